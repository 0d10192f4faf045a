// When a minor cycle's launches stop.
#pragma once
#include <climits>

namespace pg {

// The launch of the first iteration that takes no component.  One workgroup writes it during that launch, so the
// launch's other waves may read it before or after: a launch is over only when an earlier one wrote it, and every
// wave of a launch then takes the same way, whatever it reads.
struct CleanState {
  int stop;  // kCleanRuns: none yet
};
constexpr int kCleanRuns = INT_MAX;

constexpr bool clean_over(int stop, int step) { return stop < step; }
constexpr int clean_components(int stop, int max_iter) { return stop < max_iter ? stop : max_iter; }

}  // namespace pg

// Visibility binning: float64 uv snapping, w-plane choice, (plane, tile, phase)
// keys, a stable LSD radix sort and the chunked work-item list.
//
// The snapping arithmetic is written with floating-point contraction off so the
// fine-grid integers are the ones plain float64 multiply/add produces.
//
// Launch and synchronisation latency bound it at small sizes, the scattered 8-byte writes of a sort
// pass and the gather of the fine positions at large ones.  2.3M rows (25-bit keys, three passes):
// 14 launches, 280 us with the caller's allocations; with 8-bit digits on 64-bit keys and scans of
// several launches each it was 37 launches and 405 us.
#include "common.hpp"

namespace pg {
namespace {

__device__ inline int ceil_div_i(int a, int b) { return a >= 0 ? (a + b - 1) / b : -((-a) / b); }

// ---------------------------------------------------------------- stable LSD radix sort
// Digits of up to 9 bits (the fewest passes that cover the key, bits spread evenly).  A pass is three
// launches: digit counts per workgroup (the first pass's come with the keys), an exclusive scan of
// each digit's row of counts, and the scatter.  A workgroup of 16 waves takes a tile of 4096 elements,
// each wave 256 consecutive ones in four rounds of 64.  The rounds are a serial chain: with 16 (tiles
// of 16384, which write whole cache lines of a digit) 2.3M rows took 309 us and 20M 1556 us, with 8
// 315 and 1453, with 4 280 and 1443.
constexpr int kSortThreads = 1024, kSortWaves = kSortThreads / 64, kSortRounds = 4;
constexpr int kSortTile = kSortThreads * kSortRounds, kDigitBits = 9, kDigits = 1 << kDigitBits;
constexpr int64_t tiles_of(int64_t n) { return (n + kSortTile - 1) / kSortTile; }

__device__ __forceinline__ int64_t sort_index(int round) {  // element of this thread in round `round`
  return static_cast<int64_t>(blockIdx.x) * kSortTile + (threadIdx.x >> 6) * (64 * kSortRounds) + round * 64 +
         (threadIdx.x & 63);
}

template <typename KeyT>
__device__ __forceinline__ int digit_of(KeyT key, int shift, int bits) {
  return static_cast<int>(key >> shift) & ((1 << bits) - 1);
}

// Nearest plane of the ascending w_planes, the lowest index among equal distances, as a scan from plane
// 0 that keeps strictly smaller distances finds it: the rounded distances fall towards the planes
// around w and rise behind them, so it is one of those two or a lower one at the same distance.
__device__ __forceinline__ int nearest_plane(double w, const double* w_planes, int nplanes) {
#pragma clang fp contract(off)
  int lo = 0, hi = nplanes;  // planes below lo are <= w, planes from hi on are > w
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (w_planes[mid] <= w)
      lo = mid + 1;
    else
      hi = mid;
  }
  int p = lo > 0 ? lo - 1 : 0;
  double best = fabs(w - w_planes[p]);
  if (lo > 0 && lo < nplanes) {
    const double d = fabs(w - w_planes[lo]);
    if (d < best) {
      best = d;
      p = lo;
    }
  }
  while (p > 0 && fabs(w - w_planes[p - 1]) <= best) --p;
  return p;
}

template <typename KeyT>
__global__ __launch_bounds__(kSortThreads) void plan_keys_kernel(const double* __restrict__ uvw, int64_t nvis, int n,
                                                                 double ncell, double half_n, int os, int nplanes,
                                                                 const double* __restrict__ w_planes,
                                                                 const PlaneInfo* __restrict__ planes, int nt,
                                                                 KeyT drop_key, KeyT* __restrict__ keys,
                                                                 int2* __restrict__ fine_all, int digit_bits,
                                                                 int32_t* __restrict__ hist, int32_t* __restrict__ counts) {
#pragma clang fp contract(off)
  __shared__ int32_t h[kDigits];
  extern __shared__ double plane_w[];  // [nplanes] centres, then [nplanes] (support, tile)
  int2* plane_st = reinterpret_cast<int2*>(plane_w + nplanes);
  for (int p = threadIdx.x; p < nplanes; p += kSortThreads) {
    plane_w[p] = w_planes[p];
    plane_st[p] = make_int2(planes[p].support, planes[p].tile);
  }
  for (int d = threadIdx.x; d < kDigits; d += kSortThreads) h[d] = 0;
  if (blockIdx.x == 0 && threadIdx.x < 4) counts[threadIdx.x] = 0;
  __syncthreads();
  double c[kSortRounds][3];  // the rounds' coordinates are requested together
#pragma unroll
  for (int r = 0; r < kSortRounds; ++r) {
    const int64_t k = min(sort_index(r), nvis - 1);
#pragma unroll
    for (int i = 0; i < 3; ++i) c[r][i] = uvw[3 * k + i];
  }
#pragma unroll
  for (int r = 0; r < kSortRounds; ++r) {
    const int64_t k = sort_index(r);
    if (k >= nvis) continue;
    const double u = c[r][0], v = c[r][1], w = c[r][2];
    const double x = u * ncell + half_n;
    const double y = v * ncell + half_n;
    const double fxd = floor(x * static_cast<double>(os) + 0.5);
    const double fyd = floor(y * static_cast<double>(os) + 0.5);
    KeyT key = drop_key;
    int2 f = make_int2(0, 0);
    if (isfinite(fxd) && isfinite(fyd) && isfinite(w) && fabs(fxd) < 1e9 && fabs(fyd) < 1e9) {
      const int fx = static_cast<int>(fxd), fy = static_cast<int>(fyd);
      const int p = nearest_plane(w, plane_w, nplanes);
      const int2 st = plane_st[p];
      const int S = st.x, half = S * os / 2;
      const int x0 = ceil_div_i(fx - half + 1, os), y0 = ceil_div_i(fy - half + 1, os);
      const int phx = x0 * os - fx + half - 1, phy = y0 * os - fy + half - 1;
      if (x0 >= 0 && y0 >= 0 && x0 + S <= n && y0 + S <= n) {
        const KeyT ty = static_cast<KeyT>(y0 / st.y), tx = static_cast<KeyT>(x0 / st.y);
        key = (((static_cast<KeyT>(p) * nt + ty) * nt + tx) * os + static_cast<KeyT>(phy)) * os + static_cast<KeyT>(phx);
        f = make_int2(fx, fy);
      }
    }
    keys[k] = key;
    fine_all[k] = f;
    atomicAdd(&h[digit_of(key, 0, digit_bits)], 1);
  }
  __syncthreads();
  for (int d = threadIdx.x; d < (1 << digit_bits); d += kSortThreads)
    hist[static_cast<int64_t>(d) * gridDim.x + blockIdx.x] = h[d];
}

template <typename KeyT>
__global__ __launch_bounds__(kSortThreads) void radix_count(const KeyT* __restrict__ keys, int64_t n, int shift,
                                                            int digit_bits, int32_t* __restrict__ hist) {
  __shared__ int32_t h[kDigits];
  for (int d = threadIdx.x; d < kDigits; d += kSortThreads) h[d] = 0;
  __syncthreads();
#pragma unroll 4
  for (int r = 0; r < kSortRounds; ++r) {
    const int64_t k = sort_index(r);
    if (k < n) atomicAdd(&h[digit_of(keys[k], shift, digit_bits)], 1);
  }
  __syncthreads();
  for (int d = threadIdx.x; d < (1 << digit_bits); d += kSortThreads)
    hist[static_cast<int64_t>(d) * gridDim.x + blockIdx.x] = h[d];
}

// Exclusive sums over a workgroup of T threads (one value each), and their total.
template <int T>
__device__ __forceinline__ int32_t workgroup_exclusive(int32_t v, int32_t* sh, int32_t* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int32_t s = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int32_t t = __shfl_up(s, o, 64);
    if (lane >= o) s += t;
  }
  if (lane == 63) sh[wave] = s;
  __syncthreads();
  int32_t before = 0, all = 0;
#pragma unroll
  for (int w = 0; w < T / 64; ++w) {
    if (w < wave) before += sh[w];
    all += sh[w];
  }
  __syncthreads();
  *total = all;
  return before + s - v;
}

// Workgroup d: the counts of digit d over the tiles become their exclusive sums, in place; total[d].
constexpr int kRowThreads = 256;
__global__ __launch_bounds__(kRowThreads) void radix_rows(int32_t* __restrict__ hist, int64_t tiles,
                                                           int32_t* __restrict__ total) {
  __shared__ int32_t sh[kRowThreads / 64];
  int32_t* row = hist + static_cast<int64_t>(blockIdx.x) * tiles;
  int32_t carry = 0;
  for (int64_t t0 = 0; t0 < tiles; t0 += 4 * kRowThreads) {
    const int64_t t = t0 + 4 * threadIdx.x;
    int32_t v[4], sum = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      v[i] = t + i < tiles ? row[t + i] : 0;
      sum += v[i];
    }
    int32_t all;
    int32_t run = carry + workgroup_exclusive<kRowThreads>(sum, sh, &all);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (t + i < tiles) row[t + i] = run;
      run += v[i];
    }
    carry += all;
  }
  if (threadIdx.x == 0) total[blockIdx.x] = carry;
}

// The rank of an element inside its digit is the count of the lower digits, plus that of the digit in
// earlier tiles, earlier waves of this tile, and earlier rounds and lower lanes of its wave.  Each wave
// counts for itself, round after round (its LDS operations execute in program order), so the tile
// needs two barriers: 16 rounds that counted across the four waves with three barriers each took
// 27.6 us a pass at 2.3M elements.
template <typename KeyT, bool FIRST>
__global__ __launch_bounds__(kSortThreads) void radix_scatter(const KeyT* __restrict__ kin,
                                                              const int32_t* __restrict__ vin, KeyT* __restrict__ kout,
                                                              int32_t* __restrict__ vout, int64_t n, int shift,
                                                              int digit_bits, const int32_t* __restrict__ offs,
                                                              const int32_t* __restrict__ total) {
  __shared__ int32_t cnt[kSortWaves][kDigits];
  __shared__ int32_t sh[kSortWaves];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, digits = 1 << digit_bits;
  for (int d = threadIdx.x; d < kSortWaves * kDigits; d += kSortThreads) (&cnt[0][0])[d] = 0;
  KeyT key[kSortRounds];
  int32_t val[kSortRounds], rank[kSortRounds];
#pragma unroll
  for (int r = 0; r < kSortRounds; ++r) {
    const int64_t k = sort_index(r);
    key[r] = k < n ? kin[k] : KeyT(0);
    val[r] = k < n ? (FIRST ? static_cast<int32_t>(k) : vin[k]) : 0;
  }
  __syncthreads();
  volatile int32_t* mine = cnt[wave];
  const uint64_t below = (1ull << lane) - 1;
#pragma unroll
  for (int r = 0; r < kSortRounds; ++r) {
    const bool valid = sort_index(r) < n;
    const int d = digit_of(key[r], shift, digit_bits);
    uint64_t same = __ballot(valid);
    for (int b = 0; b < digit_bits; ++b) {
      const uint64_t set = __ballot((d >> b) & 1);
      same &= ((d >> b) & 1) ? set : ~set;
    }
    if (valid) {
      const int32_t old = mine[d];
      rank[r] = old + __popcll(same & below);
      __builtin_amdgcn_wave_barrier();
      if ((same & below) == 0) mine[d] = old + __popcll(same);
    }
    __builtin_amdgcn_wave_barrier();
  }
  __syncthreads();
  // digit base: lower digits, earlier tiles, then the waves in turn
  const int d = threadIdx.x;
  int32_t all;
  const int32_t base = workgroup_exclusive<kSortThreads>(d < digits ? total[d] : 0, sh, &all);
  if (d < digits) {
    int32_t at = base + offs[static_cast<int64_t>(d) * gridDim.x + blockIdx.x];
#pragma unroll
    for (int w = 0; w < kSortWaves; ++w) {
      const int32_t c = cnt[w][d];
      cnt[w][d] = at;
      at += c;
    }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kSortRounds; ++r) {
    if (sort_index(r) < n) {
      const int32_t pos = cnt[wave][digit_of(key[r], shift, digit_bits)] + rank[r];
      kout[pos] = key[r];
      vout[pos] = val[r];
    }
  }
}

// ---------------------------------------------------------------- work items
// Division by a value that is the same for the whole launch, a shift where it is a power of two.
struct Divisor {
  uint32_t by;
  int shift;  // -1: not a power of two
  explicit Divisor(uint32_t d) : by(d), shift((d & (d - 1)) == 0 ? __builtin_ctz(d) : -1) {}
  template <typename T>
  __device__ __forceinline__ T quotient(T v) const { return shift >= 0 ? v >> shift : v / by; }
  __device__ __forceinline__ bool divides(uint32_t v) const { return shift >= 0 ? (v & (by - 1)) == 0 : v % by == 0; }
};

// An item starts where a (plane, tile) run of the sorted keys starts, or a multiple of max_chunk rows
// behind that.  Tiles of the sorted keys as in the sort, kSortRounds consecutive ones per thread here; a first
// pass leaves each tile's last run start, a second counts its items (with the run start it inherits),
// a third writes them.  An item ends where the next one starts.
template <typename KeyT>
struct RunTile {
  KeyT key[kSortRounds];
  int64_t first;  // position of key[0]
  // run starts among this thread's positions; `last`: the largest (-1: none)
  __device__ __forceinline__ uint32_t load(const KeyT* __restrict__ keys, int64_t n, KeyT drop_key, Divisor os2,
                                           int64_t* last) {
    first = (static_cast<int64_t>(blockIdx.x) * kSortThreads + threadIdx.x) * kSortRounds;
#pragma unroll
    for (int i = 0; i < kSortRounds; ++i) key[i] = first + i < n ? keys[first + i] : drop_key;
    KeyT bin = first > 0 && first <= n ? os2.quotient(keys[first - 1]) : KeyT(0);
    uint32_t starts = 0;
    *last = -1;
#pragma unroll
    for (int i = 0; i < kSortRounds; ++i) {
      const KeyT b = os2.quotient(key[i]);
      if (key[i] != drop_key && (first + i == 0 || b != bin)) {
        starts |= 1u << i;
        *last = first + i;
      }
      bin = b;
    }
    return starts;
  }
};

// Largest value over the threads before this one in the workgroup (-1: none), and over all of them.
__device__ __forceinline__ int64_t workgroup_max_before(int64_t v, int64_t* sh, int64_t* all) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int64_t s = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int64_t t = __shfl_up(s, o, 64);
    if (lane >= o && t > s) s = t;
  }
  if (lane == 63) sh[wave] = s;
  int64_t m = __shfl_up(s, 1, 64);
  if (lane == 0) m = -1;
  __syncthreads();
  int64_t top = -1;
#pragma unroll
  for (int w = 0; w < kSortWaves; ++w) {
    if (w < wave && sh[w] > m) m = sh[w];
    if (sh[w] > top) top = sh[w];
  }
  __syncthreads();
  *all = top;
  return m;
}

template <typename KeyT>
__global__ __launch_bounds__(kSortThreads) void run_ends(const KeyT* __restrict__ keys, int64_t n, KeyT drop_key,
                                                         Divisor os2, int64_t* __restrict__ last_start,
                                                         int32_t* __restrict__ counts) {
  __shared__ int64_t sh[kSortWaves];
  RunTile<KeyT> t;
  int64_t last, top;
  t.load(keys, n, drop_key, os2, &last);
  workgroup_max_before(last, sh, &top);
  if (threadIdx.x == 0) last_start[blockIdx.x] = top;
#pragma unroll
  for (int i = 0; i < kSortRounds; ++i) {
    const int64_t k = t.first + i;
    if (k < n && t.key[i] != drop_key) {
      const KeyT next = i + 1 < kSortRounds ? t.key[(i + 1) % kSortRounds] : (k + 1 < n ? keys[k + 1] : drop_key);
      if (k + 1 == n || next == drop_key) counts[0] = static_cast<int32_t>(k + 1);  // rows kept
    }
  }
}

// Item starts among this thread's positions.
template <typename KeyT>
__device__ __forceinline__ uint32_t item_starts(RunTile<KeyT>& t, const KeyT* __restrict__ keys, int64_t n,
                                                KeyT drop_key, Divisor os2, Divisor max_chunk,
                                                const int64_t* __restrict__ last_start, int64_t* sh) {
  int64_t last, top;
  const uint32_t starts = t.load(keys, n, drop_key, os2, &last);
  int64_t run = workgroup_max_before(last, sh, &top);
  // the run that reaches into this tile starts in the nearest tile before it that has a start
  __shared__ int64_t inherited;
  if (threadIdx.x < 64) {
    int64_t found = -1;
    for (int64_t b = static_cast<int64_t>(blockIdx.x) - 64; found < 0 && b > -64; b -= 64) {
      int64_t v = b + threadIdx.x >= 0 ? last_start[b + threadIdx.x] : -1;
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) {
        const int64_t other = __shfl_xor(v, o, 64);
        v = other > v ? other : v;
      }
      found = v;
    }
    if (threadIdx.x == 0) inherited = found;
  }
  __syncthreads();
  if (run < 0) run = inherited;
  uint32_t items = 0;
#pragma unroll
  for (int i = 0; i < kSortRounds; ++i) {
    if (starts >> i & 1) run = t.first + i;
    if (t.key[i] != drop_key &&
        max_chunk.divides(static_cast<uint32_t>(t.first + i - run)))
      items |= 1u << i;
  }
  return items;
}

template <typename KeyT>
__global__ __launch_bounds__(kSortThreads) void item_count(const KeyT* __restrict__ keys, int64_t n, KeyT drop_key,
                                                           Divisor os2, Divisor max_chunk,
                                                           const int64_t* __restrict__ last_start,
                                                           int32_t* __restrict__ tile_items) {
  __shared__ int64_t sh[kSortWaves];
  __shared__ int32_t sum[kSortWaves];
  RunTile<KeyT> t;
  int32_t all;
  workgroup_exclusive<kSortThreads>(__popc(item_starts(t, keys, n, drop_key, os2, max_chunk, last_start, sh)), sum, &all);
  if (threadIdx.x == 0) tile_items[blockIdx.x] = all;
}

template <typename KeyT>
__global__ __launch_bounds__(kSortThreads) void item_write(const KeyT* __restrict__ keys, int64_t n, KeyT drop_key,
                                                           Divisor os2, Divisor max_chunk,
                                                           const int64_t* __restrict__ last_start,
                                                           const int32_t* __restrict__ tile_items, int nt,
                                                           const PlaneInfo* __restrict__ planes,
                                                           Item* __restrict__ items) {
  __shared__ int64_t sh[kSortWaves];
  __shared__ int32_t sum[kSortWaves];
  RunTile<KeyT> t;
  const uint32_t mask = item_starts(t, keys, n, drop_key, os2, max_chunk, last_start, sh);
  int32_t all;
  int32_t at = tile_items[blockIdx.x] + workgroup_exclusive<kSortThreads>(__popc(mask), sum, &all);
  const KeyT nt2 = static_cast<KeyT>(nt) * nt;
#pragma unroll
  for (int i = 0; i < kSortRounds; ++i) {
    if (!(mask >> i & 1)) continue;
    const KeyT bin = os2.quotient(t.key[i]), rest = bin % nt2;
    Item it;
    it.plane = static_cast<int>(bin / nt2);
    const int tile = planes[it.plane].tile;
    it.oy = static_cast<int32_t>(rest / nt) * tile;
    it.ox = static_cast<int32_t>(rest % nt) * tile;
    it.start = static_cast<int32_t>(t.first + i);
    it.end = 0;
    it.pad[0] = it.pad[1] = it.pad[2] = 0;
    items[at++] = it;
  }
}

// Fine positions in binned order, and the items' ends.
__global__ void plan_finish(const int32_t* __restrict__ perm, const int2* __restrict__ fine_all, int64_t n_kept,
                            int2* __restrict__ fine_sorted, int64_t n_items, Item* __restrict__ items) {
  const int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x;
  if (i < n_kept) fine_sorted[i] = fine_all[perm[i]];
  if (i < n_items) items[i].end = i + 1 < n_items ? items[i + 1].start : static_cast<int32_t>(n_kept);
}

template <typename T>
T* take(char*& at, int64_t count) {  // the next part of the scratch, 256-byte aligned
  T* p = reinterpret_cast<T*>(at);
  at += (static_cast<size_t>(count) * sizeof(T) + 255) / 256 * 256;
  return p;
}

struct Scratch {
  void *key[2];
  int32_t *val, *hist, *total, *tile_items, *counts;
  int64_t* last_start;
  int2* fine_all;
  size_t bytes;
};

Scratch scratch_at(char* base, int64_t nvis, int key_bytes) {
  const int64_t tiles = tiles_of(nvis);
  char* at = base;
  Scratch s;
  for (auto& k : s.key) k = take<char>(at, nvis * key_bytes);
  s.val = take<int32_t>(at, nvis);
  s.fine_all = take<int2>(at, nvis);
  s.hist = take<int32_t>(at, tiles * kDigits);
  s.total = take<int32_t>(at, kDigits);
  s.tile_items = take<int32_t>(at, tiles);
  s.last_start = take<int64_t>(at, tiles);
  s.counts = take<int32_t>(at, 4);
  s.bytes = static_cast<size_t>(at - base);
  return s;
}

int key_bytes_of(int bits) { return bits <= 32 ? 4 : 8; }
int passes_of(int bits) { return (bits + kDigitBits - 1) / kDigitBits; }

template <typename KeyT>
hipError_t run_sort(const PlanSort& a, int32_t* perm, hipStream_t s) {
  const Scratch b = scratch_at(static_cast<char*>(a.scratch), a.nvis, sizeof(KeyT));
  const dim3 tiles(static_cast<unsigned>(tiles_of(a.nvis))), threads(kSortThreads);
  const KeyT drop = static_cast<KeyT>(a.drop_key);
  const int passes = passes_of(a.bits);
  const auto digit_bits = [&](int p) { return a.bits / passes + (p < a.bits % passes ? 1 : 0); };
  KeyT* key[2] = {static_cast<KeyT*>(b.key[0]), static_cast<KeyT*>(b.key[1])};
  hipLaunchKernelGGL(plan_keys_kernel<KeyT>, tiles, threads, 16 * static_cast<size_t>(a.nplanes), s, a.uvw, a.nvis, a.n, static_cast<double>(a.n) * a.cell,
                     a.n / 2.0, a.os, a.nplanes, a.w_planes, a.planes, a.nt, drop, key[0], b.fine_all, digit_bits(0), b.hist,
                     b.counts);
  for (int p = 0, shift = 0; p < passes; ++p) {
    const int db = digit_bits(p);
    if (p > 0) hipLaunchKernelGGL(radix_count<KeyT>, tiles, threads, 0, s, key[p & 1], a.nvis, shift, db, b.hist);
    hipLaunchKernelGGL(radix_rows, dim3(1u << db), dim3(kRowThreads), 0, s, b.hist, static_cast<int64_t>(tiles.x), b.total);
    // the values alternate so that the last pass writes the permutation itself
    int32_t* out = (passes - 1 - p) % 2 == 0 ? perm : b.val;
    const int32_t* in = out == perm ? b.val : perm;
    if (p == 0)
      hipLaunchKernelGGL((radix_scatter<KeyT, true>), tiles, threads, 0, s, key[0], in, key[1], out, a.nvis, shift, db,
                         b.hist, b.total);
    else
      hipLaunchKernelGGL((radix_scatter<KeyT, false>), tiles, threads, 0, s, key[p & 1], in, key[(p + 1) & 1], out, a.nvis,
                         shift, db, b.hist, b.total);
    shift += db;
  }
  const KeyT* sorted = key[passes & 1];
  const Divisor os2(static_cast<uint32_t>(a.os) * a.os), chunk(static_cast<uint32_t>(a.max_chunk));
  hipLaunchKernelGGL(run_ends<KeyT>, tiles, threads, 0, s, sorted, a.nvis, drop, os2, b.last_start, b.counts);
  hipLaunchKernelGGL(item_count<KeyT>, tiles, threads, 0, s, sorted, a.nvis, drop, os2, chunk, b.last_start,
                     b.tile_items);
  hipLaunchKernelGGL(radix_rows, dim3(1), dim3(kRowThreads), 0, s, b.tile_items, static_cast<int64_t>(tiles.x), b.counts + 1);
  return hipGetLastError();
}

template <typename KeyT>
hipError_t run_items(const PlanSort& a, int64_t n_kept, int64_t n_items, const int32_t* perm, int2* fine, Item* items,
                     hipStream_t s) {
  const Scratch b = scratch_at(static_cast<char*>(a.scratch), a.nvis, sizeof(KeyT));
  const KeyT* sorted = static_cast<const KeyT*>(b.key[passes_of(a.bits) & 1]);
  hipLaunchKernelGGL(item_write<KeyT>, dim3(static_cast<unsigned>(tiles_of(a.nvis))),
                     dim3(kSortThreads), 0, s, sorted, a.nvis, static_cast<KeyT>(a.drop_key),
                     Divisor(static_cast<uint32_t>(a.os) * a.os), Divisor(static_cast<uint32_t>(a.max_chunk)), b.last_start, b.tile_items, a.nt, a.planes, items);
  hipLaunchKernelGGL(plan_finish, dim3(static_cast<unsigned>((n_kept + 255) / 256)), dim3(256), 0, s, perm, b.fine_all,
                     n_kept, fine, n_items, items);
  return hipGetLastError();
}

}  // namespace

size_t plan_scratch_bytes(int64_t nvis, int bits) { return scratch_at(nullptr, nvis, key_bytes_of(bits)).bytes; }

hipError_t launch_plan_sort(const PlanSort& a, int32_t* perm, const int32_t** counts, hipStream_t s) {
  *counts = scratch_at(static_cast<char*>(a.scratch), a.nvis, key_bytes_of(a.bits)).counts;
  return a.bits <= 32 ? run_sort<uint32_t>(a, perm, s) : run_sort<uint64_t>(a, perm, s);
}

hipError_t launch_plan_items(const PlanSort& a, int64_t n_kept, int64_t n_items, const int32_t* perm, int2* fine,
                             Item* items, hipStream_t s) {
  if (n_kept == 0) return hipSuccess;
  return a.bits <= 32 ? run_items<uint32_t>(a, n_kept, n_items, perm, fine, items, s)
                      : run_items<uint64_t>(a, n_kept, n_items, perm, fine, items, s);
}

}  // namespace pg

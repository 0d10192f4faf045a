// Hogbom minor cycle of Cotton-Schwab clean (Sec. 2.1), entirely on the device.
//
// The image is cut into at most kCleanTilesSide^2 tiles; the largest key of every tile (|I| over the masked
// pixels packed with the inverted pixel index into 64 bits: the largest |I| wins, ties go to the
// lowest index) is kept from one iteration to the next.  One iteration is one launch, one workgroup
// per tile, that never returns to the host:
//   peak:     every workgroup reduces the tile keys itself (they sit in the cache), so all of them
//             know the component: gain x residual[q][peak];
//   subtract: the workgroups whose tile meets the patch subtract value[q] x psf[y - py + n/2][x - px + n/2]
//             from it and find its new key; the others carry their key over.
// Keys are double-buffered (a launch reads one set and writes the other).  The component's residual
// values must be read before the launch subtracts at the peak: the owner of each tile leaves its peak
// pixel's residuals beside the key.  Below the threshold (or with no pixel) the workgroups return and
// the remaining launches of the iteration budget are empty.
// A search over the whole image, one thread to pick and a third launch to subtract took 24.4 us an
// iteration at 1536^2 x 4 with a 401^2 patch (the search alone 16 us); this takes 10.6 us, most of it
// trips past the L2 and the launch itself.  512 threads give the same; 32-pixel tiles 13.5 to 18 us
// (more records to reduce), 96- and 128-pixel tiles 16 us (too few workgroups in the patch).
// The subtraction is written without contraction (product rounded, then difference rounded) so that
// the float32 reference reproduces it bit for bit.
#include "clean_state.hpp"
#include "common.hpp"

#include <mutex>
#include <vector>

namespace pg {
namespace {

__device__ inline unsigned long long peak_key(float a, int64_t idx) {
  return (static_cast<unsigned long long>(__float_as_uint(a)) << 32) |
         static_cast<unsigned long long>(0xFFFFFFFFu - static_cast<uint32_t>(idx));
}

__global__ __launch_bounds__(256) void peak_kernel(const float* __restrict__ stokes_i, const uint8_t* __restrict__ mask,
                                                   int64_t npix, unsigned long long* __restrict__ slot) {
  unsigned long long best = 0;
  for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < npix;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x) {
    if (mask && !mask[i]) continue;
    const unsigned long long key = peak_key(fabsf(stokes_i[i]), i);
    best = key > best ? key : best;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const unsigned long long other = __shfl_xor(best, o, 64);
    best = other > best ? other : best;
  }
  __shared__ unsigned long long wbest[4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) wbest[wave] = best;
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long b = wbest[0];
    for (int w = 1; w < static_cast<int>(blockDim.x >> 6); ++w) b = wbest[w] > b ? wbest[w] : b;
    if (b) atomicMax(slot, b);
  }
}

// A tile's best pixel: its key, and its residuals of every Stokes plane.
struct __align__(32) TileBest {
  unsigned long long key;
  float value[4];
};
// One thread holds one key of the reduction, so at most 32 x 32 tiles; 64 x 64 pixels (four per
// thread, requested together) where that covers the image, larger squares of such blocks beyond 2048.
constexpr int kCleanThreads = 1024, kCleanTilesSide = 32, kCleanBlock = 64;
constexpr int kCleanRows = kCleanBlock / (kCleanThreads / kCleanBlock);  // rows of a block per thread
constexpr size_t kCleanScratchBytes = 256 + 2 * sizeof(TileBest) * kCleanTilesSide * kCleanTilesSide;

struct TileGrid {
  int n, side, across;  // image side, tile side (a multiple of kCleanBlock), tiles per row
};

TileGrid tile_grid(int n) {
  const int blocks = (n + kCleanBlock - 1) / kCleanBlock;
  const int side = (blocks + kCleanTilesSide - 1) / kCleanTilesSide * kCleanBlock;
  return TileGrid{n, side, (n + side - 1) / side};
}

// Largest key over the workgroup, in every thread.
__device__ inline unsigned long long workgroup_best(unsigned long long best, unsigned long long* wbest) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const unsigned long long other = __shfl_xor(best, o, 64);
    best = other > best ? other : best;
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) wbest[wave] = best;
  __syncthreads();
  best = wbest[lane & (kCleanThreads / 64 - 1)];
#pragma unroll
  for (int o = kCleanThreads / 128; o > 0; o >>= 1) {
    const unsigned long long other = __shfl_xor(best, o, 64);
    best = other > best ? other : best;
  }
  return best;
}

// The pixels of this workgroup's tile: subtract value[q] x psf inside rows [y0, y1), columns [x0, x1)
// (the shifted psf inside both images and the patch; empty: nothing is subtracted), then record the
// tile's best pixel.
template <int NPOL>
__device__ __forceinline__ void clean_tile(float* __restrict__ residual, const float* __restrict__ psf,
                                           const uint8_t* __restrict__ mask, const TileGrid& g, int py, int px, int y0,
                                           int y1, int x0, int x1, const float (&value)[NPOL], TileBest* out,
                                           unsigned long long* wbest) {
#pragma clang fp contract(off)
  const int64_t npix = static_cast<int64_t>(g.n) * g.n;
  const int ty = static_cast<int>(blockIdx.x) / g.across * g.side, tx = static_cast<int>(blockIdx.x) % g.across * g.side;
  unsigned long long best = 0;
  for (int by = ty; by < min(ty + g.side, g.n); by += kCleanBlock)
    for (int bx = tx; bx < min(tx + g.side, g.n); bx += kCleanBlock) {
      const int x = bx + static_cast<int>(threadIdx.x % kCleanBlock);
      const int yb = by + static_cast<int>(threadIdx.x / kCleanBlock);
      float r[kCleanRows][NPOL], p[kCleanRows];
      bool in[kCleanRows], sub[kCleanRows], on[kCleanRows];
#pragma unroll
      for (int k = 0; k < kCleanRows; ++k) {  // every load of the block's pixels before the first store
        const int y = yb + k * (kCleanBlock / kCleanRows);
        in[k] = x < g.n && y < g.n;
        sub[k] = in[k] && y >= y0 && y < y1 && x >= x0 && x < x1;
        const int64_t at = in[k] ? static_cast<int64_t>(y) * g.n + x : 0;
        on[k] = in[k] && (!mask || mask[at]);
        p[k] = sub[k] ? psf[static_cast<int64_t>(y - py + g.n / 2) * g.n + (x - px + g.n / 2)] : 0.0f;
#pragma unroll
        for (int q = 0; q < NPOL; ++q) r[k][q] = (sub[k] || (q == 0 && on[k])) ? residual[q * npix + at] : 0.0f;
      }
#pragma unroll
      for (int k = 0; k < kCleanRows; ++k) {
        const int y = yb + k * (kCleanBlock / kCleanRows);
        const int64_t at = static_cast<int64_t>(y) * g.n + x;
        if (sub[k]) {
#pragma unroll
          for (int q = 0; q < NPOL; ++q) {
            const float prod = value[q] * p[k];
            r[k][q] = r[k][q] - prod;
            residual[q * npix + at] = r[k][q];
          }
        }
        if (on[k]) {
          const unsigned long long key = peak_key(fabsf(r[k][0]), at);
          best = key > best ? key : best;
        }
      }
    }
  const unsigned long long all = workgroup_best(best, wbest);
  if (all == 0) {
    if (threadIdx.x == 0) out[blockIdx.x].key = 0;
  } else if (best == all) {  // keys hold the pixel index: one thread, which wrote that pixel if anyone did
    const int64_t at = static_cast<int64_t>(0xFFFFFFFFu - static_cast<uint32_t>(all & 0xFFFFFFFFu));
    TileBest t;
    t.key = all;
#pragma unroll
    for (int q = 0; q < NPOL; ++q) t.value[q] = residual[q * npix + at];
    out[blockIdx.x] = t;
  }
}

template <int NPOL>
__global__ __launch_bounds__(kCleanThreads) void clean_start_kernel(float* __restrict__ residual,
                                                                    const uint8_t* __restrict__ mask, TileGrid g,
                                                                    CleanState* __restrict__ st,
                                                                    TileBest* __restrict__ out) {
  __shared__ unsigned long long wbest[kCleanThreads / 64];
  if (blockIdx.x == 0 && threadIdx.x == 0) st->stop = kCleanRuns;
  const float none[NPOL] = {};
  clean_tile<NPOL>(residual, residual, mask, g, 0, 0, 0, 0, 0, 0, none, out, wbest);
}

template <int NPOL>
__global__ __launch_bounds__(kCleanThreads) void clean_step_kernel(float* __restrict__ residual,
                                                                   const float* __restrict__ psf,
                                                                   const uint8_t* __restrict__ mask, TileGrid g,
                                                                   int patch, float gain, float threshold, int step,
                                                                   CleanState* __restrict__ st,
                                                                   const TileBest* __restrict__ in,
                                                                   TileBest* __restrict__ out,
                                                                   int32_t* __restrict__ comp_pos,
                                                                   float* __restrict__ comp_val,
                                                                   float* __restrict__ model) {
  __shared__ unsigned long long wbest[kCleanThreads / 64];
  __shared__ float shared_value[NPOL];
  // thread t fetches tile t's whole record and the cycle's state at once: each is a trip past the L2
  // (another XCD wrote them), and the trips of an iteration are most of its time
  const int tiles = g.across * g.across;
  TileBest mine;
  mine.key = 0;
#pragma unroll
  for (int k = 0; k < (kCleanTilesSide * kCleanTilesSide + kCleanThreads - 1) / kCleanThreads; ++k) {
    const int t = static_cast<int>(threadIdx.x) + k * kCleanThreads;
    if (t >= tiles) break;
    const TileBest other = in[t];
    if (other.key > mine.key) mine = other;
  }
  if (clean_over(st->stop, step)) return;
  const unsigned long long key = workgroup_best(mine.key, wbest);
  const float a = __uint_as_float(static_cast<uint32_t>(key >> 32));
  if (key == 0 || !(a >= threshold)) {  // the same verdict in every workgroup
    if (blockIdx.x == 0 && threadIdx.x == 0) st->stop = step;
    return;
  }
  if (mine.key == key) {
#pragma unroll
    for (int q = 0; q < NPOL; ++q) shared_value[q] = gain * mine.value[q];
  }
  __syncthreads();
  const int idx = static_cast<int>(0xFFFFFFFFu - static_cast<uint32_t>(key & 0xFFFFFFFFu));
  const int py = idx / g.n, px = idx - py * g.n;
  const int home = py / g.side * g.across + px / g.side;
  float value[NPOL];
#pragma unroll
  for (int q = 0; q < NPOL; ++q) value[q] = shared_value[q];
  if (static_cast<int>(blockIdx.x) == home && threadIdx.x < NPOL) {
    const int64_t npix = static_cast<int64_t>(g.n) * g.n;
    const int q = threadIdx.x;
    const float v = shared_value[q];
    comp_val[static_cast<int64_t>(step) * NPOL + q] = v;
    if (model) model[q * npix + idx] += v;
    if (q == 0) comp_pos[step] = idx;
  }
  // rows and columns where the shifted psf (centre n/2) is inside both images and the patch
  const int y0 = max(max(0, py - g.n / 2), py - patch), y1 = min(min(g.n, py + g.n / 2), py + patch + 1);
  const int x0 = max(max(0, px - g.n / 2), px - patch), x1 = min(min(g.n, px + g.n / 2), px + patch + 1);
  const int ty = static_cast<int>(blockIdx.x) / g.across * g.side, tx = static_cast<int>(blockIdx.x) % g.across * g.side;
  if (ty >= y1 || ty + g.side <= y0 || tx >= x1 || tx + g.side <= x0) {  // untouched: the record carries over
    if (threadIdx.x == 0) out[blockIdx.x] = in[blockIdx.x];
    return;
  }
  clean_tile<NPOL>(residual, psf, mask, g, py, px, y0, y1, x0, x1, value, out, wbest);
}

__global__ void peak_init_kernel(unsigned long long* slot) { *slot = 0; }

__global__ void clean_count_kernel(const CleanState* st, int max_iter, int32_t* n_comp) {
  *n_comp = clean_components(st->stop, max_iter);
}

// img[i] / ref for every pixel, ref = img[ref_index] read first into `held` (one thread), so the
// division never sees a pixel already divided.
__global__ void hold_value_kernel(const float* __restrict__ img, int64_t ref_index, float* __restrict__ held) {
  if (threadIdx.x == 0 && blockIdx.x == 0) *held = img[ref_index];
}

__global__ void divide_by_held_kernel(float* __restrict__ img, int64_t count, const float* __restrict__ held) {
  const float r = *held;
  for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < count;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x)
    img[i] = img[i] / r;
}

// Scratch of the allocation-free entry point: the iteration state and two sets of tile records.  Each
// GPU holds its own copy; host code reaches it only through the address hipGetSymbolAddress returns on
// that device.
__device__ __align__(256) unsigned char scratch[kCleanScratchBytes];

std::mutex g_static_mu;
std::vector<void*> g_static_ptr;  // per device, looked up once with that device current

}  // namespace

hipError_t hogbom_static_scratch(void** out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  std::lock_guard<std::mutex> lk(g_static_mu);
  if (static_cast<size_t>(dev) >= g_static_ptr.size()) g_static_ptr.resize(dev + 1, nullptr);
  if (!g_static_ptr[dev]) {
    void* ptr = nullptr;
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    g_static_ptr[dev] = ptr;
  }
  *out = g_static_ptr[dev];
  return hipSuccess;
}

hipError_t launch_masked_peak(const float* img, const uint8_t* mask, int64_t npix, void* scratch, hipStream_t s) {
  auto* slot = reinterpret_cast<unsigned long long*>(static_cast<char*>(scratch) + 256);
  hipLaunchKernelGGL(peak_init_kernel, dim3(1), dim3(1), 0, s, slot);
  const int blocks = static_cast<int>(std::min<int64_t>((npix + 255) / 256, 1024));
  hipLaunchKernelGGL(peak_kernel, dim3(blocks), dim3(256), 0, s, img, mask, npix, slot);
  return hipGetLastError();
}

hipError_t launch_normalise_at(float* img, int64_t count, int64_t ref_index, float* held, hipStream_t s) {
  hipLaunchKernelGGL(hold_value_kernel, dim3(1), dim3(64), 0, s, img, ref_index, held);
  const unsigned blocks = static_cast<unsigned>(std::min<int64_t>((count + 255) / 256, 4096));
  hipLaunchKernelGGL(divide_by_held_kernel, dim3(blocks), dim3(256), 0, s, img, count, held);
  return hipGetLastError();
}

size_t hogbom_scratch_bytes() { return kCleanScratchBytes; }

namespace {
template <int NPOL>
hipError_t run_hogbom(float* residual, const float* psf, const uint8_t* mask, int n, float gain, float threshold,
                      int patch, int max_iter, int32_t* comp_pos, float* comp_val, float* model, int32_t* n_comp,
                      void* scratch, hipStream_t s) {
  auto* st = static_cast<CleanState*>(scratch);
  TileBest* best[2] = {reinterpret_cast<TileBest*>(static_cast<char*>(scratch) + 256), nullptr};
  best[1] = best[0] + kCleanTilesSide * kCleanTilesSide;
  const TileGrid g = tile_grid(n);
  const dim3 tiles(static_cast<unsigned>(g.across * g.across));
  hipLaunchKernelGGL(clean_start_kernel<NPOL>, tiles, dim3(kCleanThreads), 0, s, residual, mask, g, st, best[0]);
  hipError_t e = hipGetLastError();
  for (int it = 0; it < max_iter && e == hipSuccess; ++it) {
    hipLaunchKernelGGL(clean_step_kernel<NPOL>, tiles, dim3(kCleanThreads), 0, s, residual, psf, mask, g, patch, gain,
                       threshold, it, st, best[it & 1], best[(it + 1) & 1], comp_pos, comp_val, model);
    e = hipGetLastError();
  }
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(clean_count_kernel, dim3(1), dim3(1), 0, s, st, max_iter, n_comp);
  return hipGetLastError();
}
}  // namespace

hipError_t launch_hogbom(float* residual, const float* psf, const uint8_t* mask, int n, int npol, float gain,
                         float threshold, int patch, int max_iter, int32_t* comp_pos, float* comp_val, float* model,
                         int32_t* n_comp, void* scratch, hipStream_t s) {
  auto run = npol == 1 ? run_hogbom<1> : npol == 2 ? run_hogbom<2> : npol == 3 ? run_hogbom<3> : run_hogbom<4>;
  return run(residual, psf, mask, n, gain, threshold, patch, max_iter, comp_pos, comp_val, model, n_comp, scratch, s);
}

}  // namespace pg

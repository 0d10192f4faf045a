// Image-plane reprojection for image-domain mosaics (Sec. 2.2): field images made at their own
// phase centres are resampled onto a common mosaic frame, and the model image is resampled back
// onto each field before its FFT and degridding.
//
// A frame is an n x n orthographic (SIN) projection about (ra0, dec0) with pixel (row i, column j)
// at direction cosines l = (j - n/2) cell, m = (i - n/2) cell: the components of the unit
// direction vector along the frame's east, north and centre axes.  Going from one frame to the
// other is therefore a fixed rotation of (l, m, n): R[a][b] = (axis a of the source frame) .
// (axis b of the destination frame), computed once on the host in float64.  Per destination pixel:
// (l0, m0, sqrt(1 - l0^2 - m0^2)) -> R -> source (l, m, n) -> source pixel
// (x, y) -> bilinear sample of every Stokes plane and of the optional weight image.  Coordinates
// and bilinear weights are float64 (at 8192^2 the offsets need more than float32's 24 bits); the
// output is float32.  Bound: HBM, npol x (4 B read + 4 or 8 B written or read-modify-written) per
// destination pixel, plus the weight image, once the index arithmetic is out of the way.
#include <algorithm>
#include <cmath>

#include "mosaic.hpp"
#include "weight_normalise.hpp"

namespace pg {
namespace {

constexpr double kEdge = 1e-6;  // pixels: border tolerance of the covered test

struct Axes {
  double e[3], nth[3], c[3];  // east, north, centre unit vectors of a frame
};

Axes axes_of(const pg_sky_frame& f) {
  const double sa = std::sin(f.ra), ca = std::cos(f.ra), sd = std::sin(f.dec), cd = std::cos(f.dec);
  return Axes{{-sa, ca, 0.0}, {-sd * ca, -sd * sa, cd}, {cd * ca, cd * sa, sd}};
}

struct Rotation {
  double r[3][3];  // source (l, m, n) = r . destination (l, m, n)
};

Rotation rotation(const pg_sky_frame& src, const pg_sky_frame& dst) {
  const Axes s = axes_of(src), d = axes_of(dst);
  const double* sa[3] = {s.e, s.nth, s.c};
  const double* da[3] = {d.e, d.nth, d.c};
  Rotation r;
  for (int a = 0; a < 3; ++a)
    for (int b = 0; b < 3; ++b) r.r[a][b] = sa[a][0] * da[b][0] + sa[a][1] * da[b][1] + sa[a][2] * da[b][2];
  return r;
}

struct FrameD {
  int n;
  double cell, inv_cell;  // inv_cell: 1 / cell, rounded; 0 where that or the quotient's remainder may leave the normal range
};

// x / cell from the rounded reciprocal and one Newton step on the quotient (Markstein 1990), in three
// instructions; a division by an unknown takes a dozen.  The starting quotient may be further off than the
// theorem's unit in the last place, so the rounding is not proven correct; the division gave the same value for
// 2e8 random x in (-1, 1) and cells of 1e-6 to 1e-2, and a last place is 1e-16 of a pixel.
__device__ inline double over_cell(double x, FrameD f) {
  if (f.inv_cell == 0.0) return x / f.cell;
  const double q = x * f.inv_cell;
  return fma(fma(-q, f.cell, x), f.inv_cell, q);
}

// Two neighbouring samples in one load.
__device__ inline float2 pair_at(const float* p) {
  float2 v;
  __builtin_memcpy(&v, p, 8);
  return v;
}

// A workgroup takes 64 x 16 destination pixels, one column a lane and four rows a wave: the rotation is close to a
// shift, so the source rows of one tile overlap and are read into one L2.  Where nothing is added (outside
// the field, or where its weight and weighted sample are zero) an accumulated pixel is neither read nor
// written: a beam's weights are zero over most of a field image's square.
// 3000^2 onto 3750^2 accumulated with a beam's weights, and back, four planes: 94 and 79 us (164 us each
// with a linear index divided by n, a whole-image read-modify-write and scalar loads).
constexpr int kTileX = 64, kTileRows = 4, kTileY = 4 * kTileRows;

template <int NPOL>
__global__ __launch_bounds__(256) void reproject_kernel(const float* __restrict__ src,
                                                        const float* __restrict__ src_w, FrameD sf,
                                                        float* __restrict__ dst, float* __restrict__ dst_w,
                                                        FrameD df, Rotation rot, int accumulate) {
  const int64_t npix_d = static_cast<int64_t>(df.n) * df.n;
  const int64_t npix_s = static_cast<int64_t>(sf.n) * sf.n;
  const int j = blockIdx.x * kTileX + (threadIdx.x & 63);
  const int i0 = blockIdx.y * kTileY + (threadIdx.x >> 6) * kTileRows;
  if (j >= df.n) return;
  const double l0 = (j - df.n / 2) * df.cell;
#pragma unroll
  for (int row = 0; row < kTileRows; ++row) {
    const int i = i0 + row;
    if (i >= df.n) return;
    const int64_t p = static_cast<int64_t>(i) * df.n + j;
    const double m0 = (i - df.n / 2) * df.cell;
    const double r2 = l0 * l0 + m0 * m0;
    double val[NPOL] = {};
    double w = 0.0;
    if (r2 < 1.0) {
      const double n0 = sqrt(1.0 - r2);
      const double l = rot.r[0][0] * l0 + rot.r[0][1] * m0 + rot.r[0][2] * n0;
      const double m = rot.r[1][0] * l0 + rot.r[1][1] * m0 + rot.r[1][2] * n0;
      const double nn = rot.r[2][0] * l0 + rot.r[2][1] * m0 + rot.r[2][2] * n0;
      const double x = over_cell(l, sf) + sf.n / 2, y = over_cell(m, sf) + sf.n / 2;
      const double hi = sf.n - 1;
      if (nn > 0.0 && x >= -kEdge && y >= -kEdge && x <= hi + kEdge && y <= hi + kEdge) {
        const double xc = fmin(fmax(x, 0.0), hi), yc = fmin(fmax(y, 0.0), hi);
        const int x0 = min(static_cast<int>(floor(xc)), sf.n - 2), y0 = min(static_cast<int>(floor(yc)), sf.n - 2);
        const double fx = xc - x0, fy = yc - y0;
        const double w00 = (1.0 - fy) * (1.0 - fx), w01 = (1.0 - fy) * fx, w10 = fy * (1.0 - fx), w11 = fy * fx;
        const int64_t b = static_cast<int64_t>(y0) * sf.n + x0;
        float2 s0[NPOL], s1[NPOL], v0 = make_float2(0.0f, 0.0f), v1 = v0;
#pragma unroll
        for (int q = 0; q < NPOL; ++q) {
          s0[q] = pair_at(src + q * npix_s + b);
          s1[q] = pair_at(src + q * npix_s + b + sf.n);
        }
        if (src_w) {
          v0 = pair_at(src_w + b);
          v1 = pair_at(src_w + b + sf.n);
        }
#pragma unroll
        for (int q = 0; q < NPOL; ++q) val[q] = w00 * s0[q].x + w01 * s0[q].y + w10 * s1[q].x + w11 * s1[q].y;
        w = src_w ? w00 * v0.x + w01 * v0.y + w10 * v1.x + w11 * v1.y : 1.0;
      }
    }
    if (accumulate) {
      float add[NPOL];
      bool any = w != 0.0;
#pragma unroll
      for (int q = 0; q < NPOL; ++q) {
        add[q] = static_cast<float>(w * val[q]);
        any = any || add[q] != 0.0f;  // a NaN sample spreads under a zero weight too
      }
      if (!any) continue;
#pragma unroll
      for (int q = 0; q < NPOL; ++q) dst[q * npix_d + p] += add[q];
      if (dst_w) dst_w[p] += static_cast<float>(w);
    } else {
#pragma unroll
      for (int q = 0; q < NPOL; ++q) dst[q * npix_d + p] = static_cast<float>(val[q]);
      if (dst_w) dst_w[p] = static_cast<float>(w);
    }
  }
}

// HBM-bound.  V consecutive pixels a thread; a group without a pixel above the weight is not read.
// Four planes of 3750^2: 79 us (118 us with one pixel a thread, all read).
template <typename V>
__global__ __launch_bounds__(256) void weight_normalise_kernel(V* __restrict__ img, const V* __restrict__ weight,
                                                               int64_t count, int npol, float min_weight) {
  for (int64_t p = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; p < count;
       p += static_cast<int64_t>(gridDim.x) * blockDim.x) {
    const Pixels<V> w(weight[p]);
    const bool any = any_reaches(w, min_weight);
    for (int q = 0; q < npol; ++q) {
      Pixels<V> v;
      if (any) v = Pixels<V>(img[q * count + p]);
      img[q * count + p] = over_weight(v, w, min_weight);
    }
  }
}

// Phase rotation: one thread per visibility row.  uvw about the new centre = q . uvw (q[a][b] =
// axis a of the new frame . axis b of the old), and every correlation is multiplied by
// exp(2 pi i (w_old - w_new)); float64 phase, float32 products.  In place is allowed (each
// thread reads its row before writing it).  HBM-bound: 24 + 8 npol bytes in and out per row.
__global__ __launch_bounds__(256) void phase_rotate_kernel(const double* uvw_in, const float2* vis_in, int64_t nvis,
                                                           int npol, Rotation q, double* uvw_out, float2* vis_out) {
  for (int64_t k = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; k < nvis;
       k += static_cast<int64_t>(gridDim.x) * blockDim.x) {
    const double u = uvw_in[3 * k], v = uvw_in[3 * k + 1], w = uvw_in[3 * k + 2];
    const double u2 = q.r[0][0] * u + q.r[0][1] * v + q.r[0][2] * w;
    const double v2 = q.r[1][0] * u + q.r[1][1] * v + q.r[1][2] * w;
    const double w2 = q.r[2][0] * u + q.r[2][1] * v + q.r[2][2] * w;
    double s, c;
    sincospi(2.0 * (w - w2), &s, &c);
    const float cs = static_cast<float>(c), sn = static_cast<float>(s);
    for (int p = 0; p < npol; ++p) {
      const float2 a = vis_in[k * npol + p];
      vis_out[k * npol + p] = make_float2(a.x * cs - a.y * sn, a.x * sn + a.y * cs);
    }
    if (uvw_out) {
      uvw_out[3 * k] = u2;
      uvw_out[3 * k + 1] = v2;
      uvw_out[3 * k + 2] = w2;
    }
  }
}

unsigned blocks_for(int64_t n) { return static_cast<unsigned>(std::min<int64_t>((n + 255) / 256, 65536)); }

// UV-domain mosaic correction (Sec. 2.2, Eq. 1).  Pass 1: S = sum_i B_i^2 per pixel (written out as
// the mosaic weight map) and its maximum (float bits of a non-negative value order like unsigned
// integers, so one atomicMax per workgroup).  Pass 2: img *= scale sqrt(S / S_max) / S where S
// clears floor * S_max, else 0.  HBM-bound: (nfields + 1) x 4 B, then (npol x 8 + 4) B per pixel.
__global__ __launch_bounds__(256) void beam_sumsq_kernel(const float* __restrict__ beams, int nfields, int64_t npix,
                                                         float* __restrict__ sumsq, unsigned* __restrict__ max_bits) {
  float best = 0.0f;
  for (int64_t p = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; p < npix;
       p += static_cast<int64_t>(gridDim.x) * blockDim.x) {
    float s = 0.0f;
    for (int f = 0; f < nfields; ++f) {
      const float b = beams[f * npix + p];
      s = fmaf(b, b, s);
    }
    sumsq[p] = s;
    best = fmaxf(best, s);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) best = fmaxf(best, __shfl_xor(best, o, 64));
  __shared__ float wb[4];
  if ((threadIdx.x & 63) == 0) wb[threadIdx.x >> 6] = best;
  __syncthreads();
  if (threadIdx.x == 0) {
    const float b = fmaxf(fmaxf(wb[0], wb[1]), fmaxf(wb[2], wb[3]));
    atomicMax(max_bits, __float_as_uint(b));
  }
}

__global__ __launch_bounds__(256) void mosaic_gamma_kernel(const float* __restrict__ sumsq,
                                                           const unsigned* __restrict__ max_bits, float floor_frac,
                                                           float scale, int npol, int64_t npix, float* __restrict__ img) {
  const float smax = __uint_as_float(*max_bits);
  const float inv_root_max = smax > 0.0f ? 1.0f / sqrtf(smax) : 0.0f;
  for (int64_t p = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; p < npix;
       p += static_cast<int64_t>(gridDim.x) * blockDim.x) {
    const float s = sumsq[p];
    const float g = (s > 0.0f && s >= floor_frac * smax) ? scale * (sqrtf(s) * inv_root_max) / s : 0.0f;
    for (int q = 0; q < npol; ++q) img[q * npix + p] *= g;
  }
}

__global__ void zero_u32_kernel(unsigned* p) { *p = 0u; }

}  // namespace

hipError_t launch_reproject(const float* src, const float* src_w, const pg_sky_frame& sf, float* dst, float* dst_w,
                            const pg_sky_frame& df, int npol, int accumulate, hipStream_t s) {
  const dim3 grid((df.n + kTileX - 1) / kTileX, (df.n + kTileY - 1) / kTileY);
  const FrameD from{sf.n, sf.cell, sf.cell > 1e-100 && sf.cell < 1e100 ? 1.0 / sf.cell : 0.0}, to{df.n, df.cell, 0.0};
  const auto kernel = npol == 1   ? reproject_kernel<1>
                      : npol == 2 ? reproject_kernel<2>
                      : npol == 3 ? reproject_kernel<3>
                                  : reproject_kernel<4>;
  hipLaunchKernelGGL(kernel, grid, dim3(256), 0, s, src, src_w, from, dst, dst_w, to, rotation(sf, df), accumulate);
  return hipGetLastError();
}

hipError_t launch_weight_normalise(float* img, const float* weight, int n, int npol, float min_weight, hipStream_t s) {
  const int64_t npix = static_cast<int64_t>(n) * n;
  // Four pixels a thread where every plane starts on 16 bytes.
  const bool wide = npix % 4 == 0 && (reinterpret_cast<uintptr_t>(img) | reinterpret_cast<uintptr_t>(weight)) % 16 == 0;
  if (wide)
    hipLaunchKernelGGL(weight_normalise_kernel<float4>, dim3(blocks_for(npix / 4)), dim3(256), 0, s,
                       reinterpret_cast<float4*>(img), reinterpret_cast<const float4*>(weight), npix / 4, npol, min_weight);
  else
    hipLaunchKernelGGL(weight_normalise_kernel<float>, dim3(blocks_for(npix)), dim3(256), 0, s, img, weight, npix, npol,
                       min_weight);
  return hipGetLastError();
}

hipError_t launch_phase_rotate(const double* uvw_in, const void* vis_in, int64_t nvis, int npol, double ra_from,
                               double dec_from, double ra_to, double dec_to, double* uvw_out, void* vis_out,
                               hipStream_t s) {
  const pg_sky_frame from{2, 1.0, ra_from, dec_from}, to{2, 1.0, ra_to, dec_to};
  hipLaunchKernelGGL(phase_rotate_kernel, dim3(blocks_for(nvis)), dim3(256), 0, s, uvw_in,
                     static_cast<const float2*>(vis_in), nvis, npol, rotation(to, from), uvw_out,
                     static_cast<float2*>(vis_out));
  return hipGetLastError();
}

hipError_t launch_mosaic_gamma(const float* beams, int nfields, int n, double floor_frac, double scale,
                               float* weight_sum, float* img, int npol, unsigned* max_bits, hipStream_t s) {
  const int64_t npix = static_cast<int64_t>(n) * n;
  const unsigned blocks = static_cast<unsigned>(std::min<int64_t>((npix + 255) / 256, 8192));
  hipLaunchKernelGGL(zero_u32_kernel, dim3(1), dim3(1), 0, s, max_bits);
  hipLaunchKernelGGL(beam_sumsq_kernel, dim3(blocks), dim3(256), 0, s, beams, nfields, npix, weight_sum, max_bits);
  hipLaunchKernelGGL(mosaic_gamma_kernel, dim3(blocks), dim3(256), 0, s, weight_sum, max_bits,
                     static_cast<float>(floor_frac), static_cast<float>(scale), npol, npix, img);
  return hipGetLastError();
}

}  // namespace pg

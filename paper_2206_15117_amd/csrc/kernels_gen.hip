// Device side of kernel generation (Sec. 3.2): image-domain screens
// AA(l) AA(m) exp(-2 pi i w (n-1)) Phi_qc(l, m), their separable zero-padded DFT
// into the oversampled uv domain (two complex float64 matrix products per
// Mueller cell), and packing into the [phase_y][phase_x][tap_y][tap_x][q][c]
// table the gridder reads.
#include "common.hpp"
#include "mlp.hpp"
#include "mueller.hpp"

namespace pg {
namespace {

__device__ inline double2 cmul(double2 a, double2 b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}

// phi[qc][px]: the screens at one lattice sample a thread.  The 4 x 4 solve is a chain of four pivots with
// a double-precision division each; the samples are independent and the whole lattice of 256^2 takes
// less than its 4 MB of Jones matrices takes to arrive.
__global__ __launch_bounds__(64) void screens_kernel(int kind, const double* __restrict__ jones,
                                                     const double* __restrict__ jones_b, size_t npix, double4 beta4,
                                                     int convention, double2* __restrict__ phi) {
  const size_t px = blockIdx.x * static_cast<size_t>(64) + threadIdx.x;
  if (px >= npix) return;
  const cd u = stokes_u(convention);
  M4 m = mueller_at(jones, jones_b, npix, px, u);
  M4 f;
  if (kind == PG_KIND_GRID) {
    const double beta[4] = {beta4.x, beta4.y, beta4.z, beta4.w};
    regularise(m, beta);
    f = stokes(convention);
    solve(m, f);
  } else {  // (S^-1 M^S)^H
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      cd col[4], y[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) col[r] = m.a[r][c];
      stokes_inverse_times(u, col, y);
#pragma unroll
      for (int r = 0; r < 4; ++r) f.a[c][r] = conj(y[r]);
    }
  }
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int c = 0; c < 4; ++c) phi[(q * 4 + c) * npix + px] = make_double2(f.a[q][c].re, f.a[q][c].im);
}

// The screens of a few samples, solved on the host; 16 threads a sample.
__global__ void place_screens_kernel(const uint32_t* __restrict__ px, const double2* __restrict__ at, size_t count,
                                     size_t npix, double2* __restrict__ phi) {
  const size_t i = blockIdx.x * static_cast<size_t>(blockDim.x) + threadIdx.x;
  if (i < 16 * count) phi[(i % 16) * npix + px[i / 16]] = at[i];
}

__global__ void unit_screen_kernel(size_t npix, double2* __restrict__ phi) {
  const size_t px = blockIdx.x * static_cast<size_t>(blockDim.x) + threadIdx.x;
  if (px < npix) phi[px] = make_double2(1.0, 0.0);
}

// wterm[plane][b][a] = AA(l) AA(m) exp(-2 pi i w (n-1)), common to the plane's Mueller cells.
__global__ void wterm_kernel(GenRound r) {
  const int a = blockIdx.x * blockDim.x + threadIdx.x;
  const int b = blockIdx.y;
  if (a >= r.mk) return;
  const double step = r.fov / r.mk;
  const double l = (a - r.mk / 2) * step, m = (b - r.mk / 2) * step;
  const double r2 = l * l + m * m;
  const double nm1 = -r2 / (1.0 + sqrt(1.0 - r2));
  double s, c;
  sincospi(2.0 * r.w[blockIdx.z] * nm1, &s, &c);
  const double g = r.aa[a] * r.aa[b];
  r.wterm[(static_cast<size_t>(blockIdx.z) * r.mk + b) * r.mk + a] = make_double2(g * c, -g * s);
}

// twiddle[plane][d][k] = (cos, sin)(2 pi d k / (os mk)) / mk for d = 0 .. S os/2 - 1, k = 0 .. mk/2.
__global__ void twiddle_kernel(GenRound r) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x, d = blockIdx.y, mk = r.mk;
  if (k > mk / 2 || d >= r.support[blockIdx.z] * r.os / 2) return;
  const long long period = 2LL * r.os * mk;  // exp(i pi x) has period 2 in x = num / (os mk)
  const long long num = (2LL * d * k) % period;
  double s, c;
  sincospi(static_cast<double>(num) / (static_cast<double>(r.os) * mk), &s, &c);
  r.twiddle[(static_cast<size_t>(blockIdx.z) * (r.support_max * r.os / 2) + d) * (mk / 2 + 1) + k] =
      make_double2(c / mk, s / mk);
}

// The separable zero-padded DFT as two float64 matrix products per plane and Mueller cell, contracted
// over the lattice with e(d, a) = exp(+2 pi i d (a - mk/2) / (os mk)) / mk, d = di - (S os/2 - 1):
//   stage 1  half[b][dx] = sum_a (wterm[b][a] phi[qc][b][a]) e(dx, a)
//   stage 2  T[dy][dx]   = sum_b half[b][dx] e(dy, b), written to the table
//     [phase_y][phase_x][chunk][tap_y][tap_x][e] (cell qc = chunk E + e; one 16-byte chunk of 64
//     consecutive taps is 1 KiB of contiguous memory) at phase d mod os, tap d / os.
// The last row and column (d = S os / 2, outside the open footprint) are zero.
// Both are out[row][+-d] = C(row, d) +- i S(row, d) with C = sum_k even(row, k) cos(d, k),
// S = sum_k odd(row, k) sin(d, k) over k = 0 .. mk/2, even and odd the sum and difference of the samples
// k to either side of the lattice's middle: folding the samples and the outputs leaves a quarter of the
// complex product's operations.
// Bound: what is left of the float64 rate (16 FMA a clock and SIMD for vector and matrix instructions
// alike) after the loads.  A vector FMA per lane needs its LDS operands per lane, twice the LDS's
// bandwidth at 2 x 2 outputs a thread; v_mfma_f64_16x16x4 shares each among 16 lanes.  A workgroup takes 32 rows by 64
// values of d, because the folded samples (two, in stage 1 with the w-term's two) cost four times the
// bytes of the twiddles.  The next slice of the contraction is fetched into registers while one is used.
// Screened cells and the dense transform are never stored: stage 1 multiplies the screen where it
// stores it to LDS, stage 2 rounds into the table.
// 24 planes of 16 cells, mk = 256, 1.4 ms, 88 us a
// stage and round of three planes (75 us a stage and plane with vector FMAs on 32 x 32 tiles, unfolded, and 23 us
// more for storing the screened cells and packing the transform).
constexpr int kGenRows = 32, kGenCols = 64, kGenK = 16, kGenPitch = kGenK + 1;
typedef double double4_t __attribute__((ext_vector_type(4)));

template <int STAGE, typename TapT>
__global__ __launch_bounds__(256) void table_kernel(GenRound r) {
  const int mk = r.mk, mid = mk / 2, plane = blockIdx.z / r.nqc, qc = blockIdx.z % r.nqc;
  const int len = r.support[plane] * r.os, len_max = r.support_max * r.os;
  const int rows = STAGE == 1 ? mk : len, cols = len / 2;
  const int m0 = blockIdx.y * kGenRows, n0 = blockIdx.x * kGenCols;
  if (m0 >= rows || n0 >= cols) return;
  const double2* twiddle = r.twiddle + static_cast<size_t>(plane) * (len_max / 2) * (mid + 1);
  double2* half = r.half + static_cast<size_t>(blockIdx.z) * mk * len_max;
  const double2* phi = r.phi + static_cast<size_t>(qc) * mk * mk;
  const double2* wterm = r.wterm + static_cast<size_t>(plane) * mk * mk;
  __shared__ double fold[4][kGenRows * kGenPitch];  // even re, even im, odd re, odd im: [row][k]
  __shared__ double turn[2][kGenCols * kGenPitch];  // cos, sin: [d][k]

  const int t = threadIdx.x;
  const double2 zero = make_double2(0.0, 0.0);
  // Thread t holds rows / columns t / 16 + 16 i of sample t mod 16, so that 16 lanes read along the
  // contraction; stage 2's samples run along its rows: row t mod 32 of samples t / 32 + 8 i.
  double2 plus[2], minus[2], wplus[2], wminus[2], tw[4];
  const auto fetch = [&](int k0) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int row = m0 + (STAGE == 1 ? t / kGenK + 16 * i : t % kGenRows);
      const int k = k0 + (STAGE == 1 ? t % kGenK : t / kGenRows + 8 * i);
      const bool inp = row < rows && k < mid, inm = row < rows && k >= 1 && k <= mid;
      if (STAGE == 1) {
        const size_t o = static_cast<size_t>(row) * mk + mid;
        plus[i] = inp ? phi[o + k] : zero;
        minus[i] = inm ? phi[o - k] : zero;
        wplus[i] = inp ? wterm[o + k] : zero;
        wminus[i] = inm ? wterm[o - k] : zero;
      } else {
        plus[i] = inp ? half[static_cast<size_t>(mid + k) * len_max + row] : zero;
        minus[i] = inm ? half[static_cast<size_t>(mid - k) * len_max + row] : zero;
      }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int d = n0 + t / kGenK + 16 * i, k = k0 + t % kGenK;
      tw[i] = (d < cols && k <= mid) ? twiddle[static_cast<size_t>(d) * (mid + 1) + k] : zero;
    }
  };
  const auto store = [&]() {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int o = STAGE == 1 ? (t / kGenK + 16 * i) * kGenPitch + t % kGenK
                               : (t % kGenRows) * kGenPitch + t / kGenRows + 8 * i;
      const double2 p = STAGE == 1 ? cmul(wplus[i], plus[i]) : plus[i];
      const double2 m = STAGE == 1 ? cmul(wminus[i], minus[i]) : minus[i];
      fold[0][o] = p.x + m.x;
      fold[1][o] = p.y + m.y;
      fold[2][o] = p.x - m.x;
      fold[3][o] = p.y - m.y;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int o = (t / kGenK + 16 * i) * kGenPitch + t % kGenK;
      turn[0][o] = tw[i].x;
      turn[1][o] = tw[i].y;
    }
  };

  const int lane = t % 64, wave = t / 64;
  const int row0 = 16 * (wave / 2), col0 = 32 * (wave % 2);
  const int of = (row0 + lane % 16) * kGenPitch + lane / 16;
  const int ot = (col0 + lane % 16) * kGenPitch + lane / 16;
  const int tiles = (cols - n0 - col0 + 15) / 16;  // 16-column tiles of this wave that hold a column
  double4_t cr[2] = {}, ci[2] = {}, sr[2] = {}, si[2] = {};
  fetch(0);
  for (int k0 = 0; k0 <= mid; k0 += kGenK) {
    store();
    __syncthreads();
    if (k0 + kGenK <= mid) fetch(k0 + kGenK);
    const int steps = min(kGenK, mid + 1 - k0);
#pragma unroll
    for (int k = 0; k < kGenK; k += 4) {
      if (k >= steps) break;
      const double er = fold[0][of + k], ei = fold[1][of + k], dr = fold[2][of + k], di = fold[3][of + k];
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        if (j >= tiles) break;
        const double c = turn[0][ot + 16 * j * kGenPitch + k], s = turn[1][ot + 16 * j * kGenPitch + k];
        cr[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(er, c, cr[j], 0, 0, 0);
        ci[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(ei, c, ci[j], 0, 0, 0);
        sr[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(dr, s, sr[j], 0, 0, 0);
        si[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(di, s, si[j], 0, 0, 0);
      }
    }
    __syncthreads();
  }

  // out[row][d + S os/2 - 1]
  const auto put = [&](int row, int di, double re, double im) {
    if (STAGE == 1) {
      half[static_cast<size_t>(row) * len_max + di] = make_double2(re, im);
      return;
    }
    const int S = r.support[plane], os = r.os;
    const size_t chunk = static_cast<size_t>((di % os) * os + row % os) * (r.nqc / r.ce) + qc / r.ce;
    const size_t tap = static_cast<size_t>(di / os) * S + row / os;
    TapT* out = static_cast<TapT*>(r.table) + r.offset[plane] + (chunk * S * S + tap) * r.ce + qc % r.ce;
    if constexpr (sizeof(TapT) == 4) {
      // direct float64 -> float16 rounding (no intermediate float32 rounding)
      const _Float16 hr = static_cast<_Float16>(re), hi = static_cast<_Float16>(im);
      __half2 h;
      __builtin_memcpy(&h.x, &hr, 2);
      __builtin_memcpy(&h.y, &hi, 2);
      *out = h;
    } else {
      *out = make_float2(static_cast<float>(re), static_cast<float>(im));
    }
  };
  // Results of the float64 instruction: lane holds column lane mod 16 of rows lane / 16 + 4 i.
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int d = n0 + col0 + 16 * j + lane % 16;
    if (d >= cols) break;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = m0 + row0 + lane / 16 + 4 * i;
      if (row >= rows) continue;
      put(row, cols - 1 + d, cr[j][i] - si[j][i], ci[j][i] + sr[j][i]);
      if (d > 0)
        put(row, cols - 1 - d, cr[j][i] + si[j][i], ci[j][i] - sr[j][i]);
      else
        put(row, len - 1, 0.0, 0.0);
    }
  }
}

// One Mueller cell of one plane from a dense [phase_y][phase_x][tap_y][tap_x][re, im] float array
// into the chunk-major table.
// Moves Mueller cells between a chunk-major table and a plain float buffer laid out
// [plane][cell][phase_y][phase_x][tap_y][tap_x][re, im].  Planes plane0 .. plane0+nplanes-1 share
// one support, so plane i starts os^2 S^2 nqc entries after plane i-1; cells are qc0 .. qc0+ncell-1.
// to_table: table <- scale[qc] * buf (rounded to the storage type); else buf <- table.
__global__ void cell_io_kernel(void* __restrict__ table, int storage, int nqc, int ce, int os, int support,
                               int64_t offset0, int nplanes, int qc0, int ncell, float* __restrict__ buf,
                               int to_table, CellScale scale) {
  const size_t ss = static_cast<size_t>(support) * support;
  const size_t per_cell = ss * os * os;
  const size_t total = per_cell * ncell * nplanes;
  const size_t nch = nqc / ce;
  const size_t plane_stride = per_cell * nqc;
  for (size_t i = blockIdx.x * static_cast<size_t>(blockDim.x) + threadIdx.x; i < total;
       i += static_cast<size_t>(gridDim.x) * blockDim.x) {
    const size_t r = i % per_cell, pc = i / per_cell;
    const int qc = qc0 + static_cast<int>(pc % ncell);
    const size_t plane = pc / ncell;
    const size_t phase = r / ss, tap = r % ss;
    const size_t ch = qc / ce, e = qc % ce;
    const size_t dst = offset0 + plane * plane_stride + ((phase * nch + ch) * ss + tap) * ce + e;
    if (to_table) {
      const float re = buf[2 * i] * scale.v[qc], im = buf[2 * i + 1] * scale.v[qc];
      if (storage == PG_STORE_F16) {
        static_cast<__half2*>(table)[dst] = __floats2half2_rn(re, im);
      } else {
        static_cast<float2*>(table)[dst] = make_float2(re, im);
      }
    } else {
      float2 v;
      if (storage == PG_STORE_F16) {
        v = __half22float2(static_cast<const __half2*>(table)[dst]);
      } else {
        v = static_cast<const float2*>(table)[dst];
      }
      buf[2 * i] = v.x;
      buf[2 * i + 1] = v.y;
    }
  }
}

// kbound[4 p + q] = max over the entries of Mueller row q in plane p's table of |re| + |im|, the
// bound the shared-tap gridder scales its fixed point from.  A plane's table is os^2 phases of nch chunks
// of ss E entries, entry i of a chunk being tap i / E, Mueller cell chunk E + i mod E.  One pass over
// the tables, bounded by reading them: blockIdx.y is the plane, and at most 64 blocks walk its chunks,
// each with one integer atomic max a row at its end (non-negative floats order like their bits).  (One
// block and 16 atomics for each chunk queued at four addresses: 28 us a plane, now 66 us for 24.)
__device__ inline float2 entry_value(float2 t) { return t; }
__device__ inline float2 entry_value(__half2 t) { return __half22float2(t); }

template <typename TapT>
__global__ __launch_bounds__(256) void kernel_bound_kernel(const TapT* __restrict__ table,
                                                           const PlaneInfo* __restrict__ planes, int plane0, int os,
                                                           int e_per_chunk, int nch, int npol, unsigned* __restrict__ out) {
  const int plane = plane0 + blockIdx.y;
  const int per_chunk = planes[plane].support * planes[plane].support * e_per_chunk;
  table += planes[plane].offset;
  float m[4] = {0.0f, 0.0f, 0.0f, 0.0f};
  for (int c = blockIdx.x; c < os * os * nch; c += gridDim.x) {
    const TapT* blk = table + static_cast<size_t>(c) * per_chunk;
    const int cell0 = c % nch * e_per_chunk;
    for (int i = threadIdx.x; i < per_chunk; i += 256) {
      const int q = (cell0 + (i & (e_per_chunk - 1))) / npol;
      const float2 t = entry_value(blk[i]);
      const float a = fabsf(t.x) + fabsf(t.y);
#pragma unroll
      for (int qq = 0; qq < 4; ++qq)
        if (qq == q) m[qq] = fmaxf(m[qq], a);
    }
  }
  __shared__ float best[4][4];
#pragma unroll
  for (int qq = 0; qq < 4; ++qq) {
    float v = m[qq];
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) v = fmaxf(v, __shfl_xor(v, d, 64));
    if ((threadIdx.x & 63) == 0) best[qq][threadIdx.x >> 6] = v;
  }
  __syncthreads();
  if (threadIdx.x < 4) {
    const float* v = best[threadIdx.x];
    const float top = fmaxf(fmaxf(v[0], v[1]), fmaxf(v[2], v[3]));
    if (top > 0.0f) atomicMax(out + 4 * plane + threadIdx.x, __float_as_uint(top));
  }
}

}  // namespace

hipError_t cell_io(void* table, int storage, int nqc, int ce, int os, int support, int64_t offset0, int nplanes,
                   int qc0, int ncell, float* buf, bool to_table, const CellScale& scale, hipStream_t s) {
  const size_t total = static_cast<size_t>(support) * support * os * os * ncell * nplanes;
  if (total == 0) return hipSuccess;
  const int blocks = static_cast<int>(std::min<size_t>((total + 255) / 256, 65535));
  hipLaunchKernelGGL(cell_io_kernel, dim3(blocks), dim3(256), 0, s, table, storage, nqc, ce, os, support, offset0,
                     nplanes, qc0, ncell, buf, to_table ? 1 : 0, scale);
  return hipGetLastError();
}

hipError_t launch_screens(int npol, int kind, const double* jones, const double* jones_b, int mk, const double beta[4],
                          int convention, double2* phi, hipStream_t s) {
  const size_t npix = static_cast<size_t>(mk) * mk;
  if (npol == 1) {
    hipLaunchKernelGGL(unit_screen_kernel, dim3(static_cast<unsigned>((npix + 255) / 256)), dim3(256), 0, s, npix, phi);
  } else {
    hipLaunchKernelGGL(screens_kernel, dim3(static_cast<unsigned>((npix + 63) / 64)), dim3(64), 0, s, kind, jones, jones_b,
                       npix, make_double4(beta[0], beta[1], beta[2], beta[3]), convention, phi);
  }
  return hipGetLastError();
}

hipError_t launch_place_screens(const uint32_t* px, const double2* at, size_t count, size_t npix, double2* phi, hipStream_t s) {
  hipLaunchKernelGGL(place_screens_kernel, dim3(static_cast<unsigned>((16 * count + 255) / 256)), dim3(256), 0, s, px, at,
                     count, npix, phi);
  return hipGetLastError();
}

hipError_t launch_tables(const GenRound& r, hipStream_t s) {
  const unsigned len = static_cast<unsigned>(r.support_max * r.os), mk = static_cast<unsigned>(r.mk);
  const unsigned count = static_cast<unsigned>(r.count), cells = count * r.nqc;
  const auto ceil_div = [](unsigned n, unsigned d) { return (n + d - 1) / d; };
  const unsigned cols = ceil_div(len / 2, kGenCols);
  hipLaunchKernelGGL(wterm_kernel, dim3(ceil_div(mk, 128), mk, count), dim3(128), 0, s, r);
  hipLaunchKernelGGL(twiddle_kernel, dim3(ceil_div(mk / 2 + 1, 128), len / 2, count), dim3(128), 0, s, r);
  hipLaunchKernelGGL((table_kernel<1, float2>), dim3(cols, ceil_div(mk, kGenRows), cells), dim3(256), 0, s, r);
  const dim3 grid(cols, ceil_div(len, kGenRows), cells);
  if (r.storage == PG_STORE_F16)
    hipLaunchKernelGGL((table_kernel<2, __half2>), grid, dim3(256), 0, s, r);
  else
    hipLaunchKernelGGL((table_kernel<2, float2>), grid, dim3(256), 0, s, r);
  return hipGetLastError();
}

hipError_t refresh_kernel_bound(pg_kernels* k, int plane0, int nplanes, hipStream_t s) {
  if (nplanes <= 0) return hipSuccess;
  hipError_t e = launch_fill_zero(k->kbound.as<float>() + 4 * plane0, sizeof(float) * 4 * nplanes, s);
  if (e != hipSuccess) return e;
  const int nqc = k->npol * k->npol;
  const int ec = chunk_entries(k->storage, nqc), nch = nqc / ec;
  unsigned* out = k->kbound.as<unsigned>();
  for (int p = 0; p < nplanes; p += 65535) {
    const dim3 grid(static_cast<unsigned>(std::min(k->os * k->os * nch, 64)), static_cast<unsigned>(std::min(nplanes - p, 65535)));
    if (k->storage == PG_STORE_F16)
      hipLaunchKernelGGL(kernel_bound_kernel<__half2>, grid, dim3(256), 0, s, k->table.as<__half2>(),
                         k->planes.as<PlaneInfo>(), plane0 + p, k->os, ec, nch, k->npol, out);
    else
      hipLaunchKernelGGL(kernel_bound_kernel<float2>, grid, dim3(256), 0, s, k->table.as<float2>(),
                         k->planes.as<PlaneInfo>(), plane0 + p, k->os, ec, nch, k->npol, out);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace pg

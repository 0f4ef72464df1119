// Vertically implicit diffusion (vertically implicit time-discretisation
// paragraph of the time-stepping appendix of arXiv 2502.14148: the tracer
// and predictor-velocity equations (1 - dt d/dz K d/dz) X^new = X~ with a
// second-order discretisation of the vertical diffusion operator, solved
// with a tridiagonal algorithm per column).
//
// Every column of a field shares one matrix (K and the z grid do not vary
// horizontally), so everything that depends on the matrix alone is computed
// once on the host in FP64.  The elimination is written as two first-order
// linear recurrences,
//   forward:  d_q = A_q d_{q-1} + I_q x~_q      (A_q = -s_q / p_q, I_q = 1/p_q)
//   backward: x_q = d_q + B_q x_{q+1}           (B_q = -sup_q / p_q)
// with s, sup the sub- and super-diagonal and p the pivots.  The n unknowns
// of a column are split into VCH chunks of C levels, one per wavefront of a
// workgroup, each wave holding its chunk of 64 columns in registers.  A chunk
// solves its recurrences from zero; the true solution adds the incoming
// value times the precomputed products P_q = A_{q0}..A_q (forward) and
// Q_q = B_q..B_{q1-1} (backward), and the incoming values are chained across
// the chunks through LDS.  Each element is read once and written once.
#include <algorithm>
#include <vector>

#include "oc_internal.h"

namespace oc {

namespace {
constexpr int VCH = 8;      // chunks (wavefronts) per column group
constexpr int VCMAX = 32;   // levels per chunk at most (n <= 256)
}  // namespace

int vertical_chunk(int n) { return (n + VCH - 1) / VCH; }

void vertical_factors(const double* dzc, const double* dzf, int nz, double K, double dt,
                      int wface, double* out) {
  const int n = wface ? nz - 1 : nz;
  const int C = vertical_chunk(n);
  double* A = out;
  double* I = out + n;
  double* P = out + 2 * n;
  double* B = out + 3 * n;
  double* Q = out + 4 * n;
  double* PE = out + 5 * n;         // per chunk: P at its last level (1 if empty)
  double* QS = PE + VCH;            // per chunk: Q at its first level (1 if empty)
  std::vector<double> sup(n);
  double cprev = 0.0;
  for (int q = 0; q < n; ++q) {
    double lo, up, diag;
    if (wface) {
      // w on face k = q + 1, between the centres k - 1 and k (w = 0 on walls)
      const int k = q + 1;
      lo = K / (dzc[k - 1] * dzf[k]);
      up = K / (dzc[k] * dzf[k]);
      diag = 1.0 + dt * (lo + up);
      if (q == 0) lo = 0.0;
      if (q == n - 1) up = 0.0;
    } else {
      // centred cell k = q; no diffusive flux through the walls
      lo = (q > 0) ? K / (dzc[q] * dzf[q]) : 0.0;
      up = (q < n - 1) ? K / (dzc[q] * dzf[q + 1]) : 0.0;
      diag = 1.0 + dt * (lo + up);
    }
    const double s = -dt * lo;
    const double piv = diag - s * cprev;
    I[q] = 1.0 / piv;
    A[q] = -s / piv;
    sup[q] = -dt * up;
    cprev = sup[q] / piv;
    B[q] = -cprev;
  }
  for (int c = 0; c < VCH; ++c) {
    const int q0 = c * C, q1 = std::min(q0 + C, n);
    double prod = 1.0;
    for (int q = q0; q < q1; ++q) {
      prod *= A[q];
      P[q] = prod;
    }
    PE[c] = (q1 > q0) ? P[q1 - 1] : 1.0;
    prod = 1.0;
    for (int q = q1 - 1; q >= q0; --q) {
      prod *= B[q];
      Q[q] = prod;
    }
    QS[c] = (q1 > q0) ? Q[q0] : 1.0;
  }
}

int vertical_factors_len(int nz) { return 5 * nz + 2 * VCH; }

namespace {

// A uniform value the compiler can derive nothing from (nor hoist what follows
// from it out of a loop).
template <class P>
__device__ inline P opaque(P p) {
  asm volatile("" : "+s"(p));
  return p;
}

// CM: levels per chunk at most, which are the column's registers.  Memory
// bound (67 us at 5.2 TB/s for the 5 fields of 256x256x128 FP32, each read
// and written once): what counts is the waves in flight, so the registers are
// held to the column itself (the level addresses are uniform, 32 bits per
// lane), and the stores, so the halo images are not tested for level by level.
// 5 fields, with every chunk of 32 levels at most and the images tested at
// each level, and now: 256x256x128 FP32 149 -> 91 us, 256x256x200 FP32
// 199 -> 168, 128x128x64 FP64 37.5 -> 24, 128x128x256 FP64 95 -> 87, 64x64x32
// FP32 15 -> 9.6.  (16 chunks instead of 8: 123 us for the first.)  Long columns
// of short rows, by events around the launch: 64x64x256 FP32 36.3 -> 33.4, FP64
// 44.4 -> 39.9, 32x64x256 FP32 27.3 -> 25.8 (39.7, 48.9 and 30.1 with a pass of
// images for each side).
template <class T, int CM>
__global__ void __launch_bounds__(64 * VCH) vimplicit_kernel(Dims d, VImplicitArgs<T> a) {
  __shared__ T endv[VCH][64];
  __shared__ T startv[VCH][64];
  const int fld = blockIdx.y;
  T* __restrict__ f = a.f[fld];
  const int wface = a.wface[fld];
  const T* __restrict__ tab = a.fac[fld];
  const int n = wface ? d.nz - 1 : d.nz, k0 = wface ? 1 : 0;
  const int C = (n + VCH - 1) / VCH;
  const T* A = tab;
  const T* I = tab + n;
  const T* P = tab + 2 * n;
  const T* B = tab + 3 * n;
  const T* Q = tab + 4 * n;
  const T* PE = tab + 5 * n;
  const T* QS = PE + VCH;
  // the chunk is the wavefront index: uniform, so the tables are scalar loads
  const int lane = threadIdx.x & 63;
  const int c = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // Workgroups are dealt round-robin to the 8 XCDs (XCD x takes x, x + 8,
  // ...); renumber the column groups so that each XCD takes a contiguous run
  // of them: neighbouring groups share the cache lines at their ends (rows
  // are not 128-byte aligned), which then meet in one L2
  const int ng = (int)gridDim.x, bx = (int)blockIdx.x, xcd = bx % 8;
  const int grp = xcd * (ng / 8) + min(xcd, ng % 8) + bx / 8;
  const int col = grp * 64 + lane;
  const bool valid = col < d.nx * d.ny;
  const int i = valid ? col % d.nx : 0, j = valid ? col / d.nx : 0;
  const int q0 = c * C;
  const int q1 = min(q0 + C, n);
  const long sz = d.sz;
  const int H = d.h;
  const uint32_t own = (uint32_t)((j + H) * (int)d.sy + i + H);
  T x[CM];
  {
    const T* lv = f + (long)(k0 + q0 + H) * sz;
#pragma unroll
    for (int r = 0; r < CM; ++r) {
      if (q0 + r < q1) x[r] = lv[own];
      lv += sz;
    }
  }
  T pe[VCH], qs[VCH];
#pragma unroll
  for (int cc = 0; cc < VCH; ++cc) {
    pe[cc] = PE[cc];
    qs[cc] = QS[cc];
  }
  // forward recurrence within the chunk, from zero
  T dl = T(0);
#pragma unroll
  for (int r = 0; r < CM; ++r) {
    const int q = q0 + r;
    if (q < q1) {
      dl = A[q] * dl + I[q] * x[r];
      x[r] = dl;
    }
  }
  endv[c][lane] = dl;
  __syncthreads();
  T din = T(0);
  {
    T ev[VCH];
#pragma unroll
    for (int cc = 0; cc < VCH - 1; ++cc) ev[cc] = endv[cc][lane];
#pragma unroll
    for (int cc = 0; cc < VCH - 1; ++cc) din = cc < c ? pe[cc] * din + ev[cc] : din;
  }
  // backward recurrence within the chunk (after the forward correction)
  T xl = T(0);
#pragma unroll
  for (int r = CM - 1; r >= 0; --r) {
    const int q = q0 + r;
    if (q < q1) {
      xl = (x[r] + P[q] * din) + B[q] * xl;
      x[r] = xl;
    }
  }
  startv[c][lane] = xl;
  __syncthreads();
  T xin = T(0);
  {
    T sv[VCH];
#pragma unroll
    for (int cc = VCH - 1; cc > 0; --cc) sv[cc] = startv[cc][lane];
#pragma unroll
    for (int cc = VCH - 1; cc > 0; --cc) xin = cc > c ? qs[cc] * xin + sv[cc] : xin;
  }
  if (!valid) return;
#pragma unroll
  for (int r = 0; r < CM; ++r) x[r] += Q[min(q0 + r, n - 1)] * xin;
  // The column, then its periodic x / y images (of the h columns next to each
  // side): image m is shifted by a length of x (m % 3) and of y (m / 3): 1 is the
  // image past the other end, up for a column next to the start and down for one
  // next to the end (one pass for both: a wave of a row of 64 holds both); 2 the
  // second image, down, of a column within reach of both ends of an axis shorter
  // than 2H.  A combination that no lane has is passed over whole, so the
  // interior pays for it once per column and not once per level.
  const bool edge = k0 + q0 <= H || k0 + q1 >= d.nz - H;   // levels with mirror images
#pragma unroll 1
  for (int m = 0; m < 9; ++m) {
    const int mx = m % 3, my = m / 3;
    const bool xl = i < H, xh = i >= d.nx - H, yl = j < H, yh = j >= d.ny - H;
    const bool has = (mx == 0 || (mx == 1 ? xl || xh : xl && xh)) &&
                     (my == 0 || (my == 1 ? yl || yh : yl && yh));
    if (!has) continue;
    const int ox = mx == 0 ? 0 : mx == 1 && xl ? d.nx : -d.nx;
    const int oy = my == 0 ? 0 : my == 1 && yl ? d.ny : -d.ny;
    const uint32_t at = own + (uint32_t)(ox + oy * (int)d.sy);
    // (opaque: the level addresses and signed values are formed here instead
    // of being kept for all levels across the combinations, which spills)
    const int kb = opaque(k0 + q0), nl = opaque(q1 - q0), odd = opaque(wface);
    T* lv = f + (long)(kb + H) * sz;
#pragma unroll
    for (int r = 0; r < CM; ++r) {
      if (r < nl) lv[at] = x[r];
      lv += sz;
    }
    if (edge) {
      // mirror images of the levels next to the walls: even for a centred
      // field, odd about the wall faces for w
#pragma unroll
      for (int r = 0; r < CM; ++r) {
        const int k = kb + r;
        if (r < nl) {
          const T v = odd ? -x[r] : x[r];
          const int lo = wface ? -k : -1 - k, hi = wface ? 2 * d.nz - k : 2 * d.nz - 1 - k;
          if (lo >= -H) f[(long)(lo + H) * sz + at] = v;
          if (hi < d.nz + H) f[(long)(hi + H) * sz + at] = v;
        }
      }
    }
  }
}

}  // namespace

template <class T>
hipError_t launch_vertical_implicit(const Dims& d, const VImplicitArgs<T>& a, int nfields,
                                    hipStream_t s) {
  if (!d.zb || d.nz > VCH * VCMAX || nfields < 1 || nfields > MAXF) return hipErrorInvalidValue;
  const int cols = d.nx * d.ny;
  const dim3 grid((cols + 63) / 64, nfields), nt(64 * VCH);
  // by the levels of a chunk: the larger bounds hold more registers (18, 22,
  // 30 and 58 in FP32) and issue the loops of empty levels, 149 against 108 us
  // at 256x256x128 with 32 in place of 16
  const int C = vertical_chunk(d.nz);
  if (C <= 4)
    hipLaunchKernelGGL((vimplicit_kernel<T, 4>), grid, nt, 0, s, d, a);
  else if (C <= 8)
    hipLaunchKernelGGL((vimplicit_kernel<T, 8>), grid, nt, 0, s, d, a);
  else if (C <= 16)
    hipLaunchKernelGGL((vimplicit_kernel<T, 16>), grid, nt, 0, s, d, a);
  else
    hipLaunchKernelGGL((vimplicit_kernel<T, 32>), grid, nt, 0, s, d, a);
  return hipGetLastError();
}

template hipError_t launch_vertical_implicit<float>(const Dims&, const VImplicitArgs<float>&, int,
                                                    hipStream_t);
template hipError_t launch_vertical_implicit<double>(const Dims&, const VImplicitArgs<double>&,
                                                     int, hipStream_t);

}  // namespace oc

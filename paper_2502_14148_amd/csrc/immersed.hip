// Grid-fitted immersed boundaries: the vector kernels of the preconditioned
// conjugate-gradient pressure solve (pressure solver for irregular domains of
// the pressure-correction appendix of arXiv 2502.14148) and the masking of
// velocities on closed faces.
//
// The equation: on the fluid cells, the 7-point Laplacian A with no flux
// through faces next to an immersed cell (or a wall) equals b = div(u~) /
// dt_eff; gauge: zero mean over the fluid cells.  The preconditioner is P L^-1,
// L^-1 the FFT/DCT solve of the whole box (poisson.hip) and P the restriction
// to the fluid cells.
//
// A and L have the same row in every fluid cell that has no immersed
// neighbour, and P changes L^-1 x only in immersed cells.  So A P L^-1 x = x in
// all fluid cells but those next to immersed ones (the list): starting from
// the iterate P L^-1 b, every residual, and every A q of a direction q = P
// L^-1 s, is zero off the list.  The iteration therefore keeps the vectors r,
// s and A q on the list alone (1 to 2 % of the cells of a seamount), A q by its
// recurrence A q = A z + beta A q; q itself is not formed (its products are
// taken with A q, which A's symmetry allows).  It needs z = L^-1 r only on the
// list and its neighbours, and the FFT passes skip the levels and rows where the
// residual is zero or the result unused.  The steps are summed as
// sum alpha s, and the solution is p = L^-1 (b + sum alpha s), one more solve
// whose last pass is the projection's.  Against the iteration on dense
// vectors (operator, direction and residual passes of 83 bytes per cell and
// an unrestricted solve each time) a 128^3 step over a seamount went from
// 6.9 to 3.1 ms, a 256^3 one from 29.8 to 10.0 ms, with the same residuals.
//
// Vectors are FP64; the geometry comes as one byte per cell (IB_* bits: the
// cell is fluid, and which of its six faces are open).  Reductions are
// deterministic: every reducing kernel runs a grid that depends on the sizes
// alone over a fixed partition, each workgroup writes its partial sums, and
// the last one to finish adds all of them in a fixed order and updates the
// iteration's scalars on the device (no host round trip inside an iteration,
// no launch for a sum).
#include <algorithm>

#include "oc_internal.h"

namespace oc {

namespace {

constexpr int IB_NT = 256;

// Sums of K values over the workgroup, in every thread.
template <int K>
__device__ inline void block_sums(double (&v)[K], double (*sh)[IB_NT]) {
  const int t = threadIdx.x;
#pragma unroll
  for (int q = 0; q < K; ++q) sh[q][t] = v[q];
  __syncthreads();
#pragma unroll
  for (int s = IB_NT / 2; s > 0; s >>= 1) {
    if (t < s)
#pragma unroll
      for (int q = 0; q < K; ++q) sh[q][t] += sh[q][t + s];
    __syncthreads();
  }
#pragma unroll
  for (int q = 0; q < K; ++q) v[q] = sh[q][0];
  __syncthreads();
}

// Sums of K values over the grid: every workgroup leaves its partial sums
// (part[q gridDim.x + block]); the last one to arrive at the ticket adds them
// in a fixed order and gets true, with the sums in every thread.  No
// workgroup waits for another.  The partial sums pass between XCDs: written
// and read at device scope around the ticket.
template <int K>
__device__ inline bool grid_sums(double (&v)[K], double* part, unsigned* ticket,
                                 double (*sh)[IB_NT]) {
  __shared__ bool last;
  block_sums<K>(v, sh);
  if (threadIdx.x == 0) {
#pragma unroll
    for (int q = 0; q < K; ++q)
      __hip_atomic_store(&part[q * gridDim.x + blockIdx.x], v[q], __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
    last = __hip_atomic_fetch_add(ticket, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) ==
           gridDim.x - 1;
  }
  __syncthreads();
  if (!last) return false;
  __threadfence();
#pragma unroll
  for (int q = 0; q < K; ++q) {
    v[q] = 0.0;
    for (unsigned b = threadIdx.x; b < gridDim.x; b += IB_NT)
      v[q] += __hip_atomic_load(&part[q * gridDim.x + b], __ATOMIC_RELAXED,
                                __HIP_MEMORY_SCOPE_AGENT);
  }
  block_sums<K>(v, sh);
  if (threadIdx.x == 0) *ticket = 0u;   // for the next kernel
  return true;
}

// Workgroups are dealt round-robin to the 8 XCDs; the stencil kernels
// renumber them so that each XCD sweeps a contiguous range of cells in every
// round of the grid-stride loop, and the neighbouring planes a cell reads
// stay in that XCD's L2.
__device__ inline long first_cell() {
  const unsigned nb = gridDim.x, b = blockIdx.x;
  const unsigned vb = (nb % 8 == 0) ? (b % 8) * (nb / 8) + b / 8 : b;
  return (long)vb * IB_NT + threadIdx.x;
}

// (i, j, k) of a dense index (32-bit arithmetic: N < 2^31)
__device__ inline void cell_of(const Dims& d, long n, int& i, int& j, int& k) {
  const unsigned u = (unsigned)n, nx = (unsigned)d.nx, ny = (unsigned)d.ny;
  const unsigned r = u / nx;
  i = (int)(u - r * nx);
  k = (int)(r / ny);
  j = (int)(r - (unsigned)k * ny);
}

// b = div(u~) / dt_eff in fluid cells (face velocities times their open
// flags), 0 in immersed cells; partial sums of b^2.
template <class T>
__global__ void __launch_bounds__(IB_NT) ib_rhs_kernel(Dims d, const T* __restrict__ u,
                                                       const T* __restrict__ v,
                                                       const T* __restrict__ w,
                                                       const uint8_t* __restrict__ bits,
                                                       double inv_dt, double rdx, double rdy,
                                                       double rdz, CgBufs cg) {
  __shared__ double sh[1][IB_NT];
  const long N = (long)d.nx * d.ny * d.nz;
  double acc = 0.0;
  for (long n = first_cell(); n < N; n += (long)gridDim.x * IB_NT) {
    const unsigned fb = bits[n];
    double b = 0.0;
    if (fb & IB_FLUID) {
      int i, j, k;
      cell_of(d, n, i, j, k);
      const long c = pidx(d, i, j, k);
      const double ul = (fb & IB_XM) ? (double)u[c] : 0.0;
      const double ur = (fb & IB_XP) ? (double)u[pidx(d, (i + 1 == d.nx) ? 0 : i + 1, j, k)] : 0.0;
      const double vl = (fb & IB_YM) ? (double)v[c] : 0.0;
      const double vr = (fb & IB_YP) ? (double)v[pidx(d, i, (j + 1 == d.ny) ? 0 : j + 1, k)] : 0.0;
      const double wb = (fb & IB_ZM) ? (double)w[c] : 0.0;
      const double wt = (fb & IB_ZP) ? (double)w[pidx(d, i, j, (k + 1 == d.nz) ? 0 : k + 1)] : 0.0;
      b = ((ur - ul) * rdx + (vr - vl) * rdy + (wt - wb) * rdz) * inv_dt;
    }
    cg.b[n] = b;
    acc += b * b;
  }
  // partial sums only, added by ib_start_kernel: a ticket per workgroup of
  // this many would take longer than the kernel (48 us against 18 at 128^3)
  double b2[1] = {acc};
  block_sums<1>(b2, sh);
  if (threadIdx.x == 0) cg.bpart[blockIdx.x] = b2[0];
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    cg.scal[CG_IT] = 0.0;
    cg.scal[CG_DONE] = 0.0;
  }
}

// (A z)_n of the masked 7-point operator at a fluid cell: only neighbours
// across open faces are read.
struct ListGeom {
  Dims d;
  const uint8_t* bits;
  double rdx2, rdy2, rdz2;
};
__device__ inline double apply_at(const ListGeom& g, const double* __restrict__ z, int n,
                                  double z0) {
  int i, j, k;
  cell_of(g.d, n, i, j, k);
  const unsigned fb = g.bits[n];
  const int sy = g.d.nx, sz = g.d.nx * g.d.ny;
  const int xm = (i == 0) ? n + g.d.nx - 1 : n - 1, xp = (i + 1 == g.d.nx) ? n - i : n + 1;
  const int ym = (j == 0) ? n + sz - sy : n - sy, yp = (j + 1 == g.d.ny) ? n - j * sy : n + sy;
  const int zm = (k == 0) ? n + (g.d.nz - 1) * sz : n - sz, zp = (k + 1 == g.d.nz) ? n - k * sz : n + sz;
  // all six loads before the first difference (with a load in each difference
  // they wait for each other: 128^3 with 15 % of the cells immersed, a list of
  // 1 million, 19.9 ms a step instead of 14.2; loading also across closed faces
  // costs a 256^3 seamount 1 %)
  auto at = [&](unsigned bit, int m) { return (fb & bit) ? z[m] : 0.0; };
  const double vxm = at(IB_XM, xm), vxp = at(IB_XP, xp), vym = at(IB_YM, ym),
               vyp = at(IB_YP, yp), vzm = at(IB_ZM, zm), vzp = at(IB_ZP, zp);
  auto dif = [&](unsigned bit, double v) { return (fb & bit) ? v - z0 : 0.0; };
  return (dif(IB_XM, vxm) + dif(IB_XP, vxp)) * g.rdx2 +
         (dif(IB_YM, vym) + dif(IB_YP, vyp)) * g.rdy2 +
         (dif(IB_ZM, vzm) + dif(IB_ZP, vzp)) * g.rdz2;
}

// Stopping test after an iteration (an update of the iterate) with squared
// residual r2.
__device__ inline void stop_test(double* sc, double r2, double tol2, int maxiter) {
  sc[CG_RNORM2] = r2;
  sc[CG_IT] += 1.0;
  if (r2 <= tol2 * sc[CG_BNORM2] || sc[CG_IT] >= (double)maxiter) sc[CG_DONE] = 1.0;
}

// After z = L^-1 b: r = b - A P z, |b|^2 and |r|^2.  The iterate P z precedes the
// iterations that are counted and limited (k of them from here leave a smaller
// residual than k from p = 0); only where it meets the tolerance by itself is
// it one.
template <int U>
__global__ void __launch_bounds__(IB_NT) ib_start_kernel(ListGeom g, CgBufs cg,
                                                         const double* __restrict__ z,
                                                         double tol2) {
  __shared__ double sh[1][IB_NT];
  double v[1] = {0.0};
  double r[U];
  list_entries<U>(
      cg, blockIdx.x * IB_NT + threadIdx.x, gridDim.x * IB_NT,
      [&](int q, int, int n) { r[q] = cg.b[n] - apply_at(g, z, n, z[n]); },
      [&](int q, int e, int n) {
        cg.r[n] = r[q];
        cg.s[e] = 0.0;
        cg.aq[e] = 0.0;
        v[0] += r[q] * r[q];
      });
  if (!grid_sums<1>(v, cg.part, cg.ticket, sh)) return;
  double b2[1] = {0.0};
  for (int b = threadIdx.x; b < IB_NPART; b += IB_NT) b2[0] += cg.bpart[b];
  block_sums<1>(b2, sh);
  if (threadIdx.x != 0) return;
  double* sc = cg.scal;
  sc[CG_BNORM2] = b2[0];
  sc[CG_RZ] = 0.0;
  sc[CG_QAQ] = 0.0;
  sc[CG_RNORM2] = b2[0] == 0.0 ? 0.0 : v[0];
  if (b2[0] == 0.0) {   // nothing to solve: no iteration
    sc[CG_DONE] = 1.0;
  } else if (v[0] <= tol2 * b2[0]) {
    sc[CG_IT] = 1.0;
    sc[CG_DONE] = 1.0;
  }
}

// The scalars of an iteration from r.z, z.Az and z.Aq_old: beta = (r.z) / (r.z)_old
// (0 at first), and with q = z + beta q_old the q.Aq = z.Az + 2 beta z.Aq_old +
// beta^2 q_old.Aq_old (A is symmetric), so alpha is known before A q is updated.
__device__ inline void scalars(double* sc, double rz, double zaz, double zaq) {
  const double beta = sc[CG_RZ] == 0.0 ? 0.0 : rz / sc[CG_RZ];
  const double qaq = zaz + beta * (2.0 * zaq + beta * sc[CG_QAQ]);
  sc[CG_RZ] = rz;
  sc[CG_BETA] = beta;
  sc[CG_QAQ] = qaq;
  sc[CG_ALPHA] = rz / qaq;
}

// Every `stride`-th list entry from e0 on, U at a time: load(q, e, n) takes what
// entry e (cell n) needs into element q, use(q, e, n) computes and stores.  The
// loads of U entries travel together; the compiler could not move an entry's
// before the stores of the one ahead.  (Past the list's end the thread's own entry
// e is loaded again and not used: no other thread stores to it.)
template <int U, class Load, class Use>
__device__ inline void list_entries(const CgBufs& cg, int e0, int stride, Load load, Use use) {
  for (int e = e0; e < cg.n; e += U * stride) {
    int ee[U], n[U];
#pragma unroll
    for (int q = 0; q < U; ++q) {
      ee[q] = e + q * stride < cg.n ? e + q * stride : e;
      n[q] = cg.idx[ee[q]];
    }
#pragma unroll
    for (int q = 0; q < U; ++q) load(q, ee[q], n[q]);
#pragma unroll
    for (int q = 0; q < U; ++q)
      if (e + q * stride < cg.n) use(q, ee[q], n[q]);
  }
}

// A z on the list, and this thread's parts of r.z, z.Az and z.Aq_old.
template <int U>
__device__ inline void list_az(const ListGeom& g, const CgBufs& cg, const double* __restrict__ z,
                               int e0, int stride, double (&v)[3]) {
  double z0[U], az[U], r[U], aq[U];
  list_entries<U>(
      cg, e0, stride,
      [&](int q, int e, int n) {
        z0[q] = z[n];
        az[q] = apply_at(g, z, n, z0[q]);
        r[q] = cg.r[n];
        aq[q] = cg.aq[e];
      },
      [&](int q, int e, int) {
        cg.az[e] = az[q];
        v[0] += r[q] * z0[q];
        v[1] += z0[q] * az[q];
        v[2] += z0[q] * aq[q];
      });
}

// The updates: s = r + beta s, A q = A z + beta A q; the step alpha s into b;
// r -= alpha A q, and this thread's part of |r|^2.
template <int U>
__device__ inline double list_step(const CgBufs& cg, int e0, int stride, double alpha,
                                   double beta) {
  double r0[U], s0[U], az[U], aq0[U], b0[U], r2 = 0.0;
  list_entries<U>(
      cg, e0, stride,
      [&](int q, int e, int n) {
        r0[q] = cg.r[n];
        s0[q] = cg.s[e];
        az[q] = cg.az[e];
        aq0[q] = cg.aq[e];
        b0[q] = cg.b[n];
      },
      [&](int q, int e, int n) {
        const double s = r0[q] + beta * s0[q], aq = az[q] + beta * aq0[q];
        const double r = r0[q] - alpha * aq;
        cg.s[e] = s;
        cg.aq[e] = aq;
        cg.b[n] = b0[q] + alpha * s;
        cg.r[n] = r;
        r2 += r * r;
      });
  return r2;
}

// An iteration after z = L^-1 r in two launches: A z and the scalars, then the
// updates, |r|^2 and the stopping test.
template <int U>
__global__ void __launch_bounds__(IB_NT) ib_az_kernel(ListGeom g, CgBufs cg,
                                                      const double* __restrict__ z) {
  __shared__ double sh[3][IB_NT];
  if (cg.scal[CG_DONE] != 0.0) return;
  double v[3] = {0.0, 0.0, 0.0};
  list_az<U>(g, cg, z, blockIdx.x * IB_NT + threadIdx.x, gridDim.x * IB_NT, v);
  if (grid_sums<3>(v, cg.part, cg.ticket, sh) && threadIdx.x == 0)
    scalars(cg.scal, v[0], v[1], v[2]);
}

template <int U>
__global__ void __launch_bounds__(IB_NT) ib_step_kernel(CgBufs cg, double tol2, int maxiter) {
  __shared__ double sh[1][IB_NT];
  if (cg.scal[CG_DONE] != 0.0) return;
  const double alpha = cg.scal[CG_ALPHA], beta = cg.scal[CG_BETA];
  double v[1] = {
      list_step<U>(cg, blockIdx.x * IB_NT + threadIdx.x, gridDim.x * IB_NT, alpha, beta)};
  if (grid_sums<1>(v, cg.part, cg.ticket, sh) && threadIdx.x == 0)
    stop_test(cg.scal, v[0], tol2, maxiter);
}

// The whole iteration in one workgroup, for lists of up to IB_ONE_MAX entries,
// where the two launches and their tickets cost more than the work: a solve's
// iteration takes 2.9 us less with it at 596 entries and 2.2 us less at 2656;
// at 11916 one CU's gathers take 91 us against the launches' 16.
constexpr int IB_ONE = 1024, IB_ONE_U = 3, IB_ONE_MAX = IB_ONE_U * IB_ONE;

template <int K>
__device__ inline void one_block_sums(double (&v)[K], double (*sh)[IB_ONE / 64]) {
#pragma unroll
  for (int q = 0; q < K; ++q) {
#pragma unroll
    for (int h = 32; h > 0; h >>= 1) v[q] += __shfl_xor(v[q], h);
    if ((threadIdx.x & 63) == 0) sh[q][threadIdx.x >> 6] = v[q];
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < K; ++q) {
    v[q] = 0.0;
    for (int w = 0; w < IB_ONE / 64; ++w) v[q] += sh[q][w];
  }
  __syncthreads();
}

__global__ void __launch_bounds__(IB_ONE) ib_iterate_kernel(ListGeom g, CgBufs cg,
                                                            const double* __restrict__ z,
                                                            double tol2, int maxiter) {
  __shared__ double sh[3][IB_ONE / 64];
  __shared__ double sc[CG_NSCAL];
  if (cg.scal[CG_DONE] != 0.0) return;
  if (threadIdx.x < CG_NSCAL) sc[threadIdx.x] = cg.scal[threadIdx.x];
  double v[3] = {0.0, 0.0, 0.0};
  list_az<IB_ONE_U>(g, cg, z, threadIdx.x, IB_ONE, v);
  one_block_sums<3>(v, sh);
  if (threadIdx.x == 0) scalars(sc, v[0], v[1], v[2]);
  __syncthreads();
  const double alpha = sc[CG_ALPHA], beta = sc[CG_BETA];
  double r2[1] = {list_step<IB_ONE_U>(cg, threadIdx.x, IB_ONE, alpha, beta)};
  one_block_sums<1>(r2, sh);
  if (threadIdx.x == 0) stop_test(sc, r2[0], tol2, maxiter);
  __syncthreads();
  if (threadIdx.x < CG_NSCAL) cg.scal[threadIdx.x] = sc[threadIdx.x];
}

// The gauge: mean of p over the fluid cells, then the shift.
__global__ void __launch_bounds__(IB_NT) ib_mean_kernel(long N, const uint8_t* __restrict__ bits,
                                                        CgBufs cg, const double* __restrict__ p,
                                                        double nfluid) {
  __shared__ double sh[1][IB_NT];
  double v[1] = {0.0};
  for (long n = blockIdx.x * (long)IB_NT + threadIdx.x; n < N; n += (long)gridDim.x * IB_NT)
    v[0] += (bits[n] & IB_FLUID) ? p[n] : 0.0;
  if (grid_sums<1>(v, cg.part, cg.ticket, sh) && threadIdx.x == 0) cg.scal[CG_MEAN] = v[0] / nfluid;
}

__global__ void __launch_bounds__(IB_NT) ib_shift_kernel(long N, const uint8_t* __restrict__ bits,
                                                         CgBufs cg, double* __restrict__ p) {
  const double mean = cg.scal[CG_MEAN];
  for (long n = blockIdx.x * (long)IB_NT + threadIdx.x; n < N; n += (long)gridDim.x * IB_NT)
    p[n] = (bits[n] & IB_FLUID) ? p[n] - mean : 0.0;
}

// Velocities on closed faces set to zero (interior faces; halos refilled by
// the caller).  Wall faces of w are zero already.
template <class T>
__global__ void __launch_bounds__(IB_NT) ib_mask_velocity_kernel(Dims d, T* __restrict__ u,
                                                                 T* __restrict__ v,
                                                                 T* __restrict__ w,
                                                                 const T* __restrict__ mask) {
  const long N = (long)d.nx * d.ny * d.nz;
  for (long n = blockIdx.x * (long)IB_NT + threadIdx.x; n < N; n += (long)gridDim.x * IB_NT) {
    int i, j, k;
    cell_of(d, n, i, j, k);
    const long c = pidx(d, i, j, k);
    const T m0 = mask[c];
    u[c] = u[c] * (m0 * mask[c - 1]);
    v[c] = v[c] * (m0 * mask[c - d.sy]);
    if (!d.zb || k > 0) w[c] = w[c] * (m0 * mask[c - d.sz]);
  }
}

int ib_grid(long N) {
  const long b = (N + IB_NT - 1) / IB_NT;
  return (int)(b < IB_LPART ? b : IB_LPART);
}

}  // namespace

template <class T>
hipError_t launch_ib_rhs(const Dims& d, const T* u, const T* v, const T* w,
                         const uint8_t* bits, double inv_dt, double rdx, double rdy, double rdz,
                         const CgBufs& cg, hipStream_t s) {
  hipLaunchKernelGGL(ib_rhs_kernel<T>, dim3(IB_NPART), dim3(IB_NT), 0, s, d, u, v, w, bits,
                     inv_dt, rdx, rdy, rdz, cg);
  return hipGetLastError();
}

// One entry per thread up to IB_LISTWG workgroups, beyond that IB_LISTU entries at a
// time.  Every workgroup of a reducing kernel releases its sums device-wide at
// the ticket, which is what more workgroups cost: 128^3 steps over scattered cells
// with 1024, 512, 256 and 128 workgroups: 5 % of the cells immersed (a list of
// 0.5 million) 12.0, 9.3, 8.0, 7.9 ms, 15 % (1 million) 20.0, 15.3, 13.7, 14.2 ms;
// a 256^3 seamount (105 thousand) 9.18, -, 9.14, 9.10 ms.  With 128 and one entry
// at a time 15 % took 16.2 ms, with two 14.4.
constexpr int IB_LISTWG = 128, IB_LISTU = 4;
static_assert(IB_LISTWG <= IB_LPART, "room for the partial sums");
static int list_grid(const CgBufs& cg) {
  return std::max(1, std::min((cg.n + IB_NT - 1) / IB_NT, IB_LISTWG));
}
static bool batched(const CgBufs& cg) { return cg.n > IB_LISTWG * IB_NT; }

hipError_t launch_ib_start(const Dims& d, const uint8_t* bits, double rdx2, double rdy2,
                           double rdz2, const CgBufs& cg, const double* z, double tol2,
                           hipStream_t s) {
  const ListGeom g{d, bits, rdx2, rdy2, rdz2};
  hipLaunchKernelGGL(batched(cg) ? ib_start_kernel<IB_LISTU> : ib_start_kernel<1>, dim3(list_grid(cg)),
                     dim3(IB_NT), 0, s, g, cg, z, tol2);
  return hipGetLastError();
}

hipError_t launch_ib_iterate(const Dims& d, const uint8_t* bits, double rdx2, double rdy2,
                             double rdz2, const CgBufs& cg, const double* z, double tol2,
                             int maxiter, hipStream_t s) {
  const ListGeom g{d, bits, rdx2, rdy2, rdz2};
  if (cg.n <= IB_ONE_MAX) {
    hipLaunchKernelGGL(ib_iterate_kernel, dim3(1), dim3(IB_ONE), 0, s, g, cg, z, tol2, maxiter);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(batched(cg) ? ib_az_kernel<IB_LISTU> : ib_az_kernel<1>, dim3(list_grid(cg)),
                     dim3(IB_NT), 0, s, g, cg, z);
  hipLaunchKernelGGL(batched(cg) ? ib_step_kernel<IB_LISTU> : ib_step_kernel<1>, dim3(list_grid(cg)),
                     dim3(IB_NT), 0, s, cg, tol2, maxiter);
  return hipGetLastError();
}

hipError_t launch_ib_gauge(const Dims& d, const uint8_t* bits, const CgBufs& cg, double* p,
                           double nfluid, hipStream_t s) {
  const long N = (long)d.nx * d.ny * d.nz;
  hipLaunchKernelGGL(ib_mean_kernel, dim3(ib_grid(N)), dim3(IB_NT), 0, s, N, bits, cg, p, nfluid);
  hipLaunchKernelGGL(ib_shift_kernel, dim3(ib_grid(N)), dim3(IB_NT), 0, s, N, bits, cg, p);
  return hipGetLastError();
}

template <class T>
hipError_t launch_ib_mask_velocity(const Dims& d, T* u, T* v, T* w, const T* mask,
                                   hipStream_t s) {
  hipLaunchKernelGGL(ib_mask_velocity_kernel<T>, dim3(ib_grid((long)d.nx * d.ny * d.nz)),
                     dim3(IB_NT), 0, s, d, u, v, w, mask);
  return hipGetLastError();
}

#define OC_IB_INST(T)                                                                        \
  template hipError_t launch_ib_rhs<T>(const Dims&, const T*, const T*, const T*,             \
                                       const uint8_t*, double, double, double, double,        \
                                       const CgBufs&, hipStream_t);                           \
  template hipError_t launch_ib_mask_velocity<T>(const Dims&, T*, T*, T*, const T*,           \
                                                 hipStream_t);
OC_IB_INST(float)
OC_IB_INST(double)
#undef OC_IB_INST

}  // namespace oc

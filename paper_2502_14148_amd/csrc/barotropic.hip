// Split-explicit barotropic substeps of the hydrostatic model on gfx950
// (hydrostatic time-discretisation appendix of arXiv 2502.14148).
//
// A launch advances up to BHS substeps (temporal blocking, below); it reads
// (eta, U, V)^n from one buffer set and writes the state after its last
// substep to the other.  Each workgroup recomputes the substeps on a halo
// around its tile, so neither the forward (eta) and backward (U, V) halves
// of a substep nor successive substeps need a grid-wide barrier.  The
// running averages are accumulated in FP64; the last launch of a step writes
// them in place of the state, which restarts from them.  All 2D arrays are
// dense FP64, x fastest; x is periodic, y has walls (V = 0 on faces 0 and
// ny).
#include "gaddr.h"
#include "oc_internal.h"

namespace oc {

namespace {

// Up to BHS substeps in one launch.  A workgroup takes a widened tile of 64 x
// BH cells, of which the inner (64 - 2 BHS) x (BH - 2 BHS) are its own.  A wave
// holds the 64 columns of BRW rows in registers: eta, U, V and the forcing of
// a cell never go to LDS.  The x neighbours come from the next lane by DPP,
// the y neighbours from the next register, and only the row at each side of
// a wave through LDS (two 512-byte rows per wave and substep).  Each substep
// is valid on a region one cell narrower per side than the last (eta needs
// U, V one cell right/above; U, V need eta one cell left/below), so after ns
// <= BHS substeps the own tile is exact; what the edge lanes and rows compute
// from missing neighbours never reaches it.  Rows outside the domain have
// zero coefficients and hold zeros, and the wall faces V(0), V(ny) stay
// zero; x wraps periodically.
//
// Within a launch the transports are scaled, u = dtau U and v = dtau V, so that
// a substep is
//   eta -= (L_u (u_{i+1} - u_i) + L_v,{j+1} v_{j+1} - L_v,j v_j) / A,
//   u += dtau^2 GU - g H dtau^2 / dx (eta_i - eta_{i-1}),  v likewise,
// 14 FP64 operations per cell with the running averages and no division (the
// row factors and their inverses are formed once).  Bound by the
// state's 140 bytes per cell and launch and by the 2.6 cells computed per
// own cell.  On the 1440 x 560 sector a substep took 9.6 us with the tile in LDS
// (three divisions per cell, six substeps per launch), 3.8 us now.  Rows per
// wave x waves, substeps per launch, us for the 59 substeps and a correction
// of 8 levels: 4 x 16, 12: 244; 4 x 16, 10: 257; 4 x 16, 14: 297; 8 x 8, 12:
// 261; 5 x 16, 12: 260; 6 x 8, 6: 270; 3 x 16, 12: 303 (LDS tile: 577).
constexpr int BRW = 4, BNW = 16, BH = BRW * BNW, BHS = 12;
constexpr int BOX = 64 - 2 * BHS, BOY = BH - 2 * BHS;   // own tile
static_assert(BOX > 0 && BOY > 0, "an own tile is left");
struct BaroWeights {
  double w[BHS];
};

// x of the next (previous) lane; 0 past the wave's end
template <int CTRL>
__device__ inline double lane_shift(double x) {
  const unsigned long long v = __builtin_bit_cast(unsigned long long, x);
  const unsigned lo = __builtin_amdgcn_update_dpp(0u, (unsigned)v, CTRL, 0xf, 0xf, true);
  const unsigned hi = __builtin_amdgcn_update_dpp(0u, (unsigned)(v >> 32), CTRL, 0xf, 0xf, true);
  return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}
__device__ inline double lane_next(double x) { return lane_shift<0x130>(x); }   // wave_shl:1
__device__ inline double lane_prev(double x) { return lane_shift<0x138>(x); }   // wave_shr:1

__global__ void __launch_bounds__(64 * BNW) baro_multi_kernel(BaroBufs b, double dtau, double gH,
                                                              BaroWeights wts, int ns) {
  __shared__ double vrow[BNW][64], erow[BNW][64];   // a wave's first row of v, last of e
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int gx = (int)blockIdx.x * BOX - BHS + lane;
  int gi = gx % b.nx;
  if (gi < 0) gi += b.nx;
  const int j0 = (int)blockIdx.y * BOY - BHS + wave * BRW;   // the wave's first row
  const double K = gH * dtau * dtau, dtau2 = dtau * dtau;
  double e[BRW], u[BRW], v[BRW], gu[BRW], gv[BRW], se[BRW], su[BRW], sv[BRW];
  double lv[BRW + 1], ra[BRW], kx[BRW], ky[BRW];   // uniform
  lv[BRW] = b.len_v[min(max(j0 + BRW, 0), b.ny)];
#pragma unroll
  for (int r = 0; r < BRW; ++r) {
    const int gj = j0 + r;
    const bool in = gj >= 0 && gj < b.ny, vin = gj > 0 && gj < b.ny;   // uniform
    const int jc = min(max(gj, 0), b.ny - 1);
    lv[r] = b.len_v[jc];
    ra[r] = in ? b.rarea[jc] : 0.0;
    kx[r] = in ? K * b.rdx[jc] : 0.0;
    ky[r] = vin ? K * b.rdy : 0.0;
    const long c = (long)jc * b.nx + gi;
    e[r] = in ? b.eta[c] : 0.0;
    u[r] = in ? b.U[c] : 0.0;
    gu[r] = in ? b.GU[c] : 0.0;
    v[r] = vin ? b.V[c] : 0.0;
    gv[r] = vin ? b.GV[c] : 0.0;
    se[r] = su[r] = sv[r] = 0.0;
  }
#pragma unroll
  for (int r = 0; r < BRW; ++r) {
    u[r] *= dtau;
    v[r] *= dtau;
    gu[r] *= dtau2;
    gv[r] *= dtau2;
  }
  vrow[wave][lane] = v[0];
  __syncthreads();
  for (int s = 0; s < ns; ++s) {
    const double vtop = wave + 1 < BNW ? vrow[wave + 1][lane] : 0.0;
    const double wn = wts.w[s];
#pragma unroll
    for (int r = 0; r < BRW; ++r) {
      const double v1 = r + 1 < BRW ? v[r + 1] : vtop;
      double f = b.len_u * (lane_next(u[r]) - u[r]);
      f = fma(lv[r + 1], v1, f);
      f = fma(-lv[r], v[r], f);
      e[r] = fma(-ra[r], f, e[r]);
      se[r] = fma(wn, e[r], se[r]);
    }
    erow[wave][lane] = e[BRW - 1];
    __syncthreads();
    const double ebot = wave > 0 ? erow[wave - 1][lane] : 0.0;
#pragma unroll
    for (int r = 0; r < BRW; ++r) {
      const double e1 = r > 0 ? e[r - 1] : ebot;
      u[r] = fma(-kx[r], e[r] - lane_prev(e[r]), u[r]) + gu[r];
      v[r] = fma(-ky[r], e[r] - e1, v[r]) + gv[r];
      su[r] = fma(wn, u[r], su[r]);
      sv[r] = fma(wn, v[r], sv[r]);
    }
    vrow[wave][lane] = v[0];
    __syncthreads();
  }
  // the own cells (x: a tile may reach past the last column)
  if (lane < BHS || lane >= BHS + BOX || gx >= b.nx) return;
  const double rt = 1.0 / dtau;
#pragma unroll
  for (int r = 0; r < BRW; ++r) {
    const int gj = j0 + r, ty = wave * BRW + r;
    if (ty < BHS || ty >= BHS + BOY || gj >= b.ny) continue;
    const long c = (long)gj * b.nx + gx;
    double ea = se[r], ua = su[r] * rt, va = sv[r] * rt;
    if (!b.first) {
      ea += b.etab[c];
      ua += b.Ub[c];
      va += b.Vb[c];
    }
    if (b.last) {
      b.eta1[c] = ea;
      b.U1[c] = ua;
      b.V1[c] = va;
      if (gj == b.ny - 1) b.V1[c + b.nx] = 0.0;   // the northern wall
    } else {
      b.eta1[c] = e[r];
      b.U1[c] = u[r] * rt;
      b.V1[c] = v[r] * rt;
      b.etab[c] = ea;
      b.Ub[c] = ua;
      b.Vb[c] = va;
    }
  }
}

// u <- u + (Ubar - dz sum_k u) / H on every column of u (rows 0..ny-1) and v
// (the interior faces 1..ny-1), z = 0 and 1 of the grid.  Levels are fetched
// CKB at a time so that their loads are in flight together; the second read
// of a column comes from the caches.  Bound by HBM (16 bytes per cell of u and
// v).  1440 x 560 x 50 FP32: 223 us in two launches of 64-column groups with
// 64-bit addresses (a group's rows share a cache line with the next group's,
// on another XCD), 172 us with 256 columns and uniform level bases; columns
// kept in registers between the passes measured 166 us, not worth a kernel
// per column height.
template <class T>
struct CorrectArgs {
  T* f[2];
  const double* bar[2];
};
template <class T>
__global__ void __launch_bounds__(256) baro_correct_kernel(Dims d, CorrectArgs<T> a, double dz,
                                                           double inv_h) {
  const int i = blockIdx.x * 256 + threadIdx.x, z = blockIdx.z, j = z + (int)blockIdx.y;
  if (i >= d.nx || j >= d.ny) return;
  // the column's byte offset within a level; levels are a uniform base apart
  const unsigned off = (unsigned)pidx(d, i, j, -d.h) * (unsigned)sizeof(T);
  T* const f = a.f[z] + (long)d.h * d.sz;
  const double bar = glb(a.bar[z])[(long)j * d.nx + i];
  constexpr int CKB = 10;
  double sum = 0.0;
  for (int k0 = 0; k0 < d.nz; k0 += CKB) {
    T x[CKB];
#pragma unroll
    for (int q = 0; q < CKB; ++q)
      x[q] = at(uniform_ptr(f + (long)min(k0 + q, d.nz - 1) * d.sz), off);
#pragma unroll
    for (int q = 0; q < CKB; ++q)
      if (k0 + q < d.nz) sum += (double)x[q];
  }
  const double corr = (bar - dz * sum) * inv_h;
  for (int k0 = 0; k0 < d.nz; k0 += CKB) {
    T x[CKB];
#pragma unroll
    for (int q = 0; q < CKB; ++q)
      x[q] = at(uniform_ptr(f + (long)min(k0 + q, d.nz - 1) * d.sz), off);
#pragma unroll
    for (int q = 0; q < CKB; ++q)
      if (k0 + q < d.nz) at(uniform_ptr(f + (long)(k0 + q) * d.sz), off) = (T)((double)x[q] + corr);
  }
}

__global__ void baro_fill_kernel(double* a, double v, long n) {
  const long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (t < n) a[t] = v;
}

}  // namespace

hipError_t launch_baro_fill(double* a, double v, long n, hipStream_t s) {
  hipLaunchKernelGGL(baro_fill_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, a, v, n);
  return hipGetLastError();
}

int baro_max_fused() { return BHS; }

hipError_t launch_baro_substeps(const BaroBufs& b, double dtau, double gH, const double* wn,
                                int ns, hipStream_t s) {
  if (ns < 1 || ns > BHS) return hipErrorInvalidValue;
  BaroWeights w{};
  for (int q = 0; q < ns; ++q) w.w[q] = wn[q];
  dim3 grid((b.nx + BOX - 1) / BOX, (b.ny + BOY - 1) / BOY);
  hipLaunchKernelGGL(baro_multi_kernel, grid, dim3(64 * BNW), 0, s, b, dtau, gH, w, ns);
  return hipGetLastError();
}

template <class T>
hipError_t launch_baro_correct(const Dims& d, T* u, T* v, const double* ubar, const double* vbar,
                               double dz, double depth, hipStream_t s) {
  const dim3 grid((d.nx + 255) / 256, d.ny, 2), nt(256);
  const CorrectArgs<T> a{{u, v}, {ubar, vbar}};
  hipLaunchKernelGGL(baro_correct_kernel<T>, grid, nt, 0, s, d, a, dz, 1.0 / depth);
  return hipGetLastError();
}

template hipError_t launch_baro_correct<float>(const Dims&, float*, float*, const double*,
                                               const double*, double, double, hipStream_t);
template hipError_t launch_baro_correct<double>(const Dims&, double*, double*, const double*,
                                                const double*, double, double, hipStream_t);

}  // namespace oc

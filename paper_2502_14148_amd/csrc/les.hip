// Eddy-viscosity LES closures on gfx950 (closure paragraph of the
// nonhydrostatic model section of arXiv 2502.14148: the closure flux
// divergence d_m tau_nm with the SmagorinskyLilly eddy viscosity; the
// AnisotropicMinimumDissipation closure named beside it).
//
//   Smagorinsky-Lilly: nu_e = (C_s Delta)^2 |S| sqrt(max(0, 1 - C_b N^2/|S|^2)),
//     |S|^2 = 2 S_ij S_ij, Delta = (dx dy dzc)^(1/3), kappa_e = nu_e / Pr;
//   AMD (Rozema et al. 2015, Vreugdenhil & Taylor 2018):
//     nu_e = max(0, -C sum_k Delta_k^2 d_k u_i d_k u_j S_ij / |grad u|^2),
//     kappa_e = max(0, -C sum_k Delta_k^2 d_k u_i d_k c d_i c / |grad c|^2).
//
// Two kernels per substage; each workgroup owns a column tile and marches
// up a chunk of levels, keeping four levels (k-1, k, k+1 in use, k+2 on its
// way; with a one-cell halo) of every field it reads in LDS rings, so each
// value is fetched from memory once per tile instead of once per neighbour
// that reads it.  The buffer unit copies level k+2 into its slot while level k
// is computed (load-to-LDS), with one barrier per level:
//   1. the eddy viscosity (and AMD's per-tracer diffusivity) at the centres
//      from the resolved gradients: diagonal strain at the centre, the
//      off-diagonal components on the twelve surrounding edges (squared then
//      averaged for |S|, averaged for AMD's gradient tensor), N^2 from the
//      two z faces; written with their halo images;
//   2. the closure tendencies d_j(2 nu_e S_ij) of u, v, w (stresses at their
//      C-grid locations, edge viscosities the mean of four centres) and
//      d_i(kappa_e d_i c) of the tracers (face diffusivities the mean of two
//      centres); no flux through the walls.  The tendency kernel adds them.
// The kernels are instantiated for the number of fields they read, which sets
// their LDS and with it the resident workgroups, and the compiler keeps every
// ring offset an immediate.  What bounds them: vector issue together with the
// waits of a level.  At 256x256x128 FP32 (2 tracers, Smagorinsky-Lilly) the
// viscosity pass issues 198 vector and 28 LDS instructions per cell and wave
// (42 us at one per cycle; 39 us of memory traffic at 5.2 TB/s) and takes 80 us,
// the fluxes 234 and 42 (50 us; 71 us of traffic) and take 116 us.  With the
// levels brought through registers into a three-level ring, two barriers per
// level and field loops up to the largest tracer count the same passes took
// 100 and 166 us; one substage of both (with the launches between), before and
// now: Smagorinsky-Lilly 276 -> 200 us, AMD 312 -> 246 us, 64^3 75 -> 15.5 us.
#include <algorithm>

#include "oc_internal.h"
#include "tendency_tile.h"

namespace oc {

namespace {

// Tiles: TX x TY columns, chunks of kc levels.  Workgroups are dealt
// round-robin to the 8 XCDs; renumbering them gives each XCD a contiguous
// run of tiles, so the halo rows shared by neighbouring tiles stay in one L2.
struct LesTile {
  int i0, j0, kb, ke;
};

__device__ inline LesTile les_tile(const Dims& d, int tx, int ty, int kc) {
  const unsigned nb = gridDim.x;
  unsigned b = blockIdx.x;
  if (nb % 8 == 0) b = (b % 8) * (nb / 8) + b / 8;
  const int nbx = d.nx / tx, nby = d.ny / ty;
  LesTile t;
  t.i0 = (int)(b % nbx) * tx;
  t.j0 = (int)((b / nbx) % nby) * ty;
  t.kb = (int)(b / (nbx * nby)) * kc;
  t.ke = min(t.kb + kc, d.nz);
  return t;
}

// Values of field f around the own cell, read from the LDS rings: at[dk + 1]
// is the position (-1, -1) of the own cell's neighbourhood in level k + dk of
// field 0, so that every access is a compile-time offset from it.
template <class T, int PX, int PLP>
struct Ring {
  const T* S;      // ring planes of all fields, 4 PLP each
  int at[3];
  __device__ T operator()(int f, int di, int dj, int dk) const {
    return S[at[dk + 1] + f * 4 * PLP + (dj + 1) * PX + di + 1];
  }
};

// The z-march of a tile over NF fields: cell(k, ring, out) computes the NO
// results of the own cell of every level, with the rings holding levels k-1,
// k, k+1, and put(i, j, k, out) stores them.  The stores of a level are issued
// at the start of the next one: the wait for the copies at a level's end is a
// wait for every memory operation, and this way the stores have had a level's
// time as well.
template <class T, int TX, int TY, int NF, int NO, class Cell, class Put>
__device__ inline void les_march(const Dims& d, const T* const (&fld)[NF], int kc, Cell cell,
                                 Put put) {
  constexpr int PX = TX + 2, PY = TY + 2, NT = TX * TY, ES = (int)sizeof(T);
  using PC = tz::PlaneCopy<PX, PY, NT, ES>;
  constexpr int PLP = PC::PLP;
  __shared__ T S[NF * 4 * PLP];
  const LesTile t = les_tile(d, TX, TY, kc);
  const int tid = threadIdx.x, tx = tid % TX, ty = tid / TX;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  // per-lane byte offsets of the copied plane dwords from the tile corner
  const int sy = (int)d.sy;
  auto dword_off = [&](int j) -> uint32_t {
    if (j > PC::PLD - 1) j = PC::PLD - 1;
    const int e = j / PC::DPE, half = j - e * PC::DPE;
    const int ly = e / PX, lx = e - ly * PX;
    return (uint32_t)((ly * sy + lx) * ES + half * 4);
  };
  uint32_t goff[PC::NR + PC::MAXC];
#pragma unroll
  for (int r = 0; r < PC::NR; ++r) goff[r] = dword_off(r * NT + tid);
#pragma unroll
  for (int c = 0; c < PC::MAXC; ++c)
    goff[PC::NR + c] = dword_off(PC::NR * NT + (wave + c * PC::NWV) * 64 + lane);
  const uint32_t corner = (uint32_t)(((t.j0 - 1 + d.h) * sy + (t.i0 - 1 + d.h)) * ES);
  const uint32_t lvb = (uint32_t)d.sz * ES;
  auto copy_level = [&](int kk) {
    const uint32_t so = (uint32_t)(kk + d.h) * lvb + corner;
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      const __amdgpu_buffer_rsrc_t rs = tz::make_rsrc((const char*)fld[f]);
      T* dst = S + (f * 4 + (kk & 3)) * PLP;
#pragma unroll
      for (int r = 0; r < PC::NR; ++r)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (void*)(dst + (r * NT + wave * 64) / PC::DPE),
                                                 4, goff[r], so, 0, 0);
#pragma unroll
      for (int c = 0; c < PC::MAXC; ++c) {
        const int ch = wave + c * PC::NWV;
        if (ch < PC::NCH)
          __builtin_amdgcn_raw_ptr_buffer_load_lds(
              rs, (void*)(dst + (PC::NR * NT + ch * 64) / PC::DPE), 4, goff[PC::NR + c], so, 0, 0);
      }
    }
  };
  copy_level(t.kb - 1);
  copy_level(t.kb);
  copy_level(t.kb + 1);
  tz::wait_vm();
  __syncthreads();
  Ring<T, PX, PLP> r;
  r.S = S;
  const int L = ty * PX + tx;
  T out[NO];
  for (int k = t.kb; k < t.ke; ++k) {
    if (k > t.kb) put(t.i0 + tx, t.j0 + ty, k - 1, out);
    // level k - 2 is read by no one since the last barrier
    if (k + 1 < t.ke) copy_level(k + 2);
    r.at[0] = tz::opaque(((k + 3) & 3) * PLP + L);
    r.at[1] = tz::opaque((k & 3) * PLP + L);
    r.at[2] = tz::opaque(((k + 1) & 3) * PLP + L);
    cell(k, r, out);
    tz::wait_vm();      // this wave's copies have landed
    __syncthreads();
  }
  put(t.i0 + tx, t.j0 + ty, t.ke - 1, out);
}

// Ring fields of the viscosity pass: 0 u, 1 v, 2 w, then the tracers
// (Smagorinsky-Lilly: T and S when buoyant; AMD: every tracer).
template <class T, int KIND, int NTR, class R>
__device__ inline void les_viscosity_cell(const Dims& d, const LesArgs<T>& a, int k, const R& r,
                                          T* out) {
  auto U = [&](int di, int dj, int dk) { return r(0, di, dj, dk); };
  auto V = [&](int di, int dj, int dk) { return r(1, di, dj, dk); };
  auto W = [&](int di, int dj, int dk) { return r(2, di, dj, dk); };
  const T rdx = a.rdx, rdy = a.rdy, rzc = glb(a.rdzc)[k];
  const T rzf0 = glb(a.rdzf)[k], rzf1 = glb(a.rdzf)[k + 1];
  const bool wall0 = d.zb && k == 0, wall1 = d.zb && k + 1 == d.nz;
  const T ux = (U(1, 0, 0) - U(0, 0, 0)) * rdx;
  const T vy = (V(0, 1, 0) - V(0, 0, 0)) * rdy;
  const T wz = (W(0, 0, 1) - W(0, 0, 0)) * rzc;
  // off-diagonal gradients on the edges around the centre
  T uy[2][2], vx[2][2], uz[2][2], wx[2][2], vz[2][2], wy[2][2];
#pragma unroll
  for (int p = 0; p < 2; ++p)
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      // (F,F,C): x face i + p, y face j + q
      uy[p][q] = (U(p, q, 0) - U(p, q - 1, 0)) * rdy;
      vx[p][q] = (V(p, q, 0) - V(p - 1, q, 0)) * rdx;
      // (F,C,F): x face i + p, z face k + q; (C,F,F): y face j + p, z face k + q
      const bool wl = q ? wall1 : wall0;
      const T rzf = q ? rzf1 : rzf0;
      uz[p][q] = wl ? T(0) : (U(p, 0, q) - U(p, 0, q - 1)) * rzf;
      wx[p][q] = wl ? T(0) : (W(p, 0, q) - W(p - 1, 0, q)) * rdx;
      vz[p][q] = wl ? T(0) : (V(0, p, q) - V(0, p, q - 1)) * rzf;
      wy[p][q] = wl ? T(0) : (W(0, p, q) - W(0, p - 1, q)) * rdy;
    }
  T nu;
  if (KIND == OC_LES_SMAGORINSKY) {
    T sxy2 = 0, sxz2 = 0, syz2 = 0;
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const T e1 = T(0.5) * (uy[p][q] + vx[p][q]);
        const T e2 = T(0.5) * (uz[p][q] + wx[p][q]);
        const T e3 = T(0.5) * (vz[p][q] + wy[p][q]);
        sxy2 += e1 * e1;
        sxz2 += e2 * e2;
        syz2 += e3 * e3;
      }
    const T s2 = T(2) * (ux * ux + vy * vy + wz * wz) + (sxy2 + sxz2 + syz2);  // 4 x (1/4) sums
    T n2 = T(0);
    if (NTR == 2) {   // buoyant
      auto b = [&](int dk) {
        return a.g_alpha * (r(3, 0, 0, dk) - a.t_ref) - a.g_beta * (r(4, 0, 0, dk) - a.s_ref);
      };
      const T b0 = b(0);
      const T g0 = wall0 ? T(0) : (b0 - b(-1)) * rzf0;
      const T g1 = wall1 ? T(0) : (b(1) - b0) * rzf1;
      n2 = T(0.5) * (g0 + g1);
    }
    T fac = T(0);
    if (s2 > T(0)) fac = fmax(T(0), T(1) - a.cb * n2 / s2);
    nu = glb(a.delta2)[k] * sqrt(s2) * sqrt(fac);
  } else {
    // AMD: the gradient tensor at the centre (edge values averaged)
    T G[3][3];
    G[0][0] = ux;
    G[1][1] = vy;
    G[2][2] = wz;
    G[0][1] = T(0.25) * (uy[0][0] + uy[0][1] + uy[1][0] + uy[1][1]);
    G[1][0] = T(0.25) * (vx[0][0] + vx[0][1] + vx[1][0] + vx[1][1]);
    G[0][2] = T(0.25) * (uz[0][0] + uz[0][1] + uz[1][0] + uz[1][1]);
    G[2][0] = T(0.25) * (wx[0][0] + wx[0][1] + wx[1][0] + wx[1][1]);
    G[1][2] = T(0.25) * (vz[0][0] + vz[0][1] + vz[1][0] + vz[1][1]);
    G[2][1] = T(0.25) * (wy[0][0] + wy[0][1] + wy[1][0] + wy[1][1]);
    const T D2[3] = {T(1) / (rdx * rdx), T(1) / (rdy * rdy), T(1) / (rzc * rzc)};
    T num = 0, den = 0;
#pragma unroll
    for (int kk = 0; kk < 3; ++kk)
#pragma unroll
      for (int ii = 0; ii < 3; ++ii) {
        den += G[ii][kk] * G[ii][kk];
#pragma unroll
        for (int jj = 0; jj < 3; ++jj)
          num += D2[kk] * G[ii][kk] * G[jj][kk] * (T(0.5) * (G[ii][jj] + G[jj][ii]));
      }
    nu = (den > T(0)) ? fmax(T(0), -a.camd * num / den) : T(0);
    // per-tracer diffusivities
#pragma unroll
    for (int q = 0; q < NTR; ++q) {
      auto C = [&](int di, int dj, int dk) { return r(3 + q, di, dj, dk); };
      const T c0 = C(0, 0, 0);
      const T gx = T(0.5) * (C(1, 0, 0) - C(-1, 0, 0)) * rdx;
      const T gy = T(0.5) * (C(0, 1, 0) - C(0, -1, 0)) * rdy;
      const T gz0 = wall0 ? T(0) : (c0 - C(0, 0, -1)) * rzf0;
      const T gz1 = wall1 ? T(0) : (C(0, 0, 1) - c0) * rzf1;
      const T gc[3] = {gx, gy, T(0.5) * (gz0 + gz1)};
      T kn = 0;
#pragma unroll
      for (int kk = 0; kk < 3; ++kk)
#pragma unroll
        for (int ii = 0; ii < 3; ++ii) kn += D2[kk] * G[ii][kk] * gc[kk] * gc[ii];
      const T kd = gc[0] * gc[0] + gc[1] * gc[1] + gc[2] * gc[2];
      const T kap = (kd > T(0)) ? fmax(T(0), -a.camd * kn / kd) : T(0);
      out[1 + q] = kap;
    }
  }
  out[0] = nu;
}

// NTR: AMD: the tracers; Smagorinsky-Lilly: 2 (T and S) when buoyant, else 0.
template <class T, int KIND, int NTR, int TX, int TY>
__global__ void __launch_bounds__(TX * TY) les_viscosity_kernel(Dims d, LesArgs<T> a, int kc) {
  const T* fld[3 + NTR];
  fld[0] = a.u;
  fld[1] = a.v;
  fld[2] = a.w;
#pragma unroll
  for (int q = 0; q < NTR; ++q)
    fld[3 + q] = KIND == OC_LES_SMAGORINSKY ? (q ? a.c1 : a.c0) : a.tr[q];
  constexpr int NO = KIND == OC_LES_AMD ? 1 + NTR : 1;   // nu, AMD's kappas
  les_march<T, TX, TY, 3 + NTR, NO>(
      d, fld, kc,
      [&](int k, const auto& r, T* out) { les_viscosity_cell<T, KIND, NTR>(d, a, k, r, out); },
      [&](int i, int j, int k, const T* out) {
        store_with_images(a.nu, d, i, j, k, out[0], false);
#pragma unroll
        for (int q = 1; q < NO; ++q) store_with_images(a.kap[q - 1], d, i, j, k, out[q], false);
      });
}

// The closure tendencies of the cell index (i, j, k): u at x face i, v at y
// face j, w at z face k, tracers at the centre.  Ring fields: 0 u, 1 v, 2 w,
// 3 nu, 4 + q tracer q, 4 + NTR + q AMD's kappa of tracer q.
template <class T, int NTR, bool AMD, class R>
__device__ inline void les_flux_cell(const Dims& d, const LesArgs<T>& a, int k, const R& r,
                                     T* out) {
  auto U = [&](int di, int dj, int dk) { return r(0, di, dj, dk); };
  auto V = [&](int di, int dj, int dk) { return r(1, di, dj, dk); };
  auto W = [&](int di, int dj, int dk) { return r(2, di, dj, dk); };
  auto N = [&](int di, int dj, int dk) { return r(3, di, dj, dk); };
  const T rdx = a.rdx, rdy = a.rdy;
  const T rzc = glb(a.rdzc)[k], rzf0 = glb(a.rdzf)[k], rzf1 = glb(a.rdzf)[k + 1];
  const bool wall0 = d.zb && k == 0, wall1 = d.zb && k + 1 == d.nz;
  // edge viscosities: means of the four surrounding centres
  auto n_ffc = [&](int p, int q) {  // x face i + p, y face j + q
    return T(0.25) * (N(p - 1, q - 1, 0) + N(p, q - 1, 0) + N(p - 1, q, 0) + N(p, q, 0));
  };
  auto n_fcf = [&](int p, int q) {  // x face i + p, z face k + q
    return T(0.25) * (N(p - 1, 0, q - 1) + N(p, 0, q - 1) + N(p - 1, 0, q) + N(p, 0, q));
  };
  auto n_cff = [&](int p, int q) {  // y face j + p, z face k + q
    return T(0.25) * (N(0, p - 1, q - 1) + N(0, p, q - 1) + N(0, p - 1, q) + N(0, p, q));
  };
  // stresses 2 nu S at their locations
  auto txy = [&](int p, int q) {
    return n_ffc(p, q) * ((U(p, q, 0) - U(p, q - 1, 0)) * rdy + (V(p, q, 0) - V(p - 1, q, 0)) * rdx);
  };
  auto txz = [&](int p, int q) {
    if (q ? wall1 : wall0) return T(0);
    const T rzf = q ? rzf1 : rzf0;
    return n_fcf(p, q) * ((U(p, 0, q) - U(p, 0, q - 1)) * rzf + (W(p, 0, q) - W(p - 1, 0, q)) * rdx);
  };
  auto tyz = [&](int p, int q) {
    if (q ? wall1 : wall0) return T(0);
    const T rzf = q ? rzf1 : rzf0;
    return n_cff(p, q) * ((V(0, p, q) - V(0, p, q - 1)) * rzf + (W(0, p, q) - W(0, p - 1, q)) * rdy);
  };
  // u at x face i: txx at the centres i-1, i
  {
    const T t0 = T(2) * N(-1, 0, 0) * (U(0, 0, 0) - U(-1, 0, 0)) * rdx;
    const T t1 = T(2) * N(0, 0, 0) * (U(1, 0, 0) - U(0, 0, 0)) * rdx;
    const T g = (t1 - t0) * rdx + (txy(0, 1) - txy(0, 0)) * rdy + (txz(0, 1) - txz(0, 0)) * rzc;
    out[0] = g;
  }
  // v at y face j
  {
    const T t0 = T(2) * N(0, -1, 0) * (V(0, 0, 0) - V(0, -1, 0)) * rdy;
    const T t1 = T(2) * N(0, 0, 0) * (V(0, 1, 0) - V(0, 0, 0)) * rdy;
    const T g = (txy(1, 0) - txy(0, 0)) * rdx + (t1 - t0) * rdy + (tyz(0, 1) - tyz(0, 0)) * rzc;
    out[1] = g;
  }
  // w at z face k (the w cell spans the centres k-1, k: thickness dzf_k);
  // txz and tyz on face k are the q = 0 stresses of the edges with x face
  // i, i+1 (y face j, j+1)
  {
    T g = T(0);
    if (!wall0) {
      const T t0 = T(2) * N(0, 0, -1) * (W(0, 0, 0) - W(0, 0, -1)) * glb(a.rdzc)[k - 1];
      const T t1 = T(2) * N(0, 0, 0) * (W(0, 0, 1) - W(0, 0, 0)) * rzc;
      g = (txz(1, 0) - txz(0, 0)) * rdx + (tyz(1, 0) - tyz(0, 0)) * rdy + (t1 - t0) * rzf0;
    }
    out[2] = g;
  }
  // tracers: d_i(kappa d_i c), face diffusivities the mean of two centres
#pragma unroll
  for (int q = 0; q < NTR; ++q) {
    const int fk = AMD ? 4 + NTR + q : 3;
    auto C = [&](int di, int dj, int dk) { return r(4 + q, di, dj, dk); };
    auto K = [&](int di, int dj, int dk) { return r(fk, di, dj, dk); };
    const T s = AMD ? T(1) : a.rpr;
    const T c0 = C(0, 0, 0), k0 = K(0, 0, 0);
    const T fxm = T(0.5) * (K(-1, 0, 0) + k0) * (c0 - C(-1, 0, 0)) * rdx;
    const T fxp = T(0.5) * (k0 + K(1, 0, 0)) * (C(1, 0, 0) - c0) * rdx;
    const T fym = T(0.5) * (K(0, -1, 0) + k0) * (c0 - C(0, -1, 0)) * rdy;
    const T fyp = T(0.5) * (k0 + K(0, 1, 0)) * (C(0, 1, 0) - c0) * rdy;
    const T fzm = wall0 ? T(0) : T(0.5) * (K(0, 0, -1) + k0) * (c0 - C(0, 0, -1)) * rzf0;
    const T fzp = wall1 ? T(0) : T(0.5) * (k0 + K(0, 0, 1)) * (C(0, 0, 1) - c0) * rzf1;
    out[3 + q] = s * ((fxp - fxm) * rdx + (fyp - fym) * rdy + (fzp - fzm) * rzc);
  }
}

template <class T, int NTR, bool AMD, int TX, int TY>
__global__ void __launch_bounds__(TX * TY) les_flux_kernel(Dims d, LesArgs<T> a, int kc) {
  constexpr int NF = 4 + (AMD ? 2 : 1) * NTR;
  const T* fld[NF];
  fld[0] = a.u;
  fld[1] = a.v;
  fld[2] = a.w;
  fld[3] = a.nu;
#pragma unroll
  for (int q = 0; q < NTR; ++q) {
    fld[4 + q] = a.tr[q];
    if (AMD) fld[4 + NTR + q] = a.kap[q];
  }
  les_march<T, TX, TY, NF, 3 + NTR>(
      d, fld, kc,
      [&](int k, const auto& r, T* out) { les_flux_cell<T, NTR, AMD>(d, a, k, r, out); },
      [&](int i, int j, int k, const T* out) {
        const long c = pidx(d, i, j, k);
#pragma unroll
        for (int f = 0; f < 3 + NTR; ++f) glb(a.gc[f])[c] = out[f];
      });
}

}  // namespace

template <class T, int NTR, int TX, int TY>
hipError_t launch_les_tiles(const Dims& d, const LesArgs<T>& a, int kind, hipStream_t s) {
  const int tiles = (d.nx / TX) * (d.ny / TY);
  // Levels per workgroup.  A chunk copies two levels more than it computes,
  // and a workgroup's levels run one after the other, so a chunk is as long as
  // 2048 workgroups allow (8 per CU), within 2..16.  One substage with at most
  // 8, 16 and 32 levels: 256x256x128 FP32 Smagorinsky-Lilly 201, 200, 193 us,
  // AMD (its 8 fields' rings leave 2 workgroups per CU) 248, 246, 267 us; 64^3
  // with 2 levels 15.5 us, with the fixed 16 of before 75 us.
  const int kc = std::min(d.nz, std::max(2, (int)std::min(16L, (long)d.nz * tiles / 2048)));
  const dim3 grid(tiles * ((d.nz + kc - 1) / kc)), nt(TX * TY);
  if (kind == OC_LES_SMAGORINSKY) {
    if (a.buoyancy)
      hipLaunchKernelGGL((les_viscosity_kernel<T, OC_LES_SMAGORINSKY, 2, TX, TY>), grid, nt, 0, s, d,
                         a, kc);
    else
      hipLaunchKernelGGL((les_viscosity_kernel<T, OC_LES_SMAGORINSKY, 0, TX, TY>), grid, nt, 0, s, d,
                         a, kc);
    hipLaunchKernelGGL((les_flux_kernel<T, NTR, false, TX, TY>), grid, nt, 0, s, d, a, kc);
  } else if (kind == OC_LES_AMD) {
    hipLaunchKernelGGL((les_viscosity_kernel<T, OC_LES_AMD, NTR, TX, TY>), grid, nt, 0, s, d, a, kc);
    hipLaunchKernelGGL((les_flux_kernel<T, NTR, true, TX, TY>), grid, nt, 0, s, d, a, kc);
  } else {
    return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <class T, int TX, int TY>
hipError_t launch_les_tracers(const Dims& d, const LesArgs<T>& a, int kind, hipStream_t s) {
  switch (a.ntr) {
    case 1: return launch_les_tiles<T, 1, TX, TY>(d, a, kind, s);
    case 2: return launch_les_tiles<T, 2, TX, TY>(d, a, kind, s);
    case 3: return launch_les_tiles<T, 3, TX, TY>(d, a, kind, s);
    default: return launch_les_tiles<T, 4, TX, TY>(d, a, kind, s);
  }
}

template <class T>
hipError_t launch_les(const Dims& d, const LesArgs<T>& a, int kind, hipStream_t s) {
  // a field's byte offsets take 32 bits (the model's layout ensures it)
  if (a.ntr < 1 || a.ntr > OC_MAX_TRACERS || d.h < 1 ||
      (uint64_t)padded_elems(d) * sizeof(T) > 0xFFFFFFFFull)
    return hipErrorInvalidValue;
  if (d.nx % 32 == 0 && d.ny % 8 == 0) return launch_les_tracers<T, 32, 8>(d, a, kind, s);
  if (d.nx % 8 == 0 && d.ny % 8 == 0) return launch_les_tracers<T, 8, 8>(d, a, kind, s);
  return hipErrorInvalidValue;
}

template hipError_t launch_les<float>(const Dims&, const LesArgs<float>&, int, hipStream_t);
template hipError_t launch_les<double>(const Dims&, const LesArgs<double>&, int, hipStream_t);

}  // namespace oc

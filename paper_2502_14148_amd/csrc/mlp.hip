// MLP subgrid closure on gfx950: BF16 MFMA products with FP32 accumulation.
// Inference and the in-model closure run the whole network in one kernel
// (the in-model one gathers the standardised 5x5x5 (u, v, w, b)
// neighbourhood of every cell itself); training takes three launches, with
// Adam on FP32 master weights in the last.
//
// Network: 500 -> 256 -> 256 -> 4 with exact-erf GELU.  On the device the
// input width is padded to 512 with zero weights, a multiple of the 32-deep
// MFMA k step, and the output width to 16 rows (32 as a reduction).
#include "oc_internal.h"

#include <algorithm>
#include <cmath>
#include <type_traits>

namespace oc {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// The weight copies: the 16 output rows x 32 inputs that one MFMA
// takes as an operand are one contiguous kilobyte in lane order (lane l
// holds 8 consecutive k of row l % 16, k block l / 16), the k blocks of a
// row block following each other.  A wave's operand load is then one
// coalesced 16-byte load per lane.
__host__ __device__ inline int frag_at(int n, int k, int kblocks) {
  return ((n >> 4) * kblocks + (k >> 5)) * 512 + (((k >> 3) & 3) * 16 + (n & 15)) * 8 + (k & 7);
}

__device__ void mlp_write_bf16(const MlpParams& p, int t, float w) {
  // master layout: W1 (256 x 500) | b1 | W2 (256 x 256) | b2 | W3 (4 x 256) | b3
  if (t < MLP_OFF_B1) {
    const int r = t / 500, c = t % 500;
    p.W1f[frag_at(r, c, MLP_KIN / 32)] = (__bf16)w;
  } else if (t >= MLP_OFF_W2 && t < MLP_OFF_B2) {
    const int r = (t - MLP_OFF_W2) / MLP_NH, c = (t - MLP_OFF_W2) % MLP_NH;
    p.W2f[frag_at(r, c, MLP_NH / 32)] = (__bf16)w;
    p.W2Tf[frag_at(c, r, MLP_NH / 32)] = (__bf16)w;   // transposed, for the backward pass
  } else if (t >= MLP_OFF_W3 && t < MLP_OFF_B3) {
    const int r = (t - MLP_OFF_W3) / MLP_NH, c = (t - MLP_OFF_W3) % MLP_NH;
    p.W3f[frag_at(r, c, MLP_NH / 32)] = (__bf16)w;
    p.W3Tf[frag_at(c, r, 1)] = (__bf16)w;
  }
}


namespace {

// erf(z / sqrt 2) and exp(-z^2 / 2) by Abramowitz & Stegun, formula 7.1.26
// (absolute error of erf at most 1.5e-7; evaluated in FP32 5.1e-7, and 2.9e-7 in
// the GELU derivative it serves): for x >= 0, erf x = 1 - t P(t) exp(-x^2),
// t = 1 / (1 + p x), P a quartic; erf is odd.  About a dozen full-rate
// instructions, a reciprocal and an exponential: the activation epilogues
// are the bulk of the fused kernel's vector instructions.
struct ErfGauss {
  float erf, g;
};
__device__ inline ErfGauss erf_gauss(float z) {
  const float t = __builtin_amdgcn_rcpf(fmaf(0.3275911f * 0.70710678118654752f, fabsf(z), 1.0f));
  float q = fmaf(1.061405429f, t, -1.453152027f);
  q = fmaf(q, t, 1.421413741f);
  q = fmaf(q, t, -0.284496736f);
  q = fmaf(q, t, 0.254829592f);
  const float g = __builtin_amdgcn_exp2f(z * z * (-0.5f * 1.44269504088896341f));
  return {copysignf(fmaf(-(q * t), g, 1.0f), z), g};
}
// erf(z / sqrt 2) alone by Abramowitz & Stegun, formula 7.1.28 (absolute
// error at most 3e-7): for x >= 0, erf x = 1 - (1 + a1 x + ... + a6 x^6)^-16,
// here with the 1/sqrt 2 folded into the coefficients.  One reciprocal and
// no exponential.  Evaluated in FP32 the error is 1.9e-6 (the sixteenth power
// multiplies the rounding of the reciprocal, near z = 0), that of the GELU
// 7.7e-7.  Relative to the GELU it is below the rounding to BF16 (2e-3) for
// z > -3.5; in the tail beyond, where the GELU is under 8.2e-4, it reaches 2 %
// at z = -4.5 and 10 % at -5.
__device__ inline float erf_sqrt2(float z) {
  const float az = fabsf(z);
  float q = fmaf(0.0000430638f / 8.0f, az, 0.0002765672f / 5.65685424949238f);
  q = fmaf(q, az, 0.0001520143f / 4.0f);
  q = fmaf(q, az, 0.0092705272f / 2.82842712474619f);
  q = fmaf(q, az, 0.0422820123f / 2.0f);
  q = fmaf(q, az, 0.0705230784f / 1.41421356237310f);
  float r = __builtin_amdgcn_rcpf(fmaf(q, az, 1.0f));
  r *= r;
  r *= r;
  r *= r;
  r *= r;
  return copysignf(1.0f - r, z);
}
// exact-erf GELU, z Phi(z), and its derivative
__device__ inline float gelu(float z) {
  const float h = 0.5f * z;
  return fmaf(h, erf_sqrt2(z), h);
}
__device__ inline float gelu_prime(float z) {
  const ErfGauss r = erf_gauss(z);
  return fmaf(0.5f, r.erf, 0.5f) + z * r.g * 0.39894228040143268f;
}

__global__ void refresh_bf16_kernel(MlpParams p, int n) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t < n) mlp_write_bf16(p, t, p.master[t]);
}

}  // namespace

hipError_t launch_refresh_bf16(const MlpParams& p, int n, hipStream_t s) {
  hipLaunchKernelGGL(refresh_bf16_kernel, dim3((n + 255) / 256), dim3(256), 0, s, p, n);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Closure inside the model: features from the halo-padded state, and the
// conservative flux divergence of the predicted vertical fluxes.
// ---------------------------------------------------------------------------

// Standardised input f (0..499) of the cell `cell`: variable f / 125 of
// (u, v, w, b) at offset (dk, dj, di) = digits of f % 125 in base 5, minus 2.
template <class T>
__device__ inline float feature_value(const Dims& d, const T* u, const T* v, const T* w,
                                      const T* tt, const T* ss, const ClosureStats& st, long cell,
                                      int f) {
  const int i = (int)(cell % d.nx);
  const int j = (int)((cell / d.nx) % d.ny);
  const int k = (int)(cell / ((long)d.nx * d.ny));
  const int var = f / 125, o = f % 125;
  const int dk = o / 25 - 2, dj = (o / 5) % 5 - 2, di = o % 5 - 2;
  const long p = pidx(d, i + di, j + dj, k + dk);
  float x;
  if (var == 0) x = (float)u[p];
  else if (var == 1) x = (float)v[p];
  else if (var == 2) x = (float)w[p];
  else x = st.g_alpha * ((float)tt[p] - st.t_ref) - st.g_beta * ((float)ss[p] - st.s_ref);
  return (x - st.in_mean[var]) / st.in_std[var];
}

// ---------------------------------------------------------------------------
// The network on 16 MI rows (cells), from staged features to the four
// outputs, by a workgroup of four waves.  Wave wv computes outputs
// [64 wv, 64 wv + 64) of the two wide layers for every row, transposed
// (C^T = W H^T: weights as the first MFMA operand, rows as the second), so
// that a lane's four results are four consecutive outputs of one row and go
// to LDS in one 8-byte store.  The weights come from L2 straight into
// registers in operand order (one contiguous kilobyte per MFMA operand; with
// row-major weights the same loads touched sixteen 64-byte pieces each and
// the in-model kernel took 240 us at 64^3 instead of 157), NET_D chunks ahead
// of their use and across the layers.  Activations stay in LDS as the operand
// of the next layer; operands are rounded to BF16, sums are FP32 in ascending
// k.  Bound by issue: the two GELU epilogues (about 20 vector slots per
// activation, 65 us at 262144 rows) and the MFMAs (41 us) share the SIMDs
// with the staging.  64 rows, weights two chunks ahead and two workgroups'
// registers measured best at 262144 rows: 187 us, against 214 (128 rows),
// 226 (32 rows), 197 (weights one chunk ahead), 209 (a register cap for
// three waves per SIMD, spills) and 188-190 (features two or three blocks
// ahead).
//
// stage(b) writes features 64 b .. 64 b + 63 of every row to columns
// 64 (b % 2) .. of `sx` (pitch NET_SP); out(i, c) takes the outputs of row
// block i (lanes 0..15: row 16 i + lane, the four outputs in c).  `sx` and the
// stager's own tables may share LDS with `hs`: they are dead before the
// first activation is stored.
// ---------------------------------------------------------------------------
constexpr int NET_HP = MLP_NH + 8, NET_SP = 2 * 64 + 8, NET_D = 2;
constexpr int NET_S1 = MLP_KIN / 32, NET_S2 = MLP_NH / 32;   // k chunks per layer

// operand block `block` (uniform) of f: 16 bytes per lane
__device__ inline bf16x8 ldfrag(const __bf16* f, int block) {
  const __bf16* b = f + (long)block * 512;
  return ((const __attribute__((address_space(1))) bf16x8*)b)[threadIdx.x & 63];
}

template <int MI, class Stage, class Out>
__device__ inline void net_rows(const MlpParams& p, int wv, __bf16* hs, const __bf16* sx,
                                Stage& stage, const Out& out) {
  const int lane = threadIdx.x & 63;
  const int lr = lane & 15, lg = lane >> 4;
  auto load_b = [&](int s, bf16x8* b) {
#pragma unroll
    for (int j = 0; j < 4; ++j)
      b[j] = s < NET_S1 ? ldfrag(p.W1f, (wv * 4 + j) * NET_S1 + s)
                        : ldfrag(p.W2f, (wv * 4 + j) * NET_S2 + s - NET_S1);
  };
  f32x4 acc[MI][4];
  auto zero = [&]() {
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  };
  auto mma = [&](const __bf16* rows, int pitch, int k0, const bf16x8* b) {
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      const bf16x8 a = *(const bf16x8*)&rows[(i * 16 + lr) * pitch + k0 + 8 * lg];
#pragma unroll
      for (int j = 0; j < 4; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[j], a, acc[i][j], 0, 0, 0);
    }
  };
  // acc[i][j][e]: row 16 i + lane % 16, output wv 64 + 16 j + 4 (lane / 16) + e
  auto store_h = [&](const float* bias) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int n = wv * 64 + j * 16 + 4 * lg;
      const f32x4 bn = *(const __attribute__((address_space(1))) f32x4*)(bias + n);
#pragma unroll
      for (int i = 0; i < MI; ++i) {
        bf16x4 h;
#pragma unroll
        for (int e = 0; e < 4; ++e) h[e] = (__bf16)gelu(acc[i][j][e] + bn[e]);
        *(bf16x4*)&hs[(i * 16 + lr) * NET_HP + n] = h;
      }
    }
  };
  bf16x8 wb[NET_D][4];
#pragma unroll
  for (int s = 0; s < NET_D; ++s) load_b(s, wb[s]);

  // layer 1: two 32-deep chunks per barrier.  Block b uses half b % 2 of sx;
  // a wave writes a half only after the barrier of the block in between,
  // which every wave reaches after its products of the block that last read
  // the half.
  zero();
#pragma unroll
  for (int b = 0; b < NET_S1 / 2; ++b) {
    stage(b);
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int s = 2 * b + q;
      mma(sx, NET_SP, (b & 1) * 64 + q * 32, wb[s % NET_D]);
      load_b(s + NET_D, wb[s % NET_D]);
    }
  }
  __syncthreads();                  // every wave's last feature reads are done
  store_h(p.master + MLP_OFF_B1);
  __syncthreads();

  // layer 2: no barriers
  zero();
#pragma unroll
  for (int s = NET_S1; s < NET_S1 + NET_S2; ++s) {
    mma(hs, NET_HP, (s - NET_S1) * 32, wb[s % NET_D]);
    if (s + NET_D < NET_S1 + NET_S2) load_b(s + NET_D, wb[s % NET_D]);
  }
  __syncthreads();                  // every wave's reads of the layer-1 activations are done
  store_h(p.master + MLP_OFF_B2);
  __syncthreads();

  // layer 3 (outputs padded to 16): wave wv takes row blocks wv, wv + 4, ...
  const float* b3 = p.master + MLP_OFF_B3;
#pragma unroll
  for (int i0 = 0; i0 < MI; i0 += 4) {
    const int i = i0 + wv;
    if (i >= MI) break;             // uniform per wave
    f32x4 c3 = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < NET_S2; ++s)
      c3 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
          ldfrag(p.W3f, s), *(const bf16x8*)&hs[(i * 16 + lr) * NET_HP + s * 32 + 8 * lg], c3, 0,
          0, 0);
#pragma unroll
    for (int e = 0; e < MLP_NOUT; ++e) c3[e] += b3[e];
    if (lg == 0) out(i, c3);
  }
}

// Features from rows of 500 FP32 (oc_mlp_forward): a block of 64 features is
// loaded 256 bytes per row (16 bytes per lane) one block ahead, rounded and
// stored to LDS.  Rows past the batch repeat its last row.
template <int MI>
struct RowStage {
  const float* x;
  __bf16* sx;
  int row0, last;
  f32x4 r[MI];
  __device__ inline void load(int b) {
    const int f = b * 64 + (threadIdx.x & 15) * 4, t = threadIdx.x >> 4;
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      r[i] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (f < MLP_NIN) r[i] = ld4(x, (long)min(row0 + 16 * i + t, last) * MLP_NIN + f);
    }
  }
  __device__ inline void operator()(int b) {
    const int c = (b & 1) * 64 + (threadIdx.x & 15) * 4, t = threadIdx.x >> 4;
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      bf16x4 h;
#pragma unroll
      for (int e = 0; e < 4; ++e) h[e] = (__bf16)r[i][e];
      *(bf16x4*)&sx[(16 * i + t) * NET_SP + c] = h;
    }
    if (b + 1 < NET_S1 / 2) load(b + 1);
  }
};

// Inference from FP32 rows in one pass: each feature is read once (524 MB at
// 262144 rows) and only the outputs are written; 787 us (a conversion pass
// and three products through memory) -> 187 us, 2.8 TB/s.
template <int MI>
__global__ void __launch_bounds__(256, 2) mlp_forward_kernel(MlpParams p, const float* x, int B,
                                                             float* y) {
  __shared__ __attribute__((aligned(16))) __bf16 hs[MI * 16 * NET_HP];
  RowStage<MI> st;
  st.x = x;
  st.sx = hs;      // features first, activations once the first layer is done
  st.row0 = (int)blockIdx.x * MI * 16;
  st.last = B - 1;
  st.load(0);
  net_rows<MI>(p, threadIdx.x >> 6, hs, hs, st, [&](int i, f32x4 c) {
    const int row = st.row0 + 16 * i + (int)(threadIdx.x & 15);
    if (row < B)
      *(__attribute__((address_space(1))) v4u<float>*)(y + (long)row * MLP_NOUT) = c;
  });
}

// ---------------------------------------------------------------------------
// Training: gradients of the mean squared error in three launches.
//
//   1. mlp_fwdbwd_kernel: everything that is local to a row.  A workgroup
//      takes 32 rows from the FP32 features through the three layers, the
//      loss and back to both layers' errors, with the pre-activations in
//      registers; it leaves the BF16 operands of the weight gradients and
//      the FP32 bias gradients and squared error of its rows.
//   2. mlp_wgrad_kernel: dW = dZ^T H over the batch for the three layers in
//      one launch, 64 x 64 tiles, the batch split over workgroups and waves.
//   3. mlp_grad_final_kernel: the splits added in order; for a training step
//      Adam as well.
//
// The operands go between 1 and 2 in MFMA order: one kilobyte holds 32 rows
// (the k of the weight gradients) x 16 columns, lane l with column l % 16 and
// rows 4 g + 0..3, 16 + 4 g + 0..3, g = l / 16: the rows whose results a lane
// of two 16-row products already has, so they are packed in registers and
// neither side transposes.  (The sum over k takes the rows in any order, the
// same for both operands.)
//
// 4096 rows take 64 us with the loss read back (25 + 10 + 5 us of kernels).
// They took 21 launches and 279 us when the pre-activations and errors went
// through memory and the weight gradients transposed both operands two
// bytes at a time.
// ---------------------------------------------------------------------------
constexpr int TR_XP = MLP_KIN + 8;           // LDS pitch of the BF16 features
constexpr int TR_DP = 40;                    // and of the BF16 output errors

__device__ inline void stfrag(__bf16* f, int block, bf16x8 v) {
  __bf16* b = f + (long)block * 512;
  ((__attribute__((address_space(1))) bf16x8*)b)[threadIdx.x & 63] = v;
}
// the 8 rows of a lane in a 32-row block
__device__ inline bf16x8 pack_rows(f32x4 lo, f32x4 hi) {
  bf16x8 v;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    v[e] = (__bf16)lo[e];
    v[4 + e] = (__bf16)hi[e];
  }
  return v;
}
// sum over the 32 rows of a block, in every lane of the column
__device__ inline float sum_rows(f32x4 lo, f32x4 hi) {
  float s = ((lo[0] + lo[1]) + (lo[2] + lo[3])) + ((hi[0] + hi[1]) + (hi[2] + hi[3]));
  s += __shfl_xor(s, 16);
  return s + __shfl_xor(s, 32);
}

// Wave wv computes outputs [64 wv, 64 wv + 64) of every layer (rows as the
// first MFMA operand: lane l holds rows 4 (l / 16) + e of column l % 16).
// Blocks of 32 rows are dealt to at most TR_MAXWG workgroups, which keep the
// bias sums of theirs; LOOP: more blocks than workgroups (a kernel of its
// own, because the loop costs registers: 251 against 134).  Bound by latency
// at the usual batch sizes: 33 k chunks in a row, each waiting for 16 KB of
// weights from L2, two chunks in flight (four or eight: the same time, half
// the waves); 25 us at 4096 rows.
template <bool LOOP>
__global__ void __launch_bounds__(256, 2) mlp_fwdbwd_kernel(MlpParams p, MlpTrain t, const float* x,
                                                            const float* target, int B) {
  __shared__ __attribute__((aligned(16))) __bf16 xs[32 * TR_XP];   // features, then h2
  __shared__ __attribute__((aligned(16))) __bf16 hs[32 * NET_HP];  // h1, then dz2
  __shared__ __attribute__((aligned(16))) __bf16 ds[32 * TR_DP];   // dy (columns 4.. zero)
  // (the wave number made scalar: operand loads take a scalar base)
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lr = lane & 15, lg = lane >> 4;
  for (int e = threadIdx.x; e < 32 * TR_DP; e += 256) ds[e] = (__bf16)0.f;
  const float scale = 2.0f / (float)(B * 4);
  float db1[4] = {0.f, 0.f, 0.f, 0.f}, db2[4] = {0.f, 0.f, 0.f, 0.f}, db3 = 0.f;
  double loss = 0.0;
  int opaque = 0;

  f32x4 acc[2][4], z1[2][4], z2[2][4];
  // acc = rows (LDS, 32 x 32 S) * weights (operand blocks wv 4 + j, S k blocks)
  auto product = [&](const __bf16* rows, int pitch, const __bf16* wf, auto nk) {
    constexpr int S = decltype(nk)::value, D = S < 2 ? S : 2;
    static_assert(S % D == 0, "whole turns");
    bf16x8 wb[D][4];
    auto load_b = [&](int s, bf16x8* b) {
#pragma unroll
      for (int j = 0; j < 4; ++j) b[j] = ldfrag(wf + opaque, (wv * 4 + j) * S + s);
    };
#pragma unroll
    for (int s = 0; s < D; ++s) load_b(s, wb[s]);
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    // not unrolled across turns: the compiler would hoist every weight load
#pragma unroll 1
    for (int s0 = 0; s0 < S; s0 += D)
#pragma unroll
      for (int q = 0; q < D; ++q) {
        const int s = s0 + q;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const bf16x8 a = *(const bf16x8*)&rows[(i * 16 + lr) * pitch + s * 32 + 8 * lg];
#pragma unroll
          for (int j = 0; j < 4; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, wb[q][j], acc[i][j], 0, 0, 0);
        }
        if (s + D < S) load_b(s + D, wb[q]);
      }
  };
  // a layer's 32 x 64 results: to LDS as the next product's rows, to memory
  // as an operand of the weight gradients
  auto emit = [&](const f32x4 (&h)[2], int j, __bf16* rows, int pitch, __bf16* out, int kb) {
    const int n = wv * 64 + j * 16 + lr;
    if (rows) {
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) rows[(i * 16 + 4 * lg + e) * pitch + n] = (__bf16)h[i][e];
    }
    stfrag(out, kb * 16 + wv * 4 + j, pack_rows(h[0], h[1]));
  };
  auto bias_gelu = [&](const float* bias, f32x4 (&z)[2][4], __bf16* rows, int pitch, __bf16* out,
                       int kb) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float bn = bias[wv * 64 + j * 16 + lr];
      f32x4 h[2];
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          z[i][j][e] = acc[i][j][e] + bn;
          h[i][e] = gelu(z[i][j][e]);
        }
      emit(h, j, rows, pitch, out, kb);
    }
  };
  auto gelu_bwd = [&](const f32x4 (&z)[2][4], float* db, __bf16* rows, int pitch, __bf16* out,
                      int kb) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      f32x4 dz[2];
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) dz[i][e] = acc[i][j][e] * gelu_prime(z[i][j][e]);
      db[j] += sum_rows(dz[0], dz[1]);
      emit(dz, j, rows, pitch, out, kb);
    }
  };
  using K1 = std::integral_constant<int, NET_S1>;
  using K2 = std::integral_constant<int, NET_S2>;

  int kb = blockIdx.x;
  do {
    const long row0 = (long)kb * 32;
    // an offset of zero that the compiler cannot see through: it would hoist
    // the weight loads out of this loop and spill them
    if (LOOP) {
      asm volatile("" : "+s"(opaque));
      __syncthreads();   // the previous block's h2 is read
    }
    // ---- features: 8 rows x 512 bytes per pass
    {
      f32x4 r[16];
      const int c = (threadIdx.x & 31) * 4, rr = threadIdx.x >> 5;
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        const int f = (q & 3) * 128 + c;
        r[q] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (f < MLP_NIN) r[q] = ld4(x, (row0 + (q >> 2) * 8 + rr) * MLP_NIN + f);
      }
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        bf16x4 h;
#pragma unroll
        for (int e = 0; e < 4; ++e) h[e] = (__bf16)r[q][e];
        *(bf16x4*)&xs[((q >> 2) * 8 + rr) * TR_XP + (q & 3) * 128 + c] = h;
      }
    }
    __syncthreads();
    product(xs, TR_XP, p.W1f, K1{});
    // the features as an operand (8 of the 32 column blocks per wave)
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int fb = wv * 8 + q;
      bf16x8 v;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        v[e] = xs[(4 * lg + e) * TR_XP + fb * 16 + lr];
        v[4 + e] = xs[(16 + 4 * lg + e) * TR_XP + fb * 16 + lr];
      }
      stfrag(t.xf, kb * 32 + fb, v);
    }
    bias_gelu(p.master + MLP_OFF_B1, z1, hs, NET_HP, t.h1f, kb);
    __syncthreads();
    product(hs, NET_HP, p.W2f, K2{});
    bias_gelu(p.master + MLP_OFF_B2, z2, xs, NET_HP, t.h2f, kb);   // h2 over the features
    __syncthreads();
    // ---- outputs, loss and their error: the first wave
    if (wv == 0) {
      f32x4 y[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
      for (int s = 0; s < NET_S2; ++s) {
        const bf16x8 b = ldfrag(p.W3f + opaque, s);
#pragma unroll
        for (int i = 0; i < 2; ++i)
          y[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
              *(const bf16x8*)&xs[(i * 16 + lr) * NET_HP + s * 32 + 8 * lg], b, y[i], 0, 0, 0);
      }
      f32x4 dy[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
      if (lr < MLP_NOUT) {
        const float b3 = p.master[MLP_OFF_B3 + lr];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int r = i * 16 + 4 * lg + e;
            const float d = (y[i][e] + b3) - target[(row0 + r) * MLP_NOUT + lr];
            loss += (double)d * d;
            dy[i][e] = scale * d;
            ds[r * TR_DP + lr] = (__bf16)dy[i][e];
          }
      }
      db3 += sum_rows(dy[0], dy[1]);
      stfrag(t.dyf, kb, pack_rows(dy[0], dy[1]));
    }
    __syncthreads();
    product(ds, TR_DP, p.W3Tf, std::integral_constant<int, 1>{});
    gelu_bwd(z2, db2, hs, NET_HP, t.dz2f, kb);   // dz2 over h1
    __syncthreads();
    product(hs, NET_HP, p.W2Tf, K2{});
    gelu_bwd(z1, db1, nullptr, 0, t.dz1f, kb);
    kb += gridDim.x;
  } while (LOOP && kb < B / 32);

  // this workgroup's bias sums (any lane of a column) and squared error
  float* pb = t.biasp + (long)blockIdx.x * TR_NB;
  if (lg == 0)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      pb[wv * 64 + j * 16 + lr] = db1[j];
      pb[MLP_NH + wv * 64 + j * 16 + lr] = db2[j];
    }
  if (wv == 0) {
    if (lane < MLP_NOUT) pb[2 * MLP_NH + lane] = db3;
#pragma unroll
    for (int h = 32; h > 0; h >>= 1) loss += __shfl_xor(loss, h);
    if (lane == 0) t.lossp[blockIdx.x] = loss;
  }
}

// Tiles of the weight gradients: 4 x 8 of dW1 (the last column tile half
// padding), 4 x 4 of dW2, 1 x 4 of dW3 (16 rows, 4 real).  A tile's batch
// range is dealt to the four waves, whose sums are added in LDS.
constexpr int WG_T1 = 32, WG_T2 = WG_T1 + 16, WG_TILES = WG_T2 + 4;

__global__ void __launch_bounds__(256) mlp_wgrad_kernel(MlpTrain t, int nkb, int nsplit,
                                                        float* out) {
  __shared__ __attribute__((aligned(16))) float red[4][64 * 64];
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int tile = blockIdx.x, sp = blockIdx.y;
  const __bf16 *A, *Bm;
  int na, nb, a0, b0, ld, cols, off;   // operand blocks per 32 rows; this tile's first ones
  if (tile < WG_T1) {
    A = t.dz1f; na = 16; a0 = (tile >> 3) * 4;
    Bm = t.xf; nb = 32; b0 = (tile & 7) * 4;
    ld = MLP_NIN; cols = MLP_NIN; off = MLP_OFF_W1;
  } else if (tile < WG_T2) {
    A = t.dz2f; na = 16; a0 = ((tile - WG_T1) >> 2) * 4;
    Bm = t.h1f; nb = 16; b0 = ((tile - WG_T1) & 3) * 4;
    ld = MLP_NH; cols = MLP_NH; off = MLP_OFF_W2;
  } else {
    A = t.dyf; na = 1; a0 = 0;
    Bm = t.h2f; nb = 16; b0 = (tile - WG_T2) * 4;
    ld = MLP_NH; cols = MLP_NH; off = MLP_OFF_W3;
  }
  const int ni = na == 1 ? 1 : 4;   // uniform
  const int k0 = (int)((long)sp * nkb / nsplit), k1 = (int)((long)(sp + 1) * nkb / nsplit);
  f32x4 acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  bf16x8 a[2][4], b[2][4];
  auto load = [&](int kb, bf16x8* va, bf16x8* vb) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (i < ni) va[i] = ldfrag(A, kb * na + a0 + i);
#pragma unroll
    for (int j = 0; j < 4; ++j) vb[j] = ldfrag(Bm, kb * nb + b0 + j);
  };
  auto mma = [&](const bf16x8* va, const bf16x8* vb) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (i < ni)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va[i], vb[j], acc[i][j], 0, 0, 0);
  };
  int kb = k0 + wv;
  if (kb < k1) load(kb, a[0], b[0]);
  for (; kb < k1; kb += 8) {   // two blocks per turn, each loaded one ahead
    if (kb + 4 < k1) load(kb + 4, a[1], b[1]);
    mma(a[0], b[0]);
    if (kb + 4 < k1) {
      if (kb + 8 < k1) load(kb + 8, a[0], b[0]);
      mma(a[1], b[1]);
    }
  }
  // lane: rows 16 i + 4 (lane / 16) + e, column 16 j + lane % 16
  const int lr = lane & 15, lg = lane >> 4;
#pragma unroll
  for (int i = 0; i < 4; ++i)
    if (i < ni)
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          red[wv][(16 * i + 4 * lg + e) * 64 + 16 * j + lr] = acc[i][j][e];
  __syncthreads();
  float* o = out + (long)sp * MLP_NPARAM + off;
  const int rows = na == 1 ? MLP_NOUT : 64;
  for (int q = threadIdx.x; q < rows * 64; q += 256) {
    const int r = a0 * 16 + (q >> 6), c = b0 * 16 + (q & 63);
    if (c < cols) o[r * ld + c] = ((red[0][q] + red[1][q]) + red[2][q]) + red[3][q];
  }
}

// Sums of the splits, in order; biases from the workgroups' sums.  The first
// blocks take the weights (a thread per parameter), then 33 blocks of 16
// biases (16 lanes each over the workgroups, added in a fixed tree); one
// more adds the loss.  adam.lr > 0: Adam (Kingma & Ba) on the FP32
// master parameters, refreshing the BF16 copies.
struct AdamArgs {
  float *m1, *m2;
  float lr, c1, c2;   // c = 1 - beta^t
};
constexpr int GF_BIAS = (2 * MLP_NH + MLP_NOUT + 15) / 16;

__global__ void __launch_bounds__(256) mlp_grad_final_kernel(MlpParams p, MlpTrain t,
                                                             const float* part, int nsplit,
                                                             int nwg, float* grad, AdamArgs ad) {
  auto finish = [&](int q, float g) {
    grad[q] = g;
    if (ad.lr > 0.f) {
      const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
      const float mm = b1 * ad.m1[q] + (1.f - b1) * g;
      const float vv = b2 * ad.m2[q] + (1.f - b2) * g * g;
      ad.m1[q] = mm;
      ad.m2[q] = vv;
      const float w = p.master[q] - ad.lr * (mm / ad.c1) / (sqrtf(vv / ad.c2) + eps);
      p.master[q] = w;
      mlp_write_bf16(p, q, w);
    }
  };
  const int nw = (MLP_NPARAM + 255) / 256;
  if ((int)blockIdx.x < nw) {
    const int q = blockIdx.x * 256 + threadIdx.x;
    const bool bias = (q >= MLP_OFF_B1 && q < MLP_OFF_W2) || (q >= MLP_OFF_B2 && q < MLP_OFF_W3) ||
                      q >= MLP_OFF_B3;
    if (q >= MLP_NPARAM || bias) return;
    float s = 0.f;
    for (int z = 0; z < nsplit; ++z) s += part[(long)z * MLP_NPARAM + q];
    finish(q, s);
    return;
  }
  const int bb = (int)blockIdx.x - nw;
  if (bb < GF_BIAS) {
    __shared__ float red[16][17];
    const int c = threadIdx.x & 15, rl = threadIdx.x >> 4, n = bb * 16 + c;
    float s = 0.f;
    if (n < 2 * MLP_NH + MLP_NOUT)
#pragma unroll 8
      for (int w = rl; w < nwg; w += 16) s += t.biasp[(long)w * TR_NB + n];
    red[rl][c] = s;
    __syncthreads();
    if (rl == 0 && n < 2 * MLP_NH + MLP_NOUT) {
      float a = 0.f;
#pragma unroll
      for (int r = 0; r < 16; ++r) a += red[r][c];
      finish(n < MLP_NH ? MLP_OFF_B1 + n
                        : (n < 2 * MLP_NH ? MLP_OFF_B2 + n - MLP_NH : MLP_OFF_B3 + n - 2 * MLP_NH),
             a);
    }
    return;
  }
  __shared__ double sd[256];
  double s = 0.0;
  for (int w = threadIdx.x; w < nwg; w += 256) s += t.lossp[w];
  sd[threadIdx.x] = s;
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if ((int)threadIdx.x < h) sd[threadIdx.x] += sd[threadIdx.x + h];
    __syncthreads();
  }
  if (threadIdx.x == 0) t.loss[0] = sd[0];
}

// The closure network on every cell of a model: 16 MI consecutive cells per
// workgroup, whose features are the standardised (u, v, w, b) in the 5 x 5 x
// 5 neighbourhoods.
//
// Rows of GW consecutive cells share an x row, so the standardised BF16
// values over their whole 5 x 5 x (GW + 4) neighbourhood regions are loaded
// once (coalesced along x) into LDS, and each block of features is copied
// out of the region (im2col in LDS).
constexpr int RG_ROWS = 4 * 25 + 1;                         // + a row of zeros
constexpr int rg_pitch(int gw) { return gw + 8; }

// Element offset in the region buffer of input feature f: variable f / 125
// (u, v, w, b), row 25 var + 5 dk + dj and column di, where (dk, dj, di) are
// the base-5 digits of f % 125; the padding features past the 500 inputs
// read the row of zeros.
struct RgOffsets {
  unsigned short v[MLP_KIN];
};
constexpr RgOffsets make_rg_offsets(int pitch) {
  RgOffsets t{};
  for (int f = 0; f < MLP_KIN; ++f) {
    if (f >= MLP_NIN) {
      t.v[f] = (unsigned short)((RG_ROWS - 1) * pitch);
      continue;
    }
    const int var = f / 125, o = f % 125;
    t.v[f] = (unsigned short)((var * 25 + o / 5) * pitch + o % 5);
  }
  return t;
}
__constant__ RgOffsets kRgOff64 = make_rg_offsets(rg_pitch(64));
__constant__ RgOffsets kRgOff32 = make_rg_offsets(rg_pitch(32));

template <int MI, int GW>
struct RegionStage {
  const __bf16* rg;
  __bf16* sx;
  // cell `lane` + 64 m of the workgroup; wave wv copies features 64 b + 16 wv .. + 15
  __device__ inline void operator()(int b) const {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int f0 = __builtin_amdgcn_readfirstlane(b * 64 + 16 * wv);
    const unsigned short* off = GW == 64 ? kRgOff64.v : kRgOff32.v;
#pragma unroll
    for (int m = 0; m < MI / 4; ++m) {
      const int c = lane + 64 * m;
      const __bf16* r = rg + (c / GW) * (RG_ROWS * rg_pitch(GW)) + c % GW;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        bf16x8 xv;
#pragma unroll
        for (int q = 0; q < 8; ++q) xv[q] = r[off[f0 + 8 * h + q]];
        *(bf16x8*)&sx[c * NET_SP + (b & 1) * 64 + 16 * wv + 8 * h] = xv;
      }
    }
  }
};

template <class T, int MI, int GW>
__global__ void __launch_bounds__(256, 2) closure_mlp_region_kernel(Dims d, const T* u, const T* v,
                                                                const T* w, const T* tt,
                                                                const T* ss, ClosureStats st,
                                                                MlpParams p, float* y) {
  constexpr int MR = MI * 16, NG = MR / GW, RX = GW + 4, RP = rg_pitch(GW);
  constexpr int SX = MR * NET_SP, LDS = SX + NG * RG_ROWS * RP;
  constexpr int HS = MR * NET_HP;
  __shared__ __attribute__((aligned(16))) __bf16 lds[LDS > HS ? LDS : HS];
  __bf16* sx = lds;
  __bf16* rg = lds + SX;
  const int c0 = (int)blockIdx.x * MR;
  // the neighbourhood regions, standardised, in BF16 (compile-time trip
  // count: every load of a region is in flight before the first is used)
#pragma unroll
  for (int g = 0; g < NG; ++g) {
    const int cg = c0 + g * GW;
    const int i0 = cg % d.nx, jk = cg / d.nx;
    const int j0 = jk % d.ny, k0 = jk / d.ny;
    __bf16* R = rg + g * RG_ROWS * RP;
#pragma unroll
    for (int q = 0; q < (25 * RX + 255) / 256; ++q) {
      const int e = (int)threadIdx.x + q * 256;
      if (e >= 25 * RX) break;
      const int row = e / RX, x = e - row * RX;
      const int dk = row / 5, dj = row - dk * 5;
      const long pp = pidx(d, i0 - 2 + x, j0 - 2 + dj, k0 - 2 + dk);
      R[row * RP + x] = (__bf16)(((float)u[pp] - st.in_mean[0]) * st.in_rstd[0]);
      R[(25 + row) * RP + x] = (__bf16)(((float)v[pp] - st.in_mean[1]) * st.in_rstd[1]);
      R[(50 + row) * RP + x] = (__bf16)(((float)w[pp] - st.in_mean[2]) * st.in_rstd[2]);
      const float b =
          st.g_alpha * ((float)tt[pp] - st.t_ref) - st.g_beta * ((float)ss[pp] - st.s_ref);
      R[(75 + row) * RP + x] = (__bf16)((b - st.in_mean[3]) * st.in_rstd[3]);
    }
    if ((int)threadIdx.x < RP) R[(RG_ROWS - 1) * RP + threadIdx.x] = (__bf16)0.0f;
  }
  __syncthreads();
  RegionStage<MI, GW> stage{rg, sx};
  net_rows<MI>(p, __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lds, sx, stage, [&](int i, f32x4 c) {
    *(__attribute__((address_space(1))) f32x4*)(
        y + (long)(c0 + 16 * i + (int)(threadIdx.x & 15)) * MLP_NOUT) = c;
  });
}

// Any x length (rows of 8 or 16 cells): the features gathered from memory
// 64 at a time, one block ahead of their use; the walk over (variable,
// offset) is uniform per wave and runs on the scalar unit.
template <class T>
struct GatherStage {
  const T *u, *v, *w, *tt, *ss;
  const ClosureStats& st;
  __bf16* sx;
  int corner, sy, sz;   // padded offset of the neighbourhood corner (i-2, j-2, k-2)
  bool live;
  float graw[16], sraw[16];
  __device__ inline void load(int b) {
    int f = __builtin_amdgcn_readfirstlane(b * 64 + (int)(threadIdx.x >> 6) * 16);
    int var = f / 125, o = f - var * 125;
    int dk = o / 25, dj = (o - dk * 25) / 5, di = o - dk * 25 - dj * 5;
#pragma unroll
    for (int q = 0; q < 16; ++q, ++f) {
      const int off = dk * sz + dj * sy + di;
      graw[q] = 0.f;
      sraw[q] = 0.f;
      if (f < MLP_NIN) {
        if (var == 0) graw[q] = (float)u[corner + off];
        else if (var == 1) graw[q] = (float)v[corner + off];
        else if (var == 2) graw[q] = (float)w[corner + off];
        else { graw[q] = (float)tt[corner + off]; sraw[q] = (float)ss[corner + off]; }
      }
      if (++di == 5) { di = 0; if (++dj == 5) { dj = 0; if (++dk == 5) { dk = 0; ++var; } } }
    }
  }
  __device__ inline void operator()(int b) {
    int f = __builtin_amdgcn_readfirstlane(b * 64 + (int)(threadIdx.x >> 6) * 16);
    int var = f / 125;
    int o = f - var * 125;
    bf16x8 xv[2];
#pragma unroll
    for (int q = 0; q < 16; ++q, ++f) {
      const int vq = var < 4 ? var : 3;
      const float raw = vq == 3 ? st.g_alpha * (graw[q] - st.t_ref) - st.g_beta * (sraw[q] - st.s_ref)
                                : graw[q];
      const float x = (live && f < MLP_NIN) ? (raw - st.in_mean[vq]) * st.in_rstd[vq] : 0.f;
      xv[q >> 3][q & 7] = (__bf16)x;
      if (++o == 125) { o = 0; ++var; }
    }
    __bf16* at = &sx[(threadIdx.x & 63) * NET_SP + (b & 1) * 64 + (threadIdx.x >> 6) * 16];
    *(bf16x8*)at = xv[0];
    *(bf16x8*)(at + 8) = xv[1];
    if (b + 1 < NET_S1 / 2) load(b + 1);
  }
};

template <class T>
__global__ void __launch_bounds__(256) closure_mlp_gather_kernel(Dims d, const T* u, const T* v,
                                                                const T* w, const T* tt,
                                                                const T* ss, ClosureStats st,
                                                                MlpParams p, float* y) {
  __shared__ __attribute__((aligned(16))) __bf16 hs[64 * NET_HP];
  const int ncell = d.nx * d.ny * d.nz;
  const int c0 = (int)blockIdx.x * 64, cell = c0 + (int)(threadIdx.x & 63);
  const bool live = cell < ncell;
  int corner = 0;
  if (live) {
    const int jk = cell / d.nx;
    corner = (int)pidx(d, cell % d.nx - 2, jk % d.ny - 2, jk / d.ny - 2);
  }
  GatherStage<T> stage{u, v, w, tt, ss, st, hs, corner, (int)d.sy, (int)d.sz, live, {}, {}};
  stage.load(0);
  net_rows<4>(p, __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), hs, hs, stage, [&](int i, f32x4 c) {
    const int row = c0 + 16 * i + (int)(threadIdx.x & 15);
    if (row < ncell)
      *(__attribute__((address_space(1))) f32x4*)(y + (long)row * MLP_NOUT) = c;
  });
}

// FP32 rows of 500: the network input of oc_mlp_* (training data).
template <class T>
__global__ void __launch_bounds__(256) closure_features_f32_kernel(Dims d, const T* u,
                                                                   const T* v, const T* w,
                                                                   const T* tt, const T* ss,
                                                                   ClosureStats st, float* x) {
  const long ncell = (long)d.nx * d.ny * d.nz;
  const long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= ncell * 500) return;
  x[t] = feature_value(d, u, v, w, tt, ss, st, t / 500, (int)(t % 500));
}

// Physical fluxes F_q = y_q std_q + mean_q at cell centres; u takes the
// flux at (x face, z face) as the mean of the four adjacent centres, v the
// same in y, tracers the mean of the two centres about each z face (J_b
// turned into a temperature flux), w the difference of tau_ww across its
// face.  Wall fluxes are zero.  A thread reads the fluxes of its own column at
// the three levels around it (16 bytes a cell) and of its west and south
// neighbours', all at once, by 32-bit indices (a grid has at most 2^24
// cells): 64^3 5.3 us, 9.2 with 64-bit divisions and a scalar load for
// each use.  8 MB, 1.6 us at 5.2 TB/s.
template <class T>
__global__ void __launch_bounds__(256) closure_apply_kernel(Dims d, const float* y, ClosureStats st,
                                                            double rdz, T* gu, T* gv, T* gw,
                                                            T* gt) {
  typedef float f4 __attribute__((ext_vector_type(4)));
  const uint32_t nx = d.nx, ny = d.ny, nz = d.nz, plane = nx * ny;
  const uint32_t t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= plane * nz) return;
  const uint32_t i = t % nx, row = t / nx, j = row % ny, k = row / ny;
  const uint32_t tw = i == 0 ? t + nx - 1 : t - 1, ts = j == 0 ? t + plane - nx : t - nx;
  const bool low = k > 0, high = k + 1 < nz;   // the faces that are not walls
  const uint32_t dl = low ? plane : 0, dh = high ? plane : 0;
  const auto y4 = (const __attribute__((address_space(1))) f4*)y;
  const auto y1 = glb(y);
  const f4 om = y4[t - dl], o0 = y4[t], op = y4[t + dh];
  const float wm = y1[(tw - dl) * 4], w0 = y1[tw * 4], wp = y1[(tw + dh) * 4];
  const float sm = y1[(ts - dl) * 4 + 1], s0 = y1[ts * 4 + 1], sp = y1[(ts + dh) * 4 + 1];
  auto F = [&](int q, float v) { return v * st.out_std[q] + st.out_mean[q]; };
  // flux of quantity q through the face between the centres a (below) and b,
  // averaged with the neighbour's na, nb
  auto mean4 = [&](int q, float na, float a, float nb, float b) {
    return 0.25f * (F(q, na) + F(q, a) + F(q, nb) + F(q, b));
  };
  const float ul = low ? mean4(0, wm, om.x, w0, o0.x) : 0.f;
  const float uh = high ? mean4(0, w0, o0.x, wp, op.x) : 0.f;
  const float vl = low ? mean4(1, sm, om.y, s0, o0.y) : 0.f;
  const float vh = high ? mean4(1, s0, o0.y, sp, op.y) : 0.f;
  const float tl = low ? 0.5f * (F(3, om.w) + F(3, o0.w)) : 0.f;
  const float th = high ? 0.5f * (F(3, o0.w) + F(3, op.w)) : 0.f;
  const long p = pidx(d, (int)i, (int)j, (int)k);
  const float rz = (float)rdz;
  gu[p] = (T)(-(uh - ul) * rz);
  gv[p] = (T)(-(vh - vl) * rz);
  gt[p] = (T)(-(th - tl) * rz * st.inv_galpha);
  gw[p] = low ? (T)(-(F(2, o0.z) - F(2, om.z)) * rz) : (T)0;
}

// Splits of the batch in the weight gradients: enough that the 52 tiles
// occupy the 256 CUs, each wave with at least four 32-row blocks.
static int wgrad_splits(int nkb) { return std::max(1, std::min(nkb / 16, TR_MAXSPLIT)); }

hipError_t launch_mlp_gradients(const MlpParams& p, const MlpTrain& t, const float* x,
                                const float* target, int B, float* grad, float* m1, float* m2,
                                float lr, int step, hipStream_t s) {
  const int nkb = B / 32, nwg = std::min(nkb, TR_MAXWG), nsplit = wgrad_splits(nkb);
  const auto rows = nwg == nkb ? mlp_fwdbwd_kernel<false> : mlp_fwdbwd_kernel<true>;
  hipLaunchKernelGGL(rows, dim3(nwg), dim3(256), 0, s, p, t, x, target, B);
  hipLaunchKernelGGL(mlp_wgrad_kernel, dim3(WG_TILES, nsplit), dim3(256), 0, s, t, nkb, nsplit,
                     t.part);
  AdamArgs ad{m1, m2, lr, 1.f, 1.f};
  if (lr > 0.f) {
    ad.c1 = 1.f - powf(0.9f, (float)step);
    ad.c2 = 1.f - powf(0.999f, (float)step);
  }
  hipLaunchKernelGGL(mlp_grad_final_kernel, dim3((MLP_NPARAM + 255) / 256 + GF_BIAS + 1), dim3(256),
                     0, s, p, t, (const float*)t.part, nsplit, nwg, grad, ad);
  return hipGetLastError();
}

// 64-row workgroups once they fill the 256 CUs twice (65536 rows: 48 us
// against 53 with 32 rows); below that 32-row ones, twice as many and half as
// long (4096 rows: 11 us).
hipError_t launch_mlp_forward(const MlpParams& p, const float* x, int B, float* y, hipStream_t s) {
  if (B >= 2 * 256 * 64)
    hipLaunchKernelGGL(mlp_forward_kernel<4>, dim3((B + 63) / 64), dim3(256), 0, s, p, x, B, y);
  else
    hipLaunchKernelGGL(mlp_forward_kernel<2>, dim3((B + 31) / 32), dim3(256), 0, s, p, x, B, y);
  return hipGetLastError();
}

template <class T>
hipError_t launch_closure_mlp_fused(const Dims& d, const T* u, const T* v, const T* w, const T* t,
                                    const T* s, ClosureStats st, const MlpParams& p, float* y,
                                    hipStream_t stream) {
  const int n = d.nx * d.ny * d.nz;   // a multiple of 512 (grid lengths are multiples of 8)
  const dim3 nt(256);
  if (d.nx % 64 == 0)
    hipLaunchKernelGGL((closure_mlp_region_kernel<T, 4, 64>), dim3(n / 64), nt, 0, stream, d, u, v,
                       w, t, s, st, p, y);
  else if (d.nx % 32 == 0)
    hipLaunchKernelGGL((closure_mlp_region_kernel<T, 4, 32>), dim3(n / 64), nt, 0, stream, d, u, v,
                       w, t, s, st, p, y);
  else
    hipLaunchKernelGGL(closure_mlp_gather_kernel<T>, dim3((n + 63) / 64), nt, 0, stream, d, u, v,
                       w, t, s, st, p, y);
  return hipGetLastError();
}
template hipError_t launch_closure_mlp_fused<float>(const Dims&, const float*, const float*,
                                                    const float*, const float*, const float*,
                                                    ClosureStats, const MlpParams&, float*,
                                                    hipStream_t);
template hipError_t launch_closure_mlp_fused<double>(const Dims&, const double*, const double*,
                                                     const double*, const double*, const double*,
                                                     ClosureStats, const MlpParams&, float*,
                                                     hipStream_t);

template <class T>
hipError_t launch_closure_features_f32(const Dims& d, const T* u, const T* v, const T* w,
                                       const T* t, const T* s, ClosureStats st, float* x,
                                       hipStream_t stream) {
  const long n = (long)d.nx * d.ny * d.nz * 500;
  hipLaunchKernelGGL(closure_features_f32_kernel<T>, dim3((unsigned)((n + 255) / 256)), dim3(256),
                     0, stream, d, u, v, w, t, s, st, x);
  return hipGetLastError();
}
template hipError_t launch_closure_features_f32<float>(const Dims&, const float*, const float*,
                                                       const float*, const float*, const float*,
                                                       ClosureStats, float*, hipStream_t);
template hipError_t launch_closure_features_f32<double>(const Dims&, const double*,
                                                        const double*, const double*,
                                                        const double*, const double*,
                                                        ClosureStats, float*, hipStream_t);

template <class T>
hipError_t launch_closure_apply(const Dims& d, const float* y, ClosureStats st, double rdz, T* gu,
                                T* gv, T* gw, T* gt, hipStream_t stream) {
  const long n = (long)d.nx * d.ny * d.nz;
  hipLaunchKernelGGL(closure_apply_kernel<T>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0,
                     stream, d, y, st, rdz, gu, gv, gw, gt);
  return hipGetLastError();
}

template hipError_t launch_closure_apply<float>(const Dims&, const float*, ClosureStats, double,
                                                float*, float*, float*, float*, hipStream_t);
template hipError_t launch_closure_apply<double>(const Dims&, const float*, ClosureStats, double,
                                                 double*, double*, double*, double*, hipStream_t);

}  // namespace oc

// MLP subgrid closure on gfx950: BF16 MFMA GEMMs with FP32 accumulation
// for the forward and backward passes, fused bias/GELU epilogues, loss and
// bias-gradient reductions, Adam on FP32 master weights, and the gather of
// the standardised 5x5x5 (u, v, w, b) neighbourhood of every coarse cell.
//
// Network: 500 -> 256 -> 256 -> 4 with exact-erf GELU.  On the device the
// input width is padded to 512 and the output width to 32 with zero weights
// so every GEMM dimension is a multiple of the 32-deep MFMA k step.
#include "oc_internal.h"

namespace oc {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// Fragment-major weight copies: the 16 output rows x 32 inputs that one MFMA
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
    p.W1b[r * 512 + c] = (__bf16)w;
    p.W1f[frag_at(r, c, MLP_KIN / 32)] = (__bf16)w;
  } else if (t >= MLP_OFF_W2 && t < MLP_OFF_B2) {
    const int r = (t - MLP_OFF_W2) / MLP_NH, c = (t - MLP_OFF_W2) % MLP_NH;
    p.W2b[r * MLP_NH + c] = (__bf16)w;
    p.W2bT[c * MLP_NH + r] = (__bf16)w;   // transposed copy for the backward pass
    p.W2f[frag_at(r, c, MLP_NH / 32)] = (__bf16)w;
  } else if (t >= MLP_OFF_W3 && t < MLP_OFF_B3) {
    const int r = (t - MLP_OFF_W3) / MLP_NH, c = (t - MLP_OFF_W3) % MLP_NH;
    p.W3b[t - MLP_OFF_W3] = (__bf16)w;
    p.W3f[frag_at(r, c, MLP_NH / 32)] = (__bf16)w;
  }
}


namespace {

constexpr int BM = 64, BN = 64, BK = 32, LDP = BK + 8;  // LDS rows padded by 8 bf16

// erf(z / sqrt 2) and exp(-z^2 / 2) by Abramowitz & Stegun, formula 7.1.26
// (absolute error of erf at most 1.5e-7, far below the BF16 rounding the
// activations get next): for x >= 0, erf x = 1 - t P(t) exp(-x^2),
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
// no exponential.
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

// Epilogue of one output element (m, n) of a GEMM.
__device__ inline void epilogue(const GemmArgs& g, int m, int n, float v) {
  const long o = (long)m * g.ldc + n;
  switch (g.epi) {
    case EPI_STORE:
      g.C[o] = v;
      break;
    case EPI_BIAS:
      g.C[o] = v + g.bias[n];
      break;
    case EPI_BIAS_GELU: {
      const float z = v + g.bias[n];
      g.C[o] = z;                                   // pre-activation (for backward)
      g.H[(long)m * g.ldh + n] = (__bf16)gelu(z);    // activation (next layer)
      break;
    }
    case EPI_GELU_BWD: {
      const float dz = v * gelu_prime(g.Z[o]);
      g.C[o] = dz;
      g.H[(long)m * g.ldh + n] = (__bf16)dz;
      break;
    }
  }
}

// C[m][n] = sum_k A[m][k] B[k][n].  transA = 0: A[m][k] at A[m*lda + k];
// 1: at A[k*lda + m].  transB = 0: B[k][n] at B[k*ldb + n]; 1: at B[n*ldb + k].
// Tiles are staged in LDS with k contiguous, the order the MFMA operands
// need: lane l holds 8 consecutive k of row (or column) l % 16, k block l / 16.
__global__ void __launch_bounds__(256) gemm_bf16_kernel(GemmArgs g) {
  __shared__ __bf16 As[BM][LDP];
  __shared__ __bf16 Bs[BN][LDP];
  const int tid = threadIdx.x;
  const int lane = tid & 63, wv = tid >> 6;
  const int wm = wv >> 1, wn = wv & 1;
  const int m0 = blockIdx.y * BM, n0 = blockIdx.x * BN;
  // split K: this workgroup's range of the reduction
  const int kspan = g.K / g.ksplit;
  const int kbeg = blockIdx.z * kspan, kend = kbeg + kspan;
  f32x4 acc[2][2];
  for (int i = 0; i < 2; ++i)
    for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  for (int k0 = kbeg; k0 < kend; k0 += BK) {
    // ---- stage A (BM x BK) and B (BN x BK)
    if (!g.transA) {
      const int r = tid >> 2, ks = (tid & 3) * 8;
      const int m = m0 + r;
      bf16x8 v;
      if (m < g.M) v = *(const bf16x8*)(g.A + (long)m * g.lda + k0 + ks);
      else for (int e = 0; e < 8; ++e) v[e] = (__bf16)0.0f;
      *(bf16x8*)&As[r][ks] = v;
    } else {
      const int kk = tid >> 3, ms = (tid & 7) * 8;
      const __bf16* src = g.A + (long)(k0 + kk) * g.lda + m0 + ms;
      for (int e = 0; e < 8; ++e) As[ms + e][kk] = (m0 + ms + e < g.M) ? src[e] : (__bf16)0.0f;
    }
    if (g.transB) {
      const int r = tid >> 2, ks = (tid & 3) * 8;
      const int n = n0 + r;
      bf16x8 v;
      if (n < g.N) v = *(const bf16x8*)(g.B + (long)n * g.ldb + k0 + ks);
      else for (int e = 0; e < 8; ++e) v[e] = (__bf16)0.0f;
      *(bf16x8*)&Bs[r][ks] = v;
    } else {
      const int kk = tid >> 3, ns = (tid & 7) * 8;
      const __bf16* src = g.B + (long)(k0 + kk) * g.ldb + n0 + ns;
      for (int e = 0; e < 8; ++e) Bs[ns + e][kk] = (n0 + ns + e < g.N) ? src[e] : (__bf16)0.0f;
    }
    __syncthreads();
    // ---- 2 x 2 MFMA tiles of 16 x 16 per wave
    bf16x8 a[2], b[2];
    for (int i = 0; i < 2; ++i)
      a[i] = *(const bf16x8*)&As[wm * 32 + i * 16 + (lane & 15)][8 * (lane >> 4)];
    for (int j = 0; j < 2; ++j)
      b[j] = *(const bf16x8*)&Bs[wn * 32 + j * 16 + (lane & 15)][8 * (lane >> 4)];
    for (int i = 0; i < 2; ++i)
      for (int j = 0; j < 2; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
    __syncthreads();
  }

  // ---- epilogue: lane holds rows 4*(lane/16) + e of column lane % 16
  for (int i = 0; i < 2; ++i)
    for (int j = 0; j < 2; ++j) {
      const int n = n0 + wn * 32 + j * 16 + (lane & 15);
      if (n >= g.N) continue;
      for (int e = 0; e < 4; ++e) {
        const int m = m0 + wm * 32 + i * 16 + 4 * (lane >> 4) + e;
        if (m >= g.M) continue;
        const float v = acc[i][j][e];
        if (g.ksplit > 1) {
          g.part[((long)blockIdx.z * g.M + m) * g.N + n] = v;
          continue;
        }
        epilogue(g, m, n, v);
      }
    }
}

// dY = 2 (Y - T) / (B * 4) on the 4 real outputs (FP32 and BF16, padded
// columns zero); per-block partial sums of the squared error.
// C = A B with both operands k-contiguous (A[m][k] at A[m*lda + k], B[k][n]
// at B[n*ldb + k]), M any multiple of 32, N a multiple of 128, K a multiple
// of 64.  Workgroup tile 128 x 128, k step 64, four waves of 64 x 64 (4 x 4
// MFMA 16x16x32 tiles); 16-byte global loads into registers for the next
// k step while the current one is multiplied out of double-buffered LDS.
constexpr int NT_BM = 128, NT_BN = 128, NT_BK = 64, NT_LDP = NT_BK + 8;

__global__ void __launch_bounds__(256) gemm_bf16_nt_kernel(GemmArgs g) {
  __shared__ __bf16 As[2][NT_BM][NT_LDP];
  __shared__ __bf16 Bs[2][NT_BN][NT_LDP];
  const int tid = threadIdx.x;
  const int lane = tid & 63, wv = tid >> 6;
  const int wm = wv >> 1, wn = wv & 1;
  const int m0 = blockIdx.y * NT_BM, n0 = blockIdx.x * NT_BN;
  // each thread moves 4 chunks of 8 bf16 per operand and k step: rows
  // (tid >> 3) + 32 c, k offset 8 (tid & 7)
  const int lr = tid >> 3, lk = (tid & 7) * 8;
  bf16x8 ra[4], rb[4];
  auto load = [&](int k0) {
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int m = m0 + lr + 32 * c;
      if (m < g.M) ra[c] = *(const bf16x8*)(g.A + (long)m * g.lda + k0 + lk);
      else for (int e = 0; e < 8; ++e) ra[c][e] = (__bf16)0.0f;
      const int n = n0 + lr + 32 * c;
      rb[c] = *(const bf16x8*)(g.B + (long)n * g.ldb + k0 + lk);
    }
  };
  auto stash = [&](int buf) {
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      *(bf16x8*)&As[buf][lr + 32 * c][lk] = ra[c];
      *(bf16x8*)&Bs[buf][lr + 32 * c][lk] = rb[c];
    }
  };
  f32x4 acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int nk = g.K / NT_BK;
  load(0);
  stash(0);
  __syncthreads();
  for (int kt = 0; kt < nk; ++kt) {
    const int buf = kt & 1;
    if (kt + 1 < nk) load((kt + 1) * NT_BK);
#pragma unroll
    for (int ks = 0; ks < NT_BK; ks += 32) {
      bf16x8 a[4], b[4];
#pragma unroll
      for (int i = 0; i < 4; ++i)
        a[i] = *(const bf16x8*)&As[buf][wm * 64 + i * 16 + (lane & 15)][ks + 8 * (lane >> 4)];
#pragma unroll
      for (int j = 0; j < 4; ++j)
        b[j] = *(const bf16x8*)&Bs[buf][wn * 64 + j * 16 + (lane & 15)][ks + 8 * (lane >> 4)];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
    }
    if (kt + 1 < nk) stash(buf ^ 1);
    __syncthreads();
  }
  // lane holds rows 4 (lane / 16) + e of column lane % 16 of each 16 x 16 tile
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int n = n0 + wn * 64 + j * 16 + (lane & 15);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int m = m0 + wm * 64 + i * 16 + 4 * (lane >> 4) + e;
        if (m < g.M) epilogue(g, m, n, acc[i][j][e]);
      }
    }
}

__global__ void __launch_bounds__(256) loss_grad_kernel(const float* Y, int ldy, const float* T,
                                                        int B, float* dY, __bf16* dYb, int ldd,
                                                        double* partial) {
  __shared__ double red[256];
  double acc = 0.0;
  const float scale = 2.0f / (float)(B * 4);
  for (long t = (long)blockIdx.x * blockDim.x + threadIdx.x; t < (long)B * ldd;
       t += (long)gridDim.x * blockDim.x) {
    const int r = (int)(t / ldd), c = (int)(t % ldd);
    float d = 0.f;
    if (c < 4) {
      const float e = Y[(long)r * ldy + c] - T[(long)r * 4 + c];
      acc += (double)e * e;
      d = scale * e;
    }
    dY[t] = d;
    dYb[t] = (__bf16)d;
  }
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) partial[blockIdx.x] = red[0];
}

// column sums of a (rows x cols) FP32 matrix into out (bias gradients)
// Sum of the split-K partials in z order: C[m][n] = sum_z part[z][m][n].
__global__ void splitk_reduce_kernel(const float* part, int ksplit, int M, int N, float* C,
                                     int ldc) {
  const long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= (long)M * N) return;
  const long mn = (long)M * N;
  float s = 0.f;
  for (int z = 0; z < ksplit; ++z) s += part[z * mn + t];
  C[(t / N) * ldc + t % N] = s;
}

// Column sums in two levels: chunk q of the rows gives part[q][c] (a block
// of 64 columns x 4 row lanes, combined in LDS), then the chunks are added
// in order.
__global__ void __launch_bounds__(256) colsum_partial_kernel(const float* a, int rows, int cols,
                                                             int lda, int chunk, float* part) {
  __shared__ float red[4][64];
  const int cl = threadIdx.x & 63, rl = threadIdx.x >> 6;
  const int c = blockIdx.x * 64 + cl;
  const int r0 = blockIdx.y * chunk, r1 = min(r0 + chunk, rows);
  float s = 0.f;
  if (c < cols)
    for (int r = r0 + rl; r < r1; r += 4) s += a[(long)r * lda + c];
  red[rl][cl] = s;
  __syncthreads();
  if (rl == 0 && c < cols)
    part[(long)blockIdx.y * cols + c] = ((red[0][cl] + red[1][cl]) + red[2][cl]) + red[3][cl];
}

__global__ void colsum_final_kernel(const float* part, int nchunk, int cols, float* out) {
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= cols) return;
  float s = 0.f;
  for (int q = 0; q < nchunk; ++q) s += part[(long)q * cols + c];
  out[c] = s;
}

// FP32 features (B x 500) -> BF16 (B x 512), zero padding
__global__ void features_to_bf16_kernel(const float* x, int B, __bf16* xb) {
  const long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= (long)B * 512) return;
  const int r = (int)(t / 512), c = (int)(t % 512);
  xb[t] = (c < 500) ? (__bf16)x[(long)r * 500 + c] : (__bf16)0.0f;
}

// Adam (Kingma & Ba) on the FP32 master parameters; refreshes the padded
// BF16 copies used by the GEMMs.
__global__ void adam_kernel(MlpParams p, const float* grad, float* m1, float* m2, int n,
                            float lr, float b1, float b2, float eps, float c1, float c2) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n) return;
  const float g = grad[t];
  const float mm = b1 * m1[t] + (1.f - b1) * g;
  const float vv = b2 * m2[t] + (1.f - b2) * g * g;
  m1[t] = mm;
  m2[t] = vv;
  const float w = p.master[t] - lr * (mm / c1) / (sqrtf(vv / c2) + eps);
  p.master[t] = w;
  mlp_write_bf16(p, t, w);
}

__global__ void refresh_bf16_kernel(MlpParams p, int n) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t < n) mlp_write_bf16(p, t, p.master[t]);
}

}  // namespace

hipError_t launch_gemm_bf16(const GemmArgs& g, hipStream_t s) {
  const int ks = g.ksplit > 1 ? g.ksplit : 1;
  if (ks > 1 && (g.epi != EPI_STORE || g.K % (ks * BK) || !g.part ||
                 (long)ks * g.M * g.N > MLP_PART_FLOATS))
    return hipErrorInvalidValue;
  GemmArgs a = g;
  a.ksplit = ks;
  if (ks == 1 && !g.transA && g.transB && g.N % NT_BN == 0 && g.K % NT_BK == 0) {
    dim3 grid(g.N / NT_BN, (g.M + NT_BM - 1) / NT_BM);
    hipLaunchKernelGGL(gemm_bf16_nt_kernel, grid, dim3(256), 0, s, a);
    return hipGetLastError();
  }
  dim3 grid((g.N + BN - 1) / BN, (g.M + BM - 1) / BM, ks);
  hipLaunchKernelGGL(gemm_bf16_kernel, grid, dim3(256), 0, s, a);
  if (ks > 1) {
    const long n = (long)g.M * g.N;
    hipLaunchKernelGGL(splitk_reduce_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s,
                       g.part, ks, g.M, g.N, g.C, g.ldc);
  }
  return hipGetLastError();
}

hipError_t launch_loss_grad(const float* Y, int ldy, const float* T, int B, float* dY, __bf16* dYb,
                            int ldd, double* partial, int nblocks, hipStream_t s) {
  hipLaunchKernelGGL(loss_grad_kernel, dim3(nblocks), dim3(256), 0, s, Y, ldy, T, B, dY, dYb, ldd,
                     partial);
  return hipGetLastError();
}

hipError_t launch_colsum(const float* a, int rows, int cols, int lda, float* out, float* part,
                         hipStream_t s) {
  int chunk = 128;
  while ((rows + chunk - 1) / chunk > COLSUM_MAX_CHUNKS) chunk *= 2;
  const int nchunk = (rows + chunk - 1) / chunk;
  hipLaunchKernelGGL(colsum_partial_kernel, dim3((cols + 63) / 64, nchunk), dim3(256), 0, s, a,
                     rows, cols, lda, chunk, part);
  hipLaunchKernelGGL(colsum_final_kernel, dim3((cols + 127) / 128), dim3(128), 0, s, part, nchunk,
                     cols, out);
  return hipGetLastError();
}

hipError_t launch_features_to_bf16(const float* x, int B, __bf16* xb, hipStream_t s) {
  const long n = (long)B * 512;
  hipLaunchKernelGGL(features_to_bf16_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s,
                     x, B, xb);
  return hipGetLastError();
}

hipError_t launch_adam(const MlpParams& p, const float* grad, float* m1, float* m2, int n, float lr,
                       int step, hipStream_t s) {
  const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
  const float c1 = 1.f - powf(b1, (float)step), c2 = 1.f - powf(b2, (float)step);
  hipLaunchKernelGGL(adam_kernel, dim3((n + 255) / 256), dim3(256), 0, s, p, grad, m1, m2, n, lr,
                     b1, b2, eps, c1, c2);
  return hipGetLastError();
}

hipError_t launch_refresh_bf16(const MlpParams& p, int n, hipStream_t s) {
  hipLaunchKernelGGL(refresh_bf16_kernel, dim3((n + 255) / 256), dim3(256), 0, s, p, n);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Closure inside the model: features from the halo-padded state, and the
// conservative flux divergence of the predicted vertical fluxes.
// ---------------------------------------------------------------------------

// xb[cell][f], f = var * 125 + (dk+2)*25 + (dj+2)*5 + (di+2), var = u, v, w, b
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

// BF16 rows of 512 (the GEMM's padded K) for the model's own closure.
template <class T>
__global__ void __launch_bounds__(256) closure_features_kernel(Dims d, const T* u, const T* v,
                                                               const T* w, const T* tt,
                                                               const T* ss, ClosureStats st,
                                                               __bf16* xb) {
  const long ncell = (long)d.nx * d.ny * d.nz;
  const long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= ncell * 512) return;
  const long cell = t >> 9;
  const int f = (int)(t & 511);
  xb[t] = (f < 500) ? (__bf16)feature_value(d, u, v, w, tt, ss, st, cell, f) : (__bf16)0.0f;
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

__device__ inline bf16x8 ldfrag(const __bf16* f, int block) {
  return *(const __attribute__((address_space(1))) bf16x8*)(f + (long)block * 512 +
                                                            (threadIdx.x & 63) * 8);
}

template <int MI, class Stage, class Out>
__device__ inline void net_rows(const MlpParams& p, __bf16* hs, const __bf16* sx, Stage& stage,
                                const Out& out) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
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
  net_rows<MI>(p, hs, hs, st, [&](int i, f32x4 c) {
    const int row = st.row0 + 16 * i + (int)(threadIdx.x & 15);
    if (row < B)
      *(__attribute__((address_space(1))) v4u<float>*)(y + (long)row * MLP_NOUT) = c;
  });
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
  net_rows<MI>(p, lds, sx, stage, [&](int i, f32x4 c) {
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
  net_rows<4>(p, hs, hs, stage, [&](int i, f32x4 c) {
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
// face.  Wall fluxes are zero.
template <class T>
__global__ void __launch_bounds__(256) closure_apply_kernel(Dims d, const float* y, ClosureStats st,
                                                            double rdz, T* gu, T* gv, T* gw,
                                                            T* gt) {
  const long ncell = (long)d.nx * d.ny * d.nz;
  const long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= ncell) return;
  const int i = (int)(t % d.nx);
  const int j = (int)((t / d.nx) % d.ny);
  const int k = (int)(t / ((long)d.nx * d.ny));
  auto F = [&](int q, int ii, int jj, int kk) -> float {
    ii = (ii + d.nx) % d.nx;
    jj = (jj + d.ny) % d.ny;
    const long c = ((long)kk * d.ny + jj) * d.nx + ii;
    return y[c * 4 + q] * st.out_std[q] + st.out_mean[q];
  };
  // flux through the z face kk (0..nz) of quantity q averaged over x or y
  auto zface = [&](int q, int ax, int kk) -> float {
    if (kk <= 0 || kk >= d.nz) return 0.f;
    if (ax == 0) return 0.25f * (F(q, i - 1, j, kk - 1) + F(q, i, j, kk - 1) + F(q, i - 1, j, kk) +
                                 F(q, i, j, kk));
    if (ax == 1) return 0.25f * (F(q, i, j - 1, kk - 1) + F(q, i, j, kk - 1) + F(q, i, j - 1, kk) +
                                 F(q, i, j, kk));
    return 0.5f * (F(q, i, j, kk - 1) + F(q, i, j, kk));
  };
  const long p = pidx(d, i, j, k);
  const float rz = (float)rdz;
  gu[p] = (T)(-(zface(0, 0, k + 1) - zface(0, 0, k)) * rz);
  gv[p] = (T)(-(zface(1, 1, k + 1) - zface(1, 1, k)) * rz);
  gt[p] = (T)(-(zface(3, 2, k + 1) - zface(3, 2, k)) * rz * st.inv_galpha);
  gw[p] = (k == 0) ? (T)0 : (T)(-(F(2, i, j, k) - F(2, i, j, k - 1)) * rz);
}

template <class T>
hipError_t launch_closure_features(const Dims& d, const T* u, const T* v, const T* w, const T* t,
                                   const T* s, ClosureStats st, __bf16* xb, hipStream_t stream) {
  const long n = (long)d.nx * d.ny * d.nz * 512;
  hipLaunchKernelGGL(closure_features_kernel<T>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0,
                     stream, d, u, v, w, t, s, st, xb);
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

template hipError_t launch_closure_features<float>(const Dims&, const float*, const float*,
                                                   const float*, const float*, const float*,
                                                   ClosureStats, __bf16*, hipStream_t);
template hipError_t launch_closure_features<double>(const Dims&, const double*, const double*,
                                                    const double*, const double*, const double*,
                                                    ClosureStats, __bf16*, hipStream_t);
template hipError_t launch_closure_apply<float>(const Dims&, const float*, ClosureStats, double,
                                                float*, float*, float*, float*, hipStream_t);
template hipError_t launch_closure_apply<double>(const Dims&, const float*, ClosureStats, double,
                                                 double*, double*, double*, double*, hipStream_t);

}  // namespace oc

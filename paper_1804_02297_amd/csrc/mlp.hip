// Stencil-prediction network on gfx950 (a project extension of Section 3).
//
// The per-point fit (pointfit.hip) makes an interior point's stencil depend on
// the medium in its 5^3 patch.  This network predicts that dependence:
//
//   x (250)  = Re, Im of m on the 5^3 patch / 0.3 (last dimension fastest, 0 off the grid)
//   h1 = GELU(x W1 + b1) (256), h2 = GELU(h1 W2 + b2) (256), y = h2 W3 + b3 (468)
//   y encodes the 26 off-centre 3x3 blocks of alpha~_i - alpha~_class, where
//   alpha~ = alpha (alpha_centre)^-1 is the gauge with the identity as centre block
//   (S^-1 Q is invariant under alpha -> alpha X, so the gauge costs nothing).
//
// Weights are FP32 masters with BF16 copies; every product runs on BF16 MFMA
// (16x16x16 in training, 16x16x32 in inference) with FP32 accumulation.
// Training runs the layers as separate products (the backward pass needs the
// pre-activations); inference fuses the three layers per tile of rows.  GELU is
// x Phi(x) with Phi from an erfc fit good to 1.5e-7 (far below the BF16
// rounding of the activations).  Loss: mean squared error; optimiser: Adam.
//
// The learned fit predicts alpha for every interior point, orthonormalises it,
// and accepts it when its locality tr(Q^H Gram_i Q) is no larger than the
// class stencil's tr(alpha_c^H Gram_i alpha_c) on the same medium-weighted
// Gram; other points fall back to the exact per-point fit.
#include <cmath>
#include <cstdio>
#include <cstring>
#include <random>
#include <string>
#include <vector>

#include "buffers.h"
#include "common.h"
#include "mlp.h"

namespace ls {

namespace {

typedef short v4s __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));

__device__ __forceinline__ unsigned short f2bf(float x) {
  unsigned u = __float_as_uint(x);
  u += 0x7FFFu + ((u >> 16) & 1u);      // round to nearest, ties to even
  return (unsigned short)(u >> 16);
}
__device__ __forceinline__ float bf2f(unsigned short b) { return __uint_as_float(((unsigned)b) << 16); }

// erfc(z) for z >= 0 to 1.5e-7 absolute, from the rational-exponential fit of
// Abramowitz and Stegun (eq. 7.1.26), and e^{-z^2} with it
__device__ __forceinline__ float erfc_pos(float z, float& ez2) {
  const float t = __builtin_amdgcn_rcpf(fmaf(0.3275911f, z, 1.0f));
  ez2 = __builtin_amdgcn_exp2f(-z * z * 1.4426950408889634f);
  const float q = fmaf(t, fmaf(t, fmaf(t, fmaf(t, 1.061405429f, -1.453152027f), 1.421413741f), -0.284496736f),
                       0.254829592f);
  return t * q * ez2;
}
// GELU(x) = x Phi(x), Phi(x) = erfc(-x / sqrt 2) / 2
__device__ __forceinline__ float gelu(float x) {
  float e;
  const float q = erfc_pos(fabsf(x) * 0.70710678118654752f, e);
  return x >= 0.f ? x * (1.0f - 0.5f * q) : 0.5f * x * q;
}
// GELU'(x) = Phi(x) + x phi(x)
__device__ __forceinline__ float gelu_grad(float x) {
  float e;
  const float q = erfc_pos(fabsf(x) * 0.70710678118654752f, e);
  return (x >= 0.f ? 1.0f - 0.5f * q : 0.5f * q) + x * e * 0.39894228040143268f;
}

enum Epi { EPI_STORE = 0, EPI_HIDDEN = 1, EPI_OUT = 2, EPI_DACT = 3 };

struct EpiArgs {
  const float* bias;       // EPI_HIDDEN, EPI_OUT
  float* zf;               // EPI_HIDDEN: pre-activation out; EPI_DACT: dZ (f32) out
  const float* zin;        // EPI_DACT: the forward pre-activation
  unsigned short* hb;      // EPI_HIDDEN: GELU(z) as bf16; EPI_DACT: dZ as bf16
  float* cf;               // EPI_STORE / EPI_OUT
  int ld;                  // leading dimension of every output (row-major, M x ld)
  int nvalid;              // columns >= nvalid are written as zero (padding)
};

// C (M x N) = A (M x K) B (K x N), BF16 operands, FP32 accumulation.
// A(m, k) = TA ? A[k lda + m] : A[m lda + k];  B(k, n) = TB ? B[n ldb + k] : B[k ldb + n].
// Workgroup: 4 waves, 64 x 64 output tile, K in steps of 32 through LDS; each
// operand is read along its contiguous index (consecutive threads, consecutive
// addresses).  Split K (EPI_STORE only): workgroup z of gridDim.z takes the K
// range [z Kc, (z + 1) Kc) and writes its partial sums to cf + z M ld.
template <bool TA, bool TB, int EPI>
__global__ __launch_bounds__(256) void gemm_bf16_kernel(const unsigned short* __restrict__ A, int lda,
                                                        const unsigned short* __restrict__ B, int ldb, int M, int N,
                                                        int K, EpiArgs ep) {
  __shared__ unsigned short As[64][32 + 4];   // [m][k]
  __shared__ unsigned short Bs[64][32 + 4];   // [n][k]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int m0 = blockIdx.y * 64, n0 = blockIdx.x * 64;
  const int wm = (wave >> 1) * 32, wn = (wave & 1) * 32;
  const int Kc = (K + (int)gridDim.z - 1) / (int)gridDim.z;
  const int kbeg = (int)blockIdx.z * Kc, kend = min(K, kbeg + Kc);
  v4f acc[2][2];
  for (int a = 0; a < 2; ++a)
    for (int b = 0; b < 2; ++b) acc[a][b] = v4f{0.f, 0.f, 0.f, 0.f};
  for (int k0 = kbeg; k0 < kend; k0 += 32) {
    for (int e = tid; e < 64 * 32; e += 256) {
      // A: m fastest when A is stored k-major (TA), else k fastest; B likewise
      const int ra = TA ? e % 64 : e / 32, ca = TA ? e / 64 : e % 32;
      const int rb = TB ? e / 32 : e % 64, cb = TB ? e % 32 : e / 64;
      const int m = m0 + ra, ka = k0 + ca, n = n0 + rb, kb = k0 + cb;
      unsigned short av = 0, bv = 0;
      if (m < M && ka < kend) av = TA ? A[(long)ka * lda + m] : A[(long)m * lda + ka];
      if (n < N && kb < kend) bv = TB ? B[(long)n * ldb + kb] : B[(long)kb * ldb + n];
      As[ra][ca] = av;
      Bs[rb][cb] = bv;
    }
    __syncthreads();
#pragma unroll
    for (int ks = 0; ks < 32; ks += 16) {
      v4s af[2], bfr[2];
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const int kk = ks + 4 * (lane >> 4);
        const int ra = wm + 16 * t + (lane & 15);
        const int rb = wn + 16 * t + (lane & 15);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          af[t][q] = (short)As[ra][kk + q];
          bfr[t][q] = (short)Bs[rb][kk + q];
        }
      }
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(af[a], bfr[b], acc[a][b], 0, 0, 0);
    }
    __syncthreads();
  }
  // D[4 (l / 16) + r][l % 16] in register r of lane l
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = m0 + wm + 16 * a + 4 * (lane >> 4) + r;
        const int n = n0 + wn + 16 * b + (lane & 15);
        if (m >= M || n >= N) continue;
        const long o = (long)m * ep.ld + n + (long)blockIdx.z * M * ep.ld;
        const bool pad = n >= ep.nvalid;
        float v = acc[a][b][r];
        if (EPI == EPI_STORE) {
          ep.cf[o] = pad ? 0.f : v;
        } else if (EPI == EPI_OUT) {
          ep.cf[o] = pad ? 0.f : v + ep.bias[n];
        } else if (EPI == EPI_HIDDEN) {
          const float z = pad ? 0.f : v + ep.bias[n];
          ep.zf[o] = z;
          ep.hb[o] = pad ? 0 : f2bf(gelu(z));
        } else {   // EPI_DACT
          const float d = pad ? 0.f : v * gelu_grad(ep.zin[o]);
          ep.zf[o] = d;
          ep.hb[o] = f2bf(d);
        }
      }
}

template <bool TA, bool TB, int EPI>
ls_status gemm(const unsigned short* A, int lda, const unsigned short* B, int ldb, int M, int N, int K,
               const EpiArgs& ep, hipStream_t s, int splitk = 1) {
  if (splitk > 1 && EPI != EPI_STORE) return LS_EINVAL;
  dim3 grid((N + 63) / 64, (M + 63) / 64, splitk);
  hipLaunchKernelGGL((gemm_bf16_kernel<TA, TB, EPI>), grid, dim3(256), 0, s, A, lda, B, ldb, M, N, K, ep);
  return hipGetLastError() == hipSuccess ? LS_OK : LS_EHIP;
}

__global__ void f32_to_bf16_kernel(const float* __restrict__ a, unsigned short* __restrict__ b, long cnt) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < cnt) b[i] = f2bf(a[i]);
}

// copy an r x c FP32 block into a zero-padded R x Cp BF16 block (row-major)
__global__ void pad_bf16_kernel(const float* __restrict__ a, int r, int c, unsigned short* __restrict__ b, int R,
                                int Cp) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (long)R * Cp) return;
  const int row = (int)(i / Cp), col = (int)(i % Cp);
  b[i] = (row < r && col < c) ? f2bf(a[(long)row * c + col]) : (unsigned short)0;
}

// dY = 2 (Y - T) / (B * 468), padded columns zero; the block's sum of squared
// errors goes to sq[block % 256] (one atomic per block)
__global__ __launch_bounds__(256) void loss_grad_kernel(const float* __restrict__ Y, const float* __restrict__ T,
                                                        int Bm, float inv, unsigned short* __restrict__ dYb,
                                                        float* __restrict__ sq) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  float d = 0.f;
  if (i < (long)Bm * MLP_OP) {
    const int n = (int)(i % MLP_OP);
    const long m = i / MLP_OP;
    if (n < MLP_O) d = Y[i] - T[m * MLP_O + n];
    dYb[i] = f2bf(2.0f * d * inv);
  }
  float e = d * d;
  for (int o = 32; o > 0; o >>= 1) e += __shfl_xor(e, o);
  __shared__ float red[4];
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = e;
  __syncthreads();
  if (threadIdx.x == 0) atomicAdd(&sq[blockIdx.x % 256], red[0] + red[1] + red[2] + red[3]);
}

// Column sums in two deterministic stages.  Stage 1: part[c][n] = sum over
// the rows m of chunk c of (A[m][n] - B[m][n]) (B may be null); a block is 64
// columns x 4 row phases, blockIdx.y the chunk.  Stage 2: out[n] = scale sum_c.
constexpr int kColChunks = 32;
__global__ __launch_bounds__(256) void colsum_partial_kernel(const float* __restrict__ A, int lda,
                                                             const float* __restrict__ B, int ldb, int rows,
                                                             int cols, float* __restrict__ part) {
  const int cx = threadIdx.x & 63, ry = threadIdx.x >> 6;
  const int n = blockIdx.x * 64 + cx;
  const int per = (rows + kColChunks - 1) / kColChunks;
  const int m0 = blockIdx.y * per, m1 = min(rows, m0 + per);
  float acc = 0.f;
  if (n < cols)
    for (int m = m0 + ry; m < m1; m += 4) acc += A[(long)m * lda + n] - (B ? B[(long)m * ldb + n] : 0.f);
  __shared__ float red[4][64];
  red[ry][cx] = acc;
  __syncthreads();
  if (ry == 0 && n < cols) part[(long)blockIdx.y * cols + n] = red[0][cx] + red[1][cx] + red[2][cx] + red[3][cx];
}

__global__ void colsum_final_kernel(const float* __restrict__ part, int cols, float scale, float* __restrict__ out) {
  const int n = blockIdx.x * blockDim.x + threadIdx.x;
  if (n >= cols) return;
  float acc = 0.f;
  for (int c = 0; c < kColChunks; ++c) acc += part[(long)c * cols + n];
  out[n] = scale * acc;
}

static ls_status colsum(const float* A, int lda, const float* B, int ldb, int rows, int cols, float scale,
                        float* part, float* out, hipStream_t s) {
  hipLaunchKernelGGL(colsum_partial_kernel, dim3((cols + 63) / 64, kColChunks), dim3(256), 0, s, A, lda, B, ldb, rows,
                     cols, part);
  hipLaunchKernelGGL(colsum_final_kernel, dim3((cols + 255) / 256), dim3(256), 0, s, part, cols, scale, out);
  return hipGetLastError() == hipSuccess ? LS_OK : LS_EHIP;
}

// gather a row-major block of FP32 dW (rows x cols, ld) into the flat gradient,
// summing the nsplit split-K partial blocks (each Mfull x ld) in order
__global__ void gather_grad_kernel(const float* __restrict__ src, int rows, int cols, int ld, int Mfull, int nsplit,
                                   float* __restrict__ dst) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (long)rows * cols) return;
  const long o = (i / cols) * ld + i % cols;
  float v = 0.f;
  for (int z = 0; z < nsplit; ++z) v += src[o + (long)z * Mfull * ld];
  dst[i] = v;
}
// split of the batch dimension in the weight-gradient products (K = batch rows):
// 16-32 output tiles alone leave most of the chip idle
constexpr int kGradSplit = 8;

__global__ void adam_kernel(float* __restrict__ w, const float* __restrict__ g, float* __restrict__ m,
                            float* __restrict__ v, long cnt, float lr, float b1, float b2, float eps, float c1,
                            float c2) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= cnt) return;
  const float gi = g[i];
  const float mi = b1 * m[i] + (1.f - b1) * gi;
  const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  w[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}


// ---- inference: the three layers fused per tile of rows ------------------------
// y (rows x 480, FP32) = W3^T GELU(W2^T GELU(W1^T x + b1) + b2) + b3 for FR rows
// per workgroup of IW waves.  The tile's activations stay in LDS (BF16, as the
// separate layers round them); the weights stream from L2 in copies laid out
// in MFMA fragment order, so the 64 lanes' B operands of one 16-column tile
// and one k step are 1 KB contiguous (whole lines per load).  A wave owns two
// column tiles at a time and loads the fragments of its next pair while it
// multiplies the current one.  Products on v_mfma_f32_16x16x32_bf16: lane l
// gives A[l % 16][8 (l / 16) + j] and B[8 (l / 16) + j][l % 16], j < 8, and
// receives D[4 (l / 16) + r][l % 16], r < 4.  Every layer has K = 256.
constexpr int FR = 32;                 // rows per workgroup
constexpr int FRT = FR / 16;           // 16-row tiles per workgroup
constexpr int FLD = MLP_IP + 8;        // LDS row stride (bf16): 528 bytes, spreads the banks
constexpr int IW = 8;                  // waves per workgroup
constexpr int KS = MLP_IP / 32;        // k steps per product
constexpr int CTP = 2;                 // column tiles per wave and step
static_assert(MLP_H == MLP_IP, "every inference product has K = 256");

typedef __bf16 v8bf __attribute__((ext_vector_type(8)));

// wf[((nt KS + ks) 64 + l) 8 + j] = wb[(32 ks + 8 (l / 16) + j) N + 16 nt + l % 16]
// for a K = 256 by N row-major BF16 weight (N a multiple of 16)
__global__ void frag_bf16_kernel(const unsigned short* __restrict__ wb, int N, unsigned short* __restrict__ wf) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (long)MLP_IP * N) return;
  const int j = (int)(i & 7), l = (int)((i >> 3) & 63);
  const long f = i >> 9;
  const int ks = (int)(f % KS), nt = (int)(f / KS);
  wf[i] = wb[(long)(32 * ks + 8 * (l >> 4) + j) * N + 16 * nt + (l & 15)];
}

struct Frags {
  uint4 b[CTP][KS];
};

// the fragments of column tiles nt0 and nt0 + IW (zero past nct)
__device__ __forceinline__ void load_pair(Frags& F, const uint4* __restrict__ wf, int nt0, int nct, int lane) {
#pragma unroll
  for (int u = 0; u < CTP; ++u) {
    const int nt = nt0 + u * IW;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
      F.b[u][ks] = nt < nct ? wf[(nt * KS + ks) * 64 + lane] : uint4{0u, 0u, 0u, 0u};
  }
}

// the biases of column tiles nt0 and nt0 + IW at this lane's column (0 past nout)
__device__ __forceinline__ void load_bias(float* bn, const float* __restrict__ bias, int nt0, int nout, int lane) {
#pragma unroll
  for (int u = 0; u < CTP; ++u) {
    const int n = 16 * (nt0 + u * IW) + (lane & 15);
    bn[u] = n < nout ? bias[n] : 0.f;
  }
}

template <bool HIDDEN>
__device__ __forceinline__ void infer_pair(const Frags& F, const float* bn, const unsigned short* __restrict__ hin,
                                           unsigned short* __restrict__ hout, float* __restrict__ y, int r0, int Bm,
                                           int nt0, int nct, int lane) {
  v4f acc[FRT][CTP];
#pragma unroll
  for (int a = 0; a < FRT; ++a)
#pragma unroll
    for (int u = 0; u < CTP; ++u) acc[a][u] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    const int kk = 32 * ks + 8 * (lane >> 4);
    uint4 af[FRT];
#pragma unroll
    for (int a = 0; a < FRT; ++a) af[a] = *reinterpret_cast<const uint4*>(hin + (16 * a + (lane & 15)) * FLD + kk);
#pragma unroll
    for (int a = 0; a < FRT; ++a)
#pragma unroll
      for (int u = 0; u < CTP; ++u)
        acc[a][u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, af[a]),
                                                            __builtin_bit_cast(v8bf, F.b[u][ks]), acc[a][u], 0, 0,
                                                            0);
  }
#pragma unroll
  for (int u = 0; u < CTP; ++u) {
    const int nt = nt0 + u * IW;
    if (nt >= nct) continue;
    const int n = 16 * nt + (lane & 15);
#pragma unroll
    for (int a = 0; a < FRT; ++a)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = 16 * a + 4 * (lane >> 4) + r;
        if (HIDDEN) {
          hout[row * FLD + n] = f2bf(gelu(acc[a][u][r] + bn[u]));
        } else if (r0 + row < Bm) {
          y[(long)(r0 + row) * MLP_OP + n] = (n < MLP_O) ? acc[a][u][r] + bn[u] : 0.f;
        }
      }
  }
}

__global__ __launch_bounds__(64 * IW) void mlp_infer_kernel(const unsigned short* __restrict__ xb, int Bm,
                                                            const uint4* __restrict__ w1f,
                                                            const uint4* __restrict__ w2f,
                                                            const uint4* __restrict__ w3f,
                                                            const float* __restrict__ b1,
                                                            const float* __restrict__ b2,
                                                            const float* __restrict__ b3, float* __restrict__ y) {
  __shared__ __attribute__((aligned(16))) unsigned short hs[2][FR * FLD];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r0 = blockIdx.x * FR;
  // the tile's inputs, 16 bytes per load; rows past Bm are zero
  constexpr int XL = FR * (MLP_IP / 8) / (64 * IW);
  static_assert(XL * 64 * IW == FR * (MLP_IP / 8), "the input tile splits evenly over the threads");
  uint4 xv[XL];
#pragma unroll
  for (int q = 0; q < XL; ++q) {
    const int e = tid + 64 * IW * q, r = e / (MLP_IP / 8), c = e % (MLP_IP / 8);
    xv[q] = r0 + r < Bm ? *reinterpret_cast<const uint4*>(xb + (long)(r0 + r) * MLP_IP + 8 * c)
                        : uint4{0u, 0u, 0u, 0u};
  }
  // every bias this wave adds, loaded before the weights so that no wait for
  // a bias also waits for the weight fragments in flight
  float bs[4][CTP];
  load_bias(bs[0], b1, wave, MLP_H, lane);
  load_bias(bs[1], b2, wave, MLP_H, lane);
  load_bias(bs[2], b3, wave, MLP_O, lane);
  load_bias(bs[3], b3, wave + 2 * IW, MLP_O, lane);
  Frags P, Q;
  load_pair(P, w1f, wave, MLP_H / 16, lane);                // layer 1: tiles wave, wave + 8
#pragma unroll
  for (int q = 0; q < XL; ++q) {
    const int e = tid + 64 * IW * q, r = e / (MLP_IP / 8), c = e % (MLP_IP / 8);
    *reinterpret_cast<uint4*>(&hs[0][r * FLD + 8 * c]) = xv[q];
  }
  __syncthreads();
  load_pair(Q, w2f, wave, MLP_H / 16, lane);                // layer 2, loaded during layer 1
  infer_pair<true>(P, bs[0], hs[0], hs[1], nullptr, r0, Bm, wave, MLP_H / 16, lane);
  __syncthreads();
  load_pair(P, w3f, wave, MLP_OP / 16, lane);               // layer 3: tiles wave, wave + 8
  infer_pair<true>(Q, bs[1], hs[1], hs[0], nullptr, r0, Bm, wave, MLP_H / 16, lane);
  __syncthreads();
  load_pair(Q, w3f, wave + 2 * IW, MLP_OP / 16, lane);      // tiles wave + 16, wave + 24 (< 30)
  infer_pair<false>(P, bs[2], hs[0], nullptr, y, r0, Bm, wave, MLP_OP / 16, lane);
  infer_pair<false>(Q, bs[3], hs[0], nullptr, y, r0, Bm, wave + 2 * IW, MLP_OP / 16, lane);
}

inline unsigned nbk(long len, int t) { return (unsigned)((len + t - 1) / t); }

}  // namespace

// ---- host side ----------------------------------------------------------------

ls_status mlp_init(MlpState& st, const float* params_host, hipStream_t s) {
  LS_TRY(st.w.alloc(MLP_NPARAM * sizeof(float)));
  LS_TRY(st.m.alloc(MLP_NPARAM * sizeof(float)));
  LS_TRY(st.v.alloc(MLP_NPARAM * sizeof(float)));
  LS_TRY(st.grad.alloc(MLP_NPARAM * sizeof(float)));
  LS_TRY(st.w1b.alloc((size_t)MLP_IP * MLP_H * 2));
  LS_TRY(st.w2b.alloc((size_t)MLP_H * MLP_H * 2));
  LS_TRY(st.w3b.alloc((size_t)MLP_H * MLP_OP * 2));
  LS_HIP(hipMemcpyAsync(st.w.p, params_host, MLP_NPARAM * sizeof(float), hipMemcpyHostToDevice, s));
  LS_HIP(hipMemsetAsync(st.m.p, 0, st.m.bytes, s));
  LS_HIP(hipMemsetAsync(st.v.p, 0, st.v.bytes, s));
  LS_HIP(hipMemsetAsync(st.grad.p, 0, st.grad.bytes, s));
  st.t = 0;
  st.have_grad = false;
  return mlp_refresh_bf16(st, s);
}

ls_status mlp_refresh_bf16(MlpState& st, hipStream_t s) {
  const float* w = st.w.as<float>();
  hipLaunchKernelGGL(pad_bf16_kernel, dim3(nbk((long)MLP_IP * MLP_H, 256)), dim3(256), 0, s, w + MLP_OFF_W1, MLP_I,
                     MLP_H, st.w1b.as<unsigned short>(), MLP_IP, MLP_H);
  hipLaunchKernelGGL(pad_bf16_kernel, dim3(nbk((long)MLP_H * MLP_H, 256)), dim3(256), 0, s, w + MLP_OFF_W2, MLP_H,
                     MLP_H, st.w2b.as<unsigned short>(), MLP_H, MLP_H);
  hipLaunchKernelGGL(pad_bf16_kernel, dim3(nbk((long)MLP_H * MLP_OP, 256)), dim3(256), 0, s, w + MLP_OFF_W3, MLP_H,
                     MLP_O, st.w3b.as<unsigned short>(), MLP_H, MLP_OP);
  LS_HIP(hipGetLastError());
  ++st.wver;                           // the fragment-ordered inference copies are stale
  return LS_OK;
}

ls_status mlp_infer(MlpState& st, const unsigned short* xb, int Bm, hipStream_t s) {
  LS_TRY(mlp_workspace(st, Bm));
  if (st.fver != st.wver) {
    if (!st.w1f.p)
      LS_TRY(alloc_all<DevBuf>({{&st.w1f, (size_t)MLP_IP * MLP_H * 2},
                                {&st.w2f, (size_t)MLP_H * MLP_H * 2},
                                {&st.w3f, (size_t)MLP_H * MLP_OP * 2}}));
    hipLaunchKernelGGL(frag_bf16_kernel, dim3(nbk((long)MLP_IP * MLP_H, 256)), dim3(256), 0, s,
                       st.w1b.as<unsigned short>(), MLP_H, st.w1f.as<unsigned short>());
    hipLaunchKernelGGL(frag_bf16_kernel, dim3(nbk((long)MLP_H * MLP_H, 256)), dim3(256), 0, s,
                       st.w2b.as<unsigned short>(), MLP_H, st.w2f.as<unsigned short>());
    hipLaunchKernelGGL(frag_bf16_kernel, dim3(nbk((long)MLP_H * MLP_OP, 256)), dim3(256), 0, s,
                       st.w3b.as<unsigned short>(), MLP_OP, st.w3f.as<unsigned short>());
    LS_HIP(hipGetLastError());
    st.fver = st.wver;
  }
  const float* w = st.w.as<float>();
  hipLaunchKernelGGL(mlp_infer_kernel, dim3(nbk(Bm, FR)), dim3(64 * IW), 0, s, xb, Bm, st.w1f.as<uint4>(),
                     st.w2f.as<uint4>(), st.w3f.as<uint4>(), w + MLP_OFF_B1, w + MLP_OFF_B2, w + MLP_OFF_B3,
                     st.y.as<float>());
  LS_HIP(hipGetLastError());
  return LS_OK;
}

ls_status mlp_workspace(MlpState& st, int Bm) {
  if (st.ws_rows >= Bm) return LS_OK;
  st.ws_rows = 0;                      // until all are there
  LS_TRY(alloc_all<DevBuf>({{&st.z1, (size_t)Bm * MLP_H * 4},
                            {&st.z2, (size_t)Bm * MLP_H * 4},
                            {&st.h1b, (size_t)Bm * MLP_H * 2},
                            {&st.h2b, (size_t)Bm * MLP_H * 2},
                            {&st.y, (size_t)Bm * MLP_OP * 4},
                            {&st.dyb, (size_t)Bm * MLP_OP * 2},
                            {&st.dz2, (size_t)Bm * MLP_H * 4},
                            {&st.dz2b, (size_t)Bm * MLP_H * 2},
                            {&st.dz1, (size_t)Bm * MLP_H * 4},
                            {&st.dz1b, (size_t)Bm * MLP_H * 2},
                            {&st.dw, (size_t)kGradSplit * MLP_IP * MLP_OP * 4},
                            {&st.sq, (size_t)256 * 4},
                            {&st.part, (size_t)kColChunks * MLP_OP * 4}}));
  st.ws_rows = Bm;
  return LS_OK;
}

// y (Bm x 480, FP32) for inputs xb (Bm x 256, BF16)
ls_status mlp_forward(MlpState& st, const unsigned short* xb, int Bm, hipStream_t s) {
  LS_TRY(mlp_workspace(st, Bm));
  const float* w = st.w.as<float>();
  EpiArgs e1{w + MLP_OFF_B1, st.z1.as<float>(), nullptr, st.h1b.as<unsigned short>(), nullptr, MLP_H, MLP_H};
  LS_TRY((gemm<false, false, EPI_HIDDEN>(xb, MLP_IP, st.w1b.as<unsigned short>(), MLP_H, Bm, MLP_H, MLP_IP, e1, s)));
  EpiArgs e2{w + MLP_OFF_B2, st.z2.as<float>(), nullptr, st.h2b.as<unsigned short>(), nullptr, MLP_H, MLP_H};
  LS_TRY((gemm<false, false, EPI_HIDDEN>(st.h1b.as<unsigned short>(), MLP_H, st.w2b.as<unsigned short>(), MLP_H, Bm,
                                         MLP_H, MLP_H, e2, s)));
  EpiArgs e3{w + MLP_OFF_B3, nullptr, nullptr, nullptr, st.y.as<float>(), MLP_OP, MLP_O};
  LS_TRY((gemm<false, false, EPI_OUT>(st.h2b.as<unsigned short>(), MLP_H, st.w3b.as<unsigned short>(), MLP_OP, Bm,
                                      MLP_OP, MLP_H, e3, s)));
  return LS_OK;
}

// gradients of the mean squared error into st.grad (flat, like the parameters)
ls_status mlp_backward(MlpState& st, const unsigned short* xb, const float* T, int Bm, double* loss, hipStream_t s) {
  const float* w = st.w.as<float>();
  float* g = st.grad.as<float>();
  LS_HIP(hipMemsetAsync(st.sq.p, 0, 256 * 4, s));
  hipLaunchKernelGGL(loss_grad_kernel, dim3(nbk((long)Bm * MLP_OP, 256)), dim3(256), 0, s, st.y.as<float>(), T, Bm,
                     1.0f / ((float)Bm * MLP_O), st.dyb.as<unsigned short>(), st.sq.as<float>());
  LS_HIP(hipGetLastError());
  // layer 3: dW3 = h2^T dY (256 x 468), db3, dh2 = dY W3^T -> dZ2
  EpiArgs es{nullptr, nullptr, nullptr, nullptr, st.dw.as<float>(), MLP_OP, MLP_O};
  LS_TRY((gemm<true, false, EPI_STORE>(st.h2b.as<unsigned short>(), MLP_H, st.dyb.as<unsigned short>(), MLP_OP, MLP_H,
                                       MLP_OP, Bm, es, s, kGradSplit)));
  hipLaunchKernelGGL(gather_grad_kernel, dim3(nbk((long)MLP_H * MLP_O, 256)), dim3(256), 0, s, st.dw.as<float>(), MLP_H,
                     MLP_O, MLP_OP, MLP_H, kGradSplit, g + MLP_OFF_W3);
  // db3 from dY: reuse dz2 (f32) as scratch is not possible (bf16 dY); recompute from Y - T
  EpiArgs ed2{nullptr, st.dz2.as<float>(), st.z2.as<float>(), st.dz2b.as<unsigned short>(), nullptr, MLP_H, MLP_H};
  LS_TRY((gemm<false, true, EPI_DACT>(st.dyb.as<unsigned short>(), MLP_OP, st.w3b.as<unsigned short>(), MLP_OP, Bm,
                                      MLP_H, MLP_OP, ed2, s)));
  // layer 2
  es.cf = st.dw.as<float>();
  es.ld = MLP_H;
  es.nvalid = MLP_H;
  LS_TRY((gemm<true, false, EPI_STORE>(st.h1b.as<unsigned short>(), MLP_H, st.dz2b.as<unsigned short>(), MLP_H, MLP_H,
                                       MLP_H, Bm, es, s, kGradSplit)));
  hipLaunchKernelGGL(gather_grad_kernel, dim3(nbk((long)MLP_H * MLP_H, 256)), dim3(256), 0, s, st.dw.as<float>(), MLP_H,
                     MLP_H, MLP_H, MLP_H, kGradSplit, g + MLP_OFF_W2);
  LS_TRY(colsum(st.dz2.as<float>(), MLP_H, nullptr, 0, Bm, MLP_H, 1.0f, st.part.as<float>(), g + MLP_OFF_B2, s));
  EpiArgs ed1{nullptr, st.dz1.as<float>(), st.z1.as<float>(), st.dz1b.as<unsigned short>(), nullptr, MLP_H, MLP_H};
  LS_TRY((gemm<false, true, EPI_DACT>(st.dz2b.as<unsigned short>(), MLP_H, st.w2b.as<unsigned short>(), MLP_H, Bm,
                                      MLP_H, MLP_H, ed1, s)));
  // layer 1
  es.cf = st.dw.as<float>();
  LS_TRY((gemm<true, false, EPI_STORE>(xb, MLP_IP, st.dz1b.as<unsigned short>(), MLP_H, MLP_IP, MLP_H, Bm, es, s,
                                       kGradSplit)));
  hipLaunchKernelGGL(gather_grad_kernel, dim3(nbk((long)MLP_I * MLP_H, 256)), dim3(256), 0, s, st.dw.as<float>(), MLP_I,
                     MLP_H, MLP_H, MLP_IP, kGradSplit, g + MLP_OFF_W1);
  LS_TRY(colsum(st.dz1.as<float>(), MLP_H, nullptr, 0, Bm, MLP_H, 1.0f, st.part.as<float>(), g + MLP_OFF_B1, s));
  LS_HIP(hipGetLastError());
  // db3 = column sums of dY in FP32: dY = 2 (Y - T) / (B 468)
  LS_TRY(mlp_bias3_grad(st, T, Bm, g + MLP_OFF_B3, s));
  if (loss) {
    float sq[256];
    LS_HIP(hipMemcpyAsync(sq, st.sq.p, sizeof(sq), hipMemcpyDeviceToHost, s));
    LS_HIP(hipStreamSynchronize(s));
    double t = 0.0;
    for (int i = 0; i < 256; ++i) t += sq[i];
    *loss = t / ((double)Bm * MLP_O);
  }
  st.have_grad = true;
  return LS_OK;
}

ls_status mlp_bias3_grad(MlpState& st, const float* T, int Bm, float* db, hipStream_t s) {
  return colsum(st.y.as<float>(), MLP_OP, T, MLP_O, Bm, MLP_O, 2.0f / ((float)Bm * MLP_O), st.part.as<float>(), db, s);
}

ls_status mlp_adam(MlpState& st, double lr, hipStream_t s) {
  st.t += 1;
  const float b1 = 0.9f, b2 = 0.999f;
  const float c1 = 1.0f - powf(b1, (float)st.t), c2 = 1.0f - powf(b2, (float)st.t);
  hipLaunchKernelGGL(adam_kernel, dim3(nbk(MLP_NPARAM, 256)), dim3(256), 0, s, st.w.as<float>(), st.grad.as<float>(),
                     st.m.as<float>(), st.v.as<float>(), (long)MLP_NPARAM, (float)lr, b1, b2, 1e-8f, c1, c2);
  LS_HIP(hipGetLastError());
  return mlp_refresh_bf16(st, s);
}

}  // namespace ls

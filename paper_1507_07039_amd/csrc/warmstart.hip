// Kernels of the learned warm start (not in the paper): per-edge features
// of the priors, the 16-64-64-1 MLP (inference, gradient, Adam) and the
// target / prediction maps.  The MLP runs on bf16 matrix cores with FP32
// accumulation; feature statistics and the sketch bases are FP64.
//
// MLP layout.  A wave handles 32 edges at a time with both layers computed
// transposed (Z^T = W X^T), so each lane owns one edge (lane % 32) and the
// 32 x 32 result layout of v_mfma_f32_32x32x16_bf16 puts hidden units in the
// lane's registers: unit(b, r, h) = 32 b + 8 (r / 4) + 4 h + r % 4 for output
// block b, register r and lane half h = lane / 32.  The next contraction over
// those 64 units is issued in k-steps s whose element e (of lane half h) is
// the lane's own register (b = s / 2, r = 8 (s % 2) + e); the weight operand
// is gathered in the matching unit order, so activations never leave the
// registers in the forward pass.  The weight gradients contract over edges:
// they go through a per-wave LDS transpose ([unit][edge]) into accumulators
// that live across all of the wave's edges; bias gradients come from a
// constant-one column of the same products.
#include "warm_internal.h"

namespace panda {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float f4 __attribute__((ext_vector_type(4)));

constexpr int kT = 256;           // threads per block
constexpr int kWaves = kT / 64;
constexpr int NF = kMlpFeatures;  // 16
constexpr int NH = kMlpHidden;    // 64

__device__ __forceinline__ int unit_of(int b, int r, int h) {
  return 32 * b + 8 * (r >> 2) + 4 * h + (r & 3);
}
__device__ __forceinline__ int kunit(int s, int h, int e) {
  return unit_of(s >> 1, 8 * (s & 1) + e, h);
}
__device__ __forceinline__ __bf16 bq(float x) { return (__bf16)x; }
__device__ __forceinline__ float fq(__bf16 x) { return (float)x; }

// Weights of one block in LDS: bf16 matrices, FP32 biases, bf16-rounded w3.
struct MlpShared {
  alignas(16) __bf16 W1[NH][NF];
  alignas(16) __bf16 W2[NH][NH];
  float b1[NH], b2[NH], w3[NH];
  float b3;
};

__device__ __forceinline__ void load_params(const float* __restrict__ p, MlpShared& sm) {
  for (int i = threadIdx.x; i < NH * NF; i += kT) sm.W1[i / NF][i % NF] = bq(p[kOffW1 + i]);
  for (int i = threadIdx.x; i < NH * NH; i += kT) sm.W2[i / NH][i % NH] = bq(p[kOffW2 + i]);
  for (int i = threadIdx.x; i < NH; i += kT) {
    sm.b1[i] = p[kOffB1 + i];
    sm.b2[i] = p[kOffB2 + i];
    sm.w3[i] = fq(bq(p[kOffW3 + i]));
  }
  if (threadIdx.x == 0) sm.b3 = p[kOffB3];
  __syncthreads();
}

// Weight operands of one wave (constant over its edges).
struct MlpOps {
  bf16x8 A1[2];     // W1 rows 32 mb + lane%32, features 8h..8h+7
  bf16x8 A2[2][4];  // W2 rows 32 mb + lane%32, k-step s in the unit order above
  __device__ __forceinline__ void build(const MlpShared& sm, int lane) {
    const int h = lane >> 5, m = lane & 31;
#pragma unroll
    for (int mb = 0; mb < 2; ++mb) {
#pragma unroll
      for (int e = 0; e < 8; ++e) A1[mb][e] = sm.W1[32 * mb + m][8 * h + e];
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int e = 0; e < 8; ++e) A2[mb][s][e] = sm.W2[32 * mb + m][kunit(s, h, e)];
    }
  }
};

// Forward pass of the 32 edges of one wave; lane = (edge lane%32, half h).
struct MlpFwd {
  bf16x8 x;           // features 8h..8h+7 of the lane's edge (bf16)
  floatx16 z1[2];     // layer-1 pre-activations (without bias)
  bf16x8 h1[4];       // bf16 activations in k-step order
  floatx16 z2[2];     // layer-2 pre-activations (with bias after run)
  float y;
  __device__ __forceinline__ void run(const MlpShared& sm, const MlpOps& op, const float* __restrict__ F,
                                      int64_t row, bool valid, int lane) {
    const int h = lane >> 5;
    if (valid) {
      const f4 a = *reinterpret_cast<const f4*>(F + row * NF + 8 * h);
      const f4 b = *reinterpret_cast<const f4*>(F + row * NF + 8 * h + 4);
      x[0] = bq(a.x); x[1] = bq(a.y); x[2] = bq(a.z); x[3] = bq(a.w);
      x[4] = bq(b.x); x[5] = bq(b.y); x[6] = bq(b.z); x[7] = bq(b.w);
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) x[e] = bq(0.0f);
    }
#pragma unroll
    for (int mb = 0; mb < 2; ++mb) {
      floatx16 zero;
#pragma unroll
      for (int r = 0; r < 16; ++r) zero[r] = 0.0f;
      z1[mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(op.A1[mb], x, zero, 0, 0, 0);
    }
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        z1[b][r] += sm.b1[unit_of(b, r, h)];
        const float v = z1[b][r] > 0.0f ? z1[b][r] : 0.0f;
        h1[2 * b + (r >> 3)][r & 7] = bq(v);
      }
#pragma unroll
    for (int mb = 0; mb < 2; ++mb) {
#pragma unroll
      for (int r = 0; r < 16; ++r) z2[mb][r] = 0.0f;
#pragma unroll
      for (int s = 0; s < 4; ++s)
        z2[mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(op.A2[mb][s], h1[s], z2[mb], 0, 0, 0);
    }
    float part = 0.0f;
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int u = unit_of(b, r, h);
        z2[b][r] += sm.b2[u];
        part += sm.w3[u] * (z2[b][r] > 0.0f ? z2[b][r] : 0.0f);
      }
    y = part + __shfl_xor(part, 32) + sm.b3;
  }
};

// y for n feature rows.  Grid-stride over 32-edge chunks, one per wave.
__global__ __launch_bounds__(kT) void k_mlp_forward(const float* __restrict__ p,
                                                    const float* __restrict__ F, int64_t n,
                                                    float* __restrict__ y) {
  __shared__ MlpShared sm;
  load_params(p, sm);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  MlpOps op;
  op.build(sm, lane);
  const int64_t chunks = (n + 31) / 32;
  for (int64_t c = (int64_t)blockIdx.x * kWaves + wave; c < chunks;
       c += (int64_t)gridDim.x * kWaves) {
    const int64_t row = c * 32 + (lane & 31);
    MlpFwd f;
    f.run(sm, op, F, row, row < n, lane);
    if (lane < 32 && row < n) y[row] = f.y;
  }
}

// Gradient of the mean squared error over a batch of n edges (rows idx[e] of
// F and target, or e itself when idx is null).  The edges are dealt to `groups`
// groups of four waves, 32 at a time; every wave writes its partial gradient
// (and loss sum) for each group to that group's slots; k_mlp_reduce sums the slots in a
// fixed order.  All waves of a block run the same number of chunk rounds
// (masked past the end) because the LDS transposes need block barriers.
struct GradShared {
  MlpShared w;
  alignas(16) __bf16 dz2[kWaves][NH][32];  // [unit][edge] per wave
  alignas(16) __bf16 h1[kWaves][NH][32];
  alignas(16) __bf16 dz1[kWaves][NH][32];
  alignas(16) __bf16 x[kWaves][NF][32];
};

__global__ __launch_bounds__(kT) void k_mlp_grad(const float* __restrict__ p,
                                                 const float* __restrict__ F, int64_t nrows,
                                                 const float* __restrict__ target,
                                                 const int64_t* __restrict__ idx, int64_t n,
                                                 int64_t groups, float* __restrict__ part,
                                                 double* __restrict__ lpart) {
  __shared__ GradShared sm;
  load_params(p, sm.w);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int h = lane >> 5, m = lane & 31;
  MlpOps op;
  op.build(sm.w, lane);
  // A operands of dH1^T = W2^T dZ2^T: rows = layer-1 units 32 mb + m, k-step
  // s over layer-2 units in the register order of dz2
  bf16x8 A3[2][4];
#pragma unroll
  for (int mb = 0; mb < 2; ++mb)
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int e = 0; e < 8; ++e) A3[mb][s][e] = sm.w.W2[kunit(s, h, e)][32 * mb + m];
  bf16x8 ones, zeros;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    ones[e] = bq(1.0f);
    zeros[e] = bq(0.0f);
  }
  const float inv = 2.0f / (float)n;
  const int64_t chunks = (n + 31) / 32;
  const int64_t rounds = (chunks + groups * kWaves - 1) / (groups * kWaves);
#pragma unroll 1
  for (int64_t grp = blockIdx.x; grp < groups; grp += gridDim.x) {
    floatx16 g2[2][3], g1[2];  // dW2 | db2 (third block: column 0), dW1 | db1 (column 16)
#pragma unroll
    for (int a = 0; a < 2; ++a) {
#pragma unroll
      for (int r = 0; r < 16; ++r) g1[a][r] = 0.0f;
#pragma unroll
      for (int b = 0; b < 3; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r) g2[a][b][r] = 0.0f;
    }
    float gw3[2][16];
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) gw3[b][r] = 0.0f;
    float gb3 = 0.0f;
    double loss = 0.0;
    for (int64_t rd = 0; rd < rounds; ++rd) {
      const int64_t c = (rd * groups + grp) * kWaves + wave;
      const int64_t e = c * 32 + m;
      int64_t row = e < n ? (idx ? idx[e] : e) : -1;
      const bool valid = row >= 0 && row < nrows;
      if (!valid) row = 0;
      MlpFwd f;
      f.run(sm.w, op, F, row, valid, lane);
      const float err = valid ? f.y - target[row] : 0.0f;
      const float dy = inv * err;
      if (h == 0) {
        loss += (double)err * (double)err;
        gb3 += dy;
      }
      // layer 2 backward (registers: lane's units of half h)
      bf16x8 dzq[4];
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int u = unit_of(b, r, h);
          const float h2 = f.z2[b][r] > 0.0f ? f.z2[b][r] : 0.0f;
          gw3[b][r] += dy * h2;
          const float dz = f.z2[b][r] > 0.0f ? dy * sm.w.w3[u] : 0.0f;
          dzq[2 * b + (r >> 3)][r & 7] = bq(dz);
          sm.dz2[wave][u][m] = bq(dz);
        }
      // dH1^T (64 x 32 edges) = W2^T dZ2^T, then dZ1 = dH1 * (z1 > 0)
      floatx16 dh1[2];
#pragma unroll
      for (int mb = 0; mb < 2; ++mb) {
#pragma unroll
        for (int r = 0; r < 16; ++r) dh1[mb][r] = 0.0f;
#pragma unroll
        for (int s = 0; s < 4; ++s)
          dh1[mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A3[mb][s], dzq[s], dh1[mb], 0, 0, 0);
      }
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int u = unit_of(b, r, h);
          sm.dz1[wave][u][m] = bq(f.z1[b][r] > 0.0f ? dh1[b][r] : 0.0f);
          sm.h1[wave][u][m] = f.h1[2 * b + (r >> 3)][r & 7];
        }
#pragma unroll
      for (int ee = 0; ee < 8; ++ee) sm.x[wave][8 * h + ee][m] = f.x[ee];
      __syncthreads();
      // weight gradients: contractions over the wave's 32 edges in two k-steps
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const int e0 = 16 * s + 8 * h;
#pragma unroll
        for (int mb = 0; mb < 2; ++mb) {
          const bf16x8 a2 = *reinterpret_cast<const bf16x8*>(&sm.dz2[wave][32 * mb + m][e0]);
#pragma unroll
          for (int nb = 0; nb < 2; ++nb) {
            const bf16x8 b2 = *reinterpret_cast<const bf16x8*>(&sm.h1[wave][32 * nb + m][e0]);
            g2[mb][nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a2, b2, g2[mb][nb], 0, 0, 0);
          }
          g2[mb][2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a2, m == 0 ? ones : zeros, g2[mb][2],
                                                              0, 0, 0);
          const bf16x8 a1 = *reinterpret_cast<const bf16x8*>(&sm.dz1[wave][32 * mb + m][e0]);
          const bf16x8 b1 = m < NF ? *reinterpret_cast<const bf16x8*>(&sm.x[wave][m][e0])
                                   : (m == NF ? ones : zeros);
          g1[mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1, b1, g1[mb], 0, 0, 0);
        }
      }
      __syncthreads();
    }
    // dw3: sum over the 32 lanes of each half (same units, different edges)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        float v = gw3[b][r];
#pragma unroll
        for (int off = 16; off >= 1; off >>= 1) v += __shfl_xor(v, off);
        gw3[b][r] = v;
      }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
      gb3 += __shfl_xor(gb3, off);
      loss += __shfl_xor(loss, off);
    }
    const int64_t slot = grp * kWaves + wave;
    float* out = part + slot * kMlpParams;
    int mo = m, ho = h;  // the stores' addresses are formed here, not kept across groups
    asm volatile("" : "+v"(mo), "+v"(ho));
#pragma unroll
    for (int mb = 0; mb < 2; ++mb)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int row = unit_of(mb, r, ho);  // layer-2 unit (dW2, db2) / layer-1 unit (dW1, db1)
#pragma unroll
        for (int nb = 0; nb < 2; ++nb) out[kOffW2 + row * NH + 32 * nb + mo] = g2[mb][nb][r];
        if (mo == 0) out[kOffB2 + row] = g2[mb][2][r];
        if (mo < NF) out[kOffW1 + row * NF + mo] = g1[mb][r];
        if (mo == NF) out[kOffB1 + row] = g1[mb][r];
        if (mo == 0) out[kOffW3 + row] = gw3[mb][r];
      }
    if (lane == 0) {
      out[kOffB3] = gb3;
      lpart[slot] = loss;
    }
  }
}

// grad[k] = sum over slots (fixed order, FP64); loss = sum of squares / n.
// Bound by the latency of its loads: a thread per parameter walking all the
// slots is one serial chain of up to 2048 of them.  Here 32 threads share a
// parameter (slots g, g + 32, ... each, eight loads in flight) and their sums
// are added in order from LDS; the block after the last takes the loss.
// 65536 edges (2048 slots, 43 MB): 590 -> 13 us.
constexpr int kRedT = 1024, kRedC = 32, kRedG = kRedT / kRedC;
__global__ __launch_bounds__(kRedT) void k_mlp_reduce(const float* __restrict__ part, int64_t slots,
                                                      const double* __restrict__ lpart, int64_t n,
                                                      float* __restrict__ grad,
                                                      double* __restrict__ loss) {
  __shared__ double red[kRedG][kRedC + 1];
  const int c = threadIdx.x % kRedC, g = threadIdx.x / kRedC;
  const bool is_loss = (int64_t)blockIdx.x * kRedC >= kMlpParams;
  const int64_t k = (int64_t)blockIdx.x * kRedC + c;
  double s = 0.0;
  if (is_loss) {
    for (int64_t i = threadIdx.x; i < slots; i += kRedT) s += lpart[i];
  } else if (k < kMlpParams) {
    int64_t i = g;
    for (; i + 7 * kRedG < slots; i += 8 * kRedG) {
      float v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = part[(i + u * kRedG) * kMlpParams + k];
#pragma unroll
      for (int u = 0; u < 8; ++u) s += (double)v[u];
    }
    for (; i < slots; i += kRedG) s += (double)part[i * kMlpParams + k];
  }
  red[g][c] = s;
  __syncthreads();
  if (g != 0) return;
  for (int q = 1; q < kRedG; ++q) s += red[q][c];
  if (is_loss) {
#pragma unroll
    for (int off = kRedC / 2; off >= 1; off >>= 1) s += __shfl_xor(s, off);
    if (c == 0 && loss) *loss = s / (double)n;
  } else if (k < kMlpParams) {
    grad[k] = (float)s;
  }
}

// One Adam update (Kingma & Ba 2015, Algorithm 1) at step t >= 1.
__global__ __launch_bounds__(kT) void k_mlp_adam(float* __restrict__ p, float* __restrict__ mo,
                                                 float* __restrict__ vo,
                                                 const float* __restrict__ g, int32_t t, float lr,
                                                 float beta1, float beta2, float eps) {
  const int64_t k = (int64_t)blockIdx.x * kT + threadIdx.x;
  if (k >= kMlpParams) return;
  const float gk = g[k];
  const float m = beta1 * mo[k] + (1.0f - beta1) * gk;
  const float v = beta2 * vo[k] + (1.0f - beta2) * gk * gk;
  mo[k] = m;
  vo[k] = v;
  const float mh = m / (1.0f - powf(beta1, (float)t));
  const float vh = v / (1.0f - powf(beta2, (float)t));
  p[k] = p[k] - lr * mh / (sqrtf(vh) + eps);
}

// out = (a - b) * scale over n entries of two strided matrices (rows x cols).
__global__ __launch_bounds__(kT) void k_ws_affine(const float* __restrict__ A, int64_t lda,
                                                  const float* __restrict__ B, int64_t ldb,
                                                  int64_t rows, int64_t cols, double scale,
                                                  double shift_scale, float* __restrict__ out,
                                                  int64_t ldo) {
  const int64_t n = rows * cols;
  for (int64_t e = (int64_t)blockIdx.x * kT + threadIdx.x; e < n; e += (int64_t)gridDim.x * kT) {
    const int64_t i = e / cols, j = e % cols;
    const double a = A[i * lda + j], b = B[i * ldb + j];
    out[i * ldo + j] = (float)(shift_scale * b + scale * a);
  }
}

// ------------------------------------------------------------- features ---
constexpr int kSk = kSketch;  // 6

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off);
  return v;
}

// Sums over the wave of N values per lane (N = 3 * 2^h), in lanes: each of the
// first h steps adds one half of the values across lanes and keeps it, so
// N + 3 (6 - h) exchanges serve all N.  Lane l ends with the sums of values
// [at, at + 3), at = wave_sums_at<N>(l).
template <int N>
__device__ __forceinline__ void wave_sums(double (&v)[N], int lane) {
  int n = N;
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    if (n % 2 == 0 && n > 3) {
      n /= 2;
      const bool up = (lane & off) != 0;
#pragma unroll
      for (int k = 0; k < N / 2; ++k) {
        if (k >= n) break;
        const double keep = up ? v[k + n] : v[k], send = up ? v[k] : v[k + n];
        v[k] = keep + __shfl_xor(send, off);
      }
    } else {
#pragma unroll
      for (int k = 0; k < 3; ++k) v[k] += __shfl_xor(v[k], off);
    }
  }
}
template <int N>
__device__ __forceinline__ int wave_sums_at(int lane) {
  int at = 0, n = N;
  for (int off = 32; off >= 1 && n > 3; off >>= 1) {
    n /= 2;
    if (lane & off) at += n;
  }
  return at;
}

// Sums over a block of NW waves of N values per thread; red holds NW x N
// doubles and ends with the sums in red[0][..], for every thread.
template <int N, int NW>
__device__ __forceinline__ void block_sums(double (&v)[N], double (*red)[N]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  wave_sums<N>(v, lane);
  const int at = wave_sums_at<N>(lane);
#pragma unroll
  for (int k = 0; k < 3; ++k) red[wave][at + k] = v[k];  // (equal sums from equal lanes)
  __syncthreads();
  if (threadIdx.x < N) {
    double s = red[0][threadIdx.x];
#pragma unroll
    for (int w = 1; w < NW; ++w) s += red[w][threadIdx.x];
    red[0][threadIdx.x] = s;
  }
  __syncthreads();
}

// Y = M X (rows x 6, FP64) for M rows x cols (FP32, leading dimension ld) and
// X cols x 6 (FP64).  Bound by reading M where it is large, by latency where
// it is small: a block takes RB rows and its threads walk the columns side by
// side, RB entries of M and a row of X (which L2 holds) at a time, two columns
// in flight.  4000 x 4000 (64 MB): 21 us; 200 rows of 200 or 4000: 5; 57 on
// average over both as 16 rows a block, a wave to four.
template <int RB>
__global__ __launch_bounds__(kT) void k_skinny(const float* __restrict__ M, int64_t rows,
                                               int64_t cols, int64_t ld,
                                               const double* __restrict__ X,
                                               double* __restrict__ Y) {
  __shared__ double red[kWaves][RB * kSk];
  const int64_t r0 = (int64_t)blockIdx.x * RB;
  double acc[RB * kSk];
#pragma unroll
  for (int k = 0; k < RB * kSk; ++k) acc[k] = 0.0;
#pragma unroll 2
  for (int64_t c = threadIdx.x; c < cols; c += kT) {
    double x[kSk];
#pragma unroll
    for (int k = 0; k < kSk; ++k) x[k] = X[c * kSk + k];
    float m[RB];
#pragma unroll
    for (int q = 0; q < RB; ++q) {
      const int64_t r = r0 + q < rows ? r0 + q : rows - 1;
      m[q] = M[r * ld + c];
    }
#pragma unroll
    for (int q = 0; q < RB; ++q)
#pragma unroll
      for (int k = 0; k < kSk; ++k) acc[q * kSk + k] += (double)m[q] * x[k];
  }
  block_sums<RB * kSk, kWaves>(acc, red);
  if (threadIdx.x < RB * kSk && r0 + threadIdx.x / kSk < rows)
    Y[r0 * kSk + threadIdx.x] = red[0][threadIdx.x];
}

// out[j][k] = sum_i M[i][j] z[i][k] (M rows x cols).  A block takes 32 columns,
// eight threads sharing one: a thread per column was one serial chain of
// `rows` loads.  200 x 4000: 50 -> 6 us.
constexpr int kColG = 8, kColC = kT / kColG;
__global__ __launch_bounds__(kT) void k_colskinny(const float* __restrict__ M, int64_t rows,
                                                  int64_t cols, int64_t ld,
                                                  const double* __restrict__ z,
                                                  double* __restrict__ out) {
  __shared__ double red[kColG][kColC][kSk];
  const int cl = threadIdx.x % kColC, g = threadIdx.x / kColC;
  const int64_t j = (int64_t)blockIdx.x * kColC + cl, jj = j < cols ? j : cols - 1;
  double acc[kSk];
#pragma unroll
  for (int k = 0; k < kSk; ++k) acc[k] = 0.0;
#pragma unroll 4
  for (int64_t i = g; i < rows; i += kColG) {
    const double v = (double)M[i * ld + jj];
#pragma unroll
    for (int k = 0; k < kSk; ++k) acc[k] += v * z[i * kSk + k];
  }
#pragma unroll
  for (int k = 0; k < kSk; ++k) red[g][cl][k] = acc[k];
  __syncthreads();
  if (threadIdx.x < kColC * kSk) {
    const int c = threadIdx.x / kSk, k = threadIdx.x % kSk;
    double s = 0.0;
#pragma unroll
    for (int q = 0; q < kColG; ++q) s += red[q][c][k];
    const int64_t jo = (int64_t)blockIdx.x * kColC + c;
    if (jo < cols) out[jo * kSk + k] = s;
  }
}

__device__ __forceinline__ double bsum(double v, double* red) {
  v = wave_sum(v);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  return ((red[0] + red[1]) + red[2]) + red[3];
}

// Cholesky QR of Y (n x 6): G = Y^T Y (one block), L L^T = G with the pivot
// rule (stop at L_kk^2 <= rel * max diag G), Q = Y L^-T on the first k
// columns, zero after.
constexpr int kChT = 1024;
__global__ __launch_bounds__(kChT) void k_cholqr_factor(const double* __restrict__ Y, int64_t n,
                                                        double rel, double* __restrict__ Linv) {
  // the 21 products of the lower triangle in one pass (a pass each took 45 us
  // at n = 4000, this one 20); the last three are the filler block_sums wants
  constexpr int N = 24;
  __shared__ double red[kChT / 64][N];
  double v[N];
#pragma unroll
  for (int k = 0; k < N; ++k) v[k] = 0.0;
  for (int64_t i = threadIdx.x; i < n; i += kChT) {
    double y[kSk];
#pragma unroll
    for (int k = 0; k < kSk; ++k) y[k] = Y[i * kSk + k];
    int q = 0;
#pragma unroll
    for (int a = 0; a < kSk; ++a)
#pragma unroll
      for (int b = 0; b <= a; ++b) v[q++] += y[a] * y[b];
  }
  block_sums<N, kChT / 64>(v, red);
  if (threadIdx.x != 0) return;
  double G[kSk][kSk];
  for (int a = 0, q = 0; a < kSk; ++a)
    for (int b = 0; b <= a; ++b) G[a][b] = G[b][a] = red[0][q++];
  double L[kSk][kSk] = {};
  double mx = 0.0;
  for (int a = 0; a < kSk; ++a) mx = G[a][a] > mx ? G[a][a] : mx;
  const double thr = rel * mx;
  int k = kSk;
  for (int j = 0; j < kSk; ++j) {
    double piv = G[j][j];
    for (int q = 0; q < j; ++q) piv -= L[j][q] * L[j][q];
    if (!(piv > thr)) {
      k = j;
      break;
    }
    L[j][j] = sqrt(piv);
    for (int i = j + 1; i < kSk; ++i) {
      double v = G[i][j];
      for (int q = 0; q < j; ++q) v -= L[i][q] * L[j][q];
      L[i][j] = v / L[j][j];
    }
  }
  // inverse of the leading k x k block (lower triangular), forward substitution
  double Li[kSk][kSk] = {};
  for (int c = 0; c < k; ++c) {
    Li[c][c] = 1.0 / L[c][c];
    for (int i = c + 1; i < k; ++i) {
      double v = 0.0;
      for (int q = c; q < i; ++q) v -= L[i][q] * Li[q][c];
      Li[i][c] = v / L[i][i];
    }
  }
  for (int a = 0; a < kSk; ++a)
    for (int b = 0; b < kSk; ++b) Linv[a * kSk + b] = (a < k && b < k) ? Li[a][b] : 0.0;
}

// Q[i][c] = sum_m Y[i][m] Linv[c][m]  (Q = Y L^-T).
__global__ __launch_bounds__(kT) void k_cholqr_apply(const double* __restrict__ Y, int64_t n,
                                                     const double* __restrict__ Linv,
                                                     double* __restrict__ Q) {
  const int64_t i = (int64_t)blockIdx.x * kT + threadIdx.x;
  if (i >= n) return;
#pragma unroll
  for (int c = 0; c < kSk; ++c) {
    double s = 0.0;
#pragma unroll
    for (int q = 0; q < kSk; ++q) s += Y[i * kSk + q] * Linv[c * kSk + q];
    Q[i * kSk + c] = s;
  }
}

// X (rows x 6 FP64) from an FP32 input with leading dimension 6.
__global__ __launch_bounds__(kT) void k_widen6(const float* __restrict__ in, int64_t rows,
                                               double* __restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * kT + threadIdx.x;
  if (i < rows * kSk) out[i] = (double)in[i];
}

// Row sums (blocks [0, rows)) and column sums (the remaining blocks, as
// k_colskinny's) of M (FP64 results).  200 x 4000: 47 -> 6 us.
__global__ __launch_bounds__(kT) void k_degrees(const float* __restrict__ M, int64_t rows,
                                                int64_t cols, int64_t ld, double* __restrict__ dr,
                                                double* __restrict__ dc) {
  __shared__ double red[4];
  if ((int64_t)blockIdx.x < rows) {
    const int64_t i = blockIdx.x;
    double s = 0.0;
    for (int64_t j = threadIdx.x; j < cols; j += kT) s += (double)M[i * ld + j];
    const double t = bsum(s, red);
    if (threadIdx.x == 0) dr[i] = t;
    return;
  }
  __shared__ double part[kColG][kColC];
  const int cl = threadIdx.x % kColC, g = threadIdx.x / kColC;
  const int64_t j = ((int64_t)blockIdx.x - rows) * kColC + cl, jj = j < cols ? j : cols - 1;
  double s = 0.0;
#pragma unroll 4
  for (int64_t i = g; i < rows; i += kColG) s += (double)M[i * ld + jj];
  part[g][cl] = s;
  __syncthreads();
  if (g == 0 && j < cols) {
#pragma unroll
    for (int q = 1; q < kColG; ++q) s += part[q][cl];
    dc[j] = s;
  }
}

// Population mean and variance (two passes, FP64) of column `col` of an
// n x stride FP64 array; one block per vector.
struct VecRef {
  const double* v;
  int64_t n, stride;
};
__global__ __launch_bounds__(kT) void k_vec_moments(const VecRef* __restrict__ vecs,
                                                    double* __restrict__ out) {
  __shared__ double red[4];
  const VecRef r = vecs[blockIdx.x];
  double s = 0.0;
  for (int64_t i = threadIdx.x; i < r.n; i += kT) s += r.v[i * r.stride];
  const double mean = bsum(s, red) / (double)r.n;
  double q = 0.0, q2 = 0.0;
  for (int64_t i = threadIdx.x; i < r.n; i += kT) {
    const double d = r.v[i * r.stride] - mean;
    q += d * d;
    q2 += r.v[i * r.stride] * r.v[i * r.stride];
  }
  const double var = bsum(q, red) / (double)r.n;
  const double msq = bsum(q2, red) / (double)r.n;
  if (threadIdx.x == 0) {
    out[3 * blockIdx.x + 0] = mean;
    out[3 * blockIdx.x + 1] = var;
    out[3 * blockIdx.x + 2] = msq;
  }
}

// S = (R0 + A0) / 2 in place of A0.
__global__ __launch_bounds__(kT) void k_half_sum(const float* __restrict__ R, int64_t ldr,
                                                 float* __restrict__ A, int64_t lda, int64_t rows,
                                                 int64_t cols) {
  const int64_t n = rows * cols;
  for (int64_t e = (int64_t)blockIdx.x * kT + threadIdx.x; e < n; e += (int64_t)gridDim.x * kT) {
    const int64_t i = e / cols, j = e - i * cols, o = i * lda + j;
    A[o] = (float)(0.5 * ((double)R[i * ldr + j] + (double)A[o]));
  }
}

// The 16 features of every edge, z-scored with the statistics st[f] =
// (mean, 1 / std or 0 for a constant feature).
__global__ __launch_bounds__(kT) void k_ws_assemble(
    int64_t Ne, int64_t Na, const float* __restrict__ W0, const float* __restrict__ S, int64_t ld,
    const double* __restrict__ dr, const double* __restrict__ dc, const double* __restrict__ a,
    const double* __restrict__ b, const double* __restrict__ c, const double* __restrict__ d,
    const double2* __restrict__ st, float* __restrict__ F) {
  const int64_t n = Ne * Na;
  for (int64_t e = (int64_t)blockIdx.x * kT + threadIdx.x; e < n; e += (int64_t)gridDim.x * kT) {
    const int64_t i = e / Na, j = e % Na;
    double g[NF];
    g[0] = W0[i * ld + j];
    g[1] = dr[i];
    g[2] = dc[j];
#pragma unroll
    for (int k = 0; k < kSk; ++k) {
      g[3 + k] = a[i * kSk + k] * b[j * kSk + k];
      g[9 + k] = c[i * kSk + k] * d[j * kSk + k];
    }
    g[15] = S[i * ld + j];
    float o[NF];
#pragma unroll
    for (int f = 0; f < NF; ++f) o[f] = (float)((g[f] - st[f].x) * st[f].y);
    f4* dst = reinterpret_cast<f4*>(F + e * NF);
#pragma unroll
    for (int q = 0; q < NF / 4; ++q) dst[q] = f4{o[4 * q], o[4 * q + 1], o[4 * q + 2], o[4 * q + 3]};
  }
}

// Feature statistics from the vector moments (m = {mean, var, mean square}
// for dr, dc, a_0..5, b_0..5, c_0..5, d_0..5) and the two full reductions
// zW = (mean, std) of W0 and zS of S.  A product feature u_i v_j over all
// edges has mean m_u m_v and second moment E[u^2] E[v^2].
__global__ void k_ws_stats(const double* __restrict__ m, const double* __restrict__ zW,
                           const double* __restrict__ zS, double2* __restrict__ st) {
  if (threadIdx.x != 0) return;
  auto put = [&](int f, double mean, double var, double scale2) {
    // var below rounding of the mean: a constant feature
    const double sd = var > 1e-24 * scale2 ? sqrt(var) : 0.0;
    st[f] = make_double2(mean, sd > 0.0 ? 1.0 / sd : 0.0);
  };
  put(0, zW[0], zW[1] * zW[1], zW[0] * zW[0] + 1e-300);
  put(1, m[0], m[1], m[2] + 1e-300);
  put(2, m[3], m[4], m[5] + 1e-300);
  for (int k = 0; k < kSk; ++k) {
    const double* A = m + 3 * (2 + k);
    const double* B = m + 3 * (8 + k);
    const double* C = m + 3 * (14 + k);
    const double* D = m + 3 * (20 + k);
    const double mp = A[0] * B[0], mq = C[0] * D[0];
    const double sp = A[2] * B[2], sq = C[2] * D[2];
    put(3 + k, mp, sp - mp * mp, sp + 1e-300);
    put(9 + k, mq, sq - mq * mq, sq + 1e-300);
  }
  put(15, zS[0], zS[1] * zS[1], zS[0] * zS[0] + 1e-300);
}

unsigned grid_cap(int64_t n, int64_t cap) {
  int64_t b = (n + kT - 1) / kT;
  if (b > cap) b = cap;
  return (unsigned)(b < 1 ? 1 : b);
}

}  // namespace

// ------------------------------------------------------------ launchers --

int64_t mlp_grad_slots(int64_t n) {
  const int64_t chunks = (n + 31) / 32;
  int64_t groups = (chunks + kWaves - 1) / kWaves;
  if (groups > kMlpGradGroups) groups = kMlpGradGroups;
  if (groups < 1) groups = 1;
  return groups * kWaves;
}

hipError_t launch_mlp_forward(const float* p, const float* F, int64_t n, float* y, hipStream_t s) {
  const int64_t chunks = (n + 31) / 32;
  int64_t blocks = (chunks + kWaves - 1) / kWaves;
  // as many as run at once: a block's weights cost more to set up than its
  // chunks to compute (402804 edges: 51 us as 3147 blocks of a chunk per wave,
  // 16 as these)
  if (blocks > 512) blocks = 512;
  if (blocks < 1) blocks = 1;
  k_mlp_forward<<<dim3((unsigned)blocks), dim3(kT), 0, s>>>(p, F, n, y);
  return hipGetLastError();
}

hipError_t launch_mlp_grad(const float* p, const float* F, int64_t nrows, const float* target,
                           const int64_t* idx, int64_t n, float* part, double* lpart, float* grad,
                           double* loss, hipStream_t s) {
  const int64_t slots = mlp_grad_slots(n), groups = slots / kWaves;
  const unsigned grid = (unsigned)(groups < kMlpGradGrid ? groups : kMlpGradGrid);
  k_mlp_grad<<<dim3(grid), dim3(kT), 0, s>>>(p, F, nrows, target, idx, n, groups, part, lpart);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const unsigned nred = (unsigned)((kMlpParams + kRedC - 1) / kRedC) + 1;  // + the loss block
  k_mlp_reduce<<<dim3(nred), dim3(kRedT), 0, s>>>(part, slots, lpart, n, grad, loss);
  return hipGetLastError();
}

hipError_t launch_mlp_adam(float* p, float* m, float* v, const float* g, int32_t t, float lr,
                           float beta1, float beta2, float eps, hipStream_t s) {
  k_mlp_adam<<<dim3((unsigned)((kMlpParams + kT - 1) / kT)), dim3(kT), 0, s>>>(
      p, m, v, g, t, lr, beta1, beta2, eps);
  return hipGetLastError();
}

hipError_t launch_ws_affine(const float* A, int64_t lda, const float* B, int64_t ldb,
                            int64_t rows, int64_t cols, double scale, double shift_scale,
                            float* out, int64_t ldo, hipStream_t s) {
  k_ws_affine<<<grid_cap(rows * cols, 8192), dim3(kT), 0, s>>>(A, lda, B, ldb, rows, cols, scale,
                                                               shift_scale, out, ldo);
  return hipGetLastError();
}

hipError_t launch_ws_sketch(const float* M, int64_t n, int64_t ld, const double* X, double* tmp,
                            double* Y, hipStream_t s) {
  const hipError_t e = launch_skinny(M, n, n, ld, X, tmp, s);
  return e != hipSuccess ? e : launch_skinny(M, n, n, ld, tmp, Y, s);
}

// Eight rows per block once that fills the CUs; X is read once per block, so
// fewer cost more of L2 (4000 rows two at a time: 30 us; 200 by eights: 8).
hipError_t launch_skinny(const float* M, int64_t rows, int64_t cols, int64_t ld, const double* X,
                         double* Y, hipStream_t s) {
  if (rows >= 2048)
    k_skinny<8><<<dim3((unsigned)((rows + 7) / 8)), dim3(kT), 0, s>>>(M, rows, cols, ld, X, Y);
  else
    k_skinny<2><<<dim3((unsigned)((rows + 1) / 2)), dim3(kT), 0, s>>>(M, rows, cols, ld, X, Y);
  return hipGetLastError();
}

hipError_t launch_colskinny(const float* M, int64_t rows, int64_t cols, int64_t ld,
                            const double* z, double* out, hipStream_t s) {
  k_colskinny<<<dim3((unsigned)((cols + kColC - 1) / kColC)), dim3(kT), 0, s>>>(M, rows, cols, ld,
                                                                               z, out);
  return hipGetLastError();
}

hipError_t launch_cholqr(const double* Y, int64_t n, double rel, double* Linv, double* Q,
                         hipStream_t s) {
  k_cholqr_factor<<<1, kChT, 0, s>>>(Y, n, rel, Linv);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  k_cholqr_apply<<<dim3((unsigned)((n + kT - 1) / kT)), dim3(kT), 0, s>>>(Y, n, Linv, Q);
  return hipGetLastError();
}

hipError_t launch_widen6(const float* in, int64_t rows, double* out, hipStream_t s) {
  k_widen6<<<dim3((unsigned)((rows * kSk + kT - 1) / kT)), dim3(kT), 0, s>>>(in, rows, out);
  return hipGetLastError();
}

hipError_t launch_degrees(const float* M, int64_t rows, int64_t cols, int64_t ld, double* dr,
                          double* dc, hipStream_t s) {
  const unsigned nb = (unsigned)(rows + (cols + kColC - 1) / kColC);
  k_degrees<<<dim3(nb), dim3(kT), 0, s>>>(M, rows, cols, ld, dr, dc);
  return hipGetLastError();
}

hipError_t launch_vec_moments(const VecRefHost* vecs, int count, double* out, hipStream_t s) {
  static_assert(sizeof(VecRefHost) == sizeof(VecRef), "same layout");
  k_vec_moments<<<dim3((unsigned)count), dim3(kT), 0, s>>>(reinterpret_cast<const VecRef*>(vecs),
                                                           out);
  return hipGetLastError();
}

hipError_t launch_half_sum(const float* R, int64_t ldr, float* A, int64_t lda, int64_t rows,
                           int64_t cols, hipStream_t s) {
  k_half_sum<<<grid_cap(rows * cols, 8192), dim3(kT), 0, s>>>(R, ldr, A, lda, rows, cols);
  return hipGetLastError();
}

hipError_t launch_ws_stats(const double* m, const double* zW, const double* zS, double2* st,
                           hipStream_t s) {
  k_ws_stats<<<1, 64, 0, s>>>(m, zW, zS, st);
  return hipGetLastError();
}

hipError_t launch_ws_assemble(int64_t Ne, int64_t Na, const float* W0, const float* S, int64_t ld,
                              const double* dr, const double* dc, const double* a,
                              const double* b, const double* c, const double* d,
                              const double2* st, float* F, hipStream_t s) {
  k_ws_assemble<<<grid_cap(Ne * Na, 16384), dim3(kT), 0, s>>>(Ne, Na, W0, S, ld, dr, dc, a, b, c,
                                                              d, st, F);
  return hipGetLastError();
}

}  // namespace panda

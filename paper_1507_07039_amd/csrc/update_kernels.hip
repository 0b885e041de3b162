// Element-wise and reduction kernels of the PANDA iteration: the h of Eq. 7,
// the second half of the P update (Eq. 5), the diagonal rule of Eq. 6, the
// squared-norm vectors the similarity epilogues read, and the z-score
// normalisation of Sec. II-A.  All reductions are FP64 and run in a fixed
// order, so results do not depend on scheduling.
#include "update_device.h"

namespace panda {
namespace {

using upd::block_sum;
using upd::split_planes;
constexpr int kRT = upd::kUT;  // threads per block for the kernels in this file

__global__ __launch_bounds__(kRT) void k_finish_h(const double* __restrict__ hpart, int64_t n,
                                                  int64_t count, DevState* st, double tol,
                                                  int32_t update_last) {
  __shared__ double red[4];
  upd::finish_h(hpart, n, count, st, tol, update_last, red);
}

__global__ __launch_bounds__(kRT) void k_coop_finalize(
    const float* __restrict__ part, int splits, int64_t Nep, const double* __restrict__ nW,
    float* __restrict__ P, int64_t ldp, int64_t Ne, double alpha, float* __restrict__ Tside,
    Planes Pp, int np, const int32_t* gate) {
  if (*gate == 0) return;
  upd::coop_finalize_entry((int64_t)blockIdx.x * kRT + threadIdx.x, part, splits, Nep, nW, P, ldp,
                           Ne, alpha, Tside, Pp, np);
}

// Eq. 6 for both networks.  Blocks [0, Ne): row i of P; remaining blocks:
// one thread per row of C.  The diagonals live in the FP64 vectors dP, dC.
__global__ __launch_bounds__(kRT) void k_diagonals(
    const float* __restrict__ P, int64_t ldp, double* __restrict__ dP, int64_t Ne,
    const float* __restrict__ Tside, double* __restrict__ nP, double* __restrict__ dC,
    int64_t ldc, int64_t Na, const double2* __restrict__ cstat, const double* __restrict__ csq,
    int64_t nslots, double* __restrict__ nC, double alpha, int32_t diag_alpha, int32_t n_own,
    int32_t ddof, const DevState* st, int32_t sched, double keep, double g, int64_t b0) {
  __shared__ double red[4];
  if (st->run_pc == 0) return;
  upd::DiagRule dr = upd::diag_rule(alpha, diag_alpha, n_own, ddof, st->t);
  if (sched) {  // closed form of several steps (warm state)
    dr.keep = keep;
    dr.g = g;
  }
  const int64_t blk = (int64_t)blockIdx.x + b0;  // launches of one part start at b0
  if (blk < Ne) {
    upd::diag_p_row(blk, P, ldp, dP, Ne, Na, Tside, nP, dr, red);
    return;
  }
  // C: 64 rows per block; wave w adds slots w, w + 4, ... and wave 0 adds
  // the four partial sums in wave order
  __shared__ double3 part[kRT / 64][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t r = (blk - Ne) * 64 + lane;
  double s1 = 0.0, s2 = 0.0, c2 = 0.0;
  if (r < Na) {
    // slots w, w + 4, ..., added in that order; eight slots' loads are in
    // flight before the first of them is added
    constexpr int64_t kStep = kRT / 64, kU = 8;
    int64_t sl = w;
    for (; sl + (kU - 1) * kStep < nslots; sl += kU * kStep) {
      double2 v[kU];
      double q[kU];
#pragma unroll
      for (int k = 0; k < kU; ++k) {
        v[k] = cstat[(sl + k * kStep) * ldc + r];
        q[k] = csq ? csq[(sl + k * kStep) * ldc + r] : 0.0;
      }
#pragma unroll
      for (int k = 0; k < kU; ++k) {
        s1 += v[k].x;
        s2 += v[k].y;
        if (csq) c2 += q[k];
      }
    }
    for (; sl < nslots; sl += kStep) {
      const double2 v = cstat[sl * ldc + r];
      s1 += v.x;
      s2 += v.y;
      if (csq) c2 += csq[sl * ldc + r];
    }
  }
  part[w][lane] = make_double3(s1, s2, c2);
  __syncthreads();
  if (w == 0 && r < Na) {
    double3 t = part[0][lane];
    for (int k = 1; k < kRT / 64; ++k) {
      t.x += part[k][lane].x;
      t.y += part[k][lane].y;
      t.z += part[k][lane].z;
    }
    upd::diag_c_finish(r, t.x, t.y, csq ? t.z : t.y, dC, Ne, Na, nC, dr);
  }
}

// d[i] = M[i][i] and M[i][i] = 0: the diagonal moves to its FP64 vector.
__global__ __launch_bounds__(kRT) void k_take_diag(float* __restrict__ M, int64_t n, int64_t ld,
                                                   double* __restrict__ d) {
  const int64_t i = (int64_t)blockIdx.x * kRT + threadIdx.x;
  if (i >= n) return;
  d[i] = (double)M[i * ld + i];
  M[i * ld + i] = 0.0f;
}

// M[i][i] = d[i] (rounded to FP32): the diagonal back into a stored matrix.
__global__ __launch_bounds__(kRT) void k_put_diag(float* __restrict__ M, int64_t n, int64_t ld,
                                                  const double* __restrict__ d) {
  const int64_t i = (int64_t)blockIdx.x * kRT + threadIdx.x;
  if (i < n) M[i * ld + i] = (float)d[i];
}

// ---- co-expression prior (Sec. II-A) ---------------------------------------
// Pearson correlation between genes across samples.  Per row: mean and
// centred sum of squares in FP64 (two passes), one wave per row.
__global__ __launch_bounds__(kRT) void k_pearson_stats(const float* __restrict__ E, int64_t G,
                                                       int64_t S, int64_t lde,
                                                       double2* __restrict__ stat) {
  const int lane = threadIdx.x & 63;
  const int64_t i = (int64_t)blockIdx.x * (kRT / 64) + (threadIdx.x >> 6);
  if (i >= G) return;
  const float* e = E + i * lde;
  double s = 0.0;
  for (int64_t k = lane; k < S; k += 64) s += (double)e[k];
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off);
  const double mean = s / (double)S;
  double q = 0.0;
  for (int64_t k = lane; k < S; k += 64) q += ((double)e[k] - mean) * ((double)e[k] - mean);
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) q += __shfl_xor(q, off);
  // a constant row gets scale 0: its normalised entries are 0
  if (lane == 0) stat[i] = make_double2(mean, q > 0.0 ? 1.0 / sqrt(q) : 0.0);
}

// Zt[k][i] = (E[i][k] - mean_i) / sqrt(ss_i), zero-padded, through a 64 x 64
// tile in LDS so that E is read and Zt written along their rows.
__global__ __launch_bounds__(kRT) void k_pearson_z(const float* __restrict__ E, int64_t G,
                                                   int64_t S, int64_t lde,
                                                   const double2* __restrict__ stat,
                                                   float* __restrict__ Zt, int64_t Gp,
                                                   int64_t Sp) {
  __shared__ float tile[64][65];
  const int64_t r0 = (int64_t)blockIdx.y * 64, c0 = (int64_t)blockIdx.x * 64;
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  for (int rr = ty; rr < 64; rr += 4) {
    const int64_t r = r0 + rr, c = c0 + tx;
    float v = 0.0f;
    if (r < G && c < S) {
      const double2 st = stat[r];
      v = (float)(((double)E[r * lde + c] - st.x) * st.y);
    }
    tile[rr][tx] = v;
  }
  __syncthreads();
  for (int cc = ty; cc < 64; cc += 4) {
    const int64_t c = c0 + cc, r = r0 + tx;
    if (r < Gp && c < Sp) Zt[c * Gp + r] = tile[tx][cc];
  }
}

// ---- bf16 operand planes ----------------------------------------------------
// Planes of P without its diagonal (which lives in its FP64 vector).
__global__ __launch_bounds__(kRT) void k_split_offdiag(const float* __restrict__ M, int64_t n,
                                                       int64_t ld, Planes out, int np) {
  const int64_t tot = n * n;
  for (int64_t e = (int64_t)blockIdx.x * kRT + threadIdx.x; e < tot; e += (int64_t)gridDim.x * kRT) {
    const int64_t i = e / n, j = e % n;
    upd::put_planes(out, np, i, j, i != j ? M[i * ld + j] : 0.0f);
  }
}

__global__ __launch_bounds__(kRT) void k_join_planes(Planes P, int64_t cols,
                                                     float* __restrict__ out, int64_t ldo) {
  const int64_t r = blockIdx.y, k = (int64_t)blockIdx.x * kRT + threadIdx.x;
  if (k < cols) out[r * ldo + k] = join_planes(P, r, k);
}

// ---- squared norms --------------------------------------------------------
// Squared norms of the rows and columns of W in one pass (Eq. 9 needs
// |W_i.|^2 and |W_.j|^2), and with NP > 0 also its NP bf16 planes,
// row-major and gene-major.  Block (bx, by) takes the 64 x 64 tile at rows
// 64 by, columns 64 bx and writes FP64 partial sums: rowpart[bx][r] over its
// 64 columns, colpart[by][c] over its 64 rows; k_w_norms_sum adds them up in
// block order (deterministic).  The tile is staged in LDS: a column's sum is
// the thread's own (its 16 rows, then the four waves in order), a row's the
// sum of four threads' quarters (16 columns each, in order) combined within
// the quad of lanes.  The planes are written whole tiles at a time from the
// staged tile, 8 entries (16 bytes) per store; entries past Ne x Na are zero
// in the tile, so the padding of the planes stays zero.
template <int NP>
__global__ __launch_bounds__(kRT) void k_w_norms(const float* __restrict__ W, int64_t Ne,
                                                 int64_t Na, int64_t ldw, int64_t Nep,
                                                 double* __restrict__ rowpart,
                                                 double* __restrict__ colpart,
                                                 Planes Wr, Planes Wt, const int32_t* gate) {
  __shared__ float tile[64][65];
  __shared__ double cred[4][64];
  if (gate && *gate == 0) return;
  const int64_t r0 = (int64_t)blockIdx.y * 64, c0 = (int64_t)blockIdx.x * 64;
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  double cs = 0.0;
  // this thread's 16 entries, all loads in flight before the first is used
  float vals[16];
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    const int64_t r = r0 + ty + 4 * k, c = c0 + tx;
    vals[k] = (r < Ne && c < Na) ? W[r * ldw + c] : 0.0f;
  }
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    const float v = vals[k];
    tile[ty + 4 * k][tx] = v;
    cs += (double)v * (double)v;
  }
  cred[ty][tx] = cs;
  __syncthreads();
  {
    // row rr, quarter q: entries 16 q .. 16 q + 15 (pitch 65: the 64 lanes of
    // a read hit 64 distinct banks)
    const int rr = threadIdx.x >> 2, q = threadIdx.x & 3;
    double rs = 0.0;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const double v = tile[rr][16 * q + i];
      rs += v * v;
    }
    rs += __shfl_xor(rs, 1);  // (q0 + q1) and (q2 + q3) ..
    rs += __shfl_xor(rs, 2);  // .. then their sum, the same in all four lanes
    if (q == 0) rowpart[(int64_t)blockIdx.x * Nep + r0 + rr] = rs;
  }
  if (ty == 0)
    colpart[(int64_t)blockIdx.y * gridDim.x * 64 + c0 + tx] =
        ((cred[0][tx] + cred[1][tx]) + cred[2][tx]) + cred[3][tx];
  if constexpr (NP > 0) {
    // 64 lines x 8 chunks of 8 entries (16 bytes), in the planes' own order:
    // a K-tile of the planes holds CT chunks of each line, line after line, so
    // consecutive threads write consecutive bytes
    constexpr int KT = plane_kt(NP), CT = KT / 8;
#pragma unroll
    for (int pass = 0; pass < 2; ++pass) {
      const int id = (int)threadIdx.x + kRT * pass;
      const int line = (id / CT) % 64, q = id % CT + CT * (id / (64 * CT));
      constexpr int NR = NP == 3 ? kHeldPlanes : NP;  // with the lower bits (join_planes)
      unsigned r[4][4], t[3][4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        bf16_t a[3], b[3];
        const float x = tile[line][8 * q + 2 * e], y = tile[line][8 * q + 2 * e + 1];
        split_planes<NP>(x, a);  // row line, along the columns
        split_planes<NP>(y, b);
#pragma unroll
        for (int p = 0; p < NP; ++p) r[p][e] = (unsigned)a[p] | ((unsigned)b[p] << 16);
        r[3][e] = (__builtin_bit_cast(unsigned, x) & 0xffffu) | (__builtin_bit_cast(unsigned, y) << 16);
        split_planes<NP>(tile[8 * q + 2 * e][line], a);  // column line, along the rows
        split_planes<NP>(tile[8 * q + 2 * e + 1][line], b);
#pragma unroll
        for (int p = 0; p < NP; ++p) t[p][e] = (unsigned)a[p] | ((unsigned)b[p] << 16);
      }
      const int64_t ro = plane_index<KT>(Wr.rows, r0 + line, c0 + 8 * q);
      const int64_t to = plane_index<KT>(Wt.rows, c0 + line, r0 + 8 * q);
#pragma unroll
      for (int p = 0; p < NR; ++p)
        *reinterpret_cast<uint4*>(Wr.p + p * Wr.stride + ro) =
            make_uint4(r[p][0], r[p][1], r[p][2], r[p][3]);
#pragma unroll
      for (int p = 0; p < NP; ++p)
        *reinterpret_cast<uint4*>(Wt.p + p * Wt.stride + to) =
            make_uint4(t[p][0], t[p][1], t[p][2], t[p][3]);
    }
  }
}

// Sums of the partials of k_w_norms: blocks [0, Nep) one row each, then
// the columns, kRT per block.
__global__ __launch_bounds__(kRT) void k_w_norms_sum(const double* __restrict__ rowpart,
                                                     const double* __restrict__ colpart,
                                                     int64_t Nep, int64_t Nap,
                                                     double* __restrict__ nr,
                                                     double* __restrict__ nc,
                                                     const int32_t* gate) {
  __shared__ double red[kRT / 64];
  if (gate && *gate == 0) return;
  const int64_t ncb = Nap / 64, nrb = Nep / 64;
  if ((int64_t)blockIdx.x < Nep) {
    const int64_t r = blockIdx.x;
    double s = 0.0;
    for (int64_t b = threadIdx.x; b < ncb; b += kRT) s += rowpart[b * Nep + r];
    const double tot = block_sum(s, red);
    if (threadIdx.x == 0) nr[r] = tot;
    return;
  }
  const int64_t c = ((int64_t)blockIdx.x - Nep) * kRT + threadIdx.x;
  if (c >= Nap) return;
  // blocks in order; eight blocks' loads in flight before the first is added
  double s = 0.0;
  int64_t b = 0;
  for (; b + 8 <= nrb; b += 8) {
    double v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = colpart[(b + k) * Nap + c];
#pragma unroll
    for (int k = 0; k < 8; ++k) s += v[k];
  }
  for (; b < nrb; ++b) s += colpart[b * Nap + c];
  nc[c] = s;
}

// ---- z-score --------------------------------------------------------------
// Moments of a set of entries: count, mean, sum of squared deviations from
// that mean.  Two sets merge without cancellation (Chan, Golub & LeVeque,
// "Updating formulae and a pairwise algorithm for computing sample
// variances", 1979).
struct Mom {
  double n, mean, m2;
};
__device__ __forceinline__ void mom_add(Mom& a, double n, double mean, double m2) {
  if (n <= 0.0) return;
  const double tot = a.n + n, d = mean - a.mean, f = n / tot;
  a.mean += d * f;
  a.m2 += m2 + d * d * (a.n * f);
  a.n = tot;
}
// Moments of v[0 .. cnt-1]: two passes in registers.
template <int U>
__device__ __forceinline__ void mom_add_run(Mom& a, const float (&v)[U], int cnt) {
  double s = 0.0, q = 0.0;
  if (cnt == U) {  // a whole run, without the selects
#pragma unroll
    for (int k = 0; k < U; ++k) s += (double)v[k];
    const double mean = s * (1.0 / U);
#pragma unroll
    for (int k = 0; k < U; ++k) {
      const double d = (double)v[k] - mean;
      q += d * d;
    }
    mom_add(a, (double)U, mean, q);
    return;
  }
#pragma unroll
  for (int k = 0; k < U; ++k) s += k < cnt ? (double)v[k] : 0.0;
  const double mean = cnt ? s / (double)cnt : 0.0;
#pragma unroll
  for (int k = 0; k < U; ++k) {
    const double d = k < cnt ? (double)v[k] - mean : 0.0;
    q += d * d;
  }
  mom_add(a, (double)cnt, mean, q);
}
// The moments of a block's threads, merged about their common mean (the same
// in every thread).  The mean is taken relative to thread 0's, so that equal
// entries give an m2 of exactly 0 whatever their number.
__device__ __forceinline__ Mom mom_block(const Mom& a, double* red) {
  __shared__ double ref;
  __syncthreads();
  if (threadIdx.x == 0) ref = a.mean;
  __syncthreads();
  const double r = ref;
  Mom t;
  t.n = block_sum(a.n, red);
  const double off = block_sum(a.n * (a.mean - r), red);
  t.mean = t.n > 0.0 ? r + off / t.n : 0.0;
  const double d = a.mean - t.mean;
  t.m2 = block_sum(a.n > 0.0 ? a.m2 + a.n * d * d : 0.0, red);
  return t;
}

// Global scope, one pass: chunks of kRT x 4 x U entries of one row (the whole
// matrix is one row where its rows are contiguous) go to the blocks in turn;
// a thread holds its 4 U entries of a chunk in registers and takes their mean
// and squared deviations there, so the matrix is read once at the rate of
// memory and nothing cancels.  An entry that is NaN or Inf makes its block's
// m2 NaN.  Scratch: mean, std and the non-finite flag at [kZsBlocks],
// [kZsBlocks + 1], [kZsBlocks + 2]; the block moments from kZsPart on.
// 18000 x 18000: two passes of 733 us (a 64-bit division per entry to find
// its row) -> one of 0.42 ms.
template <bool VEC, int U>
__global__ __launch_bounds__(kRT) void k_zs_moments(const float* __restrict__ M, int64_t rows,
                                                    int64_t cols, int64_t ld, int64_t per_row,
                                                    double* __restrict__ scratch) {
  __shared__ double red[4];
  constexpr int64_t kChunk = (int64_t)kRT * 4 * U;
  Mom a{0.0, 0.0, 0.0};
  const int64_t nch = rows * per_row;
  for (int64_t ch = blockIdx.x; ch < nch; ch += gridDim.x) {
    const int64_t r = ch / per_row, c0 = (ch - r * per_row) * kChunk;
    const float* row = M + r * ld;
    const int64_t left = cols - c0;  // entries of the row from this chunk on
    float v[4 * U];
    int cnt = 0;
    if (VEC) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int64_t o = ((int64_t)u * kRT + threadIdx.x) * 4;
        float4 x = make_float4(0.f, 0.f, 0.f, 0.f);
        if (o + 3 < left) {
          x = *reinterpret_cast<const float4*>(row + c0 + o);
        } else if (o < left) {
          x.x = row[c0 + o];
          if (o + 1 < left) x.y = row[c0 + o + 1];
          if (o + 2 < left) x.z = row[c0 + o + 2];
        }
        v[4 * u] = x.x; v[4 * u + 1] = x.y; v[4 * u + 2] = x.z; v[4 * u + 3] = x.w;
        const int64_t k = left - o;
        cnt += k >= 4 ? 4 : k > 0 ? (int)k : 0;
      }
    } else {
#pragma unroll
      for (int u = 0; u < 4 * U; ++u) {
        const int64_t o = (int64_t)u * kRT + threadIdx.x;
        v[u] = o < left ? row[c0 + o] : 0.0f;
        cnt += o < left ? 1 : 0;
      }
    }
    mom_add_run(a, v, cnt);  // a thread's entries inside the row come first
  }
  const Mom t = mom_block(a, red);
  if (threadIdx.x == 0) {
    double* p = scratch + kZsPart + 3 * (int64_t)blockIdx.x;
    p[0] = t.n;
    p[1] = t.mean;
    p[2] = t.m2;
  }
}

// The blocks' moments merged: mean, std (divisor n - ddof; 0 when there is
// no degree of freedom) and the non-finite flag.  One block.
__global__ __launch_bounds__(kRT) void k_zs_finish(double* scratch, int nb, int ddof) {
  __shared__ double red[4];
  Mom a{0.0, 0.0, 0.0};
  double bad = 0.0;
  for (int i = threadIdx.x; i < nb; i += kRT) {
    const double* p = scratch + kZsPart + 3 * i;
    if (p[0] > 0.0 && !isfinite(p[2])) bad = 1.0;
    mom_add(a, p[0], p[1], p[2]);
  }
  const Mom t = mom_block(a, red);
  const double nbad = block_sum(bad, red);
  if (threadIdx.x == 0) {
    scratch[kZsBlocks] = t.mean;
    scratch[kZsBlocks + 1] = t.n - ddof >= 1.0 ? sqrt(t.m2 / (t.n - ddof)) : 0.0;
    scratch[kZsBlocks + 2] = nbad > 0.0 ? 1.0 : 0.0;
  }
}

// M <- (M - mean) / std, skipped where the moments were refused (std = 0 or
// a non-finite entry).  The chunks are taken from the matrix's end, whose
// entries the moments pass read last and the last-level cache still holds.
// Bound by memory: 18000 x 18000 in 463 us (5.6 TB/s); 643 us with two 64-bit
// divisions for the row and an FP64 one per entry.
template <bool VEC, int U>
__global__ __launch_bounds__(kRT) void k_zs_apply(float* __restrict__ M, int64_t rows,
                                                  int64_t cols, int64_t ld, int64_t per_row,
                                                  const double* __restrict__ scratch) {
  constexpr int64_t kChunk = (int64_t)kRT * 4 * U;
  const double mean = scratch[kZsBlocks], sd = scratch[kZsBlocks + 1];
  if (!(sd > 0.0) || scratch[kZsBlocks + 2] != 0.0) return;
  const double inv = 1.0 / sd;
  auto z = [&](float x) { return (float)(((double)x - mean) * inv); };
  const int64_t nch = rows * per_row;
  for (int64_t k = blockIdx.x; k < nch; k += gridDim.x) {
    const int64_t ch = nch - 1 - k;
    const int64_t r = ch / per_row, c0 = (ch - r * per_row) * kChunk;
    float* row = M + r * ld + c0;
    const int64_t left = cols - c0;
    if (VEC) {
      float4 x[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int64_t o = ((int64_t)u * kRT + threadIdx.x) * 4;
        if (o + 3 < left) x[u] = *reinterpret_cast<const float4*>(row + o);
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int64_t o = ((int64_t)u * kRT + threadIdx.x) * 4;
        if (o + 3 < left) {
          *reinterpret_cast<float4*>(row + o) =
              make_float4(z(x[u].x), z(x[u].y), z(x[u].z), z(x[u].w));
        } else {
          for (int64_t e = o; e < left && e < o + 4; ++e) row[e] = z(row[e]);
        }
      }
    } else {
#pragma unroll
      for (int u = 0; u < 4 * U; ++u) {
        const int64_t o = (int64_t)u * kRT + threadIdx.x;
        if (o < left) row[o] = z(row[o]);
      }
    }
  }
}

// Z-score per row, or row + column (scopes of the z-score of Sec. II-A).
// rs and cs hold (mean, 1 / std).  flags[0] = 1 if an entry is NaN/Inf,
// flags[1] = 1 if a row or column has zero spread (every writer stores the
// same 1.0).  Moments in FP64; std = 0 when fewer than ddof + 1 entries.
__device__ __forceinline__ void zs_put(double2* out, double n, double mean, double m2, int ddof,
                                       double* flags) {
  const double sd = n - ddof >= 1.0 ? sqrt(m2 / (n - ddof)) : 0.0;
  *out = make_double2(mean, 1.0 / sd);
  if (!(sd > 0.0)) flags[1] = 1.0;  // NaN too: flags[0] is set with it
}
__global__ __launch_bounds__(kRT) void k_zs_rows(const float* __restrict__ M, int64_t cols,
                                                 int64_t ld, int ddof, double2* __restrict__ rs,
                                                 double* flags) {
  __shared__ double red[4];
  constexpr int U = 16;
  const float* row = M + (int64_t)blockIdx.x * ld;
  Mom a{0.0, 0.0, 0.0};
  for (int64_t j0 = 0; j0 < cols; j0 += kRT * U) {
    float v[U];
    int cnt = 0;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t j = j0 + (int64_t)u * kRT + threadIdx.x;
      v[u] = j < cols ? row[j] : 0.0f;
      cnt += j < cols ? 1 : 0;
    }
    mom_add_run(a, v, cnt);
  }
  const Mom t = mom_block(a, red);
  if (threadIdx.x == 0) {
    if (!isfinite(t.m2)) flags[0] = 1.0;
    zs_put(rs + blockIdx.x, t.n, t.mean, t.m2, ddof, flags);
  }
}

// Column moments: a block takes kRT columns of kZsColRows rows (coalesced
// across the wave), sixteen loads in flight per thread, and leaves its
// moments in part[chunk][column]; the finish merges the chunks.  One thread
// walking a whole column leaves most of the chip idle: 18000 x 18000 in 71
// blocks.
__global__ __launch_bounds__(kRT) void k_zs_cols_part(const float* __restrict__ M, int64_t rows,
                                                      int64_t cols, int64_t ld, int64_t chunk,
                                                      double2* __restrict__ part) {
  constexpr int U = 16;
  const int64_t j = (int64_t)blockIdx.x * kRT + threadIdx.x;
  if (j >= cols) return;
  const int64_t r0 = (int64_t)blockIdx.y * chunk;
  const int64_t r1 = r0 + chunk < rows ? r0 + chunk : rows;
  Mom a{0.0, 0.0, 0.0};
  for (int64_t i = r0; i < r1; i += U) {
    float v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = i + u < r1 ? M[(i + u) * ld + j] : 0.0f;
    mom_add_run(a, v, (int)(r1 - i < U ? r1 - i : U));
  }
  part[(int64_t)blockIdx.y * cols + j] = make_double2(a.mean, a.m2);
}
__global__ __launch_bounds__(kRT) void k_zs_cols_sum(const double2* __restrict__ part, int64_t rows,
                                                     int64_t cols, int64_t chunk, int nch,
                                                     int ddof, double2* __restrict__ cs,
                                                     double* flags) {
  const int64_t j = (int64_t)blockIdx.x * kRT + threadIdx.x;
  if (j >= cols) return;
  Mom a{0.0, 0.0, 0.0};
  for (int c = 0; c < nch; ++c) {
    const double2 p = part[(int64_t)c * cols + j];
    const int64_t n = rows - (int64_t)c * chunk;
    mom_add(a, (double)(n < chunk ? n : chunk), p.x, p.y);
  }
  zs_put(cs + j, a.n, a.mean, a.m2, ddof, flags);
}

// Four columns of one row per thread; blockIdx.y walks the rows.  Skipped
// where the flags refuse the matrix.
__global__ __launch_bounds__(kRT) void k_zs_apply_rc(float* __restrict__ M, int64_t rows,
                                                     int64_t cols, int64_t ld,
                                                     const double2* __restrict__ rs,
                                                     const double2* __restrict__ cs,
                                                     const double* __restrict__ flags) {
  if (flags[0] != 0.0 || flags[1] != 0.0) return;
  constexpr int U = 4;
  const double r2 = 1.0 / sqrt(2.0);
  const int64_t j0 = (int64_t)blockIdx.x * kRT * U + threadIdx.x;
  double2 c[U];
#pragma unroll
  for (int u = 0; u < U; ++u)
    if (cs && j0 + u * kRT < cols) c[u] = cs[j0 + u * kRT];
  for (int64_t i = blockIdx.y; i < rows; i += gridDim.y) {
    const double2 r = rs[i];
    float* row = M + i * ld;
    float v[U];
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (j0 + u * kRT < cols) v[u] = row[j0 + u * kRT];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (j0 + u * kRT >= cols) continue;
      const double x = (double)v[u], zr = (x - r.x) * r.y;
      row[j0 + u * kRT] = cs ? (float)((zr + (x - c[u].x) * c[u].y) * r2) : (float)zr;
    }
  }
}

__global__ __launch_bounds__(kRT) void k_zs_flags_clear(double* flags) {
  if (threadIdx.x < 8) flags[threadIdx.x] = 0.0;
}

__global__ void k_state_set(DevState* st, int32_t t, int32_t active, int32_t run_pc) {
  if (threadIdx.x == 0) {
    st->t = t;
    st->wsel = 0;
    st->active = active;
    st->run_pc = run_pc;
  }
}

unsigned grid_for(int64_t n, int64_t cap) {
  int64_t b = (n + kRT - 1) / kRT;
  if (b > cap) b = cap;
  if (b < 1) b = 1;
  return (unsigned)b;
}

}  // namespace

hipError_t launch_finish_h(const double* hpart, int64_t n, int64_t count, DevState* st, Rule rule,
                           hipStream_t s) {
  k_finish_h<<<1, kRT, 0, s>>>(hpart, n, count, st, rule.tol, rule.update_last);
  return hipGetLastError();
}

hipError_t launch_coop_finalize(const float* part, int splits, int64_t Nep, const double* nWrow,
                                float* P, int64_t ldp, int64_t Ne, Rule rule, float* Tside,
                                Planes Pp, int np, const int32_t* gate, hipStream_t s) {
  const int64_t n = Ne * Ne;
  k_coop_finalize<<<dim3((unsigned)((n + kRT - 1) / kRT)), kRT, 0, s>>>(
      part, splits, Nep, nWrow, P, ldp, Ne, rule.alpha, Tside, Pp, np, gate);
  return hipGetLastError();
}

hipError_t launch_split_offdiag(const float* M, int64_t n, int64_t ld, Planes out, int np,
                                hipStream_t s) {
  k_split_offdiag<<<grid_for(n * n, 8192), kRT, 0, s>>>(M, n, ld, out, np);
  return hipGetLastError();
}

hipError_t launch_join_planes(const Planes& P, int64_t rows, int64_t cols, float* out, int64_t ldo,
                              hipStream_t s) {
  k_join_planes<<<dim3((unsigned)((cols + kRT - 1) / kRT), (unsigned)rows), kRT, 0, s>>>(P, cols,
                                                                                         out, ldo);
  return hipGetLastError();
}

hipError_t launch_diagonals(const float* P, int64_t ldp, double* dP, int64_t Ne,
                            const float* Tside, double* nP, double* dC, int64_t ldc, int64_t Na,
                            const double2* cstat, const double* csq, int64_t nslots, double* nC,
                            Rule rule, const DevState* st, hipStream_t s, int part) {
  const int64_t b0 = part == kDiagC ? Ne : 0;
  const int64_t nb = (part == kDiagC ? 0 : Ne) + (part == kDiagP ? 0 : (Na + 63) / 64);
  if (nb == 0) return hipSuccess;
  k_diagonals<<<dim3((unsigned)nb), kRT, 0, s>>>(P, ldp, dP, Ne, Tside, nP, dC, ldc, Na, cstat,
                                                 csq, nslots, nC, rule.alpha, rule.diag_alpha,
                                                 rule.n_own, rule.sigma_ddof, st, 0, 0.0, 0.0, b0);
  return hipGetLastError();
}

hipError_t launch_diagonals_schedule(const float* P, int64_t ldp, double* dP, int64_t Ne,
                                     const float* Tside, double* nP, double* dC, int64_t ldc,
                                     int64_t Na, const double2* cstat, const double* csq,
                                     int64_t nslots, double* nC, Rule rule, double keep, double g,
                                     const DevState* st, hipStream_t s) {
  const int64_t nb = Ne + (Na + 63) / 64;
  k_diagonals<<<dim3((unsigned)nb), kRT, 0, s>>>(P, ldp, dP, Ne, Tside, nP, dC, ldc, Na, cstat,
                                                 csq, nslots, nC, rule.alpha, rule.diag_alpha,
                                                 rule.n_own, rule.sigma_ddof, st, 1, keep, g, 0);
  return hipGetLastError();
}

hipError_t launch_pearson_z(const float* E, int64_t G, int64_t S, int64_t lde, double2* stat,
                            float* Zt, int64_t Gp, int64_t Sp, hipStream_t s) {
  if (Gp % 128 || Sp % 16 || G > Gp || S > Sp) return hipErrorInvalidValue;
  k_pearson_stats<<<dim3((unsigned)((G + kRT / 64 - 1) / (kRT / 64))), kRT, 0, s>>>(E, G, S, lde,
                                                                                  stat);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  k_pearson_z<<<dim3((unsigned)((Sp + 63) / 64), (unsigned)(Gp / 64)), kRT, 0, s>>>(
      E, G, S, lde, stat, Zt, Gp, Sp);
  return hipGetLastError();
}

hipError_t launch_take_diag(float* M, int64_t n, int64_t ld, double* d, hipStream_t s) {
  k_take_diag<<<dim3((unsigned)((n + kRT - 1) / kRT)), kRT, 0, s>>>(M, n, ld, d);
  return hipGetLastError();
}

hipError_t launch_put_diag(float* M, int64_t n, int64_t ld, const double* d, hipStream_t s) {
  k_put_diag<<<dim3((unsigned)((n + kRT - 1) / kRT)), kRT, 0, s>>>(M, n, ld, d);
  return hipGetLastError();
}

hipError_t launch_state_set(DevState* st, int32_t t, int32_t active, int32_t run_pc,
                            hipStream_t s) {
  k_state_set<<<1, 64, 0, s>>>(st, t, active, run_pc);
  return hipGetLastError();
}

size_t w_norm_scratch_doubles(int64_t Nep, int64_t Nap) {
  const size_t fused = (size_t)(Nap / 64) * (size_t)Nep + (size_t)(Nep / 64) * (size_t)Nap;
  const size_t chunks = (size_t)kColChunks * (size_t)Nap;
  return fused > chunks ? fused : chunks;
}

hipError_t launch_w_norms(const float* W, int64_t Ne, int64_t Na, int64_t ldw, int64_t Nep,
                          double* nr, double* nc, double* scr, Planes Wr, Planes Wt, int np,
                          const int32_t* gate, hipStream_t s) {
  const int64_t Nap = ldw;
  if (Nep % 64 || Nap % 64 || Ne > Nep || Na > Nap) return hipErrorInvalidValue;
  if (np && (Wr.rows != Nep || Wt.rows != Nap)) return hipErrorInvalidValue;
  double* rowpart = scr;
  double* colpart = scr + (Nap / 64) * Nep;
  const dim3 grid((unsigned)(Nap / 64), (unsigned)(Nep / 64));
  auto* fn = np == 0 ? k_w_norms<0> : np == 2 ? k_w_norms<2> : k_w_norms<3>;
  fn<<<grid, kRT, 0, s>>>(W, Ne, Na, ldw, Nep, rowpart, colpart, Wr, Wt, gate);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int64_t nb = Nep + (Nap + kRT - 1) / kRT;
  k_w_norms_sum<<<dim3((unsigned)nb), kRT, 0, s>>>(rowpart, colpart, Nep, Nap, nr, nc, gate);
  return hipGetLastError();
}

// Chunking of the global z-score's passes: the whole matrix as one row where
// its rows are contiguous; 16-byte accesses where every row starts on 16
// bytes; chunks of 8192 entries once those fill every block, else of 1024.
namespace {
struct ZsPlan {
  int64_t rows, cols, ld, per_row;
  bool vec, large;
};
ZsPlan zs_plan(const float* M, int64_t rows, int64_t cols, int64_t ld) {
  ZsPlan p;
  const bool flat = ld == cols || rows == 1;
  p.rows = flat ? 1 : rows;
  p.cols = flat ? rows * cols : cols;
  p.ld = flat ? p.cols : ld;
  p.vec = reinterpret_cast<uintptr_t>(M) % 16 == 0 && (flat || ld % 4 == 0);
  const int64_t big = (int64_t)kRT * 32;
  p.large = rows * cols >= big * kZsBlocks && p.cols >= big;
  const int64_t chunk = p.large ? big : (int64_t)kRT * 4;
  p.per_row = (p.cols + chunk - 1) / chunk;
  return p;
}
}  // namespace

hipError_t launch_zscore_stats(const float* M, int64_t rows, int64_t cols, int64_t ld,
                               double* scratch, hipStream_t s, int ddof) {
  const ZsPlan p = zs_plan(M, rows, cols, ld);
  const int64_t nch = p.rows * p.per_row;
  const unsigned nb = (unsigned)(nch < kZsBlocks ? nch : kZsBlocks);
  auto* fn = p.vec ? (p.large ? k_zs_moments<true, 8> : k_zs_moments<true, 1>)
                   : (p.large ? k_zs_moments<false, 8> : k_zs_moments<false, 1>);
  fn<<<dim3(nb), kRT, 0, s>>>(M, p.rows, p.cols, p.ld, p.per_row, scratch);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  k_zs_finish<<<1, kRT, 0, s>>>(scratch, (int)nb, ddof);
  return hipGetLastError();
}

int64_t zs_col_chunks(int64_t rows) {
  const int64_t n = (rows + 255) / 256;
  return n < kZsColChunks ? n : kZsColChunks;
}

hipError_t launch_zscore_rc_stats(const float* M, int64_t rows, int64_t cols, int64_t ld, int ddof,
                                  double* flags, double2* rs, double2* cs, double2* cpart,
                                  hipStream_t s) {
  k_zs_flags_clear<<<1, kRT, 0, s>>>(flags);
  k_zs_rows<<<dim3((unsigned)rows), kRT, 0, s>>>(M, cols, ld, ddof, rs, flags);
  if (cs) {
    const int64_t nch = zs_col_chunks(rows), chunk = (rows + nch - 1) / nch;
    const unsigned gx = (unsigned)((cols + kRT - 1) / kRT);
    const unsigned gy = (unsigned)((rows + chunk - 1) / chunk);  // no empty chunk
    k_zs_cols_part<<<dim3(gx, gy), kRT, 0, s>>>(M, rows, cols, ld, chunk, cpart);
    k_zs_cols_sum<<<dim3(gx), kRT, 0, s>>>(cpart, rows, cols, chunk, (int)gy, ddof, cs, flags);
  }
  return hipGetLastError();
}

hipError_t launch_zscore_rc_apply(float* M, int64_t rows, int64_t cols, int64_t ld,
                                  const double2* rs, const double2* cs, const double* flags,
                                  hipStream_t s) {
  const int64_t gx = (cols + kRT * 4 - 1) / (kRT * 4);
  int64_t gy = (8192 + gx - 1) / gx;
  if (gy > rows) gy = rows;
  k_zs_apply_rc<<<dim3((unsigned)gx, (unsigned)gy), kRT, 0, s>>>(M, rows, cols, ld, rs, cs, flags);
  return hipGetLastError();
}

hipError_t launch_zscore_apply(float* M, int64_t rows, int64_t cols, int64_t ld,
                               const double* scratch, hipStream_t s) {
  const ZsPlan p = zs_plan(M, rows, cols, ld);
  const int64_t nch = p.rows * p.per_row;
  const unsigned nb = (unsigned)(nch < 4096 ? nch : 4096);
  auto* fn = p.vec ? (p.large ? k_zs_apply<true, 8> : k_zs_apply<true, 1>)
                   : (p.large ? k_zs_apply<false, 8> : k_zs_apply<false, 1>);
  fn<<<dim3(nb), kRT, 0, s>>>(M, p.rows, p.cols, p.ld, p.per_row, scratch);
  return hipGetLastError();
}

}  // namespace panda

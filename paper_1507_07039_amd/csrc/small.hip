// The iteration of a small network (Sec. II-B) in three launches.  At 40 x 400
// an iteration of the tiled kernels is eleven launches of 2 to 19 us, most of
// it launch, fill and drain: 72 us for 42 MFLOP.  Here the steps that need the
// same data are one launch, and every launch covers the chip with 32 x 32
// output tiles whose K is cut over the eight waves of a block, straight from
// memory to the FP32 matrix cores (no LDS staging: a wave has all the loads
// of its share in flight at once), the waves' sums added in FP64 in LDS:
//   avail    A = T(W, C), the W update, h's partials           (Eq. 4, 2, 7)
//   update   h and the gates; P and C off the diagonal          (Eq. 7, 5)
//   finish   the diagonals of P and C; the next R = T(P, W)     (Eq. 6, 3)
// What a launch would otherwise wait for, its blocks compute for themselves:
// every block of update adds up h, every block takes the norms of the rows
// and columns it reads from its own operands, every R tile takes the spread of
// its rows of P.  A 32 x 32 tile reads 64 rows of K for 1024 entries, 8 flops
// a byte, so past about a thousand rows the larger tiles win (small_net).
//
// State: avail and update read st; block 0 of update writes the new state to
// st[1], finish reads that and its block 0 writes it back to st[0], so no
// block reads what another of its launch writes.  The diagonal of P, which
// every R tile of a row reads and one writes, alternates between two vectors
// by the parity of t.
#include "panda.h"

#include "epilogues.h"
#include "small_internal.h"
#include "update_device.h"

namespace panda {
namespace {

using gemm::f4;
using gemm::floatx16;
using gemm::tanimoto;
using gemm::tri_tile;

constexpr int kNW = 8;             // waves per block
constexpr int kNT = 64 * kNW;      // (four waves per SIMD: two blocks per CU)
constexpr int kT = (int)kSmallTile;
constexpr int kPer = kT * kT / kNT;  // entries of the tile per thread
static_assert(kPer * kNT == kT * kT, "whole passes");

// Where a lane's four k of a group of eight lie: rows K-contiguous (row r at
// p + r * ld), K-strided (k at p + k * ld), or the packed symmetric C.
enum { kRows = 0, kCols = 1, kPackedC = 2 };

// The lane's operand of group g (k = 8 g + 4 h + 0 .. 3) for row / column mn.
template <int M>
__device__ __forceinline__ f4 operand(const float* __restrict__ p, int64_t ld, int64_t mn,
                                      int64_t k) {
  if constexpr (M == kRows) {
    return *reinterpret_cast<const f4*>(p + mn * ld + k);
  } else if constexpr (M == kCols) {
    return f4{p[k * ld + mn], p[(k + 1) * ld + mn], p[(k + 2) * ld + mn], p[(k + 3) * ld + mn]};
  } else {  // four k of one packed tile: along its row above the diagonal, else down a column
    const int64_t a = mn / kPT, b = k / kPT, r = mn % kPT, c = k % kPT;
    if (a <= b) return *reinterpret_cast<const f4*>(p + packed_tile(a, b) * kPT * kPT + r * kPT + c);
    const float* q = p + packed_tile(b, a) * kPT * kPT + c * kPT + r;
    return f4{q[0], q[kPT], q[2 * kPT], q[3 * kPT]};
  }
}

// This wave's share of the 32 x 32 product at (m0, n0): groups w, w + kNW, ...
// of eight k.  xx, yy: the squares of the lane's X and Y entries (its row m0 +
// lane % 32, its column n0 + lane % 32).  U groups' loads are in flight before
// the first is used.  Operands are zero past their real extent up to a
// multiple of 64.
template <int XM, int YM, bool NX, bool NY, int U, class Seen>
__device__ __forceinline__ void product(const float* __restrict__ X, int64_t ldx, int64_t m0,
                                        const float* __restrict__ Y, int64_t ldy, int64_t n0,
                                        int64_t K, floatx16& acc, double& xx, double& yy,
                                        Seen&& seen) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t mn = lane & 31, h4 = 4 * (lane >> 5);
  const int64_t ng = (K + 7) / 8;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
  xx = yy = 0.0;
  for (int64_t g0 = w; g0 < ng; g0 += U * kNW) {
    f4 a[U], b[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t g = g0 + u * kNW;
      const bool in = g < ng;
      a[u] = in ? operand<XM>(X, ldx, m0 + mn, 8 * g + h4) : f4{0.f, 0.f, 0.f, 0.f};
      b[u] = in ? operand<YM>(Y, ldy, n0 + mn, 8 * g + h4) : f4{0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t g = g0 + u * kNW;
      if (g < ng) seen(a[u], 8 * g + h4);
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        if constexpr (NX) xx += (double)a[u][s] * (double)a[u][s];
        if constexpr (NY) yy += (double)b[u][s] * (double)b[u][s];
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[u][s], b[u][s], acc, 0, 0, 0);
      }
    }
  }
}
struct Nothing {
  __device__ __forceinline__ void operator()(const f4&, int64_t) const {}
};

struct Shared {
  float part[kNW][kT * kT];       // the waves' sums, result layout [register][lane]
  double rv[4][kNW][kT];          // per-row (and per-column) values of the waves
  double row[4][kT];              // ... added up
  double red[kNW];
  float t[kT][kT + 1], v[kT][kT + 1];
};

// Sum of one double per thread over the block, fixed order.
__device__ __forceinline__ double bsum(double v, double* red) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  double s = red[0];
#pragma unroll
  for (int w = 1; w < kNW; ++w) s += red[w];
  return s;
}

__device__ __forceinline__ void put_part(Shared& sm, const floatx16& acc) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
  for (int r = 0; r < 16; ++r) sm.part[w][r * 64 + lane] = acc[r];
}
// A lane's value of its row: both halves of the wave added, into slot q.
__device__ __forceinline__ void put_row(Shared& sm, int q, double x) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  x += __shfl_xor(x, 32);
  if (lane < 32) sm.rv[q][w][lane] = x;
}
// Slots 0 .. Q-1 added over the waves (after a barrier; one before use).
template <int Q>
__device__ __forceinline__ void sum_rows(Shared& sm) {
  if (threadIdx.x < Q * kT) {
    const int q = threadIdx.x / kT, r = threadIdx.x % kT;
    double s = sm.rv[q][0][r];
#pragma unroll
    for (int w = 1; w < kNW; ++w) s += sm.rv[q][w][r];
    sm.row[q][r] = s;
  }
}
// Entry e of the tile (result layout of v_mfma_f32_32x32x2f32).
__device__ __forceinline__ int e_row(int e) {
  const int r = e >> 6, lane = e & 63;
  return 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
}
__device__ __forceinline__ int e_col(int e) { return e & 31; }
__device__ __forceinline__ double e_dot(const Shared& sm, int e) {
  double s = sm.part[0][e];
#pragma unroll
  for (int w = 1; w < kNW; ++w) s += sm.part[w][e];
  return s;
}

template <bool BATCH>
__device__ __forceinline__ const BInst& net_of(const BInst* bi, const BInst& one) {
  if constexpr (BATCH)
    return bi[blockIdx.y];
  else
    return one;
}

template <bool BATCH, bool PK>
__global__ __launch_bounds__(kNT, 4) void k_small_avail(const BInst* __restrict__ bi, BInst one,
                                                     SmallRule rule) {
  __shared__ Shared sm;
  const BInst& d = net_of<BATCH>(bi, one);
  const int64_t nMT = (d.Ne + kT - 1) / kT, nNT = (d.Na + kT - 1) / kT;
  const int64_t tile = blockIdx.x;
  if (tile >= nMT * nNT) return;
  const int32_t active = d.st->active;
  if (BATCH && active == 0) return;  // one network: checked when the loads are back
  const int ws = BATCH ? d.st->wsel : 0;
  const float* Wold = d.W[ws];
  float* Wnew = d.W[ws ^ 1];
  const int64_t m0 = (tile % nMT) * kT, n0 = (tile / nMT) * kT;
  // the epilogue's operands, in flight under the product
  float w[kPer], rr[kPer];
  double nx[kPer], ny[kPer], cd[kPer];
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    const int e = threadIdx.x + q * kNT;
    const int64_t i = m0 + e_row(e), j = n0 + e_col(e);
    const bool in = i < d.Ne && j < d.Na;
    w[q] = in ? Wold[i * d.Nap + j] : 0.0f;
    rr[q] = in ? d.R[i * d.Nap + j] : 0.0f;
    nx[q] = in ? d.nWr[i] : 0.0;
    ny[q] = in ? d.nC[j] : 0.0;
    cd[q] = in ? d.dC[j] : 0.0;
  }
  floatx16 acc;
  double xx, yy;
  product<kRows, PK ? kPackedC : kRows, false, false, 4>(Wold, d.Nap, m0, d.C, d.Nap, n0, d.Na, acc,
                                                      xx, yy, Nothing{});
  if (active == 0) return;
  put_part(sm, acc);
  __syncthreads();
  double hs = 0.0;
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    const int e = threadIdx.x + q * kNT;
    const int64_t i = m0 + e_row(e), j = n0 + e_col(e);
    if (i < d.Ne && j < d.Na) {
      const double wd = w[q], dot = e_dot(sm, e) + wd * cd[q];
      const double a = tanimoto(dot, nx[q], ny[q]);
      const double pred = 0.5 * (a + (double)rr[q]);
      const float wn = (float)((1.0 - rule.r.alpha) * wd + rule.r.alpha * pred);
      Wnew[i * d.Nap + j] = wn;
      hs += rule.r.h_undamped ? fabs(pred - wd) : fabs((double)wn - wd);
    }
  }
  const double tot = bsum(hs, sm.red);
  if (threadIdx.x == 0) d.hpart[tile] = tot;
}

// Entry (i, j), i <= j, of C in its storage.
template <bool PK>
__device__ __forceinline__ int64_t c_index(int64_t i, int64_t j, int64_t ld) {
  if constexpr (PK)
    return packed_tile(i / kPT, j / kPT) * kPT * kPT + i % kPT * kPT + j % kPT;
  else
    return i * ld + j;
}

template <bool BATCH, bool PK>
__global__ __launch_bounds__(kNT, 4) void k_small_update(const BInst* __restrict__ bi, BInst one,
                                                      SmallRule rule, int mode) {
  __shared__ Shared sm;
  const BInst& d = net_of<BATCH>(bi, one);
  const int64_t nP = (d.Ne + kT - 1) / kT, nC = (d.Na + kT - 1) / kT;
  const int64_t uP = nP * (nP + 1) / 2, uC = nC * (nC + 1) / 2;
  if ((int64_t)blockIdx.x >= uP + uC) return;
  const bool is_p = (int64_t)blockIdx.x < uP;  // P's tiles first: the longer K where N_a > N_e
  int64_t I, J;
  tri_tile(is_p ? blockIdx.x : blockIdx.x - uP, I, J);
  DevState st = d.st[0];
  auto frozen = [&] {
    if (mode != kSmallStep || st.active != 0) return false;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      st.run_pc = 0;
      st.stepped = 0;
      d.st[1] = st;
    }
    return true;
  };
  if (BATCH && frozen()) return;  // one network: checked when the loads are back
  if (mode == kSmallLoad && I != J) return;  // norms only: the diagonal tiles hold them
  const float* W = d.W[!BATCH || (mode == kSmallStep) != (st.wsel != 0) ? 1 : 0];
  const int64_t m0 = I * kT, n0 = J * kT, n = is_p ? d.Ne : d.Na;
  // the old entries, and this thread's share of h's partials
  float old[kPer];
  double hs = 0.0;
  if (mode != kSmallLoad) {
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      const int e = threadIdx.x + q * kNT;
      const int64_t i = m0 + e_row(e), j = n0 + e_col(e);
      old[q] = i < j && j < n ? (is_p ? d.P[i * d.Nep + j] : d.C[c_index<PK>(i, j, d.Nap)]) : 0.0f;
    }
    if (mode == kSmallStep) {
      const int64_t nh = nP * nC;
      for (int64_t k = threadIdx.x; k < nh; k += kNT) hs += d.hpart[k];
    }
  }
  floatx16 acc;
  double xx, yy;
  if (is_p)
    product<kRows, kRows, true, true, 3>(W, d.Nap, m0, W, d.Nap, n0, d.Na, acc, xx, yy, Nothing{});
  else
    product<kCols, kCols, true, true, 3>(W, d.Nap, m0, W, d.Nap, n0, d.Ne, acc, xx, yy, Nothing{});
  if (!BATCH && frozen()) return;
  put_part(sm, acc);
  put_row(sm, 0, xx);
  put_row(sm, 1, yy);
  __syncthreads();
  sum_rows<2>(sm);
  bool go = true;
  if (mode == kSmallStep) {  // h (Eq. 7), the same in every block; its barriers publish the rows
    const double h = bsum(hs, sm.red) / ((double)d.Ne * (double)d.Na);
    const int conv = h < rule.r.tol;
    go = !conv || rule.r.update_last;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      st.h = h;
      st.t += 1;
      st.wsel ^= 1;
      st.conv = conv;
      st.run_pc = go ? 1 : 0;
      st.stepped = 1;
      if (conv) st.active = 0;
      d.st[1] = st;
    }
  } else {
    __syncthreads();
  }
  if (!go) return;
  if (I == J && threadIdx.x < kT && m0 + threadIdx.x < n)
    (is_p ? d.nWr : d.nWc)[m0 + threadIdx.x] = sm.row[0][threadIdx.x];
  if (mode == kSmallLoad) return;
  const double al = rule.r.alpha;
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    const int e = threadIdx.x + q * kNT;
    const int rl = e_row(e), cl = e_col(e);
    const int64_t i = m0 + rl, j = n0 + cl;
    float tv = 0.0f, v = 0.0f;
    if (i < j && j < n) {  // strictly upper and real
      const double ts = tanimoto(e_dot(sm, e), sm.row[0][rl], sm.row[1][cl]);
      tv = (float)ts;
      v = (float)((1.0 - al) * (double)old[q] + al * ts);
      if (is_p)
        d.P[i * d.Nep + j] = v;
      else
        d.C[c_index<PK>(i, j, d.Nap)] = v;
      if (is_p && rule.sigma_from_T) d.Tside[i * d.Nep + j] = tv;
    }
    sm.t[rl][cl] = tv;
    sm.v[rl][cl] = v;
  }
  __syncthreads();
  // the mirror image, along its rows (a packed off-diagonal tile has none)
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    const int e = threadIdx.x + q * kNT;
    const int rl = e / kT, cl = e % kT;  // entry (n0 + rl, m0 + cl) = tile (cl, rl)
    const int64_t j = n0 + rl, i = m0 + cl;
    if (i < j && j < n) {
      if (is_p) {
        d.P[j * d.Nep + i] = sm.v[cl][rl];
        if (rule.sigma_from_T) d.Tside[j * d.Nep + i] = sm.t[cl][rl];
      } else if (!PK) {
        d.C[j * d.Nap + i] = sm.v[cl][rl];
      } else if (j / kPT == i / kPT) {  // a packed diagonal tile holds both triangles
        d.C[packed_tile(i / kPT, i / kPT) * kPT * kPT + j % kPT * kPT + i % kPT] = sm.v[cl][rl];
      }
    }
  }
  if (is_p) return;
  // row sums of C for the sigma of Eq. 6 and |C_.j|^2: slot J of the tile's
  // rows, slot I of its columns (one slot for both on the diagonal)
  if (threadIdx.x < 2 * kT) {
    const int q = threadIdx.x % kT;
    const bool col = threadIdx.x >= kT;
    double s1 = 0.0, s2 = 0.0, c2 = 0.0;
    for (int u = 0; u < kT; ++u) {
      const double v = col ? sm.v[u][q] : sm.v[q][u];
      const double x = rule.sigma_from_T ? (double)(col ? sm.t[u][q] : sm.t[q][u]) : v;
      s1 += x;
      s2 += x * x;
      c2 += v * v;
    }
    if (I == J) {  // threads 0-31 add their column's part
      s1 += __shfl_xor(s1, 32);
      s2 += __shfl_xor(s2, 32);
      c2 += __shfl_xor(c2, 32);
      if (!col) {
        d.cstat[I * d.Nap + m0 + q] = make_double2(s1, s2);
        if (rule.sigma_from_T) d.csq[I * d.Nap + m0 + q] = c2;
      }
    } else {
      const int64_t at = col ? I * d.Nap + n0 + q : J * d.Nap + m0 + q;
      d.cstat[at] = make_double2(s1, s2);
      if (rule.sigma_from_T) d.csq[at] = c2;
    }
  }
}

// Spread of a row of P about its first off-diagonal entry: sums of x - x0,
// (x - x0)^2 and x^2 over the real off-diagonal entries.  A shift inside the
// data keeps the one-pass variance from cancelling (0 for equal entries).
struct RowSpread {
  double x0;
  int64_t i, n;
  double s, q, sq;
  __device__ __forceinline__ void add(const f4& x, int64_t k) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (k + e < n && k + e != i) {
        const double v = x[e], dv = v - x0;
        s += dv;
        q += dv * dv;
      }
    }
  }
};

template <bool BATCH>
__global__ __launch_bounds__(kNT, 4) void k_small_finish(const BInst* __restrict__ bi, BInst one,
                                                         SmallRule rule, int mode,
                                                         DevState* snap) {
  __shared__ Shared sm;
  const BInst& d = net_of<BATCH>(bi, one);
  const int64_t nMT = (d.Ne + kT - 1) / kT, nNT = (d.Na + kT - 1) / kT, nR = nMT * nNT;
  const int64_t nD = mode == kSmallLoad ? 0 : (d.Na + 63) / 64;  // blocks of C's diagonal
  if ((int64_t)blockIdx.x >= nR + nD) return;
  const DevState st = mode == kSmallLoad ? d.st[0] : d.st[1];
  if (mode == kSmallStep && blockIdx.x == 0 && threadIdx.x == 0) {
    d.st[0] = st;
    if (snap) {
      *snap = st;
      __threadfence_system();
    }
  }
  if (mode == kSmallStep && st.run_pc == 0) {
    // t went on without P (the converging iteration): its diagonal goes along
    const int64_t i = (int64_t)blockIdx.x * kT + threadIdx.x;
    if (st.stepped && (int64_t)blockIdx.x < nMT && threadIdx.x < kT && i < d.Ne)
      d.dP[(st.t & 1) * d.Nep + i] = d.dP[(~st.t & 1) * d.Nep + i];
    return;
  }
  const upd::DiagRule dr =
      upd::diag_rule(rule.r.alpha, rule.r.diag_alpha, rule.r.n_own, rule.r.sigma_ddof, st.t);
  if ((int64_t)blockIdx.x >= nR) {
    // C: 64 rows, the slots over the waves, added in wave order
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t r = ((int64_t)blockIdx.x - nR) * 64 + lane;
    double s1 = 0.0, s2 = 0.0, c2 = 0.0;
    if (r < d.Na)
      for (int64_t sl = w; sl < nNT; sl += kNW) {
        const double2 v = d.cstat[sl * d.Nap + r];
        s1 += v.x;
        s2 += v.y;
        if (rule.sigma_from_T) c2 += d.csq[sl * d.Nap + r];
      }
    double(*p)[64] = reinterpret_cast<double(*)[64]>(sm.part);
    p[w][lane] = s1;
    p[kNW + w][lane] = s2;
    p[2 * kNW + w][lane] = c2;
    __syncthreads();
    if (w != 0 || r >= d.Na) return;
#pragma unroll
    for (int k = 1; k < kNW; ++k) {
      s1 += p[k][lane];
      s2 += p[kNW + k][lane];
      c2 += p[2 * kNW + k][lane];
    }
    upd::diag_c_finish(r, s1, s2, rule.sigma_from_T ? c2 : s2, d.dC, d.Ne, d.Na, d.nC, dr);
    return;
  }
  const float* W = d.W[BATCH ? st.wsel : 1];
  const int64_t tile = blockIdx.x;
  const int64_t m0 = (tile % nMT) * kT, n0 = (tile / nMT) * kT;
  float w[kPer];
  double ny[kPer];
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    const int e = threadIdx.x + q * kNT;
    const int64_t i = m0 + e_row(e), j = n0 + e_col(e);
    const bool in = i < d.Ne && j < d.Na;
    w[q] = in ? W[i * d.Nap + j] : 0.0f;
    ny[q] = in ? d.nWc[j] : 0.0;
  }
  // P's diagonal of this t (a state just loaded has it) and of the one before
  const double* dPold = d.dP + ((st.t ^ (mode == kSmallStep ? 1 : 0)) & 1) * d.Nep;
  double* dPnew = d.dP + (st.t & 1) * d.Nep;
  const int lane = threadIdx.x & 63;
  const int64_t i = m0 + (lane & 31);
  const bool real = i < d.Ne;
  // the rows the sigma is taken over: the fresh similarities under
  // sigma_from_T, else P itself, which is also the product's operand
  const float* srow = rule.sigma_from_T ? d.Tside : d.P;
  RowSpread sp{real && d.Ne > 1 ? (double)srow[i * d.Nep + (i == 0 ? 1 : 0)] : 0.0, i,
               real ? d.Ne : 0, 0.0, 0.0, 0.0};
  floatx16 acc;
  double xx, yy;
  const bool side = rule.sigma_from_T != 0;
  product<kRows, kCols, true, false, 2>(d.P, d.Nep, m0, W, d.Nap, n0, d.Ne, acc, xx, yy,
                                     [&](const f4& x, int64_t k) {
                                       if (side)
                                         sp.add(operand<kRows>(srow, d.Nep, i, k), k);
                                       else
                                         sp.add(x, k);
                                     });
  put_part(sm, acc);
  put_row(sm, 0, sp.s);
  put_row(sm, 1, sp.q);
  put_row(sm, 2, xx);  // P holds zero on its diagonal
  __syncthreads();
  sum_rows<3>(sm);
  __syncthreads();
  if (threadIdx.x < kT && m0 + threadIdx.x < d.Ne) {
    const int r = threadIdx.x;
    const int64_t gi = m0 + r;
    double dn = dPold[gi];
    if (mode == kSmallStep) {
      const double cnt = (double)(d.Ne - 1);
      double var = 0.0;
      if (cnt - dr.ddof >= 1.0) {
        var = sm.row[1][r] - sm.row[0][r] * sm.row[0][r] / cnt;
        var = var > 0.0 ? var / (cnt - dr.ddof) : 0.0;
      }
      const double mult = dr.n_own ? (double)d.Ne : (double)d.Na;
      dn = upd::diag_round(dr.keep * dn + dr.f * mult * sqrt(var) * dr.g);
    }
    sm.row[3][r] = dn;
    sm.row[2][r] += dn * dn;
    if (n0 == 0 && mode == kSmallStep) {
      dPnew[gi] = dn;
      d.nP[gi] = sm.row[2][r];
    }
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    const int e = threadIdx.x + q * kNT;
    const int rl = e_row(e);
    const int64_t gi = m0 + rl, j = n0 + e_col(e);
    if (gi < d.Ne && j < d.Na) {
      const double dot = e_dot(sm, e) + sm.row[3][rl] * (double)w[q];
      d.R[gi * d.Nap + j] = (float)tanimoto(dot, sm.row[2][rl], ny[q]);
    }
  }
}

}  // namespace

// ------------------------------------------------------------ launchers --

// Past this line the tiled kernels win in either form: us an iteration here /
// there in the FP32 form, 1000 x 1000 142 / 131, 100 x 3000 148 / 103, 40 x
// 4000 172 / 130 (the small tiles read C at a third of its bandwidth).
// With few genes every sum over them is short, and takes no planes (kShortK).
bool small_net(int64_t Ne, int64_t Na) {
  return Na <= kShortK || (Ne <= 2048 && Na <= 2048 && Ne * Na * (Ne + Na) <= 900000000);
}

// us an iteration here / in the tiled kernels of the FP32 form / of the split
// one: 40 x 400 25 / 72 / 77, 500 x 500 39 / 93 / 102, 750 x 750 82 / 112 / 97,
// 500 x 1000 66 / 100 / 88, 300 x 1500 81 / 97 / 84, 2000 x 150 98 / 211 / 166,
// 128 x 2048 75 / 92 / 79.  With more tiles of A than CUs some CU takes two,
// each over all of K = N_a, and near the long end of the range that costs more
// than the launches saved: 129 x 1700 82 / 94 / 81, 192 x 1900 93 / 93 / 84, 192
// x 2048 97 / 93 / 81; up to 1600 genes neither form loses 3 % (288 x 1600 87 /
// 98 / 86).
constexpr int64_t kChip = 256;  // CUs
bool small_run(int64_t Ne, int64_t Na, int32_t precision) {
  const int64_t longest = precision == PANDA_PREC_BF16X3 ? 1600 : 1900;
  return small_net(Ne, Na) && (Na <= longest || small_tiles(Ne) * small_tiles(Na) <= kChip);
}

hipError_t launch_small_avail(const BInst* bi, const BInst& one, int n, SmallDims mx,
                              const SmallRule& rule, hipStream_t s) {
  const dim3 g((unsigned)(small_tiles(mx.Ne) * small_tiles(mx.Na)), (unsigned)n);
  if (bi)
    k_small_avail<true, false><<<g, kNT, 0, s>>>(bi, one, rule);
  else if (rule.packed)
    k_small_avail<false, true><<<g, kNT, 0, s>>>(bi, one, rule);
  else
    k_small_avail<false, false><<<g, kNT, 0, s>>>(bi, one, rule);
  return hipGetLastError();
}

hipError_t launch_small_update(const BInst* bi, const BInst& one, int n, SmallDims mx,
                               const SmallRule& rule, SmallMode mode, hipStream_t s) {
  const int64_t a = small_tiles(mx.Ne), b = small_tiles(mx.Na);
  const dim3 g((unsigned)(a * (a + 1) / 2 + b * (b + 1) / 2), (unsigned)n);
  if (bi)
    k_small_update<true, false><<<g, kNT, 0, s>>>(bi, one, rule, mode);
  else if (rule.packed)
    k_small_update<false, true><<<g, kNT, 0, s>>>(bi, one, rule, mode);
  else
    k_small_update<false, false><<<g, kNT, 0, s>>>(bi, one, rule, mode);
  return hipGetLastError();
}

hipError_t launch_small_finish(const BInst* bi, const BInst& one, int n, SmallDims mx,
                               const SmallRule& rule, SmallMode mode, hipStream_t s,
                               DevState* snap) {
  const dim3 g((unsigned)(small_tiles(mx.Ne) * small_tiles(mx.Na) + (mx.Na + 63) / 64), (unsigned)n);
  if (bi)
    k_small_finish<true><<<g, kNT, 0, s>>>(bi, one, rule, mode, nullptr);
  else
    k_small_finish<false><<<g, kNT, 0, s>>>(bi, one, rule, mode, snap);
  return hipGetLastError();
}

}  // namespace panda

// Device building blocks of the similarity GEMMs: operand tile loaders, the
// block-level MFMA main loops (FP32 and split-BF16), and the stream-K driver
// shared by every rectangular product.
//
// Every similarity of the method is T(X, Y)_ij = (XY)_ij / sqrt(|X_i.|^2 +
// |Y_.j|^2 - |(XY)_ij|) (Eq. 1), which Sec. II-C recasts as one matrix product
// followed by an element-wise step on row and column norms (Eq. 9).  The
// product runs on matrix cores; the element-wise step (and whatever update
// rule consumes the similarity) is the epilogue of the same kernel.
//
// Operands are zero-padded to tile multiples by the host, so main loops have
// no bounds checks; zero rows and columns add nothing to products.  The
// rectangular products share one tile schedule (whole tiles in full rounds,
// the remainder split stream-K style), described at k_rect_streamk.
#pragma once

#include <algorithm>
#include <type_traits>

#include "panda_internal.h"

namespace panda {
namespace gemm {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef unsigned int u4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// A value that is the same in every lane, for the compiler to keep as such.
__device__ __forceinline__ int64_t uniform(int64_t v) {
  const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)v);
  const int hi = __builtin_amdgcn_readfirstlane((int)(v >> 32));
  return ((int64_t)hi << 32) | lo;
}

// Logical number for block b of an n-block grid: contiguous chunks per XCD.
__device__ __forceinline__ int64_t xcd_tile(int64_t b, int64_t n) {
  const int64_t xcd = b & 7, slot = b >> 3;
  const int64_t q = n >> 3, r = n & 7;
  return xcd * q + (xcd < r ? xcd : r) + slot;
}

// (I, J) with I <= J for upper-triangular tile number u = J(J+1)/2 + I.
__device__ __forceinline__ void tri_tile(int64_t u, int64_t& I, int64_t& J) {
  int64_t j = (int64_t)((sqrt(8.0 * (double)u + 1.0) - 1.0) * 0.5);
  while (j * (j + 1) / 2 > u) --j;
  while ((j + 1) * (j + 2) / 2 <= u) ++j;
  J = j;
  I = u - j * (j + 1) / 2;
}

// Eq. 1 from the product and the two squared norms (FP64); T := 0 when the
// denominator vanishes (both vectors zero).
// The quotient is taken as dot times 1/sqrt(den): the hardware estimate
// (about 2^-23 relative) refined by one Newton step, which squares its error
// (about 1e-14 relative, far under the FP32 rounding of every result), for a
// few FMAs instead of a double divide and square root per entry.
// Computed without a branch (den <= 0 selects 0 after the fact), so that
// runs of entries compile to straight-line code.
__device__ __forceinline__ double tanimoto(double dot, double xx, double yy) {
  const double den = xx + yy - fabs(dot);
  const double y0 = __builtin_amdgcn_rsq(den);
  const double y1 = y0 * (1.5 - 0.5 * den * y0 * y0);
  return den > 0.0 ? dot * y1 : 0.0;
}

// Deterministic sum of one double per thread over the block; red holds one
// double per wave.
__device__ __forceinline__ double block_sum(double v, double* red) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  double s = red[0];
  for (int w = 1; w < (int)(blockDim.x >> 6); ++w) s += red[w];
  return s;
}

// bf16 of x rounded to nearest even, as raw bits.
__device__ __forceinline__ bf16_t to_bf16(float x) {
  return __builtin_bit_cast(bf16_t, (__bf16)x);
}
__device__ __forceinline__ float from_bf16(bf16_t b) {
  return (float)__builtin_bit_cast(__bf16, b);
}

// FP32 operands: X element (m, k) = XK ? X[m*ldx + k] : X[k*ldx + m];
// Y element (k, n) = YK ? Y[n*ldy + k] : Y[k*ldy + n].
struct OpsF32 {
  const float* X;
  int64_t ldx;
  const float* Y;
  int64_t ldy;
  int64_t xrows = INT64_MAX;  // rows (m) of X that exist (loaders may clamp to them)
  int64_t K = INT64_MAX;      // length of the contraction without its padding
};

// Entries of block GEMM g summed over kn <= kShortK terms in FP64.  fill(xs, ys)
// puts the terms of the tile's rows and columns in LDS, kShortK doubles each.
// Bound by the FP64 FMAs and the epilogue.  A similarity of 5000 x 8 x 5000 takes
// 134 us (105 on planes, 151 on FP32 matrix cores), 5000 x 3 x 5000 114 (107, 150),
// correlations of 18000 genes over 5 samples 322 (305, 383).
constexpr int kShortLd = (int)kShortK + 1;  // columns read lane by lane: in other banks
template <class G, class Fill>
__device__ __forceinline__ void short_product(G& g, int kn, char* smem, Fill&& fill) {
  double* xs = reinterpret_cast<double*>(smem);
  double* ys = xs + G::BM * kShortLd;
  static_assert((G::BM + G::BN) * kShortLd * 8 <= G::MAIN_BYTES, "within the stages");
  __syncthreads();
  fill(xs, ys);
  __syncthreads();
  double y[G::TN][kShortK];
#pragma unroll
  for (int j = 0; j < G::TN; ++j)
#pragma unroll
    for (int k = 0; k < (int)kShortK; ++k) y[j][k] = ys[g.col_of(j) * kShortLd + k];
#pragma unroll
  for (int i = 0; i < G::TM; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const double* x = xs + g.row_of(i, r) * kShortLd;
      double s[G::TN];
#pragma unroll
      for (int j = 0; j < G::TN; ++j) s[j] = 0.0;
#pragma unroll
      for (int k = 0; k < (int)kShortK; ++k) {
        if (k >= kn) break;
        const double xk = x[k];
#pragma unroll
        for (int j = 0; j < G::TN; ++j) s[j] += xk * y[j][k];
      }
#pragma unroll
      for (int j = 0; j < G::TN; ++j) g.acc[i][j][r] = (float)s[j];
    }
  __syncthreads();
}

// ================================================== split-BF16 main loop ==
// Both operands are stored as bf16 planes (see Planes; X[m][k] and Yt[n][k], Yt
// = Y transposed), multiplied on v_mfma_f32_32x32x16_bf16 with an FP32
// accumulator.
//   Two planes (x = hi + lo): hi*hi + hi*lo + lo*hi; the dropped lo*lo term
//   and the rounding of lo bound the relative error of each product term by
//   about 2^-16.
//   Three planes (x = hi + mid + lo, 8 bits each, see split_pair3):
//   the six products down to 2^-16 of the leading one; the dropped ones add up
//   to 2^-22 of a term at most (of either sign), which sums of more than
//   kShortK terms average out below what an FP32 accumulation rounds away.
struct OpsB3 {
  Planes X;
  Planes Y;
  int64_t mrows = INT64_MAX;  // rows of X that exist (loaders may clamp to them)
};
// The same with Y an FP32 symmetric matrix (Yt = Y, rows read K-contiguous)
// that is split into its planes as its fragments are read.
struct OpsB3F {
  Planes X;
  const float* Y;
  int64_t ldy;
  int64_t mrows = INT64_MAX;  // rows of X that exist (loaders may clamp to them)
};
// ... with Y stored packed (packed_tile).
struct OpsB3FP {
  Planes X;
  const float* Yp;
  int64_t mrows = INT64_MAX;
};

// MN x BK tile of one K-contiguous operand, both planes, loaded by NT
// threads.  LDS rows are BK bf16 (chunks of 8 bf16 = 16 B) with the chunk
// index XOR-swizzled by the row's bank group, so the 16 rows one
// ds_read_b128 group touches land in distinct banks.
template <int MN, int NT, int BK_>
struct TileLoadB3 {
  static constexpr int BK = BK_;
  static constexpr int CPR = BK / 8;        // 16-byte chunks per row and plane
  static constexpr int RP = NT / CPR;       // rows per pass
  static constexpr int NV = MN >= RP ? MN / RP : 1;  // chunks per thread and plane
  static constexpr bool ALL = MN >= RP;     // every thread loads (else t < MN * CPR)
  static constexpr int PLANE = MN * BK;     // bf16 per plane in LDS
  static constexpr int RG = 64 / (BK / 2);  // rows sharing a bank offset
  static_assert(ALL ? RP * NV == MN : RP % MN == 0, "loads must cover the tile");

  u4 h[NV], l[NV];

  __device__ __forceinline__ static int swz(int row, int chunk) {
    return row * BK + ((chunk ^ ((row / RG) & (CPR - 1))) << 3);
  }
  __device__ __forceinline__ void load(const Planes& P, int64_t mn0, int64_t k0, int t) {
    static_assert(BK == plane_kt(2), "one K-tile of the planes");
    if (!ALL && t >= MN * CPR) return;
    const int c = (t % CPR) * 8;
    const bf16_t* H = P.p + plane_index<BK>(P.rows, mn0, k0) + c;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int r = t / CPR + i * RP;
      h[i] = *reinterpret_cast<const u4*>(H + r * BK);
      l[i] = *reinterpret_cast<const u4*>(H + P.stride + r * BK);
    }
  }
  __device__ __forceinline__ void store(bf16_t* lds, int t) const {
    if (!ALL && t >= MN * CPR) return;
    const int c = t % CPR;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int r = t / CPR + i * RP;
      *reinterpret_cast<u4*>(lds + swz(r, c)) = h[i];
      *reinterpret_cast<u4*>(lds + PLANE + swz(r, c)) = l[i];
    }
  }
};

// Block-level split-BF16 GEMM, WM x WN waves of (BM/WM) x (BN/WN) each.
// All fragments of a K-tile are read from LDS before its MFMAs are issued,
// so the LDS latency is paid once per tile rather than once per 16-k step.
template <int BM_, int BN_, int WM, int WN, int BK_ = 32, int WPE = 1>
struct BlockGemmB3 {
  using Ops = OpsB3;
  static constexpr bool kBlockEpi = true;  // epilogue entries in runs of 8
  static constexpr int BM = BM_, BN = BN_, BK = BK_, NT = 64 * WM * WN;
  static constexpr int WAVES_PER_EU = WPE;  // occupancy asked of the compiler (1: no request)
  static constexpr int TM = BM / WM / 32;
  static constexpr int TN = BN / WN / 32;
  static constexpr int KS = BK / 16;  // MFMA k-steps per K-tile
  static_assert(TM >= 1 && TN >= 1, "wave tile below one MFMA block");
  using LX = TileLoadB3<BM, NT, BK>;
  using LY = TileLoadB3<BN, NT, BK>;
  static constexpr int XS = 2 * LX::PLANE;  // bf16 per stage
  static constexpr int YS = 2 * LY::PLANE;
  static constexpr int MAIN_BYTES = 2 * (XS + YS) * 2;

  floatx16 acc[TM][TN];
  int lane, wm, wn;

  __device__ __forceinline__ static void load_y(LY& ly, const Ops& o, int64_t n0, int64_t k0,
                                                int t) {
    ly.load(o.Y, n0, k0, t);
  }

  __device__ __forceinline__ void run(const Ops& o, int64_t m0, int64_t n0, int64_t kbeg,
                                      int64_t kend, char* smem) {
    const int t = threadIdx.x;
    lane = t & 63;
    const int w = t >> 6;
    wm = w % WM;
    wn = w / WM;
    bf16_t* xs = reinterpret_cast<bf16_t*>(smem);
    bf16_t* ys = xs + 2 * XS;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
    LX lx;
    LY ly;
    const int64_t nk = (kend - kbeg) / BK;
    if (nk > 0) {
      lx.load(o.X, m0, kbeg, t);
      load_y(ly, o, n0, kbeg, t);
      lx.store(xs, t);
      ly.store(ys, t);
    }
    __syncthreads();
    const int mrow = wm * (BM / WM) + (lane & 31);
    const int ncol = wn * (BN / WN) + (lane & 31);
    const int khalf = lane >> 5;
    for (int64_t kt = 0; kt < nk; ++kt) {
      const int cur = (int)(kt & 1);
      const bool more = kt + 1 < nk;
      if (more) {
        lx.load(o.X, m0, kbeg + (kt + 1) * BK, t);
        load_y(ly, o, n0, kbeg + (kt + 1) * BK, t);
      }
      const bf16_t* xc = xs + cur * XS;
      const bf16_t* yc = ys + cur * YS;
      bf16x8 xh[KS][TM], xl[KS][TM], yh[KS][TN], yl[KS][TN];
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const int chunk = 2 * ks + khalf;  // this lane's 8 k-values of the 16-k step
#pragma unroll
        for (int i = 0; i < TM; ++i) {
          const int off = LX::swz(mrow + i * 32, chunk);
          xh[ks][i] = *reinterpret_cast<const bf16x8*>(xc + off);
          xl[ks][i] = *reinterpret_cast<const bf16x8*>(xc + LX::PLANE + off);
        }
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          const int off = LY::swz(ncol + j * 32, chunk);
          yh[ks][j] = *reinterpret_cast<const bf16x8*>(yc + off);
          yl[ks][j] = *reinterpret_cast<const bf16x8*>(yc + LY::PLANE + off);
        }
      }
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j) {
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xh[ks][i], yl[ks][j], acc[i][j], 0, 0, 0);
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xl[ks][i], yh[ks][j], acc[i][j], 0, 0, 0);
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xh[ks][i], yh[ks][j], acc[i][j], 0, 0, 0);
          }
      if (more) {
        lx.store(xs + (cur ^ 1) * XS, t);
        ly.store(ys + (cur ^ 1) * YS, t);
      }
      __syncthreads();
    }
  }

  __device__ __forceinline__ int row_of(int i, int r) const {
    return wm * (BM / WM) + i * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
  }
  __device__ __forceinline__ int col_of(int j) const {
    return wn * (BN / WN) + j * 32 + (lane & 31);
  }
  template <class F>
  __device__ __forceinline__ void for_each(F&& f) const {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int c = col_of(j);
#pragma unroll
        for (int r = 0; r < 16; ++r) f(row_of(i, r), c, acc[i][j][r]);
      }
  }
};

// =============================== software-pipelined split-BF16 loop ==
// A x C with A given as bf16 hi/lo planes and C as FP32 (split into hi/lo
// as its fragments are read; C is symmetric, so its row n is the column the
// product needs).  Operand tiles move by direct global -> LDS loads
// (global_load_lds_dwordx4: lane l of a wave writes its 16 bytes at LDS base
// + 16 l) into STAGES (two or three) stages, so STAGES - 1 K-tiles are in
// flight without holding registers.  Which global chunk a lane fetches is chosen so that the LDS
// image is swizzled for conflict-free fragment reads:
//   bf16 planes: rows of BK bf16, slot s of row r holds chunk s ^ f(r) (as
//     TileLoadB3);
//   FP32 rows: BK floats = BK / 4 chunks, slot s of row r holds chunk
//     s ^ yswz(r), so the 16 rows one read touches at a time cover all 64
//     banks.
// The loop is also software-pipelined in registers: while the matrix cores
// work on K-tile k, the wave issues the loads of K-tile k + STAGES, reads
// the fragments of K-tile k + 1 from LDS and splits them.
//
// The direct loads are issued from inline assembly (no register results;
// the LDS base goes through M0), so the compiler's own LDS reads are not
// held back for them; ordering is explicit instead: every wave waits for its
// own loads of a stage (vmcnt), then a barrier that is also a compiler
// memory barrier makes the stage complete for all waves.  A stage is
// refilled only after the barrier that follows its last reads.
__device__ __forceinline__ void lds_dma16(unsigned voff, const void* sbase, unsigned ldsa) {
  // the base and the LDS address are wave-uniform; say so, so that they sit
  // in scalar registers whatever the compiler concluded about them
  // (the builtin returns a signed int: widen through unsigned, or a low half
  // with bit 31 set would be sign-extended into the high half)
  const uint64_t b = (uint64_t)sbase;
  const uint64_t lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)b);
  const uint64_t hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(b >> 32));
  const uint64_t bs = lo | (hi << 32);
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
               :
               : "v"(voff), "s"(bs), "s"(__builtin_amdgcn_readfirstlane(ldsa))
               : "memory", "m0");
}
// Barrier after this wave's LDS reads have completed (so no read of a stage
// can still be pending when another wave refills it); also a compiler
// memory barrier.
__device__ __forceinline__ void wave_barrier_mem() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Wait until at most n vector-memory operations of this wave are pending
// (gfx9 s_waitcnt: vmcnt in bits 3:0 and 15:14; exp and lgkm counts left at
// their maxima, i.e. not waited for).
template <int N>
__device__ __forceinline__ void wait_vmem() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 0xF) | ((N >> 4) << 14) | (0x7 << 4) | (0xF << 8));
}

// hi = RNE(a), lo = RNE(a - hi) for two floats at once (packed bf16 pairs).
__device__ __forceinline__ void split_pair(float a, float b, unsigned& h, unsigned& l) {
  typedef float fl2 __attribute__((ext_vector_type(2)));
  typedef __bf16 bh2 __attribute__((ext_vector_type(2)));
  h = __builtin_bit_cast(unsigned, __builtin_convertvector((fl2){a, b}, bh2));
  const float ha = __builtin_bit_cast(float, h << 16);
  const float hb = __builtin_bit_cast(float, h & 0xffff0000u);
  l = __builtin_bit_cast(unsigned, __builtin_convertvector((fl2){a - ha, b - hb}, bh2));
}

// Two floats as three bf16 each, x = hi + mid + lo: hi = the upper 16 bits of x
// (truncated, so that no finite x overflows), mid = RNE(x - hi), lo = x - hi -
// mid, which has at most 8 significant bits (both differences are exact; below
// 2^-110 some of those bits lie under the smallest bf16 and are lost).
__device__ __forceinline__ void split_pair3(float a, float b, unsigned (&o)[3]) {
  typedef float fl2 __attribute__((ext_vector_type(2)));
  typedef __bf16 bh2 __attribute__((ext_vector_type(2)));
  const unsigned ua = __builtin_bit_cast(unsigned, a), ub = __builtin_bit_cast(unsigned, b);
  o[0] = __builtin_amdgcn_perm(ub, ua, 0x07060302u);  // upper halves of b : a
  const float ra = a - __builtin_bit_cast(float, ua & 0xffff0000u);
  const float rb = b - __builtin_bit_cast(float, ub & 0xffff0000u);
  const unsigned m = __builtin_bit_cast(unsigned, __builtin_convertvector((fl2){ra, rb}, bh2));
  o[1] = m;
  const float la = ra - __builtin_bit_cast(float, m << 16);
  const float lb = rb - __builtin_bit_cast(float, m & 0xffff0000u);
  o[2] = __builtin_amdgcn_perm(__builtin_bit_cast(unsigned, lb), __builtin_bit_cast(unsigned, la),
                               0x07060302u);
}

// ========================================= FP32 operands on bf16 planes ==
// Block-level product of FP32 operands (OpsF32) over k in [kbeg, kend), a
// multiple of 16, on the bf16 matrix cores: each 16-deep K-tile is split into
// its three exact bf16 planes (split_pair3) between the registers it was
// loaded into and LDS, and multiplied as BlockGemmB3P<NP = 3> multiplies
// stored planes.  For operands nobody keeps planes of: batches, the
// stand-alone similarity, the correlations, the warm start.
//
// A wave of 64 x 64 has 24 MFMAs of 32 cycles per K-tile; the next tile's
// split (some 90 vector instructions) and LDS stores go between them, and two
// waves per SIMD cover each other's fragment reads and barriers.  What it took
// to keep the matrix cores fed: two K-tiles on their way in registers, loads
// known to be in global memory (flat ones are waited for with every LDS
// read), and no work for row blocks that are all padding.  Against
// v_mfma_f32_32x32x2f32 on the same operands: A + W of a batch of six
// networks (57 x 4999 to 661 x 9787, 238 GFLOP) 2.81 -> 1.62 ms (880 TFLOP/s
// of bf16), its C update 1.74 -> 1.11, W W^T 0.15 -> 0.11; a similarity of 700
// x 2001 x 5003 167 -> 94 us; correlations of 18000 genes over 200 samples
// 938 -> 668 us on average over 21 launches (871 -> 563 the shortest; with the
// 16-byte stores of corr_sym_epilogue).  The error against 64 bits falls to between
// a third and 0.8 of what it was.
//
// KS: how K is summed (KSum).  Folded as there, but in registers (a choice of
// kernel: the running sum takes 64 of the 256 registers a wave has; it cost
// 15 % where it was carried for K = 700).
template <int MN, bool KC, int NT>
struct TileLoadF3 {
  static constexpr int NI = MN * 2 / NT;  // runs of 8 k per thread
  static_assert(NI >= 1 && NI * NT == MN * 2, "whole runs per thread");
  // LDS, per plane and 8 k: 16 bytes per row.  The pad keeps the two runs of
  // a row, which neighbouring lanes of the KC case write, in other banks.
  static constexpr int RUN = MN * 16 + (KC ? 128 : 0), PLANE = 2 * RUN;
  // the next K-tile to load: uniform, and known to be in global memory (a flat
  // load would also be waited for with every LDS read)
  using Global = const __attribute__((address_space(1))) char*;
  template <class T>
  using GlobalP = const __attribute__((address_space(1))) T*;
  Global base;
  unsigned off[NI];  // bytes, per lane
  int64_t ld;        // bytes from one row in memory to the next
  float v[2][NI][8];  // two tiles on their way

  __device__ __forceinline__ static int row(int t, int i) {
    return KC ? (t + i * NT) >> 1 : (t + i * NT) % MN;
  }
  __device__ __forceinline__ static int run(int t, int i) {
    return KC ? (t + i * NT) & 1 : (t + i * NT) / MN;
  }
  // Rows past the operand's end re-read its last one; their outputs are never
  // stored.
  __device__ __forceinline__ void setup(const float* b, int64_t ld_, int64_t mn0, int64_t rows,
                                        int64_t kbeg, int t) {
    ld = uniform(4 * ld_);
    base = (Global)(size_t)uniform((int64_t)(size_t)(KC ? b + mn0 * ld_ + kbeg : b + kbeg * ld_ + mn0));
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int r = mn0 + row(t, i) < rows ? row(t, i) : (int)(rows - 1 - mn0);
      off[i] = KC ? (unsigned)(r * ld) + 32u * run(t, i) : (unsigned)(8 * run(t, i) * ld) + 4u * r;
    }
  }
  // The tile at `base` into set S; `more`: another one follows it.
  template <int S>
  __device__ __forceinline__ void load(bool more) {
#pragma unroll
    for (int e = 0; e < (KC ? 1 : 8); ++e) {
      // a uniform base per row: one 32-bit offset per run serves all its loads
      int64_t a = (int64_t)base + (KC ? 0 : e * ld);
      asm("" : "+s"(a));
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        unsigned r = off[i];
        asm("" : "+v"(r));  // (stays a 32-bit offset)
        if constexpr (KC) {
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const f4 x = *(GlobalP<f4>)((Global)a + r + 16 * h);
#pragma unroll
            for (int k = 0; k < 4; ++k) v[S][i][4 * h + k] = x[k];
          }
        } else {
          v[S][i][e] = *(GlobalP<float>)((Global)a + r);
        }
      }
    }
    base += more ? (KC ? 64 : 16 * ld) : 0;
  }
  // Piece q of 5 NI of set S: four pairs split, then the run's planes stored.
  template <int S>
  __device__ __forceinline__ void put(char* lds, int t, int q, unsigned (&o)[3][4]) {
    const int i = q / 5, s = q % 5;
    if (s < 4) {
      unsigned u[3];
      // not before its MFMA (the compiler would otherwise start with it and
      // wait for the loads there)
      asm volatile("" : "+v"(v[S][i][2 * s]), "+v"(v[S][i][2 * s + 1]));
      split_pair3(v[S][i][2 * s], v[S][i][2 * s + 1], u);
#pragma unroll
      for (int pl = 0; pl < 3; ++pl) o[pl][s] = u[pl];
    } else {
#pragma unroll
      for (int pl = 0; pl < 3; ++pl)
        *reinterpret_cast<u4*>(lds + pl * PLANE + run(t, i) * RUN + row(t, i) * 16) =
            (u4){o[pl][0], o[pl][1], o[pl][2], o[pl][3]};
    }
  }
};

template <int BM_, int BN_, int WM, int WN, bool XK, bool YK, int KS>
struct BlockGemmF3 {
  static constexpr bool LK = KS == kSumFolded || KS == kSumAny;
  using Ops = OpsF32;
  static constexpr int BM = BM_, BN = BN_, BK = 16, NT = 64 * WM * WN;
  static constexpr int WAVES_PER_EU = 2;
  static constexpr bool kPrefetchEpi = true, kBlockEpi = true;
  static constexpr int TM = BM / WM / 32;
  static constexpr int TN = BN / WN / 32;
  static_assert(TM >= 1 && TN >= 1, "wave tile below one MFMA block");
  using LX = TileLoadF3<BM, XK, NT>;
  using LY = TileLoadF3<BN, YK, NT>;
  static constexpr int STAGE = 3 * (LX::PLANE + LY::PLANE);
  static constexpr int MAIN_BYTES = 2 * STAGE;
  static constexpr int NQX = LX::NI * 5, NQ = NQX + LY::NI * 5;  // pieces of a split
  static constexpr int kFoldTiles = (int)(kFoldK / BK);

  floatx16 acc[TM][TN];
  int lane, wm, wn;

  __device__ __forceinline__ void run(const Ops& o, int64_t m0, int64_t n0, int64_t kbeg,
                                      int64_t kend, char* smem) {
    constexpr int XP[6] = {2, 0, 1, 1, 0, 0}, YP[6] = {0, 2, 1, 0, 1, 0};
    const int t = threadIdx.x;
    lane = t & 63;
    const int w = __builtin_amdgcn_readfirstlane(t >> 6);
    wm = w % WM;
    wn = w / WM;
    if constexpr (KS == kSumAny || KS == kSumShort) {
      if (KS == kSumShort || o.K <= kShortK) {
        run_short(o, m0, n0, kbeg, kend, smem);
        return;
      }
    }
    floatx16 sum[LK ? TM : 1][LK ? TN : 1];
    auto clear = [](auto& a) {
#pragma unroll
      for (auto& row : a)
#pragma unroll
        for (auto& x : row)
#pragma unroll
          for (int r = 0; r < 16; ++r) x[r] = 0.0f;
    };
    clear(acc);
    if constexpr (LK) clear(sum);

    LX lx;
    LY ly;
    lx.setup(o.X, o.ldx, m0, o.xrows, kbeg, t);
    ly.setup(o.Y, o.ldy, n0, INT64_MAX, kbeg, t);
    const int nk = (int)(uniform(kend - kbeg) / BK);
    // 32-row blocks of this wave that hold rows of X; the others (padding) take
    // no part: their outputs are never stored
    const int64_t rows = uniform(o.xrows - m0) - wm * (BM / WM);
    const int live = rows >= 32 * TM ? TM : rows <= 0 ? 0 : (int)(rows + 31) / 32;
    unsigned ox[3][4], oy[3][4];
    const int xo = (lane >> 5) * LX::RUN + (wm * (BM / WM) + (lane & 31)) * 16;
    const int yo = 3 * LX::PLANE + (lane >> 5) * LY::RUN + (wn * (BN / WN) + (lane & 31)) * 16;
    // K-tile kt: stage kt % 2 holds it, register set S tile kt + 1 and the other
    // set tile kt + 2 (or the last tile again, at the end of the range).  Tile
    // kt + 1 is split into the other stage and tile kt + 3 loaded, each piece
    // under an MFMA.
    auto step = [&](auto set, auto nl, int kt) {
      constexpr int S = decltype(set)::value;
      constexpr int TL = decltype(nl)::value;  // live row blocks
      constexpr int NM = 6 * TL * TN;          // MFMAs per K-tile
      constexpr int PM = NM > 1 ? (NQ + NM - 2) / (NM - 1) : NQ;  // pieces under each
      const char* rd = smem + (kt & 1) * STAGE;
      char* wr = smem + ((kt + 1) & 1) * STAGE;
      auto piece = [&](int q) {
        if (q < NQX)
          lx.template put<S>(wr, t, q, ox);
        else if (q < NQ)
          ly.template put<S>(wr + 3 * LX::PLANE, t, q - NQX, oy);
      };
      const bool more = kt + 4 < nk;
      if constexpr (TL == 0) {
#pragma unroll
        for (int q = 0; q < NQ; ++q) piece(q);
        lx.template load<S>(more);
        ly.template load<S>(more);
      } else {
        bf16x8 x[3][TL], y[3][TN];
#pragma unroll
        for (int pl = 0; pl < 3; ++pl) {
#pragma unroll
          for (int i = 0; i < TL; ++i)
            x[pl][i] = *reinterpret_cast<const bf16x8*>(rd + xo + pl * LX::PLANE + i * 512);
#pragma unroll
          for (int j = 0; j < TN; ++j)
            y[pl][j] = *reinterpret_cast<const bf16x8*>(rd + yo + pl * LY::PLANE + j * 512);
        }
#pragma unroll
        for (int m = 0; m < NM; ++m) {
          const int j = m % TN, i = (m / TN) % TL, p = m / TN / TL;
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[XP[p]][i], y[YP[p]][j], acc[i][j],
                                                              0, 0, 0);
#pragma unroll
          for (int q = m * PM; q < (m + 1) * PM; ++q) piece(q);
          if (m == (NQX + PM - 1) / PM) lx.template load<S>(more);
          if (m == (NQ + PM - 1) / PM) ly.template load<S>(more);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      __syncthreads();
    };
    if (nk > 0) {
      lx.template load<0>(nk > 1);
      ly.template load<0>(nk > 1);
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        if (q < NQX)
          lx.template put<0>(smem, t, q, ox);
        else
          ly.template put<0>(smem + 3 * LX::PLANE, t, q - NQX, oy);
      }
      lx.template load<0>(nk > 2);
      ly.template load<0>(nk > 2);
      lx.template load<1>(nk > 3);
      ly.template load<1>(nk > 3);
    }
    __syncthreads();
    using S0 = std::integral_constant<int, 0>;
    using S1 = std::integral_constant<int, 1>;
    auto tiles = [&](auto nl) {
      constexpr int TL = decltype(nl)::value;
      for (int kt = 0; kt < nk; kt += 2) {
        step(S0{}, nl, kt);
        if (kt + 1 < nk) step(S1{}, nl, kt + 1);
        if constexpr (LK) {
          if (kt % kFoldTiles == kFoldTiles - 2) {
#pragma unroll
            for (int i = 0; i < TL; ++i)
#pragma unroll
              for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                  sum[i][j][r] += acc[i][j][r];
                  acc[i][j][r] = 0.0f;
                }
          }
        }
      }
    };
    static_assert(TM <= 4 && TM != 3, "live row blocks");
    if (live == TM) {
      tiles(std::integral_constant<int, TM>{});
    } else if (live == 0) {
      tiles(std::integral_constant<int, 0>{});
    } else if constexpr (TM >= 2) {
      if (live == 1) tiles(std::integral_constant<int, 1>{});
      if constexpr (TM == 4) {
        if (live == 2) tiles(std::integral_constant<int, 2>{});
        if (live == 3) tiles(std::integral_constant<int, 3>{});
      }
    }
    if constexpr (LK) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[i][j][r] += sum[i][j][r];
    }
  }
  // Terms of one operand (rows rows, ld floats apart along k or across it) in LDS.
  template <bool KC, int MN>
  __device__ __forceinline__ static void put_terms(double* s, const float* p, int64_t ld, int64_t mn0,
                                                   int64_t rows, int64_t kbeg, int64_t kn) {
    for (int e = threadIdx.x; e < MN * (int)kShortK; e += NT) {
      const int k = KC ? e % (int)kShortK : e / MN, q = KC ? e / (int)kShortK : e % MN;
      const int64_t mn = mn0 + q < rows ? mn0 + q : rows - 1;
      s[q * kShortLd + k] = k < kn ? (double)(KC ? p[mn * ld + kbeg + k] : p[(kbeg + k) * ld + mn]) : 0.0;
    }
  }
  __device__ __forceinline__ void run_short(const Ops& o, int64_t m0, int64_t n0, int64_t kbeg,
                                            int64_t kend, char* smem) {
    const int64_t kn = (kend < o.K ? kend : o.K) - kbeg;  // (none in a later chunk of K)
    short_product(*this, kn > 0 ? (int)kn : 0, smem, [&](double* xs, double* ys) {
      put_terms<XK, BM>(xs, o.X, o.ldx, m0, o.xrows, kbeg, kn);
      put_terms<YK, BN>(ys, o.Y, o.ldy, n0, INT64_MAX, kbeg, kn);
    });
  }
  __device__ __forceinline__ int row_of(int i, int r) const {
    return wm * (BM / WM) + i * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
  }
  __device__ __forceinline__ int col_of(int j) const {
    return wn * (BN / WN) + j * 32 + (lane & 31);
  }
  template <class F>
  __device__ __forceinline__ void for_each(F&& f) const {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int c = col_of(j);
#pragma unroll
        for (int r = 0; r < 16; ++r) f(row_of(i, r), c, acc[i][j][r]);
      }
  }
};

// YF32: Y is the FP32 symmetric matrix split as its fragments are read;
// otherwise Y is given as bf16 hi/lo planes like X (no split arithmetic).
// The STAGES stage buffers are carved from the caller's shared memory.
// YP: Y (FP32) is stored packed (packed_tile).  The product needs row n of Y
// over the K-tile's k (Y symmetric: row n is column n).  Where the tile of
// (n, k) lies above the diagonal it holds that row directly; below it, the
// tile of (k, n) holds it as a column, so such a K-tile is loaded as it is
// stored, [k][n] rows of kPT floats, and its fragments are read with one
// 4-byte read per k.  Both rows of a fragment read's two half-waves differ
// by 8 in k, and their 16-byte chunks are XOR-swizzled by that bit, so the
// two half-waves use different banks.
// NP: planes of each operand (2 or 3), and the products of a K-step with it.
template <int BM_, int BN_, int WM, int WN, bool YF32 = true, int STAGES = 3, int BK_ = 32,
          bool YP = false, int NP = 2>
struct BlockGemmB3P {
  using Ops = typename std::conditional<
      YP, OpsB3FP, typename std::conditional<YF32, OpsB3F, OpsB3>::type>::type;
  static_assert(NP == 2 || NP == 3, "two or three planes");
  static constexpr int NPROD = NP == 2 ? 3 : 6;  // products per K-step and accumulator
  // Three planes over a long K: after every kFoldTiles K-tiles the accumulator
  // is added to a running sum and cleared (run<true>).  The matrix cores align
  // the 16 products of an MFMA to the accumulator and drop what lies below it,
  // which takes a little off every small product (hi * lo, mid * mid) once the
  // accumulator is large: over all of K = 18000 in one accumulator the sums of
  // a late iteration, whose terms are coherent, came out 6e-6 low; folded
  // every 1008 the error against 64 bits (W after five iterations at T=700,
  // G=18000: 1.1e-7) is below that of v_mfma_f32_32x32x2f32 (5.8e-7).
  static constexpr bool kFolds = NP == 3;
  static constexpr int kFoldTiles = (int)(kFoldK / BK_) / 3 * 3;
  // k of the first run of a range of `k`: what is summed before the first fold
  // (all of it where no fold follows).  The pipelined loop stops five K-tiles
  // before the end of its range and folds only inside it, so a shorter rest
  // stays in the accumulator; every layout of Y cuts a range in the same places.
  static __host__ __device__ constexpr int64_t fold_run(int64_t k) {
    return k < (int64_t)(kFoldTiles + 5) * BK_ ? k : (int64_t)kFoldTiles * BK_;
  }
  static_assert(!kFolds || (kFoldTiles + 5) * BK_ > kFoldK, "no fold where there is no scratch");
  static_assert(!YP || (YF32 && BN_ == (int)kPT && kPT % BK_ == 0 && (BK_ == 32 || BK_ == 16)),
                "packed Y: FP32 rows of one packed column block, K-tiles inside a block");
  // one block per CU (its stages fill most of the LDS): the epilogue has
  // the registers to fetch its per-entry operands 16 at a time (see epi_tile)
  static constexpr bool kPrefetchEpi = true;
  static constexpr int BM = BM_, BN = BN_, BK = BK_, NT = 64 * WM * WN;
  static constexpr int WAVES = WM * WN;
  // the block's waves spread over the CU's four SIMDs: eight waves give each
  // SIMD two, so one wave's waits are covered by the other's matrix work
  static_assert(WAVES % 4 == 0, "whole waves per SIMD");
  static constexpr int WAVES_PER_EU = WAVES / 4;
  static constexpr int TM = BM / WM / 32;
  static constexpr int TN = BN / WN / 32;
  static constexpr int KS = BK / 16;
  static_assert(TM >= 1 && TN >= 1 && (KS == 1 || KS == 2), "one or two 16-deep k-steps per K-tile");
  // Swizzle of FP32 Y rows (BK floats = BK / 4 chunks): chunk s of row r sits
  // in slot s ^ yswz(r), so the 16 rows a read touches at a time cover all
  // 64 banks (256 bytes hold 64 / BK rows).
  __device__ __forceinline__ static int yswz(int r) { return (r / (64 / BK)) % (BK / 4); }
  static_assert(STAGES == 2 || STAGES == 3, "two or three stages");
  using PX = TileLoadB3<BM, NT, BK>;  // swizzle of the bf16 planes
  using PY = TileLoadB3<BN, NT, BK>;
  static constexpr int CPR = BK / 8;  // 16-byte chunks per bf16 row
  static constexpr int XQ = BM * CPR; // chunks per X plane
  static constexpr int YQ = YF32 ? BN * (BK / 4) : NP * BN * CPR;  // chunks of the Y tile
  static constexpr int STAGE_BYTES = (NP * XQ + YQ) * 16;
  static constexpr int MAIN_BYTES = STAGES * STAGE_BYTES;
  static constexpr int XI = NP * XQ / 64, YI = YQ / 64;  // wave-instructions per stage
  static_assert((NP * XQ) % 64 == 0 && YQ % 64 == 0 && (XI + YI) % WAVES == 0, "load split");
  static constexpr int IPW = (XI + YI) / WAVES;  // loads per wave and stage
  static constexpr int YR = YF32 ? 2 : NP;       // 16-byte reads of a Y fragment
  static constexpr int PER = NP * TM + YR * TN;  // 16-byte fragment reads per k-step
  static constexpr int NR = KS * PER;
  // This wave's loads of one stage: wave-instruction q * WAVES + w of the
  // stage, so which operand (and plane) a load q reads is fixed at compile
  // time.
  static constexpr int XPW = XI / WAVES;  // X loads per wave (all planes)
  static constexpr int XPP = XPW / NP;    // ... per plane
  static constexpr int YPP = YI / WAVES / NP;  // Y loads per wave and plane (bf16 Y)
  static_assert(XI % (NP * WAVES) == 0, "X planes split evenly over the waves");
  static_assert(YF32 || YI % (NP * WAVES) == 0, "Y planes split evenly over the waves");

  floatx16 acc[TM][TN];
  int lane, wm, wn;

  struct Frag {  // operands of one K-tile
    bf16x8 x[NP][KS][TM], y[NP][KS][TN];
  };
  struct Raw {
    u4 r[NR];
  };
  using Split = unsigned[NP][KS][TN][4];  // split pairs of the FP32 Y fragments
  struct Dma {
    const char* x[NP];  // uniform bases at K-tile 0 of the range
    const char* y[NP];  // Y (FP32, y[0]) or its planes
    size_t xstep, ystep;  // bytes from one K-tile to the next
    unsigned voff[IPW];  // per lane
    unsigned wofs;       // this wave's LDS offset within a stage
    // packed Y: its base, the column block, the range start, and the per-lane
    // offsets of the K-tiles loaded as stored ([k][n])
    const char* yp;
    int64_t jb, kbeg;
    unsigned voffT[IPW];
  };
  // packed Y: whether K-tile kt of a range starting at kbeg is read as stored
  __device__ __forceinline__ static bool tr_at(const Dma& d, int kt) {
    if constexpr (!YP) return false;
    return d.jb > (d.kbeg + (int64_t)kt * BK) / kPT;
  }
  static constexpr int KT = plane_kt(NP);  // K depth of the planes' tiles
  static_assert(BK % KT == 0 && (BK == 16 || BK == 32), "whole plane tiles per K-tile");
  // bytes from a plane's (row r0, K-tile start) to row r, 16-byte chunk c of it
  __device__ __forceinline__ static unsigned plane_off(int64_t rows, int64_t r, int c) {
    return (unsigned)(((c / (KT / 8)) * rows * KT + r * KT + (c % (KT / 8)) * 8) * 2);
  }

  __device__ __forceinline__ static unsigned lds_addr(const void* p) {
    return (unsigned)(size_t)(const __attribute__((address_space(3))) char*)p;
  }

  __device__ __forceinline__ void setup(const Ops& o, int64_t m0, int64_t n0, int64_t kbeg, int w,
                                        Dma& d) const {
#pragma unroll
    for (int pl = 0; pl < NP; ++pl) {
      d.x[pl] = reinterpret_cast<const char*>(o.X.p + pl * o.X.stride +
                                              plane_index<KT>(o.X.rows, m0, kbeg));
      if constexpr (YP)
        d.y[pl] = nullptr;  // per K-tile, from the packed tile (dma_at)
      else if constexpr (YF32)
        d.y[pl] = reinterpret_cast<const char*>(o.Y + n0 * o.ldy + kbeg);
      else
        d.y[pl] = reinterpret_cast<const char*>(o.Y.p + pl * o.Y.stride +
                                                plane_index<KT>(o.Y.rows, n0, kbeg));
    }
    d.xstep = (size_t)o.X.rows * BK * 2;
    if constexpr (YP)
      d.ystep = 0;
    else if constexpr (YF32)
      d.ystep = BK * 4;
    else
      d.ystep = (size_t)o.Y.rows * BK * 2;
    d.wofs = (unsigned)w * 1024u;
    if constexpr (YP) {
      d.yp = reinterpret_cast<const char*>(o.Yp);
      d.jb = n0 / kPT;
      d.kbeg = kbeg;
    }
#pragma unroll
    for (int q = 0; q < IPW; ++q) {
      if (q < XPW) {
        const int p = ((q % XPP) * WAVES + w) * 64 + lane;  // chunk within the plane
        const int r = p / CPR, slot = p % CPR;
        const int chunk = slot ^ ((r / PX::RG) & (CPR - 1));
        // rows past the operand's end (M padded to the tile) re-read its last
        // row; their outputs are never stored
        const int64_t rr = (m0 + r < o.mrows ? m0 + r : o.mrows - 1) - m0;
        d.voff[q] = plane_off(o.X.rows, rr, chunk);
      } else if constexpr (YP) {
        const int p = ((q - XPW) * WAVES + w) * 64 + lane;
        const int r = p / (BK / 4), slot = p % (BK / 4);
        const int chunk = slot ^ yswz(r);
        d.voff[q] = (unsigned)(((int64_t)r * kPT + chunk * 4) * 4);  // rows of a packed tile
        // as stored: row kr of kPT floats (32 chunks), chunk c in slot c ^ 8 (kr / 8 % 2)
        const int kr = p / (int)(kPT / 4), s2 = p % (int)(kPT / 4);
        const int c2 = s2 ^ (((kr >> 3) & 1) << 3);
        d.voffT[q] = (unsigned)((kr * kPT + c2 * 4) * 4);
      } else if constexpr (YF32) {
        const int p = ((q - XPW) * WAVES + w) * 64 + lane;
        const int r = p / (BK / 4), slot = p % (BK / 4);
        const int chunk = slot ^ yswz(r);
        d.voff[q] = (unsigned)(((int64_t)r * o.ldy + chunk * 4) * 4);
      } else {
        const int p = (((q - XPW) % YPP) * WAVES + w) * 64 + lane;
        const int r = p / CPR, slot = p % CPR;
        const int chunk = slot ^ ((r / PY::RG) & (CPR - 1));
        d.voff[q] = plane_off(o.Y.rows, r, chunk);
      }
    }
  }

  // Direct load q of K-tile kt into the stage at LDS address sb (this wave's
  // part of it).
  __device__ __forceinline__ static void dma_at(const Dma& d, int q, int kt, unsigned sb) {
    const char* b;
    unsigned vo = d.voff[q];
    if (q < XPW) {
      b = d.x[q / XPP] + (size_t)kt * d.xstep;
    } else if constexpr (YP) {
      const int64_t k = d.kbeg + (int64_t)kt * BK, kb = k / kPT, kk = k % kPT;
      if (d.jb > kb) {  // tile (kb, jb): rows k, read as stored
        b = d.yp + (size_t)(packed_tile(kb, d.jb) * (kPT * kPT) + kk * kPT) * 4;
        vo = d.voffT[q];
      } else {          // tile (jb, kb): rows n, columns kk ..
        b = d.yp + (size_t)(packed_tile(d.jb, kb) * (kPT * kPT) + kk) * 4;
      }
    } else {
      b = d.y[YF32 ? 0 : (q - XPW) / (YPP > 0 ? YPP : 1)] + (size_t)kt * d.ystep;
    }
    lds_dma16(vo, b, sb + d.wofs + (unsigned)(q * WAVES) * 1024u);
  }
  __device__ __forceinline__ static void issue(const Dma& d, int kt, const char* st) {
#pragma unroll
    for (int q = 0; q < IPW; ++q) dma_at(d, q, kt, lds_addr(st));
  }

  // Packed Y read as stored: byte offset (within a stage) of this lane's
  // column n of fragment j, at the first of its 8 k (the rest at + kPT * 4 per k).
  __device__ __forceinline__ void read_offsets_t(unsigned (&adT)[TN]) const {
    const int khalf = lane >> 5;
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int n = wn * (BN / WN) + j * 32 + (lane & 31);
      adT[j] = (unsigned)NP * XQ * 16 + (unsigned)(8 * khalf) * (unsigned)(kPT * 4) +
               (((unsigned)(n >> 2) ^ (unsigned)(8 * khalf)) << 4) + 4u * (n & 3);
    }
  }
  // Read r of a K-tile's fragment reads: X and row-stored Y reads are 16
  // bytes at ad[r]; a packed Y K-tile read as stored takes four 4-byte reads
  // of consecutive k.
  template <bool TR>
  __device__ __forceinline__ static u4 read_r(const char* st, const unsigned (&ad)[NR],
                                              const unsigned (&adT)[TN], int r) {
    if constexpr (TR) {
      const int ks = r / PER, q = r % PER;
      if (q >= NP * TM) {
        const int j = (q - NP * TM) / 2, h = (q - NP * TM) % 2;
        const char* b = st + adT[j] + (unsigned)((16 * ks + 4 * h) * kPT * 4);
        return (u4){*reinterpret_cast<const unsigned*>(b),
                    *reinterpret_cast<const unsigned*>(b + kPT * 4),
                    *reinterpret_cast<const unsigned*>(b + 2 * kPT * 4),
                    *reinterpret_cast<const unsigned*>(b + 3 * kPT * 4)};
      }
    }
    return *reinterpret_cast<const u4*>(st + ad[r]);
  }

  // Byte offsets (within a stage) of this lane's fragment reads.
  __device__ __forceinline__ void read_offsets(unsigned (&ad)[NR]) const {
    const int mrow = wm * (BM / WM) + (lane & 31);
    const int khalf = lane >> 5;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const int chunk = 2 * ks + khalf;
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        const unsigned off = 2u * PX::swz(mrow + i * 32, chunk);
#pragma unroll
        for (int pl = 0; pl < NP; ++pl) ad[PER * ks + NP * i + pl] = off + 2u * pl * BM * BK;
      }
      const int c0 = 4 * ks + 2 * khalf;
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int n = wn * (BN / WN) + j * 32 + (lane & 31);
        if constexpr (YF32) {
          const unsigned yb = (unsigned)NP * XQ * 16 + 4u * n * BK;
          const int f = yswz(n);
          ad[PER * ks + NP * TM + 2 * j] = yb + 4u * ((c0 ^ f) << 2);
          ad[PER * ks + NP * TM + 2 * j + 1] = yb + 4u * (((c0 + 1) ^ f) << 2);
        } else {
          const unsigned off = (unsigned)NP * XQ * 16 + 2u * PY::swz(n, chunk);
#pragma unroll
          for (int pl = 0; pl < NP; ++pl)
            ad[PER * ks + NP * TM + NP * j + pl] = off + 2u * pl * BN * BK;
        }
      }
    }
  }

  template <bool TR>
  __device__ __forceinline__ static void read(const char* st, const unsigned (&ad)[NR],
                                              const unsigned (&adT)[TN], Raw& rw) {
#pragma unroll
    for (int i = 0; i < NR; ++i) rw.r[i] = read_r<TR>(st, ad, adT, i);
  }

  // Split pair sp of the next tile's FP32 Y fragments (4 pairs per fragment).
  __device__ __forceinline__ static void split_at(const Raw& rw, Split& o, int sp) {
    const int fi = sp / 4, pr = sp % 4, ks = fi / TN, j = fi % TN;
    const f4 v = __builtin_bit_cast(f4, rw.r[PER * ks + NP * TM + 2 * j + pr / 2]);
    const float a = pr % 2 == 0 ? v.x : v.z, b = pr % 2 == 0 ? v.y : v.w;
    unsigned t[3];
    if constexpr (NP == 2)
      split_pair(a, b, t[0], t[1]);
    else
      split_pair3(a, b, t);
#pragma unroll
    for (int pl = 0; pl < NP; ++pl) {
      o[pl][ks][j][pr] = t[pl];
      // keep the pair here, between its MFMAs (the compiler would otherwise
      // sink it to the end of the K-tile, next to its first use)
      asm volatile("" : "+v"(o[pl][ks][j][pr]));
    }
  }
  static constexpr int NSP = YF32 ? KS * TN * 4 : 0;  // split pairs per K-tile

  // Fragments of a K-tile from its LDS reads (and split pairs).
  __device__ __forceinline__ static void assemble(const Raw& rw, const Split& sp, Frag& f) {
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int pl = 0; pl < NP; ++pl) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
          f.x[pl][ks][i] = __builtin_bit_cast(bf16x8, rw.r[PER * ks + NP * i + pl]);
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          if constexpr (YF32)
            f.y[pl][ks][j] = __builtin_bit_cast(
                bf16x8, (u4){sp[pl][ks][j][0], sp[pl][ks][j][1], sp[pl][ks][j][2], sp[pl][ks][j][3]});
          else
            f.y[pl][ks][j] = __builtin_bit_cast(bf16x8, rw.r[PER * ks + NP * TM + NP * j + pl]);
        }
      }
  }
  __device__ __forceinline__ static void split(const Raw& rw, Frag& f) {
    Split sp;
#pragma unroll
    for (int k = 0; k < NSP; ++k) split_at(rw, sp, k);
    assemble(rw, sp, f);
  }

  // One MFMA of a K-tile: m = ((ks * NPROD + product) * TM + i) * TN + j.
  // Consecutive MFMAs go to different accumulators and never wait for each
  // other; the small products of a K-step come before the leading one.
  __device__ __forceinline__ void mfma_at(const Frag& f, int m) {
    constexpr int XP[6] = {2, 0, 1, 1, 0, 0}, YPL[6] = {0, 2, 1, 0, 1, 0};
    constexpr int X2[3] = {0, 1, 0}, Y2[3] = {1, 0, 0};
    const int j = m % TN, i = (m / TN) % TM, p = (m / TN / TM) % NPROD, ks = m / TN / TM / NPROD;
    const int xp = NP == 2 ? X2[p % 3] : XP[p], yp = NP == 2 ? Y2[p % 3] : YPL[p];
    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.x[xp][ks][i], f.y[yp][ks][j], acc[i][j],
                                                        0, 0, 0);
  }
  __device__ __forceinline__ void mfma(const Frag& f) {
#pragma unroll
    for (int m = 0; m < KS * NPROD * TM * TN; ++m) mfma_at(f, m);
  }

  // K-tile kt whose STAGES successors exist: stage `rd` holds tile kt + 1,
  // stage `fr` held tile kt (already in registers) and takes tile
  // kt + STAGES.  The MFMAs of tile kt are issued one by one, each followed
  // by work of the next tile that does not depend on them: first the direct
  // loads of tile kt + STAGES and the LDS reads of tile kt + 1, then the
  // split of tile kt + 1's C fragments.  Scheduling barriers keep this order
  // (the matrix core runs each MFMA while the wave issues what follows it).
  template <bool TR>
  __device__ __forceinline__ void full_step(const Dma& d, const unsigned (&ad)[NR],
                                            const unsigned (&adT)[TN], int kt, const char* rd,
                                            const char* fr, Frag& cur) {
    constexpr int NM = KS * TM * TN * NPROD;  // MFMAs per K-tile
    constexpr int NRM = (NR + 1) / 2;     // MFMAs followed by reads
    static_assert(IPW <= NM, "one direct load per MFMA slot at most");
    wait_vmem<(STAGES - 2) * IPW>();  // tile kt + 1 landed (later ones may be in flight)
    wave_barrier_mem();
    __builtin_amdgcn_sched_barrier(0);
    const unsigned sb = lds_addr(fr);
    Raw rw;
    Split sp;
#pragma unroll
    for (int m = 0; m < NM; ++m) {
      mfma_at(cur, m);
      if (m < IPW) dma_at(d, m, kt + STAGES, sb);
      if (m < NRM) {
#pragma unroll
        for (int r = 2 * m; r < 2 * m + 2 && r < NR; ++r) rw.r[r] = read_r<TR>(rd, ad, adT, r);
      } else if (m - NRM < NSP) {
        split_at(rw, sp, m - NRM);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int m = NM; m < NRM + NSP; ++m) split_at(rw, sp, m - NRM);  // left over
    assemble(rw, sp, cur);
  }

  // Packed Y: K-tiles [0, ksplit) of the range lie below the diagonal.
  __device__ __forceinline__ static int ksplit_of(const Dma& d, int nk) {
    const int64_t ks = (d.jb * kPT - d.kbeg + BK - 1) / BK;
    return ks <= 0 ? 0 : ks >= nk ? nk : (int)ks;
  }

  // Any K-tile (near the end of the range): the same with bounds.
  __device__ __forceinline__ void tail_step(const Dma& d, const unsigned (&ad)[NR],
                                            const unsigned (&adT)[TN], int kt, int nk,
                                            const char* rd, const char* fr, Frag& cur) {
    if (kt + 1 < nk) {
      if (STAGES == 3 && kt + 2 < nk) wait_vmem<IPW>(); else wait_vmem<0>();
      wave_barrier_mem();
      if (kt + STAGES < nk) issue(d, kt + STAGES, fr);
      Raw rw;
      if (tr_at(d, kt + 1))
        read<true>(rd, ad, adT, rw);
      else
        read<false>(rd, ad, adT, rw);
      mfma(cur);
      split(rw, cur);
    } else {
      mfma(cur);
    }
  }

  // The running sum of a thread's entries, 16 bytes per thread at a time (its
  // own entries: no other thread reads them): the first LQ of its kFoldQ
  // chunks in LDS past the stages, the others in the block's slot in memory.
  static constexpr int kFoldQ = TM * TN * 4;
  template <int LQ>
  static constexpr int fold_lds_bytes() { return LQ * NT * 16; }
  template <int LQ>
  __device__ __forceinline__ f4* fold_at(char* smem, float* slot, int c) const {
    return c < LQ ? reinterpret_cast<f4*>(smem + MAIN_BYTES) + c * NT + threadIdx.x
                  : reinterpret_cast<f4*>(slot) + (c - LQ) * NT + threadIdx.x;
  }
  template <int LQ>
  __device__ __forceinline__ void fold(char* smem, float* slot, bool first) {
#pragma unroll
    for (int c = kFoldQ - 1; c >= 0; --c) {  // (memory first: its loads take longer)
      floatx16& a = acc[c / 4 / TN][c / 4 % TN];
      f4 v;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        v[e] = a[4 * (c % 4) + e];
        a[4 * (c % 4) + e] = 0.0f;
      }
      if (!first) v += *fold_at<LQ>(smem, slot, c);
      *fold_at<LQ>(smem, slot, c) = v;
    }
  }
  template <int LQ>
  __device__ __forceinline__ void unfold(char* smem, float* slot) {
#pragma unroll
    for (int c = kFoldQ - 1; c >= 0; --c) {
      const f4 v = *fold_at<LQ>(smem, slot, c);
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[c / 4 / TN][c / 4 % TN][4 * (c % 4) + e] += v[e];
    }
  }
  // The product over a long K (three planes).  Packed Y restarts the loop
  // after every fold: its two loops with the fold between their steps spill
  // 288 registers.
  template <int LQ>
  __device__ __forceinline__ void run_long(const Ops& o, int64_t m0, int64_t n0, int64_t kbeg,
                                           int64_t kend, char* smem, float* slot) {
    if constexpr (!YP) {
      run<LQ>(o, m0, n0, kbeg, kend, smem, slot);
    } else {
      for (int64_t k = kbeg;;) {
        const int64_t n = fold_run(kend - k);
        run(o, m0, n0, k, k + n, smem);
        if (k + n >= kend) {
          if (k != kbeg) unfold<LQ>(smem, slot);
          return;
        }
        fold<LQ>(smem, slot, k == kbeg);
        k += n;
      }
    }
  }

  // The product over a short K (three planes of both operands; the planes are
  // zero past it).
  __device__ __forceinline__ void run_short(const Ops& o, int64_t m0, int64_t n0, int64_t K,
                                            char* smem) {
    static_assert(NP == 3 && !YF32 && KT >= kShortK, "whole operands, one K-tile");
    lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    wm = w % WM;
    wn = w / WM;
    auto terms = [](double* s, const Planes& P, int64_t row) {
      const bf16_t* p = P.p + plane_index<KT>(P.rows, row, 0);
      const bf16x8 hi = *reinterpret_cast<const bf16x8*>(p);
      const bf16x8 mid = *reinterpret_cast<const bf16x8*>(p + P.stride);
      const bf16x8 lo = *reinterpret_cast<const bf16x8*>(p + 2 * P.stride);
#pragma unroll
      for (int k = 0; k < (int)kShortK; ++k)
        s[k] = (double)(float)hi[k] + ((double)(float)mid[k] + (double)(float)lo[k]);
    };
    short_product(*this, (int)K, smem, [&](double* xs, double* ys) {
      for (int q = threadIdx.x; q < BM; q += NT)
        terms(xs + q * kShortLd, o.X, m0 + q < o.mrows ? m0 + q : o.mrows - 1);
      for (int q = threadIdx.x; q < BN; q += NT) terms(ys + q * kShortLd, o.Y, n0 + q);
    });
  }

  // LQ >= 0: fold a long K (see run_long).
  template <int LQ = -1>
  __device__ __forceinline__ void run(const Ops& o, int64_t m0, int64_t n0, int64_t kbeg,
                                      int64_t kend, char* smem, float* slot = nullptr) {
    constexpr bool FOLD = LQ >= 0;
    static_assert(!FOLD || STAGES == 3, "folded in the three-stage loop");
    int to_fold = kFoldTiles;
    bool folded = false;
    // n more K-tiles are in the accumulator; whether it was folded for them
    auto stepped = [&](int n) {
      to_fold -= n;
      if (to_fold > 0) return false;
      if constexpr (FOLD) fold<LQ>(smem, slot, !folded);
      folded = true;
      to_fold = kFoldTiles;
      return true;
    };
    char* const s0 = smem;
    char* const s1 = smem + STAGE_BYTES;
    char* const s2 = smem + (STAGES == 3 ? 2 * STAGE_BYTES : 0);
    lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    wm = w % WM;
    wn = w / WM;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
    const int nk = (int)((kend - kbeg) / BK);
    // Every wave of the block is done with the stages (and with whatever the
    // caller kept in the same shared memory).
    wait_vmem<0>();
    wave_barrier_mem();
    if (nk <= 0) return;
    Dma d;
    setup(o, m0, n0, kbeg, w, d);
    unsigned ad[NR];
    read_offsets(ad);
    unsigned adT[TN];
    if constexpr (YP) read_offsets_t(adT);
    issue(d, 0, s0);
    if (nk > 1) {
      issue(d, 1, s1);
      wait_vmem<IPW>();
    } else {
      wait_vmem<0>();
    }
    wave_barrier_mem();
    if (STAGES == 3 && nk > 2) issue(d, 2, s2);
    // A wave whose rows all lie past the operand's end (M padded to the tile)
    // only takes its share of the loads and barriers: no reads, no MFMAs.
    // (Only the A product pads M.)
    if (YF32 && m0 + wm * (BM / WM) >= o.mrows) {
      for (int kt = 0; kt + 1 < nk; ++kt) {
        if (STAGES == 3 && kt + 2 < nk) wait_vmem<IPW>(); else wait_vmem<0>();
        wave_barrier_mem();
        if (kt + STAGES < nk) issue(d, kt + STAGES, kt % STAGES == 0 ? s0 : kt % STAGES == 1 ? s1 : s2);
      }
      wave_barrier_mem();
      return;
    }
    Frag cur;
    {
      Raw rw;
      if (tr_at(d, 0))
        read<true>(s0, ad, adT, rw);
      else
        read<false>(s0, ad, adT, rw);
      split(rw, cur);
    }
    int kt = 0;
    if constexpr (STAGES == 3) {
      // Packed Y: the K-tiles below the diagonal (k < jb kPT, read as stored)
      // come first, then the others; each run of one orientation gets its own
      // loop (a choice between the two inside one loop costs the register
      // allocator hundreds of spilled registers).  Reads of tile kt + 1.
      const int ksplit = YP ? ksplit_of(d, nk) : 0;
      auto stg = [&](int k) { const int m = k % 3; return m == 0 ? s0 : m == 1 ? s1 : s2; };
      // runs of whole loop steps up to the next fold
      for (;;) {
        const int end = FOLD && kt + to_fold < ksplit - 3 ? kt + to_fold : ksplit - 3;
        const int kt0 = kt;
        for (; kt + 5 < nk && kt < end; kt += 3) {
          full_step<true>(d, ad, adT, kt, s1, s0, cur);
          full_step<true>(d, ad, adT, kt + 1, s2, s1, cur);
          full_step<true>(d, ad, adT, kt + 2, s0, s2, cur);
        }
        if (!FOLD || !stepped(kt - kt0)) break;
      }
      for (; kt + 5 < nk && kt + 1 < ksplit; ++kt) {
        full_step<true>(d, ad, adT, kt, stg(kt + 1), stg(kt), cur);
        if constexpr (FOLD) to_fold -= 1;
      }
      for (; kt + 5 < nk && kt % 3 != 0; ++kt) {
        full_step<false>(d, ad, adT, kt, stg(kt + 1), stg(kt), cur);
        if constexpr (FOLD) to_fold -= 1;
      }
      for (;;) {
        const int end = FOLD && kt + to_fold < nk - 5 ? kt + to_fold : nk - 5;
        const int kt0 = kt;
        for (; kt < end; kt += 3) {
          full_step<false>(d, ad, adT, kt, s1, s0, cur);
          full_step<false>(d, ad, adT, kt + 1, s2, s1, cur);
          full_step<false>(d, ad, adT, kt + 2, s0, s2, cur);
        }
        if (!FOLD || !stepped(kt - kt0)) break;
      }
      for (; kt < nk; ++kt) tail_step(d, ad, adT, kt, nk, stg(kt + 1), stg(kt), cur);
      if constexpr (FOLD) {
        if (folded) unfold<LQ>(smem, slot);
      }
    } else {
      static_assert(!YP, "packed Y takes three stages");
      for (; kt + 3 < nk; kt += 2) {
        full_step<false>(d, ad, adT, kt, s1, s0, cur);
        full_step<false>(d, ad, adT, kt + 1, s0, s1, cur);
      }
      for (; kt < nk; ++kt) {
        const bool ph = kt % 2;
        tail_step(d, ad, adT, kt, nk, ph ? s0 : s1, ph ? s1 : s0, cur);
      }
    }
    // the caller may reuse the shared memory once every wave has read its last stage
    wave_barrier_mem();
  }

  __device__ __forceinline__ int row_of(int i, int r) const {
    return wm * (BM / WM) + i * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
  }
  __device__ __forceinline__ int col_of(int j) const {
    return wn * (BN / WN) + j * 32 + (lane & 31);
  }
  template <class F>
  __device__ __forceinline__ void for_each(F&& f) const {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int c = col_of(j);
#pragma unroll
        for (int r = 0; r < 16; ++r) f(row_of(i, r), c, acc[i][j][r]);
      }
  }
};

// Block GEMMs whose sums over a long K are folded (BlockGemmB3P of three
// planes): run over [kbeg, kend) with the running sum in `slot`.
template <class G, class = void>
struct folds_k : std::false_type {};
template <class G>
struct folds_k<G, std::void_t<decltype(G::kFolds)>> : std::integral_constant<bool, G::kFolds> {};
template <class G>
__host__ __device__ constexpr int rect_fold_lds() {  // chunks of the running sum kept in LDS
  if constexpr (folds_k<G>::value) return 7;
  else return 0;
}
template <class G>
__host__ __device__ constexpr int rect_smem_bytes() {
  if constexpr (folds_k<G>::value)
    return G::MAIN_BYTES + G::template fold_lds_bytes<rect_fold_lds<G>()>();
  else
    return G::MAIN_BYTES;
}
template <class G>
__device__ __forceinline__ void run_rect(G& g, const typename G::Ops& ops, int64_t m0, int64_t n0,
                                         int64_t kbeg, int64_t kend, char* smem, float* slot) {
  if constexpr (folds_k<G>::value)
    g.template run_long<rect_fold_lds<G>()>(ops, m0, n0, kbeg, kend, smem, slot);
  else
    g.run(ops, m0, n0, kbeg, kend, smem);
}

// ======================================================= tile schedule ==
// A grid of nb blocks (as many as the GPU runs at once) covers nTiles output
// tiles of U K-steps each in two parts:
//   full rounds: with R = nTiles / nb, block L computes tiles L, L + nb, ...,
//     L + (R-1) nb whole.  Consecutive tiles (M fastest, sharing a strip of
//     the Y operand) run on one XCD at the same time, so that strip and the
//     X tiles they need are fetched from memory about once per round.
//   tail: the T = nTiles - R nb remaining tiles are cut into S equal K-chunks
//     each, and item i = c T + t (chunk c of tail tile t) goes to block i mod
//     nb.  Items are numbered chunk first, so the blocks of one XCD work on
//     the same K-chunk of neighbouring tiles at the same time and keep
//     sharing operand strips in L2, as in a full round.  With S = 1 a block
//     finishes the tile itself; otherwise it stores its partial product and
//     the fix-up kernel adds the S partials of each tile in chunk order
//     (deterministic; no block ever waits for another).  The host picks S
//     to minimise the largest tail load of a block.
// Logical block numbers are assigned XCD by XCD (the hardware hands block b to
// XCD b % 8), so one XCD works on contiguous tiles.
// The epilogue of a finished tile.  Where the block GEMM allows it
// (kPrefetchEpi) and the epilogue reads operands of its own per entry
// (fetch), those are loaded for the 16 entries of one accumulator block
// before any is used, so the loads are in flight together instead of one
// dependent load per entry.  Same arithmetic, same order, either way.
template <class E, class = void>
struct has_fetch : std::false_type {};
template <class E>
struct has_fetch<E, std::void_t<decltype(&E::fetch)>> : std::true_type {};
// Epi::Pre where the epilogue fetches its operands ahead, else a placeholder.
template <class E, class = void>
struct fetch_t {
  struct type {};
};
template <class E>
struct fetch_t<E, std::void_t<typename E::Pre>> {
  using type = typename E::Pre;
};
template <class G, class = void>
struct prefetch_epi : std::false_type {};
template <class G>
struct prefetch_epi<G, std::void_t<decltype(G::kPrefetchEpi)>>
    : std::integral_constant<bool, G::kPrefetchEpi> {};

// Epilogues with a block<N>(rows, cols, acc) member take N entries at once:
// every operand of the N entries is loaded before the first result is
// stored (a store may alias an operand buffer, so entry by entry each
// entry's loads would wait for the store before them).
template <class E, class = void>
struct has_block : std::false_type {};
template <class E>
struct has_block<E, std::void_t<decltype(&E::template block<16>)>> : std::true_type {};
// Block GEMMs whose epilogue takes entries in runs (kBlockEpi); the others
// keep their registers for occupancy (measured: the FP32 products run
// slower with the extra live operands).
template <class G, class = void>
struct block_epi : std::false_type {};
template <class G>
struct block_epi<G, std::void_t<decltype(G::kBlockEpi)>>
    : std::integral_constant<bool, G::kBlockEpi> {};

// The epilogue of a tile in runs of NB entries of one column (Epi::block):
// all operands of a run are loaded before any of its results is stored.
template <int NB, class G, class Epi>
__device__ __forceinline__ void epi_tile_runs(const G& g, Epi& epi, int64_t m0, int64_t n0) {
  static_assert(16 % NB == 0, "whole runs per accumulator column");
#pragma unroll
  for (int i = 0; i < G::TM; ++i)
#pragma unroll
    for (int j = 0; j < G::TN; ++j)
#pragma unroll
      for (int r0 = 0; r0 < 16; r0 += NB) {
        int64_t rs[NB], cs[NB];
        float a[NB];
#pragma unroll
        for (int r = 0; r < NB; ++r) {
          rs[r] = m0 + g.row_of(i, r0 + r);
          cs[r] = n0 + g.col_of(j);
          a[r] = g.acc[i][j][r0 + r];
        }
        epi.template block<NB>(rs, cs, a);
      }
}

template <class G, class Epi>
__device__ __forceinline__ void epi_tile(const G& g, Epi& epi, int64_t m0, int64_t n0) {
  if constexpr (has_fetch<Epi>::value && prefetch_epi<G>::value) {
#pragma unroll
    for (int i = 0; i < G::TM; ++i)
#pragma unroll
      for (int j = 0; j < G::TN; ++j) {
        const int64_t c = n0 + g.col_of(j);
        typename Epi::Pre pre[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) pre[r] = epi.fetch(m0 + g.row_of(i, r), c);
#pragma unroll
        for (int r = 0; r < 16; ++r) epi.element_pre(m0 + g.row_of(i, r), c, g.acc[i][j][r], pre[r]);
      }
  } else if constexpr (has_block<Epi>::value && block_epi<G>::value) {
    epi_tile_runs<8>(g, epi, m0, n0);
  } else {
    g.for_each([&](int rr, int c, float v) { epi.element(m0 + rr, n0 + c, v); });
  }
}

template <class G, class Epi>
__global__ __launch_bounds__(G::NT) __attribute__((amdgpu_waves_per_eu(G::WAVES_PER_EU)))
void k_rect_streamk(typename G::Ops ops, int64_t nMT, int64_t nTiles, int64_t U, int64_t S,
                    Epi epi, float* __restrict__ part, float* __restrict__ fold,
                    const int32_t* gate) {
  if (gate && *gate == 0) return;
  __shared__ __align__(16) char smem[rect_smem_bytes<G>()];
  float* const slot = fold + (int64_t)blockIdx.x * (G::BM * G::BN);
  __shared__ double red[G::NT / 64];
  const int64_t nb = gridDim.x;
  const int64_t L = xcd_tile(blockIdx.x, nb);
  const int64_t R = nTiles / nb, nFull = R * nb, T = nTiles - nFull;
  G g;
  for (int64_t r = 0; r < R; ++r) {
    const int64_t tile = r * nb + L;
    const int64_t m0 = (tile % nMT) * G::BM, n0 = (tile / nMT) * G::BN;
    run_rect(g, ops, m0, n0, 0, U * G::BK, smem, slot);
    epi_tile(g, epi, m0, n0);
    epi.end_tile(tile, red);
  }
  for (int64_t i = L; i < T * S; i += nb) {
    const int64_t c = i / T, tile = nFull + i % T;
    const int64_t m0 = (tile % nMT) * G::BM, n0 = (tile / nMT) * G::BN;
    run_rect(g, ops, m0, n0, c * U / S * G::BK, (c + 1) * U / S * G::BK, smem, slot);
    if (S == 1) {
      epi_tile(g, epi, m0, n0);
      epi.end_tile(tile, red);
    } else {
      float* ps = part + i * (int64_t)(G::BM * G::BN);
      g.for_each([&](int rr, int c2, float v) { ps[rr * G::BN + c2] = v; });
    }
  }
}

// Tail tiles computed in S > 1 K-chunks: add the partial products in chunk
// order (deterministic) and run the epilogue.  1024 threads per block: the
// epilogue's loads form a dependent chain per element, so the fix-up runs as
// many waves per tile as a block holds, and a tile of more than 8 entries per
// thread is shared by kFixParts(G) blocks of 8 entries per thread each (one
// round of loads per thread instead of several in a row).  Block part q > 0
// of tile `tile` leaves its share of the h sum in slot q * nTiles + tile of
// the epilogue's per-tile partials, part 0 in slot `tile`.
constexpr int kFixThreads = 1024;
template <class G>
constexpr int kFixParts = (G::BM * G::BN) / kFixThreads > 8 ? (G::BM * G::BN) / kFixThreads / 8 : 1;
template <class G, class Epi>
__global__ __launch_bounds__(kFixThreads) void k_rect_fixup(int64_t nMT, int64_t nTiles, int64_t nb,
                                                            int64_t S,
                                                            const float* __restrict__ part, Epi epi,
                                                            const int32_t* gate) {
  if (gate && *gate == 0) return;
  __shared__ double red[kFixThreads / 64];
  constexpr int Q = kFixParts<G>;
  const int64_t nFull = (nTiles / nb) * nb, T = nTiles - nFull;
  const int64_t t = blockIdx.x / Q, tile = nFull + t;
  const int qb = (int)(blockIdx.x % Q);
  const int64_t m0 = (tile % nMT) * G::BM, n0 = (tile / nMT) * G::BN;
  constexpr int E = G::BM * G::BN;
  static_assert(E % (kFixThreads * Q) == 0, "whole passes");
  // entries e = threadIdx.x + q kFixThreads, q in this block's share [q_lo,
  // q_lo + PER), taken GRP at a time: their partials (and the epilogue's own
  // operands) are loaded together, then summed in chunk order and finished
  // in the order of q
  constexpr int PER = E / kFixThreads / Q, GRP = PER < 8 ? PER : 8;
  static_assert(PER % GRP == 0, "whole groups");
  const int q_lo = qb * PER;
  for (int q0 = q_lo; q0 < q_lo + PER; q0 += GRP) {
    // the epilogue's own operands first, then the partials of up to two
    // chunks at a time, all in flight before they are added in chunk order
    typename fetch_t<Epi>::type pre[GRP];
    if constexpr (has_fetch<Epi>::value) {
#pragma unroll
      for (int q = 0; q < GRP; ++q) {
        const int e = threadIdx.x + (q0 + q) * kFixThreads;
        pre[q] = epi.fetch(m0 + e / G::BN, n0 + e % G::BN);
      }
    }
    float s[GRP];
#pragma unroll
    for (int q = 0; q < GRP; ++q) s[q] = part[t * E + threadIdx.x + (q0 + q) * kFixThreads];
    constexpr int CH = 2;
    for (int64_t c = 1; c < S; c += CH) {
      float v[CH][GRP];
#pragma unroll
      for (int k = 0; k < CH; ++k)
        if (c + k < S)
#pragma unroll
          for (int q = 0; q < GRP; ++q)
            v[k][q] = part[((c + k) * T + t) * E + threadIdx.x + (q0 + q) * kFixThreads];
#pragma unroll
      for (int k = 0; k < CH; ++k)
        if (c + k < S)
#pragma unroll
          for (int q = 0; q < GRP; ++q) s[q] += v[k][q];
    }
    if constexpr (has_block<Epi>::value && !has_fetch<Epi>::value) {
      int64_t rs[GRP], cs[GRP];
#pragma unroll
      for (int q = 0; q < GRP; ++q) {
        const int e = threadIdx.x + (q0 + q) * kFixThreads;
        rs[q] = m0 + e / G::BN;
        cs[q] = n0 + e % G::BN;
      }
      epi.template block<GRP>(rs, cs, s);
    } else if constexpr (has_fetch<Epi>::value) {
#pragma unroll
      for (int q = 0; q < GRP; ++q) {
        const int e = threadIdx.x + (q0 + q) * kFixThreads;
        epi.element_pre(m0 + e / G::BN, n0 + e % G::BN, s[q], pre[q]);
      }
    } else {
#pragma unroll
      for (int q = 0; q < GRP; ++q) {
        const int e = threadIdx.x + (q0 + q) * kFixThreads;
        epi.element(m0 + e / G::BN, n0 + e % G::BN, s[q]);
      }
    }
  }
  epi.end_tile(qb * nTiles + tile, red);
}

constexpr int64_t kPartTile = 64 * 128;  // floats of a unit of split-tile scratch
constexpr int64_t kFoldBlocks = 256;  // folding slots of a rectangular product

inline int64_t device_cus() {
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      cus <= 0)
    cus = 256;
  return cus;
}

// Blocks of kernel `fn` (nt threads each) the whole GPU runs at once.
inline int64_t resident_blocks(const void* fn, int nt = kThreads) {
  const int64_t cus = device_cus();
  int occ = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, fn, nt, 0) != hipSuccess || occ <= 0)
    occ = 1;
  return cus * occ;
}

// Launch of a rectangular product over an Mp x Np output with K = Kp; part
// holds 2 * kMaxStreamKBlocks tiles of split-tile scratch.
template <class G, class Epi>
hipError_t launch_rect(const typename G::Ops& ops, int64_t Mp, int64_t Np, int64_t Kp, Epi epi,
                       float* part, const int32_t* gate, hipStream_t s, float* fold = nullptr) {
  // computed once per kernel (a function-local static: thread-safe initialisation)
  static const int64_t fits =
      resident_blocks(reinterpret_cast<const void*>(&k_rect_streamk<G, Epi>), G::NT);
  int64_t resident = fits;
  static const int64_t cus = device_cus();
  // blocks with a folding slot of their own
  if (folds_k<G>::value && resident > kFoldBlocks) resident = kFoldBlocks;
  if (folds_k<G>::value && Kp > kFoldK && !fold) return hipErrorInvalidValue;
  const int64_t nMT = Mp / G::BM, nNT = Np / G::BN;
  const int64_t nTiles = nMT * nNT, U = Kp / G::BK;
  // K-chunks per tail tile: the smallest S with the least cost, counted in
  // K-steps: the largest block load (with start-up per item) plus the fix-up,
  // which reads S partials per entry; the partials must fit the scratch
  // (2 * kMaxStreamKBlocks tiles of 64 x 128).
  const int64_t cap = 2 * kMaxStreamKBlocks * kPartTile / (G::BM * G::BN);
  constexpr int64_t kItemCost = 8;
  // A product of fewer tiles than CUs is all tail: with S = 1 a block per
  // tile would leave the other CUs idle for the whole of K.  Blocks of one CU
  // share its matrix cores (n of them run about 0.6 n times as long as one
  // alone), and cutting must save more than the fix-up's launch (about ten
  // K-steps).  A + W at 200 x 4000 split-BF16 (32 tiles): 151 -> 33 + 13 us; a
  // product of 440 tiles gains nothing from it (0.97x).
  const bool starved = nTiles < cus;
  const int64_t T = starved ? nTiles : nTiles % std::min(resident, nTiles);
  int64_t S = 1, best = T ? ((T + resident - 1) / resident) * (U + kItemCost) : 0;
  for (int64_t c = 2; T && c <= 64 && c <= U && T * c <= cap; ++c) {
    const int64_t steps = (U + c - 1) / c + kItemCost, per_cu = (T * c + cus - 1) / cus;
    const int64_t load = starved ? (per_cu > 1 ? 6 * per_cu * steps / 10 : steps) + c + 10
                                 : ((T * c + resident - 1) / resident) * steps + c;
    if (load < best) {
      best = load;
      S = c;
    }
  }
  // whole rounds of `nb` tiles, then the items of the tail (see the kernel)
  const int64_t nb = starved ? std::min(T * S, resident) : std::min(resident, nTiles);
  k_rect_streamk<G, Epi><<<dim3((unsigned)nb), dim3(G::NT), 0, s>>>(ops, nMT, nTiles, U, S, epi,
                                                                     part, fold, gate);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (T == 0 || S == 1) return hipSuccess;  // (starved with S = 1: one whole round)
  k_rect_fixup<G, Epi><<<dim3((unsigned)(T * kFixParts<G>)), dim3(kFixThreads), 0, s>>>(
      nMT, nTiles, nb, S, part, epi, gate);
  return hipGetLastError();
}

}  // namespace gemm
}  // namespace panda

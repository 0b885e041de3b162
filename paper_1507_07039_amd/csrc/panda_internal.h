// Internal declarations shared by the HIP sources of libpanda.so.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace panda {

// Device-resident iteration state.  Kernels read the gates and skip their
// work once the run has converged, so the host can enqueue iterations ahead
// of reading h back.
struct DevState {
  double h;        // h of the last completed iteration (Eq. 7)
  int32_t t;       // number of completed iterations (t of Eq. 6 during the P/C phase)
  int32_t active;  // 1 while h >= tol: gates R, A, W and h
  int32_t run_pc;  // 1 when the current iteration updates P and C: gates Eq. 5-6
  int32_t conv;    // 1 once h < tol
  int32_t wsel;    // index (0/1) of the buffer holding the current W; flipped with t
  int32_t stepped; // small kernels: whether the last launched iteration advanced t
};

// Scalars of the update rules.
struct Rule {
  double alpha;
  double tol;
  int32_t diag_alpha;
  int32_t sigma_from_T;
  int32_t n_own;
  int32_t h_undamped;
  int32_t update_last;
  int32_t sigma_ddof;
};

typedef unsigned short bf16_t;           // raw bits of a bfloat16

// An FP32 matrix (rows x K, products contract over K) given as bf16 planes,
// plane q at p + q * stride, leading term first: two planes x = hi + lo to
// 2^-17, three planes x = hi + mid + lo, exactly from 2^-110 up (and at 0); below
// it to 2^-134, what is left there being finer than the smallest bf16.  A plane is stored K-tile by
// K-tile, [K / KT][rows][KT] with KT = plane_kt(planes), the K-tile depth of
// the products: the direct-to-LDS loads of a tile then read whole cache lines
// (row-major, a K-tile of 16 took 32 bytes of each row, 32 lines per load
// instruction instead of 8, and the loads bound the C update).
struct Planes {
  bf16_t* p;
  int64_t stride;
  int64_t rows;
};
__host__ __device__ constexpr int plane_kt(int planes) { return planes == 2 ? 32 : 16; }
template <int KT>
__host__ __device__ constexpr int64_t plane_index(int64_t rows, int64_t r, int64_t k) {
  return (k / KT * rows + r) * KT + k % KT;
}
// Where three planes are all that holds a matrix (W of a single network in the
// FP32 form), a fourth keeps the lower 16 bits of each entry, whose upper 16 are
// hi: entry (r, k), bit for bit.
constexpr int kHeldPlanes = 4;
__device__ __forceinline__ float join_planes(const Planes& P, int64_t r, int64_t k) {
  const bf16_t* p = P.p + plane_index<plane_kt(3)>(P.rows, r, k);
  return __builtin_bit_cast(float, ((unsigned)p[0] << 16) | p[3 * P.stride]);
}

constexpr int kThreads = 256;            // threads per block (4 waves of 64)
constexpr int64_t kMaxStreamKBlocks = 1024;
constexpr int kColChunks = 64;           // row chunks of the column-norm kernel

// Padding of the internal state: TF dimension to 64, gene dimension to 128.
constexpr int64_t kPadE = 64;
constexpr int64_t kPadA = 128;
constexpr int64_t kPadK = 32;            // K of a stand-alone similarity product
constexpr int64_t kCoopTile = 64;        // tile side of the W W^T partial products
inline int64_t round_up(int64_t x, int64_t m) { return (x + m - 1) / m * m; }

// Packed-symmetric storage of C (an option of the single-network context):
// only the upper kPT x kPT tiles (a <= b) of the padded N_a x N_a matrix,
// tile (a, b) at index b (b + 1) / 2 + a, each tile row-major with its own
// row length kPT.  An upper tile serves both triangles: C[i][j] for i in
// block a, j in block b is tile (a, b) entry (i mod kPT, j mod kPT), and
// C[j][i] is the same entry.  Diagonal tiles hold both of their triangles
// (they are symmetric), so any row of them can be read directly.
constexpr int64_t kPT = 128;
__host__ __device__ inline int64_t packed_tile(int64_t a, int64_t b) { return b * (b + 1) / 2 + a; }
inline int64_t packed_floats(int64_t Nap) {
  const int64_t nT = Nap / kPT;
  return nT * (nT + 1) / 2 * kPT * kPT;
}

// ------------------------------------------------------------ launchers --
// Rectangular similarity products (stream-K).  X is Mp x Kp (k contiguous),
// Y is Kp x Np (n contiguous); Mp % 64 == 0, Np % 128 == 0, Kp % 32 == 0.
// nx / ny are the FP64 squared norms of the rows of X / columns of Y.
// part: rect_partial_floats() floats of split-tile scratch.
// h partial slots of the A + W product: one per tile and fix-up block part
// (slots of tiles the fix-up never splits stay zero)
int64_t avail_hpart_slots(int64_t Mp, int64_t Np);
size_t rect_partial_floats();
// K up to which a product of three planes stays in one accumulator (see
// BlockGemmB3P::kFolds), and the A product's scratch for longer ones.
constexpr int64_t kFoldK = 1024;
// K up to which the products of the FP32 form are summed term by term in FP64
// from the whole operands.  What three planes leave out (mid * lo, lo * mid,
// lo * lo: 2^-22 of a term at most) is lost in a longer sum, but not in one or
// a few terms.  Error of a similarity in units of 2^-24 sum |x y| / sqrt(den),
// rms (largest of 3.6e6), on planes / on FP32 matrix cores: K = 1 0.98 (7.3) /
// 0.69 (2.4), K = 3 0.66 (5.7) / 0.62 (4.2), K = 5 0.53 (5.0) / 0.59 (4.5), K = 8
// 0.43 (4.2) / 0.56 (4.7), and below the cores' from there on.
constexpr int64_t kShortK = 8;
// How a product of FP32 operands sums over K: in one accumulator; folded where
// K is past kFoldK; that, but term by term where K is at most kShortK (of a
// batch's networks some may have a short one); all of it term by term.
enum KSum { kSumOnce = 0, kSumFolded = 1, kSumAny = 2, kSumShort = 3 };
size_t rect_fold_floats(int64_t Kp, int np);

// Out[i][j] = T(X, Y)_ij for i < M, j < N, over K (zeros from there to Kp).  yd (optional): Y is square with
// its diagonal held apart in this FP64 vector (and zero in Y).
hipError_t launch_tanimoto_store(const float* X, int64_t ldx, const float* Y, int64_t ldy,
                                 int64_t Mp, int64_t Np, int64_t Kp, int64_t M, int64_t N, int64_t K,
                                 const double* nx, const double* ny, float* Out, int64_t ldo,
                                 float* part, const int32_t* gate, hipStream_t s,
                                 const double* yd = nullptr);

// The diagonals of P and C are held apart in FP64 vectors dP, dC (the
// matrices hold zero there); the products add their terms in the epilogues.
// R = T(P, W) of the iteration (Eq. 3).
hipError_t launch_resp(const float* P, int64_t ldp, const double* dP, const float* W, int64_t ldw,
                       int64_t Nep, int64_t Nap, int64_t Ne, int64_t Na, const double* nP,
                       const double* nWc, float* R, int64_t ldr, float* part, const int32_t* gate,
                       hipStream_t s);

// A = T(W, C) fused with the W update of Eq. 2 and per-tile h partials (Eq. 7).
// (C is symmetric: its row n is the column n the product needs; it is split
// into planes as it is read.)  With three planes the old W is read from them
// (Wold unused) and Wnew may be R itself; fold holds rect_fold_floats().
hipError_t launch_avail_wupdate(const Planes& Wr, int np, const float* Wold, const float* C,
                                const double* dC, const float* R, float* Wnew, int64_t ld,
                                int64_t Nep, int64_t Nap, int64_t Ne, int64_t Na,
                                const double* nWrow, const double* nC, Rule rule, double* hpart,
                                float* part, float* fold, const int32_t* gate, hipStream_t s,
                                bool packed);

// C update (Eq. 5) on the upper tiles of T(W^T, W) with mirror writes and
// per-row partial sums for the sigma of Eq. 6 (and |C_.j|^2).  order holds
// the upper tiles (I | J << 16) in launch order, see launch_order.
hipError_t launch_coreg_update(const Planes& Wt, int np, int64_t Ne, int64_t Nep, float* C,
                               int64_t ldc, int64_t Nap, int64_t Na, const double* nWcol,
                               Rule rule, double2* cstat, double* csq, const uint32_t* order,
                               const int32_t* gate, hipStream_t s, bool packed);
int64_t coreg_slots(int64_t Nap);
// Upper tiles of the C product (Nap / 128 per side) and their launch order:
// group x group super-tiles (column of super-tiles by column, downwards, a
// super-tile's tiles column by column), so the tiles running together on one
// XCD share 2 * group operand strips in its L2.
int64_t coreg_tiles(int64_t Nap);
#ifndef PANDA_COREG_GROUP
#define PANDA_COREG_GROUP 6
#endif
constexpr int kCoregGroup = PANDA_COREG_GROUP;

// P update, split over K: partial products of W W^T on upper tiles.
hipError_t launch_coop_partial(const Planes& Wr, int np, int64_t Nep, int64_t Nap, int splits,
                               float* part, const int32_t* gate, hipStream_t s);
// K chunks of the partial products, for about `blocks` blocks in all (at
// T=700, G=18000 the split-BF16 products run best at 512: more partial sums
// cost the finalise more than they save; the FP32 form takes 1024, whose
// shorter sums also round less).
int coop_splits(int64_t Nep, int64_t Nap, int64_t blocks);

// R = T(P, W) (Eq. 3) on 128 x 128 tiles (next_r_tiles of them), alone or
// inside the C update's launch: that launch runs the C tiles and the R tiles
// of order_r, so the next iteration's R is ready when the C update ends (P, its diagonal dP and norms nP, and W's
// planes and column norms must be the new ones).  Both compute R the same
// way, bit for bit.  W, R: leading dimension ldw (R may be W itself: an entry
// of W is read by the thread that stores R there).
int64_t next_r_row_tiles(int64_t Nep);
int64_t next_r_tiles(int64_t Nep, int64_t Nap);
// An entry of order_r with this bit set is R tile (entry & 0xffff, (entry >>
// 16) & 0x7fff) (row tile of P, column tile of W); the others are C tiles (I,
// J) = (entry & 0xffff, entry >> 16).  Each XCD's share of the launch (the
// ranges xcd_tile maps block indices to) takes its share of the C tiles in
// their order, then its share of the R tiles, column tile by column tile (R
// tiles of one column share W's strip): they fill the end of its work.
constexpr uint32_t kNextRTile = 0x80000000u;
hipError_t launch_resp_tiles(const Planes& Pp, const Planes& Wt, int np, int64_t ldp,
                             const double* dP, int64_t Nap, int64_t Ne, int64_t Na,
                             const float* W, int64_t ldw, const double* nP, const double* nWc,
                             float* R, const int32_t* gate, hipStream_t s);
hipError_t launch_coreg_update_next_r(const Planes& Wt, int np, int64_t Nep,
                                      float* C, int64_t ldc, int64_t Nap, int64_t Na,
                                      const double* nWcol, Rule rule, double2* cstat, double* csq,
                                      const uint32_t* order_r, const int32_t* gate, hipStream_t s,
                                      bool packed, const Planes& Pp, const double* dP,
                                      const double* nP, const float* W, int64_t ldw, int64_t Ne,
                                      float* R);
// out[r][k] of the matrix that planes hold (join_planes; rows x cols, leading dimension ldo).
hipError_t launch_join_planes(const Planes& P, int64_t rows, int64_t cols, float* out, int64_t ldo,
                              hipStream_t s);
// The np planes of an n x n matrix with its diagonal left zero.
hipError_t launch_split_offdiag(const float* M, int64_t n, int64_t ld, Planes out, int np,
                                hipStream_t s);

// Packed C (see packed_tile).  load: the upper tiles of the n x n symmetric
// matrix src (row length n; its upper triangle is read, and mirrored inside
// diagonal tiles; the identity dval / oval where null), zero past n and on the
// diagonal, which goes to diag; norms[j] = sum_i C[i][j]^2 with the diagonal
// (j < Nap, FP64), through slots (nT x Nap doubles, nT = Nap / kPT).  unpack:
// the full n x n matrix into dst (leading dimension ldd).  sum_slots: out[j] =
// sum_k slots[k][j], j < Nap.
hipError_t launch_unpack_sym(const float* src, int64_t n, int64_t Nap, float* dst, int64_t ldd,
                             hipStream_t s);
hipError_t launch_sum_slots(const double* slots, int64_t Nap, int64_t nslots, double* out,
                            hipStream_t s);
hipError_t launch_load_packed(const float* src, int64_t n, int64_t Nap, float dval, float oval,
                              float* dst, double* diag, double* slots, double* norms,
                              hipStream_t s);

// Rest of the iteration: h, P finalisation, both diagonals, norm vectors.
hipError_t launch_finish_h(const double* hpart, int64_t n, int64_t count, DevState* st,
                           Rule rule, hipStream_t s);
hipError_t launch_coop_finalize(const float* part, int splits, int64_t Nep, const double* nWrow,
                                float* P, int64_t ldp, int64_t Ne, Rule rule, float* Tside,
                                Planes Pp, int np, const int32_t* gate, hipStream_t s);
// part: kDiagBoth, or kDiagP / kDiagC for P's rows (dP, nP: they need only
// the new P) or C's rows (dC, nC: they need the C update's row sums) alone.
constexpr int kDiagBoth = 0, kDiagP = 1, kDiagC = 2;
hipError_t launch_diagonals(const float* P, int64_t ldp, double* dP, int64_t Ne,
                            const float* Tside, double* nP, double* dC, int64_t ldc, int64_t Na,
                            const double2* cstat, const double* csq, int64_t nslots, double* nC,
                            Rule rule, const DevState* st, hipStream_t s, int part = kDiagBoth);
// The same with the diagonal rule new = keep * old + f * N * sigma * g given
// (closed form of several steps of Eq. 6).
hipError_t launch_diagonals_schedule(const float* P, int64_t ldp, double* dP, int64_t Ne,
                                     const float* Tside, double* nP, double* dC, int64_t ldc,
                                     int64_t Na, const double2* cstat, const double* csq,
                                     int64_t nslots, double* nC, Rule rule, double keep, double g,
                                     const DevState* st, hipStream_t s);
// The diagonal of an n x n matrix into / out of its FP64 vector (take also
// sets the matrix diagonal to zero).
hipError_t launch_take_diag(float* M, int64_t n, int64_t ld, double* d, hipStream_t s);
hipError_t launch_put_diag(float* M, int64_t n, int64_t ld, const double* d, hipStream_t s);
// t, the gates, and the current-W selector back to buffer 0.
hipError_t launch_state_set(DevState* st, int32_t t, int32_t active, int32_t run_pc,
                            hipStream_t s);
// Row and column squared norms of W (padded Nep x ldw, real Ne x Na) in one
// pass over it, plus its np bf16 planes (of W, Wr, with the lower bits where np
// is 3; of W^T, Wt).  scr holds w_norm_scratch_doubles().
size_t w_norm_scratch_doubles(int64_t Nep, int64_t Nap);
hipError_t launch_w_norms(const float* W, int64_t Ne, int64_t Na, int64_t ldw, int64_t Nep,
                          double* nr, double* nc, double* scr, Planes Wr, Planes Wt, int np,
                          const int32_t* gate, hipStream_t s);
// Z-score (Sec. II-A) on a strided matrix; scratch holds kZsScratch doubles:
// the moments (mean, std, non-finite flag) at kZsBlocks, the blocks' moments
// (3 doubles each) from kZsPart on.
constexpr int kZsBlocks = 1024;
constexpr int kZsPart = kZsBlocks + 8;
constexpr size_t kZsScratch = kZsPart + 3 * (size_t)kZsBlocks;
hipError_t launch_zscore_stats(const float* M, int64_t rows, int64_t cols, int64_t ld,
                               double* scratch, hipStream_t s, int ddof = 0);
// Per-row moments (rs, one per row) and, when cs is given, per-column
// moments (cs, one per column) as (mean, 1 / std); cpart: zs_col_chunks(rows)
// x cols double2 of scratch for the columns.  flags[0] / flags[1] are set for
// a NaN/Inf entry / a row or column of zero spread, and then the matrix is
// left alone by apply: per-row z-score, or (row z + column z) / sqrt 2 when
// cs is given.
constexpr int64_t kZsColChunks = 64;
int64_t zs_col_chunks(int64_t rows);
hipError_t launch_zscore_rc_stats(const float* M, int64_t rows, int64_t cols, int64_t ld, int ddof,
                                  double* flags, double2* rs, double2* cs, double2* cpart,
                                  hipStream_t s);
hipError_t launch_zscore_rc_apply(float* M, int64_t rows, int64_t cols, int64_t ld,
                                  const double2* rs, const double2* cs, const double* flags,
                                  hipStream_t s);
// Skipped on the device where the moments refuse the matrix.
hipError_t launch_zscore_apply(float* M, int64_t rows, int64_t cols, int64_t ld,
                               const double* scratch, hipStream_t s);
// Pearson correlation of the G rows of E (G x S, leading dimension lde):
// row statistics, then the centred rows scaled to unit norm, stored
// sample-major as Zt (Sp x Gp, zero-padded; Gp a multiple of 128, Sp of 16);
// then C = Z Z^T on the upper 128 x 128 tiles, mirrored, 1 on the diagonal.
hipError_t launch_pearson_z(const float* E, int64_t G, int64_t S, int64_t lde, double2* stat,
                            float* Zt, int64_t Gp, int64_t Sp, hipStream_t s);
hipError_t launch_corr(const float* Zt, int64_t Gp, int64_t Sp, int64_t S, int64_t G, float* C,
                       int64_t ldc, hipStream_t s);


}  // namespace panda

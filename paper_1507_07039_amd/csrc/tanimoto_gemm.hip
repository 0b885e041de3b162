// The similarity products of one PANDA iteration, in the two arithmetic
// forms the library offers, with the update rules fused into the epilogues:
//   R = T(P, W)                 Eq. 3, stored (also the stand-alone Tfunction)
//   A = T(W, C) + W update      Eq. 4 folded into Eq. 2, h partials of Eq. 7
//   C update                    Eq. 5 on upper tiles of T(W^T, W), mirrored,
//                               with the per-row sums for the sigma of Eq. 6
//   W W^T partial products      first half of the P update (Eq. 5), split-K
// The iteration's products run on bf16 planes of their operands
// (v_mfma_f32_32x32x16_bf16, FP32 accumulator): two planes and three products
// in the split-BF16 form, three exact planes and six products in the FP32
// form.  The stand-alone Tfunction and the correlations split their FP32
// operands into the three planes as they are loaded.  The diagonals of P and C
// (which grow like exp(2 alpha t), Eq. 6) are kept out of the operands and
// added back in FP64 in the epilogue (P_ii W_ij in R, W_ij C_jj in A).  Norms,
// denominators and h stay FP64 in both forms.
#include "epilogues.h"

namespace panda {
namespace {

using namespace gemm;

// R = T(P, W) (Eq. 3) on 128 x 128 tiles of the symmetric product's block,
// the same K = N_e as the C update: X = P's planes (rows past N_e clamped), Y
// = W^T's planes; rows past N_e are never stored.  The next iteration's R is
// computed inside the C update's launch, as soon as P, its diagonal and W's
// norms and planes are new: its tiles fill the launch's last wave of C tiles.
template <class G>
struct NextR {
  typename G::Ops ops;
  EpiStoreT epi;
};
// R's epilogue: W entries of runs of 16 rows of a column loaded together.
constexpr int kNextRRun = 16;

// The product of the tile, then the update in its epilogue (two blocks per
// CU, so one block's epilogue overlaps the other's products).  With NR the
// order also holds R tiles (kNextRTile).
// KS (three planes): K past kFoldK is folded through LDS behind the stages
// (kSumFolded), K of at most kShortK summed term by term (kSumShort).
template <class G, bool SIGT, int KS>
constexpr int coreg_kernel_bytes() {
  constexpr int main = G::MAIN_BYTES + (KS == kSumFolded ? G::BM * G::BN * 4 : 0);
  return main > coreg_smem_bytes<G, SIGT>() ? main : coreg_smem_bytes<G, SIGT>();
}
template <int KS, class G>
__device__ __forceinline__ void run_ks(G& g, const typename G::Ops& ops, int64_t m0, int64_t n0,
                                       int64_t kbeg, int64_t kend, char* smem, int64_t K = 0) {
  if constexpr (KS == kSumShort)
    g.run_short(ops, m0, n0, K, smem);
  else if constexpr (KS == kSumFolded)
    g.template run_long<G::kFoldQ>(ops, m0, n0, kbeg, kend, smem, nullptr);
  else
    g.run(ops, m0, n0, kbeg, kend, smem);
}

template <class G, bool SIGT, bool PK, bool NR, int KS>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2))) void k_coreg_update(
    typename G::Ops ops, int64_t Ne, int64_t Kp, float* __restrict__ C, int64_t ldc, int64_t Na,
    const double* __restrict__ ncol, double alpha, double2* __restrict__ cstat,
    double* __restrict__ csq, int64_t ldstat, const uint32_t* __restrict__ order,
    const int32_t* gate, NextR<G> nr) {
  if (gate && *gate == 0) return;
  __shared__ __align__(16) char smem[coreg_kernel_bytes<G, SIGT, KS>()];
  const uint32_t ij = order[xcd_tile(blockIdx.x, gridDim.x)];
  if constexpr (NR) {
    if (ij & kNextRTile) {
      const int64_t m0 = (int64_t)(ij & 0xffff) * kCB, n0 = (int64_t)((ij >> 16) & 0x7fff) * kCB;
      G g;
      run_ks<KS>(g, nr.ops, m0, n0, 0, Kp, smem, nr.epi.M);
      store_t_tile_xd<kNextRRun>(g, smem, nr.epi, m0, n0);
      return;
    }
  }
  const int64_t I = ij & 0xffff, J = ij >> 16;
  const int64_t m0 = I * kCB, n0 = J * kCB;
  const double nval = coreg_norm_load(ncol, I, J, Na);
  G g;
  run_ks<KS>(g, ops, m0, n0, 0, Kp, smem, Ne);
  coreg_epilogue<SIGT, PK>(g, smem, I, J, C, ldc, Na, nval, alpha, cstat, csq, ldstat);
}

// R alone on the same tiles (same arithmetic, so R is the same bit for bit
// whichever launch computed it): block b is tile (b % nRT, b / nRT).
template <class G, int KS>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2))) void k_resp_tiles(
    NextR<G> nr, int64_t Kp, int64_t nRT, const int32_t* gate) {
  if (gate && *gate == 0) return;
  __shared__ __align__(16) char smem[G::MAIN_BYTES + (KS == kSumFolded ? G::BM * G::BN * 4 : 0)];
  const int64_t b = xcd_tile(blockIdx.x, gridDim.x);
  const int64_t m0 = (b % nRT) * kCB, n0 = (b / nRT) * kCB;
  G g;
  run_ks<KS>(g, nr.ops, m0, n0, 0, Kp, smem, nr.epi.M);
  store_t_tile_xd<kNextRRun>(g, smem, nr.epi, m0, n0);
}

// Pearson correlations: one upper 128 x 128 tile of Z Z^T per block, both
// operands read from Z^T (samples x genes), stored at the tile and mirrored.
template <class G>
__global__ __launch_bounds__(G::NT) __attribute__((amdgpu_waves_per_eu(G::WAVES_PER_EU)))
void k_corr_sym(typename G::Ops ops, int64_t Kp, float* __restrict__ C, int64_t ldc, int64_t n) {
  __shared__ __align__(16) char smem[corr_smem_bytes<G>()];
  int64_t I, J;
  tri_tile(xcd_tile(blockIdx.x, gridDim.x), I, J);
  G g;
  g.run(ops, I * kCB, J * kCB, 0, Kp, smem);
  corr_sym_epilogue(g, smem, I, J, C, ldc, n);
}

// ------------------------------------------------------------------------
// P update, first half: each block writes the partial product of one upper
// tile over one K chunk.

template <class G, bool LK>
__global__ __launch_bounds__(kThreads) void k_coop_partial(typename G::Ops ops, int64_t Nep,
                                                           int64_t nU, int64_t chunk, int64_t Nap,
                                                           float* __restrict__ part,
                                                           const int32_t* gate) {
  if (gate && *gate == 0) return;
  static_assert(G::BM == kPB && G::BN == kPB, "square tiles");
  __shared__ __align__(16) char smem[G::MAIN_BYTES + (LK ? G::BM * G::BN * 4 : 0)];
  const int64_t idx = xcd_tile(blockIdx.x, gridDim.x);
  const int64_t u = idx % nU, s = idx / nU;
  int64_t I, J;
  tri_tile(u, I, J);
  const int64_t m0 = I * kPB, n0 = J * kPB;
  int64_t kb = s * chunk, ke = kb + chunk;
  if (kb > Nap) kb = Nap;
  if (ke > Nap) ke = Nap;
  G g;
  run_ks<LK ? kSumFolded : kSumOnce>(g, ops, m0, n0, kb, ke, smem);
  float* ps = part + s * Nep * Nep;
  g.for_each([&](int r, int c, float v) { ps[(m0 + r) * Nep + n0 + c] = v; });
}

}  // namespace

// ---------------------------------------------------------------- launch --

template <int NP>
constexpr bool kOneAvailGrid = Tiles<NP>::Rect::BM == Tiles<2>::Rect::BM &&
                               Tiles<NP>::Rect::BN == Tiles<2>::Rect::BN &&
                               Tiles<NP>::RectP::BM == Tiles<2>::Rect::BM &&
                               Tiles<NP>::RectP::BN == Tiles<2>::Rect::BN;
static_assert(kOneAvailGrid<2> && kOneAvailGrid<3>, "one slot layout for both forms and layouts");
int64_t avail_hpart_slots(int64_t Mp, int64_t Np) {
  using G = Tiles<2>::Rect;
  return (Mp + G::BM - 1) / G::BM * (Np / G::BN) * kFixParts<G>;
}
size_t rect_fold_floats(int64_t Kp, int np) {
  using G = Tiles<3>::Rect;
  return np == 3 && Kp > kFoldK ? (size_t)kFoldBlocks * G::BM * G::BN : 0;
}
size_t rect_partial_floats() {
  return (size_t)2 * (size_t)kMaxStreamKBlocks * (size_t)kPartTile;
}

static hipError_t rect_f32(const OpsF32& ops, int64_t Mp, int64_t Np, int64_t Kp,
                           const EpiStoreT& epi, float* part, const int32_t* gate, hipStream_t s) {
  auto run = [&](auto g) {
    using G = decltype(g);
    return launch_rect<G>(ops, round_up(Mp, G::BM), Np, Kp, epi, part, gate, s);
  };
  if (ops.K <= kShortK) return run(RectF32<kSumShort>{});
  return Kp > kFoldK ? run(RectF32<kSumFolded>{}) : run(RectF32<kSumOnce>{});
}

hipError_t launch_tanimoto_store(const float* X, int64_t ldx, const float* Y, int64_t ldy,
                                 int64_t Mp, int64_t Np, int64_t Kp, int64_t M, int64_t N, int64_t K,
                                 const double* nx, const double* ny, float* Out, int64_t ldo,
                                 float* part, const int32_t* gate, hipStream_t s,
                                 const double* yd) {
  EpiStoreT epi{Out, ldo, M, N, nx, ny};
  if (yd) {  // Y's diagonal held apart: its term X_ij Y_jj (X square with Y)
    epi.yd = yd;
    epi.xv = X;
    epi.ldxv = ldx;
  }
  return rect_f32(OpsF32{X, ldx, Y, ldy, M, K}, Mp, Np, Kp, epi, part, gate, s);
}

hipError_t launch_corr(const float* Zt, int64_t Gp, int64_t Sp, int64_t S, int64_t G, float* C,
                       int64_t ldc, hipStream_t s) {
  // X = Z stored sample-major (Z^T), as W^T is read from W in the C update.
  const int64_t nT = Gp / kCB;
  auto run = [&](auto g) {
    using Gm = decltype(g);
    if (Gp % kCB || Sp % Gm::BK || G > Gp) return hipErrorInvalidValue;
    k_corr_sym<Gm><<<dim3((unsigned)(nT * (nT + 1) / 2)), dim3(Gm::NT), 0, s>>>(
        OpsF32{Zt, Gp, Zt, Gp, Gp, S}, Sp, C, ldc, G);
    return hipGetLastError();
  };
  if (S <= kShortK) return run(SymF32<kSumShort>{});
  return Sp > kFoldK ? run(SymF32<kSumFolded>{}) : run(SymF32<kSumOnce>{});
}

hipError_t launch_resp(const float* P, int64_t ldp, const double* dP, const float* W, int64_t ldw,
                       int64_t Nep, int64_t Nap, int64_t Ne, int64_t Na, const double* nP,
                       const double* nWc, float* R, int64_t ldr, float* part, const int32_t* gate,
                       hipStream_t s) {
  EpiStoreT epi{R, ldr, Ne, Na, nP, nWc, dP, W, ldw};
  return rect_f32(OpsF32{P, ldp, W, ldw, Ne, Ne}, Nep, Nap, Nep, epi, part, gate, s);
}

template <int NP, class Epi>
static hipError_t avail_np(const Planes& Wr, const float* C, int64_t ld, int64_t Nep, int64_t Nap,
                           const Epi& epi, float* part, float* fold, const int32_t* gate,
                           hipStream_t s, bool packed) {
  using T = Tiles<NP>;
  const int64_t Mp = round_up(Nep, T::Rect::BM);
  if (packed)
    return launch_rect<typename T::RectP>(OpsB3FP{Wr, C, Nep}, Mp, Nap, Nap, epi, part, gate, s, fold);
  return launch_rect<typename T::Rect>(OpsB3F{Wr, C, ld, Nep}, Mp, Nap, Nap, epi, part, gate, s, fold);
}

hipError_t launch_avail_wupdate(const Planes& Wr, int np, const float* Wold, const float* C,
                                const double* dC, const float* R, float* Wnew, int64_t ld,
                                int64_t Nep, int64_t Nap, int64_t Ne, int64_t Na,
                                const double* nWrow, const double* nC, Rule rule, double* hpart,
                                float* part, float* fold, const int32_t* gate, hipStream_t s,
                                bool packed) {
  if (np == 2) {
    const EpiWUpdate epi{Wold, R,  Wnew,       ld,              Ne,    Na, nWrow,
                         nC,   dC, rule.alpha, rule.h_undamped, hpart, 0.0};
    return avail_np<2>(Wr, C, ld, Nep, Nap, epi, part, nullptr, gate, s, packed);
  }
  const EpiWUpdateT<true> epi{nullptr, R,  Wnew,       ld,              Ne,    Na,  nWrow,
                              nC,      dC, rule.alpha, rule.h_undamped, hpart, 0.0, Wr};
  return avail_np<3>(Wr, C, ld, Nep, Nap, epi, part, fold, gate, s, packed);
}

int64_t coreg_slots(int64_t Nap) { return Nap / kCB; }
int64_t coreg_tiles(int64_t Nap) { return (Nap / kCB) * (Nap / kCB + 1) / 2; }

template <class G, bool PK, bool NR>
static hipError_t coreg_launch_pk(const typename G::Ops& ops, int64_t Ne, int64_t Nep, float* C, int64_t ldc,
                                  int64_t Nap, int64_t Na, const double* nWcol, Rule rule,
                                  double2* cstat, double* csq, const uint32_t* order,
                                  const int32_t* gate, hipStream_t s, const NextR<G>& nr,
                                  int64_t extra) {
  const dim3 nb((unsigned)(coreg_tiles(Nap) + extra));
  auto go = [&](auto* fn) {
    fn<<<nb, dim3(kThreads), 0, s>>>(ops, Ne, Nep, C, ldc, Na, nWcol, rule.alpha, cstat, csq, Nap,
                                     order, gate, nr);
  };
  auto with = [&](auto ks) {
    constexpr int KS = decltype(ks)::value;
    if (rule.sigma_from_T)
      go(k_coreg_update<G, true, PK, NR, KS>);
    else
      go(k_coreg_update<G, false, PK, NR, KS>);
    return hipGetLastError();
  };
  if constexpr (folds_k<G>::value) {
    if (Ne <= kShortK) return with(std::integral_constant<int, kSumShort>{});
    if (Nep > kFoldK) return with(std::integral_constant<int, kSumFolded>{});
  }
  return with(std::integral_constant<int, kSumOnce>{});
}

template <class G, bool NR = false>
static hipError_t coreg_launch(const typename G::Ops& ops, int64_t Ne, int64_t Nep, float* C, int64_t ldc,
                               int64_t Nap, int64_t Na, const double* nWcol, Rule rule,
                               double2* cstat, double* csq, const uint32_t* order,
                               const int32_t* gate, hipStream_t s, bool packed,
                               const NextR<G>& nr = NextR<G>{}, int64_t extra = 0) {
  return packed ? coreg_launch_pk<G, true, NR>(ops, Ne, Nep, C, ldc, Nap, Na, nWcol, rule, cstat,
                                               csq, order, gate, s, nr, extra)
                : coreg_launch_pk<G, false, NR>(ops, Ne, Nep, C, ldc, Nap, Na, nWcol, rule, cstat,
                                                csq, order, gate, s, nr, extra);
}

hipError_t launch_coreg_update(const Planes& Wt, int np, int64_t Ne, int64_t Nep, float* C,
                               int64_t ldc, int64_t Nap, int64_t Na, const double* nWcol,
                               Rule rule, double2* cstat, double* csq, const uint32_t* order,
                               const int32_t* gate, hipStream_t s, bool packed) {
  // X = Yt = W^T stored gene-major: row m of W^T is column m of W.  Only the
  // FP32 C is written; the next A product splits it while staging.
  const OpsB3 ops{Wt, Wt};
  return np == 2 ? coreg_launch<Tiles<2>::Sym>(ops, Ne, Nep, C, ldc, Nap, Na, nWcol, rule, cstat, csq,
                                               order, gate, s, packed)
                 : coreg_launch<Tiles<3>::Sym>(ops, Ne, Nep, C, ldc, Nap, Na, nWcol, rule, cstat, csq,
                                               order, gate, s, packed);
}

int64_t next_r_row_tiles(int64_t Nep) { return (Nep + kCB - 1) / kCB; }
int64_t next_r_tiles(int64_t Nep, int64_t Nap) { return next_r_row_tiles(Nep) * (Nap / kCB); }

template <class G>
static NextR<G> next_r_args(const Planes& Pp, const double* dP, const double* nP,
                            const Planes& Wt, const float* W, int64_t ldw, int64_t Ne,
                            int64_t Na, const double* nWc, float* R) {
  NextR<G> nr;
  nr.ops = OpsB3{Pp, Wt, Pp.rows};  // P has N_e (padded) rows
  nr.epi = EpiStoreT{R, ldw, Ne, Na, nP, nWc, dP, W, ldw};
  return nr;
}

template <class G, int KS>
static hipError_t resp_tiles_launch(const NextR<G>& nr, int64_t ldp, int64_t Nap,
                                    const int32_t* gate, hipStream_t s) {
  k_resp_tiles<G, KS><<<dim3((unsigned)next_r_tiles(ldp, Nap)), dim3(kThreads), 0, s>>>(
      nr, ldp, next_r_row_tiles(ldp), gate);
  return hipGetLastError();
}

hipError_t launch_resp_tiles(const Planes& Pp, const Planes& Wt, int np, int64_t ldp,
                             const double* dP, int64_t Nap, int64_t Ne, int64_t Na,
                             const float* W, int64_t ldw, const double* nP, const double* nWc,
                             float* R, const int32_t* gate, hipStream_t s) {
  if (ldp % SymB3::BK || Nap % kCB) return hipErrorInvalidValue;
  using G2 = Tiles<2>::Sym;
  using G3 = Tiles<3>::Sym;
  if (np == 2)
    return resp_tiles_launch<G2, kSumOnce>(next_r_args<G2>(Pp, dP, nP, Wt, W, ldw, Ne, Na, nWc, R),
                                        ldp, Nap, gate, s);
  const NextR<G3> nr = next_r_args<G3>(Pp, dP, nP, Wt, W, ldw, Ne, Na, nWc, R);
  if (Ne <= kShortK) return resp_tiles_launch<G3, kSumShort>(nr, ldp, Nap, gate, s);
  return ldp > kFoldK ? resp_tiles_launch<G3, kSumFolded>(nr, ldp, Nap, gate, s)
                      : resp_tiles_launch<G3, kSumOnce>(nr, ldp, Nap, gate, s);
}

hipError_t launch_coreg_update_next_r(const Planes& Wt, int np, int64_t Nep,
                                      float* C, int64_t ldc, int64_t Nap, int64_t Na,
                                      const double* nWcol, Rule rule, double2* cstat, double* csq,
                                      const uint32_t* order_r, const int32_t* gate, hipStream_t s,
                                      bool packed, const Planes& Pp, const double* dP,
                                      const double* nP, const float* W, int64_t ldw, int64_t Ne,
                                      float* R) {
  if (Nep % SymB3::BK || Nap % kCB) return hipErrorInvalidValue;
  using G2 = Tiles<2>::Sym;
  using G3 = Tiles<3>::Sym;
  const OpsB3 ops{Wt, Wt};
  const int64_t extra = next_r_tiles(Nep, Nap);
  if (np == 2)
    return coreg_launch<G2, true>(ops, Ne, Nep, C, ldc, Nap, Na, nWcol, rule, cstat, csq, order_r, gate,
                                  s, packed,
                                  next_r_args<G2>(Pp, dP, nP, Wt, W, ldw, Ne, Na, nWcol, R), extra);
  return coreg_launch<G3, true>(ops, Ne, Nep, C, ldc, Nap, Na, nWcol, rule, cstat, csq, order_r, gate, s,
                                packed, next_r_args<G3>(Pp, dP, nP, Wt, W, ldw, Ne, Na, nWcol, R),
                                extra);
}

int coop_splits(int64_t Nep, int64_t Nap, int64_t blocks) {
  const int64_t nT = Nep / kPB, nU = nT * (nT + 1) / 2;
  int64_t s = (blocks + nU - 1) / nU;
  const int64_t maxs = Nap / (4 * CoopB3::BK);  // at least 4 K-steps per block
  if (s > maxs) s = maxs;
  if (s < 1) s = 1;
  return (int)s;
}

static int64_t coop_chunk(int64_t Nap, int splits) {
  return round_up((Nap + splits - 1) / splits, CoopB3::BK);
}

hipError_t launch_coop_partial(const Planes& Wr, int np, int64_t Nep, int64_t Nap, int splits,
                               float* part, const int32_t* gate, hipStream_t s) {
  const int64_t nT = Nep / kPB, nU = nT * (nT + 1) / 2, chunk = coop_chunk(Nap, splits);
  auto* fn = np == 2          ? k_coop_partial<Tiles<2>::Coop, false>
             : chunk > kFoldK ? k_coop_partial<Tiles<3>::Coop, true>
                              : k_coop_partial<Tiles<3>::Coop, false>;
  fn<<<dim3((unsigned)(nU * splits)), dim3(kThreads), 0, s>>>(OpsB3{Wr, Wr}, Nep, nU, chunk, Nap,
                                                              part, gate);
  return hipGetLastError();
}

}  // namespace panda

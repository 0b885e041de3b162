// Host side of libpanda.so: argument checks, workspace layout, the
// iteration sequence of Sec. II-B and the C ABI declared in include/panda.h.
#include <math.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <mutex>
#include <new>
#include <vector>

#include "host_internal.h"

using namespace panda;

namespace panda {

thread_local char g_err[512] = "";

panda_status fail(panda_status st, const char* fmt, const char* what) {
  snprintf(g_err, sizeof g_err, fmt, what);
  return st;
}

panda_status hip_fail(hipError_t e, const char* where) {
  snprintf(g_err, sizeof g_err, "%s: %s", where, hipGetErrorString(e));
  return PANDA_ERR_HIP;
}

}  // namespace panda

namespace panda {

Rule rule_of(const panda_options& o) {
  Rule r;
  r.alpha = o.alpha;
  r.tol = o.tol;
  r.diag_alpha = o.diag_alpha;
  r.sigma_from_T = o.sigma_from_T;
  r.n_own = o.n_own;
  r.h_undamped = o.h_undamped;
  r.update_last = o.update_last;
  r.sigma_ddof = o.sigma_ddof;
  return r;
}

panda_status check_options(const panda_options& o) {
  if (!(o.alpha > 0.0) || !(o.alpha <= 1.0)) return fail(PANDA_ERR_ARG, "alpha must be in (0, 1]%s");
  if (!(o.tol >= 0.0) || !isfinite(o.tol)) return fail(PANDA_ERR_ARG, "tol must be finite and >= 0%s");
  if (o.max_iter < 1) return fail(PANDA_ERR_ARG, "max_iter must be >= 1%s");
  if (o.poll_every < 1) return fail(PANDA_ERR_ARG, "poll_every must be >= 1%s");
  if (o.precision != PANDA_PREC_FP32 && o.precision != PANDA_PREC_BF16X3)
    return fail(PANDA_ERR_ARG, "unknown precision%s");
  if (o.sigma_ddof != 0 && o.sigma_ddof != 1) return fail(PANDA_ERR_ARG, "sigma_ddof must be 0 or 1%s");
  if (o.packed_c != 0 && o.packed_c != 1) return fail(PANDA_ERR_ARG, "packed_c must be 0 or 1%s");
  if (o.zscore_mode < PANDA_ZSCORE_GLOBAL || o.zscore_mode > PANDA_ZSCORE_ROWCOL)
    return fail(PANDA_ERR_ARG, "unknown zscore_mode%s");
  return PANDA_OK;
}

// Dimensions that keep every index and the tiled grids within range.
bool dims_ok(int64_t Ne, int64_t Na) {
  return Ne >= 1 && Na >= 1 && Ne <= (1 << 16) && Na <= (1 << 18);
}

}  // namespace panda

namespace panda {

LayoutSpec single_spec(int64_t Ne, int64_t Na, bool packed_c, int32_t precision) {
  const int64_t Nep = round_up(Ne, kPadE), Nap = round_up(Na, kPadA);
  // K chunks of W W^T: the FP32 form's are kept short enough for one
  // accumulator where that at most doubles their number
  const bool fp32 = precision != PANDA_PREC_BF16X3;
  int64_t splits = coop_splits(Nep, Nap, fp32 ? 1024 : 512);
  const int64_t whole = (Nap + kFoldK - 1) / kFoldK;
  if (fp32 && whole <= 2 * splits) splits = std::max(splits, whole);
  return LayoutSpec{false, avail_hpart_slots(Nep, Nap), splits, packed_c};
}

// Workspace layout shared by the size queries and the contexts.
size_t ctx_layout(int64_t Ne, int64_t Na, int32_t precision, const LayoutSpec& spec, panda_ctx* c,
                  char* base) {
  const int64_t Nep = round_up(Ne, kPadE), Nap = round_up(Na, kPadA);
  Carver cv{base};
  const size_t nw = (size_t)Nep * (size_t)Nap;
  // bf16 planes of the operands: two, or three for the FP32 form
  const bool sm = spec.batched ? small_net(Ne, Na) : small_run(Ne, Na, precision);
  const int np = sm && !spec.batched ? 0 : precision == PANDA_PREC_BF16X3 ? 2 : spec.batched ? 0 : 3;
  const bool in_place = np == 3;  // one buffer for W and R
  float* w0 = cv.take<float>(nw);
  float* w1 = in_place ? w0 : cv.take<float>(nw);
  float* r = in_place ? w0 : cv.take<float>(nw);
  float* p = cv.take<float>((size_t)Nep * Nep);
  float* cc = cv.take<float>(spec.packed_c ? (size_t)packed_floats(Nap) : (size_t)Nap * Nap);
  float* ts = cv.take<float>((size_t)Nep * Nep);
  const int splits = (int)spec.ppart_splits;
  // Of the FP32 form's buffers two share memory with others: the W W^T partials
  // (from the partial products to the P finalisation), then the C update's sums
  // of squares (to its diagonal; or a load's), then the A product's folding
  // scratch; the A product's split tiles, then the planes of W^T, which are
  // written after it and last read by the C update before the next one.
  const int64_t nslots = sm ? std::max(coreg_slots(Nap), small_tiles(Na)) : coreg_slots(Nap);
  const size_t npp = (size_t)splits * Nep * Nep, nfold = rect_fold_floats(Nap, np);
  const size_t ncsq = (size_t)nslots * Nap;
  float* pp = cv.take<float>(in_place ? std::max({npp, nfold, 2 * ncsq}) : npp);
  const size_t nsk = spec.batched ? 0 : rect_partial_floats();
  float* sk = cv.take<float>(in_place ? std::max(nsk, (3 * nw + 1) / 2) : nsk);
  if (spec.batched) sk = nullptr;
  double* dp = cv.take<double>((size_t)Nep * (sm ? 2 : 1));
  double* dc = cv.take<double>((size_t)Nap);
  double* np_ = cv.take<double>((size_t)Nep);
  double* nc = cv.take<double>((size_t)Nap);
  double* nwr = cv.take<double>((size_t)Nep);
  double* nwc = cv.take<double>((size_t)Nap);
  double* scr = cv.take<double>(w_norm_scratch_doubles(Nep, Nap));
  const int64_t nh = sm ? std::max(spec.hpart_tiles, small_h_slots(Ne, Na)) : spec.hpart_tiles;
  double* hp = cv.take<double>((size_t)nh);
  double2* cs = cv.take<double2>(ncsq);
  double* cq = in_place ? reinterpret_cast<double*>(pp) : cv.take<double>(ncsq);
  uint32_t* co = cv.take<uint32_t>((size_t)coreg_tiles(Nap));
  DevState* st = cv.take<DevState>(2);  // the second: the small kernels' next state
  uint32_t* cor = !spec.batched
                      ? cv.take<uint32_t>((size_t)(coreg_tiles(Nap) + next_r_tiles(Nep, Nap)))
                      : nullptr;
  Planes wr{nullptr, (int64_t)nw, Nep}, wt{nullptr, (int64_t)nw, Nap}, pl{nullptr, Nep * Nep, Nep};
  if (np) {
    wr.p = cv.take<bf16_t>((in_place ? kHeldPlanes : np) * nw);  // W
    wt.p = in_place ? reinterpret_cast<bf16_t*>(sk) : cv.take<bf16_t>(np * nw);  // W^T
    pl.p = cv.take<bf16_t>(np * (size_t)Nep * Nep);  // P, zero diagonal
  }
  if (c) {
    c->Nep = Nep;
    c->Nap = Nap;
    c->W[0] = w0;
    c->W[1] = w1;
    c->R = r;
    c->P = p;
    c->C = cc;
    c->Tside = ts;
    c->ppart = pp;
    c->skpart = sk;
    c->fold = nfold ? pp : nullptr;
    c->dP = dp;
    c->dC = dc;
    c->nP = np_;
    c->nC = nc;
    c->nWr = nwr;
    c->nWc = nwc;
    c->colscr = scr;
    c->splits = splits;
    c->hpart = hp;
    c->nh = spec.hpart_tiles;  // h partials that the tiled A + W products may add up
    c->cstat = cs;
    c->csq = cq;
    c->crows = sm ? kSmallTile : kPT;
    c->corder = co;
    c->corder_r = cor;
    c->small = sm && !spec.batched;
    c->w_in_place = in_place;
    c->r_next = false;
    c->st = st;
    c->np = np;
    c->packed = spec.packed_c;
    c->Wr = wr;
    c->Wt = wt;
    c->Pp = pl;
  }
  return cv.off;
}

panda_status ctx_setup(panda_ctx* c, int64_t Ne, int64_t Na, const panda_options& o,
                       const LayoutSpec& spec, char* base, hipStream_t stream) {
  c->Ne = Ne;
  c->Na = Na;
  c->opt = o;
  c->rule = rule_of(o);
  c->stream = stream;
  ctx_layout(Ne, Na, o.precision, spec, c, base);
  HIP_TRY(hipHostMalloc(reinterpret_cast<void**>(&c->host), sizeof(DevState),
                        hipHostMallocDefault));
  c->loaded = false;
  return PANDA_OK;
}

panda_status ctx_fill_order(panda_ctx* c) {
  HIP_TRY(launch_order(c->Nep, c->Nap, kCoregGroup, c->corder, c->corder_r, c->stream));
  return PANDA_OK;
}

void ctx_free(panda_ctx* c) {
  if (c->snap) {
    // an iteration queued behind the converged one may still write it
    (void)hipStreamSynchronize(c->stream);
    (void)hipHostFree(c->snap);
    for (hipEvent_t& e : c->snap_ev) (void)hipEventDestroy(e);
  }
  c->snap = nullptr;
  if (c->host) (void)hipHostFree(c->host);
  c->host = nullptr;
  if (c->ev[0][0])
    for (int i = 0; i < kMaxPending; ++i)
      for (int p = 0; p <= PANDA_NPHASE; ++p) (void)hipEventDestroy(c->ev[i][p]);
  c->ev[0][0] = nullptr;
}

// The z-scored identity of order n (Sec. II-A: an absent prior is the
// identity, z-scored like any network) in closed form: every row, every
// column and the whole matrix hold one 1 among zeros, so the result has one
// value on the diagonal (dv) and one off it (ov).  Mean m = 1/n; sum of
// squared deviations over n^2 entries n (1 - m)^2 + (n^2 - n) m^2 = n - 1,
// over a row (1 - m)^2 + (n - 1) m^2; the row + column scope gives
// (Zr + Zc) / sqrt 2 = sqrt 2 Zr.  False when the std is 0 (n = 1).
bool identity_zscore(int64_t n, int32_t mode, int32_t ddof, double* dv, double* ov) {
  const double m = 1.0 / (double)n, nn = (double)n;
  const double cnt = mode == PANDA_ZSCORE_GLOBAL ? nn * nn : nn;
  const double ss = mode == PANDA_ZSCORE_GLOBAL ? nn * (1.0 - m) * (1.0 - m) + (nn * nn - nn) * m * m
                                                : (1.0 - m) * (1.0 - m) + (nn - 1.0) * m * m;
  if (cnt - ddof < 1.0) return false;
  const double sd = sqrt(ss / (cnt - ddof));
  if (!(sd > 0.0)) return false;
  const double f = mode == PANDA_ZSCORE_ROWCOL ? sqrt(2.0) : 1.0;
  *dv = f * (1.0 - m) / sd;
  *ov = f * (-m) / sd;
  return true;
}

size_t zscore_scratch_doubles(int64_t rows, int64_t cols, int32_t mode) {
  if (mode == PANDA_ZSCORE_GLOBAL) return kZsScratch;
  const size_t rc = 8 + 2 * (size_t)rows +
                    (mode == PANDA_ZSCORE_ROWCOL
                         ? 2 * (size_t)cols * (1 + (size_t)zs_col_chunks(rows)) : 0);
  return rc > kZsScratch ? rc : kZsScratch;
}

panda_status zscore(float* M, int64_t rows, int64_t cols, int64_t ld, int32_t mode, int32_t ddof,
                    double* scratch, hipStream_t s) {
  // apply skips a refused matrix on the device, so it is enqueued before the
  // verdict is read back and the GPU does not wait for the host
  if (mode == PANDA_ZSCORE_GLOBAL) {
    HIP_TRY(launch_zscore_stats(M, rows, cols, ld, scratch, s, ddof));
    HIP_TRY(launch_zscore_apply(M, rows, cols, ld, scratch, s));
    double tail[3];
    HIP_TRY(hipMemcpyAsync(tail, scratch + kZsBlocks, sizeof tail, hipMemcpyDeviceToHost, s));
    HIP_TRY(hipStreamSynchronize(s));
    if (tail[2] != 0.0) return fail(PANDA_ERR_NONFINITE, "network contains NaN or Inf%s");
    if (!(tail[1] > 0.0)) return fail(PANDA_ERR_DEGENERATE, "network is constant (std = 0)%s");
    return PANDA_OK;
  }
  double* flags = scratch;
  double2* rs = reinterpret_cast<double2*>(scratch + 8);
  double2* cs = mode == PANDA_ZSCORE_ROWCOL ? rs + rows : nullptr;
  HIP_TRY(launch_zscore_rc_stats(M, rows, cols, ld, ddof, flags, rs, cs, cs ? cs + cols : nullptr,
                                 s));
  HIP_TRY(launch_zscore_rc_apply(M, rows, cols, ld, rs, cs, flags, s));
  double f[2];
  HIP_TRY(hipMemcpyAsync(f, flags, sizeof f, hipMemcpyDeviceToHost, s));
  HIP_TRY(hipStreamSynchronize(s));
  if (f[0] != 0.0) return fail(PANDA_ERR_NONFINITE, "network contains NaN or Inf%s");
  if (f[1] != 0.0)
    return fail(PANDA_ERR_DEGENERATE, "a row or column of the network is constant (std = 0)%s");
  return PANDA_OK;
}

SmallRule small_rule_of(const panda_ctx* c) {
  return SmallRule{c->rule, c->rule.sigma_from_T, c->packed ? 1 : 0};
}

BInst inst_of(const panda_ctx* c) {
  BInst d{};
  d.Ne = c->Ne;
  d.Na = c->Na;
  d.Nep = c->Nep;
  d.Nap = c->Nap;
  d.W[0] = c->W[0];
  d.W[1] = c->W[1];
  d.R = c->R;
  d.P = c->P;
  d.C = c->C;
  d.Tside = c->Tside;
  d.ppart = c->ppart;
  d.dP = c->dP;
  d.dC = c->dC;
  d.nP = c->nP;
  d.nC = c->nC;
  d.nWr = c->nWr;
  d.nWc = c->nWc;
  d.colscr = c->colscr;
  d.hpart = c->hpart;
  d.cstat = c->cstat;
  d.csq = c->csq;
  d.corder = c->corder;
  d.st = c->st;
  d.Wr = c->Wr;
  d.Wt = c->Wt;
  d.Pp = c->Pp;
  d.np = c->np;
  return d;
}

BInst small_inst_of(const panda_ctx* c, int64_t k) {
  BInst d = inst_of(c);
  const int64_t at = k >= 0 ? k : -k - 1;
  d.W[0] = c->W[at & 1];
  d.W[1] = c->W[(k >= 0 ? at + 1 : at) & 1];
  return d;
}

}  // namespace panda

namespace {

// Phase boundary marker: records event `p` of the current pending
// iteration when timing is on.
panda_status mark(panda_ctx* c, int p) {
  if (!c->timing) return PANDA_OK;
  HIP_TRY(hipEventRecord(c->ev[c->npend][p], c->stream));
  return PANDA_OK;
}

// Sum the elapsed times of the pending timed iterations (stream synced).
panda_status collect_times(panda_ctx* c) {
  for (int i = 0; i < c->npend; ++i)
    for (int p = 0; p < PANDA_NPHASE; ++p) {
      float ms = 0.0f;
      HIP_TRY(hipEventElapsedTime(&ms, c->ev[i][p], c->ev[i][p + 1]));
      c->tot_ms[p] += ms;
      c->cnt[p] += 1;
    }
  c->npend = 0;
  return PANDA_OK;
}

// Read the device state back (synchronises the stream).
panda_status read_state(panda_ctx* c) {
  HIP_TRY(hipMemcpyAsync(c->host, c->st, sizeof(DevState), hipMemcpyDeviceToHost, c->stream));
  HIP_TRY(hipStreamSynchronize(c->stream));
  c->executed = c->host->t - c->t0;
  c->fresh = true;
  return collect_times(c);
}

// Enqueue one iteration: R, A + W update, h, P update, C update, diagonals.
// Iteration k (counted from the load) reads W[k % 2] and writes W[(k+1) % 2];
// iterations past convergence are skipped on the device, so the executed
// ones are always a prefix of the enqueued ones.
panda_status enqueue_iteration(panda_ctx* c) {
  c->fresh = false;
  if (c->timing && c->npend == kMaxPending) PANDA_TRY(read_state(c));
  const int64_t k = c->enqueued;
  float* Wold = c->W[k & 1];
  float* Wnew = c->W[(k + 1) & 1];
  hipStream_t s = c->stream;
  const int32_t* active = &c->st->active;
  const int32_t* run_pc = &c->st->run_pc;
  PANDA_TRY(mark(c, PANDA_PHASE_R));
  if (c->small) {  // three launches: the P phases are empty, R belongs to the last
    const BInst d = small_inst_of(c, k);
    const SmallDims mx{c->Ne, c->Na};
    const SmallRule rule = small_rule_of(c);
    PANDA_TRY(mark(c, PANDA_PHASE_AW));
    HIP_TRY(launch_small_avail(nullptr, d, 1, mx, rule, s));
    for (int p : {PANDA_PHASE_H, PANDA_PHASE_PPART, PANDA_PHASE_PFIN, PANDA_PHASE_C})
      PANDA_TRY(mark(c, p));
    HIP_TRY(launch_small_update(nullptr, d, 1, mx, rule, kSmallStep, s));
    PANDA_TRY(mark(c, PANDA_PHASE_DIAG));
    HIP_TRY(launch_small_finish(nullptr, d, 1, mx, rule, kSmallStep, s, c->snap_to));
    PANDA_TRY(mark(c, PANDA_NPHASE));
    if (c->timing) c->npend += 1;
    c->enqueued += 1;
    return PANDA_OK;
  }
  // Eq. 3: R = T(P, W), K = N_e (computed by the last C update unless the
  // state is new)
  if (!c->r_next)
    HIP_TRY(launch_resp_tiles(c->Pp, c->Wt, c->np, c->Nep, c->dP, c->Nap, c->Ne, c->Na, Wold,
                              c->Nap, c->nP, c->nWc, c->R, active, s));
  PANDA_TRY(mark(c, PANDA_PHASE_AW));
  // Eq. 4 + Eq. 2 + Eq. 7 partials: A = T(W, C), K = N_a
  HIP_TRY(launch_avail_wupdate(c->Wr, c->np, Wold, c->C, c->dC, c->R, Wnew, c->Nap, c->Nep, c->Nap,
                               c->Ne, c->Na, c->nWr, c->nC, c->rule, c->hpart, c->skpart,
                               c->fold, active, s, c->packed));
  PANDA_TRY(mark(c, PANDA_PHASE_H));
  HIP_TRY(launch_finish_h(c->hpart, c->nh, c->Ne * c->Na, c->st, c->rule, s));
  // squared norms and planes of the new W
  HIP_TRY(launch_w_norms(Wnew, c->Ne, c->Na, c->Nap, c->Nep, c->nWr, c->nWc, c->colscr, c->Wr,
                         c->Wt, c->np, run_pc, s));
  PANDA_TRY(mark(c, PANDA_PHASE_PPART));
  // Eq. 5, P: T(W_i., W_m.) of the new W
  HIP_TRY(launch_coop_partial(c->Wr, c->np, c->Nep, c->Nap, c->splits, c->ppart, run_pc, s));
  PANDA_TRY(mark(c, PANDA_PHASE_PFIN));
  float* const tside = c->rule.sigma_from_T ? c->Tside : nullptr;
  double* const csq = c->rule.sigma_from_T ? c->csq : nullptr;
  HIP_TRY(launch_coop_finalize(c->ppart, c->splits, c->Nep, c->nWr, c->P, c->Nep, c->Ne, c->rule,
                               tside, c->Pp, c->np, run_pc, s));
  // Eq. 6 for P, and |P_i.|^2, before the C update, which also computes the
  // next R (which needs them)
  HIP_TRY(launch_diagonals(c->P, c->Nep, c->dP, c->Ne, tside, c->nP, c->dC, c->Nap, c->Na, c->cstat,
                           csq, coreg_slots(c->Nap), c->nC, c->rule, c->st, s, kDiagP));
  PANDA_TRY(mark(c, PANDA_PHASE_C));
  // Eq. 5, C: T(W_.k, W_.j) of the new W, upper tiles, mirrored (and the
  // next iteration's R = T(P, W) of the new P and W)
  HIP_TRY(launch_coreg_update_next_r(c->Wt, c->np, c->Nep, c->C, c->Nap, c->Nap, c->Na,
                                     c->nWc, c->rule, c->cstat, c->csq, c->corder_r, run_pc, s,
                                     c->packed, c->Pp, c->dP, c->nP, Wnew, c->Nap, c->Ne, c->R));
  PANDA_TRY(mark(c, PANDA_PHASE_DIAG));
  // Eq. 6 for C, and |C_.j|^2 for the next iteration
  HIP_TRY(launch_diagonals(c->P, c->Nep, c->dP, c->Ne, tside, c->nP, c->dC, c->Nap, c->Na, c->cstat,
                           csq, coreg_slots(c->Nap), c->nC, c->rule, c->st, s, kDiagC));
  c->r_next = true;
  PANDA_TRY(mark(c, PANDA_NPHASE));
  if (c->timing) c->npend += 1;
  c->enqueued += 1;
  return PANDA_OK;
}

// Whether the buffer that W shares holds R and the planes alone hold W.  An
// iteration that updates P and C ends that way: it writes the planes of its
// new W and the next R over W.  One that does not (the converging one without
// update_last) leaves its W in the buffer, and in the planes the W before.
// The state is that of the last read-back.
bool w_in_planes(const panda_ctx* c) {
  return c->w_in_place && c->r_next && (!c->host->conv || c->rule.update_last);
}

}  // namespace

namespace panda {

panda_status ctx_set_small(panda_ctx* c, bool small) {
  if (!c->loaded || c->small == small) {
    c->small = small;
    return PANDA_OK;
  }
  PANDA_TRY(read_state(c));
  const size_t n = (size_t)c->Nep * sizeof(double);
  if (c->host->t & 1)  // P's diagonal lies in the second vector in the small kernels
    HIP_TRY(hipMemcpyAsync(c->dP + (small ? c->Nep : 0), c->dP + (small ? 0 : c->Nep), n,
                           hipMemcpyDeviceToDevice, c->stream));
  c->small = small;
  if (!small && c->np) {  // the planes that the grouped kernels expect (and W's norms again)
    HIP_TRY(hipMemsetAsync(c->Pp.p, 0, (size_t)c->np * c->Nep * c->Nep * 2, c->stream));
    HIP_TRY(launch_split_offdiag(c->P, c->Ne, c->Nep, c->Pp, c->np, c->stream));
    HIP_TRY(launch_w_norms(c->W[c->executed & 1], c->Ne, c->Na, c->Nap, c->Nep, c->nWr, c->nWc,
                           c->colscr, c->Wr, c->Wt, c->np, nullptr, c->stream));
  }
  if (small)  // they expect R of the state they step from
    HIP_TRY(launch_small_finish(nullptr, small_inst_of(c, -c->executed - 1), 1,
                                SmallDims{c->Ne, c->Na}, small_rule_of(c), kSmallLoad, c->stream));
  return PANDA_OK;
}

panda_status ctx_current_w(panda_ctx* c, float** W) {
  *W = c->W[c->executed & 1];
  if (w_in_planes(c)) {
    HIP_TRY(launch_join_planes(c->Wr, c->Ne, c->Na, *W, c->Nap, c->stream));
    c->r_next = false;
  }
  return PANDA_OK;
}

panda_status ctx_load(panda_ctx* c, const float* W, const float* P, const float* C,
                      int32_t t) {
  if (!c || !W || t < 0) return fail(PANDA_ERR_ARG, "ctx_load: bad arguments%s");
  hipStream_t s = c->stream;
  const int64_t Ne = c->Ne, Na = c->Na, Nep = c->Nep, Nap = c->Nap;
  // an absent prior is the z-scored identity
  auto prior = [&](const float* src, int64_t n, PriorSrc* p) {
    double dv = 0.0, ov = 0.0;
    if (!src && !identity_zscore(n, c->opt.zscore_mode, c->opt.sigma_ddof, &dv, &ov)) return false;
    *p = PriorSrc{src, (float)dv, (float)ov};
    return true;
  };
  LoadArgs a{};
  if (!prior(P, Ne, &a.Psrc) || !prior(C, Na, &a.Csrc))
    return fail(PANDA_ERR_DEGENERATE, "identity prior of order 1 has std 0%s");
  a.Wsrc = W;
  a.Ne = Ne;
  a.Na = Na;
  a.Nep = Nep;
  a.Nap = Nap;
  a.W = c->W[0];
  a.W1 = c->w_in_place ? nullptr : c->W[1];
  a.P = c->P;
  a.C = c->packed ? nullptr : c->C;
  a.dP = diag_p_of(c, t);
  a.dC = c->dC;
  a.nP = c->nP;
  a.nC = c->nC;
  a.nWr = c->nWr;
  a.nWc = c->nWc;
  a.hpart = c->hpart;  // partials the A + W product never writes add zeros
  a.nh = c->nh;
  a.slots = c->csq;
  a.crows = c->crows;
  a.Pp = c->Pp;
  a.np = c->np;
  a.t = t;
  a.st = c->st;
  HIP_TRY(launch_load(a, s));
  if (c->packed)
    HIP_TRY(launch_load_packed(C, Na, Nap, a.Csrc.dval, a.Csrc.oval, c->C, c->dC, c->csq, c->nC, s));
  // norms (and planes) of W exactly as an iteration computes them, so a
  // stored state resumes bit for bit
  if (c->small) {
    const BInst d = small_inst_of(c, -1);
    const SmallDims mx{Ne, Na};
    const SmallRule rule = small_rule_of(c);
    HIP_TRY(launch_small_update(nullptr, d, 1, mx, rule, kSmallLoad, s));
    HIP_TRY(launch_small_finish(nullptr, d, 1, mx, rule, kSmallLoad, s));
  } else {
    HIP_TRY(launch_w_norms(c->W[0], Ne, Na, Nap, Nep, c->nWr, c->nWc, c->colscr, c->Wr, c->Wt,
                           c->np, nullptr, s));
    PANDA_TRY(ctx_fill_order(c));
  }
  c->r_next = false;
  c->t0 = t;
  c->executed = 0;
  c->enqueued = 0;
  c->host->h = 0.0;
  c->host->t = t;
  c->host->active = 1;
  c->host->conv = 0;
  c->loaded = true;
  c->fresh = false;
  return PANDA_OK;
}

// Iterate to convergence or max_iter.  The host never makes the device wait
// for it: the state after a polled iteration is copied to a pinned slot (with
// an event) as soon as that iteration is enqueued, and the host looks at it
// only after enqueueing the next iteration, so the device always has work
// queued while the host waits.  The one iteration enqueued after convergence
// runs gated (its kernels return at once: the executed iterations are always
// a prefix of the enqueued ones), so the result is that of polling at once.
panda_status run_loaded(panda_ctx* c) {
  const int64_t max_iter = c->opt.max_iter, poll = c->opt.poll_every;
  if (!c->snap) {
    HIP_TRY(hipHostMalloc(reinterpret_cast<void**>(&c->snap), 2 * sizeof(DevState),
                          hipHostMallocDefault));
    for (hipEvent_t& e : c->snap_ev) HIP_TRY(hipEventCreateWithFlags(&e, hipEventDisableTiming));
  }
  int64_t pending = -1;  // polled iteration whose state copy is awaited
  while (c->enqueued < max_iter) {
    const bool polled = (c->enqueued + 1) % poll == 0 && c->enqueued + 1 < max_iter;
    c->snap_to = c->small && polled ? &c->snap[(c->enqueued + 1) & 1] : nullptr;
    const panda_status st = enqueue_iteration(c);
    const bool copied = c->snap_to != nullptr;
    c->snap_to = nullptr;
    PANDA_TRY(st);
    const int64_t k = c->enqueued;
    if (pending >= 0) {
      HIP_TRY(hipEventSynchronize(c->snap_ev[pending & 1]));
      if (!c->snap[pending & 1].active) {
        // the state of the converging iteration is the final one: what is
        // queued behind it does nothing
        if (c->timing) break;
        *c->host = c->snap[pending & 1];
        c->executed = c->enqueued = c->host->t - c->t0;
        c->fresh = true;
        return PANDA_OK;
      }
      pending = -1;
    }
    if (polled) {
      if (!copied)
        HIP_TRY(hipMemcpyAsync(&c->snap[k & 1], c->st, sizeof(DevState), hipMemcpyDeviceToHost,
                               c->stream));
      HIP_TRY(hipEventRecord(c->snap_ev[k & 1], c->stream));
      pending = k;
    }
  }
  PANDA_TRY(read_state(c));
  c->enqueued = c->executed;
  return PANDA_OK;
}

}  // namespace panda

extern "C" {

void panda_default_options(panda_options* o) {
  if (!o) return;
  o->alpha = 0.1;
  o->tol = 1e-3;
  o->max_iter = 200;
  o->diag_alpha = 1;
  o->sigma_from_T = 0;
  o->n_own = 0;
  o->h_undamped = 0;
  o->update_last = 0;
  o->poll_every = 1;
  o->precision = PANDA_PREC_FP32;
  o->sigma_ddof = 0;
  o->zscore_mode = PANDA_ZSCORE_GLOBAL;
  o->packed_c = 0;
}

panda_status panda_ctx_set_timing(panda_ctx* c, int32_t enable) {
  if (!c) return fail(PANDA_ERR_ARG, "set_timing: NULL context%s");
  if (enable && !c->ev[0][0]) {
    for (int i = 0; i < kMaxPending; ++i)
      for (int p = 0; p <= PANDA_NPHASE; ++p) HIP_TRY(hipEventCreate(&c->ev[i][p]));
  }
  if (!enable && c->timing) {
    HIP_TRY(hipStreamSynchronize(c->stream));
    panda_status st = collect_times(c);
    if (st != PANDA_OK) return st;
  }
  c->timing = enable != 0;
  for (int p = 0; p < PANDA_NPHASE; ++p) {
    c->tot_ms[p] = 0.0;
    c->cnt[p] = 0;
  }
  return PANDA_OK;
}

panda_status panda_ctx_phase_times(panda_ctx* c, double* total_ms, int64_t* count) {
  if (!c) return fail(PANDA_ERR_ARG, "phase_times: NULL context%s");
  if (c->timing && c->npend) {
    HIP_TRY(hipStreamSynchronize(c->stream));
    panda_status st = collect_times(c);
    if (st != PANDA_OK) return st;
  }
  for (int p = 0; p < PANDA_NPHASE; ++p) {
    if (total_ms) total_ms[p] = c->tot_ms[p];
    if (count) count[p] = c->cnt[p];
  }
  return PANDA_OK;
}

const char* panda_status_string(panda_status s) {
  switch (s) {
    case PANDA_OK: return "ok";
    case PANDA_NOT_CONVERGED: return "not converged";
    case PANDA_ERR_ARG: return "invalid argument";
    case PANDA_ERR_DEGENERATE: return "degenerate network (std = 0)";
    case PANDA_ERR_NONFINITE: return "non-finite input";
    case PANDA_ERR_HIP: return "HIP runtime error";
    case PANDA_ERR_WORKSPACE: return "workspace too small or misaligned";
    case PANDA_STATUS_MAX_ENUM: break;  // sizes the enum, no status
  }
  return "unknown status";
}

const char* panda_last_error(void) { return g_err; }

size_t panda_normalize_workspace_bytes(void) { return align_up(kZsScratch * sizeof(double)); }

panda_status panda_normalize(float* M, int64_t rows, int64_t cols, void* workspace,
                             size_t ws_bytes, hipStream_t stream) {
  if (!M || rows < 1 || cols < 1) return fail(PANDA_ERR_ARG, "normalize: bad matrix%s");
  if (!workspace || ws_bytes < panda_normalize_workspace_bytes() ||
      (reinterpret_cast<uintptr_t>(workspace) % kAlign))
    return fail(PANDA_ERR_WORKSPACE, "normalize: workspace too small or misaligned%s");
  return zscore(M, rows, cols, cols, PANDA_ZSCORE_GLOBAL, 0, static_cast<double*>(workspace),
                stream);
}

size_t panda_normalize_ex_workspace_bytes(int64_t rows, int64_t cols, int32_t zscore_mode) {
  if (rows < 1 || cols < 1 || zscore_mode < PANDA_ZSCORE_GLOBAL ||
      zscore_mode > PANDA_ZSCORE_ROWCOL)
    return 0;
  return align_up(zscore_scratch_doubles(rows, cols, zscore_mode) * sizeof(double));
}

panda_status panda_normalize_ex(float* M, int64_t rows, int64_t cols, int32_t zscore_mode,
                                int32_t ddof, void* workspace, size_t ws_bytes,
                                hipStream_t stream) {
  if (!M || rows < 1 || cols < 1) return fail(PANDA_ERR_ARG, "normalize_ex: bad matrix%s");
  if (zscore_mode < PANDA_ZSCORE_GLOBAL || zscore_mode > PANDA_ZSCORE_ROWCOL || ddof < 0 ||
      ddof > 1)
    return fail(PANDA_ERR_ARG, "normalize_ex: unknown zscore_mode or ddof%s");
  if (!workspace || ws_bytes < panda_normalize_ex_workspace_bytes(rows, cols, zscore_mode) ||
      (reinterpret_cast<uintptr_t>(workspace) % kAlign))
    return fail(PANDA_ERR_WORKSPACE, "normalize_ex: workspace too small or misaligned%s");
  return zscore(M, rows, cols, cols, zscore_mode, ddof, static_cast<double*>(workspace), stream);
}

namespace {
struct TaniLayout {
  float *Xp, *Yp, *part;
  double *nx, *ny, *scr;
};
static size_t tanimoto_layout(int64_t M, int64_t K, int64_t N, char* base, TaniLayout* L) {
  const int64_t Mp = round_up(M, kPadE), Kp = round_up(K, kPadK), Np = round_up(N, kPadA);
  Carver cv{base};
  float* xp = cv.take<float>((size_t)Mp * Kp);
  float* yp = cv.take<float>((size_t)Kp * Np);
  float* pt = cv.take<float>(rect_partial_floats());
  double* nx = cv.take<double>((size_t)Mp);
  double* ny = cv.take<double>((size_t)Np);
  double* sc = cv.take<double>((size_t)kColChunks * (size_t)Np);
  if (L) *L = TaniLayout{xp, yp, pt, nx, ny, sc};
  return cv.off;
}
}  // namespace

size_t panda_tanimoto_workspace_bytes(int64_t M, int64_t K, int64_t N) {
  if (M < 1 || K < 1 || N < 1) return 0;
  return tanimoto_layout(M, K, N, nullptr, nullptr);
}

panda_status panda_tanimoto(const float* X, const float* Y, int64_t M, int64_t K, int64_t N,
                            float* Out, void* workspace, size_t ws_bytes, hipStream_t s) {
  if (!X || !Y || !Out || M < 1 || K < 1 || N < 1 || M > (1 << 20) || N > (1 << 20) ||
      K > (1 << 20))
    return fail(PANDA_ERR_ARG, "tanimoto: bad arguments%s");
  const size_t need = panda_tanimoto_workspace_bytes(M, K, N);
  if (!workspace || ws_bytes < need || (reinterpret_cast<uintptr_t>(workspace) % kAlign))
    return fail(PANDA_ERR_WORKSPACE, "tanimoto: workspace too small or misaligned%s");
  const int64_t Mp = round_up(M, kPadE), Kp = round_up(K, kPadK), Np = round_up(N, kPadA);
  TaniLayout L;
  tanimoto_layout(M, K, N, static_cast<char*>(workspace), &L);
  PackArgs a{X, Y, M, K, N, Mp, Kp, Np, L.Xp, L.Yp, L.nx, L.ny, L.scr, 0};
  a.rows = std::max<int64_t>(32, round_up((Kp + kColChunks - 1) / kColChunks, 8));
  HIP_TRY(launch_pack_xy(a, s));
  HIP_TRY(launch_tanimoto_store(L.Xp, Kp, L.Yp, Np, Mp, Np, Kp, M, N, K, L.nx, L.ny, Out, N, L.part,
                                nullptr, s));
  return PANDA_OK;
}

namespace {
struct PearsonLayout {
  double2* stat;
  float* Zt;
};
static size_t pearson_layout(int64_t G, int64_t S, char* base, PearsonLayout* L) {
  const int64_t Gp = round_up(G, kPadA), Sp = round_up(S, kPadK);
  Carver cv{base};
  double2* st = cv.take<double2>((size_t)G);
  float* zt = cv.take<float>((size_t)Sp * Gp);
  if (L) *L = PearsonLayout{st, zt};
  return cv.off;
}
}  // namespace

size_t panda_pearson_workspace_bytes(int64_t G, int64_t S) {
  if (G < 1 || S < 2) return 0;
  return pearson_layout(G, S, nullptr, nullptr);
}

namespace {
bool pearson_args_ok(const float* E, int64_t G, int64_t S, int64_t lde, const float* C,
                     int64_t ldc) {
  return E && C && G >= 1 && S >= 2 && G <= (1 << 18) && S <= (1 << 20) && lde >= S && ldc >= G;
}

// The two kernels of the prior on a scratch region laid out by
// pearson_layout; every byte of it that they read they have written first.
panda_status pearson_enqueue(const float* E, int64_t G, int64_t S, int64_t lde, float* C,
                             int64_t ldc, char* base, hipStream_t s) {
  const int64_t Gp = round_up(G, kPadA), Sp = round_up(S, kPadK);
  PearsonLayout L;
  pearson_layout(G, S, base, &L);
  HIP_TRY(launch_pearson_z(E, G, S, lde, L.stat, L.Zt, Gp, Sp, s));
  HIP_TRY(launch_corr(L.Zt, Gp, Sp, S, G, C, ldc, s));
  return PANDA_OK;
}

// Scratch of panda_pearson_noalloc, one copy on every GPU the library runs
// on, held until the process ends.  In host code `scratch` names a host-side
// stand-in, not the device array: its device address comes from
// hipGetSymbolAddress, once per device, and only that address is used.
static __device__ __align__(256) unsigned char scratch[PANDA_NOALLOC_SCRATCH_BYTES];
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_dev[kMaxDevices];

panda_status scratch_address(void** out) {
  int dev = -1;
  HIP_TRY(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) return fail(PANDA_ERR_ARG, "pearson_noalloc: device id out of range%s");
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_dev[dev]) {
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return hip_fail(e, "hipGetSymbolAddress(scratch)");
    if (!p) return fail(PANDA_ERR_HIP, "pearson_noalloc: no device address for the scratch array%s");
    g_scratch_dev[dev] = p;
  }
  *out = g_scratch_dev[dev];
  return PANDA_OK;
}
}  // namespace

panda_status panda_pearson(const float* E, int64_t G, int64_t S, int64_t lde, float* C,
                           int64_t ldc, void* workspace, size_t ws_bytes, hipStream_t s) {
  if (!pearson_args_ok(E, G, S, lde, C, ldc)) return fail(PANDA_ERR_ARG, "pearson: bad arguments%s");
  const size_t need = panda_pearson_workspace_bytes(G, S);
  if (!workspace || ws_bytes < need || (reinterpret_cast<uintptr_t>(workspace) % kAlign))
    return fail(PANDA_ERR_WORKSPACE, "pearson: workspace too small or misaligned%s");
  return pearson_enqueue(E, G, S, lde, C, ldc, static_cast<char*>(workspace), s);
}

panda_status panda_pearson_noalloc(const float* E, int64_t G, int64_t S, int64_t lde, float* C,
                                   int64_t ldc, hipStream_t s) {
  if (!pearson_args_ok(E, G, S, lde, C, ldc))
    return fail(PANDA_ERR_ARG, "pearson_noalloc: bad arguments%s");
  const size_t need = panda_pearson_workspace_bytes(G, S);
  if (need > (size_t)PANDA_NOALLOC_SCRATCH_BYTES) {
    snprintf(g_err, sizeof g_err,
             "pearson_noalloc: G = %lld genes x S = %lld samples need %zu bytes of scratch, more "
             "than the %zu the library holds; use panda_pearson with a workspace",
             (long long)G, (long long)S, need, (size_t)PANDA_NOALLOC_SCRATCH_BYTES);
    return PANDA_ERR_ARG;
  }
  void* base = nullptr;
  PANDA_TRY(scratch_address(&base));
  return pearson_enqueue(E, G, S, lde, C, ldc, static_cast<char*>(base), s);
}

size_t panda_workspace_bytes(int64_t Ne, int64_t Na, const panda_options* opt) {
  (void)opt;
  if (!dims_ok(Ne, Na)) return 0;
  return ctx_layout(Ne, Na, opt ? opt->precision : PANDA_PREC_FP32,
                    single_spec(Ne, Na, opt && opt->packed_c,
                                opt ? opt->precision : PANDA_PREC_FP32),
                    nullptr, nullptr);
}

panda_status panda_ctx_create(int64_t Ne, int64_t Na, const panda_options* opt, void* workspace,
                              size_t ws_bytes, hipStream_t stream, panda_ctx** out) {
  if (!out) return fail(PANDA_ERR_ARG, "ctx_create: out is NULL%s");
  *out = nullptr;
  if (!dims_ok(Ne, Na)) return fail(PANDA_ERR_ARG, "ctx_create: bad dimensions%s");
  panda_options o;
  if (opt)
    o = *opt;
  else
    panda_default_options(&o);
  panda_status st = check_options(o);
  if (st != PANDA_OK) return st;
  if (!workspace || ws_bytes < panda_workspace_bytes(Ne, Na, &o) ||
      (reinterpret_cast<uintptr_t>(workspace) % kAlign))
    return fail(PANDA_ERR_WORKSPACE, "ctx_create: workspace too small or misaligned%s");
  panda_ctx* c = new (std::nothrow) panda_ctx();
  if (!c) return fail(PANDA_ERR_ARG, "ctx_create: out of host memory%s");
  st = ctx_setup(c, Ne, Na, o, single_spec(Ne, Na, o.packed_c != 0, o.precision),
                 static_cast<char*>(workspace), stream);
  if (st != PANDA_OK) {
    delete c;
    return st;
  }
  *out = c;
  return PANDA_OK;
}

void panda_ctx_destroy(panda_ctx* c) {
  if (!c) return;
  ctx_free(c);
  delete c;
}

panda_status panda_ctx_load(panda_ctx* c, const float* W, const float* P, const float* C,
                            int32_t t) {
  PANDA_TRY(ctx_load(c, W, P, C, t));
  // the caller may free or reuse its buffers, which need not belong to the
  // context's stream
  HIP_TRY(hipStreamSynchronize(c->stream));
  return PANDA_OK;
}

panda_status panda_iterate(panda_ctx* c, double* h, int32_t* t) {
  if (!c || !c->loaded) return fail(PANDA_ERR_ARG, "iterate: context not loaded%s");
  if (c->host->active) {
    panda_status st = enqueue_iteration(c);
    if (st != PANDA_OK) return st;
  }
  panda_status st = read_state(c);
  if (st != PANDA_OK) return st;
  c->enqueued = c->executed;
  if (h) *h = c->host->h;
  if (t) *t = c->host->t;
  return PANDA_OK;
}

panda_status panda_ctx_store(panda_ctx* c, float* W, float* P, float* C, double* h, int32_t* t) {
  if (!c || !c->loaded) return fail(PANDA_ERR_ARG, "ctx_store: context not loaded%s");
  if (!c->fresh) PANDA_TRY(read_state(c));
  StoreArgs a{};
  a.Wbuf = w_in_planes(c) ? nullptr : c->W[c->executed & 1];
  a.Wr = c->Wr;
  a.P = c->P;
  a.C = c->C;
  a.dP = diag_p_of(c, c->host->t);
  a.dC = c->dC;
  a.Ne = c->Ne;
  a.Na = c->Na;
  a.Nep = c->Nep;
  a.Nap = c->Nap;
  a.W = W;
  a.Pout = P;
  a.Cout = c->packed ? nullptr : C;
  HIP_TRY(launch_store(a, c->stream));
  if (C && c->packed) {
    HIP_TRY(launch_unpack_sym(c->C, c->Na, c->Nap, C, c->Na, c->stream));
    HIP_TRY(launch_put_diag(C, c->Na, c->Na, c->dC, c->stream));
  }
  if (h) *h = c->host->h;
  if (t) *t = c->host->t;
  return PANDA_OK;
}

panda_status panda_run(const float* W0, const float* P0, const float* C0, int64_t Ne, int64_t Na,
                       double alpha, double tol, int32_t max_iter, float* W, float* P, float* C,
                       void* workspace, size_t ws_bytes, const panda_options* opt,
                       int32_t* iters, double* h, hipStream_t stream) {
  if (!W0 || !W || !P || !C) return fail(PANDA_ERR_ARG, "run: NULL matrix pointer%s");
  panda_options o;
  if (opt)
    o = *opt;
  else
    panda_default_options(&o);
  o.alpha = alpha;
  o.tol = tol;
  o.max_iter = max_iter;
  panda_ctx* c = nullptr;
  panda_status st = panda_ctx_create(Ne, Na, &o, workspace, ws_bytes, stream, &c);
  if (st != PANDA_OK) return st;
  st = ctx_load(c, W0, P0, C0, 0);
  if (st == PANDA_OK) st = run_loaded(c);
  if (st == PANDA_OK) st = panda_ctx_store(c, W, P, C, h, iters);
  if (st == PANDA_OK && c->host->active) st = PANDA_NOT_CONVERGED;
  panda_ctx_destroy(c);
  return st;
}

}  // extern "C"

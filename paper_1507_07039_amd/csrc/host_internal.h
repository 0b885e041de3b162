// Host-side internals shared by the single-network API (panda_api.hip) and
// the batched API (batch_api.hip): error reporting, the workspace carver, the
// per-network context and its workspace layout.
#pragma once

#include "panda.h"

#include <stdio.h>

#include "load_internal.h"
#include "small_internal.h"

namespace panda {

// Error text of the calling thread (panda_last_error); returns st.
panda_status fail(panda_status st, const char* fmt, const char* what = "");
panda_status hip_fail(hipError_t e, const char* where);

#define HIP_TRY(call)                                         \
  do {                                                        \
    hipError_t e_ = (call);                                   \
    if (e_ != hipSuccess) return panda::hip_fail(e_, #call);  \
  } while (0)

#define PANDA_TRY(call)                      \
  do {                                       \
    panda_status s_ = (call);                \
    if (s_ != PANDA_OK) return s_;           \
  } while (0)

constexpr size_t kAlign = 256;
inline size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

// Bump allocator over the caller's workspace (sizes only when base is null).
struct Carver {
  char* base;
  size_t off = 0;
  template <typename T>
  T* take(size_t count) {
    T* p = base ? reinterpret_cast<T*>(base + off) : nullptr;
    off += align_up(count * sizeof(T));
    return p;
  }
};

// Scratch (doubles) of a z-score of a rows x cols network with the given
// scope: the global form's block moments, or 8 flags plus the per-row and
// per-column moments and the column chunks' moments.
size_t zscore_scratch_doubles(int64_t rows, int64_t cols, int32_t mode);
// Diagonal and off-diagonal value of the z-scored identity of order n; false
// if its standard deviation is 0.
bool identity_zscore(int64_t n, int32_t mode, int32_t ddof, double* dv, double* ov);
// Z-score in place (Sec. II-A) with the scope and normaliser of the
// options; synchronises the stream to read the degeneracy flags.
panda_status zscore(float* M, int64_t rows, int64_t cols, int64_t ld, int32_t mode, int32_t ddof,
                    double* scratch, hipStream_t s);
constexpr int kMaxPending = 16;               // timed iterations between read-backs

Rule rule_of(const panda_options& o);
panda_status check_options(const panda_options& o);
// PANDA() from a loaded context until h < tol or max_iter (panda_run's loop).
panda_status run_loaded(panda_ctx* c);
bool dims_ok(int64_t Ne, int64_t Na);

// Sizes of the buffers whose extent depends on the tile schedule.  The
// single-network schedule fixes them; a batch sizes them for the smallest
// tile and K chunk among its candidates, and needs no stream-K scratch.
struct LayoutSpec {
  bool batched;
  int64_t hpart_tiles;  // per-tile h partials of the A + W product
  int64_t ppart_splits; // K splits of the W W^T partial products
  bool packed_c = false; // C as its upper tiles (packed_tile)
};
LayoutSpec single_spec(int64_t Ne, int64_t Na, bool packed_c, int32_t precision);
// A network of a batch, sized for every tile candidate: the smallest A + W tile
// (64 x 64) and the smallest W W^T chunk.
LayoutSpec batch_spec(int64_t Ne, int64_t Na);
// Whether a batch of n networks, all of them small (small_net), runs faster in
// the small kernels than in the grouped ones.
bool small_batch(int32_t n, const int64_t* Ne, const int64_t* Na, int32_t precision);

}  // namespace panda

struct panda_ctx {
  int64_t Ne, Na, Nep, Nap;
  panda_options opt;
  panda::Rule rule;
  hipStream_t stream;
  // W, the W being written, and R.  In the FP32 form of a single network the
  // three are one buffer: the planes hold W (join_planes), A reads R there and
  // leaves the new W in its place, and the next R replaces that (see w_in_place)
  float* W[2];
  float* R;
  float* P;
  float* C;
  float* Tside;
  float* ppart;   // split-K partial products of W W^T
  float* skpart;  // stream-K partial tiles (single-network schedule only)
  float* fold;    // running sums of the A product over long K (FP32 form, else null)
  double* dP;     // diagonal of P (FP64; P holds zero there; see diag_p_of)
  double* dC;     // diagonal of C
  double* nP;     // |P_i.|^2
  double* nC;     // |C_.j|^2
  double* nWr;    // |W_i.|^2
  double* nWc;    // |W_.j|^2
  double* colscr; // column-norm scratch
  double* hpart;
  double2* cstat;
  double* csq;
  int64_t crows;    // rows of C whose squares a load sums in one slot of csq
  uint32_t* corder;  // launch order of the upper C tiles
  uint32_t* corder_r;  // the same with the R tiles of the next iteration (not in a batch)
  bool small;       // iterates in the small kernels (small_internal.h)
  bool w_in_place;  // W and R share a buffer (FP32 form of a single network)
  bool r_next;  // R holds T(P, W) of the current state (computed by the last C update)
  panda::DevState* st;
  int np;       // bf16 planes of the operands: 2 (split-BF16) or 3 (FP32); 0: none (FP32 batch)
  bool packed;  // C stored as its upper tiles (packed_tile)
  panda::Planes Wr, Wt, Pp;  // of W, W^T and P without its diagonal (C stays FP32)
  panda::DevState* host;  // pinned
  panda::DevState* snap;  // pinned, two slots: states copied ahead (run_loaded)
  hipEvent_t snap_ev[2];
  panda::DevState* snap_to;  // slot that the iteration being enqueued fills itself (small), or null
  int splits;
  int64_t nh;
  int32_t t0;
  int64_t executed;  // iterations known to have run since load
  int64_t enqueued;  // iterations enqueued since load
  bool loaded;
  bool fresh;  // host holds the state of everything enqueued
  // phase timing
  bool timing;
  int npend;
  hipEvent_t ev[16][PANDA_NPHASE + 1];
  double tot_ms[PANDA_NPHASE];
  int64_t cnt[PANDA_NPHASE];
};

namespace panda {

// Workspace layout of one network: fills c (when not null) with pointers
// into base and returns the bytes used.
size_t ctx_layout(int64_t Ne, int64_t Na, int32_t precision, const LayoutSpec& spec, panda_ctx* c,
                  char* base);
// Context over an already carved workspace (no argument checks), with its
// pinned state mirror; ctx_free releases what ctx_setup acquired.
panda_status ctx_setup(panda_ctx* c, int64_t Ne, int64_t Na, const panda_options& o,
                       const LayoutSpec& spec, char* base, hipStream_t stream);
void ctx_free(panda_ctx* c);
// P's diagonal at iteration t: the small kernels alternate between two vectors.
inline double* diag_p_of(const panda_ctx* c, int32_t t) {
  return c->dP + (c->small && (t & 1) ? c->Nep : 0);
}
// Rules and descriptor of a network for the small and grouped kernels.
SmallRule small_rule_of(const panda_ctx* c);
BInst inst_of(const panda_ctx* c);
// The same for the small kernels of one network, step k since the load (k < 0:
// outside a step, after -k - 1 of them).
BInst small_inst_of(const panda_ctx* c, int64_t k);
// Into (or out of) the small kernels: a loaded state is carried over.
panda_status ctx_set_small(panda_ctx* c, bool small);
// The current W of a loaded context as an FP32 matrix (leading dimension
// Nap), for callers between iterations; R, which may share its buffer, is
// computed again by the next iteration.
panda_status ctx_current_w(panda_ctx* c, float** W);
// panda_ctx_load without its wait for the copies out of W, P and C.
panda_status ctx_load(panda_ctx* c, const float* W, const float* P, const float* C, int32_t t);
// Launch-order tables of the upper C tiles, enqueued on the context's stream.
panda_status ctx_fill_order(panda_ctx* c);

}  // namespace panda

// Moving a network's state into and out of a context's workspace (load.hip).
#pragma once

#include "panda_internal.h"

namespace panda {

// A prior that is the z-scored identity when src is null: dval on the
// diagonal, oval off it.
struct PriorSrc {
  const float* src;
  float dval, oval;
};

// Everything a load writes, in one launch: W (and zeros in W1 where given), P
// and C padded with zeros and without their diagonals, the diagonals, the
// squared norms of P's rows and C's columns, P's planes, zeros in nWr, nWc and
// hpart, and the iteration state at t.  C's norms go through `slots`, Nap
// doubles for each chunk of crows rows.  C null: it is stored packed
// (launch_load_packed).
struct LoadArgs {
  const float* Wsrc;
  PriorSrc Psrc, Csrc;
  int64_t Ne, Na, Nep, Nap;
  float *W, *W1, *P, *C;
  double *dP, *dC, *nP, *nC, *nWr, *nWc, *hpart;
  int64_t nh;
  double* slots;
  int64_t crows;
  Planes Pp;
  int32_t np, t;
  DevState* st;
};
hipError_t launch_load(const LoadArgs& a, hipStream_t s);

// The state out of a context: W (from its buffer, or from three planes where
// Wbuf is null), P and C with their diagonals back; null outputs are skipped.
struct StoreArgs {
  const float *Wbuf, *P, *C;
  Planes Wr;
  const double *dP, *dC;
  int64_t Ne, Na, Nep, Nap;
  float *W, *Pout, *Cout;
};
hipError_t launch_store(const StoreArgs& a, hipStream_t s);

// Operands of a stand-alone similarity, padded with zeros, and the squared
// norms of X's rows and Y's columns (the latter through `slots`, Np doubles
// for each chunk of `rows` rows of Y).  Two launches where copies, fills and
// norms by themselves took seven: 700 x 2001 x 5003 went from 85 us beside the
// product's 94 to 29.
struct PackArgs {
  const float *X, *Y;
  int64_t M, K, N, Mp, Kp, Np;
  float *Xp, *Yp;
  double *nx, *ny, *slots;
  int64_t rows;
};
hipError_t launch_pack_xy(const PackArgs& a, hipStream_t s);

// The launch orders of the C update, written on the device: the upper tiles by
// super-tiles of group x group, and, unless corder_r is null, the same order
// with the next R's tiles after each XCD's share of C tiles.
hipError_t launch_order(int64_t Nep, int64_t Nap, int group, uint32_t* corder, uint32_t* corder_r,
                        hipStream_t s);

}  // namespace panda

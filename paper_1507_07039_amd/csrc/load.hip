// Loading and storing a context's state.  Both are bound by memory, or for a
// small network by launches: each entry is read once and written once, with
// its norm and its diagonal taken on the way, in one launch (and one for the
// sum of C's column norms).  P and C of 700 and 18000 are loaded in 0.55 ms
// and stored in 0.53 (2.6 GB each: 4.8 TB/s, a copy's rate); as fills, strided
// copies, norms and diagonals by themselves they took 1.2 and 0.6 ms.  500 x
// 500: 29 us on the device, where some twenty launches and two synchronised
// copies of host-built order tables took about 200.
#include "load_internal.h"

#include "update_device.h"

namespace panda {
namespace {

constexpr int kLT = upd::kUT;
typedef float f4 __attribute__((ext_vector_type(4)));

// Four entries c .. c + 3 of a row of n (16-byte loads where `al`); zero past n.
__device__ __forceinline__ f4 row4(const float* __restrict__ row, int64_t c, int64_t n, bool al) {
  if (al && c + 3 < n) return *reinterpret_cast<const f4*>(row + c);
  f4 v;
#pragma unroll
  for (int e = 0; e < 4; ++e) v[e] = c + e < n ? row[c + e] : 0.0f;
  return v;
}
__device__ __forceinline__ void put4(float* __restrict__ row, int64_t c, int64_t n, bool al,
                                     const f4& v) {
  if (al && c + 3 < n) {
    __builtin_nontemporal_store(v, reinterpret_cast<f4*>(row + c));
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (c + e < n) row[c + e] = v[e];
  }
}
__host__ __device__ constexpr int64_t c_strips(int64_t Nap) {
  return (Nap + 4 * kLT - 1) / (4 * kLT);
}
__device__ __forceinline__ bool aligned16(const void* p, int64_t ld) {
  return (reinterpret_cast<uintptr_t>(p) & 15) == 0 && ld % 4 == 0;
}

// Entries c .. c + 3 of row i of a prior of order n; zero past n.
__device__ __forceinline__ f4 prior4(const PriorSrc& s, int64_t i, int64_t c, int64_t n, bool al) {
  f4 v = {0.f, 0.f, 0.f, 0.f};
  if (i >= n || c >= n) return v;
  if (s.src) return row4(s.src + i * n, c, n, al);
#pragma unroll
  for (int e = 0; e < 4; ++e) v[e] = c + e >= n ? 0.0f : c + e == i ? s.dval : s.oval;
  return v;
}

// Row i of P (order n, leading dimension ld, zero past n), its diagonal
// entry, its squared norm and its planes.
__device__ __forceinline__ void load_p_row(const PriorSrc& s, int64_t i, int64_t n,
                                           float* __restrict__ dst, int64_t ld,
                                           double* __restrict__ diag, double* __restrict__ norm,
                                           const Planes& pl, int np, double* red) {
  constexpr int U = 4;
  const bool al = s.src && aligned16(s.src, n);
  float* out = dst + i * ld;
  double q = 0.0;
  for (int64_t c0 = 4 * threadIdx.x; c0 < ld; c0 += 4 * kLT * U) {
    f4 v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t c = c0 + u * 4 * kLT;
      v[u] = prior4(s, i, c, n, al);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t c = c0 + u * 4 * kLT;
      if (c >= ld) continue;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        q += (double)v[u][e] * (double)v[u][e];
        if (c + e == i && i < n) {
          diag[i] = (double)v[u][e];
          v[u][e] = 0.0f;
        }
        if (np) upd::put_planes(pl, np, i, c + e, v[u][e]);
      }
      *reinterpret_cast<f4*>(out + c) = v[u];
    }
  }
  const double tot = upd::block_sum(q, red);
  if (threadIdx.x == 0) norm[i] = tot;
}

// Rows [i0, i1) of 1024 columns of C (order n, leading dimension ld): four
// columns per thread, their sums of squares over the rows to `slot`.
__device__ __forceinline__ void load_c_part(const PriorSrc& s, int64_t i0, int64_t i1, int64_t c,
                                            int64_t n, float* __restrict__ dst, int64_t ld,
                                            double* __restrict__ diag,
                                            double* __restrict__ slot) {
  constexpr int U = 8;
  if (c >= ld) return;
  const bool al = s.src && aligned16(s.src, n);
  double q[4] = {0.0, 0.0, 0.0, 0.0};
  for (int64_t r0 = i0; r0 < i1; r0 += U) {
    f4 v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = prior4(s, r0 + u < i1 ? r0 + u : n, c, n, al);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t i = r0 + u;
      if (i >= i1) break;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        q[e] += (double)v[u][e] * (double)v[u][e];
        if (c + e == i && i < n) {
          diag[i] = (double)v[u][e];
          v[u][e] = 0.0f;
        }
      }
      *reinterpret_cast<f4*>(dst + i * ld + c) = v[u];
    }
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) slot[c + e] = q[e];
}

__global__ __launch_bounds__(kLT) void k_load(LoadArgs a) {
  __shared__ double red[4];
  int64_t b = blockIdx.x;
  if (b < a.Nep) {  // W
    const bool al = aligned16(a.Wsrc, a.Na);
    for (int64_t c = 4 * threadIdx.x; c < a.Nap; c += 4 * kLT) {
      const f4 z = {0.f, 0.f, 0.f, 0.f};
      *reinterpret_cast<f4*>(a.W + b * a.Nap + c) =
          b < a.Ne && c < a.Na ? row4(a.Wsrc + b * a.Na, c, a.Na, al) : z;
      if (a.W1) *reinterpret_cast<f4*>(a.W1 + b * a.Nap + c) = z;
    }
    return;
  }
  b -= a.Nep;
  if (b < a.Nep) {
    load_p_row(a.Psrc, b, a.Ne, a.P, a.Nep, a.dP, a.nP, a.Pp, a.np, red);
    return;
  }
  b -= a.Nep;
  if (a.C) {
    const int64_t strips = c_strips(a.Nap), nq = (a.Na + a.crows - 1) / a.crows;
    if (b < strips * nq) {
      const int64_t k = b / strips;  // chunk of rows; the last takes the padding
      load_c_part(a.Csrc, k * a.crows, k + 1 == nq ? a.Nap : (k + 1) * a.crows,
                  4 * kLT * (b % strips) + 4 * threadIdx.x, a.Na, a.C, a.Nap, a.dC,
                  a.slots + k * a.Nap);
      return;
    }
    b -= strips * nq;
  }
  // the vectors that start at zero, and the state
  int64_t k = b * kLT + threadIdx.x;
  if (k == 0) *a.st = DevState{0.0, a.t, 1, 0, 0, 0, 0};
  if (k < a.Nep) a.nWr[k] = 0.0;
  if (k < a.Nap) a.nWc[k] = 0.0;
  if (k < a.nh) a.hpart[k] = 0.0;
}

// Blocks [0, Mp): a row of X each, padded, with its squared norm; then (chunk
// of rows, 1024 columns) of Y, padded, with the columns' partial sums of
// squares.
__global__ __launch_bounds__(kLT) void k_pack_xy(PackArgs a) {
  __shared__ double red[4];
  constexpr int U = 8;
  const int64_t b = blockIdx.x;
  if (b < a.Mp) {
    const bool al = aligned16(a.X, a.K);
    double q = 0.0;
    for (int64_t c = 4 * threadIdx.x; c < a.Kp; c += 4 * kLT) {
      f4 v = {0.f, 0.f, 0.f, 0.f};
      if (b < a.M && c < a.K) v = row4(a.X + b * a.K, c, a.K, al);
#pragma unroll
      for (int e = 0; e < 4; ++e) q += (double)v[e] * (double)v[e];
      *reinterpret_cast<f4*>(a.Xp + b * a.Kp + c) = v;
    }
    const double tot = upd::block_sum(q, red);
    if (threadIdx.x == 0) a.nx[b] = tot;
    return;
  }
  const int64_t strips = c_strips(a.Np), k = (b - a.Mp) / strips;
  const int64_t c = 4 * kLT * ((b - a.Mp) % strips) + 4 * threadIdx.x;
  if (c >= a.Np) return;
  const int64_t i0 = k * a.rows, i1 = i0 + a.rows < a.Kp ? i0 + a.rows : a.Kp;
  const bool al = aligned16(a.Y, a.N);
  double q[4] = {0.0, 0.0, 0.0, 0.0};
  for (int64_t r0 = i0; r0 < i1; r0 += U) {
    f4 v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      v[u] = f4{0.f, 0.f, 0.f, 0.f};
      if (r0 + u < i1 && r0 + u < a.K && c < a.N) v[u] = row4(a.Y + (r0 + u) * a.N, c, a.N, al);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (r0 + u >= i1) break;
#pragma unroll
      for (int e = 0; e < 4; ++e) q[e] += (double)v[u][e] * (double)v[u][e];
      *reinterpret_cast<f4*>(a.Yp + (r0 + u) * a.Np + c) = v[u];
    }
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) a.slots[k * a.Np + c + e] = q[e];
}

__global__ __launch_bounds__(kLT) void k_store(StoreArgs a) {
  int64_t b = blockIdx.x;
  if (a.W) {
    if (b < a.Ne) {
      const bool al = aligned16(a.W, a.Na);
      for (int64_t c = 4 * threadIdx.x; c < a.Na; c += 4 * kLT) {
        f4 v;
        if (a.Wbuf) {
          v = *reinterpret_cast<const f4*>(a.Wbuf + b * a.Nap + c);
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = join_planes(a.Wr, b, c + e);  // (zero past Na)
        }
        put4(a.W + b * a.Na, c, a.Na, al, v);
      }
      return;
    }
    b -= a.Ne;
  }
  const bool is_p = a.Pout && b < a.Ne;
  if (a.Pout && !is_p) b -= a.Ne;
  const int64_t n = is_p ? a.Ne : a.Na, ld = is_p ? a.Nep : a.Nap;
  const float* src = (is_p ? a.P : a.C) + b * ld;
  float* dst = (is_p ? a.Pout : a.Cout) + b * n;
  const float d = (float)(is_p ? a.dP : a.dC)[b];
  const bool al = aligned16(is_p ? a.Pout : a.Cout, n);
  constexpr int U = 4;
  for (int64_t c0 = 4 * threadIdx.x; c0 < n; c0 += 4 * kLT * U) {
    f4 v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t c = c0 + u * 4 * kLT;
      if (c < n) v[u] = __builtin_nontemporal_load(reinterpret_cast<const f4*>(src + c));
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t c = c0 + u * 4 * kLT;
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (c + e == b) v[u][e] = d;
      if (c < n) put4(dst, c, n, al, v[u]);
    }
  }
}

// The order of the upper C tiles (kCoregGroup): super-tiles of g x g tiles,
// column of super-tiles after column and downwards in each, the tiles of one
// column by column.  So tile (I, J) comes after the columns of super-tiles
// before J's, the super-tiles above I's in its own, and the tiles before it
// there.
__device__ __forceinline__ int64_t order_of(int64_t I, int64_t J, int64_t nT, int64_t g) {
  const int64_t J0 = J / g * g, J1 = J0 + g < nT ? J0 + g : nT, I0 = I / g * g;
  const int64_t before = J0 * (J0 + 1) / 2 + I0 * (J1 - J0);
  return before + (I0 == J0 ? (J - J0) * (J - J0 + 1) / 2 + (I - I0) : (J - J0) * g + (I - I0));
}

__global__ __launch_bounds__(kLT) void k_order(int64_t nT, int64_t g, int64_t nRT, int64_t nR,
                                               uint32_t r_tile, uint32_t* __restrict__ corder,
                                               uint32_t* __restrict__ corder_r) {
  const int64_t nC = nT * (nT + 1) / 2, n = nC + nR;
  const int64_t k = (int64_t)blockIdx.x * kLT + threadIdx.x;
  if (k >= n) return;
  uint32_t entry;
  int64_t item;  // among the C tiles (in their order), or among the R tiles
  if (k < nC) {
    int64_t J = (int64_t)((sqrt(8.0 * (double)k + 1.0) - 1.0) * 0.5);
    while (J * (J + 1) / 2 > k) --J;
    while ((J + 1) * (J + 2) / 2 <= k) ++J;
    const int64_t I = k - J * (J + 1) / 2;
    entry = (uint32_t)(I | (J << 16));
    item = order_of(I, J, nT, g);
    corder[item] = entry;
  } else {
    item = k - nC;
    entry = r_tile | (uint32_t)(item % nRT) | ((uint32_t)(item / nRT) << 16);
  }
  if (!corder_r) return;
  // each XCD's share of the launch: its C tiles, then its R tiles
  int64_t pos = 0, c0 = 0, r0 = 0;
  for (int64_t x = 0; x < 8; ++x) {
    const int64_t size = n / 8 + (x < n % 8 ? 1 : 0), nr = nR / 8 + (x < nR % 8 ? 1 : 0);
    if (k < nC ? item < c0 + size - nr : item < r0 + nr) {
      corder_r[pos + (k < nC ? item - c0 : size - nr + item - r0)] = entry;
      return;
    }
    pos += size;
    c0 += size - nr;
    r0 += nr;
  }
}

}  // namespace

hipError_t launch_load(const LoadArgs& a, hipStream_t s) {
  const int64_t most = a.nh > a.Nap ? (a.nh > a.Nep ? a.nh : a.Nep) : (a.Nap > a.Nep ? a.Nap : a.Nep);
  const int64_t nq = (a.Na + a.crows - 1) / a.crows;
  const int64_t nb = 2 * a.Nep + (a.C ? c_strips(a.Nap) * nq : 0) + (most + kLT - 1) / kLT;
  k_load<<<dim3((unsigned)nb), kLT, 0, s>>>(a);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess || !a.C) return e;
  return launch_sum_slots(a.slots, a.Nap, nq, a.nC, s);
}

hipError_t launch_pack_xy(const PackArgs& a, hipStream_t s) {
  const int64_t nq = (a.Kp + a.rows - 1) / a.rows, nb = a.Mp + c_strips(a.Np) * nq;
  k_pack_xy<<<dim3((unsigned)nb), kLT, 0, s>>>(a);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return launch_sum_slots(a.slots, a.Np, nq, a.ny, s);
}

hipError_t launch_store(const StoreArgs& a, hipStream_t s) {
  const int64_t nb = (a.W ? a.Ne : 0) + (a.Pout ? a.Ne : 0) + (a.Cout ? a.Na : 0);
  if (nb == 0) return hipSuccess;
  k_store<<<dim3((unsigned)nb), kLT, 0, s>>>(a);
  return hipGetLastError();
}

hipError_t launch_order(int64_t Nep, int64_t Nap, int group, uint32_t* corder, uint32_t* corder_r,
                        hipStream_t s) {
  const int64_t nC = coreg_tiles(Nap), nR = corder_r ? next_r_tiles(Nep, Nap) : 0;
  k_order<<<dim3((unsigned)((nC + nR + kLT - 1) / kLT)), kLT, 0, s>>>(
      Nap / kPT, group, next_r_row_tiles(Nep), nR, kNextRTile, corder, corder_r);
  return hipGetLastError();
}

}  // namespace panda

// Weight gradients of the network adjoints: dW = sum over rows of X^T Y, where
// the adjoint kernels leave both row tables in global memory.
//
// The rows come in units (the rows of a group of walkers, or of one
// coordinate chunk of a walker).  Every unit's product is formed on the
// matrix cores from zero, reducing 32 rows per step (lane group g takes rows
// 8 g .. 8 g + 7 of a step), and added to the running sum of its slot; a slot
// takes a fixed sequence of units, so the result depends on nothing else that
// runs on the device.
//
// One wavefront owns a strip of NA x NB output tiles of one matrix and keeps
// its running sums in registers across the slot's units (adding every unit's
// product to a gradient slot in memory costs a read and a write of all
// parameters per unit).  A lane's columns are adjacent (column NA c + a of X,
// NB c + b of Y for tile a or b), so that one load serves all tiles of a row.
// Bound by the reads of the row tables: the blocks of a slot sit on one XCD,
// whose L2 then serves the strips that share rows.
#pragma once
#include <algorithm>

#include "mfma_gemm.h"
#include "pn_internal.h"

namespace pn {

constexpr int kMaxWMats = 4 * kMaxLayers + 5;

template <typename TN>
struct WMat {
  const TN* X;   // [rows][A]
  const TN* Y;   // [rows][B]
  int64_t out;   // offset of the [A][B] result in a slot
  int64_t xu, yu;  // elements from one unit to the next (chunks; the walkers' tables are contiguous)
  int A, B;
  int rows;      // rows per walker, or per chunk (0: those of the chunk's electrons)
  int strip0;    // first strip of this matrix among its launch
};

template <typename TN>
struct WMats {
  WMat<TN> m[kMaxWMats];
  int n;
};

// Units of the value-path adjoint: groups of wb walkers, taken s, s + slots, ...
struct UnitsOfWalkers {
  int64_t nw;
  int wb, slots;
  __device__ int64_t slot(int64_t s) const { return s; }
  __device__ bool keep(int64_t) const { return false; }  // one launch makes a slot
  __device__ int64_t count(int64_t s) const {
    const int64_t ng = (nw + wb - 1) / wb;
    return s < ng ? (ng - s + slots - 1) / slots : 0;
  }
  __device__ int group(int64_t s, int64_t k, int64_t& w0) const {  // first walker and their number
    w0 = (s + k * slots) * wb;
    return (int)min((int64_t)wb, nw - w0);
  }
  template <typename M>
  __device__ void rows(int64_t s, int64_t k, const M& m, int64_t& x0, int64_t& y0, int& n) const {
    int64_t w0;
    n = group(s, k, w0) * m.rows;
    x0 = w0 * m.rows * m.A;
    y0 = w0 * m.rows * m.B;
  }
};

// rows r0 .. r0 + 31 of a unit: NC adjacent columns per lane, zero past the
// unit's n rows
template <typename TN, int NC>
__device__ __forceinline__ void load_rows(const TN* p, int ld, int r0, int n, TN (&f)[NC][8]) {
  typedef TN vec __attribute__((ext_vector_type(NC)));
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    const int r = r0 + s;
    if constexpr (NC == 1) {
      const TN v = p[(int64_t)min(r, n - 1) * ld];
      f[0][s] = r < n ? v : TN(0);
    } else {
      const vec v = *reinterpret_cast<const vec*>(p + (int64_t)min(r, n - 1) * ld);
#pragma unroll
      for (int c = 0; c < NC; ++c) f[c][s] = r < n ? v[c] : TN(0);
    }
  }
}

// UNITS: slot() is the slot of local index s, keep() whether it already holds
// the sum of earlier units (else it is set), rows() where a unit's rows are.
template <typename TN, typename UNITS, int NA, int NB>
__global__ __launch_bounds__(256) void k_wgrad(WMats<TN> mats, UNITS units, int n_slots, int n_strips, int bps,
                                               TN* __restrict__ slots, int64_t slot_len) {
  typedef typename MfmaTile<TN>::acc_t acc_t;
  const int lane = threadIdx.x & 63, g = lane >> 4, c16 = lane & 15;
  // blocks b, b + 8, ... run on one XCD: a slot's bps blocks stay together
  const int64_t s = (int64_t)(blockIdx.x >> 3) / bps * 8 + (blockIdx.x & 7);
  const int strip = (int)((blockIdx.x >> 3) % bps) * 4 + ((int)threadIdx.x >> 6);
  if (s >= n_slots || strip >= n_strips) return;
  int k = 0;
  while (k + 1 < mats.n && strip >= mats.m[k + 1].strip0) ++k;
  const WMat<TN> m = mats.m[k];
  const int nbs = m.B / (16 * NB), local = strip - m.strip0;
  const int a0 = local / nbs * (16 * NA), b0 = local % nbs * (16 * NB);
  const TN* X = m.X + a0 + NA * c16;
  const TN* Y = m.Y + b0 + NB * c16;
  TN* out = slots + units.slot(s) * slot_len + m.out;
  const bool keep = units.keep(s);
  acc_t acc[NA][NB];
  const int64_t nu = units.count(s);
#pragma unroll
  for (int a = 0; a < NA; ++a)
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int v = 0; v < 4; ++v)
        acc[a][b][v] = keep ? out[(a0 + NA * MfmaTile<TN>::row_of(lane, v) + a) * m.B + b0 + NB * c16 + b] : TN(0);
  for (int64_t u = 0; u < nu; ++u) {
    int64_t x0, y0;
    int n;
    units.rows(s, u, m, x0, y0, n);
    const TN* xu = X + x0;
    const TN* yu = Y + y0;
    acc_t c[NA][NB];
#pragma unroll
    for (int a = 0; a < NA; ++a)
#pragma unroll
      for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int v = 0; v < 4; ++v) c[a][b][v] = TN(0);
    for (int r0 = 0; r0 < n; r0 += 32) {
      TN xf[NA][8], yf[NB][8];
      load_rows<TN, NA>(xu, m.A, r0 + g * 8, n, xf);
      load_rows<TN, NB>(yu, m.B, r0 + g * 8, n, yf);
#pragma unroll
      for (int a = 0; a < NA; ++a)
#pragma unroll
        for (int b = 0; b < NB; ++b) c[a][b] = MfmaChain<TN, 8>::run(xf[a], yf[b], c[a][b], false);
    }
    const bool set = u == 0 && !keep;
#pragma unroll
    for (int a = 0; a < NA; ++a)
#pragma unroll
      for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[a][b][v] = set ? c[a][b][v] : acc[a][b][v] + c[a][b][v];
  }
#pragma unroll
  for (int a = 0; a < NA; ++a)
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
      for (int b = 0; b < NB; ++b)
        out[(a0 + NA * MfmaTile<TN>::row_of(lane, v) + a) * m.B + b0 + NB * c16 + b] = acc[a][b][v];
}

// All matrices of `all`, one launch per strip shape.  FP32 strips are two
// tiles high where A allows it; FP64 accumulators take twice the registers.
template <typename TN, typename UNITS>
void launch_wgrad(hipStream_t s, const WMats<TN>& all, const UNITS& units, int n_slots, TN* slots,
                  int64_t slot_len) {
  auto launch = [&](auto na, auto nb) {
    constexpr int NA = decltype(na)::value, NB = decltype(nb)::value;
    WMats<TN> ms;
    ms.n = 0;
    int strips = 0;
    for (int k = 0; k < all.n; ++k) {
      WMat<TN> m = all.m[k];
      const int want_a = sizeof(TN) == 4 && m.A % 32 == 0 ? 2 : 1;
      const int want_b = m.B % 64 == 0 ? 4 : (m.B % 32 == 0 ? 2 : 1);
      if (want_a != NA || want_b != NB) continue;
      m.strip0 = strips;
      strips += (m.A / (16 * NA)) * (m.B / (16 * NB));
      ms.m[ms.n++] = m;
    }
    if (!ms.n) return;
    const int bps = (strips + 3) / 4;
    const unsigned grid = (unsigned)((n_slots + 7) / 8 * 8 * bps);
    hipLaunchKernelGGL((k_wgrad<TN, UNITS, NA, NB>), dim3(grid), dim3(256), 0, s, ms, units, n_slots, strips, bps,
                       slots, slot_len);
  };
  using one = std::integral_constant<int, 1>;
  using two = std::integral_constant<int, 2>;
  using four = std::integral_constant<int, 4>;
  launch(one(), one());
  launch(one(), two());
  launch(one(), four());
  if constexpr (sizeof(TN) == 4) {
    launch(two(), one());
    launch(two(), two());
    launch(two(), four());
  }
}

}  // namespace pn

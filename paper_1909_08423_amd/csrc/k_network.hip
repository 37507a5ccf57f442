// SchNet-style interaction layers and the Jastrow / backflow heads
// (Methods, "PauliNet extension of SchNet"; Results, J = eta(sum_i x_i),
// f_i = kappa(x_i)), in two passes:
//
//  value pass   (k_net_value)   one block per group of walkers; computes the
//               activations and stores what the tangent pass needs: h^(n)
//               values and the ssp'(u), ssp''(u) of every head hidden unit.
//
//  tangent pass (k_net_tangent, in k_tangent.hip) one block per (walker,
//               coordinate chunk), using what the value pass stored.
#include "gemm_lds.h"
#include "mfma_gemm.h"
#include "pn_internal.h"

namespace pn {
namespace {

// ---------------------------------------------------------------- values --
// Output epilogues of the value pass (each stores its tile itself, so a
// product, its bias, its activation and its stores take one phase).
// rows = walker-local electron rows (wl, i) or walkers (Jastrow head).

// h = x W_h + b_h: to LDS for the messages and to the table of the tangent pass
template <typename TN>
struct HOut {
  static constexpr bool kOwnStore = true;
  TN* H;
  int ld, rows, DZ;
  RowDiv N;
  const TN* b;
  TN* hval;       // h table at this layer and the block's first walker
  int64_t wstep;  // its walker stride
  template <typename A>
  __device__ void operator()(int, int, A&) const {}
  template <typename A>
  __device__ void store(int rt, int col, const A& c) const {
    const TN bc = b[col];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int row = (rt << 4) + MfmaTile<TN>::row_of((int)threadIdx.x & 63, v);
      if (row >= rows) continue;
      const TN y = c[v] + bc;
      H[row * ld + col] = y;
      hval[N.div(row) * wstep + N.mod(row) * DZ + col] = y;
    }
  }
};

// y = ssp(u), u = x W + b, with ssp'(u), ssp''(u) kept for the tangent pass:
// coef[walker][layer][2][N][DX] (Jastrow head: N = 1, rows are walkers)
template <typename TN>
struct HeadOut {
  static constexpr bool kOwnStore = true;
  TN* Y;
  int ld, rows, DX;
  RowDiv N;
  const TN* b;
  TN* coef;  // at this hidden layer and the block's first walker
  template <typename A>
  __device__ void operator()(int, int, A&) const {}
  template <typename A>
  __device__ void store(int rt, int col, const A& c) const {
    const TN bc = b[col];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int row = (rt << 4) + MfmaTile<TN>::row_of((int)threadIdx.x & 63, v);
      if (row >= rows) continue;
      const TN u = c[v] + bc;
      const TN sg = sigmoid_d(u);
      TN* k = coef + (int64_t)(N.div(row) * 4 * N.N + N.mod(row)) * DX + col;
      k[0] = sg;
      k[N.N * DX] = sg * (TN(1) - sg);
      Y[row * ld + col] = ssp(u);
    }
  }
};

// f = 1 + y W3 + b3, in FP64
template <typename TN>
struct FOut {
  static constexpr bool kOwnStore = true;
  int rows, M;
  const TN* b;
  double* f;  // [walker][N][M] at the block's first walker: rows are contiguous
  template <typename A>
  __device__ void operator()(int, int, A&) const {}
  template <typename A>
  __device__ void store(int rt, int col, const A& c) const {
    if (col >= M) return;
    const TN bc = b[col];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int row = (rt << 4) + MfmaTile<TN>::row_of((int)threadIdx.x & 63, v);
      if (row < rows) f[(int64_t)row * M + col] = 1.0 + (double)(c[v] + bc);
    }
  }
};

// The kernel's products are small (some tens of rows), so a block's time is
// its chain of barriers and load latencies, not a unit.  A layer therefore
// has three phases: the h product (bias and stores in its epilogue), the
// messages of all three channels, and the three channels' products (each
// output element stays with one lane, so they follow each other without a
// barrier); the two heads share four phases.  Eight partners' filter values
// are requested per step of a message sum.
// Measured per launch against the form with one phase per product, per
// bias and per activation and a block of 64 rows for every batch: 305 ->
// 192 us at 4096 walkers of a ten-electron atom (FP32), 680 -> 469 us at 8192
// walkers of a ten-atom chain (FP32), 46 -> 32 us at 512 walkers of H2 (FP64).
// ZCH: channels whose messages are in LDS together, 3, or 1 where a block of
// one walker does not hold three message tables (from 43 electrons of widths
// 128 / 64 in FP64): the channels then follow each other through one table,
// with the same sums in the same order.
template <typename TN, int ZCH>
__global__ __launch_bounds__(kThreads, sizeof(TN) == 4 ? 3 : 2) void k_net_value(
    Dims d, DevTables t, int64_t nw, int WPB, const TN* __restrict__ P, ParamLayout pl, int jets, const TN* __restrict__ filt,
    TN* __restrict__ hval, TN* __restrict__ kcoef, TN* __restrict__ ecoef, double* __restrict__ fval,
    double* __restrict__ jval, TN* __restrict__ xval) {
  extern __shared__ __align__(16) char smem[];
  const int N = d.N, DX = d.DX, DZ = d.DZ, M = d.M;
  const int64_t w0 = (int64_t)blockIdx.x * WPB;
  const int nwb = (int)min((int64_t)WPB, nw - w0);
  if (nwb <= 0) return;
  const int R = nwb * N;
  const int LDX = ld_pad<TN>(DX), LDZ = ld_pad<TN>(DZ), LDW = max(LDX, LDZ);
  int* pidx = reinterpret_cast<int*>(smem);                  // [N][N]
  TN* X = reinterpret_cast<TN*>(pidx + ((N * N + 3) & ~3));  // [WPB*N][LDX]
  TN* H = X + WPB * N * LDX;                                 // [WPB*N][LDW] h, later the backflow head
  TN* Z = H + WPB * N * LDW;                                 // [ZCH][WPB*N][LDZ] messages
  TN* E = Z + ZCH * WPB * N * LDZ;                           // [2][WPB][LDX] Jastrow head
  const int64_t fl_stride = (int64_t)jets * d.n_pairs * DZ;  // per layer
  const int64_t fw_stride = fl_stride * d.L;               // per walker
  // the tangent pass takes h walker by walker, the value-path adjoint layer by layer
  const int64_t h_walker = jets == 1 ? 1 : d.L, h_layer = jets == 1 ? nw : 1;
  const int ZS = WPB * N * LDZ;
  const int sx = log2_of(DX), sz = log2_of(DZ);
  const RowDiv rN(N);

  for (int q = threadIdx.x; q < N * N; q += blockDim.x) pidx[q] = t.pair_index[q];
  for (int q = threadIdx.x; q < R * DX; q += blockDim.x) X[(q >> sx) * LDX + (q & (DX - 1))] = P[pl.x0 + (q & (DX - 1))];
  __syncthreads();
  auto save_x = [&](int n) {  // x^(n), for the adjoints
    for (int q = threadIdx.x; q < R * DX; q += blockDim.x) {
      const int row = q >> sx, x = q & (DX - 1);
      xval[((n * nw + w0) * N) * DX + q] = X[row * LDX + x];
    }
  };
  for (int n = 0; n < d.L; ++n) {
    const ParamLayout::Layer& Lp = pl.layer[n];
    if (xval) save_x(n);
    gemm_mfma<TN, false, HOut<TN>>(X, LDX, R, DX, P + Lp.hW, DZ, H, LDW, false, false,
                                   HOut<TN>{H, LDW, R, DZ, rN, P + Lp.hb, hval + (w0 * h_walker + n * h_layer) * N * DZ,
                                            h_walker * N * DZ});
    __syncthreads();
    for (int ch0 = 0; ch0 < 3; ch0 += ZCH) {
      for (int q = threadIdx.x; q < ZCH * R * DZ; q += blockDim.x) {
        const int q3 = q >> sz, cz = ZCH == 1 ? 0 : (q3 >= R) + (q3 >= 2 * R), row = q3 - cz * R, z = q & (DZ - 1);
        const int ch = ch0 + cz;
        const int wl = rN.div(row), i = row - wl * N;
        const TN* fw = filt + (w0 + wl) * fw_stride + n * fl_stride + z;  // jet 0 = value
        TN acc = 0;
        if (ch < 2) {
          // electrons of this channel: same spin (ch 0) or opposite spin
          // (ch 1); j = i contributes w = 0
          const bool want_up = (ch == 0) == (i < d.n_up);
          const int j_lo = want_up ? 0 : d.n_up, j_hi = want_up ? d.n_up : N;
          const TN* hw = H + wl * N * LDW + z;
          for (int j = j_lo; j < j_hi; j += 8) {
            TN wv[8], hv[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) {
              const int jj = min(j + k, j_hi - 1);
              wv[k] = fw[max(pidx[i * N + jj], 0) * DZ];
              hv[k] = hw[jj * LDW];
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int k = 0; k < 8; ++k) acc += (j + k < j_hi && j + k != i) ? wv[k] * hv[k] : TN(0);
          }
        } else {
          for (int I = 0; I < d.NN; I += 4) {
            TN wv[4], yv[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
              const int II = min(I + k, d.NN - 1);
              wv[k] = fw[(d.n_ee + i * d.NN + II) * DZ];
              yv[k] = P[pl.Y + II * DZ + z];
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int k = 0; k < 4; ++k) acc += I + k < d.NN ? wv[k] * yv[k] : TN(0);
          }
        }
        Z[cz * ZS + row * LDZ + z] = acc;
      }
      __syncthreads();
      for (int cz = 0; cz < ZCH; ++cz)
        gemm_mfma<TN>(Z + cz * ZS, LDZ, R, DZ, P + Lp.gW[ch0 + cz], DX, X, LDX, true, false);
      __syncthreads();
    }
    // the three channels' biases, added once
    for (int q = threadIdx.x; q < R * DX; q += blockDim.x) {
      const int x = q & (DX - 1);
      X[(q >> sx) * LDX + x] += P[Lp.gb[0] + x] + P[Lp.gb[1] + x] + P[Lp.gb[2] + x];
    }
    __syncthreads();
  }
  if (xval) save_x(d.L);
  // ---- heads: Jastrow on s = sum_i x_i (rows = walkers), backflow per
  // electron row; the two advance together, one step of each per phase ----
  const bool do_j = !(d.flags & PN_NET_NO_JASTROW), do_k = !(d.flags & PN_NET_NO_BACKFLOW);
  TN* S = E;                // [WPB][LDX]
  TN* U = E + WPB * LDX;    // [WPB][LDX]
  TN* ec = ecoef + w0 * 4 * DX;
  TN* kc = kcoef + w0 * 4 * N * DX;
  if (do_j) {
    for (int q = threadIdx.x; q < nwb * DX; q += blockDim.x) {
      const int wl = q >> sx, x = q & (DX - 1);
      TN s = 0;
      for (int i = 0; i < N; ++i) s += X[(wl * N + i) * LDX + x];
      S[wl * LDX + x] = s;
    }
  } else {
    for (int wl = threadIdx.x; wl < nwb; wl += blockDim.x) jval[w0 + wl] = 0.0;
  }
  if (do_k)
    gemm_mfma<TN, false, HeadOut<TN>>(X, LDX, R, DX, P + pl.kW1, DX, H, LDW, false, false,
                                      HeadOut<TN>{H, LDW, R, DX, rN, P + pl.kb1, kc});
  else
    for (int q = threadIdx.x; q < R * M; q += blockDim.x) fval[w0 * N * M + q] = 1.0;
  __syncthreads();
  if (do_j)
    gemm_mfma<TN, false, HeadOut<TN>>(S, LDX, nwb, DX, P + pl.eW1, DX, U, LDX, false, false,
                                      HeadOut<TN>{U, LDX, nwb, DX, RowDiv(1), P + pl.eb1, ec});
  if (do_k)
    gemm_mfma<TN, false, HeadOut<TN>>(H, LDW, R, DX, P + pl.kW2, DX, X, LDX, false, false,
                                      HeadOut<TN>{X, LDX, R, DX, rN, P + pl.kb2, kc + 2 * N * DX});
  __syncthreads();
  if (do_j)
    gemm_mfma<TN, false, HeadOut<TN>>(U, LDX, nwb, DX, P + pl.eW2, DX, S, LDX, false, false,
                                      HeadOut<TN>{S, LDX, nwb, DX, RowDiv(1), P + pl.eb2, ec + 2 * DX});
  if (do_k)
    gemm_mfma_cols<TN, FOut<TN>>(X, LDX, R, DX, P + pl.kW3, M, H, LDW, false, false,
                                 FOut<TN>{R, M, P + pl.kb3, fval + w0 * N * M});
  if (!do_j) return;
  __syncthreads();
  for (int wl = threadIdx.x; wl < nwb; wl += blockDim.x) {
    TN acc = P[pl.eb3];
    for (int x = 0; x < DX; x += 16) {  // DX is a multiple of 16; the sum runs in order of x
      TN sv[16], wv[16];
#pragma unroll
      for (int k = 0; k < 16; ++k) {
        sv[k] = S[wl * LDX + x + k];
        wv[k] = P[pl.eW3 + x + k];
      }
#pragma unroll
      for (int k = 0; k < 16; ++k) acc += sv[k] * wv[k];
    }
    jval[w0 + wl] = (double)acc;
  }
}

}  // namespace

// LDS of the value pass: three message tables, or one where a single walker's
// block does not hold them.
template <typename TN>
static size_t value_lds_channels(const Dims& d, int wpb, int channels) {
  const int LDX = ld_pad<TN>(d.DX), LDZ = ld_pad<TN>(d.DZ), LDW = std::max(LDX, LDZ);
  return (size_t)((d.N * d.N + 3) & ~3) * sizeof(int) +
         ((size_t)wpb * d.N * (LDX + LDW + channels * LDZ) + 2 * (size_t)wpb * LDX) * sizeof(TN);
}

template <typename TN>
size_t value_lds_bytes(const Dims& d, int wpb) {
  const size_t three = value_lds_channels<TN>(d, wpb, 3);
  return wpb > 1 || three <= 160 * 1024 ? three : value_lds_channels<TN>(d, wpb, 1);
}

template <typename TN>
void launch_net_value(const pn_ctx* c, hipStream_t s, int64_t nw, const TN* P, char* ws, const WsLayout& L) {
  const Dims& d = c->d;
  int64_t nb = (nw + L.wpb_value - 1) / L.wpb_value;
  auto kern = L.lds_value == value_lds_channels<TN>(d, L.wpb_value, 3) ? &k_net_value<TN, 3> : &k_net_value<TN, 1>;
  if (L.lds_value > 65536)
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)L.lds_value);
  hipLaunchKernelGGL(kern, dim3((unsigned)nb), dim3(kThreads), L.lds_value, s, d, c->t, nw, L.wpb_value,
                     P, c->pl, L.jets, reinterpret_cast<const TN*>(ws + L.filt), reinterpret_cast<TN*>(ws + L.hval),
                     reinterpret_cast<TN*>(ws + L.kcoef), reinterpret_cast<TN*>(ws + L.ecoef),
                     reinterpret_cast<double*>(ws + L.fval), reinterpret_cast<double*>(ws + L.jval),
                     L.xval ? reinterpret_cast<TN*>(ws + L.xval) : nullptr);
}

template void launch_net_value<double>(const pn_ctx*, hipStream_t, int64_t, const double*, char*, const WsLayout&);
template void launch_net_value<float>(const pn_ctx*, hipStream_t, int64_t, const float*, char*, const WsLayout&);
template size_t value_lds_bytes<double>(const Dims&, int);
template size_t value_lds_bytes<float>(const Dims&, int);

}  // namespace pn

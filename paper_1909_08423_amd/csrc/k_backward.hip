// Value-path adjoint: grad_theta += sum_w ct_w d ln|psi_w| / d theta.
//
// The Hermitian gradient estimator (Methods, eq. "trainig") needs only the
// parameter gradient of ln|psi| weighted per walker by 2 (E_loc - L) / B,
// which is this adjoint with ct_w = that weight.  ln|psi| = gamma + J +
// ln|Psi_d| depends on theta through J and through the backflow f inside
// the determinants:
//   d ln|Psi_d| / d A_p^s[k][i] = w_p (A_p^s)^{-1}[i][k],  w_p = c_p D_p / Psi_d
//   A_p^s[k][i] = phi_mu(r_i) f_{i mu},  mu = mu_p^s(k)
// so  d ln|psi| / d f_{i mu} = phi_mu(r_i) sum_p w_p sum_{k: mu_p(k) = mu} G_p[i][k].
// From there the reverse sweep runs through kappa, eta, the interaction
// layers (messages, h and the three g) and finally the filter networks.
//
// Kernels (the forward values come from the value pass, run just before):
//  k_bwd_net     groups of WB walkers: the reverse sweep.  Leaves both row
//                tables of every weight gradient, the sums of the bias-like
//                parameters of its group, and the filter outputs' cotangents.
//  k_wgrad       (wgrad.h) weight gradients from the row tables, k_wgrad_small
//                those of the last backflow layer and the bias-like ones; each
//                into the gradient slot of its group (slot = group mod 512).
//  k_bwd_filter  per (layer, channel) and a fixed set of blocks striding
//                over (walker, pair) rows; recomputes features and the
//                hidden layer, accumulates the filter gradients in registers.
//  k_bwd_reduce  sums the slots in a fixed order into the FP64 gradient.
// The fixed groups and slot order make the result independent of anything
// else running on the device.
#include "adj_util.h"
#include "gemm_lds.h"
#include "mfma_gemm.h"
#include "pn_internal.h"
#include "wgrad.h"

namespace pn {
namespace {

constexpr int kSlotsNet = 512;     // gradient slots of the network weights, at most
constexpr int kSlotsFilter = 256;  // blocks per (layer, channel) of k_bwd_filter, at most
constexpr int kFiltRows = 32;      // (walker, pair) rows per tile of k_bwd_filter, at most

// What k_bwd_net leaves behind for the weight gradients ([walker][row]
// tables, contiguous over the walkers of a launch) and, per group of walkers,
// the sums of the parameters that are no matrix: offsets into one block.
template <typename TN>
struct NetOps {
  TN *z, *cx, *ch;             // [L][3][nw N][DZ] messages, [L][nw N][DX] cotangents of x^(n+1), [L][nw N][DZ] of h
  TN *a1, *c2, *c1, *a2, *cf;  // backflow head: [nw N][DX] activations and cotangents, [nw N][M] cotangent of f
  TN *s, *e1, *ec1, *ec2;      // Jastrow head: [nw][DX]
  TN* small;                   // [groups][SmallSums::total]
};

struct SmallSums {
  int eW3, eb3, eb2, eb1, kb3, kb2, kb1, x0, layer, gb, hb, Y, step, total;  // layer n at layer + n step + gb | hb | Y
  __host__ __device__ explicit SmallSums(const Dims& d) {
    int o = 0;
    auto take = [&](int n) {
      const int at = o;
      o += n;
      return at;
    };
    eW3 = take(d.DX), eb3 = take(1), eb2 = take(d.DX), eb1 = take(d.DX);
    kb3 = take(d.M), kb2 = take(d.DX), kb1 = take(d.DX), x0 = take(d.DX);
    layer = o;
    gb = 0, hb = d.DX, Y = hb + d.DZ, step = Y + d.NN * d.DZ;
    total = layer + d.L * step;
  }
};

// out[b] = sum_r Y[r][b]
template <typename TN>
__device__ __forceinline__ void colsum(const TN* Y, int ldy, int B, int rows, TN* out) {
  for (int b = threadIdx.x; b < B; b += blockDim.x) {
    TN s = 0;
    for (int r = 0; r < rows; ++r) s += Y[r * ldy + b];
    out[b] = s;
  }
}

// The sweep's products are small (a group has some tens of rows), so its time
// is latency: of the barriers, of the filter values (each read once, for the
// message and for the cotangent of h together, eight partners at a time), and
// of the index arithmetic.  The weight gradients, which would read and write
// every parameter of a slot once per group, are left to k_wgrad.
// Measured per launch (FP32): 14.2 -> 2.9 ms (+ 0.5 ms of weight gradients) at
// 2048 walkers of the 30-electron diatomic, 1.44 -> 0.57 ms at 4096 walkers of
// a ten-electron atom, against one kernel that added every group's weight
// gradients to slots in memory and took the channels one after the other.
template <typename TN, int NT>
__global__ __launch_bounds__(NT, 512 / NT) void k_bwd_net(Dims d, DevTables t, int64_t nw, int WB,
                                                          const TN* __restrict__ P, ParamLayout pl,
                                                          const TN* __restrict__ xval, const TN* hval,
                                                          int jets, const TN* __restrict__ filt,
                                                          const double* __restrict__ phi,
                                                          const double* __restrict__ ginv,
                                                          const double* __restrict__ wdet,
                                                          const double* __restrict__ ct_logabs, TN* __restrict__ ctw,
                                                          const double* __restrict__ ctfpart, int n_chunks,
                                                          const TN* __restrict__ cthv, const TN* __restrict__ ctkc,
                                                          const TN* __restrict__ ctec, NetOps<TN> op,
                                                          TN* __restrict__ arena, int64_t arena_elems) {
  extern __shared__ __align__(16) char smem[];
  const int N = d.N, DX = d.DX, DZ = d.DZ, M = d.M, L = d.L, NU = d.n_up, P2 = 2 * d.P;
  const int LDX = ld_pad<TN>(DX), LDZ = ld_pad<TN>(DZ), LDM = ld_pad<TN>((M + 15) & ~15);
  const int RW = WB * N;
  const int sx = log2_of(DX), sz = log2_of(DZ);
  const RowDiv rN(N);
  const SmallSums sm(d);
  int* pidx = reinterpret_cast<int*>(smem);                              // [N][N]
  unsigned short* pij = reinterpret_cast<unsigned short*>(pidx + ((N * N + 3) & ~3));  // [n_ee] i + 256 j
  signed char* inv = reinterpret_cast<signed char*>(pij + ((d.n_ee + 7) & ~7));  // [P][2][M] slot of an orbital
  TN* cw = reinterpret_cast<TN*>(inv + ((P2 * M + 15) & ~15));           // [WB]
  TN* CX = cw + ((WB + 3) & ~3);                                         // [RW][LDX]
  // union region (heads, then layers): in LDS, or in this block's part of a
  // global arena when it does not fit beside CX
  TN* UN = arena ? arena + (size_t)blockIdx.x * arena_elems : CX + RW * LDX;
  // heads view
  TN* X = UN;                  // [RW][LDX] x^(L), then the second pre-activation and its product
  TN* A = X + RW * LDX;        // [RW][LDX] first pre-activation
  TN* B = A + RW * LDX;        // [RW][LDX] first activation, then the second's cotangent
  TN* CF = B + RW * LDX;       // [RW][LDM] cotangent of f
  TN* Sv = CF + RW * LDM;      // [WB][LDX] sum_i x_i
  TN* U1 = Sv + WB * LDX;      // pre-activations of the Jastrow head
  TN* U2 = U1 + WB * LDX;
  TN* Y1 = U2 + WB * LDX;
  TN* C1 = Y1 + WB * LDX;      // cotangents
  TN* C2 = C1 + WB * LDX;
  // layers view
  TN* H = UN;                  // [RW][LDZ]
  TN* CZ = H + RW * LDZ;       // [3][RW][LDZ]
  TN* CH = CZ + 3 * RW * LDZ;  // [RW][LDZ]
  const int64_t fl_stride = (int64_t)jets * d.n_pairs * DZ;
  const int64_t h_walker = jets == 1 ? 1 : L, h_layer = jets == 1 ? nw : 1;  // h table, in units of a walker's layer
  const int64_t ng = (nw + WB - 1) / WB;
  const int n_same = (d.n_up * (d.n_up - 1) + d.n_dn * (d.n_dn - 1)) / 2;
  const TN jas = (d.flags & PN_NET_NO_JASTROW) ? TN(0) : TN(1);  // a removed Jastrow factor gets no cotangent
  for (int q = threadIdx.x; q < N * N; q += blockDim.x) pidx[q] = t.pair_index[q];
  for (int q = threadIdx.x; q < d.n_ee; q += blockDim.x)
    pij[q] = (unsigned short)(t.pair_ij[2 * q] + 256 * t.pair_ij[2 * q + 1]);
  for (int q = threadIdx.x; q < P2 * M; q += blockDim.x) inv[q] = -1;
  __syncthreads();
  for (int q = threadIdx.x; q < d.P * N; q += blockDim.x) {
    const int p = q / N, k = q % N;
    const bool up = k < NU;
    inv[(2 * p + !up) * M + (up ? t.det_up[p * d.n_up + k] : t.det_dn[p * d.n_dn + k - NU])] =
        (signed char)(up ? k : k - NU);
  }
  for (int64_t grp = blockIdx.x; grp < ng; grp += gridDim.x) {
    const int64_t w0 = grp * WB, row0 = w0 * N;
    const int nwb = (int)min((int64_t)WB, nw - w0);
    const int R = nwb * N;
    TN* small = op.small + grp * sm.total;
    __syncthreads();
    for (int q = threadIdx.x; q < nwb; q += blockDim.x) cw[q] = (TN)ct_logabs[w0 + q];
    const TN* xl = xval + ((int64_t)L * nw * N + row0) * DX;
    for (int q = threadIdx.x; q < R * DX; q += blockDim.x) X[(q >> sx) * LDX + (q & (DX - 1))] = xl[q];
    __syncthreads();
    // ---- cotangent of the backflow, from the determinants; the sum of the
    // embeddings; the first products of both heads ----
    const int gsz = d.n_up * d.n_up + d.n_dn * d.n_dn;
    for (int q = threadIdx.x; q < R * LDM; q += blockDim.x) {
      const int row = q / LDM, mu = q - row * LDM, wl = rN.div(row), i = row - wl * N;
      const int64_t w = w0 + wl;
      TN cf = 0;
      if (mu < M && !(d.flags & PN_NET_NO_BACKFLOW)) {  // f = 1 does not depend on theta
        if (ctfpart) {
          // full adjoint: the determinant part supplies the cotangent of f
          // (its ln|psi| share included), summed over the coordinate chunks
          double v = 0.0;
          for (int c = 0; c < n_chunks; ++c) v += ctfpart[((w * n_chunks + c) * N + i) * M + mu];
          cf = (TN)v;
        } else {
          const bool up = i < NU;
          const int n = up ? d.n_up : d.n_dn, ii = up ? i : i - NU;
          const double* G = ginv + w * d.P * gsz + (up ? 0 : d.n_up * d.n_up) + ii * n;
          const double* wd = wdet + w * d.P;
          for (int p = 0; p < d.P; p += 4) {
            double gv[4], wv[4];
            int kk[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
              const int pu = min(p + u, d.P - 1);
              kk[u] = p + u < d.P ? inv[(2 * pu + !up) * M + mu] : -1;
              gv[u] = G[(int64_t)pu * gsz + max(kk[u], 0)];
              wv[u] = wd[pu];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
              if (kk[u] >= 0) cf += (TN)(wv[u] * gv[u]);
          }
          cf *= (TN)(phi[((w * N + i) * M + mu) * 7]) * cw[wl];
        }
      }
      CF[q] = cf;
      if (mu < M) op.cf[(row0 + row) * M + mu] = cf;
    }
    for (int q = threadIdx.x; q < nwb * DX; q += blockDim.x) {
      const int wl = q >> sx, x = q & (DX - 1);
      TN s = 0;
      for (int i = 0; i < N; ++i) s += X[(wl * N + i) * LDX + x];
      Sv[wl * LDX + x] = s;
      op.s[w0 * DX + q] = s;
    }
    gemm_mfma<TN>(X, LDX, R, DX, P + pl.kW1, DX, A, LDX, false, false);
    __syncthreads();
    gemm_mfma<TN>(Sv, LDX, nwb, DX, P + pl.eW1, DX, U1, LDX, false, false);
    for (int q = threadIdx.x; q < R * DX; q += blockDim.x) {
      const int o = (q >> sx) * LDX + (q & (DX - 1));
      const TN u1 = A[o] + P[pl.kb1 + (q & (DX - 1))];
      const TN y = ssp(u1);
      A[o] = u1;
      B[o] = y;
      op.a1[row0 * DX + q] = y;
    }
    colsum<TN>(CF, LDM, M, R, small + sm.kb3);
    __syncthreads();
    for (int q = threadIdx.x; q < nwb * DX; q += blockDim.x) {
      const int o = (q >> sx) * LDX + (q & (DX - 1));
      const TN u1 = U1[o] + P[pl.eb1 + (q & (DX - 1))];
      const TN y = ssp(u1);
      U1[o] = u1;
      Y1[o] = y;
      op.e1[w0 * DX + q] = y;
    }
    gemm_mfma<TN>(B, LDX, R, DX, P + pl.kW2, DX, X, LDX, false, false);
    __syncthreads();
    gemm_mfma<TN>(Y1, LDX, nwb, DX, P + pl.eW2, DX, U2, LDX, false, false);
    // d/d y2 = CF W3^T (W3 is [DX][M]), eight rows per read of W3; then d/d u2
    for (int q = threadIdx.x; q < ((R + 7) >> 3) * DX; q += blockDim.x) {
      const int x = q & (DX - 1), r0 = (q >> sx) * 8, nr = min(8, R - r0);
      const TN* w3 = P + pl.kW3 + x * M;
      TN sv[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) sv[k] = 0;
      for (int mu = 0; mu < M; ++mu) {
        const TN w = w3[mu];
#pragma unroll
        for (int k = 0; k < 8; ++k) sv[k] += CF[min(r0 + k, R - 1) * LDM + mu] * w;
      }
      const TN b2 = P[pl.kb2 + x];
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        if (k >= nr) break;
        const int r = r0 + k;
        const TN u2 = X[r * LDX + x] + b2;
        TN c2 = sv[k] * sig(u2);  // d/d u2
        if (ctkc) {
          const int wl = rN.div(r);
          const TN* ck = ctkc + ((w0 + wl) * 4 + 2) * N * DX + (r - wl * N) * DX + x;
          c2 += ck[0] * ssp2(u2) + ck[N * DX] * ssp3(u2);
        }
        B[r * LDX + x] = c2;
        op.a2[(row0 + r) * DX + x] = ssp(u2);
        op.c2[(row0 + r) * DX + x] = c2;
      }
    }
    __syncthreads();
    for (int x = threadIdx.x; x < DX; x += blockDim.x) {
      TN s = 0;
      const TN b2 = P[pl.eb2 + x], w3 = P[pl.eW3 + x];
      for (int r = 0; r < nwb; ++r) {
        // d/d u2 = cJ * W3[x] * ssp'(u2)
        const TN u2 = U2[r * LDX + x] + b2;
        TN c2 = jas * cw[r] * w3 * sig(u2);
        if (ctec) {  // tangent-pass cotangents of ssp'(u2), ssp''(u2)
          const TN* ce = ctec + ((w0 + r) * 2 + 1) * 2 * DX;
          c2 += ce[x] * ssp2(u2) + ce[DX + x] * ssp3(u2);
        }
        C2[r * LDX + x] = c2;
        op.ec2[(w0 + r) * DX + x] = c2;
        s += jas * ssp(u2) * cw[r];
      }
      small[sm.eW3 + x] = s;
    }
    if (threadIdx.x == 0) {
      TN s = 0;
      for (int r = 0; r < nwb; ++r) s += jas * cw[r];
      small[sm.eb3] = s;
    }
    gemm_mfma_wt<TN>(B, LDX, R, DX, P + pl.kW2, DX, X, LDX, false);
    colsum<TN>(B, LDX, DX, R, small + sm.kb2);
    __syncthreads();
    gemm_mfma_wt<TN>(C2, LDX, nwb, DX, P + pl.eW2, DX, C1, LDX, false);
    colsum<TN>(C2, LDX, DX, nwb, small + sm.eb2);
    for (int q = threadIdx.x; q < R * DX; q += blockDim.x) {
      const int r = q >> sx, x = q & (DX - 1);
      const TN u1 = A[r * LDX + x];
      TN c1 = X[r * LDX + x] * sig(u1);  // d/d u1
      if (ctkc) {
        const int wl = rN.div(r);
        const TN* ck = ctkc + (w0 + wl) * 4 * N * DX + (r - wl * N) * DX + x;
        c1 += ck[0] * ssp2(u1) + ck[N * DX] * ssp3(u1);
      }
      X[r * LDX + x] = c1;
      op.c1[row0 * DX + q] = c1;
    }
    __syncthreads();
    for (int q = threadIdx.x; q < nwb * DX; q += blockDim.x) {
      const int r = q >> sx, x = q & (DX - 1);
      const TN u1 = U1[r * LDX + x];
      TN c1 = C1[r * LDX + x] * sig(u1);
      if (ctec) {
        const TN* ce = ctec + (w0 + r) * 4 * DX;
        c1 += ce[x] * ssp2(u1) + ce[DX + x] * ssp3(u1);
      }
      C1[r * LDX + x] = c1;
      op.ec1[w0 * DX + q] = c1;
    }
    colsum<TN>(X, LDX, DX, R, small + sm.kb1);
    __syncthreads();
    gemm_mfma_wt<TN>(C1, LDX, nwb, DX, P + pl.eW1, DX, C2, LDX, false);  // d/d s
    colsum<TN>(C1, LDX, DX, nwb, small + sm.eb1);
    __syncthreads();
    for (int q = threadIdx.x; q < R * DX; q += blockDim.x) {
      const int row = q >> sx, x = q & (DX - 1);
      CX[row * LDX + x] = C2[rN.div(row) * LDX + x];
    }
    __syncthreads();
    gemm_mfma_wt<TN>(X, LDX, R, DX, P + pl.kW1, DX, CX, LDX, true);
    __syncthreads();
    // ---- interaction layers, last to first ----
    for (int n = L - 1; n >= 0; --n) {
      const ParamLayout::Layer& Lp = pl.layer[n];
      TN* sml = small + sm.layer + n * sm.step;
      for (int q = threadIdx.x; q < R * DZ; q += blockDim.x) {
        const int row = q >> sz, z = q & (DZ - 1), wl = rN.div(row);
        H[row * LDZ + z] = hval[(((w0 + wl) * h_walker + n * h_layer) * N + (row - wl * N)) * DZ + z];
        // the tangent pass's cotangent of the h values seeds the h adjoint
        CH[row * LDZ + z] = cthv ? cthv[(((w0 + wl) * L + n) * N + (row - wl * N)) * DZ + z] : TN(0);
      }
      {
        TN* oc = op.cx + ((int64_t)n * nw * N + row0) * DX;
        for (int q = threadIdx.x; q < R * DX; q += blockDim.x) oc[q] = CX[(q >> sx) * LDX + (q & (DX - 1))];
      }
      colsum<TN>(CX, LDX, DX, R, sml + sm.gb);  // the same for the three channels' biases
      for (int ch = 0; ch < 3; ++ch)            // d/d z
        gemm_mfma_wt<TN>(CX, LDX, R, DX, P + Lp.gW[ch], DZ, CZ + ch * RW * LDZ, LDZ, false);
      __syncthreads();
      // messages z_i = sum_j w_ij h_j (recomputed for the weight gradients)
      // and d/d h_i += sum_j w_ij d/d z_j, from the same filter values
      TN* oz = op.z + ((int64_t)n * 3 * nw * N + row0) * DZ;
      const int64_t oz_ch = nw * N * DZ;
      for (int q = threadIdx.x; q < R * DZ; q += blockDim.x) {
        const int row = q >> sz, z = q & (DZ - 1), wl = rN.div(row), i = row - wl * N;
        const TN* fv = filt + (w0 + wl) * fl_stride * L + n * fl_stride + z;
        TN chv = CH[row * LDZ + z];
        for (int ch = 0; ch < 2; ++ch) {
          const bool want_up = (ch == 0) == (i < NU);
          const int j_lo = want_up ? 0 : NU, j_hi = want_up ? NU : N;
          const TN* hz = H + wl * N * LDZ + z;
          const TN* cz = CZ + (ch * RW + wl * N) * LDZ + z;
          TN acc = 0, cac = 0;
          for (int j = j_lo; j < j_hi; j += 8) {
            TN wv[8], hv[8], cv[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) {
              const int jj = min(j + k, j_hi - 1);
              wv[k] = fv[max(pidx[i * N + jj], 0) * DZ];
              hv[k] = hz[jj * LDZ];
              cv[k] = cz[jj * LDZ];
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int k = 0; k < 8; ++k) {
              const bool on = j + k < j_hi && j + k != i;  // else both terms are exact zeros
              const TN w = on ? wv[k] : TN(0);
              acc += w * (on ? hv[k] : TN(0));
              cac += w * (on ? cv[k] : TN(0));
            }
          }
          oz[ch * oz_ch + q] = acc;
          chv += cac;
        }
        CH[row * LDZ + z] = chv;
        TN acc = 0;
        for (int I = 0; I < d.NN; ++I) acc += fv[(d.n_ee + i * d.NN + I) * DZ] * P[pl.Y + I * DZ + z];
        oz[2 * oz_ch + q] = acc;
      }
      // cotangents of the filter outputs
      for (int wl = 0; wl < nwb; ++wl) {
        TN* cwp = ctw + ((w0 + wl) * L + n) * (int64_t)d.n_pairs * DZ;
        const TN* hz = H + wl * N * LDZ;
        for (int q = threadIdx.x; q < d.n_ee * DZ; q += blockDim.x) {
          const int p = q >> sz, z = q & (DZ - 1), i = pij[p] & 255, j = pij[p] >> 8;
          const TN* cz = CZ + ((p < n_same ? 0 : RW) + wl * N) * LDZ + z;
          const TN v = cz[i * LDZ] * hz[j * LDZ + z] + cz[j * LDZ] * hz[i * LDZ + z];
          cwp[q] = v;
        }
        const TN* cn = CZ + (2 * RW + wl * N) * LDZ;
        for (int q = threadIdx.x; q < N * d.NN * DZ; q += blockDim.x) {
          const int iI = q >> sz, z = q & (DZ - 1), i = iI / d.NN, I = iI - i * d.NN;
          cwp[d.n_ee * DZ + q] = cn[i * LDZ + z] * P[pl.Y + I * DZ + z];
        }
      }
      // d/d Y_I = sum over layers and electrons of w_iI d/d z_i (this layer's share)
      for (int q = threadIdx.x; q < d.NN * DZ; q += blockDim.x) {
        const int I = q >> sz, z = q & (DZ - 1);
        TN s = 0;
        for (int r0 = 0; r0 < R; r0 += 8) {
          TN fv[8], cv[8];
#pragma unroll
          for (int k = 0; k < 8; ++k) {
            const int row = min(r0 + k, R - 1), wl = rN.div(row), i = row - wl * N;
            fv[k] = filt[((w0 + wl) * L + n) * fl_stride + (d.n_ee + i * d.NN + I) * DZ + z];
            cv[k] = CZ[(2 * RW + row) * LDZ + z];
          }
#pragma unroll
          for (int k = 0; k < 8; ++k)
            if (r0 + k < R) s += fv[k] * cv[k];
        }
        sml[sm.Y + q] = s;
      }
      __syncthreads();
      // h = x W_h + b_h
      {
        TN* oc = op.ch + ((int64_t)n * nw * N + row0) * DZ;
        for (int q = threadIdx.x; q < R * DZ; q += blockDim.x) oc[q] = CH[(q >> sz) * LDZ + (q & (DZ - 1))];
      }
      colsum<TN>(CH, LDZ, DZ, R, sml + sm.hb);
      gemm_mfma_wt<TN>(CH, LDZ, R, DZ, P + Lp.hW, DX, CX, LDX, true);
      __syncthreads();
    }
    // x^(0) = x0 for every electron
    colsum<TN>(CX, LDX, DX, R, small + sm.x0);
  }
}

// The parameters that are no weight matrix of k_wgrad, per (slot, parameter):
// the last backflow layer W3 [DX][M] (M is no tile width: a thread per entry,
// the rows of a group in order), then the groups' sums.
template <typename TN>
__global__ __launch_bounds__(kThreads) void k_wgrad_small(Dims d, ParamLayout pl, UnitsOfWalkers units,
                                                          const TN* __restrict__ a2, const TN* __restrict__ cf,
                                                          const TN* __restrict__ small, TN* __restrict__ slots,
                                                          int64_t slot_len) {
  const SmallSums sm(d);
  const int64_t s = blockIdx.y;
  const int q = blockIdx.x * blockDim.x + threadIdx.x, n3 = d.DX * d.M;
  TN* out = slots + s * slot_len;
  const int64_t nu = units.count(s);
  if (q < n3) {
    const int a = q / d.M, b = q - a * d.M;
    TN acc = 0;
    for (int64_t u = 0; u < nu; ++u) {
      int64_t w0;
      const int n = units.group(s, u, w0) * d.N;
      const TN* x = a2 + w0 * d.N * d.DX + a;
      const TN* y = cf + w0 * d.N * d.M + b;
      TN v = 0;
      for (int r0 = 0; r0 < n; r0 += 8) {
        TN xv[8], yv[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          const int r = min(r0 + k, n - 1);
          xv[k] = x[r * d.DX];
          yv[k] = y[r * d.M];
        }
#pragma unroll
        for (int k = 0; k < 8; ++k)
          if (r0 + k < n) v += xv[k] * yv[k];
      }
      acc = u == 0 ? v : acc + v;
    }
    out[pl.kW3 + q] = acc;
    return;
  }
  const int e = q - n3;
  if (e >= sm.total) return;
  auto sum = [&](int at) {
    TN acc = 0;
    for (int64_t u = 0; u < nu; ++u) {
      const TN v = small[(s + u * units.slots) * sm.total + at];
      acc = u == 0 ? v : acc + v;
    }
    return acc;
  };
  if (e < sm.layer) {
    const int at[8] = {sm.eW3, sm.eb3, sm.eb2, sm.eb1, sm.kb3, sm.kb2, sm.kb1, sm.x0};
    const int64_t to[8] = {pl.eW3, pl.eb3, pl.eb2, pl.eb1, pl.kb3, pl.kb2, pl.kb1, pl.x0};
#pragma unroll
    for (int k = 7; k >= 0; --k)
      if (e >= at[k]) {
        out[to[k] + e - at[k]] = sum(e);
        break;
      }
    return;
  }
  const int n = (e - sm.layer) / sm.step, o = (e - sm.layer) % sm.step;
  if (o < sm.hb) {
    const TN v = sum(e);
    for (int ch = 0; ch < 3; ++ch) out[pl.layer[n].gb[ch] + o] = v;
  } else if (o < sm.Y) {
    out[pl.layer[n].hb + o - sm.hb] = sum(e);
  } else if (n == 0) {  // one embedding for all layers: summed layer by layer, last to first
    TN acc = 0;
    for (int64_t u = 0; u < nu; ++u)
      for (int l = d.L - 1; l >= 0; --l) {
        const TN v = small[(s + u * units.slots) * sm.total + sm.layer + l * sm.step + o];
        acc = u == 0 && l == d.L - 1 ? v : acc + v;
      }
    out[pl.Y + o - sm.Y] = acc;
  }
}

// JETS: the cotangents also reach the radial derivatives (w'/d and w'') of
// the filter outputs (full adjoint).  With the jets of the hidden layer
//   u = e W1 + b1, ud = (e'/d) W1, u2 = e'' W1,
//   a0 = ssp(u), a1 = s ud, a2 = s u2 + s' (d ud)^2   (s = ssp'(u), s' = ssp''(u))
//   w = a0 W2 + b2, w'/d = a1 W2, w'' = a2 W2
// the reverse is
//   ct a_k = ct w_k W2^T,  dW2 += sum_k a_k^T ct w_k,  db2 += ct w
//   ct u  = ct a0 s + ct a1 s' ud + ct a2 (s' u2 + s'' (d ud)^2)
//   ct ud = ct a1 s + 2 ct a2 s' d (d ud),   ct u2 = ct a2 s
//   dW1 += e^T ct u + (e'/d)^T ct ud + e''^T ct u2,  db1 += ct u.
// A block walks row tiles of PT (walker, pair) rows with its weight slabs in
// registers.  Per tile: features and filter cotangents to LDS, then (one wave
// per 16 x 16 tile of the hidden layer) both products and the activation's
// reverse in the accumulators, then the weight gradients.  The next tile's
// distances are computed, and its cotangents requested, one tile ahead.  Bound
// by the latency of those steps (two blocks per CU), not by a unit.
// Measured per launch: 5.8 -> 2.8 ms at 2048 walkers of the 30-electron
// diatomic and 0.57 -> 0.22 ms at 4096 walkers of a ten-electron atom (FP32),
// 1.27 -> 0.57 ms with jets at 1024 walkers of a ten-atom chain (FP64).
template <typename TN, bool JETS, int PT, int KQ1, int KQ2>
__global__ __launch_bounds__(KQ2 == 16 ? 512 : 256, JETS || sizeof(TN) == 8 ? 2 : 4) void k_bwd_filter(
    Dims d, DevTables t, int64_t nw, const double* __restrict__ r, const TN* __restrict__ P, ParamLayout pl,
    const TN* __restrict__ ctw, const TN* __restrict__ ctww, const TN* __restrict__ ctwd, const TN* __restrict__ ctw2,
    TN* __restrict__ fslot, int n_same) {
  extern __shared__ __align__(16) char smem[];
  typedef typename MfmaTile<TN>::acc_t acc_t;
  constexpr int NJ = JETS ? 3 : 1, K = 4 * KQ1, DZ = 4 * KQ2, NT = KQ2 == 16 ? 512 : 256, NW = NT / 64;
  constexpr int LDK = ld_pad<TN>(K), LDZ = ld_pad<TN>(DZ);
  constexpr int RPG = PT / 4;  // rows of a tile per lane group of the MFMA reduction
  constexpr int nz = DZ / 16, nt1 = (K / 16) * nz, nt = nt1 + nz * nz, kTiles = (nt + NW - 1) / NW;
  constexpr int nh = nz * (PT / 16), kHid = (nh + NW - 1) / NW;  // hidden-layer tiles, per wave
  constexpr int kCw = PT * DZ / NT;                              // cotangent entries per thread and jet
  const int layer = blockIdx.y / 3, ch = blockIdx.y % 3, L = d.L;
  const int p_lo = ch == 0 ? 0 : (ch == 1 ? n_same : d.n_ee);
  const int p_hi = ch == 0 ? n_same : (ch == 1 ? d.n_ee : d.n_pairs);
  const int np = p_hi - p_lo;
  const int64_t nrows = nw * np;
  double* dd = reinterpret_cast<double*>(smem);                  // [2][PT] distances, this tile's and the next's
  int64_t* oc = reinterpret_cast<int64_t*>(dd + 2 * PT);         // [2][PT] offset of a row in the pair tables
  int64_t* oe = oc + 2 * PT;                                     // [2][PT] in the ee table, -1 for e-n pairs
  TN* E = reinterpret_cast<TN*>(oe + 2 * PT);    // [NJ][PT][LDK] feature jets
  TN* U = E + NJ * PT * LDK;                     // [NJ][PT][LDZ] activations
  TN* CW = U + NJ * PT * LDZ;                    // [NJ][PT][LDZ] d/d (w, w'/d, w'')
  TN* CU = CW + NJ * PT * LDZ;                   // [NJ][PT][LDZ] d/d hidden jets
  const ParamLayout::Layer& Lp = pl.layer[layer];
  constexpr int fsz = K * DZ + DZ + DZ * DZ + DZ;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, g = lane >> 4, c16 = lane & 15;
  acc_t accs[kTiles];
#pragma unroll
  for (int k = 0; k < kTiles; ++k)
#pragma unroll
    for (int v = 0; v < 4; ++v) accs[k][v] = 0;
  TN bacc = 0;  // thread z < DZ owns db1[z], thread DZ + z db2[z] (different waves where DZ is a wave)
  // weight slabs of this wave's column of hidden tiles (ct = wv % nz for each of them)
  const int col = (wv % nz) * 16 + c16;
  TN w1[KQ1], w2[KQ2];
#pragma unroll
  for (int s = 0; s < KQ1; ++s) w1[s] = P[Lp.w1W[ch] + (g * KQ1 + s) * DZ + col];
#pragma unroll
  for (int s = 0; s < KQ2; ++s) w2[s] = P[Lp.w2W[ch] + col * DZ + g * KQ2 + s];
  const TN b1 = P[Lp.w1b[ch] + col];
  // distance and table offsets of row q of the tile at row0
  auto locate = [&](int64_t row0, int buf) {
    const int q = (int)threadIdx.x - (NT - PT);  // the last threads: the first ones sum the biases
    if (q < 0) return;
    double v = 1.0;
    int64_t o = 0, e = -1;
    if (row0 + q < nrows) {
      const int gq = (int)(row0 + q), w = gq / np, p = p_lo + gq - w * np;
      const double* rw = r + (int64_t)w * d.N * 3;
      double x, y, z;
      if (p < d.n_ee) {
        const int i = t.pair_ij[2 * p], j = t.pair_ij[2 * p + 1];
        x = rw[3 * i] - rw[3 * j];
        y = rw[3 * i + 1] - rw[3 * j + 1];
        z = rw[3 * i + 2] - rw[3 * j + 2];
        e = (((int64_t)w * L + layer) * d.n_ee + p) * DZ;
      } else {
        const int q2 = p - d.n_ee, i = q2 / d.NN, I = q2 - i * d.NN;
        x = rw[3 * i] - t.nuc_xyz[3 * I];
        y = rw[3 * i + 1] - t.nuc_xyz[3 * I + 1];
        z = rw[3 * i + 2] - t.nuc_xyz[3 * I + 2];
      }
      v = sqrt(x * x + y * y + z * z);
      o = (((int64_t)w * L + layer) * d.n_pairs + p) * DZ;
    }
    dd[buf * PT + q] = v;
    oc[buf * PT + q] = o;
    oe[buf * PT + q] = e;
  };
  // this thread's entries of the filter cotangents (rows past the end: zero)
  TN cw[NJ][kCw];
  auto request = [&](int64_t row0, int buf) {
    const int rows = (int)min((int64_t)PT, nrows - row0);
#pragma unroll
    for (int k = 0; k < kCw; ++k) {
      const int q = (int)threadIdx.x + k * NT, row = q / DZ, z = q % DZ;
      const int64_t o = oc[buf * PT + row] + z;
      cw[0][k] = ctw[o];
      if constexpr (JETS) {
        const int64_t e = oe[buf * PT + row];
        if (e >= 0) cw[0][k] += ctww[e + z];
        cw[NJ / 2][k] = ctwd[o];
        cw[NJ - 1][k] = ctw2[o];
      }
#pragma unroll
      for (int jet = 0; jet < NJ; ++jet) cw[jet][k] = row < rows ? cw[jet][k] : TN(0);
    }
  };
  const int64_t step = (int64_t)gridDim.x * PT;
  int64_t row0 = (int64_t)blockIdx.x * PT;
  int buf = 0;
  if (row0 < nrows) locate(row0, 0);
  __syncthreads();
  if (row0 < nrows) request(row0, 0);
  for (; row0 < nrows; row0 += step, buf ^= 1) {
    const int rows = (int)min((int64_t)PT, nrows - row0);
    const double* dc = dd + buf * PT;
    const bool more = row0 + step < nrows;
    for (int q = threadIdx.x; q < PT * K; q += NT) {
      const int row = q / K, k = q % K;
      TN e0 = 0, e1 = 0, e2 = 0;
      if (row < rows) {
        const double dv = dc[row], dm = dv - t.feat_mu[k], sg = t.feat_sig2inv[k];
        const double eg = exp(-dv - dm * dm * sg);
        e0 = (TN)(dv * dv * eg);
        if (JETS) {
          const double g1 = -1.0 - 2.0 * dm * sg, g2 = -2.0 * sg;
          e1 = (TN)((2.0 + dv * g1) * eg);                                  // e'/d
          e2 = (TN)((2.0 + 4.0 * dv * g1 + dv * dv * (g1 * g1 + g2)) * eg);  // e''
        }
      }
      E[row * LDK + k] = e0;
      if (JETS) {
        E[(PT + row) * LDK + k] = e1;
        E[(2 * PT + row) * LDK + k] = e2;
      }
    }
#pragma unroll
    for (int jet = 0; jet < NJ; ++jet)
#pragma unroll
      for (int k = 0; k < kCw; ++k) {
        const int q = (int)threadIdx.x + k * NT;
        CW[(jet * PT + q / DZ) * LDZ + q % DZ] = cw[jet][k];
      }
    if (more) locate(row0 + step, buf ^ 1);
    __syncthreads();
    if (more) request(row0 + step, buf ^ 1);
    // ---- hidden layer: both products, activation and its reverse ----
#pragma unroll
    for (int h = 0; h < kHid; ++h) {
      const int tile = wv + h * NW;
      if (tile < nh) {
        const int rt = tile / nz;
        acc_t cu[NJ], cc[NJ];
#pragma unroll
        for (int jet = 0; jet < NJ; ++jet) {
          TN a[KQ1], c[KQ2];
          const TN* xr = E + (jet * PT + rt * 16 + c16) * LDK + g * KQ1;
          const TN* cr = CW + (jet * PT + rt * 16 + c16) * LDZ + g * KQ2;
#pragma unroll
          for (int s = 0; s < KQ1; ++s) a[s] = xr[s];
#pragma unroll
          for (int s = 0; s < KQ2; ++s) c[s] = cr[s];
          acc_t z;
#pragma unroll
          for (int v = 0; v < 4; ++v) z[v] = TN(0);
          cu[jet] = MfmaChain<TN, KQ1>::run(a, w1, z, false);
          cc[jet] = MfmaChain<TN, KQ2>::run(c, w2, z, false);
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int row = rt * 16 + MfmaTile<TN>::row_of(lane, v);
          const bool ok = row < rows;
          TN* u0 = U + row * LDZ + col;
          TN* c0 = CU + row * LDZ + col;
          const TN u = cu[0][v] + b1;
          const TN s = sig(u);
          if constexpr (!JETS) {
            c0[0] = ok ? cc[0][v] * s : TN(0);
            u0[0] = ok ? ssp(u) : TN(0);  // hidden activation (zero on padding rows)
          } else {
            const TN s1 = ssp2(u), s2 = ssp3(u), dv = (TN)dc[row];
            const TN ud = cu[NJ / 2][v], u2 = cu[NJ - 1][v], up = dv * ud;
            const TN ca0 = cc[0][v], ca1 = cc[NJ / 2][v], ca2 = cc[NJ - 1][v];
            // (the fused steps are named: they are part of the FP32 rounding)
            c0[0] = ok ? fma(ca2, fma(s1, u2, s2 * up * up), fma(ca0, s, ca1 * s1 * ud)) : TN(0);
            c0[PT * LDZ] = ok ? fma(TN(2) * ca2 * s1 * dv, up, ca1 * s) : TN(0);
            c0[2 * PT * LDZ] = ok ? ca2 * s : TN(0);
            u0[0] = ok ? ssp(u) : TN(0);
            u0[PT * LDZ] = ok ? s * ud : TN(0);
            u0[2 * PT * LDZ] = ok ? fma(s, u2, s1 * up * up) : TN(0);
          }
        }
      }
    }
    __syncthreads();
    // ---- weight gradients dW1 = sum_k E_k^T CU_k and dW2 = sum_k U_k^T CW_k:
    // every wave keeps its 16 x 16 output tiles in registers across the tiles ----
#pragma unroll
    for (int k = 0; k < kTiles; ++k) {
      const int tt = wv + k * NW;
      if (tt < nt) {
        const bool first_mat = tt < nt1;
        const int a0 = (first_mat ? tt / nz : (tt - nt1) / nz) * 16, b0 = (first_mat ? tt % nz : (tt - nt1) % nz) * 16;
        const TN* X = (first_mat ? E : U) + a0 + c16;
        const TN* Y = (first_mat ? CU : CW) + b0 + c16;
        const int ldx = first_mat ? LDK : LDZ;
#pragma unroll
        for (int jet = 0; jet < NJ; ++jet) {
          TN af[RPG], bf[RPG];
#pragma unroll
          for (int s2 = 0; s2 < RPG; ++s2) {
            af[s2] = X[(jet * PT + g * RPG + s2) * ldx];
            bf[s2] = Y[(jet * PT + g * RPG + s2) * LDZ];
          }
          accs[k] = MfmaChain<TN, RPG>::run(af, bf, accs[k], false);
        }
      }
    }
    if (threadIdx.x < 2 * DZ) {
      const TN* y = (threadIdx.x < DZ ? CU : CW) + threadIdx.x % DZ;
      for (int r0 = 0; r0 < rows; r0 += 8) {
        TN v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = y[min(r0 + k, PT - 1) * LDZ];
#pragma unroll
        for (int k = 0; k < 8; ++k)
          if (r0 + k < rows) bacc += v[k];
      }
    }
    __syncthreads();
  }
  TN* out = fslot + ((size_t)blockIdx.x * L * 3 + blockIdx.y) * fsz;
  // layout of a filter block: [w1W K x DZ][w1b DZ][w2W DZ x DZ][w2b DZ]
#pragma unroll
  for (int k = 0; k < kTiles; ++k) {
    const int tt = wv + k * NW;
    if (tt < nt) {
      const bool first_mat = tt < nt1;
      const int a0 = (first_mat ? tt / nz : (tt - nt1) / nz) * 16, b0 = (first_mat ? tt % nz : (tt - nt1) % nz) * 16;
      const int base = first_mat ? 0 : K * DZ + DZ;
#pragma unroll
      for (int v = 0; v < 4; ++v) out[base + (a0 + MfmaTile<TN>::row_of(lane, v)) * DZ + b0 + c16] = accs[k][v];
    }
  }
  if (threadIdx.x < 2 * DZ)
    out[K * DZ + (threadIdx.x < DZ ? 0 : DZ + DZ * DZ) + threadIdx.x % DZ] = bacc;
}

// sum_b p[b * stride], b = 0 .. n-1 in order, in FP64; sixteen slots requested
// together (the slots are far apart: one load at a time made this kernel 4 % of
// a training step, 0.25 instead of 0.05 ms at 4096 walkers of a ten-electron atom)
template <typename TN>
__device__ __forceinline__ double slot_sum(const TN* __restrict__ p, size_t stride, int n, double s) {
  for (int b = 0; b < n; b += 16) {
    TN v[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) v[k] = p[(size_t)min(b + k, n - 1) * stride];
#pragma unroll
    for (int k = 0; k < 16; ++k)
      if (b + k < n) s += (double)v[k];
  }
  return s;
}

template <typename TN>
__global__ __launch_bounds__(kThreads) void k_bwd_reduce(Dims d, ParamLayout pl, int64_t n_params, int n_net,
                                                         const TN* __restrict__ gslot, int n_filt,
                                                         const TN* __restrict__ fslot, int n_tan,
                                                         const TN* __restrict__ tslot, double* __restrict__ grad) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= n_params) return;
  const int fsz = d.K * d.DZ + d.DZ + d.DZ * d.DZ + d.DZ;
  // is q inside a filter block?
  for (int n = 0; n < d.L; ++n) {
    const int64_t f0 = pl.layer[n].w1W[0];
    if (q >= f0 && q < f0 + 3 * fsz) {
      const int seg = n * 3 + (int)((q - f0) / fsz), o = (int)((q - f0) % fsz);
      grad[q] += slot_sum(fslot + (size_t)seg * fsz + o, (size_t)d.L * 3 * fsz, n_filt, 0.0);
      return;
    }
  }
  double s = slot_sum(gslot + q, n_params, n_net, 0.0);
  // the tangent adjoint's slots hold what depends on the tangents: the
  // products without a bias, from layer 1 on for h, and the nuclear embeddings
  bool tan = (q >= pl.Y && q < pl.Y + d.NN * d.DZ);
  for (int n = 0; n < d.L; ++n) {
    const ParamLayout::Layer& Lp = pl.layer[n];
    const int64_t xz = (int64_t)d.DX * d.DZ;
    tan = tan || (n > 0 && q >= Lp.hW && q < Lp.hW + xz);
    for (int ch = 0; ch < 3; ++ch) tan = tan || (q >= Lp.gW[ch] && q < Lp.gW[ch] + xz);
  }
  const int64_t xx = (int64_t)d.DX * d.DX;
  if (!(d.flags & PN_NET_NO_JASTROW))
    tan = tan || (q >= pl.eW1 && q < pl.eW1 + xx) || (q >= pl.eW2 && q < pl.eW2 + xx) ||
          (q >= pl.eW3 && q < pl.eW3 + d.DX);
  if (!(d.flags & PN_NET_NO_BACKFLOW))
    tan = tan || (q >= pl.kW1 && q < pl.kW1 + xx) || (q >= pl.kW2 && q < pl.kW2 + xx) ||
          (q >= pl.kW3 && q < pl.kW3 + (int64_t)d.DX * d.M);
  if (tan && n_tan > 0) s = slot_sum(tslot + q, n_params, n_tan, s);
  grad[q] += s;
}

}  // namespace

// elements of k_bwd_net's union region (head buffers, or layer buffers)
template <typename TN>
static size_t bwd_net_union(const Dims& d, int WB) {
  const int LDX = ld_pad<TN>(d.DX), LDZ = ld_pad<TN>(d.DZ), LDM = ld_pad<TN>((d.M + 15) & ~15);
  const size_t RW = (size_t)WB * d.N;
  const size_t heads = 3 * RW * LDX + RW * LDM + 6 * (size_t)WB * LDX;  // kappa buffers, then the eta ones
  const size_t layers = 5 * RW * LDZ;
  return std::max(heads, layers);
}

// LDS of k_bwd_net; with `arena` the union region lives in global memory
template <typename TN>
static size_t bwd_net_lds(const Dims& d, int WB, bool arena = false) {
  const size_t RW = (size_t)WB * d.N;
  return (size_t)((d.N * d.N + 3) & ~3) * sizeof(int) + (size_t)((d.n_ee + 7) & ~7) * 2 +
         (size_t)((2 * d.P * d.M + 15) & ~15) +
         ((size_t)((WB + 3) & ~3) + RW * ld_pad<TN>(d.DX) + (arena ? 0 : bwd_net_union<TN>(d, WB))) * sizeof(TN);
}

// Walkers per group: the unit of every sum over rows in the gradient (and so
// part of its FP32 rounding).  About 64 rows, as far as a block that also
// holds the layer inputs stays within half a CU's LDS.
template <typename TN>
static int bwd_wb(const Dims& d) {
  auto bytes = [&](int wb) {
    const size_t LDX = ld_pad<TN>(d.DX), LDZ = ld_pad<TN>(d.DZ), LDM = ld_pad<TN>((d.M + 15) & ~15);
    const size_t RW = (size_t)wb * d.N;
    return (size_t)((d.N * d.N + 3) & ~3) * sizeof(int) +
           ((size_t)((wb + 3) & ~3) + 2 * RW * LDX +
            std::max(3 * RW * LDX + RW * LDM + 6 * (size_t)wb * LDX, 4 * RW * LDZ)) *
               sizeof(TN);
  };
  int wb = std::max(1, 64 / d.N);
  while (wb > 1 && bytes(wb) > 80 * 1024) --wb;
  return wb;
}

// k_bwd_net keeps its union region in a global arena when the whole block
// does not fit in LDS (40 electrons of width 128 in FP64)
template <typename TN>
static bool bwd_net_arena(const Dims& d) {
  return bwd_net_lds<TN>(d, bwd_wb<TN>(d)) > 160 * 1024;
}

template <typename TN>
static size_t bwd_filter_lds(const Dims& d, int PT, bool full) {
  return (size_t)PT * 48 + (size_t)(full ? 3 : 1) * PT * (ld_pad<TN>(d.K) + 3 * ld_pad<TN>(d.DZ)) * sizeof(TN);
}

// Rows per tile of k_bwd_filter: 32, or 16 where the row tables of 32 exceed
// the LDS (the rule is part of the FP32 rounding of the filters' gradients).
static int bwd_filter_rows(const Dims& d, bool fp32, bool full) {
  const int nj = full ? 3 : 1;
  const size_t tn = fp32 ? sizeof(float) : sizeof(double);
  const size_t ldk = fp32 ? ld_pad<float>(d.K) : ld_pad<double>(d.K);
  const size_t ldz = fp32 ? ld_pad<float>(d.DZ) : ld_pad<double>(d.DZ);
  for (int pt = kFiltRows; pt >= 16; pt /= 2)
    if (pt * sizeof(double) + (size_t)nj * pt * (ldk + 3 * ldz) * tn <= 160 * 1024) return pt;
  return 16;
}

static size_t filt_fsz(const Dims& d) { return (size_t)d.K * d.DZ + d.DZ + (size_t)d.DZ * d.DZ + d.DZ; }

// gradient slots in use: one per group of walkers, one per block of filter rows
static int64_t net_slots(int64_t nw, int wb) { return std::min<int64_t>((nw + wb - 1) / wb, kSlotsNet); }
static int64_t filter_slots(const Dims& d, int64_t nw, int pt) {
  const int n_same = d.n_up * (d.n_up - 1) / 2 + d.n_dn * (d.n_dn - 1) / 2;
  const int64_t max_np = std::max<int64_t>(std::max(n_same, d.n_ee - n_same), (int64_t)d.N * d.NN);
  return std::min<int64_t>((nw * max_np + pt - 1) / pt, kSlotsFilter);
}

// Scratch of a tile.  The row tables for the weight gradients are here as far
// as no region of the value pass that is read no more holds them (run_backward).
size_t backward_scratch_bytes(const pn_ctx* c, int64_t tile, bool fp32, bool full) {
  const Dims& d = c->d;
  const size_t tn = fp32 ? sizeof(float) : sizeof(double);
  const bool arena = fp32 ? bwd_net_arena<float>(d) : bwd_net_arena<double>(d);
  const int wb = fp32 ? bwd_wb<float>(d) : bwd_wb<double>(d);
  const size_t slots = net_slots(tile, wb), groups = (tile + wb - 1) / wb;
  size_t e = slots * c->pl.total;                                                          // net slots
  e += filter_slots(d, tile, bwd_filter_rows(d, fp32, full)) * d.L * 3 * filt_fsz(d);       // filter slots
  e += (size_t)tile * d.L * d.n_pairs * d.DZ;                                               // filter cotangents
  if (arena) e += slots * (fp32 ? bwd_net_union<float>(d, wb) : bwd_net_union<double>(d, wb));
  e += (size_t)d.L * tile * d.N * ((full ? 4 : 3) * (size_t)d.DZ + d.DX);                   // row tables
  e += groups * SmallSums(d).total;                                                         // group sums
  return e * tn + 8 * 256;
}

bool backward_supported(const pn_ctx* c, bool fp32) {
  const Dims& d = c->d;
  if ((d.K / 16 + d.DZ / 16) * (d.DZ / 16) > 8 * (kThreads / 64)) return false;  // accumulator tiles per wave
  size_t lds = fp32 ? bwd_net_lds<float>(d, bwd_wb<float>(d), bwd_net_arena<float>(d))
                    : bwd_net_lds<double>(d, bwd_wb<double>(d), bwd_net_arena<double>(d));
  return lds <= 160 * 1024;
}

template <typename TN>
static void run_backward(const pn_ctx* c, hipStream_t s, int64_t nw, const double* r, const TN* P, const double* ct,
                         char* ws, const WsLayout& L, double* grad, bool full) {
  const Dims& d = c->d;
  const int64_t np = c->pl.total;
  const int WB = bwd_wb<TN>(d), PT = bwd_filter_rows(d, sizeof(TN) == sizeof(float), full);
  TN* gslot = reinterpret_cast<TN*>(ws + L.gpart);
  TN* fslot = gslot + net_slots(L.tile, WB) * np;
  TN* ctw = fslot + filter_slots(d, L.tile, PT) * d.L * 3 * filt_fsz(d);
  const int64_t ng = (nw + WB - 1) / WB;
  const int64_t rows = nw * d.N;
  const SmallSums sm(d);
  // what follows the filter cotangents, in 256-byte steps
  TN* at = ctw + (size_t)L.tile * d.L * d.n_pairs * d.DZ;
  auto take = [&](size_t elems) {
    at = reinterpret_cast<TN*>((reinterpret_cast<uintptr_t>(at) + 255) & ~(uintptr_t)255);
    TN* p = at;
    at += elems;
    return p;
  };
  const bool use_arena = bwd_net_arena<TN>(d);
  const int64_t arena_elems = use_arena ? (int64_t)bwd_net_union<TN>(d, WB) : 0;
  TN* arena = use_arena ? take(net_slots(L.tile, WB) * arena_elems) : nullptr;
  // row tables take the place of what only the value pass and the tangent
  // kernels before this one read: the heads' slopes (as many tables of the same
  // size) and the backflow; without tangents also that of h, which a block
  // reads before it writes the cotangent there
  NetOps<TN> op;
  op.z = take((size_t)d.L * 3 * rows * d.DZ);
  op.cx = take((size_t)d.L * rows * d.DX);
  op.ch = full ? take((size_t)d.L * rows * d.DZ) : reinterpret_cast<TN*>(ws + L.hval);
  op.a1 = reinterpret_cast<TN*>(ws + L.kcoef);
  op.c2 = op.a1 + rows * d.DX;
  op.c1 = op.c2 + rows * d.DX;
  op.a2 = op.c1 + rows * d.DX;
  op.cf = reinterpret_cast<TN*>(ws + L.fval);
  op.s = reinterpret_cast<TN*>(ws + L.ecoef);
  op.e1 = op.s + nw * d.DX;
  op.ec1 = op.e1 + nw * d.DX;
  op.ec2 = op.ec1 + nw * d.DX;
  op.small = take((size_t)ng * sm.total);
  const TN* xval = reinterpret_cast<const TN*>(ws + L.xval);
  const size_t lds = bwd_net_lds<TN>(d, WB, use_arena);
  // a block that takes more than half the CU's LDS runs alone on it
  const int nt = lds > 80 * 1024 ? 512 : 256;
  auto net_kernel = nt == 512 ? &k_bwd_net<TN, 512> : &k_bwd_net<TN, 256>;
  if (lds > 65536)
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(net_kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)lds);
  const int nb_net = (int)net_slots(nw, WB);
  hipLaunchKernelGGL(net_kernel, dim3((unsigned)(use_arena ? nb_net : ng)), dim3(nt), lds, s, d, c->t, nw, WB, P, c->pl,
                     xval, reinterpret_cast<const TN*>(ws + L.hval), L.jets, reinterpret_cast<const TN*>(ws + L.filt),
                     reinterpret_cast<const double*>(ws + L.phi), reinterpret_cast<const double*>(ws + L.ginv),
                     reinterpret_cast<const double*>(ws + L.wdet), ct, ctw,
                     full ? reinterpret_cast<const double*>(ws + L.ctfpart) : nullptr, L.n_chunks,
                     full ? reinterpret_cast<const TN*>(ws + L.cthv) : nullptr,
                     full ? reinterpret_cast<const TN*>(ws + L.ctkc) : nullptr,
                     full ? reinterpret_cast<const TN*>(ws + L.ctec) : nullptr, op, arena, arena_elems);
  const UnitsOfWalkers units{nw, WB, kSlotsNet};
  WMats<TN> mats;
  mats.n = 0;
  auto mat = [&](const TN* X, const TN* Y, int64_t out, int A, int B, int rpw) {
    mats.m[mats.n++] = WMat<TN>{X, Y, out, 0, 0, A, B, rpw, 0};
  };
  for (int n = 0; n < d.L; ++n) {
    for (int ch = 0; ch < 3; ++ch)
      mat(op.z + (size_t)(n * 3 + ch) * rows * d.DZ, op.cx + (size_t)n * rows * d.DX, c->pl.layer[n].gW[ch], d.DZ, d.DX,
          d.N);
    mat(xval + (size_t)n * rows * d.DX, op.ch + (size_t)n * rows * d.DZ, c->pl.layer[n].hW, d.DX, d.DZ, d.N);
  }
  mat(op.a1, op.c2, c->pl.kW2, d.DX, d.DX, d.N);
  mat(xval + (size_t)d.L * rows * d.DX, op.c1, c->pl.kW1, d.DX, d.DX, d.N);
  mat(op.e1, op.ec2, c->pl.eW2, d.DX, d.DX, 1);
  mat(op.s, op.ec1, c->pl.eW1, d.DX, d.DX, 1);
  launch_wgrad<TN>(s, mats, units, nb_net, gslot, np);
  hipLaunchKernelGGL(k_wgrad_small<TN>, dim3((unsigned)((d.DX * d.M + sm.total + kThreads - 1) / kThreads), nb_net),
                     dim3(kThreads), 0, s, d, c->pl, units, op.a2, op.cf, op.small, gslot, np);
  const int n_same = d.n_up * (d.n_up - 1) / 2 + d.n_dn * (d.n_dn - 1) / 2;
  const int nb_f = (int)filter_slots(d, nw, PT);
  const size_t lds_f = bwd_filter_lds<TN>(d, PT, full);
  auto go = [&](auto kern, int nt) {
    if (lds_f > 65536)
      (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)lds_f);
    hipLaunchKernelGGL(kern, dim3(nb_f, d.L * 3), dim3(nt), lds_f, s, d, c->t, nw, r, P, c->pl, ctw,
                       full ? reinterpret_cast<const TN*>(ws + L.ctww) : nullptr,
                       full ? reinterpret_cast<const TN*>(ws + L.ctwd) : nullptr,
                       full ? reinterpret_cast<const TN*>(ws + L.ctw2) : nullptr, fslot, n_same);
  };
  auto by_rows = [&](auto k1, auto k2) {
    constexpr int KQ1 = decltype(k1)::value, KQ2 = decltype(k2)::value, nt = KQ2 == 16 ? 512 : 256;
    if (PT == 32)
      full ? go(&k_bwd_filter<TN, true, 32, KQ1, KQ2>, nt) : go(&k_bwd_filter<TN, false, 32, KQ1, KQ2>, nt);
    else
      full ? go(&k_bwd_filter<TN, true, 16, KQ1, KQ2>, nt) : go(&k_bwd_filter<TN, false, 16, KQ1, KQ2>, nt);
  };
  auto by_width = [&](auto k1) {
    if (d.DZ == 16)
      by_rows(k1, std::integral_constant<int, 4>());
    else if (d.DZ == 32)
      by_rows(k1, std::integral_constant<int, 8>());
    else  // the accumulators' limit on K and DZ excludes 128
      by_rows(k1, std::integral_constant<int, 16>());
  };
  if (d.K == 16)
    by_width(std::integral_constant<int, 4>());
  else if (d.K == 32)
    by_width(std::integral_constant<int, 8>());
  else
    by_width(std::integral_constant<int, 16>());
  const int n_tan = full ? (int)std::min<int64_t>(nw, kSlotsTanAdj) : 0;
  hipLaunchKernelGGL(k_bwd_reduce<TN>, dim3((unsigned)((np + kThreads - 1) / kThreads)), dim3(kThreads), 0, s, d,
                     c->pl, np, nb_net, gslot, nb_f, fslot, n_tan, full ? reinterpret_cast<const TN*>(ws + L.tslot) : nullptr,
                     grad);
}

void launch_backward(const pn_ctx* c, hipStream_t s, int64_t nw, const double* r, const void* P, bool fp32, bool bf16,
                     const double* ct, char* ws, const WsLayout& L, double* grad_params, bool full) {
  (void)bf16;
  if (fp32)
    run_backward<float>(c, s, nw, r, static_cast<const float*>(P), ct, ws, L, grad_params, full);
  else
    run_backward<double>(c, s, nw, r, static_cast<const double*>(P), ct, ws, L, grad_params, full);
}

size_t backward_filter_lds_bytes(const Dims& d, bool fp32, bool full) {
  const int pt = bwd_filter_rows(d, fp32, full);
  return fp32 ? bwd_filter_lds<float>(d, pt, full) : bwd_filter_lds<double>(d, pt, full);
}

}  // namespace pn

// Adjoint of the network tangent pass: the parameter gradient of the
// coordinate derivatives of J and f (first derivatives and Laplacian), the
// second-order part of the full parameter adjoint (Methods, "PauliNet
// extension of SchNet"; J = eta(sum_i x_i), f_i = 1 + kappa(x_i)).
//
// The tangent pass maps, per coordinate chunk, the tangent columns and the
// partial-Laplacian column of the embeddings through
//   Linear  y_a = x_a W,                  y_L = x_L W
//   ssp     y_a = s1 u_a,                 y_L = s1 u_L + s2 sum_a u_a^2
//           (s1 = ssp'(u), s2 = ssp''(u) at the value-pass point u)
//   message z_a = sum_j (w_ij h_{j,a} + d_a w_ij h_j)
//           z_L = sum_j (w_ij h_{j,L} + sum_a (d2_a w_ij h_j + 2 d_a w_ij h_{j,a}))
// Its reverse, per (walker, chunk), with the cotangents of the backflow
// tangents and of J's tangents as input:
//   Linear  ct x = ct y W^T,              dW += x^T ct y   (rows = (electron, column))
//   ssp     ct u_a = s1 ct y_a + 2 s2 u_a ct y_L,  ct u_L = s1 ct y_L,
//           ct s1 = sum_a u_a ct y_a + u_L ct y_L,  ct s2 = ct y_L sum_a u_a^2
//   message ct h_{j,.} = sum_i w_ij ct z_{i,.} + 2 sum_a d_a w_ij ct z_{i,L}  (w_ij = w_ji)
//           ct w_ij   = sum_cols (h_{j,c} ct z_{i,c} + h_{i,c} ct z_{j,c})
//           and the source terms give cotangents of the value-pass h_j, of
//           w'/d and w'' per pair, and of the nuclear embeddings Y_I.
// The cotangents of the value-pass quantities (h values, ssp' and ssp'' of
// the heads, the filter values and radial derivatives) are summed over the
// walker's chunks and handed to the value-path adjoint.
//
// Three kernels and the weight gradients of wgrad.h:
//  k_tan_adj     one block per (walker, chunk): the reverse of the chunk.
//                Leaves both row tables of every weight gradient and the
//                chunk's share of the value-pass cotangents.
//  k_tan_ww      cotangents of the filter values, summed over the chunks.
//  k_tan_sum     the chunks' shares of the other value-pass cotangents, added
//                in chunk order.
//  k_tan_small   parameter gradients that are no tile product.
// Slots take walkers w, w + 512, ... and a walker's chunks in order, so every
// sum has a fixed order.  The layer inputs x^(n) come from the forward tangent
// pass (saved per chunk); h = x W_h, the messages and the head pre-activations
// are recomputed.  The tables of one chunk are 1.4 MB at the 30-electron
// diatomic in FP32, so the walkers of a tile are taken in batches.
#pragma once
#include "adj_util.h"
#include "gemm_lds.h"
#include "mfma_gemm.h"
#include "pn_internal.h"
#include "wgrad.h"

namespace pn {

// Per-walker outputs of the tangent adjoint (sums over the walker's chunks).
template <typename TN>
struct TanAdjOut {
  TN* hv;  // [nw][L][N][DZ]        cotangent of the value-pass h
  TN* ww;  // [nw][L][n_ee][DZ]     cotangent of the ee filter values w
  TN* wd;  // [nw][L][n_pairs][DZ]  cotangent of w'/d
  TN* w2;  // [nw][L][n_pairs][DZ]  cotangent of w''
  TN* kc;  // [nw][2][2][N][DX]     cotangents of the backflow head's ssp', ssp''
  TN* ec;  // [nw][2][2][DX]        same for the Jastrow head
};

constexpr int tadj_nce_max(int T) { return (T + 4) / 3; }  // electrons a chunk of T coordinates touches

namespace {

// sum_a e_a^2 over the C - 1 tangent columns.  (This and the sums below name
// their fused steps: an expression leaves their order to the compiler, and
// the FP32 rounding of every gradient depends on it.)
template <typename TN, int C>
__device__ __forceinline__ TN tangent_sq(const TN (&e)[C]) {
  if constexpr (C == 2) return e[0] * e[0];
  TN sq = fma(e[0], e[0], e[1] * e[1]);
#pragma unroll
  for (int col = 2; col < C - 1; ++col) sq = fma(e[col], e[col], sq);
  return sq;
}
// Forward activation of a head layer on the jets of one row group: columns
// 0..C-2 are tangents, column C-1 the partial Laplacian.
template <typename TN, int C>
__device__ __forceinline__ void jet_act(const TN (&e)[C], TN s1, TN s2, TN (&a)[C]) {
#pragma unroll
  for (int col = 0; col < C - 1; ++col) a[col] = s1 * e[col];
  a[C - 1] = fma(s2, tangent_sq<TN, C>(e), s1 * e[C - 1]);
}
// Its reverse, in place on the cotangent c (becomes the cotangent of e);
// returns the cotangent of s1 and the factors cl and sq of that of s2.
template <typename TN, int C>
__device__ __forceinline__ void jet_act_adj(const TN (&e)[C], TN (&c)[C], TN s1, TN s2, TN& cs1, TN& cl, TN& sq) {
  cl = c[C - 1];
  sq = tangent_sq<TN, C>(e);
  cs1 = fma(e[C - 1], cl, e[0] * c[0]);
#pragma unroll
  for (int col = 1; col < C - 1; ++col) cs1 = fma(e[col], c[col], cs1);
#pragma unroll
  for (int col = 0; col < C - 1; ++col) c[col] = fma(s1, c[col], TN(2) * s2 * e[col] * cl);
  c[C - 1] = s1 * cl;
}
// The C columns of one row group at one feature, strided by ld.
template <typename TN, int C>
__device__ __forceinline__ void get_cols(const TN* p, int ld, TN (&v)[C]) {
#pragma unroll
  for (int col = 0; col < C; ++col) v[col] = p[col * ld];
}
template <typename TN, int C>
__device__ __forceinline__ void put_cols(TN* p, int ld, const TN (&v)[C]) {
#pragma unroll
  for (int col = 0; col < C; ++col) p[col * ld] = v[col];
}

// Tables that k_tan_adj leaves, one block of `len` elements per task (walker
// of the batch, chunk); offsets into it.  Row tables have contiguous rows.
struct TanOps {
  int64_t s0, a1j, ct1j, ct2j;          // Jastrow head [C][DX]: sum, first activation, cotangents of both layers
  int64_t a1, a2, c1, c2, cf;           // backflow head [R][DX]: activations, cotangents; cf [R][M]
  int64_t kc, ec, ew3;                  // slopes of the heads: [layer][ct s1, cl, sq][N][DX] and [..][DX]; [DX] share of the Jastrow head's dW3
  int64_t layer, step;                  // layer n at layer + n * step:
  int64_t z, zn, cx, ch, hb, cz, hv, wd, w2, Y;
  int64_t arena, len;                   // row buffers of a block whose LDS does not hold them
  __host__ __device__ TanOps(const Dims& d, int T, int64_t arena_elems) {
    const int64_t C = T + 1, R = d.N * C, NC = tadj_nce_max(T), NP = d.N + d.NN;
    int64_t o = 0;
    auto take = [&](int64_t n) {
      const int64_t at = o;
      o += (n + 63) / 64 * 64;
      return at;
    };
    s0 = take(C * d.DX), a1j = take(C * d.DX), ct1j = take(C * d.DX), ct2j = take(C * d.DX);
    a1 = take(R * d.DX), a2 = take(R * d.DX), c1 = take(R * d.DX), c2 = take(R * d.DX), cf = take(R * d.M);
    kc = take(6 * (int64_t)d.N * d.DX), ec = take(6 * d.DX), ew3 = take(d.DX);
    layer = o;
    z = take(2 * R * d.DZ) - layer, zn = take(NC * C * d.DZ) - layer, cx = take(R * d.DX) - layer;
    ch = take(R * d.DZ) - layer, hb = take(R * d.DZ) - layer, cz = take(2 * R * d.DZ) - layer;
    hv = take((int64_t)d.N * d.DZ) - layer;
    wd = take(NC * NP * d.DZ) - layer, w2 = take(NC * NP * d.DZ) - layer, Y = take((int64_t)d.NN * d.DZ) - layer;
    step = o - layer;
    o = layer + d.L * step;
    arena = take(arena_elems);
    len = o;
  }
};

// The units of the chunks: local slot l holds walkers l, l + 512, ... of the
// batch (whose first walker is `first` within the tile), chunk by chunk.
struct UnitsOfChunks {
  int64_t nw, first;
  int n_chunks, T, C, N3, R, slots;
  __device__ int64_t slot(int64_t l) const { return (first + l) % slots; }
  __device__ bool keep(int64_t l) const { return first + l >= slots; }
  __device__ int64_t count(int64_t l) const { return (nw - l + slots - 1) / slots * n_chunks; }
  __device__ int64_t task(int64_t l, int64_t k) const { return (l + k / n_chunks * slots) * n_chunks + k % n_chunks; }
  template <typename M>
  __device__ void rows(int64_t l, int64_t k, const M& m, int64_t& x0, int64_t& y0, int& n) const {
    const int64_t u = task(l, k);
    x0 = u * m.xu;
    y0 = u * m.yu;
    n = m.rows;
    if (m.rows == 0) {  // the chunk electrons' rows
      const int a0 = (int)(k % n_chunks) * T, e_lo = a0 / 3, e_hi = (min(a0 + T, N3) - 1) / 3;
      n = (e_hi - e_lo + 1) * C;
      y0 += (int64_t)e_lo * C * m.B;
    }
  }
};

// Bound by the matrix products' operand reads from LDS and the partner loops;
// what it replaced took a walker's chunks one after the other in one block
// (one wave per SIMD at 256 walkers) with its row buffers in global memory.
// Two row buffers P0 and P1 of [R][max(LDX, 2 LDZ)] hold, in turn, a head's
// activations and cotangents, and in a layer the cotangents of both channels'
// messages beside the h tangents and their cotangent; a product whose result
// finds no place goes through the block's tables (they are written anyway).
// Measured, all kernels of this file and the weight gradients: 86.4 -> 29 ms at
// 256 walkers of the 30-electron diatomic (FP32), 12.7 -> 7.0 ms at 1024
// walkers of a ten-atom chain (FP64).
template <typename TN, int C, bool GA, int NT, int SX, int WPE = 2>
__global__ __launch_bounds__(NT, WPE) void k_tan_adj(
    Dims d, DevTables t, int n_chunks, const double* __restrict__ r, const TN* __restrict__ P, ParamLayout pl,
    const TN* __restrict__ filt, const TN* __restrict__ hval, const TN* __restrict__ kcoef,
    const TN* __restrict__ ecoef, const TN* __restrict__ xsave, const double* __restrict__ ctftan,
    const double* __restrict__ ctc, TanOps to, TN* __restrict__ ops) {
  constexpr int T = C - 1, LC = T;
  constexpr int NCEM = tadj_nce_max(T);
  extern __shared__ __align__(16) char smem[];
  const int64_t task = blockIdx.x, w = task / n_chunks;
  const int chunk = (int)(task % n_chunks);
  const int N = d.N, DX = SX ? SX : d.DX, DZ = SX ? SX / 2 : d.DZ, M = d.M, NU = d.n_up, NN = d.NN, L = d.L,
            N3 = 3 * d.N;
  const int R = N * C, NP = N + NN;
  const int LDX = ld_pad<TN>(DX), LDZ = ld_pad<TN>(DZ);
  const int sx = log2_of(DX), sz = log2_of(DZ);
  TN* ob = ops + task * to.len;
  double* rs = reinterpret_cast<double*>(smem);                // [N][3]
  int* pidx = reinterpret_cast<int*>(rs + ((N3 + 1) & ~1));    // [N][N]
  TN* cg = reinterpret_cast<TN*>(pidx + ((N * N + 3) & ~3));   // [NCEM][N][4]  r_i - r_k, 1/|r_i - r_k|
  TN* cgn = cg + NCEM * N * 4;                                 // [NCEM][NN][4] r_k - R_I, 1/|r_k - R_I|
  TN* cj = cgn + NCEM * NN * 4;                                // [C][LDX] cotangent of sum_i x_i
  TN* czn = cj + C * LDX;                                      // [NCEM C][LDZ] cotangent of the nuclear messages
  TN* eA = czn + NCEM * C * LDZ;                               // [2][NCEM][C + 1][DZ] pass A's share of chunk rows
  TN* eB = eA + 2 * NCEM * (C + 1) * DZ;                       // [2][NCEM][4][DZ] pass B's
  TN* P0 = GA ? ob + to.arena : eB + 2 * NCEM * 4 * DZ;
  TN* P1 = P0 + R * max(LDX, 2 * LDZ);
  const int a0 = chunk * T, Tc = min(T, N3 - a0);
  const int e_lo = a0 / 3, e_hi = (a0 + Tc - 1) / 3, NCE = e_hi - e_lo + 1;
  const TN* xs_base = xsave + (size_t)task * L * R * DX;
  const double* cc = ctc + w * (N3 + 2);
  const int64_t fl_stride = (int64_t)3 * d.n_pairs * DZ;
  const bool do_j = !(d.flags & PN_NET_NO_JASTROW), do_k = !(d.flags & PN_NET_NO_BACKFLOW);
  for (int q = threadIdx.x; q < N * N; q += blockDim.x) pidx[q] = t.pair_index[q];
  for (int q = threadIdx.x; q < N3; q += blockDim.x) rs[q] = r[w * N3 + q];
  {
    const TN* xl = xs_base + (size_t)(L - 1) * R * DX;
    for (int q = threadIdx.x; q < R * DX; q += blockDim.x) P0[(q >> sx) * LDX + (q & (DX - 1))] = xl[q];
  }
  __syncthreads();
  for (int q = threadIdx.x; q < NCE * N; q += blockDim.x) {
    const int k = e_lo + q / N, i = q % N;
    const double ux = rs[3 * i] - rs[3 * k], uy = rs[3 * i + 1] - rs[3 * k + 1], uz = rs[3 * i + 2] - rs[3 * k + 2];
    cg[4 * q + 0] = (TN)ux;
    cg[4 * q + 1] = (TN)uy;
    cg[4 * q + 2] = (TN)uz;
    cg[4 * q + 3] = i == k ? TN(0) : (TN)(1.0 / sqrt(ux * ux + uy * uy + uz * uz));
  }
  for (int q = threadIdx.x; q < NCE * NN; q += blockDim.x) {
    const int k = e_lo + q / NN, I = q % NN;
    const double ux = rs[3 * k] - t.nuc_xyz[3 * I], uy = rs[3 * k + 1] - t.nuc_xyz[3 * I + 1],
                 uz = rs[3 * k + 2] - t.nuc_xyz[3 * I + 2];
    cgn[4 * q + 0] = (TN)ux;
    cgn[4 * q + 1] = (TN)uy;
    cgn[4 * q + 2] = (TN)uz;
    cgn[4 * q + 3] = (TN)(1.0 / sqrt(ux * ux + uy * uy + uz * uz));
  }
  // ================= Jastrow head, rows = columns =================
  if (!do_j) {
    for (int q = threadIdx.x; q < C * LDX; q += blockDim.x) cj[q] = 0;
  } else {
    TN* S0 = P1;
    TN* E1 = S0 + C * LDX;
    TN* A1 = E1 + C * LDX;
    TN* E2 = A1 + C * LDX;
    TN* CT = E2 + C * LDX;
    TN* CT2 = CT + C * LDX;
    const TN* ec0 = ecoef + (w * 2 + 0) * 2 * DX;
    const TN* ec1 = ecoef + (w * 2 + 1) * 2 * DX;
    TN* oec = ob + to.ec;
    for (int q = threadIdx.x; q < C * DX; q += blockDim.x) {
      const int col = q >> sx, x = q & (DX - 1);
      TN s = 0;
      for (int i = 0; i < N; ++i) s += P0[(i * C + col) * LDX + x];
      S0[col * LDX + x] = s;
      ob[to.s0 + q] = s;
    }
    __syncthreads();
    gemm_mfma<TN>(S0, LDX, C, DX, P + pl.eW1, DX, E1, LDX, false, false);
    __syncthreads();
    for (int x = threadIdx.x; x < DX; x += blockDim.x) {
      TN e[C], a[C];
      get_cols<TN, C>(E1 + x, LDX, e);
      jet_act<TN, C>(e, ec0[x], ec0[DX + x], a);
      put_cols<TN, C>(A1 + x, LDX, a);
      put_cols<TN, C>(ob + to.a1j + x, DX, a);
    }
    __syncthreads();
    gemm_mfma<TN>(A1, LDX, C, DX, P + pl.eW2, DX, E2, LDX, false, false);
    __syncthreads();
    for (int x = threadIdx.x; x < DX; x += blockDim.x) {
      TN e[C], a[C], c[C];
      get_cols<TN, C>(E2 + x, LDX, e);
      jet_act<TN, C>(e, ec1[x], ec1[DX + x], a);
      TN s = 0;
      const TN w3 = P[pl.eW3 + x];
#pragma unroll
      for (int col = 0; col < C; ++col) {
        const TN cjc = col < LC ? (col < Tc ? (TN)cc[a0 + col] : TN(0)) : (TN)cc[N3];
        s += a[col] * cjc;
        c[col] = cjc * w3;
      }
      ob[to.ew3 + x] = s;
      jet_act_adj<TN, C>(e, c, ec1[x], ec1[DX + x], oec[3 * DX + x], oec[4 * DX + x], oec[5 * DX + x]);
      put_cols<TN, C>(CT + x, LDX, c);
      put_cols<TN, C>(ob + to.ct2j + x, DX, c);
    }
    __syncthreads();
    gemm_mfma_wt<TN>(CT, LDX, C, DX, P + pl.eW2, DX, CT2, LDX, false);
    __syncthreads();
    for (int x = threadIdx.x; x < DX; x += blockDim.x) {
      TN e[C], c[C];
      get_cols<TN, C>(E1 + x, LDX, e);
      get_cols<TN, C>(CT2 + x, LDX, c);
      jet_act_adj<TN, C>(e, c, ec0[x], ec0[DX + x], oec[x], oec[DX + x], oec[2 * DX + x]);
      put_cols<TN, C>(CT2 + x, LDX, c);
      put_cols<TN, C>(ob + to.ct1j + x, DX, c);
    }
    __syncthreads();
    gemm_mfma_wt<TN>(CT2, LDX, C, DX, P + pl.eW1, DX, cj, LDX, false);  // cotangent of sum_i x_i
  }
  __syncthreads();
  // ================= backflow head, rows = (electron, column) =================
  if (do_k) {
    const double* cf = ctftan + (size_t)task * R * M;
    TN* ocf = ob + to.cf;
    for (int q = threadIdx.x; q < R * M; q += blockDim.x) ocf[q] = (TN)cf[q];
    gemm_mfma<TN>(P0, LDX, R, DX, P + pl.kW1, DX, P1, LDX, false, false);  // K1
    __syncthreads();
    const TN* kc0 = kcoef + (w * 2 + 0) * 2 * N * DX;
    const TN* kc1 = kcoef + (w * 2 + 1) * 2 * N * DX;
    TN* okc = ob + to.kc;
    for (int q = threadIdx.x; q < N * DX; q += blockDim.x) {
      const int i = q >> sx, x = q & (DX - 1);
      TN e[C], a[C];
      get_cols<TN, C>(P1 + i * C * LDX + x, LDX, e);
      jet_act<TN, C>(e, kc0[q], kc0[N * DX + q], a);
      put_cols<TN, C>(P0 + i * C * LDX + x, LDX, a);
      put_cols<TN, C>(ob + to.a1 + i * C * DX + x, DX, a);
    }
    __syncthreads();
    TN* ok2 = ob + to.c2;  // K2, then its cotangent
    gemm_mfma<TN>(P0, LDX, R, DX, P + pl.kW2, DX, ok2, DX, false, false);
    __syncthreads();
    // second activation, the cotangent CF W3^T (W3 is [DX][M]) and its reverse;
    // two electrons per read of W3
    for (int q = threadIdx.x; q < ((N + 1) >> 1) * DX; q += blockDim.x) {
      const int i0 = (q >> sx) * 2, x = q & (DX - 1);
      const TN* w3 = P + pl.kW3 + x * M;
      const TN* cfa = ocf + i0 * C * M;
      const TN* cfb = ocf + min(i0 + 1, N - 1) * C * M;
      TN sv[2][C];
#pragma unroll
      for (int e = 0; e < 2; ++e)
#pragma unroll
        for (int col = 0; col < C; ++col) sv[e][col] = 0;
      for (int mu = 0; mu < M; ++mu) {
        const TN wv = w3[mu];
#pragma unroll
        for (int col = 0; col < C; ++col) {
          sv[0][col] += cfa[col * M + mu] * wv;
          sv[1][col] += cfb[col * M + mu] * wv;
        }
      }
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const int i = i0 + e, qi = i * DX + x;
        if (i >= N) break;
        TN k2[C], a[C];
        get_cols<TN, C>(ok2 + i * C * DX + x, DX, k2);
        jet_act<TN, C>(k2, kc1[qi], kc1[N * DX + qi], a);
        put_cols<TN, C>(ob + to.a2 + i * C * DX + x, DX, a);
        jet_act_adj<TN, C>(k2, sv[e], kc1[qi], kc1[N * DX + qi], okc[3 * N * DX + qi], okc[4 * N * DX + qi],
                           okc[5 * N * DX + qi]);
        put_cols<TN, C>(P0 + i * C * LDX + x, LDX, sv[e]);
        put_cols<TN, C>(ok2 + i * C * DX + x, DX, sv[e]);
      }
    }
    __syncthreads();
    TN* ok1 = ob + to.c1;  // cotangent of the first activation, then of K1
    gemm_mfma_wt<TN>(P0, LDX, R, DX, P + pl.kW2, DX, ok1, DX, false);
    __syncthreads();
    for (int q = threadIdx.x; q < N * DX; q += blockDim.x) {
      const int i = q >> sx, x = q & (DX - 1);
      TN e[C], c[C];
      get_cols<TN, C>(P1 + i * C * LDX + x, LDX, e);
      get_cols<TN, C>(ok1 + i * C * DX + x, DX, c);
      jet_act_adj<TN, C>(e, c, kc0[q], kc0[N * DX + q], okc[q], okc[N * DX + q], okc[2 * N * DX + q]);
      put_cols<TN, C>(P0 + i * C * LDX + x, LDX, c);
      put_cols<TN, C>(ok1 + i * C * DX + x, DX, c);
    }
    __syncthreads();
  }
  for (int q = threadIdx.x; q < R * DX; q += blockDim.x) {
    const int row = q >> sx, x = q & (DX - 1);
    P1[row * LDX + x] = cj[(row % C) * LDX + x];
  }
  __syncthreads();
  if (do_k) {
    gemm_mfma_wt<TN>(P0, LDX, R, DX, P + pl.kW1, DX, P1, LDX, true);
    __syncthreads();
  }
  // ================= interaction layers, last to first =================
  TN* CXB = P1;  // cotangent of the layer's output; the other buffer is free
  TN* FB = P0;
  for (int n = L - 1; n >= 0; --n) {
    const ParamLayout::Layer& Lp = pl.layer[n];
    const bool hn = n > 0;  // x^(0) is the same for every walker: no h tangents in layer 0
    const TN* fv = filt + (w * L + n) * fl_stride;
    const TN* fd = fv + (int64_t)d.n_pairs * DZ;
    const TN* f2 = fv + (int64_t)2 * d.n_pairs * DZ;
    const TN* hvs = hval + (w * L + n) * N * DZ;
    TN* ol = ob + to.layer + n * to.step;
    TN* ocx = ol + to.cx;
    TN* ohb = ol + to.hb;
    TN* twd = ol + to.wd;  // [NCEM][NP][DZ]
    TN* tw2 = ol + to.w2;
    TN* cthv = ol + to.hv;
    for (int q = threadIdx.x; q < R * DX; q += blockDim.x) {
      const int o = (q >> sx) * LDX + (q & (DX - 1));
      ocx[q] = CXB[o];
      if (hn) FB[o] = xs_base[(size_t)(n - 1) * R * DX + q];
    }
    __syncthreads();
    if (hn) {
      gemm_mfma<TN>(FB, LDX, R, DX, P + Lp.hW, DZ, ohb, DZ, false, false);
      __syncthreads();
    }
    // cotangents of the three channels' messages
    TN* CZ = FB;  // [2][R][LDZ]
    const int czs = R * LDZ;
    for (int ch = 0; ch < 2; ++ch) gemm_mfma_wt<TN>(CXB, LDX, R, DX, P + Lp.gW[ch], DZ, CZ + ch * czs, LDZ, false);
    gemm_mfma_wt<TN>(CXB + e_lo * C * LDX, LDX, NCE * C, DX, P + Lp.gW[2], DZ, czn, LDZ, false);
    __syncthreads();
    TN* HB = CXB;            // [R][LDZ] h tangents
    TN* CH = CXB + R * LDZ;  // [R][LDZ] their cotangent
    if (hn) {
      TN* ocz = ol + to.cz;
      for (int q = threadIdx.x; q < R * DZ; q += blockDim.x) {
        const int o = (q >> sz) * LDZ + (q & (DZ - 1));
        HB[o] = ohb[q];
        ocz[q] = CZ[o];
        ocz[R * DZ + q] = CZ[czs + o];
      }
      __syncthreads();
    }
    // ---- rows i: this channel's messages (for the weight gradients), the
    // cotangents through w_ij (pass A), and the sources of the chunk
    // electrons e != i on row e; one read of the filter values for both ----
    for (int q = threadIdx.x; q < N * DZ; q += blockDim.x) {
      const int i = q >> sz, z = q & (DZ - 1);
      const bool own = i >= e_lo && i <= e_hi;
      TN chs[C];
      TN chv_sum = 0;
#pragma unroll
      for (int c = 0; c < C; ++c) chs[c] = 0;
      for (int ch = 0; ch < 2; ++ch) {
        const bool want_up = (ch == 0) == (i < NU);
        const int j_lo = want_up ? 0 : NU, j_hi = want_up ? NU : N;
        const TN* cz = CZ + ch * czs + z;
        TN acc[C], cac[C];
#pragma unroll
        for (int c = 0; c < C; ++c) acc[c] = cac[c] = 0;
        if (hn) {
          for (int j0 = j_lo; j0 < j_hi; j0 += 4) {
            TN wv[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) wv[k] = fv[max(pidx[i * N + min(j0 + k, j_hi - 1)], 0) * DZ + z];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
              const int j = j0 + k;
              if (j >= j_hi || j == i) continue;
              const TN* hj = HB + j * C * LDZ + z;
              const TN* cj2 = cz + j * C * LDZ;
#pragma unroll
              for (int c = 0; c < C; ++c) acc[c] += wv[k] * hj[c * LDZ];
#pragma unroll
              for (int c = 0; c < C; ++c) cac[c] += wv[k] * cj2[c * LDZ];
            }
          }
        }
        TN lap = acc[LC];
        if (own) {
          const TN* gi = cg + (i - e_lo) * N * 4;
          const int c0 = 3 * i - a0;
          TN sv0 = 0, sv1 = 0, sv2 = 0;
          for (int j = j_lo; j < j_hi; ++j) {
            if (j == i) continue;
            const int p = pidx[i * N + j] * DZ + z;
            const TN wd = fd[p], w2 = f2[p];
            const TN hj = hvs[j * DZ + z], inv = gi[4 * j + 3];
            const TN* hjc = HB + j * C * LDZ + z;
#pragma unroll
            for (int al = 0; al < 3; ++al) {
              const int c = c0 + al;
              if (c < 0 || c >= Tc) continue;
              const TN ua = -gi[4 * j + al], ur = ua * inv, dw = wd * ua;
              if (al == 0) sv0 += dw * hj;
              if (al == 1) sv1 += dw * hj;
              if (al == 2) sv2 += dw * hj;
              lap += (w2 * ur * ur + wd * (TN(1) - ur * ur)) * hj;
              if (hn) lap += TN(2) * dw * hjc[c * LDZ];
            }
          }
#pragma unroll
          for (int c = 0; c < C; ++c) {
            const int al = c - c0;
            if (al == 0) acc[c] += sv0;
            if (al == 1) acc[c] += sv1;
            if (al == 2) acc[c] += sv2;
          }
        }
        // chunk electrons e of this channel: sources on row i (message) and,
        // from row e's cotangent, on h_i (pass A)
        TN chv = 0;
        const TN hvi = hvs[i * DZ + z];
        for (int e = max(e_lo, j_lo); e <= min(e_hi, j_hi - 1); ++e) {
          if (e == i) continue;
          const TN* gk = cg + ((e - e_lo) * N + i) * 4;  // r_i - r_e
          const int p = pidx[i * N + e] * DZ + z;
          const TN wd = fd[p], w2 = f2[p];
          const TN hk = hvs[e * DZ + z];
          const TN* hkc = HB + e * C * LDZ + z;
          const TN* cze = cz + e * C * LDZ;
          const TN ctzL = cze[LC * LDZ];
          const int c0 = 3 * e - a0;
          TN cwd = 0, cw2 = 0, s0 = 0, s1 = 0, s2 = 0;
#pragma unroll
          for (int al = 0; al < 3; ++al) {
            const int c = c0 + al;
            if (c < 0 || c >= Tc) continue;
            {
              const TN ua = gk[al], ur = ua * gk[3], dw = -wd * ua;
#pragma unroll
              for (int c2 = 0; c2 < LC; ++c2)
                if (c2 == c) acc[c2] = fma(dw, hk, acc[c2]);
              lap += (w2 * ur * ur + wd * (TN(1) - ur * ur)) * hk;
              if (hn) lap += TN(2) * dw * hkc[c * LDZ];
            }
            const TN ua = -gk[al], ur = ua * gk[3], ur2 = ur * ur;
            const TN ctzc = cze[c * LDZ];
            const TN d2 = w2 * ur2 + wd * (TN(1) - ur2);
            chv += wd * ua * ctzc + d2 * ctzL;
            cwd += ua * hvi * ctzc + (TN(1) - ur2) * hvi * ctzL;
            cw2 += ur2 * hvi * ctzL;
            if (hn) {
              const TN v = TN(2) * wd * ua * ctzL;
              if (al == 0) s0 += v;
              if (al == 1) s1 += v;
              if (al == 2) s2 += v;
              cwd += TN(2) * ua * HB[(i * C + c) * LDZ + z] * ctzL;
            }
          }
#pragma unroll
          for (int c = 0; c < C; ++c) {
            const int al = c - c0;
            if (al == 0) cac[c] += s0;
            if (al == 1) cac[c] += s1;
            if (al == 2) cac[c] += s2;
          }
          twd[((e - e_lo) * NP + i) * DZ + z] = cwd;
          tw2[((e - e_lo) * NP + i) * DZ + z] = cw2;
        }
        TN* oz = ol + to.z + (int64_t)ch * R * DZ + i * C * DZ + z;
#pragma unroll
        for (int c = 0; c < LC; ++c) oz[c * DZ] = acc[c];
        oz[LC * DZ] = lap;
        if (own) {  // pass B adds to these rows between the channels
          TN* ea = eA + ((ch * NCEM + i - e_lo) * (C + 1)) * DZ + z;
#pragma unroll
          for (int c = 0; c < C; ++c) ea[c * DZ] = cac[c];
          ea[C * DZ] = chv;
        } else {
#pragma unroll
          for (int c = 0; c < C; ++c) chs[c] += cac[c];
          chv_sum += chv;
        }
      }
      if (!own) {
        if (hn) put_cols<TN, C>(CH + i * C * LDZ + z, LDZ, chs);
        cthv[i * DZ + z] = chv_sum;
      }
    }
    // nuclear channel: messages, their cotangent's share of w'/d and w'' (rows
    // of the chunk's own electrons only), and d/dY_I
    for (int q = threadIdx.x; q < NCE * DZ; q += blockDim.x) {
      const int e = e_lo + (q >> sz), z = q & (DZ - 1);
      TN acc[C];
#pragma unroll
      for (int c = 0; c < C; ++c) acc[c] = 0;
      const int c0 = 3 * e - a0;
      const TN* cze = czn + (e - e_lo) * C * LDZ + z;
      const TN ctzL = cze[LC * LDZ];
      for (int I = 0; I < NN; ++I) {
        const TN* gn = cgn + ((e - e_lo) * NN + I) * 4;
        const TN y = P[pl.Y + I * DZ + z];
        const int p = (d.n_ee + e * NN + I) * DZ + z;
        const TN wd = fd[p], w2 = f2[p];
#pragma unroll
        for (int c = 0; c < T; ++c) {
          const int al = c - c0;
          if (al < 0 || al > 2 || c >= Tc) continue;
          const TN ua = gn[al], ur = ua * gn[3];
          acc[c] += wd * ua * y;
          acc[LC] += (w2 * ur * ur + wd * (TN(1) - ur * ur)) * y;
        }
        TN cwd = 0, cw2 = 0;
#pragma unroll
        for (int al = 0; al < 3; ++al) {
          const int c = c0 + al;
          if (c < 0 || c >= Tc) continue;
          const TN ua = gn[al], ur = ua * gn[3], ur2 = ur * ur;
          const TN ctzc = cze[c * LDZ];
          cwd += ua * y * ctzc + (TN(1) - ur2) * y * ctzL;
          cw2 += ur2 * y * ctzL;
        }
        twd[((e - e_lo) * NP + N + I) * DZ + z] = cwd;
        tw2[((e - e_lo) * NP + N + I) * DZ + z] = cw2;
      }
      put_cols<TN, C>(ol + to.zn + (e - e_lo) * C * DZ + z, DZ, acc);
    }
    for (int q = threadIdx.x; q < NN * DZ; q += blockDim.x) {
      const int I = q >> sz, z = q & (DZ - 1);
      TN s = 0;
      for (int e = e_lo; e <= e_hi; ++e) {
        const TN* gn = cgn + ((e - e_lo) * NN + I) * 4;
        const int p = (d.n_ee + e * NN + I) * DZ + z;
        const TN wd = fd[p], w2 = f2[p];
        const TN* cze = czn + (e - e_lo) * C * LDZ + z;
        const TN ctzL = cze[LC * LDZ];
        const int c0 = 3 * e - a0;
#pragma unroll
        for (int al = 0; al < 3; ++al) {
          const int c = c0 + al;
          if (c < 0 || c >= Tc) continue;
          const TN ua = gn[al], ur = ua * gn[3], ur2 = ur * ur;
          const TN ctzc = cze[c * LDZ];
          s += wd * ua * ctzc + (w2 * ur2 + wd * (TN(1) - ur2)) * ctzL;
        }
      }
      ol[to.Y + q] = s;
    }
    __syncthreads();
    // ---- pass B: chunk electrons e; the sources of e's coordinates on rows j ----
    for (int q = threadIdx.x; q < 2 * NCE * DZ; q += blockDim.x) {
      const int ce = q >> sz, z = q & (DZ - 1), ch = ce >= NCE, el = ce - ch * NCE, e = e_lo + el;
      const bool want_up = (ch == 0) == (e < NU);
      const int j_lo = want_up ? 0 : NU, j_hi = want_up ? NU : N;
      const TN* gi = cg + el * N * 4;  // r_j - r_e
      const TN hve = hvs[e * DZ + z];
      const TN* cz = CZ + ch * czs + z;
      const int c0 = 3 * e - a0;
      TN chv = 0, s0 = 0, s1 = 0, s2 = 0;
      for (int jb = j_lo; jb < j_hi; jb += 4) {
        TN wdv[4], w2v[4], td[4], t2[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const int j = min(jb + k, j_hi - 1), p = max(pidx[e * N + j], 0) * DZ + z, o = (el * NP + j) * DZ + z;
          wdv[k] = fd[p];
          w2v[k] = f2[p];
          td[k] = twd[o];
          t2[k] = tw2[o];
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const int j = jb + k;
          if (j >= j_hi || j == e) continue;
          const TN wd = wdv[k], w2 = w2v[k];
          const TN inv = gi[4 * j + 3];
          const TN ctzL = cz[(j * C + LC) * LDZ];
          TN cwd = 0, cw2 = 0;
#pragma unroll
          for (int al = 0; al < 3; ++al) {
            const int c = c0 + al;
            if (c < 0 || c >= Tc) continue;
            const TN ua = -gi[4 * j + al], ur = ua * inv, ur2 = ur * ur;
            const TN ctzc = cz[(j * C + c) * LDZ];
            const TN d2 = w2 * ur2 + wd * (TN(1) - ur2);
            chv += wd * ua * ctzc + d2 * ctzL;
            cwd += ua * hve * ctzc + (TN(1) - ur2) * hve * ctzL;
            cw2 += ur2 * hve * ctzL;
            if (hn) {
              const TN v = TN(2) * wd * ua * ctzL;
              if (al == 0) s0 += v;
              if (al == 1) s1 += v;
              if (al == 2) s2 += v;
              cwd += TN(2) * ua * HB[(e * C + c) * LDZ + z] * ctzL;
            }
          }
          twd[(el * NP + j) * DZ + z] = td[k] + cwd;
          tw2[(el * NP + j) * DZ + z] = t2[k] + cw2;
        }
      }
      TN* eb = eB + (ch * NCEM + el) * 4 * DZ + z;
      eb[0] = s0;
      eb[DZ] = s1;
      eb[2 * DZ] = s2;
      eb[3 * DZ] = chv;
    }
    __syncthreads();
    // chunk electrons' rows: pass A, then pass B, channel by channel
    for (int q = threadIdx.x; q < NCE * DZ; q += blockDim.x) {
      const int el = q >> sz, z = q & (DZ - 1), e = e_lo + el, c0 = 3 * e - a0;
      TN cs[C], chv = 0;
#pragma unroll
      for (int c = 0; c < C; ++c) cs[c] = 0;
      for (int ch = 0; ch < 2; ++ch) {
        const TN* ea = eA + (ch * NCEM + el) * (C + 1) * DZ + z;
        const TN* eb = eB + (ch * NCEM + el) * 4 * DZ + z;
#pragma unroll
        for (int c = 0; c < C; ++c) {
          cs[c] += ea[c * DZ];
          const int al = c - c0;
          if (al >= 0 && al < 3 && c < Tc) cs[c] += eb[al * DZ];
        }
        chv += ea[C * DZ];
        chv += eb[3 * DZ];
      }
      if (hn) put_cols<TN, C>(CH + e * C * LDZ + z, LDZ, cs);
      cthv[e * DZ + z] = chv;
    }
    if (!hn) break;
    // ---- cotangent of x^(n): that of x^(n+1) plus CH W_h^T ----
    for (int q = threadIdx.x; q < R * DX; q += blockDim.x) FB[(q >> sx) * LDX + (q & (DX - 1))] = ocx[q];
    __syncthreads();
    {
      TN* och = ol + to.ch;
      for (int q = threadIdx.x; q < R * DZ; q += blockDim.x) och[q] = CH[(q >> sz) * LDZ + (q & (DZ - 1))];
    }
    gemm_mfma_wt<TN>(CH, LDZ, R, DZ, P + Lp.hW, DX, FB, LDX, true);
    __syncthreads();
    TN* swap = CXB;
    CXB = FB;
    FB = swap;
  }
}

// ct w_ij = sum over chunks of sum_cols (h_{j,c} ct z_{i,c} + h_{i,c} ct z_{j,c}),
// added chunk by chunk.  Block: one walker, layer and 16 features, 16 x kWP
// pairs; a chunk's 16 columns of the three tables go through LDS with the jet
// columns of an electron and feature side by side.  Bound by those LDS reads.
constexpr int kWP = 16;
template <typename TN, int C>
__global__ __launch_bounds__(256) void k_tan_ww(Dims d, DevTables t, int n_chunks, const TN* __restrict__ ops,
                                                TanOps to, TN* __restrict__ ww) {
  extern __shared__ __align__(16) char smem[];
  const int N = d.N, DZ = d.DZ, R = N * C, nz = DZ / 16;
  const int64_t w = blockIdx.x;
  const int n = 1 + blockIdx.y / nz, z0 = (blockIdx.y % nz) * 16, z = threadIdx.x & 15;
  const int p0 = blockIdx.z * 16 * kWP + (int)(threadIdx.x >> 4);
  const int n_same = (d.n_up * (d.n_up - 1) + d.n_dn * (d.n_dn - 1)) / 2;
  TN* hb = reinterpret_cast<TN*>(smem);  // [N][16][C], then the two channels' ct z
  TN* cz = hb + R * 16;
  TN acc[kWP];
  int ij[kWP];
#pragma unroll
  for (int k = 0; k < kWP; ++k) {
    acc[k] = 0;
    const int p = min(p0 + 16 * k, d.n_ee - 1);
    ij[k] = t.pair_ij[2 * p] + 256 * t.pair_ij[2 * p + 1] + (p < n_same ? 0 : 65536);
  }
  for (int chunk = 0; chunk < n_chunks; ++chunk) {
    const TN* ol = ops + (w * n_chunks + chunk) * to.len + to.layer + n * to.step;
    __syncthreads();
    for (int q = threadIdx.x; q < 3 * R * 16; q += blockDim.x) {
      const int zz = q & 15, row3 = q >> 4, row = row3 % R, i = row / C, c = row - i * C, tab = row3 / R;
      const TN v = tab == 0 ? ol[to.hb + row * DZ + z0 + zz] : ol[to.cz + ((tab - 1) * R + row) * DZ + z0 + zz];
      hb[tab * R * 16 + (i * 16 + zz) * C + c] = v;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kWP; ++k) {
      const int i = ij[k] & 255, j = (ij[k] >> 8) & 255;
      const TN* hi = hb + (i * 16 + z) * C;
      const TN* hj = hb + (j * 16 + z) * C;
      const TN* zt = cz + (ij[k] >> 16) * R * 16;
      const TN* zi = zt + (i * 16 + z) * C;
      const TN* zj = zt + (j * 16 + z) * C;
      TN s = 0;
#pragma unroll
      for (int c = 0; c < C; ++c) s += hj[c] * zi[c] + hi[c] * zj[c];
      acc[k] += s;
    }
  }
#pragma unroll
  for (int k = 0; k < kWP; ++k) {
    const int p = p0 + 16 * k;
    if (p < d.n_ee) ww[((w * d.L + n) * d.n_ee + p) * DZ + z0 + z] = acc[k];
  }
}

// The other value-pass cotangents: one thread per element, chunks in order;
// bpw blocks per walker (a batch of a small system has more walkers than a
// grid has blocks in y).
template <typename TN>
__global__ __launch_bounds__(kThreads) void k_tan_sum(Dims d, int n_chunks, int T, int bpw, const TN* __restrict__ ops,
                                                      TanOps to, TanAdjOut<TN> out) {
  const int64_t w = blockIdx.x / (unsigned)bpw;
  const int N = d.N, DX = d.DX, DZ = d.DZ, L = d.L, NN = d.NN, NP = N + NN, N3 = 3 * N;
  const int n_hv = L * N * DZ, n_pw = L * d.n_pairs * DZ, n_kc = 4 * N * DX, n_ec = 4 * DX, n_w0 = d.n_ee * DZ;
  int q = (int)(blockIdx.x % (unsigned)bpw) * blockDim.x + threadIdx.x;
  const TN* base = ops + w * n_chunks * to.len;
  auto sum = [&](int64_t at) {
    TN v = 0;
    for (int c = 0; c < n_chunks; ++c) v += base[c * to.len + at];
    return v;
  };
  if (q < n_hv) {
    const int n = q / (N * DZ);
    out.hv[w * n_hv + q] = sum(to.layer + n * to.step + to.hv + q - n * N * DZ);
    return;
  }
  q -= n_hv;
  // slopes of a head's hidden unit: ct s1, or ct s2 = sum cl sq
  auto slope = [&](int64_t at, int width, int o) {
    const int lay = o / (2 * width), x = o % width;
    const int64_t a = at + lay * 3 * width + x;
    if (((o / width) & 1) == 0) return sum(a);
    TN v = 0;
    for (int c = 0; c < n_chunks; ++c) v = fma(base[c * to.len + a + width], base[c * to.len + a + 2 * width], v);
    return v;
  };
  if (q < n_kc) {
    out.kc[w * n_kc + q] = (d.flags & PN_NET_NO_BACKFLOW) ? TN(0) : slope(to.kc, N * DX, q);
    return;
  }
  q -= n_kc;
  if (q < n_ec) {
    out.ec[w * n_ec + q] = (d.flags & PN_NET_NO_JASTROW) ? TN(0) : slope(to.ec, DX, q);
    return;
  }
  q -= n_ec;
  if (q < n_w0) {  // layer 0 has no h tangents
    out.ww[w * (int64_t)L * d.n_ee * DZ + q] = 0;
    return;
  }
  q -= n_w0;
  if (q >= n_pw) return;
  // pair p of layer n: the chunks of its electrons (e-n pairs: one electron)
  const int n = q / (d.n_pairs * DZ), o = q - n * d.n_pairs * DZ, p = o / DZ, z = o % DZ;
  int i, j;
  if (p < d.n_ee) {
    // same-spin pairs of the up block, of the down block, opposite-spin pairs,
    // each with i < j ascending
    const int nu = d.n_up, nd = d.n_dn, su = nu * (nu - 1) / 2, sd = nd * (nd - 1) / 2;
    if (p < su + sd) {
      const int b = p < su ? 0 : nu, m = p < su ? nu : nd;
      int k = p < su ? p : p - su;
      i = 0;
      while (k >= m - 1 - i) k -= m - 1 - i, ++i;
      j = b + i + 1 + k;
      i += b;
    } else {
      i = (p - su - sd) / nd;
      j = nu + (p - su - sd) % nd;
    }
  } else {
    i = (p - d.n_ee) / NN;
    j = N + (p - d.n_ee) % NN;  // partner column N + I of the chunk tables
  }
  const int64_t lo = to.layer + n * to.step;
  TN vd = 0, v2 = 0;
  auto add = [&](int c, int e, int part, bool both) {
    const int e_lo = c * T / 3;
    const TN* b = base + c * to.len + lo;
    const int at = ((e - e_lo) * NP + part) * DZ + z;
    TN xd = b[to.wd + at], x2 = b[to.w2 + at];
    if (both) {  // both electrons in the chunk: its two entries together
      const int a2 = ((part - e_lo) * NP + e) * DZ + z;
      xd += b[to.wd + a2];
      x2 += b[to.w2 + a2];
    }
    vd += xd;
    v2 += x2;
  };
  for (int c = 0; c < n_chunks; ++c) {
    const int e_lo = c * T / 3, e_hi = (min(c * T + T, N3) - 1) / 3;
    const bool hi = i >= e_lo && i <= e_hi, hj = j < N && j >= e_lo && j <= e_hi;
    if (hi)
      add(c, i, j, hj);
    else if (hj)
      add(c, j, i, false);
  }
  out.wd[w * n_pw + q] = vd;
  out.w2[w * n_pw + q] = v2;
}

// Gradients that are no tile product, per slot: W3 of the backflow head (a
// thread per entry, the rows of a chunk in order), W3 of the Jastrow head and
// the nuclear embeddings (shares of each chunk, layer by layer).
template <typename TN>
__global__ __launch_bounds__(kThreads) void k_tan_small(Dims d, ParamLayout pl, UnitsOfChunks units,
                                                        const TN* __restrict__ ops, TanOps to, TN* __restrict__ slots,
                                                        int64_t slot_len) {
  const int64_t l = blockIdx.y;
  int q = blockIdx.x * blockDim.x + threadIdx.x;
  const int n3 = d.DX * d.M;
  TN* out = slots + units.slot(l) * slot_len;
  const bool keep = units.keep(l);
  const int64_t nu = units.count(l);
  if (q < n3) {
    if (d.flags & PN_NET_NO_BACKFLOW) return;
    const int a = q / d.M, b = q - a * d.M;
    TN acc = keep ? out[pl.kW3 + q] : TN(0);
    for (int64_t u = 0; u < nu; ++u) {
      const TN* x = ops + units.task(l, u) * to.len + to.a2 + a;
      const TN* y = ops + units.task(l, u) * to.len + to.cf + b;
      TN v = 0;
      for (int r0 = 0; r0 < units.R; r0 += 8) {
        TN xv[8], yv[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          const int r = min(r0 + k, units.R - 1);
          xv[k] = x[r * d.DX];
          yv[k] = y[r * d.M];
        }
#pragma unroll
        for (int k = 0; k < 8; ++k)
          if (r0 + k < units.R) v += xv[k] * yv[k];
      }
      acc += v;
    }
    out[pl.kW3 + q] = acc;
    return;
  }
  q -= n3;
  if (q < d.DX) {
    if (d.flags & PN_NET_NO_JASTROW) return;
    TN acc = keep ? out[pl.eW3 + q] : TN(0);
    for (int64_t u = 0; u < nu; ++u) acc += ops[units.task(l, u) * to.len + to.ew3 + q];
    out[pl.eW3 + q] = acc;
    return;
  }
  q -= d.DX;
  if (q >= d.NN * d.DZ) return;
  TN acc = keep ? out[pl.Y + q] : TN(0);
  for (int64_t u = 0; u < nu; ++u)
    for (int n = d.L - 1; n >= 0; --n) acc += ops[units.task(l, u) * to.len + to.layer + n * to.step + to.Y + q];
  out[pl.Y + q] = acc;
}

template <typename TN>
size_t tan_adj_small_lds(const Dims& d, int T) {
  const int NC = tadj_nce_max(T), C = T + 1;
  const size_t LDX = ld_pad<TN>(d.DX), LDZ = ld_pad<TN>(d.DZ);
  return ((size_t)(3 * d.N + 1) & ~(size_t)1) * sizeof(double) + (size_t)((d.N * d.N + 3) & ~3) * sizeof(int) +
         ((size_t)NC * (d.N + d.NN) * 4 + C * LDX + NC * C * LDZ + 2 * (size_t)NC * (C + 5) * d.DZ) * sizeof(TN);
}
template <typename TN>
size_t tan_adj_rows(const Dims& d, int T) {  // elements of P0 and P1
  const size_t C = T + 1, R = d.N * C, LDX = ld_pad<TN>(d.DX), LDZ = ld_pad<TN>(d.DZ);
  return R * std::max(LDX, 2 * LDZ) + std::max(R * std::max(LDX, 2 * LDZ), 6 * C * LDX);
}
// row buffers of a block in its tables where they exceed the LDS
template <typename TN>
bool tan_adj_global(const Dims& d, int T) {
  return tan_adj_small_lds<TN>(d, T) + tan_adj_rows<TN>(d, T) * sizeof(TN) > 160 * 1024;
}
template <typename TN>
TanOps tan_ops(const Dims& d, int T) {
  return TanOps(d, T, tan_adj_global<TN>(d, T) ? (int64_t)tan_adj_rows<TN>(d, T) : 0);
}
// walkers per batch: about 2 GiB of tables
template <typename TN>
int64_t tan_batch(const Dims& d, int T, int64_t nw) {
  const int n_chunks = (3 * d.N + T - 1) / T;
  const int64_t fit = (int64_t)((size_t(2) << 30) / ((size_t)tan_ops<TN>(d, T).len * n_chunks * sizeof(TN)));
  return std::max<int64_t>(1, std::min(fit, nw));
}

template <typename TN, int C, int SX>
void launch_ta_c(const pn_ctx* c, hipStream_t s, int64_t nw, const double* r, const TN* P, char* ws,
                 const WsLayout& L) {
  const Dims& d = c->d;
  constexpr int T = C - 1;
  const int R = d.N * C, nch = L.n_chunks;
  const TanOps to = tan_ops<TN>(d, T);
  TN* tslot = reinterpret_cast<TN*>(ws + L.tslot);
  TN* ops = reinterpret_cast<TN*>(ws + L.tanops);
  const int64_t np = c->pl.total, batch = tan_batch<TN>(d, T, nw), NN = d.n_pairs;
  const bool ga = tan_adj_global<TN>(d, T);
  const size_t lds = tan_adj_small_lds<TN>(d, T) + (ga ? 0 : tan_adj_rows<TN>(d, T) * sizeof(TN));
  // A block that takes more than half the CU's LDS runs alone on it, with 512
  // threads.  Four waves per SIMD (two 512-thread blocks) where the LDS holds two blocks
  // and 128 registers suffice, as in the tangent pass: full adjoints of 1024
  // walkers of ten electrons FP64 11.85 -> 11.2 ms, 512 of 18 electrons FP32
  // 9.5 -> 8.8.
  constexpr bool kFour = SX == 64 && (sizeof(TN) == 4 || C <= 4);
  constexpr int W = kFour ? 4 : 2;
  const bool two = kFour && lds > 160 * 1024 / 3 && lds <= 80 * 1024;
  const int nt = two || lds > 80 * 1024 ? 512 : 256;
  auto kern = two  ? (ga ? &k_tan_adj<TN, C, true, 512, SX, W> : &k_tan_adj<TN, C, false, 512, SX, W>)
              : ga ? (nt == 512 ? &k_tan_adj<TN, C, true, 512, SX> : &k_tan_adj<TN, C, true, 256, SX>)
                 : (nt == 512 ? &k_tan_adj<TN, C, false, 512, SX> : &k_tan_adj<TN, C, false, 256, SX>);
  if (lds > 65536)
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  const size_t lds_ww = (size_t)3 * R * 16 * sizeof(TN);
  if (lds_ww > 65536)
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&k_tan_ww<TN, C>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_ww);
  WMats<TN> mats;
  mats.n = 0;
  auto mat = [&](const TN* X, int64_t xu, int64_t yo, int64_t out, int A, int B, int rows) {
    mats.m[mats.n++] = WMat<TN>{X, ops + yo, out, xu, to.len, A, B, rows, 0};
  };
  for (int64_t w0 = 0; w0 < nw; w0 += batch) {
    const int64_t n = std::min(batch, nw - w0);
    const TN* xs = reinterpret_cast<const TN*>(ws + L.xsave) + (size_t)w0 * nch * d.L * R * d.DX;
    const int64_t xu = (int64_t)d.L * R * d.DX;
    hipLaunchKernelGGL(kern, dim3((unsigned)(n * nch)), dim3(nt), lds, s, d, c->t, nch, r + w0 * 3 * d.N, P, c->pl,
                       reinterpret_cast<const TN*>(ws + L.filt) + (size_t)w0 * d.L * 3 * d.n_pairs * d.DZ,
                       reinterpret_cast<const TN*>(ws + L.hval) + (size_t)w0 * d.L * d.N * d.DZ,
                       reinterpret_cast<const TN*>(ws + L.kcoef) + (size_t)w0 * 4 * d.N * d.DX,
                       reinterpret_cast<const TN*>(ws + L.ecoef) + (size_t)w0 * 4 * d.DX, xs,
                       reinterpret_cast<const double*>(ws + L.ctftan) + (size_t)w0 * nch * R * d.M,
                       reinterpret_cast<const double*>(ws + L.ctc) + (size_t)w0 * (3 * d.N + 2), to, ops);
    mats.n = 0;
    for (int l = 0; l < d.L; ++l) {
      const int64_t at = to.layer + l * to.step;
      for (int ch = 0; ch < 2; ++ch)
        mat(ops + at + to.z + (int64_t)ch * R * d.DZ, to.len, at + to.cx, c->pl.layer[l].gW[ch], d.DZ, d.DX, R);
      mat(ops + at + to.zn, to.len, at + to.cx, c->pl.layer[l].gW[2], d.DZ, d.DX, 0);
      if (l > 0) mat(xs + (size_t)(l - 1) * R * d.DX, xu, at + to.ch, c->pl.layer[l].hW, d.DX, d.DZ, R);
    }
    if (!(d.flags & PN_NET_NO_BACKFLOW)) {
      mat(ops + to.a1, to.len, to.c2, c->pl.kW2, d.DX, d.DX, R);
      mat(xs + (size_t)(d.L - 1) * R * d.DX, xu, to.c1, c->pl.kW1, d.DX, d.DX, R);
    }
    if (!(d.flags & PN_NET_NO_JASTROW)) {
      mat(ops + to.a1j, to.len, to.ct2j, c->pl.eW2, d.DX, d.DX, C);
      mat(ops + to.s0, to.len, to.ct1j, c->pl.eW1, d.DX, d.DX, C);
    }
    const UnitsOfChunks units{n, w0, nch, T, C, 3 * d.N, R, kSlotsTanAdj};
    const int n_slots = (int)std::min<int64_t>(n, kSlotsTanAdj);
    launch_wgrad<TN>(s, mats, units, n_slots, tslot, np);
    hipLaunchKernelGGL(k_tan_small<TN>,
                       dim3((unsigned)((d.DX * d.M + d.DX + d.NN * d.DZ + kThreads - 1) / kThreads), n_slots),
                       dim3(kThreads), 0, s, d, c->pl, units, ops, to, tslot, np);
    TanAdjOut<TN> o{reinterpret_cast<TN*>(ws + L.cthv) + (size_t)w0 * d.L * d.N * d.DZ,
                    reinterpret_cast<TN*>(ws + L.ctww) + (size_t)w0 * d.L * d.n_ee * d.DZ,
                    reinterpret_cast<TN*>(ws + L.ctwd) + (size_t)w0 * d.L * NN * d.DZ,
                    reinterpret_cast<TN*>(ws + L.ctw2) + (size_t)w0 * d.L * NN * d.DZ,
                    reinterpret_cast<TN*>(ws + L.ctkc) + (size_t)w0 * 4 * d.N * d.DX,
                    reinterpret_cast<TN*>(ws + L.ctec) + (size_t)w0 * 4 * d.DX};
    if (d.L > 1 && d.n_ee > 0)
      hipLaunchKernelGGL((k_tan_ww<TN, C>),
                         dim3((unsigned)n, (d.L - 1) * (d.DZ / 16), (d.n_ee + 16 * kWP - 1) / (16 * kWP)), dim3(256),
                         lds_ww, s, d, c->t, nch, ops, to, o.ww);
    const int64_t elems = (int64_t)d.L * d.N * d.DZ + 4 * d.N * d.DX + 4 * d.DX + d.n_ee * d.DZ +
                          (int64_t)d.L * d.n_pairs * d.DZ;
    const int bpw = (int)((elems + kThreads - 1) / kThreads);
    hipLaunchKernelGGL(k_tan_sum<TN>, dim3((unsigned)(n * bpw)), dim3(kThreads), 0, s, d, nch, T, bpw, ops, to, o);
  }
}

}  // namespace

// The chunk rule of the full adjoint (its chunks are part of the FP32
// rounding of every gradient): LDS of a block that holds five row tables of a
// chunk beside the tables of its pairs, or the latter alone.
template <typename TN>
size_t tangent_adj_arena_elems(const Dims& d, int T) {
  const int C = T + 1, R = d.N * C;
  const size_t LDX = ld_pad<TN>(d.DX), LDZ = ld_pad<TN>(d.DZ), LDM = ld_pad<TN>((d.M + 15) & ~15);
  const size_t u = std::max(std::max(3 * R * LDZ, 3 * R * LDX + R * LDM), 7 * (size_t)C * LDX);
  return 2 * R * LDX + u;
}
template <typename TN>
size_t tangent_adj_lds_bytes(const Dims& d, int T, bool global_arena) {
  const int NCEM = tadj_nce_max(T), NP = d.N + d.NN;
  size_t tn = (size_t)NCEM * (d.N + d.NN) * 4 + 2 * (size_t)d.N * d.DZ + 2 * (size_t)NCEM * NP * d.DZ;
  if (!global_arena) tn += tangent_adj_arena_elems<TN>(d, T);
  return 3 * kMaxElec * sizeof(double) + (size_t)((d.N * d.N + 3) & ~3) * sizeof(int) + tn * sizeof(TN);
}
// bytes of the batch's tables
template <typename TN>
size_t tangent_adj_ops_bytes(const Dims& d, int T, int64_t nw) {
  const int64_t n_chunks = (3 * d.N + T - 1) / T;
  return (size_t)tan_batch<TN>(d, T, nw) * n_chunks * tan_ops<TN>(d, T).len * sizeof(TN);
}

// SX: the embedding width as a compile-time constant (DZ = SX / 2), 0 for any
// widths, as in the tangent pass (129 to 184 registers become 76 to 155).
// Measured, full adjoints: ten electrons FP64 12.55 -> 11.85 ms (1024 walkers),
// 30 electrons FP32 49.5 -> 46.5 ms (256); bitwise the same.
template <typename TN, int SX>
void launch_net_tangent_adj_w(const pn_ctx* c, hipStream_t s, int64_t nw, const double* r, const TN* P, char* ws,
                            const WsLayout& L) {
  switch (L.T + 1) {
    case 2: launch_ta_c<TN, 2, SX>(c, s, nw, r, P, ws, L); break;
    case 3: launch_ta_c<TN, 3, SX>(c, s, nw, r, P, ws, L); break;
    case 4: launch_ta_c<TN, 4, SX>(c, s, nw, r, P, ws, L); break;
    case 5: launch_ta_c<TN, 5, SX>(c, s, nw, r, P, ws, L); break;
    case 6: launch_ta_c<TN, 6, SX>(c, s, nw, r, P, ws, L); break;
    case 7: launch_ta_c<TN, 7, SX>(c, s, nw, r, P, ws, L); break;
    default: break;  // the planner only picks T in 1..6 for the full adjoint
  }
}

}  // namespace pn

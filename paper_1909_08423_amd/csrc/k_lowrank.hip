// Multideterminant expansion through one LU per spin (all FP64).
//
// The expansion sum_p c_p det A_p^up det A_p^down (Results, eq. "ansatz")
// has members that differ from the first determinant in a few orbitals.
// Write A_0 for the first determinant's matrix of one spin, G_0 = A_0^{-1}
// and Theta = Phi~ G_0 (rows: the orbitals occupied in some determinant but
// not in the first, "virtual rows"; columns: the first determinant's slots).
// If determinant p replaces the orbitals of slots h_1..h_k by v_1..v_k, the
// matrix determinant lemma gives
//
//   det A_p = s_p det A_0 det D_p,   D_p[j][l] = Theta[v_j][h_l]   (k x k),
//
// with s_p the sign of the row order.  For a coordinate a, with
// T_a = d_a Phi~ (the table derivative), B_a = T_a G_0 and N_a = the first
// determinant's rows of B_a (= d_a A_0 G_0):
//
//   d_a ln det A_0 = tr N_a,        Xi_a = d_a Theta = B_a - Theta N_a,
//   d_a ln det D_p = tr(D_p^{-1} Xi_a[v][h]),
//
// and with L the Laplacian of the table, Lambda = L G_0 and S = sum_a Xi_a N_a:
//
//   lap ln det A_0 = tr Lambda[occ] - sum_a tr(N_a^2),
//   sum_a d2_a Theta = Lambda - Theta Lambda[occ] - 2 S,
//   lap ln det D_p = tr(D_p^{-1} (sum_a d2_a Theta)[v][h])
//                    - sum_a tr((D_p^{-1} Xi_a[v][h])^2).
//
// The per-coordinate work is one product T_a G_0 per spin instead of one
// per determinant.  The formulas divide by det A_0 through G_0: a walker
// whose first determinant is singular, or small against another member
// (|det D_p| > kRatioMax), is handed to the direct per-determinant kernels
// through a device-side list.
//
//  k_lr_value    one wavefront per (walker, spin): Theta, each D_p, its
//                determinant and inverse (Gauss-Jordan in registers), the
//                members' (ln|det|, sign) in the direct path's layout, and
//                the hand-back flag.
//  k_lr_list     one block per tile: the flagged walkers, ascending, and
//                their count.
//  k_lr_tangent  one block per walker, over the coordinate chunks of the
//                network tangent pass: the table derivatives, B_a and Xi_a,
//                the members' gradients, the determinant sum per coordinate
//                (as in the direct path), then the Laplacian terms; writes
//                the gradient and the walker's Laplacian / |grad|^2 partials.
#include <math.h>

#include <type_traits>

#include <algorithm>

#include "pn_internal.h"

namespace pn {
namespace {

constexpr int kWaves = kThreads / 64;
constexpr double kRatioMax = 1e4;

__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// In-place inverse of the leading k x k block of a (identity beyond it) by
// Gauss-Jordan elimination with partial pivoting (largest |a[r][c]|, ties to
// the lowest row); returns the determinant, 0 for a singular block (a is then
// undefined).
__device__ __forceinline__ double gj_inverse(double (&a)[kMaxExc][kMaxExc], int k) {
  int piv[kMaxExc];
  double det = 1.0;
#pragma unroll
  for (int c = 0; c < kMaxExc; ++c) {
    int bi = c;
    double best = fabs(a[c][c]);
#pragma unroll
    for (int r = c + 1; r < kMaxExc; ++r) {
      const double v = fabs(a[r][c]);
      if (r < k && v > best) {
        best = v;
        bi = r;
      }
    }
    piv[c] = bi;
    if (bi != c) det = -det;
#pragma unroll
    for (int r = c + 1; r < kMaxExc; ++r) {
      if (r == bi) {
#pragma unroll
        for (int col = 0; col < kMaxExc; ++col) {
          const double tmp = a[c][col];
          a[c][col] = a[r][col];
          a[r][col] = tmp;
        }
      }
    }
    const double pv = a[c][c];
    if (pv == 0.0) return 0.0;
    det *= pv;
    const double inv = 1.0 / pv;
    a[c][c] = 1.0;
#pragma unroll
    for (int col = 0; col < kMaxExc; ++col) a[c][col] *= inv;
#pragma unroll
    for (int r = 0; r < kMaxExc; ++r) {
      if (r == c) continue;
      const double f = a[r][c];
      a[r][c] = 0.0;
#pragma unroll
      for (int col = 0; col < kMaxExc; ++col) a[r][col] -= f * a[c][col];
    }
  }
#pragma unroll
  for (int c = kMaxExc - 1; c >= 0; --c) {
#pragma unroll
    for (int col = c + 1; col < kMaxExc; ++col) {
      if (piv[c] == col) {
#pragma unroll
        for (int r = 0; r < kMaxExc; ++r) {
          const double tmp = a[r][c];
          a[r][c] = a[r][col];
          a[r][col] = tmp;
        }
      }
    }
  }
  return det;
}

__device__ __forceinline__ int theta_size(const Dims& d) { return d.nv[0] * d.n_up + d.nv[1] * d.n_dn; }

__global__ __launch_bounds__(kThreads) void k_lr_value(Dims d, DevTables t, int64_t nw,
                                                       const double* __restrict__ phi,
                                                       const double* __restrict__ fval,
                                                       const double* __restrict__ g0,
                                                       const double* __restrict__ ld0,
                                                       double* __restrict__ theta, double* __restrict__ dinv,
                                                       double* __restrict__ ldet, int* __restrict__ flag) {
  extern __shared__ __align__(16) double lsm[];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int64_t task = (int64_t)blockIdx.x * kWaves + wv;
  if (task >= nw * 2) return;
  const int64_t w = task >> 1;
  const int s = (int)(task & 1);
  const int n = s ? d.n_dn : d.n_up, e0 = s ? d.n_up : 0, nv = s ? d.nv[1] : d.nv[0];
  const int N = d.N, M = d.M, P = d.P;
  const int gsz = d.n_up * d.n_up + d.n_dn * d.n_dn;
  const int nvmax = max(d.nv[0], d.nv[1]), nmax = max(d.n_up, d.n_dn);
  double* ts = lsm + (size_t)wv * nvmax * nmax;
  if (n == 0) {
    for (int p = lane; p < P; p += 64) {
      ldet[((w * P + p) * 2 + s) * 2] = 0.0;
      ldet[((w * P + p) * 2 + s) * 2 + 1] = 1.0;
    }
    if (lane == 0) flag[w * 2 + s] = 0;
    return;
  }
  const double* G = g0 + w * gsz + (s ? d.n_up * d.n_up : 0);
  const double l0 = ld0[(w * 2 + s) * 2], s0 = ld0[(w * 2 + s) * 2 + 1];
  const bool ref_ok = l0 > -INFINITY;
  double* Th = theta + w * theta_size(d) + (s ? d.nv[0] * d.n_up : 0);
  if (ref_ok) {
    const double* ph = phi + w * N * M * 7;
    const double* fv = fval + w * N * M;
    for (int q = lane; q < nv * n; q += 64) {
      const int v = q / n, k = q % n, orb = t.lr_vorb[s * M + v];
      double acc = 0.0;
      for (int i = 0; i < n; ++i) {
        const size_t e = (size_t)(e0 + i) * M + orb;
        acc += ph[e * 7] * fv[e] * G[i * n + k];
      }
      Th[q] = acc;
      ts[q] = acc;
    }
  }
  wave_sync();
  bool bad = !ref_ok;
  for (int p = lane; p < P; p += 64) {
    const int k = t.lr_k[p * 2 + s];
    double* di = dinv + ((w * P + p) * 2 + s) * (kMaxExc * kMaxExc);
    double lnd = 0.0, sd = 1.0;
    if (!ref_ok) {
      lnd = -INFINITY;
      sd = 0.0;
    } else if (k > 0) {
      const int* hl = t.lr_hole + (p * 2 + s) * kMaxExc;
      const int* pt = t.lr_part + (p * 2 + s) * kMaxExc;
      double a[kMaxExc][kMaxExc];
#pragma unroll
      for (int j = 0; j < kMaxExc; ++j)
#pragma unroll
        for (int l = 0; l < kMaxExc; ++l)
          a[j][l] = (j < k && l < k) ? ts[pt[j] * n + hl[l]] : (j == l ? 1.0 : 0.0);
      const double det = gj_inverse(a, k);
      if (det == 0.0) {
        lnd = -INFINITY;
        sd = 0.0;
#pragma unroll
        for (int q = 0; q < kMaxExc * kMaxExc; ++q) di[q] = 0.0;
      } else {
        lnd = log(fabs(det));
        sd = det > 0 ? 1.0 : -1.0;
        if (fabs(det) > kRatioMax) bad = true;
#pragma unroll
        for (int j = 0; j < kMaxExc; ++j)
#pragma unroll
          for (int l = 0; l < kMaxExc; ++l) di[j * kMaxExc + l] = a[j][l];
      }
    }
    ldet[((w * P + p) * 2 + s) * 2] = l0 + lnd;
    ldet[((w * P + p) * 2 + s) * 2 + 1] = s0 * sd * t.lr_sign[p * 2 + s];
  }
  const unsigned long long any_bad = __ballot(bad);
  if (lane == 0) flag[w * 2 + s] = any_bad ? 1 : 0;
}

// The walkers of the tile with either spin flagged, ascending, in list[0..],
// and their count in list[nw] (one block of 1024 threads).
__global__ __launch_bounds__(1024) void k_lr_list(int64_t nw, const int* __restrict__ flag, int* __restrict__ list) {
  __shared__ int scan[1024];
  __shared__ int base;
  if (threadIdx.x == 0) base = 0;
  __syncthreads();
  for (int64_t w0 = 0; w0 < nw; w0 += 1024) {
    const int64_t w = w0 + threadIdx.x;
    const int f = (w < nw) ? ((flag[2 * w] | flag[2 * w + 1]) ? 1 : 0) : 0;
    scan[threadIdx.x] = f;
    __syncthreads();
    for (int o = 1; o < 1024; o <<= 1) {
      const int v = threadIdx.x >= (unsigned)o ? scan[threadIdx.x - o] : 0;
      __syncthreads();
      scan[threadIdx.x] += v;
      __syncthreads();
    }
    if (f) list[base + scan[threadIdx.x] - 1] = (int)w;
    __syncthreads();
    if (threadIdx.x == 1023) base += scan[1023];
    __syncthreads();
  }
  if (threadIdx.x == 0) list[nw] = base;
}

// Element offsets of the tangent kernel's LDS regions (doubles, then ints).
struct LrLds {
  int gsz, thsz, bsz, R0, R1;
  size_t G0, TH, TB, LT, BM, SS, YY, TRN, TRN2, GPA, QACC, DELTA, DINV, WD, LAPC, SQC, SCAL, PF, n_dbl;
  size_t ROWORB, n_int;
};

__host__ __device__ inline LrLds lr_lds(const Dims& d, int T) {
  LrLds o{};
  o.gsz = d.n_up * d.n_up + d.n_dn * d.n_dn;
  o.thsz = d.nv[0] * d.n_up + d.nv[1] * d.n_dn;
  o.R0 = d.n_up + d.nv[0];
  o.R1 = d.n_dn + d.nv[1];
  o.bsz = o.R0 * d.n_up + o.R1 * d.n_dn;
  size_t off = 0;
  auto take = [&](size_t n) {
    size_t r = off;
    off += (n + 1) & ~size_t(1);  // keep 16-byte alignment
    return r;
  };
  o.G0 = take(o.gsz);
  o.TH = take(o.thsz);
  o.TB = take((size_t)T * d.M * d.N);
  o.LT = take((size_t)d.M * d.N);
  o.BM = take((size_t)T * o.bsz);
  o.SS = take(o.thsz);
  o.YY = take(o.thsz);
  o.TRN = take((size_t)T * 2);
  o.TRN2 = take((size_t)T * 2);
  o.GPA = take((size_t)d.P * T * 2);
  o.QACC = take((size_t)d.P * 2);
  o.DELTA = take(d.P);
  o.DINV = take((size_t)d.P * 2 * kMaxExc * kMaxExc);
  o.WD = take(d.P);
  o.LAPC = take(T);
  o.SQC = take(T);
  o.SCAL = take(8);
  o.PF = take((size_t)2 * d.N * d.M);
  o.n_dbl = off;
  o.ROWORB = 0;
  o.n_int = o.R0 + o.R1;
  return o;
}

// NB: the spins' largest electron number where it is at most 8 (4 stands for
// less): an item of steps 2 and 3 is then one row with all its slots, sums in
// registers, every operand requested before the first is used.  NB = 0 for
// larger spins: kSL consecutive slots of one row.
// WIDE: spins of 8 or more electrons, blocks of over 40 KB of LDS (at most
// two per CU, so a wave may hold up to 256 registers): the next chunk's
// tangents of the first kItems step-1 items requested a chunk ahead.
// Otherwise at most 128 registers (four blocks per CU), requested at the start of the step.
//
// At these sizes (ten electrons, 16 members: 20 k multiply-adds per chunk) a
// block waits for latency, not for arithmetic: what counts is the number of
// dependent LDS and cache round trips between two barriers and the index
// arithmetic around them, so there is no runtime division in the chunk loop,
// the Laplacian's terms of a coordinate's own electron are items of their own
// (among the others they held every wave up), the sums over rows and members
// run on as many lanes as they have terms instead of a wave each, and members
// replacing at most two orbitals of a spin work on 2 x 2 blocks.  Measured
// against the form without these: 4096 walkers of ten electrons with 16
// members 0.50 -> 0.20 ms, 1001 of them 0.138 -> 0.080 ms, 2048 of seven
// electrons 0.151 -> 0.100 ms, a launch of the 30-electron diatomic's large
// batch with 64 members 3.6 -> 2.35 ms.
constexpr int kSL = 4;
constexpr int kItems = 8;  // step-1 items per thread with their tangents in registers

// The sum over the 64 lanes of a wave whose lanes from width on hold zeros,
// in the order of the full butterfly.
__device__ __forceinline__ double sum_lanes(double v, int width) {
  for (int off = width >> 1; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}
__device__ __forceinline__ int pow2_lanes(int n) { return n <= 1 ? 1 : min(64, 1 << (32 - __builtin_clz((unsigned)(n - 1)))); }

// KX: members replace at most KX orbitals of a spin (2 or kMaxExc).
template <int NB, bool WIDE, int KX>
__global__ __launch_bounds__(kThreads, WIDE ? 2 : 4) void k_lr_tangent(Dims d, DevTables t, int64_t nw, int T, int n_chunks,
                                                         const double* __restrict__ geo,
                                                         const double* __restrict__ phi,
                                                         const double* __restrict__ fval,
                                                         const double* __restrict__ ftan,
                                                         const double* __restrict__ jtan,
                                                         const double* __restrict__ g0,
                                                         const double* __restrict__ theta,
                                                         const double* __restrict__ dinv,
                                                         const double* __restrict__ wdet,
                                                         const int* __restrict__ flag, double* __restrict__ grad,
                                                         double* __restrict__ partial) {
  extern __shared__ __align__(16) double sm[];
  const int64_t w = blockIdx.x;
  if (w >= nw || (flag[2 * w] | flag[2 * w + 1])) return;  // the direct path takes this walker
  const LrLds o = lr_lds(d, T);
  const int N = d.N, M = d.M, P = d.P, nu = d.n_up, nd = d.n_dn;
  const int tid = threadIdx.x;
  constexpr int nth = kThreads;
  double* G0s = sm + o.G0;
  double* THs = sm + o.TH;
  double* TB = sm + o.TB;      // [T][N][M] table derivatives of the chunk (orbital fastest)
  double* LT = sm + o.LT;      // [M][N] Laplacian of the table, summed over chunks
  double* BM = sm + o.BM;      // [T][bsz] B_a rows (first determinant's, then virtual) per spin
  double* SS = sm + o.SS;      // [thsz] S = sum_a Xi_a N_a
  double* YY = sm + o.YY;      // [thsz] sum_a d2_a Theta on the virtual rows
  double* TRN = sm + o.TRN;    // [T][2] tr N_a
  double* TRN2 = sm + o.TRN2;  // [T][2] tr N_a^2
  double* GPA = sm + o.GPA;    // [P][T][2] d_a ln|D_p|, each spin's minor
  double* QACC = sm + o.QACC;  // [P][2] sum_a tr((D^-1 Xi_a)^2), each spin
  double* DELTA = sm + o.DELTA;
  double* DI = sm + o.DINV;    // [P][2][kMaxExc^2]
  double* WD = sm + o.WD;      // [P]
  double* LAPC = sm + o.LAPC;
  double* SQC = sm + o.SQC;
  double* SCAL = sm + o.SCAL;  // lap, |grad|^2, sum tr N^2 (up, down), tr Lambda[occ] (up, down)
  double* PF = sm + o.PF;      // [2][N][M] phi_mu(r_i) and f_{i mu} of the walker
  int* ROWORB = reinterpret_cast<int*>(sm + o.n_dbl);

  const int gsz = o.gsz, thsz = o.thsz, bsz = o.bsz;
  const int sB1 = o.R0 * nu, sT1 = d.nv[0] * nu;  // offsets of the down-spin rows
  auto soffB = [&](int s) { return s ? sB1 : 0; };
  auto soffT = [&](int s) { return s ? sT1 : 0; };
  auto ns = [&](int s) { return s ? nd : nu; };
  auto e0s = [&](int s) { return s ? nu : 0; };

  for (int q = tid; q < gsz; q += nth) G0s[q] = g0[w * gsz + q];
  for (int q = tid; q < thsz; q += nth) {
    THs[q] = theta[w * thsz + q];
    SS[q] = 0.0;
  }
  for (int q = tid; q < M * N; q += nth) LT[q] = 0.0;
  for (int q = tid; q < P * 2 * kMaxExc * kMaxExc; q += nth) DI[q] = dinv[w * P * 2 * kMaxExc * kMaxExc + q];
  for (int q = tid; q < P; q += nth) {
    WD[q] = wdet[w * P + q];
    QACC[2 * q] = QACC[2 * q + 1] = 0.0;
  }
  for (int q = tid; q < o.R0 + o.R1; q += nth) {
    const int s = q >= o.R0, r = s ? q - o.R0 : q, n = ns(s);
    ROWORB[q] = r < n ? (s ? t.det_dn[r] : t.det_up[r]) : t.lr_vorb[s * M + (r - n)];
  }
  if (tid < 8) SCAL[tid] = 0.0;
  for (int q = tid; q < N * M; q += nth) {
    PF[q] = phi[((size_t)w * N * M + q) * 7];
    PF[N * M + q] = fval[(size_t)w * N * M + q];
  }
  // offsets of Xi[v][h] in a spin's rows, in the third row of the member's
  // inverse (an identity row that nothing reads)
  if constexpr (KX == 2) {
    __syncthreads();
    for (int q = tid; q < 2 * P; q += nth) {
      const int s = q & 1, n = ns(s), k = t.lr_k[q];
      int* off = reinterpret_cast<int*>(DI + q * kMaxExc * kMaxExc + 2 * kMaxExc);
      for (int j = 0; j < 2; ++j)
        for (int l = 0; l < 2; ++l)
          off[2 * j + l] = (j < k && l < k) ? (n + t.lr_part[q * kMaxExc + j]) * n + t.lr_hole[q * kMaxExc + l] : -1;
    }
  }
  __syncthreads();

  const double* ph = phi + w * N * M * 7;
  const double* g = geo + w * kGeoStride(N);
  const int Tp = T + 1, NTM = N * Tp * M;
  // the items' (i, column, mu) of step 1, the same in every chunk: those of the
  // first kItems decoded once (M <= 128 and columns <= 17 fit their 8-bit
  // fields), the others' from the last by adding nth in these digits
  constexpr int kHeld = WIDE ? kItems : 0;
  double ftv[kItems];
  int pk[kItems];
  const int nth_i = nth / (Tp * M), nth_c = (nth / M) % Tp, nth_m = nth % M;
  auto advance = [&](int& i, int& col, int& mu) {
    mu += nth_m;
    col += nth_c;
    i += nth_i;
    if (mu >= M) {
      mu -= M;
      ++col;
    }
    if (col >= Tp) {
      col -= Tp;
      ++i;
    }
  };
  int i8, c8, m8;  // the item after the last of pk
  {
    int i = tid / (Tp * M), col = (tid / M) % Tp, mu = tid % M;
#pragma unroll
    for (int u = 0; u < kHeld; ++u) {
      pk[u] = (i << 16) | (col << 8) | mu;
      advance(i, col, mu);
    }
    i8 = i;
    c8 = col;
    m8 = mu;
  }
  auto request = [&](const double* f) {
#pragma unroll
    for (int u = 0; u < kItems; ++u) ftv[u] = f[min(tid + u * nth, NTM - 1)];
  };
  if constexpr (WIDE) request(ftan + (size_t)w * n_chunks * NTM);
  // the (column, row) that a thread starts with in steps 2 and 3
  const int nr2 = NB ? o.R0 + o.R1 : o.R0 * ((nu + kSL - 1) / kSL) + o.R1 * ((nd + kSL - 1) / kSL);
  const int nr3 = NB ? d.nv[0] + d.nv[1] : d.nv[0] * ((nu + kSL - 1) / kSL) + d.nv[1] * ((nd + kSL - 1) / kSL);
  const int col2 = tid / nr2, rem2 = tid - col2 * nr2;
  const int col3 = nr3 ? tid / nr3 : 0, rem3 = tid - col3 * nr3;
  const int nmx = max(nu, nd), lanes_n = pow2_lanes(nmx), lanes_p = pow2_lanes(P);
  for (int chunk = 0; chunk < n_chunks; ++chunk) {
    const int a0 = chunk * T, Tc = min(T, 3 * N - a0);
    const double* ft = ftan + ((size_t)w * n_chunks + chunk) * NTM;
    const double* jt = jtan + ((size_t)w * n_chunks + chunk) * Tp;
    // 1. table derivatives T_a[mu][i] and the chunk's part of the table
    //    Laplacian, the former read in the memory order of the network
    //    tangents
    {
      auto put = [&](int i, int col, int mu, double f) {  // coordinates of other electrons
        if (col < Tc && (unsigned)(a0 + col - 3 * i) >= 3u) TB[(col * N + i) * M + mu] = PF[i * M + mu] * f;
      };
#pragma unroll
      for (int u = 0; u < kHeld; ++u) {
        if (tid + u * nth < NTM) put(pk[u] >> 16, (pk[u] >> 8) & 255, pk[u] & 255, ftv[u]);
      }
      int i = i8, col = c8, mu = m8;
      for (int q = tid + kHeld * nth; q < NTM; q += kItems * nth) {
        double f[kItems];
#pragma unroll
        for (int u = 0; u < kItems; ++u) f[u] = ft[min(q + u * nth, NTM - 1)];
#pragma unroll
        for (int u = 0; u < kItems; ++u) {
          if (q + u * nth < NTM) put(i, col, mu, f[u]);
          advance(i, col, mu);
        }
      }
      for (int q = tid; q < N * M; q += nth) {  // an electron's own coordinates, and the Laplacian
        const int i = q / M, mu = q - i * M;
        const double* pj = ph + (size_t)q * 7;
        const double* fi = ft + (size_t)i * Tp * M + mu;
        const double p0 = PF[q], f = PF[N * M + q];
        double v = p0 * fi[(size_t)T * M];
#pragma unroll
        for (int al = 0; al < 3; ++al) {
          const int c = 3 * i + al - a0;
          if ((unsigned)c >= (unsigned)Tc) continue;
          const double fc = fi[(size_t)c * M];
          TB[(c * N + i) * M + mu] = fma(pj[1 + al], f, p0 * fc);
          v += fma(pj[4 + al], f, 2.0 * pj[1 + al] * fc);
        }
        LT[mu * N + i] += v;
      }
      if constexpr (WIDE) {
        if (chunk + 1 < n_chunks) request(ft + NTM);  // the next chunk's tangents follow this chunk's
      }
    }
    __syncthreads();
    // 2. B_a = T_a G_0 on the first determinant's rows and the virtual rows
    {
      int col = col2, rem = rem2;
      for (; col < Tc;) {
        if constexpr (NB > 0) {
          const int s = rem >= o.R0, n = ns(s);
          const double* tb = TB + (col * N + e0s(s)) * M + ROWORB[rem];
          const double* Gs = G0s + (s ? nu * nu : 0);
          double* B = BM + col * bsz + soffB(s) + (rem - (s ? o.R0 : 0)) * n;
          double x[NB], acc[NB];
#pragma unroll
          for (int i = 0; i < NB; ++i) {
            x[i] = i < n ? tb[i * M] : 0.0;
            acc[i] = 0.0;
          }
#pragma unroll
          for (int i = 0; i < NB; ++i)
#pragma unroll
            for (int k = 0; k < NB; ++k)
              if (i < n && k < n) acc[k] += x[i] * Gs[i * n + k];
#pragma unroll
          for (int k = 0; k < NB; ++k)
            if (k < n) B[k] = acc[k];
        } else {
          const int nq0 = o.R0 * ((nu + kSL - 1) / kSL);
          const int s = rem >= nq0, rq = rem - (s ? nq0 : 0), n = ns(s), nks = (n + kSL - 1) / kSL;
          const int r = rq / nks, k0 = (rq - r * nks) * kSL;
          const double* tb = TB + (col * N + e0s(s)) * M + ROWORB[s * o.R0 + r];
          const double* Gs = G0s + (s ? nu * nu : 0);
          double acc[kSL];
#pragma unroll
          for (int u = 0; u < kSL; ++u) acc[u] = 0.0;
          for (int i = 0; i < n; ++i) {
            const double x = tb[i * M];
#pragma unroll
            for (int u = 0; u < kSL; ++u) acc[u] += x * Gs[i * n + min(k0 + u, n - 1)];
          }
          double* B = BM + col * bsz + soffB(s) + r * n;
#pragma unroll
          for (int u = 0; u < kSL; ++u)
            if (k0 + u < n) B[k0 + u] = acc[u];
        }
        for (rem += nth; rem >= nr2; rem -= nr2) ++col;
      }
    }
    __syncthreads();
    // 3. Xi_a = B_a - Theta N_a on the virtual rows (in place), and tr N_a,
    //    tr N_a^2 per (coordinate, spin), a lane per row, summed across the
    //    lanes in a fixed order
    {
      int col = col3, rem = rem3;
      for (; nr3 > 0 && col < Tc;) {
        if constexpr (NB > 0) {
          const int s = rem >= d.nv[0], n = ns(s), v = rem - (s ? d.nv[0] : 0);
          double* B = BM + col * bsz + soffB(s);
          const double* th = THs + soffT(s) + v * n;
          double x[NB], acc[NB];
#pragma unroll
          for (int k = 0; k < NB; ++k) {
            x[k] = k < n ? th[k] : 0.0;
            acc[k] = k < n ? B[(n + v) * n + k] : 0.0;
          }
#pragma unroll
          for (int l = 0; l < NB; ++l)
#pragma unroll
            for (int k = 0; k < NB; ++k)
              if (l < n && k < n) acc[k] -= x[l] * B[l * n + k];
#pragma unroll
          for (int k = 0; k < NB; ++k)
            if (k < n) B[(n + v) * n + k] = acc[k];
        } else {
          const int nq0 = d.nv[0] * ((nu + kSL - 1) / kSL);
          const int s = rem >= nq0, rq = rem - (s ? nq0 : 0), n = ns(s), nks = (n + kSL - 1) / kSL;
          const int v = rq / nks, k0 = (rq - v * nks) * kSL;
          double* B = BM + col * bsz + soffB(s);
          const double* th = THs + soffT(s) + v * n;
          double acc[kSL];
#pragma unroll
          for (int u = 0; u < kSL; ++u) acc[u] = B[(n + v) * n + min(k0 + u, n - 1)];
          for (int l = 0; l < n; ++l) {
            const double x = th[l];
#pragma unroll
            for (int u = 0; u < kSL; ++u) acc[u] -= x * B[l * n + min(k0 + u, n - 1)];
          }
#pragma unroll
          for (int u = 0; u < kSL; ++u)
            if (k0 + u < n) B[(n + v) * n + k0 + u] = acc[u];
        }
        for (rem += nth; rem >= nr3; rem -= nr3) ++col;
      }
      const int sh = log2_of(lanes_n), lane = tid & (lanes_n - 1);
      for (int cs = tid >> sh; cs < ((Tc * 2 + (nth >> sh) - 1) & ~((nth >> sh) - 1)); cs += nth >> sh) {
        const int col = min(cs >> 1, Tc - 1), s = cs & 1, n = ns(s);
        const double* B = BM + col * bsz + soffB(s);
        double tr = 0.0, tr2 = 0.0;
        if (lane < n) {
          tr = B[lane * n + lane];
#pragma unroll 4
          for (int l = 0; l < n; ++l) tr2 += B[lane * n + l] * B[l * n + lane];
        }
        tr = sum_lanes(tr, lanes_n);
        tr2 = sum_lanes(tr2, lanes_n);
        if (lane == 0 && cs < Tc * 2) {
          TRN[cs] = tr;
          TRN2[cs] = tr2;
        }
      }
    }
    __syncthreads();
    // 4. S += sum_a Xi_a N_a (virtual rows x all slots), and per member
    //    d_a ln|D_p| = tr(D_p^-1 Xi_a[v][h]) and tr((D_p^-1 Xi_a[v][h])^2),
    //    members from the next whole wave on
    const int th64 = (thsz + 63) & ~63;
    for (int q = tid; q < th64 + 2 * P; q += nth) {
      if (q < th64) {
        if (q >= thsz) continue;
        const int s = q >= sT1, rr = q - soffT(s), n = ns(s);
        const int v = rr / n, h = rr - v * n;
        double acc = SS[q];
        for (int col = 0; col < Tc; ++col) {
          const double* B = BM + col * bsz + soffB(s);
          if constexpr (NB > 0) {
            double x[NB], y[NB];
#pragma unroll
            for (int k = 0; k < NB; ++k) {
              if (k < n) {
                x[k] = B[(n + v) * n + k];
                y[k] = B[k * n + h];
              }
            }
#pragma unroll
            for (int k = 0; k < NB; ++k)
              if (k < n) acc += x[k] * y[k];
          } else {
#pragma unroll 4
            for (int k = 0; k < n; ++k) acc += B[(n + v) * n + k] * B[k * n + h];
          }
        }
        SS[q] = acc;
        continue;
      }
      const int ps = q - th64, p = ps >> 1, s = ps & 1, n = ns(s);
      const double* Di = DI + ps * kMaxExc * kMaxExc;
      double qsum = QACC[ps];
      if constexpr (KX == 2) {
        const int* off = reinterpret_cast<const int*>(Di + 2 * kMaxExc);
        const int o00 = off[0], o01 = off[1], o10 = off[2], o11 = off[3];
        const double d00 = Di[0], d01 = Di[1], d10 = Di[kMaxExc], d11 = Di[kMaxExc + 1];
#pragma unroll 3
        for (int col = 0; col < Tc; ++col) {
          double gp = 0.0;
          if (o00 >= 0) {
            const double* B = BM + col * bsz + soffB(s);
            const double x00 = B[o00], x01 = o01 >= 0 ? B[o01] : 0.0, x10 = o10 >= 0 ? B[o10] : 0.0,
                         x11 = o11 >= 0 ? B[o11] : 0.0;
            const double m00 = fma(d01, x10, d00 * x00), m01 = fma(d01, x11, d00 * x01);
            const double m10 = fma(d11, x10, d10 * x00), m11 = fma(d11, x11, d10 * x01);
            gp = m00 + m11;
            qsum = fma(m00, m00, qsum);
            qsum = fma(m01, m10, qsum);
            qsum = fma(m10, m01, qsum);
            qsum = fma(m11, m11, qsum);
          }
          GPA[(p * T + col) * 2 + s] = gp;
        }
      } else {
        const int k = t.lr_k[ps];
        const int* hl = t.lr_hole + ps * kMaxExc;
        const int* pt = t.lr_part + ps * kMaxExc;
        for (int col = 0; col < Tc; ++col) {
          double gp = 0.0;
          if (k > 0) {
            const double* B = BM + col * bsz + soffB(s);
            double X[kMaxExc][kMaxExc], Mx[kMaxExc][kMaxExc];
#pragma unroll
            for (int j = 0; j < kMaxExc; ++j)
#pragma unroll
              for (int l = 0; l < kMaxExc; ++l) X[j][l] = (j < k && l < k) ? B[(n + pt[j]) * n + hl[l]] : 0.0;
#pragma unroll
            for (int l = 0; l < kMaxExc; ++l)
#pragma unroll
              for (int l2 = 0; l2 < kMaxExc; ++l2) {
                double acc = 0.0;
#pragma unroll
                for (int j = 0; j < kMaxExc; ++j) acc += Di[l * kMaxExc + j] * X[j][l2];
                Mx[l][l2] = acc;
              }
#pragma unroll
            for (int l = 0; l < kMaxExc; ++l) {
              gp += Mx[l][l];
#pragma unroll
              for (int l2 = 0; l2 < kMaxExc; ++l2) qsum += Mx[l][l2] * Mx[l2][l];
            }
          }
          GPA[(p * T + col) * 2 + s] = gp;
        }
      }
      QACC[ps] = qsum;
    }
    __syncthreads();
    // 5. determinant sum per coordinate (lanes over members, summed across
    //    the lanes in a fixed order), gamma and J
    {
      const int sh = log2_of(lanes_p), lane = tid & (lanes_p - 1), cols = nth >> sh;
      for (int c = tid >> sh; c < (Tc + cols - 1) / cols * cols; c += cols) {
        const int col = min(c, Tc - 1), a = a0 + col, k = a / 3, al = a - 3 * k;
        const double trn = TRN[col * 2] + TRN[col * 2 + 1];
        double gj = 0.0, gl = 0.0, jc = 0.0;
        if (lane == 0) {
          gj = g[4 + 6 * k + al];
          gl = g[4 + 6 * k + 3 + al];
          jc = jt[col];
        }
        double dpsi = 0.0, wsq = 0.0;
        for (int p = lane; p < P; p += 64) {
          const double gp = trn + GPA[(p * T + col) * 2] + GPA[(p * T + col) * 2 + 1];
          dpsi += WD[p] * gp;
          wsq += WD[p] * gp * gp;
        }
        dpsi = sum_lanes(dpsi, lanes_p);
        wsq = sum_lanes(wsq, lanes_p);
        if (lane == 0 && c < Tc) {
          const double gtot = gj + jc + dpsi;
          grad[w * N * 3 + a] = gtot;
          LAPC[col] = wsq - dpsi * dpsi + gl;
          SQC[col] = gtot * gtot;
        }
      }
    }
    __syncthreads();
    if (tid < 4) {  // lap, |grad|^2, sum tr N^2 of either spin
      const double* x = tid == 0 ? LAPC : (tid == 1 ? SQC : TRN2 + (tid - 2));
      const int step = tid < 2 ? 1 : 2;
      double acc = SCAL[tid];
#pragma unroll 4
      for (int col = 0; col < Tc; ++col) acc += x[col * step];
      SCAL[tid] = tid == 0 ? acc + jt[T] : acc;
    }
    // the next chunk's first writes (TB, LT) are not read by these threads here,
    // and its TRN2 writes follow two more barriers
  }
  __syncthreads();
  // 6. Lambda = L G_0 on all rows (into the B buffer)
  for (int q = tid; q < bsz; q += nth) {
    const int s = q >= sB1, rr = q - soffB(s), n = ns(s);
    const int r = rr / n, k = rr % n;
    const double* lt = LT + (size_t)ROWORB[s * o.R0 + r] * N + e0s(s);
    const double* Gs = G0s + (s ? nu * nu : 0);
    double acc = 0.0;
    for (int i = 0; i < n; ++i) acc += lt[i] * Gs[i * n + k];
    BM[q] = acc;
  }
  __syncthreads();
  // 7. Y = Lambda[virtual] - Theta Lambda[occ] - 2 S; tr Lambda[occ]
  for (int q = tid; q < thsz + 2; q += nth) {
    if (q < thsz) {
      const int s = q >= sT1, rr = q - soffT(s), n = ns(s);
      const int v = rr / n, h = rr % n;
      const double* Lm = BM + soffB(s);
      const double* th = THs + soffT(s) + v * n;
      double acc = Lm[(n + v) * n + h] - 2.0 * SS[q];
      for (int l = 0; l < n; ++l) acc -= th[l] * Lm[l * n + h];
      YY[q] = acc;
    } else {
      const int s = q - thsz, n = ns(s);
      const double* Lm = BM + soffB(s);
      double tr = 0.0;
      for (int k = 0; k < n; ++k) tr += Lm[k * n + k];
      SCAL[4 + s] = tr;
    }
  }
  __syncthreads();
  // 8. each member's Laplacian of ln|det|, both spins
  for (int p = tid; p < P; p += nth) {
    double dl = SCAL[4] + SCAL[5] - SCAL[2] - SCAL[3] - QACC[2 * p] - QACC[2 * p + 1];
    for (int s = 0; s < 2; ++s) {
      const int k = t.lr_k[p * 2 + s];
      if (k == 0) continue;
      const int n = ns(s);
      const int* hl = t.lr_hole + (p * 2 + s) * kMaxExc;
      const int* pt = t.lr_part + (p * 2 + s) * kMaxExc;
      const double* Di = DI + (p * 2 + s) * kMaxExc * kMaxExc;
      const double* Y = YY + soffT(s);
      for (int l = 0; l < k; ++l)
        for (int j = 0; j < k; ++j) dl += Di[l * kMaxExc + j] * Y[pt[j] * n + hl[l]];
    }
    DELTA[p] = dl;
  }
  __syncthreads();
  double* pw = partial + (size_t)w * n_chunks * 2;
  for (int q = tid; q < n_chunks * 2; q += nth) {
    if (q >= 2) pw[q] = 0.0;
  }
  if (tid == 0) {
    double dl = 0.0;
#pragma unroll 8
    for (int p = 0; p < P; ++p) dl += WD[p] * DELTA[p];
    pw[0] = SCAL[0] + dl;
    pw[1] = SCAL[1];
  }
}

}  // namespace

size_t lowrank_tangent_lds_bytes(const Dims& d, int T) {
  const LrLds o = lr_lds(d, T);
  return o.n_dbl * sizeof(double) + o.n_int * sizeof(int);
}

void launch_lowrank_value(const pn_ctx* c, hipStream_t s, int64_t nw, char* ws, const WsLayout& L, double* logabs,
                          double* sign) {
  const Dims& d = c->d;
  double* g0 = reinterpret_cast<double*>(ws + L.g0);
  double* ld0 = reinterpret_cast<double*>(ws + L.ld0);
  int* flag = reinterpret_cast<int*>(ws + L.lrflag);
  int* list = reinterpret_cast<int*>(ws + L.lrlist);
  // 1. the first determinant's LU per spin
  Dims d1 = d;
  d1.P = 1;
  launch_slater_lu(c, d1, s, nw, ws, L, g0, ld0, nullptr, nullptr, (nw * 2 + kThreads - 1) / kThreads,
                   (nw * 2 + kWaves - 1) / kWaves);
  // 2. excitation table, members' minors, hand-back flags
  const size_t lds = (size_t)kWaves * std::max(d.nv[0], d.nv[1]) * std::max(d.n_up, d.n_dn) * sizeof(double);
  hipLaunchKernelGGL(k_lr_value, dim3((unsigned)((nw * 2 + kWaves - 1) / kWaves)), dim3(kThreads), lds, s, d, c->t,
                     nw, reinterpret_cast<const double*>(ws + L.phi), reinterpret_cast<const double*>(ws + L.fval), g0,
                     ld0, reinterpret_cast<double*>(ws + L.theta), reinterpret_cast<double*>(ws + L.dinv),
                     reinterpret_cast<double*>(ws + L.ldet), flag);
  // 3. the handed-back walkers go through the direct LU of every member
  hipLaunchKernelGGL(k_lr_list, dim3(1), dim3(1024), 0, s, nw, flag, list);
  const int64_t nmat = nw * d.P * 2;
  launch_slater_lu(c, d, s, nw, ws, L, reinterpret_cast<double*>(ws + L.ginv), reinterpret_cast<double*>(ws + L.ldet),
                   list, list + nw, std::min<int64_t>((nmat + kThreads - 1) / kThreads, kListGrid),
                   std::min<int64_t>((nmat + kWaves - 1) / kWaves, kListGrid));
  launch_combine_value(c, s, nw, ws, L, logabs, sign);
}

void launch_lowrank_tangent(const pn_ctx* c, hipStream_t s, int64_t nw, char* ws, const WsLayout& L, double* grad) {
  const Dims& d = c->d;
  const int* flag = reinterpret_cast<const int*>(ws + L.lrflag);
  const int* list = reinterpret_cast<const int*>(ws + L.lrlist);
  auto go = [&](auto kern) {
    if (L.lds_lr > 65536)
      (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)L.lds_lr);
    hipLaunchKernelGGL(kern, dim3((unsigned)nw), dim3(kThreads), L.lds_lr, s, d, c->t, nw, L.T, L.n_chunks,
                       reinterpret_cast<const double*>(ws + L.geo), reinterpret_cast<const double*>(ws + L.phi),
                       reinterpret_cast<const double*>(ws + L.fval), reinterpret_cast<const double*>(ws + L.ftan),
                       reinterpret_cast<const double*>(ws + L.jtan), reinterpret_cast<const double*>(ws + L.g0),
                       reinterpret_cast<const double*>(ws + L.theta), reinterpret_cast<const double*>(ws + L.dinv),
                       reinterpret_cast<const double*>(ws + L.wdet), flag, grad,
                       reinterpret_cast<double*>(ws + L.partial));
  };
  const int n = std::max(d.n_up, d.n_dn);
  auto pick = [&](auto kx_tag) {
    constexpr int KX = decltype(kx_tag)::value;
    if (n >= 8 && L.lds_lr > 40 * 1024)
      n == 8 ? go(&k_lr_tangent<8, true, KX>) : go(&k_lr_tangent<0, true, KX>);
    else if (n <= 4)
      go(&k_lr_tangent<4, false, KX>);
    else if (n <= 8)
      n == 5 ? go(&k_lr_tangent<5, false, KX>) : n == 6 ? go(&k_lr_tangent<6, false, KX>)
      : n == 7 ? go(&k_lr_tangent<7, false, KX>) : go(&k_lr_tangent<8, false, KX>);
    else
      go(&k_lr_tangent<0, false, KX>);
  };
  if (c->lr_kmax <= 2)
    pick(std::integral_constant<int, 2>());
  else
    pick(std::integral_constant<int, kMaxExc>());
  // the handed-back walkers: direct determinant tangents
  launch_slater_tangent(c, s, nw, nullptr, ws, L, grad, nullptr, list, list + nw);
}

}  // namespace pn

// Ritz step for bases of at most 112 columns (gfx950): the steps of ritz.hip with the matrix
// being factorised or reduced held in registers.
//
// What bounds it: one workgroup per problem slot runs two chains of q dependent steps (pivots,
// reflectors), a bisection and a back-transformation; the arithmetic (about 40 q^3 flops) is
// small, the latency of each step is everything.  So every step is kept short:
//  * thread (ty, tx) of a TY x 16 grid holds the entries (ty + TY a, tx + 16 b); a row of the
//    grid is one row of 16 lanes, so that sums over a matrix row are DPP adds;
//  * the pivoted Cholesky sweeps the whole matrix (Gauss-Jordan): the columns of pivots already
//    taken hold -L^{-1}'s rows in progress, so the pivot row that is broadcast at step k is also
//    row k of L^{-1} and Z needs no triangular inversion; every wave keeps the diagonal in its
//    lanes and finds the next pivot itself (value and index packed in one double), which leaves
//    one barrier per step;
//  * square roots and divisions are Newton-refined hardware reciprocals;
//  * blocks of rows or columns that are finished are skipped;
//  * eigenvalues: every thread counts at one point of a logarithmic grid first, then eight lanes
//    per eigenvalue bisect; the Sturm sequence is the determinant recurrence, one fused
//    multiply-add deep per row, on the matrix scaled by a power of two so that eight rows need
//    no overflow or underflow check;
//  * eigenvectors: two lanes per vector run the two factorisations of the twisted form at once;
//  * the back-transformation keeps the vectors in registers and loads the next reflector while
//    the current one is applied.
// One call takes 77 / 166 / 261 / 488 / 536 / 776 us at q = 24 / 48 / 64 / 84 / 96 / 112 for q / 2
// values, against 154 / 354 / 608 / 1018 / 1282 / 2140 us with the matrix in LDS or global memory
// and the steps of ritz.hip.  At q = 84: Cholesky 114 us, H' 70 (half of it the matrix cores' own
// time on one compute unit), reduction 171, eigenvalues 51, vectors 19, back-transformation 62.
// Beyond 96 columns the registers do not hold everything: 88 of a thread's values go to scratch.
#include "ritz_ops.h"

#include <type_traits>

namespace bl {

namespace {

// 1 / sqrt(x) from the hardware estimate and two Newton steps, for x well inside the range
__device__ __forceinline__ double rsq_nr(double x) {
  double r = __builtin_amdgcn_rsq(x);
  r = fma(0.5 * r, fma(-x * r, r, 1.0), r);
  r = fma(0.5 * r, fma(-x * r, r, 1.0), r);
  return r;
}

// Keeps a value loaded here in registers: selects on it stay selects (the compiler otherwise moves
// the load under a branch of its own, and the step waits for LDS once per value instead of once).
__device__ __forceinline__ void keep(c2& x) { asm volatile("" : "+v"(x.r), "+v"(x.i)); }

__device__ __forceinline__ double wave_max(double m) {
  m = fmax(m, dpp_d<kDppXor1>(m));
  m = fmax(m, dpp_d<kDppXor2>(m));
  m = fmax(m, dpp_d<kDppHalfMirror>(m));
  m = fmax(m, dpp_d<kDppMirror>(m));
  return fmax(fmax(readlane_d(m, 0), readlane_d(m, 16)), fmax(readlane_d(m, 32), readlane_d(m, 48)));
}

// A diagonal entry with its index (< 128) in the low mantissa bits: the larger double is the
// larger entry, ties (to 2^-45) to the smaller index.
__device__ __forceinline__ double pack_pivot(double d, int i) {
  const long long b = __builtin_bit_cast(long long, d);
  return __builtin_bit_cast(double, (b & ~127LL) | (long long)(127 - i));
}

// Number of eigenvalues below x of the real symmetric tridiagonal (d, e) with entries of at most
// one in size, from the signs of the leading minors p_i of T - x I:
// p_{i+1} = (d_i - x) p_i - e_{i-1}^2 p_{i-1}.  e2 holds the squares, none below 1e-40 (an
// exact zero minor then passes its neighbour's sign on); a pair of minors shrinks by at most
// 1e-160 in eight rows and, |x| being at most four, grows by at most (1 + 4 + 1)^8, after which it is
// rescaled.  (A larger x would overflow between two rescalings.)
__device__ __forceinline__ int sturm_scaled(const double* d, const double* e2, int r, double x) {
  double pm = 1.0, p = d[0] - x;
  int c = p < 0 ? 1 : 0;
  auto row = [&](double di, double ei) {
    const double pn = fma(di - x, p, -(ei * pm));
    c += ((__builtin_bit_cast(long long, pn) ^ __builtin_bit_cast(long long, p)) < 0) ? 1 : 0;
    pm = p;
    p = pn;
  };
  int i = 1;
  for (; i + 8 <= r; i += 8) {
    double dv[8], ev[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      dv[u] = d[i + u];
      ev[u] = e2[i - 1 + u];
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) row(dv[u], ev[u]);
    const int ex = __builtin_amdgcn_frexp_exp(fmax(fabs(p), fabs(pm)));
    p = ldexp(p, -ex);
    pm = ldexp(pm, -ex);
  }
  for (; i < r; ++i) row(d[i], e2[i - 1]);
  return c;
}

// C = op(X) op(Y) as mm_mfma, with the operands of four steps of four loaded ahead, with UPPER only
// the output tiles on and above the diagonal (square C), and with HERM (X square) op(X) the Hermitian
// part of X, which is X itself, bit for bit, where X is Hermitian.
template <bool CX, bool TRY, bool UPPER, bool HERM = false>
__device__ __forceinline__ void mm_ahead(const c2* X, int ldx, const c2* Y, int ldy, c2* C, int ldc, int M, int N,
                                         int K, int NB) {
  constexpr int PF = 4;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, nw = (int)blockDim.x >> 6;
  const int tm = (M + 15) / 16, tn = (N + 15) / 16;
  const int r16 = lane & 15, k4 = lane >> 4;
  for (int t = wv; t < tm * tn; t += nw) {
    if (UPPER && t / tn > t % tn) continue;
    const int i0 = (t / tn) * 16, j0 = (t % tn) * 16;
    const int ia = i0 + r16, jb = j0 + r16;
    auto load = [&](int l0, double* ar, double* ai, double* br, double* bi) {
#pragma unroll
      for (int u = 0; u < PF; ++u) {
        const int l = l0 + 4 * u + k4;
        const bool oa = ia < M && l < K, ob = jb < NB && l < K;
        const c2 a = X[oa ? (CX ? l * ldx + ia : ia * ldx + l) : 0];
        const c2 b = Y[ob ? (TRY ? jb * ldy + l : l * ldy + jb) : 0];
        if (HERM) {
          const c2 t = X[oa ? (CX ? ia * ldx + l : l * ldx + ia) : 0];
          ar[u] = oa ? 0.5 * (a.r + t.r) : 0.0;
          ai[u] = oa ? 0.5 * (CX ? t.i - a.i : a.i - t.i) : 0.0;
        } else {
          ar[u] = oa ? a.r : 0.0;
          ai[u] = oa ? (CX ? -a.i : a.i) : 0.0;
        }
        br[u] = ob ? b.r : 0.0;
        bi[u] = ob ? b.i : 0.0;
      }
    };
    rd4 cr = {0.0, 0.0, 0.0, 0.0}, ci = {0.0, 0.0, 0.0, 0.0};
    double ar[PF], ai[PF], br[PF], bi[PF];
    load(0, ar, ai, br, bi);
    for (int l0 = 0; l0 < K; l0 += 4 * PF) {
      double nar[PF], nai[PF], nbr[PF], nbi[PF];
      load(l0 + 4 * PF, nar, nai, nbr, nbi);
#pragma unroll
      for (int u = 0; u < PF; ++u) {
        cr = __builtin_amdgcn_mfma_f64_16x16x4f64(ar[u], br[u], cr, 0, 0, 0);
        ci = __builtin_amdgcn_mfma_f64_16x16x4f64(ar[u], bi[u], ci, 0, 0, 0);
        cr = __builtin_amdgcn_mfma_f64_16x16x4f64(-ai[u], bi[u], cr, 0, 0, 0);
        ci = __builtin_amdgcn_mfma_f64_16x16x4f64(ai[u], br[u], ci, 0, 0, 0);
      }
#pragma unroll
      for (int u = 0; u < PF; ++u) {
        ar[u] = nar[u];
        ai[u] = nai[u];
        br[u] = nbr[u];
        bi[u] = nbi[u];
      }
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int i = i0 + 4 * v + k4, j = j0 + r16;
      if (i < M && j < N) C[i * ldc + j] = c2{cr[v], ci[v]};
    }
  }
}

// Unit vectors x of the tridiagonal (dd, ee) for the eigenvalues lam (ascending), up to the
// factors sc: vector j at ws + vs j + 3 r.  ws: vs >= 4 r doubles per vector.  An isolated
// eigenvalue's vector comes from the twisted factorisation, two lanes per vector; eigenvalues
// closer than 1e-6 tn form a cluster (cluster_vectors).
__device__ __forceinline__ void tri_vectors(double* ws, int vs, const double* dd, const double* ee, const double* lam,
                                            double* sc, int r, int ns, double tn, double tiny) {
  const int tid = threadIdx.x, nt = (int)blockDim.x, lane = tid & 63;
  auto in_cluster = [&](int j) {
    return (j > 0 && lam[j] - lam[j - 1] <= 1e-6 * tn) || (j + 1 < ns && lam[j + 1] - lam[j] <= 1e-6 * tn);
  };
  for (int jb = 0; jb < ns; jb += nt / 2) {
    const int j = jb + (tid >> 1), h = tid & 1;
    const bool mine = j < ns && !in_cluster(j);
    double* blk = ws + (size_t)(mine ? j : 0) * vs;
    double *up = blk, *lp = blk + r, *lm = blk + 2 * r, *um = blk + 3 * r;
    const double shift = mine ? lam[j] : 0.0;
    if (mine) {
      // lane 0: L+ D+ from the top, lane 1: U- D- from the bottom
      double* pd = h ? um : up;
      double* pl = h ? lm : lp;
      const int st = h ? -1 : 1, co = h ? -1 : 0;
      int i = h ? r - 1 : 0;
      double dv = dd[i] - shift;
      double en = r > 1 ? ee[i + co] : 0.0, dn = r > 1 ? dd[i + st] : 0.0;
#pragma unroll 2
      for (int s = 0; s + 1 < r; ++s) {
        const double e = en, dx = dn;
        if (s + 2 < r) {   // the next row's entries, ahead of their use
          en = ee[i + st + co];
          dn = dd[i + 2 * st];
        }
        if (fabs(dv) < tiny) dv = dv < 0 ? -tiny : tiny;
        pd[i] = dv;
        const double l = e * rcp_nr(dv);
        pl[i + co] = l;
        dv = dx - shift - l * e;
        i += st;
      }
      if (fabs(dv) < tiny) dv = dv < 0 ? -tiny : tiny;
      pd[i] = dv;
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    // the twist: the row where |D+ + D- - (d - lambda)| is least (ties to the larger index)
    double best = INFINITY;
    int kt = -1;
    if (mine) {
#pragma unroll 4
      for (int i = h; i < r; i += 2) {
        const double gam = fabs(up[i] + um[i] - (dd[i] - shift));
        if (gam <= best) {
          best = gam;
          kt = i;
        }
      }
    }
    const double ob = dpp_d<kDppXor1>(best);
    const int ok = dpp_i<kDppXor1>(kt);
    if (ob < best || (ob == best && ok > kt)) kt = ok;
    if (kt < 0) kt = 0;
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    double nrm = 0.0;
    if (mine) {   // z_kt = 1, lane 0 upwards through L+, lane 1 downwards through U-
      double* x = um;
      const int st = h ? 1 : -1, co = h ? 0 : -1, cnt = h ? r - 1 - kt : kt;
      const double* pl = h ? lm : lp;
      if (!h) {
        x[kt] = 1.0;
        nrm = 1.0;
      }
      double xv = 1.0;
      int i = kt;
#pragma unroll 4
      for (int s = 0; s < cnt; ++s) {
        xv *= -pl[i + co];
        i += st;
        x[i] = xv;
        nrm += xv * xv;
      }
    }
    nrm += dpp_d<kDppXor1>(nrm);
    if (mine && !h) sc[j] = 1.0 / sqrt(nrm);
  }
  cluster_vectors(
      dd, ee, lam, r, ns, tn, tiny, [&](int c) { return ws + (size_t)c * vs; }, [&](int c) { return ws + (size_t)c * vs + 3 * r; },
      [&](int c) { sc[c] = 1.0; });
}

// size of the per-index arrays in complex units: two complex (phase, subdiagonal phases) and seven
// doubles per basis index, and three broadcast buffers of qp (the thread grid's extent) complex
__host__ __device__ inline int reg_index_c2(int q, int qp) { return 2 * q + 3 * qp + (7 * q + 1) / 2; }

// MODE 2: all matrices in LDS; 1: Z in LDS, the others in the work array; 0: all in the work
// array.  WL: the eigenvector work (4 q doubles per wanted vector) in LDS, over matrices that
// are free by then.
template <int TY, int RY, int RX, int MODE, bool WL>
__global__ __launch_bounds__(TY * 16) void k_ritz_reg(const c2* __restrict__ G, const c2* __restrict__ H, int q,
                                                      int nfix, int want, const double* __restrict__ zthr,
                                                      double drop_rel, double* __restrict__ work, size_t work_stride,
                                                      c2* __restrict__ Y, double* __restrict__ theta,
                                                      int* __restrict__ count, const int* __restrict__ slots) {
  constexpr int NT = TY * 16;
  constexpr int QM = (TY * RY < 16 * RX) ? TY * RY : 16 * RX;   // largest q
  constexpr int QP = (TY * RY > 16 * RX) ? TY * RY : 16 * RX;   // extent of the thread grid
  constexpr bool L2 = QM > 64;                                  // two indices per lane
  extern __shared__ c2 smem[];
  __shared__ double red_s[16];
  const int slot = slots ? slots[blockIdx.x] : (int)blockIdx.x;
  G += (size_t)slot * q * q;
  H += (size_t)slot * q * q;
  work += (size_t)slot * work_stride;
  Y += (size_t)slot * q * want;
  theta += (size_t)slot * want;
  count += slot;
  const double zero_thr = zthr ? zthr[slot] : -INFINITY;
  c2* phase = smem;
  c2* sub = phase + q;       // phases of the subdiagonal
  c2* rowb = sub + q;        // [2][QP] broadcast pivot rows / columns, by step parity
  c2* pv = rowb + 2 * QP;    // [QP]
  double* dsc = reinterpret_cast<double*>(pv + QP);
  double* dd = dsc + q;
  double* ee = dd + q;
  double* ee2 = ee + q;
  double* tau = ee2 + q;
  double* lam = tau + q;
  double* xsc = lam + q;
  const int lz = q | 1;      // odd row stride of every matrix
  c2* lm0 = smem + reg_index_c2(q, QP);
  c2* gw = reinterpret_cast<c2*>(work);
  c2* Z = MODE >= 1 ? lm0 : gw;
  c2* T = MODE == 2 ? lm0 + q * lz : gw + q * lz;
  c2* A = MODE == 2 ? lm0 + 2 * q * lz : gw + 2 * q * lz;
  c2* V = MODE == 2 ? lm0 + 3 * q * lz : gw + 3 * q * lz;
  const int tid = threadIdx.x, lane = tid & 63, tx = tid & 15, ty = tid >> 4;
  double* stamp = work + 10 * q * q + 8 * q + 1;
  if (tid == 0) { stamp[0] = (double)wall_clock64(); stamp[7] = (double)clock64(); }

  // ---- 1. scaled G, pivoted Cholesky by sweeps, Z = D P [L^{-*}; 0] ---------------------------
  for (int i = tid; i < q; i += NT) {
    const double gd = G[i * q + i].r;
    dsc[i] = gd > 0 ? 1.0 / sqrt(gd) : 0.0;
  }
  __syncthreads();
  double ar[RY][RX], ai[RY][RX];
#pragma unroll
  for (int a = 0; a < RY; ++a)
#pragma unroll
    for (int b = 0; b < RX; ++b) {
      const int i = ty + TY * a, j = tx + 16 * b;
      const bool ok = i < q && j < q;
      const c2 g = G[ok ? i * q + j : 0], gt = G[ok ? j * q + i : 0];
      const double s = ok ? dsc[ok ? i : 0] * dsc[ok ? j : 0] : 0.0;
      ar[a][b] = 0.5 * (g.r + gt.r) * s;
      ai[a][b] = 0.5 * (g.i - gt.i) * s;
    }
  // the remaining diagonal: entries lane (and lane + 64) in every wave, -1 once taken
  double d0 = -1.0, d1 = -1.0;
  if (lane < q) d0 = G[lane * q + lane].r * dsc[lane] * dsc[lane];
  if (L2 && lane + 64 < q) d1 = G[(lane + 64) * q + lane + 64].r * dsc[lane + 64] * dsc[lane + 64];
  int r = 0;
  bool second = false;
  // the scalings of Z's rows, and which indices have been pivots, at the lane's indices
  const double sc0 = dsc[lane < q ? lane : 0], sc1 = L2 ? dsc[lane + 64 < q ? lane + 64 : 0] : 0.0;
  bool tk0 = false, tk1 = false;
  for (int k = 0; k < q; ++k) {
    int idx = k;
    if (k >= nfix) {
      double mx = pack_pivot(d0, lane);
      if (L2) mx = fmax(mx, pack_pivot(d1, lane + 64));
      idx = 127 - (int)(__builtin_bit_cast(long long, wave_max(mx)) & 127);
    }
    idx = __builtin_amdgcn_readfirstlane(idx);
    if (idx >= q) break;   // (non-finite input: no valid pivot)
    const double v = (L2 && idx >= 64) ? readlane_d(d1, idx & 63) : readlane_d(d0, idx & 63);
    if (!(v > drop_rel)) break;
    second = second || v < 1e-4;
    c2* row = rowb + (k & 1) * QP;
    if (ty == idx % TY) {
#pragma unroll
      for (int a = 0; a < RY; ++a)
        if (a == idx / TY)
#pragma unroll
          for (int b = 0; b < RX; ++b) row[tx + 16 * b] = c2{ar[a][b], ai[a][b]};
    }
    const double rpiv = rsq_nr(v), invd = rpiv * rpiv;
    __syncthreads();
    c2 xl = row[lane < QP ? lane : 0], xh = {0.0, 0.0}, xj[RX], xi[RY];
    if (L2) xh = row[lane + 64 < QP ? lane + 64 : 0];
#pragma unroll
    for (int b = 0; b < RX; ++b) xj[b] = row[tx + 16 * b];
#pragma unroll
    for (int a = 0; a < RY; ++a) xi[a] = row[ty + TY * a];
    keep(xl);
    if (L2) keep(xh);
#pragma unroll
    for (int b = 0; b < RX; ++b) keep(xj[b]);
#pragma unroll
    for (int a = 0; a < RY; ++a) keep(xi[a]);
    // column k of Z: conj(row k of L^{-1}), rows scaled by D; the first wave holds the row
    if (tid < 64) {
      if (lane < q) Z[lane * lz + k] = lane == idx ? c2{sc0 * rpiv, 0.0} : (tk0 ? c2{sc0 * rpiv * xl.r, -sc0 * rpiv * xl.i} : c2{0.0, 0.0});
      if (L2 && lane + 64 < q)
        Z[(lane + 64) * lz + k] = lane + 64 == idx ? c2{sc1 * rpiv, 0.0} : (tk1 ? c2{sc1 * rpiv * xh.r, -sc1 * rpiv * xh.i} : c2{0.0, 0.0});
    }
    tk0 = tk0 || lane == idx;
    const double n0 = fma(-(xl.r * xl.r + xl.i * xl.i), invd, d0);
    d0 = tk0 || lane >= q ? -1.0 : n0;
    if (L2) {
      tk1 = tk1 || lane + 64 == idx;
      const double n1 = fma(-(xh.r * xh.r + xh.i * xh.i), invd, d1);
      d1 = tk1 || lane + 64 >= q ? -1.0 : n1;
    }
    // the pivot's column is replaced by -L^{-1}'s: zero before the update, which adds one times
    // the multipliers there
    if (tx == (idx & 15)) {
#pragma unroll
      for (int b = 0; b < RX; ++b)
        if (b == (idx >> 4)) {
          xj[b] = c2{1.0, 0.0};
#pragma unroll
          for (int a = 0; a < RY; ++a) ar[a][b] = ai[a][b] = 0.0;
        }
    }
    const int done = k < nfix ? k : nfix;   // rows below `done` are finished (fixed order)
#pragma unroll
    for (int a = 0; a < RY; ++a) {
      if (RY * RX > 9 && done >= TY * (a + 1)) continue;
      const double cr = -xi[a].r * invd, ci = xi[a].i * invd;   // -conj(x) / pivot
#pragma unroll
      for (int b = 0; b < RX; ++b) {
        ar[a][b] = fma(-ci, xj[b].i, fma(cr, xj[b].r, ar[a][b]));
        ai[a][b] = fma(ci, xj[b].r, fma(cr, xj[b].i, ai[a][b]));
      }
    }
    r = k + 1;
  }
  __syncthreads();
  if (tid == 0) stamp[1] = (double)wall_clock64();

  // ---- 2. orthonormality of Z restored when a kept pivot was small ----------------------------
  if (second) {   // G2 = Z^* G Z = L2 L2^*, Z <- Z L2^{-*}
    mm_ahead<true, false, false>(G, q, Z, lz, T, lz, q, r, q, r);   // (G is Hermitian)
    __syncthreads();
    mm_ahead<true, false, false>(Z, lz, T, lz, A, lz, r, r, q, r);
    __syncthreads();
    // distance of G2 from the identity (max entry); when it is small, one Newton-Schulz step
    // Z <- Z (3I - G2) / 2 restores orthonormality to O(dev^2), else the Cholesky route
    double dloc = 0;
    for (int e = tid; e < r * r; e += NT) {
      const int i = e / r, j = e % r;
      const c2 x = A[i * lz + j];
      dloc = fmax(dloc, fabs(x.r - (i == j ? 1.0 : 0.0)) + fabs(x.i));
    }
    for (int o = 32; o > 0; o >>= 1) dloc = fmax(dloc, __shfl_xor(dloc, o, 64));
    if (lane == 0) red_s[tid >> 6] = dloc;
    __syncthreads();
    double dev = 0;
    for (int w = 0; w < NT / 64; ++w) dev = fmax(dev, red_s[w]);
    if (dev < 1e-3) {
      for (int e = tid; e < r * r; e += NT) {
        const int i = e / r, j = e % r;
        const c2 x = A[i * lz + j];
        A[i * lz + j] = (i == j) ? c2{1.5 - 0.5 * x.r, -0.5 * x.i} : c2{-0.5 * x.r, -0.5 * x.i};
      }
      __syncthreads();
      mm_ahead<false, false, false>(Z, lz, A, lz, T, lz, q, r, r, r);
    } else {
      chol(A, V, r, lz);
      lower_inv(V, lz, A, lz, r);
      for (int e = tid; e < q * r; e += NT) {
        const int i = e / r, c = e % r;
        c2 s = {0, 0};
        for (int l = 0; l <= c; ++l) {
          const c2 t = cmulc(A[c * lz + l], Z[i * lz + l]);
          s.r += t.r;
          s.i += t.i;
        }
        T[i * lz + c] = s;
      }
    }
    __syncthreads();
    for (int e = tid; e < q * r; e += NT) Z[(e / r) * lz + e % r] = T[(e / r) * lz + e % r];
    __syncthreads();
  }
  if (tid == 0) stamp[2] = (double)wall_clock64();

  // ---- 3. H' = Z^* H Z, then its tridiagonal form --------------------------------------------
  // (of H its Hermitian part, so that one triangle of the second product holds all of H')
  mm_ahead<true, false, false, true>(H, q, Z, lz, T, lz, q, r, q, r);
  __syncthreads();
  mm_ahead<true, false, true>(Z, lz, T, lz, A, lz, r, r, q, r);
  if (MODE == 1 && WL)   // Z's LDS is reused from the eigenvectors on
    for (int e = tid; e < q * r; e += NT) gw[(e / r) * lz + e % r] = Z[(e / r) * lz + e % r];
  __syncthreads();
#pragma unroll
  for (int a = 0; a < RY; ++a)
#pragma unroll
    for (int b = 0; b < RX; ++b) {
      const int i = ty + TY * a, j = tx + 16 * b;
      const bool ok = i < r && j < r;
      const c2 x = A[ok ? (i <= j ? i * lz + j : j * lz + i) : 0];
      ar[a][b] = ok ? x.r : 0.0;
      ai[a][b] = (ok && i != j) ? (i < j ? x.i : -x.i) : 0.0;
    }
  if (tid == 0) stamp[3] = (double)wall_clock64();
  // Householder: at step k the column below the diagonal, x = A[k+1:, k], is mapped to beta e1
  // by H_k = I - tau v v^* (v in row k of V); the trailing block becomes H_k A22 H_k via
  // p = tau A22 v, w = p - (tau/2)(v^* p) v, A22 <- A22 - v w^* - w v^*.  Every wave forms the
  // column norm and v^* p itself (same lanes, same order: identical values in all waves).
  // The steps of one block of 16 columns run with that block's index as a constant, without the
  // finished blocks (whose entries are no longer kept).  The published column is zero down to
  // row k + 1; its entry there, x0, and the diagonal go to the buffer's side.
  for (int e = tid; e < QP; e += NT)
    if (e >= r) rowb[e] = rowb[QP + e] = c2{0.0, 0.0};
  auto block = [&](auto bc) {
    constexpr int S0 = decltype(bc)::value, A0 = 16 * S0 / TY;
    const int kend = min(16 * S0 + 16, r - 2);
    for (int k = 16 * S0; k < kend; ++k) {
      c2* col = rowb + (k & 1) * QP;
      c2* side = sub + k;   // x0 until the step's end, then the subdiagonal's phase
      if (tx == (k & 15)) {
#pragma unroll
        for (int a = A0; a < RY; ++a) {
          const int i = ty + TY * a;
          const c2 x = {ar[a][S0], ai[a][S0]};
          const bool below = i > k + 1;
          if (i < r) col[i] = c2{below ? x.r : 0.0, below ? x.i : 0.0};
          if (i == k + 1) *side = x;
          if (i == k) dd[k] = x.r;
        }
      }
      __syncthreads();
      c2 x0 = *side, vl = col[lane < QP ? lane : 0], vh = {0.0, 0.0}, vj[RX], vi[RY];
      if (L2) vh = col[lane + 64 < QP ? lane + 64 : 0];
#pragma unroll
      for (int b = S0; b < RX; ++b) vj[b] = col[tx + 16 * b];
#pragma unroll
      for (int a = A0; a < RY; ++a) vi[a] = col[ty + TY * a];
      keep(x0);
      keep(vl);
      if (L2) keep(vh);
#pragma unroll
      for (int b = S0; b < RX; ++b) keep(vj[b]);
#pragma unroll
      for (int a = A0; a < RY; ++a) keep(vi[a]);
      const bool ml = lane > k + 1 && lane < r, mh = lane + 64 > k + 1 && lane + 64 < r;
      double part = ml ? vl.r * vl.r + vl.i * vl.i : 0.0;
      if (L2) part += mh ? vh.r * vh.r + vh.i * vh.i : 0.0;
      const double sig = wave_sum(part);
      const double ax2 = x0.r * x0.r + x0.i * x0.i, xn2 = sig + ax2;
      double xn, tk;
      c2 ph0;
      if (ax2 > 1e-250 && sig > 1e-30 * xn2) {
        const double ra = rsq_nr(ax2);
        xn = xn2 * rsq_nr(xn2);
        ph0 = c2{x0.r * ra, x0.i * ra};
        tk = rcp_nr(fma(xn, ax2 * ra, xn2));   // 2 / (v^* v)
      } else {
        const double ax0 = sqrt(ax2);
        ph0 = ax0 > 0 ? c2{x0.r / ax0, x0.i / ax0} : c2{1.0, 0.0};
        if (!(sig > 1e-30 * xn2)) {   // already reduced in this column
          __syncthreads();   // (x0 has been read by every wave)
          if (tid == 0) {
            tau[k] = 0.0;
            ee[k] = ax0;
            *side = ph0;
          }
          continue;
        }
        xn = sqrt(xn2);
        tk = 1.0 / (xn2 + xn * ax0);
      }
      // v: x0 - beta = x0 + ph0 xn at row k + 1, the published column below
      const c2 v0 = {fma(ph0.r, xn, x0.r), fma(ph0.i, xn, x0.i)};
      vl = lane == k + 1 ? v0 : c2{ml ? vl.r : 0.0, ml ? vl.i : 0.0};
      if (L2) vh = lane + 64 == k + 1 ? v0 : c2{mh ? vh.r : 0.0, mh ? vh.i : 0.0};
#pragma unroll
      for (int b = S0; b < RX; ++b) {
        const bool at = tx + 16 * b == k + 1;
        vj[b] = c2{at ? v0.r : vj[b].r, at ? v0.i : vj[b].i};
      }
#pragma unroll
      for (int a = A0; a < RY; ++a) {
        const bool at = ty + TY * a == k + 1;
        vi[a] = c2{at ? v0.r : vi[a].r, at ? v0.i : vi[a].i};
      }
      // p = tau A22 v for the held rows: sums over the held columns, then over the row's lanes
      c2 pi[RY];
#pragma unroll
      for (int a = A0; a < RY; ++a) {
        double sr = 0.0, si = 0.0;
#pragma unroll
        for (int b = S0; b < RX; ++b) {
          sr = fma(-ai[a][b], vj[b].i, fma(ar[a][b], vj[b].r, sr));
          si = fma(ai[a][b], vj[b].r, fma(ar[a][b], vj[b].i, si));
        }
        pi[a] = c2{tk * sum16(sr), tk * sum16(si)};
      }
      if (tx == 0)
#pragma unroll
        for (int a = A0; a < RY; ++a) pv[ty + TY * a] = pi[a];
      __syncthreads();
      c2 pl = pv[lane < QP ? lane : 0], ph = {0.0, 0.0}, wj[RX];
      if (L2) ph = pv[lane + 64 < QP ? lane + 64 : 0];
#pragma unroll
      for (int b = S0; b < RX; ++b) wj[b] = pv[tx + 16 * b];
      keep(pl);
      if (L2) keep(ph);
#pragma unroll
      for (int b = S0; b < RX; ++b) keep(wj[b]);
      double kp = ml || lane == k + 1 ? vl.r * pl.r + vl.i * pl.i : 0.0;
      if (L2) kp += mh || lane + 64 == k + 1 ? vh.r * ph.r + vh.i * ph.i : 0.0;
      const double Kh = 0.5 * tk * wave_sum(kp);
#pragma unroll
      for (int a = A0; a < RY; ++a) pi[a] = c2{fma(-Kh, vi[a].r, pi[a].r), fma(-Kh, vi[a].i, pi[a].i)};   // w_i
#pragma unroll
      for (int b = S0; b < RX; ++b) {
        wj[b] = c2{fma(-Kh, vj[b].r, wj[b].r), fma(-Kh, vj[b].i, wj[b].i)};
#pragma unroll
        for (int a = A0; a < RY; ++a) {   // minus v_i conj(w_j) + w_i conj(v_j)
          ar[a][b] = fma(-pi[a].i, vj[b].i, fma(-pi[a].r, vj[b].r, fma(-vi[a].i, wj[b].i, fma(-vi[a].r, wj[b].r, ar[a][b]))));
          ai[a][b] = fma(pi[a].r, vj[b].i, fma(-pi[a].i, vj[b].r, fma(vi[a].r, wj[b].i, fma(-vi[a].i, wj[b].r, ai[a][b]))));
        }
      }
      if (tid < 64) {   // the reflector (zero up to row k) and the step's scalars
        if (lane < r) V[k * lz + lane] = vl;
        if (L2 && lane + 64 < r) V[k * lz + lane + 64] = vh;
        if (lane == 0) {
          tau[k] = tk;
          ee[k] = xn;
          *side = c2{-ph0.r, -ph0.i};
        }
      }
    }
  };
  __syncthreads();
  block(std::integral_constant<int, 0>{});
  if constexpr (RX > 1) block(std::integral_constant<int, 1>{});
  if constexpr (RX > 2) block(std::integral_constant<int, 2>{});
  if constexpr (RX > 3) block(std::integral_constant<int, 3>{});
  if constexpr (RX > 4) block(std::integral_constant<int, 4>{});
  if constexpr (RX > 5) block(std::integral_constant<int, 5>{});
  if constexpr (RX > 6) block(std::integral_constant<int, 6>{});
  __syncthreads();
  // the last 2 x 2 block
#pragma unroll
  for (int a = 0; a < RY; ++a)
#pragma unroll
    for (int b = 0; b < RX; ++b) {
      const int i = ty + TY * a, j = tx + 16 * b;
      if (i < r && i + 2 >= r && j == i) dd[i] = ar[a][b];
      if (r >= 2 && i == r - 1 && j == r - 2) {
        const double ax = sqrt(ar[a][b] * ar[a][b] + ai[a][b] * ai[a][b]);
        ee[r - 2] = ax;
        sub[r - 2] = ax > 0 ? c2{ar[a][b] / ax, ai[a][b] / ax} : c2{1.0, 0.0};
      }
    }
  if (tid == 0 && r >= 1) ee[r - 1] = 0.0;
  __syncthreads();
  // real tridiagonal: T' = Phi^* T Phi with Phi = diag(phase), off-diagonals |T_{k+1,k}|
  if (tid == 0) {
    c2 ph = {1.0, 0.0};
    phase[0] = ph;
#pragma unroll 4
    for (int k = 0; k + 1 < r; ++k) {
      ph = cmul(ph, sub[k]);
      phase[k + 1] = ph;
    }
  }
  // its infinity norm, and the scaled entries (largest power of two below the norm) for the
  // eigenvalue counts
  double tn = 0.0;
  for (int i = lane; i < r; i += 64) tn = fmax(tn, fabs(dd[i]) + (i > 0 ? ee[i - 1] : 0.0) + ee[i]);
  tn = wave_max(tn);
  const int tex = tn > 0.0 && tn < INFINITY ? __builtin_amdgcn_frexp_exp(tn) : 0;
  double* ds = reinterpret_cast<double*>(pv);   // (r doubles; the p buffer is free)
  for (int i = tid; i < r; i += NT) {
    const double es = ldexp(ee[i], -tex);
    ds[i] = ldexp(dd[i], -tex);
    ee2[i] = fmax(es * es, 1e-40);
  }
  __syncthreads();
  if (tid == 0) stamp[4] = (double)wall_clock64();

  // ---- 4. wanted eigenvalues (scaled by 2^-tex during the search) ------------------------------
  const double tiny = 1e-300 + 1e-16 * tn * 1e-10;
  const double lo0 = -1.5, hi0 = 1.5;   // entries and norm are below one
  // (a threshold beyond [lo0, hi0], where no value lies, counts as its end)
  const double zs = fmin(fmax(ldexp(zero_thr * (1 + 1e-14) + 1e-300, -tex), lo0), hi0);
  const int nz = (zero_thr > -tn - 1.0 && r > 0) ? sturm_scaled(ds, ee2, r, zs) : 0;
  const int ns = min(want, r - nz);
  {
    // counts at NT points, NT / 64 per octave from 2^-62 to 2^2
    constexpr int PO = NT / 64;
    int* cnt = reinterpret_cast<int*>(rowb);   // 2 QP complex
    auto grid = [&](int t) { return ldexp(1.0 + (double)(t % PO) / PO, t / PO - 62); };
    constexpr bool first = 8 * QP >= NT;   // room for NT counts
    if (first && r > 0) cnt[tid] = sturm_scaled(ds, ee2, r, grid(tid));
    __syncthreads();
    // eight lanes per eigenvalue: each round splits [lo, hi] at 7 interior points and keeps
    // the eighth that holds the (nz + j)-th eigenvalue (all lanes of a group agree)
    const int sb = tid % GS;
    for (int jb = 0; jb < ns; jb += NT / GS) {
      const int j = jb + tid / GS;
      if (j < ns) {
        const int target = nz + j;
        double lo = lo0, hi = hi0;
        if (first) {   // the first grid point whose count exceeds the target
          int a = 0, b = NT;
          while (a < b) {
            const int c = (a + b) >> 1;
            if (cnt[c] > target) b = c;
            else a = c + 1;
          }
          if (a > 0) lo = fmin(grid(a - 1), hi0);
          if (a < NT) hi = fmin(grid(a), hi0);
        }
        for (int it = 0; it < 100; ++it) {
          if (!(hi - lo > 4e-16 * fmax(fabs(lo), fabs(hi)) + 1e-300)) break;
          const double x = lo + (hi - lo) * (double)(sb + 1) / (double)GS;
          const bool inside = sb < GS - 1 && x > lo && x < hi;
          const int c = inside ? sturm_scaled(ds, ee2, r, x) : -1;
          double nlo = (inside && c <= target) ? x : lo;
          double nhi = (inside && c > target) ? x : hi;
          // combine the group of eight (GS) lanes: max of the lower, min of the upper ends
          nlo = fmax(nlo, dpp_d<kDppXor1>(nlo));
          nhi = fmin(nhi, dpp_d<kDppXor1>(nhi));
          nlo = fmax(nlo, dpp_d<kDppXor2>(nlo));
          nhi = fmin(nhi, dpp_d<kDppXor2>(nhi));
          nlo = fmax(nlo, dpp_d<kDppHalfMirror>(nlo));
          nhi = fmin(nhi, dpp_d<kDppHalfMirror>(nhi));
          if (nlo == lo && nhi == hi) break;   // no representable interior point left
          lo = nlo;
          hi = nhi;
        }
        if (sb == 0) lam[j] = ldexp(0.5 * (lo + hi), tex);
      }
    }
  }
  __syncthreads();
  if (tid == 0) stamp[9] = (double)wall_clock64();

  // ---- eigenvectors of the tridiagonal ---------------------------------------------------------
  // (the work lies over A and T, or over Z, in LDS; else over A and T in the work array)
  double* ws = WL ? reinterpret_cast<double*>(MODE == 2 ? T : lm0) : reinterpret_cast<double*>(T);
  // stride of a vector's work, odd in complex units where there is room (LDS banks)
  const int vs = ((MODE == 1 && WL) || (size_t)want * (4 * r + 2) <= (size_t)4 * q * lz) ? 4 * r + 2 : 4 * r;
  tri_vectors(ws, vs, dd, ee, lam, xsc, r, ns, tn, tiny);
  __syncthreads();
  if (tid == 0) stamp[5] = (double)wall_clock64();

  // ---- 5. back-transformation: y = H_0 ... H_{r-3} Phi x, then Y = Z y ------------------------
  // eight lanes per vector, lane sb owning the rows sb mod 8, in registers; a finished vector's r
  // complex entries go to the head of its block of the eigenvector work
  const c2* Zy = (MODE == 1 && WL) ? gw : Z;
  c2* yv = reinterpret_cast<c2*>(ws);
  const int ly = vs / 2;
  {
    constexpr int NC = (QM + GS - 1) / GS;
    const int sb = tid % GS;
    for (int cb = 0; cb < ns; cb += NT / GS) {
      const int c = cb + tid / GS;
      const bool act = c < ns;
      const double* x = ws + (size_t)(act ? c : 0) * vs + 3 * r;
      const double xs = act ? xsc[c] : 0.0;
      double yr[NC], yi[NC];
#pragma unroll
      for (int u = 0; u < NC; ++u) {
        const int i = sb + GS * u;
        const double xv = i < r ? x[i] * xs : 0.0;
        const c2 ph = phase[i < r ? i : 0];
        yr[u] = ph.r * xv;
        yi[u] = ph.i * xv;
      }
      // (entry 0 of every reflector is zero: what rows past r read)
      int at[NC];
#pragma unroll
      for (int u = 0; u < NC; ++u) at[u] = sb + GS * u < r ? sb + GS * u : 0;
      auto back = [&](auto bc) {   // the reflectors of a block of 16 rows: rows above it are done
        constexpr int S0 = decltype(bc)::value, U0 = 2 * S0;
        const int ktop = min(16 * S0 + 15, r - 3);
        if (ktop < 16 * S0) return;
        c2 v[NC];
        double tk = tau[ktop];
#pragma unroll
        for (int u = U0; u < NC; ++u) v[u] = V[ktop * lz + at[u]];
        for (int k = ktop; k >= 16 * S0; --k) {
          c2 vn[NC];   // the next reflector, ahead of its use
          const int kn = k > 16 * S0 ? k - 1 : k;
          const double tn1 = tau[kn];
#pragma unroll
          for (int u = U0; u < NC; ++u) vn[u] = V[kn * lz + at[u]];
          if (tk != 0.0) {
            double sr = 0.0, si = 0.0;
#pragma unroll
            for (int u = U0; u < NC; ++u) {
              sr = fma(v[u].i, yi[u], fma(v[u].r, yr[u], sr));
              si = fma(-v[u].i, yr[u], fma(v[u].r, yi[u], si));
            }
            sr = tk * sum8(sr);
            si = tk * sum8(si);
#pragma unroll
            for (int u = U0; u < NC; ++u) {
              yr[u] = fma(v[u].i, si, fma(-v[u].r, sr, yr[u]));
              yi[u] = fma(-v[u].i, sr, fma(-v[u].r, si, yi[u]));
            }
          }
          tk = tn1;
#pragma unroll
          for (int u = U0; u < NC; ++u) v[u] = vn[u];
        }
      };
      if constexpr (RX > 6) back(std::integral_constant<int, 6>{});
      if constexpr (RX > 5) back(std::integral_constant<int, 5>{});
      if constexpr (RX > 4) back(std::integral_constant<int, 4>{});
      if constexpr (RX > 3) back(std::integral_constant<int, 3>{});
      if constexpr (RX > 2) back(std::integral_constant<int, 2>{});
      if constexpr (RX > 1) back(std::integral_constant<int, 1>{});
      back(std::integral_constant<int, 0>{});
      if (act) {
#pragma unroll
        for (int u = 0; u < NC; ++u)
          if (sb + GS * u < r) yv[(size_t)c * ly + sb + GS * u] = c2{yr[u], yi[u]};
      }
    }
  }
  __syncthreads();
  // Y (q x want) = Z (q x r) y; columns ns..want-1 zero
  mm_ahead<false, true, false>(Zy, lz, yv, ly, Y, want, q, want, r, ns);
  for (int c = tid; c < want; c += NT) theta[c] = c < ns ? lam[c] : 0.0;
  if (tid == 0) {
    *count = ns;
    work[10 * q * q + 8 * q] = (double)r;       // diagnostic: kept rank
    stamp[6] = (double)wall_clock64();
    stamp[8] = (double)clock64();
  }
}

template <int TY, int RY, int RX, int MODE, bool WL>
bool go(size_t lds, const c2* g, const c2* h, int q, int nfix, int want, const double* zthr, double drop_rel,
        double* work, size_t work_stride, c2* y, double* theta, int* count, const Launch& L) {
  static const bool ok = hipFuncSetAttribute((const void*)k_ritz_reg<TY, RY, RX, MODE, WL>,
                                             hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024 - 512) == hipSuccess;
  if (!ok) {
    (void)hipGetLastError();
    return false;
  }
  k_ritz_reg<TY, RY, RX, MODE, WL><<<L.nact, TY * 16, lds, L.st>>>(g, h, q, nfix, want, zthr, drop_rel, work,
                                                                  work_stride, y, theta, count, L.slots);
  return true;
}

}  // namespace

bool ritz_registers(const double* G, const double* H, int q, int nfix, int want, const double* zthr, double drop_rel,
                    double* work, size_t work_stride, double* Y, double* theta, int* count, const Launch& L) {
  if (q > 112) return false;
  // dynamic LDS beside the kernel's 128 static bytes, in 160 KB
  const size_t cap = 160 * 1024 - 512;
  const int qp = q <= 16 ? 16 : q <= 32 ? 32 : q <= 48 ? 48 : q <= 64 ? 64 : q <= 96 ? 96 : 128;
  const size_t idx = (size_t)reg_index_c2(q, qp) * sizeof(c2), mat = (size_t)q * (q | 1) * sizeof(c2);
  const size_t vec = (size_t)want * (4 * q + 2) * sizeof(double);
  const c2* g = reinterpret_cast<const c2*>(G);
  const c2* h = reinterpret_cast<const c2*>(H);
  c2* y = reinterpret_cast<c2*>(Y);
#define BL_GO(TY, RY, RX, MODE, WL, LDS) \
  go<TY, RY, RX, MODE, WL>(LDS, g, h, q, nfix, want, zthr, drop_rel, work, work_stride, y, theta, count, L)
  // Up to 48 columns all four matrices fit LDS (and the eigenvector work lies over two of them:
  // 4 q want <= 4 q^2 doubles); up to 96 columns Z does, and after it the eigenvector work where
  // that fits beside the index arrays.
  if (q <= 16) return BL_GO(16, 1, 1, 2, true, idx + 4 * mat);
  if (q <= 32) return BL_GO(16, 2, 2, 2, true, idx + 4 * mat);
  if (q <= 48) return BL_GO(16, 3, 3, 2, true, idx + 4 * mat);
  const bool wl = idx + vec <= cap;
  const size_t zl = idx + (wl && vec > mat ? vec : mat);
  if (q <= 64) return wl ? BL_GO(32, 2, 4, 1, true, zl) : BL_GO(32, 2, 4, 1, false, idx + mat);
  if (q <= 96) return wl ? BL_GO(32, 3, 6, 1, true, zl) : BL_GO(32, 3, 6, 1, false, idx + mat);
  return BL_GO(32, 4, 7, 0, false, idx);
#undef BL_GO
}

}  // namespace bl

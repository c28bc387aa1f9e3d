// Ritz step of the block iteration (Section 4, Ritz vectors and values) for gfx950: the
// generalised Hermitian eigenproblem  H y = theta G y  of the basis S (q <= 512 columns),
// G = S^* M S and H = S^* A S, solved in one workgroup per problem slot (bases of at most 112
// columns: ritz_reg.hip, the same steps with the matrix in registers):
//
//  1. unit-diagonal scaling D; pivoted Cholesky P^T (D G D) P = L L^* (the first nfix
//     columns, previous Ritz vectors, keep their order), stopped when the largest remaining
//     pivot is below drop_rel: numerically dependent directions of S are dropped (rank r);
//  2. Z = D P [L^{-*}; 0] (q x r) spans the kept directions M-orthonormally; if a kept pivot
//     was small, G2 = Z^* G Z is formed and orthonormality restored to rounding: by one
//     Newton-Schulz step Z <- Z (3I - G2)/2 when G2 is within 1e-3 of the identity (its error
//     squares), else by a second Cholesky pass;
//  3. H' = Z^* H Z (r x r) is reduced to real symmetric tridiagonal form by Householder
//     reflections and a diagonal unitary scaling;
//  4. the wanted eigenvalues (the `want` smallest above zero_thr) by Sturm-count
//     multisection, eight lanes per eigenvalue; eigenvectors of isolated eigenvalues from
//     the twisted factorisation, of clusters of close eigenvalues by inverse iteration with
//     the tridiagonal LU, re-orthogonalised inside the cluster;
//  5. back-transformation through the scaling and the reflections (eight lanes per vector,
//     each lane owning a fixed residue class of the rows), Y = Z y.
//
// The sequential parts (pivot steps, reflector steps) keep few barriers per step: the
// Cholesky pivots without moving data (one barrier per step), pivot searches and vector
// reductions are wave-level shuffle reductions, every wave computes the small reductions it
// needs itself instead of waiting for one thread, and the recurrences use a Newton-refined
// hardware reciprocal instead of division.
#include "ritz_ops.h"

#include <cmath>
#include <cstdio>
#include <cstdlib>

namespace bl {

namespace {

// Bytes of dynamic LDS per basis index: one complex, six doubles and two ints, then either the pivot
// search's two doubles and two ints or, once it is over, a reflector and p (a complex each).
constexpr size_t kIndexBytes = 16 + 6 * 8 + 2 * 4, kSearchBytes = 2 * 8 + 2 * 4, kReflectorBytes = 2 * 16;
constexpr int kMaxRitz = 512;
static_assert(kReflectorBytes >= kSearchBytes, "the reflector's place holds the pivot search");
static_assert(kMaxRitz * (kIndexBytes + kReflectorBytes) + 256 <= 64 * 1024, "LDS that every launch is granted");

// Number of eigenvalues of the real symmetric tridiagonal (d, e; e[i] couples i, i+1)
// that are below x (Sturm sequence of the LDL^T factorisation of T - x I).
__device__ __forceinline__ int sturm_count(const double* d, const double* e2, int r, double x, double tiny) {
  int c = 0;
  double qv = d[0] - x;
  if (qv < 0) ++c;
#pragma unroll 8
  for (int i = 1; i < r; ++i) {
    if (fabs(qv) < tiny) qv = qv < 0 ? -tiny : tiny;
    qv = d[i] - x - e2[i - 1] * rcp_nr(qv);
    if (qv < 0) ++c;
  }
  return c;
}

}  // namespace

// 4 matrices of q rows and stride q | 1 (at most 8 q (q + 1) doubles), then diagnostics at
// 10 q^2 + 8 q
size_t ritz_small_work_doubles(int q) { return (size_t)10 * q * q + 8 * (size_t)q + 64; }

// Bases wider than the register kernel takes (ritz_reg.hip): four matrices of q rows of stride
// q | 1 in the work array; LDS holds the index arrays, the current reflector and p (53 KB at 512
// columns, within what any launch may take).
constexpr int TG = 32;   // TG x TG threads
__global__ __launch_bounds__(TG * TG) void k_ritz(const c2* __restrict__ G, const c2* __restrict__ H, int q,
                                             int nfix, int want, const double* __restrict__ zthr,
                                             double drop_rel, double* __restrict__ work,
                                             size_t work_stride, c2* __restrict__ Y,
                                             double* __restrict__ theta, int* __restrict__ count,
                                             const int* __restrict__ slots) {
  extern __shared__ c2 smem[];
  // one workgroup per problem slot
  const int slot = slots ? slots[blockIdx.x] : (int)blockIdx.x;
  G += (size_t)slot * q * q;
  H += (size_t)slot * q * q;
  work += (size_t)slot * work_stride;
  Y += (size_t)slot * q * want;
  theta += (size_t)slot * want;
  count += slot;
  const double zero_thr = zthr ? zthr[slot] : -INFINITY;
  __shared__ int rank_s, second_s;
  __shared__ double red_s[16];
  c2* phase = smem;
  double* dsc = reinterpret_cast<double*>(phase + q);
  double* dd = dsc + q;
  double* ee = dd + q;
  double* ee2 = ee + q;
  double* tau = ee2 + q;
  double* lam = tau + q;
  int* perm = reinterpret_cast<int*>(lam + q);
  int* pinv = perm + q;
  c2* gw = reinterpret_cast<c2*>(work);
  // row strides are odd (q | 1, r | 1 once the rank is known)
  const int lq = q | 1;
  c2* A = gw;
  c2* B = A + q * lq;
  c2* Z = B + q * lq;
  c2* T = Z + q * lq;
  const int tid = threadIdx.x, nt = blockDim.x, lane = tid & 63;
  double* stamp = work + 10 * q * q + 8 * q + 1;
  if (tid == 0) { stamp[0] = (double)wall_clock64(); stamp[7] = (double)clock64(); }

  // ---- 1. scaled G and pivoted Cholesky -----------------------------------------------------
  // Implicit pivoting: A keeps the original index order; the remaining indices are a compact
  // list and the current diagonal a separate array, both double-buffered by step parity, so
  // that a step needs one barrier (pivot search and update read this step's buffers, the
  // update writes the next step's).  L_{i,k} of the original index i goes to B[i][k]; the
  // rows are put in pivot order afterwards.
  double* dg = reinterpret_cast<double*>(reinterpret_cast<char*>(smem) + kIndexBytes * q);   // [2][q]
  int* rem = reinterpret_cast<int*>(dg + 2 * q);      // [2][q]
  for (int i = tid; i < q; i += nt) {
    const double gd = G[i * q + i].r;
    dsc[i] = gd > 0 ? 1.0 / sqrt(gd) : 0.0;
    rem[i] = i;
  }
  if (tid == 0) second_s = 0;
  __syncthreads();
  int r = 0;
  const int ty = tid / TG, tx = tid % TG;   // TG x TG thread grid
  for (int e = tid; e < q * q; e += nt) {
    const int i = e / q, j = e % q;
    const c2 g = G[e], gt = G[j * q + i];
    const double s = dsc[i] * dsc[j];
    const c2 a = {0.5 * (g.r + gt.r) * s, 0.5 * (g.i - gt.i) * s};
    A[i * lq + j] = a;
    if (i == j) dg[i] = a.r;
  }
  __syncthreads();
  for (int k = 0; k < q; ++k) {
    const double* dcur = dg + (k & 1) * q;
    double* dnext = dg + ((k + 1) & 1) * q;
    const int* rcur = rem + (k & 1) * q;
    int* rnext = rem + ((k + 1) & 1) * q;
    const int nr = q - k;
    // pivot: largest remaining diagonal, ties to the smaller index (the first nfix stay in
    // order: they lead the list); every wave finds it itself (same lanes, same order)
    double v;
    int idx, pos;
    if (k < nfix) {
      pos = 0;
      idx = rcur[0];
      v = dcur[idx];
    } else {
      v = -1.0;
      idx = q;
      pos = q;
      for (int t = lane; t < nr; t += 64) {
        const int i = rcur[t];
        const double dv = dcur[i];
        if (dv > v || (dv == v && i < idx)) { v = dv; idx = i; pos = t; }
      }
      pick_max<kDppXor1>(v, idx, pos);
      pick_max<kDppXor2>(v, idx, pos);
      pick_max<kDppHalfMirror>(v, idx, pos);
      pick_max<kDppMirror>(v, idx, pos);
      // the four rows' winners, in row order (uniform values)
      double bv = readlane_d(v, 0);
      int bi = __builtin_amdgcn_readlane(idx, 0), bp = __builtin_amdgcn_readlane(pos, 0);
      for (int rw = 16; rw < 64; rw += 16) {
        const double ov = readlane_d(v, rw);
        const int oi = __builtin_amdgcn_readlane(idx, rw), op = __builtin_amdgcn_readlane(pos, rw);
        if (ov > bv || (ov == bv && oi < bi)) { bv = ov; bi = oi; bp = op; }
      }
      v = bv;
      idx = bi;
      pos = bp;
    }
    if (!(v > drop_rel)) break;
    if (tid == 0) {
      if (v < 1e-4) second_s = 1;
      perm[k] = idx;
    }
    const double piv = sqrt(v), invd = 1.0 / v;
    // factor column k (original rows) and the next step's list
    for (int t = tid; t < nr; t += nt) {
      const int i = rcur[t];
      const c2 a = A[i * lq + idx];
      B[i * lq + k] = (i == idx) ? c2{piv, 0.0} : c2{a.r / piv, a.i / piv};
      if (t != pos) rnext[t < pos ? t : t - 1] = i;
    }
    // trailing update of the remaining indices but idx (column idx is only read here)
    for (int a = ty; a < nr; a += TG) {
      if (a == pos) continue;
      const int i = rcur[a];
      const c2 aik = A[i * lq + idx];
      for (int b = tx; b < nr; b += TG) {
        if (b == pos) continue;
        const int j = rcur[b];
        const c2 t = cmulc(A[j * lq + idx], aik);
        const c2 nv = {A[i * lq + j].r - t.r * invd, A[i * lq + j].i - t.i * invd};
        A[i * lq + j] = nv;
        if (a == b) dnext[i] = nv.r;
      }
    }
    __syncthreads();
    r = k + 1;
  }

  // pivot order of the dropped indices (after the kept ones), and the factor's rows in pivot
  // order into T (rows of A are free from here on)
  for (int t = tid; t < q - r; t += nt) perm[r + t] = rem[(r & 1) * q + t];
  __syncthreads();
  for (int e = tid; e < r * r; e += nt) {
    const int ip = e / r, k = e % r;
    if (k <= ip) T[ip * lq + k] = B[perm[ip] * lq + k];
  }
  if (tid == 0) rank_s = r;
  __syncthreads();
  r = rank_s;
  const int lr = r | 1;
  if (tid == 0) stamp[1] = (double)wall_clock64();

  // ---- 2. Z = D P [L^{-*}; 0] -------------------------------------------------------------
  lower_inv(T, lq, A, lq, r);
  for (int i = tid; i < q; i += nt) pinv[perm[i]] = i;
  __syncthreads();
  for (int e = tid; e < q * r; e += nt) {
    const int i = e / r, c = e % r;
    const int pi = pinv[i];
    c2 z = {0.0, 0.0};
    if (pi < r && pi <= c) {
      const c2 l = A[c * lq + pi];
      z = {dsc[i] * l.r, -dsc[i] * l.i};
    }
    Z[i * lr + c] = z;
  }
  __syncthreads();
  if (second_s) {   // G2 = Z^* G Z = L2 L2^*, Z <- Z L2^{-*}
    for (int e = tid; e < q * q; e += nt) B[(e / q) * lq + e % q] = G[e];   // G into the free B region
    __syncthreads();
    mm_mfma<false, false>(B, lq, Z, lr, T, lr, q, r, q, r);
    __syncthreads();
    mm_mfma<true, false>(Z, lr, T, lr, A, lr, r, r, q, r);
    __syncthreads();
    // distance of G2 from the identity (max entry); when it is small, one Newton-Schulz step
    // Z <- Z (3I - G2) / 2 restores orthonormality to O(dev^2), else the Cholesky route
    double dloc = 0;
    for (int e = tid; e < r * r; e += nt) {
      const int i = e / r, j = e % r;
      const c2 a = A[i * lr + j];
      dloc = fmax(dloc, fabs(a.r - (i == j ? 1.0 : 0.0)) + fabs(a.i));
    }
    for (int o = 32; o > 0; o >>= 1) dloc = fmax(dloc, __shfl_xor(dloc, o, 64));
    if (lane == 0) red_s[tid >> 6] = dloc;
    __syncthreads();
    double dev = 0;
    for (int w = 0; w < (nt >> 6); ++w) dev = fmax(dev, red_s[w]);
    if (dev < 1e-3) {
      for (int e = tid; e < r * r; e += nt) {
        const int i = e / r, j = e % r;
        const c2 a = A[i * lr + j];
        A[i * lr + j] = (i == j) ? c2{1.5 - 0.5 * a.r, -0.5 * a.i} : c2{-0.5 * a.r, -0.5 * a.i};
      }
      __syncthreads();
      mm_mfma<false, false>(Z, lr, A, lr, T, lr, q, r, r, r);
    } else {
      chol(A, B, r, lr);
      lower_inv(B, lr, A, lr, r);
      for (int e = tid; e < q * r; e += nt) {
        const int i = e / r, c = e % r;
        c2 s = {0, 0};
        for (int l = 0; l <= c; ++l) {
          const c2 t = cmulc(A[c * lr + l], Z[i * lr + l]);
          s.r += t.r;
          s.i += t.i;
        }
        T[i * lr + c] = s;
      }
    }
    __syncthreads();
    for (int e = tid; e < q * lr; e += nt) Z[e] = T[e];
    __syncthreads();
  }
  if (tid == 0) stamp[2] = (double)wall_clock64();

  // ---- 3. H' = Z^* H Z (A, stride r), Hermitian part, then tridiagonalisation ----------------
  for (int e = tid; e < q * q; e += nt) B[(e / q) * lq + e % q] = H[e];   // H into the free B region
  __syncthreads();
  mm_mfma<false, false>(B, lq, Z, lr, T, lr, q, r, q, r);
  __syncthreads();
  mm_mfma<true, false>(Z, lr, T, lr, A, lr, r, r, q, r);
  __syncthreads();
  for (int e = tid; e < r * r; e += nt) {
    const int a = e / r, b = e % r;
    if (a < b) {
      const c2 x = A[a * lr + b], y = A[b * lr + a];
      const c2 h = {0.5 * (x.r + y.r), 0.5 * (x.i - y.i)};
      A[a * lr + b] = h;
      A[b * lr + a] = {h.r, -h.i};
    } else if (a == b) {
      A[a * lr + a].i = 0.0;
    }
  }
  __syncthreads();
  if (tid == 0) stamp[3] = (double)wall_clock64();
  // Householder: at step k the column below the diagonal, x = A[k+1:, k], is mapped to
  // beta e1 by H_k = I - tau v v^* (v stored in row k of B, entries k+1..r-1); the trailing
  // block becomes H_k A22 H_k via p = tau A22 v, w = p - (tau/2)(v^* p) v,
  // A22 <- A22 - v w^* - w v^*.  T holds p.  Every wave forms the column norm and v^* p
  // itself (same lanes, same order: identical values in all waves).
  // the reflector and p are kept in LDS for the products; the reflector also goes to B for the
  // back-transformation
  // (over the pivot search's arrays)
  c2* vst = reinterpret_cast<c2*>(dg);
  c2* pv = vst + q;
  for (int k = 0; k + 2 < r; ++k) {
    const int m = r - k - 1;
    double part = 0;
    for (int j = lane; j < m; j += 64) {
      const c2 x = A[(k + 1 + j) * lr + k];
      part += x.r * x.r + x.i * x.i;
    }
    const double xn2 = wave_sum(part);
    const c2 x0 = A[(k + 1) * lr + k];
    const double ax0 = sqrt(x0.r * x0.r + x0.i * x0.i);
    const double sig = xn2 - ax0 * ax0;
    if (sig <= 1e-30 * xn2 || xn2 == 0.0) {   // already reduced in this column
      if (tid == 0) { tau[k] = 0.0; dd[k] = A[k * lr + k].r; }
      for (int j = tid; j < r; j += nt) B[k * lr + j] = {0.0, 0.0};
      __syncthreads();
      continue;
    }
    const double xn = sqrt(xn2);
    const c2 ph0 = ax0 > 0 ? c2{x0.r / ax0, x0.i / ax0} : c2{1.0, 0.0};
    const c2 beta = {-ph0.r * xn, -ph0.i * xn};
    const double tk = 1.0 / (xn2 + xn * ax0);      // 2 / (v^* v)
    for (int j = tid; j < r; j += nt) {
      c2 vj = {0.0, 0.0};
      if (j == k + 1) vj = {x0.r - beta.r, x0.i - beta.i};
      else if (j > k + 1) vj = A[j * lr + k];
      B[k * lr + j] = vj;
      vst[j] = vj;
    }
    if (tid == 0) { tau[k] = tk; dd[k] = A[k * lr + k].r; }
    __syncthreads();
    const c2* v = vst;
    {   // p = tau A22 v, four lanes per row
      const int sub = tid & 3;
      for (int rb = 0; rb < m; rb += nt / 4) {
        const int i = rb + tid / 4;
        c2 s = {0, 0};
        if (i < m) {
          const c2* row = A + (k + 1 + i) * lr + k + 1;
          for (int l = sub; l < m; l += 4) {
            const c2 t = cmul(row[l], v[k + 1 + l]);
            s.r += t.r;
            s.i += t.i;
          }
        }
        s.r = sum4(s.r);
        s.i = sum4(s.i);
        if (sub == 0 && i < m) pv[i] = {tk * s.r, tk * s.i};
      }
    }
    __syncthreads();
    double kp = 0;
    for (int i = lane; i < m; i += 64) kp += cmulc(v[k + 1 + i], pv[i]).r;
    const double Kh = 0.5 * tk * wave_sum(kp);
    for (int i = ty; i < m; i += TG) {
      const c2 vi = v[k + 1 + i];
      const c2 wi = {pv[i].r - Kh * vi.r, pv[i].i - Kh * vi.i};
      for (int j = tx; j < m; j += TG) {
        const c2 vj = v[k + 1 + j];
        const c2 wj = {pv[j].r - Kh * vj.r, pv[j].i - Kh * vj.i};
        const c2 t1 = cmulc(wj, vi), t2 = cmulc(vj, wi);   // v_i conj(w_j), w_i conj(v_j)
        c2& a = A[(k + 1 + i) * lr + k + 1 + j];
        a = {a.r - t1.r - t2.r, a.i - t1.i - t2.i};
      }
    }
    if (tid == 0) A[(k + 1) * lr + k] = beta;   // column k: outside the updated block
    __syncthreads();
  }
  // real tridiagonal: T' = Phi^* T Phi with Phi = diag(phase), off-diagonals |T_{k+1,k}|
  if (tid == 0) {
    for (int k = (r >= 2 ? r - 2 : 0); k < r; ++k) dd[k] = A[k * lr + k].r;
    phase[0] = {1.0, 0.0};
    for (int k = 0; k + 1 < r; ++k) {
      const c2 b = A[(k + 1) * lr + k];
      const double ab = sqrt(b.r * b.r + b.i * b.i);
      ee[k] = ab;
      ee2[k] = ab * ab;
      // phase[k+1] = phase[k] * b / |b|
      const c2 u = ab > 0 ? c2{b.r / ab, b.i / ab} : c2{1.0, 0.0};
      phase[k + 1] = cmul(phase[k], u);
    }
    if (r >= 1) { ee[r - 1] = 0.0; ee2[r - 1] = 0.0; }
  }
  __syncthreads();
  if (tid == 0) stamp[4] = (double)wall_clock64();

  // ---- 4. wanted eigenvalues (multisection) and eigenvectors (inverse iteration) ----------
  double tn = 0;   // infinity norm of the tridiagonal
  for (int i = 0; i < r; ++i) tn = fmax(tn, fabs(dd[i]) + (i > 0 ? ee[i - 1] : 0.0) + ee[i]);
  const double lo0 = -tn - 1.0, hi0 = tn + 1.0;
  const double tiny = 1e-300 + 1e-16 * tn * 1e-10;
  const int nz = (zero_thr > lo0) ? sturm_count(dd, ee2, r, zero_thr * (1 + 1e-14) + 1e-300, tiny) : 0;
  const int ns = min(want, r - nz);
  {
    // eight lanes per eigenvalue: each round splits [lo, hi] at 7 interior points and keeps
    // the eighth that holds the (nz + j)-th eigenvalue (all lanes of a group agree)
    const int sub = tid % GS;
    for (int jb = 0; jb < ns; jb += nt / GS) {
      const int j = jb + tid / GS;
      if (j < ns) {
        const int target = nz + j;
        double lo = lo0, hi = hi0;
        for (int it = 0; it < 100; ++it) {
          if (!(hi - lo > 4e-16 * fmax(fabs(lo), fabs(hi)) + 1e-300)) break;
          const double x = lo + (hi - lo) * (double)(sub + 1) / (double)GS;
          const bool inside = sub < GS - 1 && x > lo && x < hi;
          const int c = inside ? sturm_count(dd, ee2, r, x, tiny) : -1;
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
        if (sub == 0) lam[j] = 0.5 * (lo + hi);
      }
    }
  }
  __syncthreads();
  if (tid == 0) stamp[9] = (double)wall_clock64();
  // Eigenvectors: an isolated eigenvalue's from the twisted factorisation (one thread each);
  // eigenvalues closer than 1e-6 tn form a cluster (cluster_vectors).  Real vectors of length r
  // are kept in T (as doubles): vec j at xs + j*r.  Per index j the LU of T' - lambda_j I
  // (3 arrays of length r) lies in the free A region, continued in T's tail (at most want*r +
  // 3*want*r <= 4 q^2 doubles, the size of A and T together).
  double* xs = reinterpret_cast<double*>(T);
  const int clus_in_a = (2 * q * q) / (3 * r > 0 ? 3 * r : 1);
  auto lu_at = [&](int j) -> double* {
    return j < clus_in_a ? reinterpret_cast<double*>(A) + (size_t)j * 3 * r
                         : xs + (size_t)want * r + (size_t)(j - clus_in_a) * 3 * r;
  };
  auto in_cluster = [&](int j) {
    return (j > 0 && lam[j] - lam[j - 1] <= 1e-6 * tn) || (j + 1 < ns && lam[j + 1] - lam[j] <= 1e-6 * tn);
  };
  for (int j = tid; j < ns; j += nt) {
    if (in_cluster(j)) continue;
    double* u = lu_at(j);
    double* u1 = u + r;        // L+ / D+ of the twisted factorisation
    double* lm = u1 + r;
    {
      // an isolated eigenvalue: its vector from the twisted factorisation of T' - lambda I
      // (one forward LDL^T and one backward UDU^T pass; the twist index k minimises
      // |gamma_k| = |D+_k + D-_k - (d_k - lambda)|, and z_k = 1 is propagated both ways)
      double* x = xs + (size_t)j * r;
      const double shift = lam[j];
      double dp = dd[0] - shift;
      for (int i = 0; i + 1 < r; ++i) {
        if (fabs(dp) < tiny) dp = dp < 0 ? -tiny : tiny;
        u[i] = dp;                           // D+_i
        const double l = ee[i] * rcp_nr(dp);
        u1[i] = l;                           // L+_i
        dp = dd[i + 1] - shift - l * ee[i];
      }
      if (fabs(dp) < tiny) dp = dp < 0 ? -tiny : tiny;
      u[r - 1] = dp;
      double dm = dd[r - 1] - shift;
      double best = fabs(u[r - 1]);
      int kt = r - 1;
      for (int i = r - 2; i >= 0; --i) {
        if (fabs(dm) < tiny) dm = dm < 0 ? -tiny : tiny;
        const double uu = ee[i] * rcp_nr(dm);
        lm[i] = uu;                          // U-_i
        dm = dd[i] - shift - uu * ee[i];     // D-_i
        const double gam = fabs(u[i] + dm - (dd[i] - shift));
        if (gam < best) { best = gam; kt = i; }
      }
      x[kt] = 1.0;
      double nrm = 1.0;
      for (int i = kt - 1; i >= 0; --i) {
        x[i] = -u1[i] * x[i + 1];
        nrm += x[i] * x[i];
      }
      for (int i = kt + 1; i < r; ++i) {
        x[i] = -lm[i - 1] * x[i - 1];
        nrm += x[i] * x[i];
      }
      const double inv = 1.0 / sqrt(nrm);
      for (int i = 0; i < r; ++i) x[i] *= inv;
    }
  }
  cluster_vectors(
      dd, ee, lam, r, ns, tn, tiny, lu_at, [&](int c) { return xs + (size_t)c * r; }, [](int) {});
  __syncthreads();
  if (tid == 0) stamp[5] = (double)wall_clock64();

  // ---- 5. back-transformation: y = H_0 ... H_{r-3} Phi x, then Y = Z y ----------------------
  // complex vectors of length r, column-major in the A region: yv[c * lr + i]
  c2* yv = A;
  for (int e = tid; e < ns * r; e += nt) {
    const int c = e / r, i = e % r;
    const double xv = xs[(size_t)c * r + i];
    yv[c * lr + i] = {phase[i].r * xv, phase[i].i * xv};
  }
  __syncthreads();
  {
    // eight lanes per vector; lane `sub` owns the rows i = sub mod 8 throughout, so the
    // reflections need no barrier (v^* y is combined by shuffles inside the group)
    const int sub = tid % GS;
    for (int cb = 0; cb < ns; cb += nt / GS) {
      const int c = cb + tid / GS;
      if (c < ns) {
        c2* y = yv + (size_t)c * lr;
        for (int k = r - 3; k >= 0; --k) {
          const double tk = tau[k];
          if (tk == 0.0) continue;
          const c2* v = B + k * lr;
          const int i0 = k + 1 + ((sub - (k + 1)) % GS + GS) % GS;
          c2 s = {0, 0};
          for (int i = i0; i < r; i += GS) {
            const c2 t = cmulc(v[i], y[i]);
            s.r += t.r;
            s.i += t.i;
          }
          s.r = sum8(s.r);   // the vector's eight lanes (GS)
          s.i = sum8(s.i);
          for (int i = i0; i < r; i += GS) {
            const c2 t = cmul(v[i], s);
            y[i] = {y[i].r - tk * t.r, y[i].i - tk * t.i};
          }
        }
      }
    }
  }
  __syncthreads();
  // Y (q x want) = Z (q x r) y; columns ns..want-1 zero
  mm_mfma<false, true>(Z, lr, yv, lr, Y, want, q, want, r, ns);
  for (int c = tid; c < want; c += nt) theta[c] = c < ns ? lam[c] : 0.0;
  if (tid == 0) {
    *count = ns;
    work[10 * q * q + 8 * q] = (double)r;       // diagnostic: kept rank
    stamp[5 + 1] = (double)wall_clock64();
    stamp[8] = (double)clock64();
  }
}

void ritz_small(const double* G, const double* H, int q, int nfix, int want, const double* zthr,
                double drop_rel, double* work, size_t work_stride, double* Y, double* theta,
                int* count, const Launch& L) {
  if (L.nact <= 0) return;
  // up to 112 columns the matrix being reduced fits a workgroup's registers (where the device
  // grants its LDS): 0.49 ms there against 1.02 ms here at q = 84, 0.78 against 2.1 at q = 112
  if (ritz_registers(G, H, q, nfix, want, zthr, drop_rel, work, work_stride, Y, theta, count, L)) return;
  const size_t lds = (size_t)q * (kIndexBytes + kReflectorBytes);
  k_ritz<<<L.nact, TG * TG, lds, L.st>>>(reinterpret_cast<const c2*>(G), reinterpret_cast<const c2*>(H), q, nfix, want,
                                         zthr, drop_rel, work, work_stride, reinterpret_cast<c2*>(Y), theta, count,
                                         L.slots);
}

}  // namespace bl

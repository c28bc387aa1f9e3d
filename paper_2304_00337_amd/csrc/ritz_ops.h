// Device helpers shared by the Ritz-step kernels (ritz.hip, ritz_reg.hip): complex arithmetic,
// Newton-refined reciprocals, cross-lane exchanges, small matrix products on the matrix cores
// and the triangular factor routines of the orthonormality repair.
#pragma once

#include "internal.h"

namespace bl {

namespace {

struct c2 {
  double r, i;
};
__device__ __forceinline__ c2 cmul(c2 a, c2 b) { return {a.r * b.r - a.i * b.i, a.r * b.i + a.i * b.r}; }
__device__ __forceinline__ c2 cmulc(c2 a, c2 b) { return {a.r * b.r + a.i * b.i, a.r * b.i - a.i * b.r}; }  // conj(a) b

constexpr int GS = 8;     // lanes per eigenvalue / eigenvector group

// 1 / x from the hardware reciprocal and two Newton steps (full FP64 accuracy, without the
// long division sequence on the Sturm and factorisation recurrences)
__device__ __forceinline__ double rcp_nr(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = fma(fma(-x, r, 1.0), r, r);
  r = fma(fma(-x, r, 1.0), r, r);
  return r;
}

// Cross-lane exchanges through DPP (data-parallel primitives: operand swizzles of the vector
// ALU, a few cycles) instead of LDS permutes (a round trip through the LDS crossbar each).
// Patterns within rows of 16 lanes: partner lane^1 and lane^2 (quad permutations), then the
// mirror within 8 lanes and within 16 lanes, which after the first two stages reach the
// other quad / the other half-row.  All lanes of the wave must be active.
constexpr int kDppXor1 = 0xB1;         // quad_perm [1, 0, 3, 2]
constexpr int kDppXor2 = 0x4E;         // quad_perm [2, 3, 0, 1]
constexpr int kDppHalfMirror = 0x141;  // lane i <-> 7 - i within 8 lanes
constexpr int kDppMirror = 0x140;      // lane i <-> 15 - i within 16 lanes

template <int CTRL>
__device__ __forceinline__ int dpp_i(int x) {
  return __builtin_amdgcn_mov_dpp(x, CTRL, 0xF, 0xF, false);
}
template <int CTRL>
__device__ __forceinline__ double dpp_d(double x) {
  const long long b = __builtin_bit_cast(long long, x);
  const int lo = dpp_i<CTRL>((int)(b & 0xffffffffLL)), hi = dpp_i<CTRL>((int)(b >> 32));
  return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned int)lo);
}
__device__ __forceinline__ double readlane_d(double x, int l) {
  const long long b = __builtin_bit_cast(long long, x);
  const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffffLL), l);
  const int hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
  return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned int)lo);
}
// sum over groups of 4 / 8 / 16 aligned lanes, the same value in every lane of the group
// (each stage adds two equal-order pairs, so partners agree bit for bit)
__device__ __forceinline__ double sum4(double a) {
  a += dpp_d<kDppXor1>(a);
  return a + dpp_d<kDppXor2>(a);
}
__device__ __forceinline__ double sum8(double a) { a = sum4(a); return a + dpp_d<kDppHalfMirror>(a); }
__device__ __forceinline__ double sum16(double a) { a = sum8(a); return a + dpp_d<kDppMirror>(a); }

__device__ __forceinline__ double wave_sum(double a) {
  a = sum16(a);
  return (readlane_d(a, 0) + readlane_d(a, 16)) + (readlane_d(a, 32) + readlane_d(a, 48));
}

// (v, idx, pos) of the partner lane replaces this lane's when larger, ties to the smaller
// index (a strict order, so both partners keep the same triple)
template <int CTRL>
__device__ __forceinline__ void pick_max(double& v, int& idx, int& pos) {
  const double ov = dpp_d<CTRL>(v);
  const int oi = dpp_i<CTRL>(idx), op = dpp_i<CTRL>(pos);
  if (ov > v || (ov == v && oi < idx)) { v = ov; idx = oi; pos = op; }
}

// C (M x N, row-major, leading dimension ldc) = op(X) op(Y) on the matrix cores (FP64 MFMA
// 16x16x4, four real products per complex one), every wave of the workgroup taking 16 x 16
// output tiles in turn; op(X) = X (M x K, row-major) or, with CX, X^* for X stored K x M;
// op(Y) = Y (K x N, row-major) or, with TY, the transpose of Y stored N x K.  Columns j >= NB
// of op(Y) are taken as zero.  Operands may live in LDS or global memory; the next four-wide
// step's operands are loaded while the current one is multiplied.  Call between barriers.
typedef double rd4 __attribute__((ext_vector_type(4)));
template <bool CX, bool TY>
__device__ __forceinline__ void mm_mfma(const c2* X, int ldx, const c2* Y, int ldy, c2* C, int ldc, int M, int N,
                                        int K, int NB) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, nw = (int)blockDim.x >> 6;
  const int tm = (M + 15) / 16, tn = (N + 15) / 16;
  const int r16 = lane & 15, k4 = lane >> 4;
  for (int t = wv; t < tm * tn; t += nw) {
    const int i0 = (t / tn) * 16, j0 = (t % tn) * 16;
    const int ia = i0 + r16, jb = j0 + r16;   // the operand row of X and column of Y this lane supplies
    auto lda = [&](int l) -> c2 {
      if (ia >= M || l >= K) return c2{0.0, 0.0};
      if (CX) {
        const c2 v = X[(int64_t)l * ldx + ia];
        return c2{v.r, -v.i};
      }
      return X[(int64_t)ia * ldx + l];
    };
    auto ldb = [&](int l) -> c2 {
      if (jb >= NB || l >= K) return c2{0.0, 0.0};
      return TY ? Y[(int64_t)jb * ldy + l] : Y[(int64_t)l * ldy + jb];
    };
    rd4 cr = {0.0, 0.0, 0.0, 0.0}, ci = {0.0, 0.0, 0.0, 0.0};
    c2 a = lda(k4), b = ldb(k4);
    for (int l0 = 0; l0 < K; l0 += 4) {
      const c2 an = lda(l0 + 4 + k4), bn = ldb(l0 + 4 + k4);
      cr = __builtin_amdgcn_mfma_f64_16x16x4f64(a.r, b.r, cr, 0, 0, 0);
      cr = __builtin_amdgcn_mfma_f64_16x16x4f64(-a.i, b.i, cr, 0, 0, 0);
      ci = __builtin_amdgcn_mfma_f64_16x16x4f64(a.r, b.i, ci, 0, 0, 0);
      ci = __builtin_amdgcn_mfma_f64_16x16x4f64(a.i, b.r, ci, 0, 0, 0);
      a = an;
      b = bn;
    }
    // accumulator entry v of lane (k4, r16) is C[i0 + 4 v + k4][j0 + r16]
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int i = i0 + 4 * v + k4, j = j0 + r16;
      if (i < M && j < N) C[(int64_t)i * ldc + j] = c2{cr[v], ci[v]};
    }
  }
}

// Linv (stride ldv) = L^{-1} for lower-triangular L (stride ld, r x r).  Row i of the
// inverse depends on rows < i; four lanes share each column's inner sum.
__device__ __forceinline__ void lower_inv(const c2* L, int ld, c2* Linv, int ldv, int r) {
  const int tid = threadIdx.x, sub = tid & 3;
  for (int i = 0; i < r; ++i) {
    const double d = L[i * ld + i].r;
    for (int cb = 0; cb < r; cb += (int)blockDim.x / 4) {
      const int c = cb + tid / 4;
      c2 s = {0, 0};
      if (c < i)
        for (int l = c + sub; l < i; l += 4) {
          const c2 t = cmul(L[i * ld + l], Linv[l * ldv + c]);
          s.r += t.r;
          s.i += t.i;
        }
      s.r = sum4(s.r);
      s.i = sum4(s.i);
      if (sub == 0 && c < r) {
        c2 v = {0, 0};
        if (c == i) v = {1.0, 0.0};
        else if (c < i) v = {-s.r, -s.i};
        Linv[i * ldv + c] = {v.r / d, v.i / d};
      }
    }
    __syncthreads();
  }
}

// Unpivoted Cholesky of the Hermitian positive definite r x r matrix A (full square kept,
// overwritten); the factor's columns go to L (stride ld, lower triangle).
__device__ __forceinline__ void chol(c2* A, c2* L, int r, int ld) {
  const int tid = threadIdx.x, nt = blockDim.x;
  for (int k = 0; k < r; ++k) {
    double d = A[k * ld + k].r;
    d = d > 1e-300 ? d : 1e-300;
    const double piv = sqrt(d), invd = 1.0 / d;
    const int rem = r - k;
    for (int e = tid; e < rem * rem; e += nt) {
      const int i = k + e / rem, j = k + e % rem;
      if (j == k) {
        L[i * ld + k] = (i == k) ? c2{piv, 0.0} : c2{A[i * ld + k].r / piv, A[i * ld + k].i / piv};
      } else if (i > k) {
        const c2 t = cmulc(A[j * ld + k], A[i * ld + k]);
        A[i * ld + j] = {A[i * ld + j].r - t.r * invd, A[i * ld + j].i - t.i * invd};
      }
    }
    __syncthreads();
  }
}

// Unit vectors of the real symmetric tridiagonal (dd, ee) for the eigenvalues lam (ascending, ns of them)
// in clusters, that is closer than 1e-6 tn to a neighbour: inverse iteration on T - lambda I with
// partial pivoting, one wave per cluster, every lane factorising and solving for one member; after each
// of the three solves the members are Gram-Schmidt-orthogonalised in order (lanes over the rows).
// lu(c): 3 r doubles for member c's factors; vec(c): its vector, r doubles; done(c): called by one lane
// when vec(c) has been normalised.
template <typename LU, typename Vec, typename Done>
__device__ __forceinline__ void cluster_vectors(const double* dd, const double* ee, const double* lam, int r, int ns,
                                                double tn, double tiny, const LU& lu, const Vec& vec, const Done& done) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, nw = (int)blockDim.x >> 6;
  int ci = 0;
  for (int j = 0; j < ns;) {
    int jend = j + 1;
    while (jend < ns && lam[jend] - lam[jend - 1] <= 1e-6 * tn) ++jend;
    if (jend - j > 1 && (ci++ % nw) == wv) {
      const int k = jend - j;
      for (int c0 = 0; c0 < k; c0 += 64) {   // members, 64 at a time (lanes)
        const int c = j + c0 + lane;
        if (c0 + lane < k) {
          double* u = lu(c);
          double* u1 = u + r;    // U: reciprocal diagonal and first super-diagonal; the second
          double* lm = u1 + r;   // super-diagonal is e_{i+1} after a row swap, else 0.
                                 // Multipliers; a row swap is encoded as -(mult) - 4.
          const double shift = lam[c];
          // elimination with partial pivoting: the carried row has entries (a_i, b_i) in
          // columns (i, i+1); the next row is (e_i, d_{i+1} - shift, e_{i+1})
          double a_i = dd[0] - shift, b_i = ee[0];
          for (int i = 0; i < r - 1; ++i) {
            const double sub = ee[i];
            const double dnext = dd[i + 1] - shift, bnext = ee[i + 1];
            if (fabs(sub) > fabs(a_i)) {              // swap rows i and i+1
              const double rs = rcp_nr(sub);
              const double mlt = a_i * rs;
              u[i] = rs;
              u1[i] = dnext;
              lm[i] = -mlt - 4.0;                     // |mult| <= 1, so lm <= -3 marks a swap
              a_i = b_i - mlt * dnext;
              b_i = -mlt * bnext;
            } else {
              const double aa = fabs(a_i) > tiny ? a_i : (a_i < 0 ? -tiny : tiny);
              const double ra = rcp_nr(aa);
              const double mlt = sub * ra;
              u[i] = ra;
              u1[i] = b_i;
              lm[i] = mlt;                            // |mult| <= 1
              a_i = dnext - mlt * b_i;
              b_i = bnext;
            }
          }
          u[r - 1] = rcp_nr(fabs(a_i) > tiny ? a_i : (a_i < 0 ? -tiny : tiny));
          u1[r - 1] = 0.0;
          lm[r - 1] = 0.0;
          double* x = vec(c);
          for (int i = 0; i < r; ++i) x[i] = 1.0 + 0.0625 * (double)((i * 7 + c * 3) % 11);
        }
      }
      for (int rep = 0; rep < 3; ++rep) {
        for (int c0 = 0; c0 < k; c0 += 64) {
          const int c = j + c0 + lane;
          if (c0 + lane < k) {
            const double* u = lu(c);
            const double* u1 = u + r;
            const double* lm = u1 + r;
            double* x = vec(c);
            // forward: apply the row operations to x (the running entry carried in a register)
            double xi = x[0];
            for (int i = 0; i < r - 1; ++i) {
              const double l = lm[i], xn = x[i + 1];
              if (l <= -3.0) {   // swapped: new row i <- old row i+1; row i+1 <- old i - mult*old i+1
                const double mlt = -(l + 4.0);
                x[i] = xn;
                xi = xi - mlt * xn;
              } else {
                x[i] = xi;
                xi = xn - l * xi;
              }
            }
            x[r - 1] = xi;
            // back substitution with U (the two entries below carried in registers)
            double x1 = 0.0, x2 = 0.0;
            for (int i = r - 1; i >= 0; --i) {
              double sacc = x[i];
              if (i + 1 < r) sacc -= u1[i] * x1;
              if (i + 2 < r && lm[i] <= -3.0) sacc -= ee[i + 1] * x2;
              const double xv = sacc * u[i];
              x[i] = xv;
              x2 = x1;
              x1 = xv;
            }
          }
        }
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
        // orthogonalise each member against the earlier ones, normalise (lanes over rows)
        for (int c = j; c < jend; ++c) {
          double* x = vec(c);
          for (int pc = j; pc < c; ++pc) {
            const double* y = vec(pc);
            double part = 0;
            for (int i = lane; i < r; i += 64) part += y[i] * x[i];
            const double dot = wave_sum(part);
            for (int i = lane; i < r; i += 64) x[i] -= dot * y[i];
          }
          double part = 0;
          for (int i = lane; i < r; i += 64) part += x[i] * x[i];
          const double nrm = sqrt(wave_sum(part));
          const double inv = nrm > 0 ? 1.0 / nrm : 0.0;
          for (int i = lane; i < r; i += 64) x[i] *= inv;
          if (lane == 0) done(c);
          __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
          __builtin_amdgcn_wave_barrier();
        }
      }
    }
    j = jend;
  }
}

}  // namespace

}  // namespace bl

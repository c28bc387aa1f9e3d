// Dense kernels of the iteration (Section 4 and 5) for gfx950:
//  * coarsest-level direct solve: the coarse operator is assembled by applying the stencil
//    to unit vectors, inverted in place by block Gauss-Jordan steps (Hermitian positive
//    definite, no pivoting), and applied as a dense matrix-vector product;
//  * tall-skinny Gram products X^* W of planar FP64 blocks (LDS-staged, register-tiled);
//  * block recombination S Y.
#include "stencil_common.h"

#include <type_traits>

#include <cmath>
#include <cstdio>
#include <cstdlib>

// The coarse solve is repeated inside the fused coarse cycles (coarse.hip) with the same
// operations; no contraction on either side keeps the two bit-identical.
#pragma clang fp contract(off)

namespace bl {

struct c2 {
  double r, i;
};
__device__ __forceinline__ c2 cm(c2 a, c2 b) { return {a.r * b.r - a.i * b.i, a.r * b.i + a.i * b.r}; }
__device__ __forceinline__ c2 cmc(c2 a, c2 b) { return {a.r * b.r + a.i * b.i, a.r * b.i - a.i * b.r}; }  // conj(a)*b

// ------------------------------------------------------------------------------------------
__global__ void k_identity_block(double* __restrict__ out, int64_t n) {
  const int64_t j = blockIdx.y;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  out[j * 2 * n + i] = (i == j) ? 1.0 : 0.0;
  out[j * 2 * n + n + i] = 0.0;
}
void identity_block(double* out, int64_t n, hipStream_t st) {
  dim3 grid((unsigned)((n + 255) / 256), (unsigned)n);
  k_identity_block<<<grid, 256, 0, st>>>(out, n);
}

// mat_s (row-major interleaved) [i][j] = column j of slot s's probe result at row i
__global__ void k_planar_to_matrix(const double* __restrict__ cols, int64_t n, double* __restrict__ mat,
                                   const int* __restrict__ slots) {
  const int64_t j = blockIdx.y;
  const int64_t s = slots ? slots[blockIdx.z] : blockIdx.z;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double* c = cols + s * n * 2 * n;
  double* o = mat + s * n * n * 2;
  o[2 * (i * n + j)] = c[j * 2 * n + i];
  o[2 * (i * n + j) + 1] = c[j * 2 * n + n + i];
}
void planar_to_matrix(const double* cols, int64_t n, double* mat, const Launch& L) {
  if (L.nact <= 0) return;
  dim3 grid((unsigned)((n + 255) / 256), (unsigned)n, (unsigned)L.nact);
  k_planar_to_matrix<<<grid, 256, 0, L.st>>>(cols, n, mat, L.slots);
}

__global__ void k_add_rank_one(double* __restrict__ mat, int64_t n, double gamma, const int* __restrict__ slots) {
  const int64_t s = slots ? slots[blockIdx.y] : blockIdx.y;
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e < n * n) mat[s * n * n * 2 + 2 * e] += gamma / (double)n;
}
void add_constant_rank_one(double* mat, int64_t n, double gamma, const Launch& L) {
  if (L.nact <= 0) return;
  k_add_rank_one<<<dim3((unsigned)((n * n + 255) / 256), (unsigned)L.nact), 256, 0, L.st>>>(mat, n, gamma, L.slots);
}

// In-place inversion of Hermitian positive definite matrices by block Gauss-Jordan steps (no
// pivoting), one launch per block column of IB unknowns, a workgroup per IB x IB tile, all slots
// and both coarse matrices of a slot (edge and nodal) in the same launches.
//
// Bound by latency: n dependent pivots.  One workgroup per matrix sweeping scalar pivots streams
// the whole matrix through one compute unit at each of them: 618 + 176 us for the 128 edges and
// 64 nodes of an 8 x 8 level, 4.9 + 1.2 ms for the 270 and 135 of a 15 x 9 one.  Here a step
// takes IB pivots at once and its tiles spread over the device, so the chain is n / IB launches
// of 19 us: 81 us and 176 us for both matrices.  Every workgroup inverts the pivot block itself
// (32 short steps in registers, one barrier each): less than another dependent launch costs.
//
// Step k replaces, with P the inverse of the pivot block, A_kk by P, A_kj by P A_kj, A_ik by
// -A_ik P and A_ij by A_ij - A_ik P A_kj.  The other tiles of the step still read block row and
// column k, so their new values go to panels (by step parity) and are read from there by step
// k + 1, which writes them back; k_invert_finish writes the last step's panels back and the
// single-precision copy.
constexpr int IB = 32;

struct InvMat {
  c2* a;          // n x n per slot
  float* a32;     // single-precision copy (2 n n values per slot)
  c2* panel;      // 4 IB n per slot: row panels (2 x IB x n), then column panels (2 x n x IB)
  int n;
};

// Tile (I, J) before step k: in the panels of step k - 1 or in the matrix (the same choice for
// the whole workgroup, so that all of its loads can be issued together).
struct InvTile {
  const c2* p;
  int64_t stride;
};
__device__ __forceinline__ InvTile inv_tile(const InvMat& M, int64_t slot, int k, int I, int J) {
  const int64_t n = M.n, par = (k - 1) & 1;
  const c2* pan = M.panel + slot * 4 * IB * n;
  if (k > 0 && I == k - 1) return {pan + par * IB * n + J * IB, n};
  if (k > 0 && J == k - 1) return {pan + 2 * IB * n + (par * n + (int64_t)I * IB) * IB, IB};
  return {M.a + slot * n * n + (int64_t)I * IB * n + (int64_t)J * IB, n};
}

__global__ __launch_bounds__(256) void k_invert_step(InvMat me, InvMat mn, int k, const int* __restrict__ slots) {
  const InvMat M = (blockIdx.z & 1) ? mn : me;
  const int64_t slot = slots ? slots[blockIdx.z >> 1] : (int)(blockIdx.z >> 1);
  const int nb = (M.n + IB - 1) / IB;
  const int I = (int)blockIdx.y, J = (int)blockIdx.x;
  if (k >= nb || I >= nb || J >= nb) return;
  __shared__ c2 P[IB][IB + 1], X[IB][IB + 1], Y[IB][IB + 1];
  __shared__ c2 rowb[2][IB], colb[2][IB];
  const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
  // pivot block, own tile, and the tile's blocks of block column and row k: every load issued
  // before the first use (entries past the matrix read entry 0 of their tile and are replaced by
  // the identity in the pivot block, by zero elsewhere)
  double er[2][2], ei[2][2];   // (apart, so that the selects below keep them in registers)
  c2 own[2][2], xv[2][2], yv[2][2];
  const InvTile tp = inv_tile(M, slot, k, k, k), to = inv_tile(M, slot, k, I, J), tc = inv_tile(M, slot, k, I, k),
                tr = inv_tile(M, slot, k, k, J);
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const int i = ty + 16 * a, j = tx + 16 * b;
      const bool pi = IB * k + i < M.n, pj = IB * k + j < M.n, oi = IB * I + i < M.n, oj = IB * J + j < M.n;
      const c2 v = tp.p[pi && pj ? i * tp.stride + j : 0];
      own[a][b] = to.p[oi && oj ? i * to.stride + j : 0];
      xv[a][b] = tc.p[oi && pj ? i * tc.stride + j : 0];
      yv[a][b] = tr.p[pi && oj ? i * tr.stride + j : 0];
      er[a][b] = v.r;
      ei[a][b] = v.i;
    }
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const int i = ty + 16 * a, j = tx + 16 * b;
      const bool pi = IB * k + i < M.n, pj = IB * k + j < M.n, oi = IB * I + i < M.n, oj = IB * J + j < M.n;
      er[a][b] = pi && pj ? er[a][b] : (i == j ? 1.0 : 0.0);
      ei[a][b] = pi && pj ? ei[a][b] : 0.0;
      X[i][j] = c2{oi && pj ? xv[a][b].r : 0.0, oi && pj ? xv[a][b].i : 0.0};
      Y[i][j] = c2{pi && oj ? yv[a][b].r : 0.0, pi && oj ? yv[a][b].i : 0.0};
    }
#pragma unroll
  for (int hi = 0; hi < 2; ++hi)   // the pivot's register row and column are compile-time indices
#pragma unroll 1
  for (int lo = 0; lo < 16; ++lo) {
    const int s = 16 * hi + lo, par = s & 1;
    if (ty == lo) {
#pragma unroll
      for (int b = 0; b < 2; ++b) rowb[par][tx + 16 * b] = c2{er[hi][b], ei[hi][b]};
    }
    if (tx == lo) {
#pragma unroll
      for (int a = 0; a < 2; ++a) colb[par][ty + 16 * a] = c2{er[a][hi], ei[a][hi]};
    }
    __syncthreads();
    const c2 pv = rowb[par][s];
    const c2 r0 = rowb[par][tx], r1 = rowb[par][tx + 16], f0 = colb[par][ty], f1 = colb[par][ty + 16];
    const double d = 1.0 / (pv.r * pv.r + pv.i * pv.i);
    const c2 p = {pv.r * d, -pv.i * d};
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const bool pc = tx + 16 * b == s;   // the pivot column
      const c2 q = cm(b ? r1 : r0, p);
      const double qr = pc ? p.r : q.r, qi = pc ? p.i : q.i;
#pragma unroll
      for (int a = 0; a < 2; ++a) {
        const bool prow = ty + 16 * a == s;   // the pivot row
        const c2 v = cm(a ? f1 : f0, c2{qr, qi});
        er[a][b] = prow ? qr : (pc ? 0.0 : er[a][b]) - v.r;
        ei[a][b] = prow ? qi : (pc ? 0.0 : ei[a][b]) - v.i;
      }
    }
  }
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) P[ty + 16 * a][tx + 16 * b] = c2{er[a][b], ei[a][b]};
  __syncthreads();
  // C = A B over the 32-wide blocks, 2 x 2 entries per thread
  auto mul = [&](const c2(*A)[IB + 1], const c2(*B)[IB + 1], c2(&c)[2][2]) {
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b) c[a][b] = c2{0.0, 0.0};
#pragma unroll 4
    for (int l = 0; l < IB; ++l) {
      const c2 a0 = A[ty][l], a1 = A[ty + 16][l], b0 = B[l][tx], b1 = B[l][tx + 16];
      const c2 av[2] = {a0, a1}, bv[2] = {b0, b1};
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          c[a][b].r = fma(-av[a].i, bv[b].i, fma(av[a].r, bv[b].r, c[a][b].r));
          c[a][b].i = fma(av[a].i, bv[b].r, fma(av[a].r, bv[b].i, c[a][b].i));
        }
    }
  };
  c2 out[2][2];
  if (I == k && J == k) {
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b) out[a][b] = c2{er[a][b], ei[a][b]};
  } else if (I == k) {
    mul(P, Y, out);
  } else if (J == k) {
    mul(X, P, out);
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b) out[a][b] = c2{-out[a][b].r, -out[a][b].i};
  } else {
    c2 t[2][2];
    mul(P, Y, t);
    __syncthreads();   // (uniform over the workgroup) Y is replaced by P Y
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b) Y[ty + 16 * a][tx + 16 * b] = t[a][b];
    __syncthreads();
    mul(X, Y, t);
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b) out[a][b] = c2{own[a][b].r - t[a][b].r, own[a][b].i - t[a][b].i};
  }
  const int64_t n = M.n, par = k & 1;
  c2* pan = M.panel + slot * 4 * IB * n;
  c2* A = M.a + slot * n * n;
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const int i = IB * I + ty + 16 * a, j = IB * J + tx + 16 * b;
      if (i >= n || j >= n) continue;
      if (I == k) pan[(par * IB + i % IB) * n + j] = out[a][b];
      else if (J == k) pan[2 * IB * n + (par * n + i) * IB + j % IB] = out[a][b];
      else A[(int64_t)i * n + j] = out[a][b];
    }
}

// The last step's panels back into the matrix, and its single-precision copy.
__global__ __launch_bounds__(256) void k_invert_finish(InvMat me, InvMat mn, const int* __restrict__ slots) {
  const InvMat M = (blockIdx.y & 1) ? mn : me;
  const int64_t slot = slots ? slots[blockIdx.y >> 1] : (int)(blockIdx.y >> 1);
  const int64_t n = M.n, e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n * n) return;
  const int i = (int)(e / n), j = (int)(e % n), nb = (M.n + IB - 1) / IB;
  const InvTile t = inv_tile(M, slot, nb, i / IB, j / IB);
  const c2 v = t.p[(int64_t)(i % IB) * t.stride + j % IB];
  if (i / IB == nb - 1 || j / IB == nb - 1) M.a[slot * n * n + e] = v;
  float* o = M.a32 + 2 * (slot * n * n + e);
  o[0] = (float)v.r;
  o[1] = (float)v.i;
}

size_t invert_panel_doubles(int64_t ne, int64_t nn) { return (size_t)8 * IB * (ne + nn); }

void invert_coarse(double* ke, float* ke32, int64_t ne, double* kn, float* kn32, int64_t nn, int nslots, double* panel,
                   const Launch& L) {
  if (L.nact <= 0) return;
  const InvMat me{reinterpret_cast<c2*>(ke), ke32, reinterpret_cast<c2*>(panel), (int)ne};
  const InvMat mn{reinterpret_cast<c2*>(kn), kn32, reinterpret_cast<c2*>(panel) + (size_t)nslots * 4 * IB * ne, (int)nn};
  const int64_t big = ne > nn ? ne : nn;
  const unsigned nb = (unsigned)((big + IB - 1) / IB);
  for (unsigned k = 0; k < nb; ++k)
    k_invert_step<<<dim3(nb, nb, (unsigned)(2 * L.nact)), 256, 0, L.st>>>(me, mn, (int)k, L.slots);
  k_invert_finish<<<dim3((unsigned)((big * big + 255) / 256), (unsigned)(2 * L.nact)), 256, 0, L.st>>>(me, mn, L.slots);
}

// x = Inv_s b: 64 rows per workgroup, one per lane, for NC columns; each of the eight waves sums one of a
// row's parts (dense_part), which then combine in LDS.  Bound by latency, but where the matrix exceeds an
// XCD's L2 (4 MB) by reading it, the workgroups of the columns being at different places of it: 1800
// edges FP64, 48 columns 102 us with four columns a workgroup, 349 with one.
template <typename T, int NC>
__global__ __launch_bounds__(64 * kDenseParts) void k_dense_apply_parts(const T* __restrict__ inv, int n, View<const T> bv,
                                                                        View<T> xv, const int* __restrict__ slots, int ncps) {
  __shared__ T part[NC][2 * kDenseParts][64];
  const SJ g = slot_col(slots, (ncps + NC - 1) / NC);
  const int lane = (int)threadIdx.x & 63, k = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int i = (int)blockIdx.x * 64 + lane;
  inv += (int64_t)g.slot * n * n * 2;
  const T* b[NC];   // (columns past the last: the last one again, not stored)
#pragma unroll
  for (int c = 0; c < NC; ++c) b[c] = colp(bv, SJ{g.slot, min(g.j * NC + c, ncps - 1)}, n);
  if (i < n) {
    Cx<T> v[NC];
    dense_part<NC>(inv, n, b, i, n * k / kDenseParts, n * (k + 1) / kDenseParts, v);
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      part[c][2 * k][lane] = v[c].re;
      part[c][2 * k + 1][lane] = v[c].im;
    }
  }
  __syncthreads();
  const int c = k >> 1, p = k & 1;   // real, then imaginary parts
  if (c < NC && g.j * NC + c < ncps && i < n)
    colp(xv, SJ{g.slot, g.j * NC + c}, n)[p * n + i] = dense_sum([&](int q) { return part[c][2 * q + p][lane]; });
}
// The same with the terms one after the other: 64 rows per workgroup, one per lane.
template <typename T>
__global__ __launch_bounds__(64) void k_dense_apply(const T* __restrict__ inv, int n, View<const T> bv, View<T> xv,
                                                    const int* __restrict__ slots, int ncps) {
  const SJ sj = slot_col(slots, ncps);
  const int i = (int)(blockIdx.x * 64 + threadIdx.x);
  if (i >= n) return;
  const Cx<T> v = dense_row<T>(inv + (int64_t)sj.slot * n * n * 2, n, colp(bv, sj, n), i);
  T* xc = colp(xv, sj, n);
  xc[i] = v.re;
  xc[n + i] = v.im;
}
template <typename T>
void dense_apply(const void* inv, int64_t n, bool edge, View<const T> b, View<T> x, const Launch& L) {
  const unsigned rows = (unsigned)((n + 63) / 64);
  if (L.nact * L.ncps == 0) return;
  const T* m = reinterpret_cast<const T*>(inv);
  if constexpr (!dense_in_parts<T>(false))
    if (!edge) {
      k_dense_apply<T><<<dim3(rows, (unsigned)(L.nact * L.ncps)), 64, 0, L.st>>>(m, (int)n, b, x, L.slots, L.ncps);
      return;
    }
  // several columns a workgroup where the matrix exceeds an XCD's L2, as long as every compute unit has one
  auto go = [&](auto ncc) {
    constexpr int NC = decltype(ncc)::value;
    const unsigned cols = (unsigned)(L.nact * ((L.ncps + NC - 1) / NC));
    if (NC > 1 && (2 * n * n * (int64_t)sizeof(T) <= (4 << 20) || rows * cols < 256)) return false;
    k_dense_apply_parts<T, NC><<<dim3(rows, cols), 64 * kDenseParts, 0, L.st>>>(m, (int)n, b, x, L.slots, L.ncps);
    return true;
  };
  if (!go(std::integral_constant<int, 4>{}) && !go(std::integral_constant<int, 2>{})) go(std::integral_constant<int, 1>{});
}
template void dense_apply<double>(const void*, int64_t, bool, View<const double>, View<double>, const Launch&);
template void dense_apply<float>(const void*, int64_t, bool, View<const float>, View<float>, const Launch&);

// ------------------------------------------------------------------------------------------
// Gram products.  Block (16 x 16 threads) computes a 64 x 64 tile of X^* W over a range of
// rows; rows are staged through LDS 16 at a time; each thread owns a 4 x 4 register tile.
constexpr int GB = 64, GTR = 16;

__global__ __launch_bounds__(256) void k_gram(View<const double> Xv, int q, View<const double> Wv, int r,
                                              int64_t len, int64_t rows_per_blk,
                                              double* __restrict__ partial,
                                              const int* __restrict__ slots) {
  __shared__ double xr[GTR][GB], xi[GTR][GB], wr[GTR][GB], wi[GTR][GB];
  const int slot = slots ? slots[blockIdx.z] : (int)blockIdx.z;
  const double* X = Xv.p + ((int64_t)slot * Xv.cps + Xv.off) * 2 * len;
  const double* W = Wv.p + ((int64_t)slot * Wv.cps + Wv.off) * 2 * len;
  const int ntj = (r + GB - 1) / GB;
  const int i0 = (blockIdx.y / ntj) * GB, j0 = (blockIdx.y % ntj) * GB;
  const int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4;
  const int64_t rs = (int64_t)blockIdx.x * rows_per_blk;
  const int64_t re = rs + rows_per_blk < len ? rs + rows_per_blk : len;
  double ar[4][4], ai[4][4];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) { ar[a][b] = 0; ai[a][b] = 0; }
  for (int64_t r0 = rs; r0 < re; r0 += GTR) {
    for (int e = tid; e < GTR * GB; e += 256) {
      const int rr = e % GTR, cc = e / GTR;
      const int64_t row = r0 + rr;
      const bool okr = row < re;
      const int cx = i0 + cc, cw = j0 + cc;
      xr[rr][cc] = (okr && cx < q) ? X[(int64_t)cx * 2 * len + row] : 0.0;
      xi[rr][cc] = (okr && cx < q) ? X[(int64_t)cx * 2 * len + len + row] : 0.0;
      wr[rr][cc] = (okr && cw < r) ? W[(int64_t)cw * 2 * len + row] : 0.0;
      wi[rr][cc] = (okr && cw < r) ? W[(int64_t)cw * 2 * len + len + row] : 0.0;
    }
    __syncthreads();
#pragma unroll 4
    for (int rr = 0; rr < GTR; ++rr) {
      double x_r[4], x_i[4], w_r[4], w_i[4];
#pragma unroll
      for (int a = 0; a < 4; ++a) { x_r[a] = xr[rr][ty * 4 + a]; x_i[a] = xi[rr][ty * 4 + a]; }
#pragma unroll
      for (int b = 0; b < 4; ++b) { w_r[b] = wr[rr][tx * 4 + b]; w_i[b] = wi[rr][tx * 4 + b]; }
#pragma unroll
      for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          ar[a][b] += x_r[a] * w_r[b] + x_i[a] * w_i[b];
          ai[a][b] += x_r[a] * w_i[b] - x_i[a] * w_r[b];
        }
    }
    __syncthreads();
  }
  double* pp = partial + ((int64_t)blockIdx.z * gridDim.x + blockIdx.x) * q * r * 2;
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const int i = i0 + ty * 4 + a, j = j0 + tx * 4 + b;
      if (i < q && j < r) {
        pp[2 * ((int64_t)i * r + j)] = ar[a][b];
        pp[2 * ((int64_t)i * r + j) + 1] = ai[a][b];
      }
    }
}

// out_s = sum over the row blocks of the launch entry z (slot s = slots[z]) in block order
__global__ void k_gram_reduce(const double* __restrict__ partial, int nblk, int64_t count,
                              double* __restrict__ out, const int* __restrict__ slots) {
  const int z = blockIdx.y;
  const int64_t slot = slots ? slots[z] : z;
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= count) return;
  const double* p = partial + (int64_t)z * nblk * count;
  double s = 0;
  for (int b = 0; b < nblk; ++b) s += p[(int64_t)b * count + e];
  out[slot * count + e] = s;
}

// Row blocks of one Gram product: a function of the vector length only, so that a slot's
// sums do not depend on which other slots share the launch.
int gram_blocks(int64_t len) {
  int64_t nb = (len + 1023) / 1024;
  if (nb > 256) nb = 256;
  if (nb < 1) nb = 1;
  int64_t rpb = (len + nb - 1) / nb;
  rpb = (rpb + GTR - 1) / GTR * GTR;
  return (int)((len + rpb - 1) / rpb);
}

int gram(View<const double> X, int q, View<const double> W, int r, int64_t len, double* partial,
         int64_t partial_cap, double* out, const Launch& L) {
  if (L.nact <= 0) return 0;
  const int nb = gram_blocks(len);
  if ((int64_t)nb * q * r * 2 * L.nact > partial_cap) return -1;
  int64_t rpb = (len + nb - 1) / nb;
  rpb = (rpb + GTR - 1) / GTR * GTR;
  const int nti = (q + GB - 1) / GB, ntj = (r + GB - 1) / GB;
  dim3 grid((unsigned)nb, (unsigned)(nti * ntj), (unsigned)L.nact);
  k_gram<<<grid, 256, 0, L.st>>>(X, q, W, r, len, rpb, partial, L.slots);
  const int64_t count = (int64_t)q * r * 2;
  k_gram_reduce<<<dim3((unsigned)((count + 255) / 256), (unsigned)L.nact), 256, 0, L.st>>>(partial, nb, count, out, L.slots);
  return 0;
}

// ------------------------------------------------------------------------------------------
// out_s[:, j] = sum_l S_s[:, l] Y_s[l][j]; thread per row, 8 output columns per workgroup.  The
// column blocks of one row range are neighbouring workgroups (blockIdx.x = range * blocks +
// column block), so they run together and read the basis rows through L2 once from memory.
namespace {

// Block combination out_s = S_s Y_s on the matrix cores (FP64 MFMA 16x16x4), computed as
// out^T = Y^T S^T so that each lane's results are consecutive rows of one output column
// (coalesced stores): the A operand is Y (staged in LDS once per workgroup, real and
// imaginary parts apart, zero-padded to whole tiles), the B operand the basis rows straight
// from memory.  A complex product takes three real ones (Gauss's three-multiplication form):
//   P1 = Yr Sr,  P2 = Yi Si,  P3 = (Yr + Yi)(Sr + Si),  Re = P1 - P2,  Im = P3 - P1 - P2,
// each summed over the basis columns in its own accumulator.  The workgroups are persistent:
// each wave walks row tiles of BCR rows (tile t, t + stride, ...) for the NTC output column
// tiles of its workgroup (blockIdx.y selects the tile group when the block is wider), one
// stream of steps of four basis columns across its tiles, with the columns two steps ahead
// (possibly of the next tile) loaded while the current ones are multiplied.  (The file is
// compiled with MFMA results in ordinary VGPRs, so the accumulators stay put across the loop.)
typedef double bd4 __attribute__((ext_vector_type(4)));
constexpr int BCW = 4;    // waves per workgroup
constexpr int BCR = 32;   // rows per tile (two 16-row MFMA tiles)

template <int NTC>
__global__ __launch_bounds__(64 * BCW) void k_block_combine(View<const double> Sv, int q, const c2* __restrict__ Y,
                                                            int want, int64_t len, View<double> ov,
                                                            const int* __restrict__ slots) {
  extern __shared__ double yl[];   // yr then yi, each q4 x 16 NTC
  constexpr int WC = 16 * NTC;
  const int q4 = (q + 3) & ~3;
  const int cbase = (int)blockIdx.y * WC;   // first output column of the workgroup
  const int slot = slots ? slots[blockIdx.z] : (int)blockIdx.z;
  const double* S = Sv.p + ((int64_t)slot * Sv.cps + Sv.off) * 2 * len;
  double* out = ov.p + ((int64_t)slot * ov.cps + ov.off) * 2 * len;
  Y += (int64_t)slot * q * want;
  double* yr = yl;
  double* yi = yl + (size_t)q4 * WC;
  {
    // all of a thread's loads first, then the stores
    constexpr int PER = 8;
    for (int e0 = threadIdx.x; e0 < q4 * WC; e0 += PER * (int)blockDim.x) {
      c2 v[PER];
#pragma unroll
      for (int u = 0; u < PER; ++u) {
        const int e = e0 + u * (int)blockDim.x, l = e / WC, c = cbase + e % WC;
        v[u] = (e < q4 * WC && l < q && c < want) ? Y[(int64_t)l * want + c] : c2{0, 0};
      }
#pragma unroll
      for (int u = 0; u < PER; ++u) {
        const int e = e0 + u * (int)blockDim.x;
        if (e < q4 * WC) {
          yr[e] = v[u].r;
          yi[e] = v[u].i;
        }
      }
    }
  }
  __syncthreads();
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int64_t ntiles = (len + BCR - 1) / BCR;
  const int64_t tstride = (int64_t)gridDim.x * BCW;
  int64_t ct = (int64_t)blockIdx.x * BCW + wv;   // tile being multiplied
  if (ct >= ntiles) return;
  const int kk = lane >> 4, cc = lane & 15;
  bd4 p1[2][NTC], p2[2][NTC], p3[2][NTC];
#pragma unroll
  for (int rt = 0; rt < 2; ++rt)
#pragma unroll
    for (int c = 0; c < NTC; ++c) p1[rt][c] = p2[rt][c] = p3[rt][c] = bd4{0, 0, 0, 0};
  // basis column l0 + kk of this lane's two rows of tile t (zero past the basis, the rows or
  // the last tile)
  auto load = [&](int64_t t, int l0, double* sr, double* si) {
    const int l = l0 + kk;
    const int64_t off = (int64_t)(l < q ? l : q - 1) * 2 * len;
#pragma unroll
    for (int rt = 0; rt < 2; ++rt) {
      const int64_t row = t * BCR + 16 * rt + cc;
      const bool ok = t < ntiles && l < q && row < len;
      const double* rp = S + (ok ? row : 0) + (ok ? off : 0);
      const double a = rp[0], b = rp[len];
      sr[rt] = ok ? a : 0.0;
      si[rt] = ok ? b : 0.0;
    }
  };
  // prefetch position (tile pt, columns pl0 ..), two steps ahead of the multiplication
  int64_t pt = ct;
  int pl0 = 0;
  auto advance = [&]() {
    pl0 += 4;
    if (pl0 >= q4) {
      pl0 = 0;
      pt += tstride;
    }
  };
  double s0r[2], s0i[2], s1r[2], s1i[2], s2r[2], s2i[2];
  load(pt, pl0, s0r, s0i);
  advance();
  load(pt, pl0, s1r, s1i);
  advance();
  int cl0 = 0;
  for (;;) {
    load(pt, pl0, s2r, s2i);
    advance();
    const int l = cl0 + kk;
    double ss[2];
#pragma unroll
    for (int rt = 0; rt < 2; ++rt) ss[rt] = s0r[rt] + s0i[rt];
#pragma unroll
    for (int c = 0; c < NTC; ++c) {
      const double yre = yr[l * WC + 16 * c + cc], yim = yi[l * WC + 16 * c + cc];
      const double ys = yre + yim;
#pragma unroll
      for (int rt = 0; rt < 2; ++rt) {
        p1[rt][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(yre, s0r[rt], p1[rt][c], 0, 0, 0);
        p2[rt][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(yim, s0i[rt], p2[rt][c], 0, 0, 0);
        p3[rt][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(ys, ss[rt], p3[rt][c], 0, 0, 0);
      }
    }
#pragma unroll
    for (int rt = 0; rt < 2; ++rt) {
      s0r[rt] = s1r[rt];
      s0i[rt] = s1i[rt];
      s1r[rt] = s2r[rt];
      s1i[rt] = s2i[rt];
    }
    cl0 += 4;
    if (cl0 < q4) continue;
    // tile ct done: accumulator entry v of lane (kk, cc) is output column 16 c + 4 v + kk of
    // row 16 rt + cc of the tile (the 16 x 16 result of the instruction has row 4 v + lane / 16
    // and column lane % 16)
#pragma unroll
    for (int rt = 0; rt < 2; ++rt) {
      const int64_t row = ct * BCR + 16 * rt + cc;
#pragma unroll
      for (int c = 0; c < NTC; ++c)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int col = cbase + 16 * c + 4 * v + kk;
          if (col < want && row < len) {
            const double a = p1[rt][c][v], b = p2[rt][c][v];
            out[(int64_t)col * 2 * len + row] = a - b;
            out[(int64_t)col * 2 * len + len + row] = (p3[rt][c][v] - a) - b;
          }
        }
    }
    ct += tstride;
    if (ct >= ntiles) break;
    cl0 = 0;
#pragma unroll
    for (int rt = 0; rt < 2; ++rt)
#pragma unroll
      for (int c = 0; c < NTC; ++c) p1[rt][c] = p2[rt][c] = p3[rt][c] = bd4{0, 0, 0, 0};
  }
}

}  // namespace

void block_combine(View<const double> S, int q, const double* Y, int want, int64_t len,
                   View<double> out, const Launch& L) {
  if (L.nact <= 0 || want <= 0) return;
  const int q4 = (q + 3) & ~3;
  const int ntc = (want + 15) / 16;
  // column tiles per workgroup: up to three, as many as the staged Y allows in 160 KB of LDS
  const size_t tile_lds = (size_t)2 * q4 * 16 * sizeof(double);
  int per = 3;
  while (per > 1 && tile_lds * per > (size_t)160 * 1024) --per;
  if (per > ntc) per = ntc;
  const int ny = (ntc + per - 1) / per;
  // persistent workgroups: as many as stay resident together (by LDS, at most two per compute
  // unit), spread over the column groups and slots of the launch
  static const int cus = [] {   // initialised once, thread-safely
    int dev = 0, c = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&c, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || c <= 0)
      c = 256;
    return c;
  }();
  const int per_cu = tile_lds * per <= (size_t)80 * 1024 ? 2 : 1;
  const int64_t tiles_wg = ((len + BCR - 1) / BCR + BCW - 1) / BCW;
  int64_t nx = ((int64_t)cus * per_cu + (int64_t)ny * L.nact - 1) / ((int64_t)ny * L.nact);
  if (nx < 1) nx = 1;
  if (nx > tiles_wg) nx = tiles_wg;
  const dim3 grid((unsigned)nx, (unsigned)ny, (unsigned)L.nact);
  auto go = [&](auto nt) {
    constexpr int NTC = decltype(nt)::value;
    static const bool attr = [&] {   // once per instantiation, thread-safely
      (void)hipFuncSetAttribute((const void*)k_block_combine<NTC>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                160 * 1024);
      return true;
    }();
    (void)attr;
    k_block_combine<NTC><<<grid, 64 * BCW, tile_lds * NTC, L.st>>>(S, q, reinterpret_cast<const c2*>(Y), want, len,
                                                                  out, L.slots);
  };
  if (per == 1) go(std::integral_constant<int, 1>{});
  else if (per == 2) go(std::integral_constant<int, 2>{});
  else go(std::integral_constant<int, 3>{});
}

// ------------------------------------------------------------------------------------------
// In-place column compaction: column k of the view receives column src[k] (k < ncols,
// src[k] >= k, strictly increasing per slot).  Every thread owns one 16-byte position of
// all columns, so threads never touch each other's data; a thread loads a chunk of source
// columns before it stores them (a destination may be the source of a later column of the
// chunk), and a later chunk's sources lie above every earlier destination.
template <typename T>
__global__ void k_compact_cols(View<T> v, int64_t len, const int* __restrict__ src, int src_stride, int ncols,
                               const int* __restrict__ slots) {
  using V = typename std::conditional<sizeof(T) == 4, float4, double2>::type;
  constexpr int CH = 8;
  const int z = blockIdx.y;
  const int sl = slots ? slots[z] : z;
  const int* sk = src + (int64_t)z * src_stride;
  const int64_t nvec = 2 * len * (int64_t)sizeof(T) / (int64_t)sizeof(V);
  V* base = reinterpret_cast<V*>(v.p + ((int64_t)sl * v.cps + v.off) * 2 * len);
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nvec; i += (int64_t)gridDim.x * blockDim.x) {
    for (int k0 = 0; k0 < ncols; k0 += CH) {
      V buf[CH];
#pragma unroll
      for (int u = 0; u < CH; ++u) {
        const int k = k0 + u;
        if (k < ncols && sk[k] != k) buf[u] = base[(int64_t)sk[k] * nvec + i];
      }
#pragma unroll
      for (int u = 0; u < CH; ++u) {
        const int k = k0 + u;
        if (k < ncols && sk[k] != k) base[(int64_t)k * nvec + i] = buf[u];
      }
    }
  }
}
template <typename T>
void compact_cols(View<T> v, int64_t len, const int* src, int src_stride, int ncols, const Launch& L) {
  if (L.nact <= 0 || ncols <= 0) return;
  const int64_t nvec = 2 * len * (int64_t)sizeof(T) / 16;
  int64_t nb = (nvec + 255) / 256;
  if (nb > 2048) nb = 2048;
  k_compact_cols<T><<<dim3((unsigned)nb, (unsigned)L.nact), 256, 0, L.st>>>(v, len, src, src_stride, ncols, L.slots);
}
template void compact_cols<float>(View<float>, int64_t, const int*, int, int, const Launch&);
template void compact_cols<double>(View<double>, int64_t, const int*, int, int, const Launch&);

}  // namespace bl

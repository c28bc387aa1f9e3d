// Device helpers shared by the stencil kernels: complex arithmetic, Bloch-extended reads
// and writes ("extended" coordinates: a vector index outside [0,n) x [0,m) is read through
// the Bloch extension u(j1 + s1 n, j2 + s2 m) = alpha^s1 beta^s2 u(j1, j2)), slot/column
// addressing of batched launches and the cell curl.
#pragma once

#include "internal.h"

#include <type_traits>

// No contraction into FMAs in these helpers either: they are inlined into the per-level
// kernels and the fused coarse cycles alike, which must round identically.
#pragma clang fp contract(off)

namespace bl {

template <typename T>
struct Cx {
  T re, im;
};

template <typename T>
__device__ __forceinline__ Cx<T> operator+(Cx<T> a, Cx<T> b) { return {a.re + b.re, a.im + b.im}; }
template <typename T>
__device__ __forceinline__ Cx<T> operator-(Cx<T> a, Cx<T> b) { return {a.re - b.re, a.im - b.im}; }
template <typename T>
__device__ __forceinline__ Cx<T> operator*(T s, Cx<T> a) { return {s * a.re, s * a.im}; }
template <typename T>
__device__ __forceinline__ Cx<T> cmul(Cx<T> a, T br, T bi) {
  return {a.re * br - a.im * bi, a.re * bi + a.im * br};
}

// Phases in the kernel's arithmetic type.
template <typename T>
struct Ph {
  T ar, ai, br, bi;
};
template <typename T>
__host__ __device__ inline Ph<T> cast_phase(const Phase& p) {
  return {(T)p.ar, (T)p.ai, (T)p.br, (T)p.bi};
}

// Read component `off` (0 for x-edges / nodes, nm for y-edges) at extended (j1, j2),
// j1 in [-n, 2n), j2 in [-m, 2m).
template <typename TS, typename T>
__device__ __forceinline__ Cx<T> fetch(const TS* __restrict__ col, int64_t N, int n, int m,
                                       int64_t off, int j1, int j2, const Ph<T>& p) {
  int s1 = 0, s2 = 0;
  if (j1 < 0) { j1 += n; s1 = -1; } else if (j1 >= n) { j1 -= n; s1 = 1; }
  if (j2 < 0) { j2 += m; s2 = -1; } else if (j2 >= m) { j2 -= m; s2 = 1; }
  const int64_t i = off + (int64_t)j2 * n + j1;
  Cx<T> v = {(T)col[i], (T)col[N + i]};
  if (s1 > 0) v = cmul(v, p.ar, p.ai);
  else if (s1 < 0) v = cmul(v, p.ar, -p.ai);
  if (s2 > 0) v = cmul(v, p.br, p.bi);
  else if (s2 < 0) v = cmul(v, p.br, -p.bi);
  return v;
}

// Add delta (given in extended coordinates) to the stored value at extended (j1, j2),
// j1 in [-1, n), j2 in [-1, m): u_can = conj(phase) * u_ext.
template <typename TS, typename T>
__device__ __forceinline__ void add_ext(TS* __restrict__ col, int64_t N, int n, int m, int64_t off,
                                        int j1, int j2, Cx<T> d, const Ph<T>& p) {
  if (j1 < 0) { j1 += n; d = cmul(d, p.ar, p.ai); }
  if (j2 < 0) { j2 += m; d = cmul(d, p.br, p.bi); }
  const int64_t i = off + (int64_t)j2 * n + j1;
  col[i] = (TS)((T)col[i] + d.re);
  col[N + i] = (TS)((T)col[N + i] + d.im);
}

__device__ __forceinline__ int wrapi(int j, int n) { return j < 0 ? j + n : (j >= n ? j - n : j); }

// Slot and in-slot column of this block (grid.y = active slots * columns per slot).
struct SJ {
  int slot, j;
};
__device__ __forceinline__ SJ slot_col(const int* slots, int ncps) {
  const int si = (int)blockIdx.y / ncps;
  return {slots ? slots[si] : si, (int)blockIdx.y % ncps};
}
template <typename T>
__device__ __forceinline__ T* colp(View<T> v, SJ s, int64_t N) {
  return v.p + ((int64_t)s.slot * v.cps + v.off + s.j) * 2 * N;
}

// The neighbouring lane's value (lane ^ 1).
__device__ __forceinline__ float lane_xor1(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), 0xB1, 0xF, 0xF, false));
}
__device__ __forceinline__ double lane_xor1(double x) {
  const long long b = __builtin_bit_cast(long long, x);
  const int lo = __builtin_amdgcn_mov_dpp((int)(b & 0xffffffffLL), 0xB1, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), 0xB1, 0xF, 0xF, false);
  return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned int)lo);
}

// Explicit fused multiply-adds (contraction is otherwise off), so that every kernel sharing
// these bodies rounds the same way.
template <typename T>
__device__ __forceinline__ T fmat(T a, T b, T c);
template <>
__device__ __forceinline__ float fmat<float>(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
template <>
__device__ __forceinline__ double fmat<double>(double a, double b, double c) { return __builtin_fma(a, b, c); }

// Part of row i of x = Inv b for a Hermitian n x n Inv (row i read as the conjugate of column i, so
// that the lanes of a wave, one row each, read consecutive entries), for NC columns of b: terms l0 ..
// l1 - 1, in order, the loads of 16 in flight.  l0 and l1 are the same for the whole wave.  A row is
// summed in kDenseParts parts [n k / 8, n (k + 1) / 8), which dense_sum combines.
constexpr int kDenseParts = 8;
template <int U, int NC, typename T>
__device__ __forceinline__ void dense_terms(const T* __restrict__ inv, int n, const T* const (&b)[NC], int i, int l, int l1,
                                            Cx<T> (&s)[NC]) {
  struct alignas(2 * sizeof(T)) Pair {
    T r, i;
  };
  Pair a[U];
  T br[U], bi[U];
  auto load_b = [&](int c, int u) {
    const int k = l + u < l1 ? l + u : l1 - 1;
    br[u] = l + u < l1 ? b[c][k] : (T)0;
    bi[u] = l + u < l1 ? b[c][n + k] : (T)0;
  };
#pragma unroll
  for (int u = 0; u < U; ++u) {   // past the end: zeros times the last entry
    const int k = l + u < l1 ? l + u : l1 - 1;
    a[u] = reinterpret_cast<const Pair*>(inv + 2 * (int64_t)k * n)[i];
    if (NC == 1) load_b(0, u);
  }
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    if (NC > 1)
#pragma unroll
      for (int u = 0; u < U; ++u) load_b(c, u);
#pragma unroll
    for (int u = 0; u < U; ++u) {   // s += conj(a) b
      s[c].re = fmat<T>(a[u].i, bi[u], fmat<T>(a[u].r, br[u], s[c].re));
      s[c].im = fmat<T>(-a[u].i, br[u], fmat<T>(a[u].r, bi[u], s[c].im));
    }
  }
}
template <int NC, typename T>
__device__ __forceinline__ void dense_part(const T* __restrict__ inv, int n, const T* const (&b)[NC], int i, int l0, int l1,
                                           Cx<T> (&s)[NC]) {
#pragma unroll
  for (int c = 0; c < NC; ++c) s[c] = Cx<T>{0, 0};
  int l = l0;
#pragma unroll 1
  for (; l + 16 <= l1; l += 16) dense_terms<16, NC>(inv, n, b, i, l, l + 16, s);
#pragma unroll 1
  for (; l < l1; l += 8) dense_terms<8, NC>(inv, n, b, i, l, l1, s);
}
// part(k): part k's value of a row
template <typename F>
__device__ __forceinline__ auto dense_sum(const F& part) {
  return ((part(0) + part(1)) + (part(2) + part(3))) + ((part(4) + part(5)) + (part(6) + part(7)));
}

// Whether the coarsest solves sum their rows in parts.  FP32 nodal cycles do not: the projection puts
// their results into FP64 vectors, which another order of the terms would move by FP32 roundings (the
// edge cycles only precondition).  Their matrices are the smallest ones.
template <typename T>
constexpr bool dense_in_parts(bool edge) { return edge || sizeof(T) == 8; }

// Row i of the same product, the terms one after the other.  One row a lane; l and n are the same for the
// whole wave, so that b's entries are scalar loads or LDS broadcasts.  Bound by load latency: eight terms
// are loaded while the eight before them are added (more make the code longer than its loads are slow).
// 900 nodes, 24 columns: 50 us, against 56 with eight loads at a time and 121 with two lanes per row,
// whose b entries then are vector loads; the fused cycle from 62 x 62 nodes 139 us, against 165 and 285.
template <typename T>
struct DenseTerms {
  static constexpr int U = 8;
  struct alignas(2 * sizeof(T)) Pair {
    T r, i;
  } a[U];
  T br[U], bi[U];
  template <bool TAIL>
  __device__ __forceinline__ void load(const T* __restrict__ inv, int n, const T* b, int i, int l) {
#pragma unroll
    for (int u = 0; u < U; ++u) {   // past the end: the last entry, to be added times zero
      const int k = !TAIL || l + u < n ? l + u : n - 1;
      a[u] = reinterpret_cast<const Pair*>(inv + 2 * (int64_t)k * n)[i];
      br[u] = b[k];
      bi[u] = b[n + k];
    }
  }
  template <bool TAIL>
  __device__ __forceinline__ void add(int n, int l, Cx<T>& s) const {
#pragma unroll
    for (int u = 0; u < U; ++u) {   // conj(a) b: ar br + ai bi, ar bi - ai br
      const bool in = !TAIL || l + u < n;
      const T r = in ? br[u] : (T)0, q = in ? bi[u] : (T)0;
      s.re = s.re + (a[u].r * r + a[u].i * q);
      s.im = s.im + (a[u].r * q + -a[u].i * r);
    }
  }
};
template <typename T>
__device__ __forceinline__ Cx<T> dense_row(const T* __restrict__ inv, int n, const T* b, int i) {
  constexpr int U = DenseTerms<T>::U;
  Cx<T> s = {0, 0};
  DenseTerms<T> x, y;
  int l = 0;
  if (n >= 3 * U) {
    x.template load<false>(inv, n, b, i, 0);
#pragma unroll 1
    for (; l + 3 * U <= n; l += 2 * U) {
      y.template load<false>(inv, n, b, i, l + U);
      x.template add<false>(n, l, s);
      x.template load<false>(inv, n, b, i, l + 2 * U);
      y.template add<false>(n, l + U, s);
    }
  } else {
    x.template load<true>(inv, n, b, i, 0);
  }
  // the last one to three groups (x holds the first)
  const bool more = l + U < n;
  if (more) y.template load<true>(inv, n, b, i, l + U);
  x.template add<true>(n, l, s);
  if (more) {
    x.template load<true>(inv, n, b, i, l + 2 * U);
    y.template add<true>(n, l + U, s);
    x.template add<true>(n, l + 2 * U, s);
  }
  return s;
}

// Plane wave w_j = exp(i t1 j1) exp(i t2 j2) of a slot from its factor tables.
__device__ __forceinline__ Cx<double> pw_value(const PWDefl& d, int slot, int n, int j1, int j2) {
  const double* t = d.tab + (int64_t)slot * d.tabstride;
  const double ar = t[2 * j1], ai = t[2 * j1 + 1];
  const double br = t[2 * (n + j2)], bi = t[2 * (n + j2) + 1];
  return {ar * br - ai * bi, ar * bi + ai * br};
}

// Sum of (a, b) over the workgroup (waves of 64, at most 1024 threads) in a fixed order;
// thread 0 stores it at out[0..1].
__device__ __forceinline__ void block_sum2(double a, double b, double* out) {
  __shared__ double sh[2][16];
  for (int o = 32; o > 0; o >>= 1) {
    a += __shfl_down(a, o, 64);
    b += __shfl_down(b, o, 64);
  }
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  if (lane == 0) { sh[0][wv] = a; sh[1][wv] = b; }
  __syncthreads();
  if (threadIdx.x == 0) {
    double ta = 0, tb = 0;
    for (int w = 0; w < (int)((blockDim.x + 63) >> 6); ++w) { ta += sh[0][w]; tb += sh[1][w]; }
    out[0] = ta;
    out[1] = tb;
  }
}

// (i mod n, i / n) in 32-bit unsigned arithmetic, for 0 <= i < 2^32 (node and edge indices of
// a level fit); a 64-bit division costs several times as many instructions
__device__ __forceinline__ void split_index(int64_t i, int n, int& j1, int& j2) {
  const unsigned u = (unsigned)i, q = u / (unsigned)n;
  j2 = (int)q;
  j1 = (int)(u - q * (unsigned)n);
}

// Block order that gives each of the 8 XCDs (which receive the blocks round-robin) one
// contiguous range of logical blocks, so that the rows shared by neighbouring blocks stay in
// one L2.  A bijection of [0, nb).
__device__ __forceinline__ int xcd_block(int b, int nb) {
  const int x = b & 7, i = b >> 3, q = nb >> 3, r = nb & 7;
  return x * q + (x < r ? x : r) + i;
}

// The value `off` bytes past a base that is uniform in the wave: the base stays in scalar registers and
// the lane's part of the address is 32 bits, which a plane of any grid accepted (kMaxCells) stays below.
template <typename T>
__device__ __forceinline__ T& at32(T* base, unsigned off) {
  using C = typename std::conditional<std::is_const<T>::value, const char, char>::type;
  return *reinterpret_cast<T*>(reinterpret_cast<C*>(base) + off);
}

template <typename T>
__device__ __forceinline__ T kap(const double* k64, const float* k32, int64_t i);
template <>
__device__ __forceinline__ double kap<double>(const double* k64, const float*, int64_t i) { return k64[i]; }
template <>
__device__ __forceinline__ float kap<float>(const double*, const float* k32, int64_t i) { return k32[i]; }

// Cell curl (circulation) of cell (c1, c2), extended c in [-1, n).
template <typename TS, typename T>
__device__ __forceinline__ Cx<T> cell_curl(const TS* col, int64_t N, int n, int m, int64_t nm,
                                           int c1, int c2, const Ph<T>& p) {
  return fetch<TS, T>(col, N, n, m, 0, c1, c2 + 1, p) - fetch<TS, T>(col, N, n, m, 0, c1, c2, p) +
         fetch<TS, T>(col, N, n, m, nm, c1, c2, p) - fetch<TS, T>(col, N, n, m, nm, c1 + 1, c2, p);
}

}  // namespace bl

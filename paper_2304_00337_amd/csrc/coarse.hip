// Fused coarse levels of the V-cycles (Section 5) for gfx950.  Below a size where the
// per-level launches are latency-bound (a few microseconds of dispatch for a few thousand
// unknowns), the rest of a V-cycle — smoothing, residual, restriction, the dense coarsest
// solve, prolongation and post-smoothing on every remaining level — runs in one workgroup
// per column, with all levels' vectors in LDS and a barrier between dependent passes.  The
// per-point bodies are those of the per-level kernels (stencil_ops.h) and the coarsest solve
// is dense_apply's (dense_part, dense_row), so a fused cycle reproduces the per-level one bit for bit.
//
// What bounds it: a chain of some 40 short dependent passes, one workgroup per column, so the
// latency of a pass is what counts.  Therefore
//  * a thread owns a coarse node of a level, that is the 2 x 2 fine nodes around it, in every pass:
//    the rows and columns that its passes read (wrapped at the period) are worked out once per
//    level, and its patches' coefficients are loaded once per level, ahead of their use, and kept
//    for the sweeps and the residual;
//  * a pass loads its neighbourhood first and then applies the Bloch phases of a crossing, in one
//    branch per direction that only the threads at the period's edge take;
//  * where the threads suffice, two neighbouring lanes share a coarse node, one for the real and one
//    for the imaginary parts (the stencils are real; only the phases mix them): twice the waves and
//    half the instructions of each;
//  * values are interleaved complex and the even and the odd columns of a row stand apart, so that
//    the lanes of a colour read consecutive words;
//  * in the dense solve a lane takes a row and a wave an eighth of its terms, 16 loads in flight
//    (FP32 nodal cycles: see dense_in_parts).
// From a 32 x 32 level down (FP64): 28 us for edges and 15 us for nodes, against 76 and 41 us
// with every read wrapped and phased by itself, coefficients loaded per pass and one thread per row of
// the dense solve.
// (Not all fits the registers: of the FP64 kernels, nodes with one lane per coarse node spill 17 of them,
// edges with two lanes one.)
// A nodal solve of several cycles whose finest level is fused runs them all here, residuals and sums
// included: two cycles of a 32 x 32 grid take 28 us instead of two launches of 15 with a residual (9) and
// a sum (5) between.
#include "stencil_ops.h"

#include <cstdlib>

#pragma clang fp contract(off)

namespace bl {

namespace {

// Largest workgroups: the registers that the coefficients take (edges) or the dense solve's loads
// (FP64) allow no more waves; the LDS that a cycle takes (at least 112 bytes per node of its first
// level for FP64 edges, 56 for FP32 edges and FP64 nodes, of 160 KB) keeps the coarse nodes below these.
template <typename T, int LP>
constexpr int edge_threads() { return sizeof(T) == 8 || LP == 2 ? 512 : 768; }
template <typename T, int LP>
constexpr int nodal_threads() { return sizeof(T) == 4 ? 1024 : LP == 2 ? 512 : 768; }

template <typename T>
__device__ __forceinline__ const T* pickp(const double* a, const float* b);
template <>
__device__ __forceinline__ const double* pickp<double>(const double* a, const float*) { return a; }
template <>
__device__ __forceinline__ const float* pickp<float>(const double*, const float* b) { return b; }

// A vector of a level in LDS: per component (two for edges, one for nodes) a plane of n x m complex
// values; a row holds its even columns first, then the odd ones.  With LP = 2 lanes per coarse node
// each lane handles its part (0: real, 1: imaginary), passed around in the .re of a value.
template <typename T, int LP>
struct Plane {
  T* q;
  int H, W, plane, part;
  __device__ __forceinline__ Plane(T* base, const Geo& g)
      : q(base), H((g.n + 1) >> 1), W(2 * H), plane(W * g.m), part(LP == 2 ? (int)threadIdx.x & 1 : 0) {}
  __device__ __forceinline__ int index(int j1, int j2) const { return j2 * W + (j1 & 1) * H + (j1 >> 1); }
  __device__ __forceinline__ Cx<T> load(int c, int i) const {
    const T* v = q + 2 * (c * plane + i);
    if (LP == 2) return {v[part], 0};
    return {v[0], v[1]};
  }
  __device__ __forceinline__ void store(int c, int i, Cx<T> v) const {
    T* d = q + 2 * (c * plane + i);
    if (LP == 2) {
      d[part] = v.re;
    } else {
      d[0] = v.re;
      d[1] = v.im;
    }
  }
};
// Values of a column in memory: N real, then N imaginary parts.
template <typename T, int LP>
__device__ __forceinline__ Cx<T> planar(const T* c, int64_t N, int i) {
  if (LP == 2) return {c[(threadIdx.x & 1) * N + i], 0};
  return {c[i], c[N + i]};
}
template <typename T, int LP>
__device__ __forceinline__ void set_planar(T* c, int64_t N, int i, Cx<T> v) {
  if (LP == 2) {
    c[(threadIdx.x & 1) * N + i] = v.re;
  } else {
    c[i] = v.re;
    c[N + i] = v.im;
  }
}
// v times the phase ar + i ai (both lanes of a pair are here together)
template <typename T, int LP>
__device__ __forceinline__ Cx<T> rotate(Cx<T> v, T ar, T ai) {
  if (LP == 1) return cmul(v, ar, ai);
  const T other = lane_xor1(v.re), own = v.re * ar, mix = other * ai;
  return {(threadIdx.x & 1) ? mix + own : own - mix, 0};
}

// A thread's coarse node (a, b) of a level (on = false beyond the last): LDS rows and columns
// 2 b - 1 .. 2 b + 2 and 2 a - 1 .. 2 a + 2 of a fine plane, wrapped at the period, and whether the
// first and last of them are across it.
struct Site {
  int a, b, n, row[4], col[4];
  bool on, xl, xh, yl, yh;
  template <int LP>
  __device__ __forceinline__ void place(const Geo& g) {
    const int nh = g.n >> 1, mh = g.m >> 1, t = (int)threadIdx.x / LP;
    on = t < nh * mh;
    split_index(on ? t : 0, nh, a, b);
    n = g.n;
    xl = a == 0;
    xh = a == nh - 1;
    yl = b == 0;
    yh = b == mh - 1;
    col[0] = nh + (xl ? nh - 1 : a - 1);
    col[1] = a;
    col[2] = nh + a;
    col[3] = xh ? 0 : a + 1;
    row[0] = (yl ? g.m - 1 : 2 * b - 1) * n;
    row[1] = 2 * b * n;
    row[2] = row[1] + n;
    row[3] = yh ? 0 : row[2] + n;
  }
  // the fine node of colour c in a planar column
  __device__ __forceinline__ int node(int c) const { return (2 * b + (c >> 1)) * n + 2 * a + (c & 1); }
  // Runs f(integral_constant<int, c>) for the four colours c in order, or in reverse.  The rows are
  // made opaque before each, so that the compiler does not keep all colours' addresses in registers.
  template <bool REV = false, typename F>
  __device__ __forceinline__ void each_colour(const F& f) {
    auto one = [&](auto c) {
      asm volatile("" : "+v"(row[0]), "+v"(row[1]), "+v"(row[2]), "+v"(row[3]));
      f(c);
    };
    one(std::integral_constant<int, REV ? 3 : 0>{});
    one(std::integral_constant<int, REV ? 2 : 1>{});
    one(std::integral_constant<int, REV ? 1 : 2>{});
    one(std::integral_constant<int, REV ? 0 : 3>{});
  }
};

// The values around the fine node of colour C of a site, in Bloch-extended coordinates (as fetch():
// the x phase first), for the shared point bodies.  What a body does not read is not loaded.
template <typename T, int LP, int C, int COMPS>
struct Near {
  static constexpr int PX = C & 1, PY = C >> 1;
  const Plane<T, LP>& X;
  const Site& s;
  Cx<T> v[COMPS][3][3], raw[2];   // raw: the stored x-edge (-1, 0) and y-edge (0, -1)
  __device__ __forceinline__ int at(int d1, int d2) const { return s.row[PY + d2 + 1] + s.col[PX + d1 + 1]; }
  __device__ __forceinline__ Near(const Plane<T, LP>& x, const Site& site) : X(x), s(site) {
#pragma unroll
    for (int c = 0; c < COMPS; ++c)
#pragma unroll
      for (int d2 = -1; d2 <= 1; ++d2)
#pragma unroll
        for (int d1 = -1; d1 <= 1; ++d1) v[c][d2 + 1][d1 + 1] = X.load(c, at(d1, d2));
    raw[0] = v[0][1][0];
    raw[1] = v[COMPS - 1][0][1];
  }
  // the phases of the values across the period in x, in y (callers branch on the site's flags)
  __device__ __forceinline__ void cross_x(const Ph<T>& p) {
#pragma unroll
    for (int c = 0; c < COMPS; ++c)
#pragma unroll
      for (int d = 0; d < 3; ++d)
        v[c][d][PX ? 2 : 0] = rotate<T, LP>(v[c][d][PX ? 2 : 0], p.ar, PX ? p.ai : -p.ai);
  }
  __device__ __forceinline__ void cross_y(const Ph<T>& p) {
#pragma unroll
    for (int c = 0; c < COMPS; ++c)
#pragma unroll
      for (int d = 0; d < 3; ++d)
        v[c][PY ? 2 : 0][d] = rotate<T, LP>(v[c][PY ? 2 : 0][d], p.br, PY ? p.bi : -p.bi);
  }
  __device__ __forceinline__ bool at_x() const { return PX ? s.xh : s.xl; }
  __device__ __forceinline__ bool at_y() const { return PY ? s.yh : s.yl; }
  __device__ __forceinline__ Near& cross(const Ph<T>& p) {
    if (at_x()) cross_x(p);
    if (at_y()) cross_y(p);
    return *this;
  }
};
template <typename T, int LP, int C>
struct EdgesNear : Near<T, LP, C, 2> {
  using N = Near<T, LP, C, 2>;
  const Ph<T>& p;
  __device__ __forceinline__ EdgesNear(const Plane<T, LP>& x, const Site& site, const Ph<T>& ph) : N(x, site), p(ph) {}
  __device__ __forceinline__ Cx<T> get(int c, int d1, int d2) const { return N::v[c][d2 + 1][d1 + 1]; }
  // as add_ext(): a value written one period back is stored times alpha (beta)
  __device__ __forceinline__ void add(int c, int d1, int d2, Cx<T> u) const {
    if (d1 < 0 && N::PX == 0 && N::s.xl) u = rotate<T, LP>(u, p.ar, p.ai);
    if (d2 < 0 && N::PY == 0 && N::s.yl) u = rotate<T, LP>(u, p.br, p.bi);
    const Cx<T> old = c == 0 && d1 < 0 ? N::raw[0] : c == 1 && d2 < 0 ? N::raw[1] : get(c, d1, d2);
    N::X.store(c, N::at(d1, d2), old + u);
  }
};
template <typename T, int LP, int C>
struct NodesNear : Near<T, LP, C, 1> {
  using N = Near<T, LP, C, 1>;
  __device__ __forceinline__ NodesNear(const Plane<T, LP>& x, const Site& site, const Ph<T>& p) : N(x, site) { N::cross(p); }
  __device__ __forceinline__ Cx<T> get(int d1, int d2) const { return N::v[0][d2 + 1][d1 + 1]; }
};

// The coefficients of a thread's four patches: kappa of the 3 x 3 cells around its fine nodes, and
// the patch inverses (colour c: node (2 a + (c & 1), 2 b + (c >> 1))).
template <typename T>
struct PatchCoef {
  T k[3][3], w[4][kPatchW];
};
template <typename T>
__device__ __forceinline__ void load_coef(const CoarseLevel& lv, int slot, const Site& s, PatchCoef<T>& K) {
  struct alignas(2 * sizeof(T)) Pair {
    T x, y;
  };
  static_assert(kPatchW % 2 == 0, "pairs of entries");
  const int n = lv.g.n, m = lv.g.m, a = s.a, b = s.b;
  const Pair* si = reinterpret_cast<const Pair*>(pickp<T>(lv.si64, lv.si32) + kPatchW * (int64_t)slot * lv.g.nm);
#pragma unroll
  for (int c = 0; c < 4; ++c)
#pragma unroll
    for (int u = 0; u < kPatchW / 2; ++u) {
      const Pair v = si[kPatchW / 2 * s.node(c) + u];
      K.w[c][2 * u] = v.x;
      K.w[c][2 * u + 1] = v.y;
    }
  const double* k64 = lv.k64 + (int64_t)slot * lv.g.nm;
  const float* k32 = lv.k32 + (int64_t)slot * lv.g.nm;
  const int x[3] = {a > 0 ? 2 * a - 1 : n - 1, 2 * a, 2 * a + 1}, y[3] = {b > 0 ? 2 * b - 1 : m - 1, 2 * b, 2 * b + 1};
#pragma unroll
  for (int v = 0; v < 3; ++v)
#pragma unroll
    for (int u = 0; u < 3; ++u) K.k[v][u] = kap<T>(k64, k32, y[v] * n + x[u]);
}

template <typename T, int LP, bool BWD>
__device__ __forceinline__ void edge_sweep(const Plane<T, LP>& X, const Plane<T, LP>& B, const CoarseLevel& lv,
                                           const PatchCoef<T>& K, Site& site, const Ph<T>& p, T mu) {
  const T s = (T)lv.g.s, mmx = mu * (T)lv.g.mx, mmy = mu * (T)lv.g.my;
  site.each_colour<BWD>([&](auto colour) {
    constexpr int c = decltype(colour)::value, px = c & 1, py = c >> 1;
    if (site.on) {
      EdgesNear<T, LP, c> x(X, site, p), b(B, site, p);
      if (x.at_x()) {
        x.cross_x(p);
        if (!px) b.cross_x(p);
      }
      if (x.at_y()) {
        x.cross_y(p);
        if (!py) b.cross_y(p);
      }
      patch_update<T>(x, b, K.k[py + 1][px + 1], K.k[py + 1][px], K.k[py][px], K.k[py][px + 1], K.w[c], s, mmx, mmy);
    }
    __syncthreads();
  });
}

// The coarsest solve, x = Inv b, over the whole workgroup: a wave sums a part of 64 rows at a time
// into `part` (room for `groups` groups of 64 rows), then a thread combines and stores a row.
template <typename T, typename Store>
__device__ __forceinline__ void dense_solve(const T* inv, int n, const T* b, T* part, int groups, const Store& store) {
  const int lane = (int)threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int waves = (int)blockDim.x >> 6, all = (n + 63) >> 6;
#pragma unroll 1
  for (int g0 = 0; g0 < all; g0 += groups) {
    const int ng = groups < all - g0 ? groups : all - g0;
#pragma unroll 1
    for (int t = wave; t < ng * kDenseParts; t += waves) {
      const int k = t % kDenseParts, r = t / kDenseParts * 64 + lane, i = g0 * 64 + r;
      if (i < n) {
        const T* const bc[1] = {b};
        Cx<T> v[1];
        dense_part<1>(inv, n, bc, i, n * k / kDenseParts, n * (k + 1) / kDenseParts, v);
        part[(2 * k) * (ng * 64) + r] = v[0].re;
        part[(2 * k + 1) * (ng * 64) + r] = v[0].im;
      }
    }
    __syncthreads();
    for (int r = (int)threadIdx.x; r < ng * 64 && g0 * 64 + r < n; r += (int)blockDim.x)
      store(g0 * 64 + r, Cx<T>{dense_sum([&](int k) { return part[2 * k * (ng * 64) + r]; }),
                               dense_sum([&](int k) { return part[(2 * k + 1) * (ng * 64) + r]; })});
    __syncthreads();
  }
}

template <typename T, int LP>
__global__ __launch_bounds__((edge_threads<T, LP>())) void k_edge_vcycle_fused(
    View<const T> bv, View<T> xv, CoarseCycle C, const Phase* __restrict__ phs, const double* __restrict__ mus,
    const int* __restrict__ slots, int ncps) {
  using P1 = Plane<T, 1>;
  using PL = Plane<T, LP>;
  extern __shared__ unsigned char lds_raw[];
  const int zi = (int)blockIdx.x / ncps;
  const int slot = slots ? slots[zi] : zi;
  const SJ sj{slot, (int)blockIdx.x % ncps};
  T* const base = reinterpret_cast<T*>(lds_raw);
  const int tid = threadIdx.x, nt = blockDim.x;
  const int last = C.nlev - 1;
  const T* const inv = static_cast<const T*>(C.inv) + (int64_t)slot * C.nc * C.nc * 2;
  Site site;
  PatchCoef<T> K;
  site.place<LP>(C.L[0].g);
  {
    const Geo& g = C.L[0].g;
    const T* bg = colp(bv, sj, g.ne);
    const PL B(base + C.bo[0], g);
    Cx<T> bx[4], by[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      bx[c] = planar<T, LP>(bg, g.ne, site.node(c));
      by[c] = planar<T, LP>(bg + g.nm, g.ne, site.node(c));
    }
    load_coef<T>(C.L[0], slot, site, K);
    for (int l = 0; l < last; ++l) {
      T* x = base + C.xo[l];
      const int len = 4 * (int)C.L[l].g.nm;
      for (int i = tid; i < len; i += nt) x[i] = (T)0;
    }
    if (site.on)
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        B.store(0, site.row[(c >> 1) + 1] + site.col[(c & 1) + 1], bx[c]);
        B.store(1, site.row[(c >> 1) + 1] + site.col[(c & 1) + 1], by[c]);
      }
  }
  const Ph<T> p = cast_phase<T>(phs[slot]);
  const T mu = (T)mus[slot];
  __syncthreads();
#pragma unroll 1
  for (int l = 0; l < last; ++l) {
    const Geo& g = C.L[l].g;
    const Geo& gc = C.L[l + 1].g;
    const PL X(base + C.xo[l], g), B(base + C.bo[l], g), R(base + C.ro, g);
#pragma unroll 1
    for (int it = 0; it < C.nu_pre; ++it) edge_sweep<T, LP, false>(X, B, C.L[l], K, site, p, mu);
    const T s = (T)g.s, mx = (T)g.mx, my = (T)g.my;
    if (site.on)
      site.each_colour([&](auto colour) {
        constexpr int c = decltype(colour)::value, px = c & 1, py = c >> 1;
        EdgesNear<T, LP, c> x(X, site, p);
        x.cross(p);
        const int i = x.at(0, 0);
        Cx<T> Au, Mu;
        edge_AM_acc<T>(x, 0, K.k[py][px + 1], K.k[py + 1][px + 1], s, mx, Au, Mu);
        R.store(0, i, B.load(0, i) - (Au + (mu * Mu)));
        edge_AM_acc<T>(x, 1, K.k[py + 1][px + 1], K.k[py + 1][px], s, my, Au, Mu);
        R.store(1, i, B.load(1, i) - (Au + (mu * Mu)));
      });
    // the next level's coefficients are on their way while this one is restricted
    const Site fine = site;
    if (l + 1 < last) {
      site.place<LP>(gc);
      load_coef<T>(C.L[l + 1], slot, site, K);
    }
    __syncthreads();
    if (fine.on) {
      EdgesNear<T, LP, 0> r(R, fine, p);
      r.cross(p);
      const Cx<T> vx = edge_restrict_acc<T>(r, 0), vy = edge_restrict_acc<T>(r, 1);
      T* bc = base + C.bo[l + 1];
      const PL Bc(bc, gc);
      if (l + 1 < last) {
        Bc.store(0, Bc.index(fine.a, fine.b), vx);
        Bc.store(1, Bc.index(fine.a, fine.b), vy);
      } else {
        set_planar<T, LP>(bc, gc.ne, fine.b * gc.n + fine.a, vx);
        set_planar<T, LP>(bc + gc.nm, gc.ne, fine.b * gc.n + fine.a, vy);
      }
    }
    __syncthreads();
  }
  {
    const Geo& g = C.L[last].g;
    const P1 X(base + C.xo[last], g);
    const int nm = (int)g.nm;
    dense_solve<T>(inv, (int)C.nc, base + C.bo[last],
                   base + C.ro, C.groups, [&](int i, Cx<T> v) {
                     const int c = i >= nm ? 1 : 0;
                     int j1, j2;
                     split_index(i - c * nm, g.n, j1, j2);
                     X.store(c, X.index(j1, j2), v);
                   });
  }
#pragma unroll 1
  for (int l = last - 1; l >= 0; --l) {
    const Geo& g = C.L[l].g;
    const PL X(base + C.xo[l], g), B(base + C.bo[l], g), Xc(base + C.xo[l + 1], C.L[l + 1].g);
    if (l < last - 1) {
      site.place<LP>(g);
      load_coef<T>(C.L[l], slot, site, K);
    }
    if (site.on) {
      const int a = site.a, b = site.b, i = Xc.index(a, b);
      const Cx<T> x00 = Xc.load(0, i), y00 = Xc.load(1, i);
      Cx<T> x01 = Xc.load(0, Xc.index(a, site.yh ? 0 : b + 1)), y10 = Xc.load(1, Xc.index(site.xh ? 0 : a + 1, b));
      if (site.xh) y10 = rotate<T, LP>(y10, p.ar, p.ai);
      if (site.yh) x01 = rotate<T, LP>(x01, p.br, p.bi);
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int i = site.row[(c >> 1) + 1] + site.col[(c & 1) + 1];
        X.store(0, i, X.load(0, i) + edge_prolong_combine<T>(x00, x01, c >> 1));
        X.store(1, i, X.load(1, i) + edge_prolong_combine<T>(y00, y10, c & 1));
      }
    }
    __syncthreads();
#pragma unroll 1
    for (int it = 0; it < C.nu_post; ++it) edge_sweep<T, LP, true>(X, B, C.L[l], K, site, p, mu);
  }
  const Geo& g = C.L[0].g;
  T* xg = colp(xv, sj, g.ne);
  const PL X(base + C.xo[0], g);
  if (site.on)
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int i = site.row[(c >> 1) + 1] + site.col[(c & 1) + 1];
      set_planar<T, LP>(xg, g.ne, site.node(c), X.load(0, i));
      set_planar<T, LP>(xg + g.nm, g.ne, site.node(c), X.load(1, i));
    }
}

template <typename T, int LP, bool BWD>
__device__ __forceinline__ void nodal_sweep(const Plane<T, LP>& X, const Cx<T> (&rhs)[4], const NodalStencil& st,
                                            Site& site, const Ph<T>& p) {
  const T inv = (T)1 / (T)st.c0;
  site.each_colour<BWD>([&](auto colour) {
    constexpr int c = decltype(colour)::value;
    if (site.on) {
      const NodesNear<T, LP, c> x(X, site, p);
      const Cx<T> r = rhs[c] - nodal_stencil_at<T>(x, st), u = x.get(0, 0);
      X.store(0, x.at(0, 0), Cx<T>{u.re + inv * r.re, u.im + inv * r.im});
    }
    __syncthreads();
  });
}

template <typename T, int LP>
__global__ __launch_bounds__((nodal_threads<T, LP>())) void k_nodal_vcycle_fused(View<const T> bv, View<T> xv, CoarseCycle C,
                                                                                 const Phase* __restrict__ phs,
                                                                                 const int* __restrict__ slots, int ncps) {
  using P1 = Plane<T, 1>;
  using PL = Plane<T, LP>;
  extern __shared__ unsigned char lds_raw[];
  const int zi = (int)blockIdx.x / ncps;
  const int slot = slots ? slots[zi] : zi;
  const SJ sj{slot, (int)blockIdx.x % ncps};
  T* const base = reinterpret_cast<T*>(lds_raw);
  const int tid = threadIdx.x, nt = blockDim.x;
  const int last = C.nlev - 1;
  const T* const inv = static_cast<const T*>(C.inv) + (int64_t)slot * C.nc * C.nc * 2;
  Site site;
  // the right-hand side is read at the thread's own nodes only: plain planes, and registers
  Cx<T> rhs[4];
  auto load_rhs = [&](const T* src, const Geo& g) {
#pragma unroll
    for (int c = 0; c < 4; ++c) rhs[c] = planar<T, LP>(src, g.nm, site.node(c));
  };
  site.place<LP>(C.L[0].g);
  const T* bg = colp(bv, sj, C.L[0].g.nm);
  load_rhs(bg, C.L[0].g);
  const Ph<T> p = cast_phase<T>(phs[slot]);
  T* const xg = colp(xv, sj, C.L[0].g.nm);
  // one pass of this loop per cycle, the later ones on the residual of the sum so far (in xg)
#pragma unroll 1
  for (int cycle = 0;; ++cycle) {
    for (int l = 0; l < last; ++l) {
      T* x = base + C.xo[l];
      const int len = 2 * (int)C.L[l].g.nm;
      for (int i = tid; i < len; i += nt) x[i] = (T)0;
    }
    if (site.on)
#pragma unroll
      for (int c = 0; c < 4; ++c) set_planar<T, LP>(base + C.bo[0], C.L[0].g.nm, site.node(c), rhs[c]);
    __syncthreads();
#pragma unroll 1
    for (int l = 0; l < last; ++l) {
      const Geo& g = C.L[l].g;
      const Geo& gc = C.L[l + 1].g;
      const PL X(base + C.xo[l], g), R(base + C.ro, g);
      if (l > 0) {
        site.place<LP>(g);
        load_rhs(base + C.bo[l], g);
      }
#pragma unroll 1
      for (int it = 0; it < C.nu_pre; ++it) nodal_sweep<T, LP, false>(X, rhs, C.ns, site, p);
      if (site.on)
        site.each_colour([&](auto colour) {
          constexpr int c = decltype(colour)::value;
          const NodesNear<T, LP, c> x(X, site, p);
          R.store(0, x.at(0, 0), rhs[c] - nodal_stencil_at<T>(x, C.ns));
        });
      __syncthreads();
      if (site.on) {
        const Cx<T> v = nodal_restrict_acc<T>(NodesNear<T, LP, 0>(R, site, p));
        set_planar<T, LP>(base + C.bo[l + 1], gc.nm, site.b * gc.n + site.a, v);
      }
      __syncthreads();
    }
    {
      const Geo& g = C.L[last].g;
      const int nc = (int)C.nc;
      int j1, j2;
      if constexpr (dense_in_parts<T>(false)) {
        const P1 X(base + C.xo[last], g);
        dense_solve<T>(inv, nc, base + C.bo[last], base + C.ro, C.groups, [&](int i, Cx<T> v) {
          split_index(i, g.n, j1, j2);
          X.store(0, X.index(j1, j2), v);
        });
      } else {
        const P1 X(base + C.xo[last], g);
#pragma unroll 1
        for (int i = tid; i < nc; i += nt) {
          const Cx<T> v = dense_row<T>(inv, nc, base + C.bo[last], i);
          split_index(i, g.n, j1, j2);
          X.store(0, X.index(j1, j2), v);
        }
        __syncthreads();
      }
    }
#pragma unroll 1
    for (int l = last - 1; l >= 0; --l) {
      const Geo& g = C.L[l].g;
      const PL X(base + C.xo[l], g), Xc(base + C.xo[l + 1], C.L[l + 1].g);
      if (l < last - 1) {
        site.place<LP>(g);
        load_rhs(base + C.bo[l], g);
      }
      if (site.on) {
        const int a = site.a, b = site.b, a1 = site.xh ? 0 : a + 1, b1 = site.yh ? 0 : b + 1;
        const Cx<T> c00 = Xc.load(0, Xc.index(a, b));
        Cx<T> c10 = Xc.load(0, Xc.index(a1, b)), c01 = Xc.load(0, Xc.index(a, b1)), c11 = Xc.load(0, Xc.index(a1, b1));
        if (site.xh) {
          c10 = rotate<T, LP>(c10, p.ar, p.ai);
          c11 = rotate<T, LP>(c11, p.ar, p.ai);
        }
        if (site.yh) {
          c01 = rotate<T, LP>(c01, p.br, p.bi);
          c11 = rotate<T, LP>(c11, p.br, p.bi);
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const int i = site.row[(c >> 1) + 1] + site.col[(c & 1) + 1];
          X.store(0, i, X.load(0, i) + nodal_prolong_combine<T>(c00, c10, c01, c11, c & 1, c >> 1));
        }
      }
      __syncthreads();
#pragma unroll 1
      for (int it = 0; it < C.nu_post; ++it) nodal_sweep<T, LP, true>(X, rhs, C.ns, site, p);
    }
    const Geo& g = C.L[0].g;
    const PL X(base + C.xo[0], g);
    auto own = [&](int c) { return site.row[(c >> 1) + 1] + site.col[(c & 1) + 1]; };
    if (site.on)
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        Cx<T> v = X.load(0, own(c));
        if (cycle) {
          v = planar<T, LP>(xg, g.nm, site.node(c)) + v;
          X.store(0, own(c), v);
        }
        set_planar<T, LP>(xg, g.nm, site.node(c), v);
      }
    if (cycle + 1 == C.cycles) break;
    __syncthreads();
    load_rhs(bg, g);
    if (site.on)
      site.each_colour([&](auto colour) {
        constexpr int c = decltype(colour)::value;
        rhs[c] = rhs[c] - nodal_stencil_at<T>(NodesNear<T, LP, c>(X, site, p), C.ns);
      });
    __syncthreads();
  }
}

int g_lds_cap = -1;

int lds_cap() {
  if (g_lds_cap < 0) {
    int dev = 0, cap = 65536;
    (void)hipGetDevice(&dev);
    if (hipDeviceGetAttribute(&cap, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess) cap = 65536;
    const void* ks[] = {(const void*)k_edge_vcycle_fused<double, 1>,  (const void*)k_edge_vcycle_fused<double, 2>,
                        (const void*)k_edge_vcycle_fused<float, 1>,   (const void*)k_edge_vcycle_fused<float, 2>,
                        (const void*)k_nodal_vcycle_fused<double, 1>, (const void*)k_nodal_vcycle_fused<double, 2>,
                        (const void*)k_nodal_vcycle_fused<float, 1>,  (const void*)k_nodal_vcycle_fused<float, 2>};
    for (const void* k : ks)
      if (hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, cap) != hipSuccess) cap = 65536;
    g_lds_cap = cap;
  }
  return g_lds_cap;
}

// LDS offsets of a cycle's vectors (elements); returns their total.  The residual lives only
// between a level's smoothing and its restriction: one buffer, sized for the first level, which
// also holds the dense solve's parts (for as many groups of 64 rows at a time as fit, at least one).
int64_t fused_layout(CoarseCycle& C, bool edge) {
  const int64_t comps = edge ? 4 : 2;
  int64_t o = 0;
  for (int l = 0; l < C.nlev; ++l) {
    const Geo& g = C.L[l].g;
    C.xo[l] = (int)o;
    o += comps * (2 * ((g.n + 1) / 2)) * g.m;
    C.bo[l] = (int)o;
    o += comps * g.nm;
  }
  const int64_t parts = 64 * 2 * kDenseParts, r = comps * C.L[0].g.nm;
  C.ro = (int)o;
  C.groups = r >= parts ? (int)(r / parts) : 1;
  return o + (r >= parts ? r : parts);
}

}  // namespace

size_t fused_lds_bytes(const CoarseCycle& C, bool edge, size_t elem) {
  CoarseCycle c = C;
  return (size_t)fused_layout(c, edge) * elem;
}

size_t fused_lds_limit() { return (size_t)lds_cap(); }

namespace {
// lanes * (coarse nodes below the first fused level) threads, in whole waves, and at least 256 for
// the dense solve.
int fused_threads(const CoarseCycle& C, int lanes) {
  const int64_t t = lanes * (C.L[0].g.nm / 4);
  return t <= 256 ? 256 : (int)((t + 63) / 64 * 64);
}
}  // namespace

// Two lanes per coarse node where the workgroup has them (see the head of this file).
template <typename T>
void edge_vcycle_fused(View<const T> b, View<T> x, const CoarseCycle& cyc, const Phase* ph, const double* mu,
                       const Launch& L) {
  const int nb = L.nact * L.ncps;
  if (nb <= 0) return;
  CoarseCycle C = cyc;
  const size_t lds = (size_t)fused_layout(C, true) * sizeof(T);
  (void)lds_cap();
  if (fused_threads(C, 2) <= edge_threads<T, 2>())
    k_edge_vcycle_fused<T, 2><<<nb, fused_threads(C, 2), lds, L.st>>>(b, x, C, ph, mu, L.slots, L.ncps);
  else
    k_edge_vcycle_fused<T, 1><<<nb, fused_threads(C, 1), lds, L.st>>>(b, x, C, ph, mu, L.slots, L.ncps);
}
template <typename T>
void nodal_vcycle_fused(View<const T> b, View<T> x, const CoarseCycle& cyc, const Phase* ph, const Launch& L) {
  const int nb = L.nact * L.ncps;
  if (nb <= 0) return;
  CoarseCycle C = cyc;
  const size_t lds = (size_t)fused_layout(C, false) * sizeof(T);
  (void)lds_cap();
  if (fused_threads(C, 2) <= nodal_threads<T, 2>())
    k_nodal_vcycle_fused<T, 2><<<nb, fused_threads(C, 2), lds, L.st>>>(b, x, C, ph, L.slots, L.ncps);
  else
    k_nodal_vcycle_fused<T, 1><<<nb, fused_threads(C, 1), lds, L.st>>>(b, x, C, ph, L.slots, L.ncps);
}
template void edge_vcycle_fused<double>(View<const double>, View<double>, const CoarseCycle&, const Phase*, const double*, const Launch&);
template void edge_vcycle_fused<float>(View<const float>, View<float>, const CoarseCycle&, const Phase*, const double*, const Launch&);
template void nodal_vcycle_fused<double>(View<const double>, View<double>, const CoarseCycle&, const Phase*, const Launch&);
template void nodal_vcycle_fused<float>(View<const float>, View<float>, const CoarseCycle&, const Phase*, const Launch&);

}  // namespace bl

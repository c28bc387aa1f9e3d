// Tiled smoother sweeps (Section 5) for gfx950: one launch performs a whole sweep of the
// four-colour node-patch block Gauss-Seidel (edge smoother) or of the four-colour point
// Gauss-Seidel (nodal smoother) instead of one launch per colour.
//
// Each workgroup owns a TX x TY tile of nodes of one column and keeps in LDS the iterate on
// the tile plus a halo (kLo nodes below/left, kHi above/right).  The four colour passes run
// on the LDS copy, updating every patch whose stencil lies inside the box, halo included;
// values near the box edge go stale (their neighbours outside are not updated), but the
// staleness moves inwards by at most one node per pass on the low side and two on the high
// side, so after four passes the tile itself holds exactly what the per-colour launches
// produce.  The halo widths are the smallest for which this holds for both colour orders
// (checked by propagating the set of exact values through the passes).  Patches are
// computed by the same per-point code as the per-colour kernels, through accessors that
// read the LDS copy with the same Bloch-phase arithmetic, so the results agree bit for bit.
//
// LDS layout: the box is split by node parity into four sub-grids, so that the patches of
// one colour, which are two nodes apart, sit at consecutive addresses (no bank conflicts)
// and every neighbour of a patch is at a compile-time offset from it.  Only workgroups whose
// box crosses the periodic seam run the phase checks of the Bloch extension.
//
// The sweep reads the iterate from one buffer and writes it to another: a tile's halo is the
// neighbours' state before the sweep, which an in-place update could already have replaced.
//
// HBM traffic per sweep and column: the right-hand side once, the iterate once (not at all
// when the sweep starts from zero) and the iterate written once, against four reads of the
// iterate and two of the right-hand side for four colour launches.
#include "stencil_ops.h"

#pragma clang fp contract(off)

namespace bl {

namespace {

constexpr int kLo = 4;    // halo below / left of a tile, nodes (even: keeps colour parity)
constexpr int kHiE = 5;   // halo above / right, edge sweeps
constexpr int kHiN = 4;   // halo above / right, nodal sweeps

// MODE bits of a sweep with level transfers folded in: kRestrict (forward sweeps) also forms
// the residual of the result and restricts it to the coarse right-hand side; kProlong starts
// from xin + Pr xc; kBase writes base + result.  The residual at the fine nodes that the
// restriction reads (one node below/left of the tile to its last row/column) needs the swept
// iterate two nodes below/left and one node above/right of the tile: the halos grow to kLoR
// below (nodal and edge) and kHiER above (edge; the nodal forward sweep's kHiN suffices).
constexpr int kRestrict = 1, kProlong = 2, kBase = 4;
// kResid (nodal backward sweeps): the sweep also writes the residual b - P x of its result at
// the tile's nodes (as the residual kernel computes it), for which the iterate must be exact
// one node around the tile.
constexpr int kResid = 8;
// kZero (forward sweeps): the iterate is zero on entry and not read; nodal sweeps store a node in its own
// pass first and leave out the neighbours that no pass has reached, edge sweeps take the edges that no
// pass has written as zero.
constexpr int kZero = 16;
constexpr int kLoR = 6;
constexpr int kHiER = 6;

__device__ __forceinline__ int wrapm(int v, int n) {
  const int r = v % n;
  return r < 0 ? r + n : r;
}

template <typename T>
__device__ __forceinline__ const T* pick_si(const double* a, const float* b);
template <>
__device__ __forceinline__ const double* pick_si<double>(const double* a, const float*) { return a; }
template <>
__device__ __forceinline__ const float* pick_si<float>(const double*, const float* b) { return b; }

// Parity-split box: position (bx, by) of a BX x BY box is entry (by/2) HX + bx/2 of
// sub-grid (bx mod 2) + 2 (by mod 2).
template <int BX, int BY>
struct Split {
  static constexpr int HX = (BX + 1) / 2, HY = (BY + 1) / 2, SUB = HX * HY, N = 4 * SUB;
  __device__ static __forceinline__ int at(int bx, int by) {
    return ((bx & 1) + 2 * (by & 1)) * SUB + (by >> 1) * HX + (bx >> 1);
  }
};

// Which neighbours of a node lie across the periodic seam: for a node at canonical (p1, p2)
// the neighbour at offset d1 = -1 crosses when p1 = 0, d1 = +1 when p1 = n - 1 (y alike).
// Only the directions in which the box crosses the seam (CX, CY) are checked.
template <bool CX, bool CY>
struct Seam {
  bool lx, hx, ly, hy;
  __device__ __forceinline__ Seam(int p1, int p2, int n, int m)
      : lx(CX && p1 == 0), hx(CX && p1 == n - 1), ly(CY && p2 == 0), hy(CY && p2 == m - 1) {}
  __device__ __forceinline__ bool cross_x(int d1) const { return CX && ((d1 < 0 && lx) || (d1 > 0 && hx)); }
  __device__ __forceinline__ bool cross_y(int d2) const { return CY && ((d2 < 0 && ly) || (d2 > 0 && hy)); }
};

template <typename T>
__device__ __forceinline__ Cx<T> pick(bool c, Cx<T> a, Cx<T> b) {
  return {c ? a.re : b.re, c ? a.im : b.im};
}

// The value at offset (d1, d2) as fetch() returns it: times alpha (one period ahead) or
// conj(alpha) (one period back) across the x seam, then beta likewise across the y seam.
// The products are formed unconditionally and selected per lane, so that workgroups on the
// seam run the same instructions in every lane.
template <bool CX, bool CY, typename T>
__device__ __forceinline__ Cx<T> phased(Cx<T> v, int d1, int d2, const Seam<CX, CY>& sm, const Ph<T>& p) {
  if (CX && d1 != 0) v = pick(sm.cross_x(d1), cmul(v, p.ar, d1 > 0 ? p.ai : -p.ai), v);
  if (CY && d2 != 0) v = pick(sm.cross_y(d2), cmul(v, p.br, d2 > 0 ? p.bi : -p.bi), v);
  return v;
}

// Patches each colour pass has to update.  Walking the passes backwards from the region that
// must be exact after the sweep (the tile, or the residual window's inputs), a pass needs the
// patches of its colour that write into the region still required, and the values those
// patches read must then be exact before it; every other patch of the box only feeds values
// that never reach the tile.  The bounding rectangle of the needed patches (box positions,
// inclusive) is formed at compile time for every box shape and colour order.
struct PassRect {
  int x0, x1, y0, y1;
};
struct SweepRects {
  PassRect r[4];   // in sweep order
  bool ok;         // no needed patch lies on the box's outermost ring (the halo suffices)
};
constexpr int kMaxBox = 80;
constexpr SweepRects sweep_rects(bool edge, int BX, int BY, int LO, int TX, int TY, int EA, int EB, bool bwd) {
  // need[c][by][bx]: component c (x-edge / y-edge; nodal values use c = 0) must be exact
  bool need[2][kMaxBox][kMaxBox] = {};
  for (int y = LO - EA; y < LO + TY + EB; ++y)
    for (int x = LO - EA; x < LO + TX + EB; ++x) need[0][y][x] = need[1][y][x] = true;
  // an edge patch at P reads x-edges at P + XR and y-edges at P + YR (patch_update) and writes
  // the x-edges of P and P - (1, 0) and the y-edges of P and P - (0, 1); a nodal point reads
  // its 3 x 3 neighbourhood and writes P
  constexpr int XR[6][2] = {{0, 0}, {0, 1}, {0, -1}, {-1, 0}, {-1, 1}, {-1, -1}};
  constexpr int YR[6][2] = {{0, 0}, {1, 0}, {-1, 0}, {0, -1}, {1, -1}, {-1, -1}};
  SweepRects out{};
  out.ok = BX <= kMaxBox && BY <= kMaxBox;
  for (int k = 3; k >= 0; --k) {
    const int colour = bwd ? 3 - k : k;
    const int px = colour & 1, py = colour >> 1;
    PassRect r{kMaxBox, -1, kMaxBox, -1};
    bool hit[kMaxBox][kMaxBox] = {};
    for (int y = 0; y < BY; ++y)
      for (int x = 0; x < BX; ++x) {
        if ((x & 1) != px || (y & 1) != py) continue;
        hit[y][x] = edge ? (need[0][y][x] || (x > 0 && need[0][y][x - 1]) || need[1][y][x] ||
                            (y > 0 && need[1][y - 1][x]))
                         : need[0][y][x];
        if (!hit[y][x]) continue;
        if (x == 0 || y == 0 || x == BX - 1 || y == BY - 1) {   // not updatable: the halo is short
          out.ok = false;
          continue;
        }
        if (x < r.x0) r.x0 = x;
        if (x > r.x1) r.x1 = x;
        if (y < r.y0) r.y0 = y;
        if (y > r.y1) r.y1 = y;
      }
    // the needed patches' reads must be exact before the pass (the other patches of the
    // rectangle are updated too, but nothing needed reads what they write)
    for (int y = 1; y < BY - 1; ++y)
      for (int x = 1; x < BX - 1; ++x) {
        if (!hit[y][x]) continue;
        if (edge) {
          for (int q = 0; q < 6; ++q) {
            need[0][y + XR[q][1]][x + XR[q][0]] = true;
            need[1][y + YR[q][1]][x + YR[q][0]] = true;
          }
        } else {
          for (int dy = -1; dy <= 1; ++dy)
            for (int dx = -1; dx <= 1; ++dx) need[0][y + dy][x + dx] = true;
        }
      }
    out.r[k] = r;
  }
  return out;
}

// Column and tile of this workgroup: blockIdx.y = active slot x column, blockIdx.x = tile
// (XCD-major order when there are at least 8 tiles, so that neighbouring tiles share an L2).
struct TileRef {
  int slot, j, t0x, t0y;
};
__device__ __forceinline__ TileRef tile_ref(const int* slots, int ncps, int tiles_x, int TX, int TY) {
  const int si = (int)blockIdx.y / ncps;
  const int nb = (int)gridDim.x;
  const int t = nb >= 8 ? xcd_block((int)blockIdx.x, nb) : (int)blockIdx.x;
  return {slots ? slots[si] : si, (int)blockIdx.y % ncps, (t % tiles_x) * TX, (t / tiles_x) * TY};
}

struct EdgeArgs {
  const double* k64;
  const float* k32;
  const double* si64;
  const float* si32;
  double s, mx, my;
};

// ---- edge sweeps ----------------------------------------------------------------------------
// A thread owns one 2 x 2 block of the box's nodes (blocks of HX a row, so that block t is entry t of
// every parity sub-grid) in all passes: its addresses, its seam flags, kappa around it and in FP32 its
// right-hand side are worked out and loaded once, with the iterate; a sweep from zero neither reads nor
// stores zeros, and the residual that a restricting sweep forms takes over the iterate's planes, so
// that the box fits the static LDS in FP64 too.  Loads bound it, two workgroups of 512 threads to a
// compute unit (FP32: 92 to 121 registers) or one (FP64: 132 to 160) being few to hide them behind: in
// FP32, without its arithmetic the sweep takes as long, without the patch inverses a fifth less.  Sweeps
// without transfers are not the faster form everywhere: 512 x 512 FP32, 24 columns 154 us forward and
// backward, against 143 and 155 with the patches dealt out; 704 x 640, 48 columns 523 and 520 against
// 512 and 558.  1024 x 1024 FP32, 24 columns, the five
// sweep levels of a V-cycle: restricting 778 us, prolongating 949, against 970 and 1028 with the
// colours' patches dealt out anew in each pass; 256 x 256 FP64, three levels: 134 and 115 us against
// 182 and 224 with the residual and the transfers in launches of their own.
constexpr int kTile = 32, kThreads = 512;

// The values of a block's four nodes in a column, colour by colour: off is the byte offset of its
// first node in a plane, row that of a row; wide: two neighbouring values in one load.
template <typename T>
__device__ __forceinline__ void load_block(const T* c, int64_t N, unsigned off, unsigned row, bool wide, Cx<T> (&v)[4]) {
  struct alignas(2 * sizeof(T)) Pair {
    T a, b;
  };
  if (wide) {
#pragma unroll
    for (int y = 0; y < 2; ++y) {
      const Pair re = at32(reinterpret_cast<const Pair*>(c), off + y * row);
      const Pair im = at32(reinterpret_cast<const Pair*>(c + N), off + y * row);
      v[2 * y] = {re.a, im.a};
      v[2 * y + 1] = {re.b, im.b};
    }
  } else {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const unsigned o = off + (k >> 1) * row + (k & 1) * (unsigned)sizeof(T);
      v[k] = {at32(c, o), at32(c + N, o)};
    }
  }
}

// Runs f(integral_constant<int, 0 .. 3>).
template <typename F>
__device__ __forceinline__ void four(const F& f) {
  f(std::integral_constant<int, 0>{});
  f(std::integral_constant<int, 1>{});
  f(std::integral_constant<int, 2>{});
  f(std::integral_constant<int, 3>{});
}

// The edges around a node of block t in the iterate's planes (x-edge re, x-edge im, y-edge re, y-edge
// im).  In pass PASS of a forward sweep from zero (4: everything is stored) the edges that no earlier
// pass has written are zero: all of them in pass 0, x-edges of odd rows up to pass 2, y-edges of odd
// columns up to pass 1.
template <typename T, typename S, int PX, int PY, bool CX, bool CY, int PASS = 4>
struct BlockEdges {
  T* pl;   // at entry t
  Seam<CX, CY> sm;
  const Ph<T>& p;
  static constexpr bool unset(int c, int d1, int d2) {
    return c == 0 ? PASS == 0 || (PASS <= 2 && ((PY + d2) & 1)) : PASS == 0 || (PASS <= 1 && ((PX + d1) & 1));
  }
  __device__ __forceinline__ T* at(int c, int d1, int d2) const {
    const int sx = (PX + d1) & 1, sy = (PY + d2) & 1;
    return pl + c * 2 * S::N + (sx + 2 * sy) * S::SUB + ((PY + d2) >> 1) * S::HX + ((PX + d1) >> 1);
  }
  __device__ __forceinline__ Cx<T> get(int c, int d1, int d2) const {
    if (unset(c, d1, d2)) return {0, 0};
    const T* q = at(c, d1, d2);
    return phased<CX, CY, T>(Cx<T>{q[0], q[S::N]}, d1, d2, sm, p);
  }
  // as add_ext(): a value written one period back is stored times alpha (beta)
  __device__ __forceinline__ void add(int c, int d1, int d2, Cx<T> v) const {
    if (CX && d1 < 0) v = pick(sm.lx, cmul(v, p.ar, p.ai), v);
    if (CY && d2 < 0) v = pick(sm.ly, cmul(v, p.br, p.bi), v);
    T* q = at(c, d1, d2);
    q[0] = (unset(c, d1, d2) ? (T)0 : q[0]) + v.re;
    q[S::N] = (unset(c, d1, d2) ? (T)0 : q[S::N]) + v.im;
  }
};
// The right-hand side on a patch's edges: x (0, 0), x (-1, 0), y (0, 0), y (0, -1).
template <typename T>
struct PatchRhs {
  Cx<T> q[4];
  __device__ __forceinline__ Cx<T> get(int c, int d1, int d2) const { return q[2 * c + (d1 < 0 || d2 < 0 ? 1 : 0)]; }
};

template <typename T, bool BWD, int MODE>
struct EdgeShape {
  static constexpr bool RES = (MODE & kRestrict) != 0, PRO = (MODE & kProlong) != 0, ZERO = (MODE & kZero) != 0;
  static constexpr int TX = kTile, LO = RES ? kLoR : kLo, BX = TX + LO + (RES ? kHiER : kHiE);
  using S = Split<BX, BX>;
  static constexpr int EA = RES ? 2 : 0, EB = RES ? 1 : 0;   // exact margin the residual window needs
  static constexpr SweepRects R = sweep_rects(true, BX, BX, LO, TX, TX, EA, EB, BWD);
  static_assert(R.ok, "the halo does not cover the sweep's dependency cone");
  static_assert(S::SUB <= kThreads, "a block per thread");
};

template <typename T, bool BWD, int MODE, bool CX, bool CY>
__device__ __forceinline__ void edge_tile(T* pl, const T* xc, T* xo, const T* bc, const T* cc, T* bco, const EdgeArgs& e,
                                          int slot, int t0x, int t0y, int n, int m, int64_t N, int64_t nm, const Geo& gc,
                                          T mu, const Ph<T>& p, bool wide) {
  using H = EdgeShape<T, BWD, MODE>;
  using S = typename H::S;
  struct alignas(2 * sizeof(T)) Pair {
    T a, b;
  };
  // FP32 keeps the block's right-hand side and loads a pass's patch inverse one pass ahead (24 columns at
  // 1024 x 1024: 645 and 617 us, against 679 and 695 without); FP64 loads both in the pass.  There one
  // workgroup fits a compute unit either way (154 to 160 registers, 162 to 200 with the loads ahead)
  constexpr bool AHEAD = sizeof(T) == 4;
  constexpr int LO = H::LO, BX = H::BX, TX = H::TX;
  constexpr SweepRects R = H::R;
  const int tid = (int)threadIdx.x;
  const bool live = tid < S::SUB;
  const int t = live ? tid : 0, a = t % S::HX, b = t / S::HX;
  const int ox = t0x - LO, oy = t0y - LO;   // canonical node of box position 0 (unwrapped)
  // canonical first node of the block (n, m, ox and oy are even: a block never straddles the seam,
  // and where the box has an odd number of nodes its last block still lies in the grid)
  const int p1 = CX ? wrapm(ox + 2 * a, n) : ox + 2 * a, p2 = CY ? wrapm(oy + 2 * b, m) : oy + 2 * b;
  constexpr unsigned E = (unsigned)sizeof(T);
  const unsigned off = (unsigned)(p2 * n + p1) * E, row = (unsigned)n * E;
  // the column left of the block and the row below it, wrapped
  const unsigned left = CX && p1 == 0 ? off + row - E : off - E, low = CY && p2 == 0 ? (unsigned)((m - 1) * n + p1) * E : off - row;
  const unsigned corner = CX && p1 == 0 ? low + row - E : low - E;
  Cx<T> bx[4], by[4], bl[2], bd[2];   // right-hand side: the block's edges, x-edges left, y-edges below
  auto load_left = [&](int y) {
    const Cx<T> v{at32(bc, left + y * row), at32(bc + N, left + y * row)};
    return CX ? pick(p1 == 0, cmul(v, p.ar, -p.ai), v) : v;
  };
  auto load_low = [&](int x) {
    const Cx<T> v{at32(bc + nm, low + x * E), at32(bc + N + nm, low + x * E)};
    return CY ? pick(p2 == 0, cmul(v, p.br, -p.bi), v) : v;
  };
  auto load_own = [&](int comp, int c) {
    const T* q = comp ? bc + nm : bc;
    const unsigned o = off + (c >> 1) * row + (c & 1) * E;
    return Cx<T>{at32(q, o), at32(q + N, o)};
  };
  if constexpr (AHEAD) {
    load_block(bc, N, off, row, wide, bx);
    load_block(bc + nm, N, off, row, wide, by);
    for (int k = 0; k < 2; ++k) {
      bl[k] = load_left(k);
      bd[k] = load_low(k);
    }
  }
  // kappa of the 3 x 3 cells around the block, from the one below and left of it
  const T* kp = pick_si<T>(e.k64, e.k32);
  kp += (int64_t)slot * nm;
  const T kap9[3][3] = {{at32(kp, corner), at32(kp, low), at32(kp, low + E)},
                        {at32(kp, left), at32(kp, off), at32(kp, off + E)},
                        {at32(kp, left + row), at32(kp, off + row), at32(kp, off + row + E)}};
  const T* wp = pick_si<T>(e.si64, e.si32) + kPatchW * ((int64_t)slot * nm + (int64_t)p2 * n + p1);
  T w[2][kPatchW];
  auto load_w = [&](int c, T (&v)[kPatchW]) {
    const Pair* q = reinterpret_cast<const Pair*>(wp + kPatchW * ((int64_t)(c >> 1) * n + (c & 1)));
#pragma unroll
    for (int k = 0; k < kPatchW / 2; ++k) {
      const Pair u = q[k];
      v[2 * k] = u.a;
      v[2 * k + 1] = u.b;
    }
  };
  if constexpr (AHEAD) load_w(BWD ? 3 : 0, w[0]);
  T* pt = pl + t;
  if constexpr (!H::ZERO) {
    Cx<T> ux[4], uy[4];
    load_block(xc, N, off, row, wide, ux);
    load_block(xc + nm, N, off, row, wide, uy);
    if constexpr (H::PRO) {   // as the prolongation kernel: x + Pr xc
      // a coarse value across the period takes its phase as fetch() has it
      const bool xh = p1 == n - 2, yh = p2 == m - 2;
      const unsigned j = (unsigned)((p2 >> 1) * gc.n + (p1 >> 1)) * E;
      const unsigned jx = xh ? j + E - (unsigned)gc.n * E : j + E, jy = yh ? (unsigned)(p1 >> 1) * E : j + (unsigned)gc.n * E;
      const T *cx = cc, *cy = cc + gc.nm;
      const Cx<T> x00{at32(cx, j), at32(cx + gc.ne, j)}, y00{at32(cy, j), at32(cy + gc.ne, j)};
      Cx<T> x01{at32(cx, jy), at32(cx + gc.ne, jy)}, y10{at32(cy, jx), at32(cy + gc.ne, jx)};
      if (yh) x01 = cmul(x01, p.br, p.bi);
      if (xh) y10 = cmul(y10, p.ar, p.ai);
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        ux[c] = ux[c] + edge_prolong_combine<T>(x00, x01, c >> 1);
        uy[c] = uy[c] + edge_prolong_combine<T>(y00, y10, c & 1);
      }
    }
    if (live)
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        pt[c * S::SUB] = ux[c].re;
        pt[S::N + c * S::SUB] = ux[c].im;
        pt[2 * S::N + c * S::SUB] = uy[c].re;
        pt[3 * S::N + c * S::SUB] = uy[c].im;
      }
    __syncthreads();
  }
  const T s = (T)e.s, mx = (T)e.mx, my = (T)e.my, mmx = mu * mx, mmy = mu * my;
  four([&](auto order) {
    constexpr int k = decltype(order)::value, c = BWD ? 3 - k : k, px = c & 1, py = c >> 1;
    constexpr PassRect r = R.r[k];
    static_assert((r.x0 & 1) == px && (r.y0 & 1) == py && r.x0 >= 1 && r.y0 >= 1 && r.x1 <= BX - 2 && r.y1 <= BX - 2,
                  "pass rectangle");
    if constexpr (AHEAD && k < 3) load_w(BWD ? 2 - k : k + 1, w[(k + 1) & 1]);
    if (live && a >= (r.x0 >> 1) && a <= (r.x1 >> 1) && b >= (r.y0 >> 1) && b <= (r.y1 >> 1)) {
      PatchRhs<T> rhs;
      if constexpr (AHEAD) {
        rhs.q[0] = bx[c];
        rhs.q[1] = px ? bx[c & 2] : bl[py];
        rhs.q[2] = by[c];
        rhs.q[3] = py ? by[c & 1] : bd[px];
      } else {
        load_w(c, w[k & 1]);
        rhs.q[0] = load_own(0, c);
        rhs.q[1] = px ? load_own(0, c & 2) : load_left(py);
        rhs.q[2] = load_own(1, c);
        rhs.q[3] = py ? load_own(1, c & 1) : load_low(px);
      }
      const BlockEdges<T, S, px, py, CX, CY, H::ZERO ? k : 4> x{pt, Seam<CX, CY>(p1 + px, p2 + py, n, m), p};
      if constexpr (H::ZERO && k == 0)
        patch_solve<T>(x, w[k & 1], rhs.q[0], rhs.q[1], rhs.q[2], rhs.q[3]);
      else
        patch_update<T>(x, rhs, kap9[py + 1][px + 1], kap9[py + 1][px], kap9[py][px], kap9[py][px + 1], w[k & 1], s, mmx, mmy);
    }
    __syncthreads();
  });
  // the tile, whole rows at a time
  constexpr int ROWS = kThreads / TX, RK = TX / ROWS;
  const int ix = tid % TX, iy = tid / TX;
#pragma unroll
  for (int k = 0; k < RK; ++k) {
    const int c1 = t0x + ix, c2 = t0y + iy + k * ROWS;
    if (c1 >= n || c2 >= m) continue;
    const T* q = pl + S::at(ix + LO, iy + k * ROWS + LO);
    const unsigned i = (unsigned)(c2 * n + c1) * E;
    at32(xo, i) = q[0];
    at32(xo + N, i) = q[S::N];
    at32(xo + nm, i) = q[2 * S::N];
    at32(xo + N + nm, i) = q[3 * S::N];
  }
  if constexpr (H::RES) {
    // the residual b - (A + mu M) x (as the residual kernel computes it) in the window from one node
    // below and left of the tile that the restriction to the tile's coarse edges reads
    constexpr int W0 = LO - 1, W1 = LO + TX - 1;
    Cx<T> rx[4], ry[4];
    four([&](auto colour) {
      constexpr int c = decltype(colour)::value, px = c & 1, py = c >> 1;
      const int qx = 2 * a + px, qy = 2 * b + py;
      rx[c] = ry[c] = {0, 0};
      if (live && qx >= W0 && qx <= W1 && qy >= W0 && qy <= W1) {
        const BlockEdges<T, S, px, py, CX, CY> x{pt, Seam<CX, CY>(p1 + px, p2 + py, n, m), p};
        const Cx<T> ox0 = AHEAD ? bx[c] : load_own(0, c), oy0 = AHEAD ? by[c] : load_own(1, c);
        Cx<T> Au, Mu;
        edge_AM_acc<T>(x, 0, kap9[py][px + 1], kap9[py + 1][px + 1], s, mx, Au, Mu);
        rx[c] = ox0 - (Au + (mu * Mu));
        edge_AM_acc<T>(x, 1, kap9[py + 1][px + 1], kap9[py + 1][px], s, my, Au, Mu);
        ry[c] = oy0 - (Au + (mu * Mu));
      }
    });
    __syncthreads();   // the iterate has been read: its planes take the residual
    if (live)
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        pt[c * S::SUB] = rx[c].re;
        pt[S::N + c * S::SUB] = rx[c].im;
        pt[2 * S::N + c * S::SUB] = ry[c].re;
        pt[3 * S::N + c * S::SUB] = ry[c].im;
      }
    __syncthreads();
    const int f1 = ox + 2 * a, f2 = oy + 2 * b;
    if (live && a >= LO / 2 && a < (LO + TX) / 2 && b >= LO / 2 && b < (LO + TX) / 2 && f1 < n && f2 < m) {
      const BlockEdges<T, S, 0, 0, CX, CY> r{pt, Seam<CX, CY>(p1, p2, n, m), p};
      const Cx<T> vx = edge_restrict_acc<T>(r, 0), vy = edge_restrict_acc<T>(r, 1);
      const unsigned J = (unsigned)((f2 >> 1) * gc.n + (f1 >> 1)) * E;
      at32(bco, J) = vx.re;
      at32(bco + gc.ne, J) = vx.im;
      at32(bco + gc.nm, J) = vy.re;
      at32(bco + gc.ne + gc.nm, J) = vy.im;
    }
  }
}

template <typename T, bool BWD, int MODE>
__global__ __launch_bounds__(kThreads) void k_edge_sweep(View<const T> xin, View<T> xout, View<const T> bv, EdgeArgs a, Geo g,
                                                      const Phase* __restrict__ phs, const double* __restrict__ mus,
                                                      int wide, const int* __restrict__ slots, int ncps, int tiles_x,
                                                      SweepFuse<T> fz) {
  static_assert(!((MODE & (kRestrict | kZero)) && BWD), "the order of the colours");
  static_assert(!(MODE & (kBase | kResid)), "nodal sweeps only");
  using H = EdgeShape<T, BWD, MODE>;
  __shared__ T pl[4 * H::S::N];
  const TileRef tr = tile_ref(slots, ncps, tiles_x, H::TX, H::TX);
  const int n = g.n, m = g.m;
  const int64_t N = g.ne, nm = g.nm;
  const int ox = tr.t0x - H::LO, oy = tr.t0y - H::LO;
  const bool cx = !(ox >= 0 && ox + H::BX <= n), cy = !(oy >= 0 && oy + H::BX <= m);
  const SJ sj{tr.slot, tr.j};
  T* xo = colp(xout, sj, N);
  const T* bc = colp(bv, sj, N);
  const T* xc = H::ZERO ? nullptr : colp(xin, sj, N);
  const T* cc = H::PRO ? colp(fz.xc, sj, fz.gc.ne) : nullptr;
  T* bco = H::RES ? colp(fz.bc, sj, fz.gc.ne) : nullptr;
  const Ph<T> p = cast_phase<T>(phs[tr.slot]);
  const T mu = (T)mus[tr.slot];
#define BL_TILE(CX, CY) \
  edge_tile<T, BWD, MODE, CX, CY>(pl, xc, xo, bc, cc, bco, a, tr.slot, tr.t0x, tr.t0y, n, m, N, nm, fz.gc, mu, p, wide != 0)
  if (!cx && !cy) BL_TILE(false, false);
  else if (!cy) BL_TILE(true, false);
  else if (!cx) BL_TILE(false, true);
  else BL_TILE(true, true);
#undef BL_TILE
}

// ---- nodal sweeps ---------------------------------------------------------------------------
// A thread owns one 2 x 2 block of the box's nodes (blocks of HX a row, so that block t is entry t of
// every parity sub-grid) in all passes: its addresses, its seam flags and its right-hand side are
// worked out and loaded once, with the iterate, and a pass is LDS reads at constant offsets and
// arithmetic.  Passes that dealt out a colour's nodes anew each time were bound by the vector units:
// 230 to 330 instructions per node, three quarters of them addressing and reloading; this form takes
// 160 to 240.  A sweep from zero (84 % of the vector issue) leaves out what is still zero; the
// prolongating ones wait for memory half the time.  1024 x 1024 FP32, 48 columns, finest level:
// restricting sweep 295 us, prolongating with residual 484, prolongating onto the base 416, against
// 395, 624 and 486; 256 x 256 FP64: 73 and 48 us for the last two, against 103 and 84.
// The values around a node of block t in the iterate's planes; colours from FIRST on are still zero.
template <typename T, typename S, int PX, int PY, bool CX, bool CY, int FIRST = 4>
struct BlockNodes {
  const T* pl;   // at entry t
  Seam<CX, CY> sm;
  const Ph<T>& p;
  __device__ __forceinline__ Cx<T> get(int d1, int d2) const {
    const int sx = (PX + d1) & 1, sy = (PY + d2) & 1;
    if (sx + 2 * sy >= FIRST) return {0, 0};
    const T* q = pl + (sx + 2 * sy) * S::SUB + ((PY + d2) >> 1) * S::HX + ((PX + d1) >> 1);
    return phased<CX, CY, T>(Cx<T>{q[0], q[S::N]}, d1, d2, sm, p);
  }
};

template <typename T, bool BWD, int MODE>
struct NodalShape {
  static constexpr bool RES = (MODE & kRestrict) != 0, PRO = (MODE & kProlong) != 0, BAS = (MODE & kBase) != 0;
  static constexpr bool TRES = (MODE & kResid) != 0, ZERO = (MODE & kZero) != 0;
  static constexpr int TX = kTile, LO = RES ? kLoR : kLo;
  static constexpr int HI = TRES ? kHiN + 1 : kHiN;   // (the tile residual: exact one node above / right too)
  static constexpr int BX = TX + LO + HI;
  using S = Split<BX, BX>;
  // coarse nodes under the box: fine box position b lies over coarse box position b >> 1 and its
  // neighbours one up
  static constexpr int CBX = (BX - 1) / 2 + 2, CB = CBX * CBX;
  // exact margin the residual window (restriction) or the tile residual needs
  static constexpr int EA = RES ? 2 : (TRES ? 1 : 0), EB = (RES || TRES) ? 1 : 0;
  static constexpr SweepRects R = sweep_rects(false, BX, BX, LO, TX, TX, EA, EB, BWD);
  static_assert(R.ok, "the halo does not cover the sweep's dependency cone");
  static_assert(S::SUB <= kThreads && CB <= kThreads, "a block per thread");
};

template <typename T, bool BWD, int MODE, bool CX, bool CY>
__device__ __forceinline__ void nodal_tile(T* pl, T* cl, const T* xc, T* xo, const T* bc, const T* cc, T* bco, const T* bs,
                                           T* ro, const NodalStencil& st, int t0x, int t0y, int n, int m, int64_t N,
                                           const Geo& gc, const Ph<T>& p, bool wide) {
  using H = NodalShape<T, BWD, MODE>;
  using S = typename H::S;
  constexpr int LO = H::LO, BX = H::BX, TX = H::TX;
  constexpr SweepRects R = H::R;
  const int tid = (int)threadIdx.x;
  const bool live = tid < S::SUB;
  const int t = live ? tid : 0, a = t % S::HX, b = t / S::HX;
  const int ox = t0x - LO, oy = t0y - LO;   // canonical node of box position 0 (unwrapped)
  // canonical first node of the block (n, m, ox and oy are even: a block never straddles the seam,
  // and where the box has an odd number of nodes its last block still lies in the grid)
  const int p1 = CX ? wrapm(ox + 2 * a, n) : ox + 2 * a, p2 = CY ? wrapm(oy + 2 * b, m) : oy + 2 * b;
  const unsigned off = (unsigned)(p2 * n + p1) * (unsigned)sizeof(T), row = (unsigned)n * (unsigned)sizeof(T);
  Cx<T> rhs[4], u[4];
  load_block(bc, N, off, row, wide, rhs);
  if constexpr (!H::ZERO) load_block(xc, N, off, row, wide, u);
  // the tile, whole rows at a time
  constexpr int ROWS = kThreads / TX, RK = TX / ROWS;
  const int ix = tid % TX, iy = tid / TX;
  Cx<T> base[RK];
  if constexpr (H::BAS)
#pragma unroll
    for (int k = 0; k < RK; ++k) {
      const int c1 = t0x + ix, c2 = t0y + iy + k * ROWS;
      const unsigned i = c1 < n && c2 < m ? (unsigned)(c2 * n + c1) * (unsigned)sizeof(T) : 0u;
      base[k] = Cx<T>{at32(bs, i), at32(bs + N, i)};
    }
  T* pt = pl + t;
  if constexpr (H::PRO) {   // as the prolongation kernel: x + Pr xc
    // the coarse values under the box; a value across the period takes its phase as fetch() has it
    if (tid < H::CB) {
      const int J1 = wrapm((ox >> 1) + tid % H::CBX, gc.n), J2 = wrapm((oy >> 1) + tid / H::CBX, gc.m);
      const unsigned i = (unsigned)(J2 * gc.n + J1) * (unsigned)sizeof(T);
      cl[tid] = at32(cc, i);
      cl[H::CB + tid] = at32(cc + gc.nm, i);
    }
    __syncthreads();
    const T* q = cl + b * H::CBX + a;
    const Cx<T> c00{q[0], q[H::CB]};
    Cx<T> c10{q[1], q[H::CB + 1]}, c01{q[H::CBX], q[H::CB + H::CBX]}, c11{q[H::CBX + 1], q[H::CB + H::CBX + 1]};
    if (p1 == n - 2) {
      c10 = cmul(c10, p.ar, p.ai);
      c11 = cmul(c11, p.ar, p.ai);
    }
    if (p2 == m - 2) {
      c01 = cmul(c01, p.br, p.bi);
      c11 = cmul(c11, p.br, p.bi);
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) u[c] = u[c] + nodal_prolong_combine<T>(c00, c10, c01, c11, c & 1, c >> 1);
  }
  if constexpr (!H::ZERO) {
    if (live)
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        pt[c * S::SUB] = u[c].re;
        pt[S::N + c * S::SUB] = u[c].im;
      }
    __syncthreads();
  }
  const T inv = (T)1 / (T)st.c0;
  auto node = [&](auto colour) {
    constexpr int c = decltype(colour)::value;
    return BlockNodes<T, S, (c & 1), (c >> 1), CX, CY>{pt, Seam<CX, CY>(p1 + (c & 1), p2 + (c >> 1), n, m), p};
  };
  auto pass = [&](auto order) {
    constexpr int k = decltype(order)::value, c = BWD ? 3 - k : k;
    constexpr PassRect r = R.r[k];
    static_assert((r.x0 & 1) == (c & 1) && (r.y0 & 1) == (c >> 1) && r.x0 >= 1 && r.y0 >= 1 && r.x1 <= BX - 2 && r.y1 <= BX - 2,
                  "pass rectangle");
    if (live && a >= (r.x0 >> 1) && a <= (r.x1 >> 1) && b >= (r.y0 >> 1) && b <= (r.y1 >> 1)) {
      const BlockNodes<T, S, (c & 1), (c >> 1), CX, CY, H::ZERO ? c : 4> x{
          pt, Seam<CX, CY>(p1 + (c & 1), p2 + (c >> 1), n, m), p};
      const Cx<T> v = rhs[c] - nodal_stencil_at<T>(x, st), o = x.get(0, 0);
      pt[c * S::SUB] = o.re + inv * v.re;
      pt[S::N + c * S::SUB] = o.im + inv * v.im;
    }
    __syncthreads();
  };
  pass(std::integral_constant<int, 0>{});
  pass(std::integral_constant<int, 1>{});
  pass(std::integral_constant<int, 2>{});
  pass(std::integral_constant<int, 3>{});
#pragma unroll
  for (int k = 0; k < RK; ++k) {
    const int c1 = t0x + ix, c2 = t0y + iy + k * ROWS;
    if (c1 >= n || c2 >= m) continue;
    const int q = S::at(ix + LO, iy + k * ROWS + LO);
    const unsigned i = (unsigned)(c2 * n + c1) * (unsigned)sizeof(T);
    Cx<T> v{pl[q], pl[S::N + q]};
    if constexpr (H::BAS) v = base[k] + v;   // as the update kernel: base + x
    at32(xo, i) = v.re;
    at32(xo + N, i) = v.im;
  }
  if constexpr (H::TRES || H::RES) {
    // the residual b - P x, as the residual kernel computes it, at the nodes of the block in the
    // tile (TRES), or in the window from one node below and left of it that the restriction to the
    // tile's coarse nodes reads
    constexpr int W0 = LO - (H::RES ? 1 : 0), W1 = LO + TX - 1;
    Cx<T> r[4];
    auto resid = [&](auto colour) {
      constexpr int c = decltype(colour)::value;
      const int bx = 2 * a + (c & 1), by = 2 * b + (c >> 1);
      r[c] = {0, 0};
      if (live && bx >= W0 && bx <= W1 && by >= W0 && by <= W1) r[c] = rhs[c] - nodal_stencil_at<T>(node(colour), st);
    };
    resid(std::integral_constant<int, 0>{});
    resid(std::integral_constant<int, 1>{});
    resid(std::integral_constant<int, 2>{});
    resid(std::integral_constant<int, 3>{});
    __syncthreads();   // the iterate has been read: its planes take the residual
    if (live)
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        pt[c * S::SUB] = r[c].re;
        pt[S::N + c * S::SUB] = r[c].im;
      }
    __syncthreads();
    if constexpr (H::TRES) {
#pragma unroll
      for (int k = 0; k < RK; ++k) {
        const int c1 = t0x + ix, c2 = t0y + iy + k * ROWS;
        if (c1 >= n || c2 >= m) continue;
        const int q = S::at(ix + LO, iy + k * ROWS + LO);
        const unsigned i = (unsigned)(c2 * n + c1) * (unsigned)sizeof(T);
        at32(ro, i) = pl[q];
        at32(ro + N, i) = pl[S::N + q];
      }
    } else {
      const int f1 = ox + 2 * a, f2 = oy + 2 * b;
      if (live && a >= LO / 2 && a < (LO + TX) / 2 && b >= LO / 2 && b < (LO + TX) / 2 && f1 < n && f2 < m) {
        const Cx<T> v = nodal_restrict_acc<T>(node(std::integral_constant<int, 0>{}));
        const unsigned J = (unsigned)((f2 >> 1) * gc.n + (f1 >> 1)) * (unsigned)sizeof(T);
        at32(bco, J) = v.re;
        at32(bco + gc.nm, J) = v.im;
      }
    }
  }
}

template <typename T, bool BWD, int MODE>
__global__ __launch_bounds__(kThreads) void k_nodal_sweep(View<const T> xin, View<T> xout, View<const T> bv, Geo g,
                                                            const Phase* __restrict__ phs, NodalStencil st,
                                                            int wide, const int* __restrict__ slots, int ncps,
                                                            int tiles_x, SweepFuse<T> fz) {
  static_assert(!((MODE & kRestrict) && BWD), "the residual window halo is sized for forward sweeps");
  static_assert(!((MODE & kResid) && !BWD), "the tile residual rides on backward sweeps");
  static_assert(!((MODE & kZero) && BWD), "the order of the colours in a sweep from zero");
  using H = NodalShape<T, BWD, MODE>;
  __shared__ T pl[2 * H::S::N];
  __shared__ T cl[H::PRO ? 2 * H::CB : 1];
  const TileRef tr = tile_ref(slots, ncps, tiles_x, H::TX, H::TX);
  const int n = g.n, m = g.m;
  const int64_t N = g.nm;
  const int ox = tr.t0x - H::LO, oy = tr.t0y - H::LO;
  const bool cx = !(ox >= 0 && ox + H::BX <= n), cy = !(oy >= 0 && oy + H::BX <= m);
  const SJ sj{tr.slot, tr.j};
  T* xo = colp(xout, sj, N);
  const T* bc = colp(bv, sj, N);
  const T* xc = H::ZERO ? nullptr : colp(xin, sj, N);
  const T* cc = H::PRO ? colp(fz.xc, sj, fz.gc.nm) : nullptr;
  T* bco = H::RES ? colp(fz.bc, sj, fz.gc.nm) : nullptr;
  const T* bs = H::BAS ? colp(fz.base, sj, N) : nullptr;
  T* ro = H::TRES ? colp(fz.res, sj, N) : nullptr;
  const Ph<T> p = cast_phase<T>(phs[tr.slot]);
  if (!cx && !cy)
    nodal_tile<T, BWD, MODE, false, false>(pl, cl, xc, xo, bc, cc, bco, bs, ro, st, tr.t0x, tr.t0y, n, m, N, fz.gc, p, wide != 0);
  else if (!cy)
    nodal_tile<T, BWD, MODE, true, false>(pl, cl, xc, xo, bc, cc, bco, bs, ro, st, tr.t0x, tr.t0y, n, m, N, fz.gc, p, wide != 0);
  else if (!cx)
    nodal_tile<T, BWD, MODE, false, true>(pl, cl, xc, xo, bc, cc, bco, bs, ro, st, tr.t0x, tr.t0y, n, m, N, fz.gc, p, wide != 0);
  else
    nodal_tile<T, BWD, MODE, true, true>(pl, cl, xc, xo, bc, cc, bco, bs, ro, st, tr.t0x, tr.t0y, n, m, N, fz.gc, p, wide != 0);
}

// Two values a load where the columns (whole numbers of pairs) start on a pair.
template <typename T>
int wide_loads(View<const T> b, View<const T> x) {
  return (((uintptr_t)b.p | (uintptr_t)x.p) & (2 * sizeof(T) - 1)) == 0 ? 1 : 0;
}

template <typename T, bool BWD, int MODE>
void edge_go(View<const T> xin, View<T> xout, View<const T> b, const EdgeArgs& a, const Geo& g, const Phase* ph,
             const double* mu, const SweepFuse<T>& fz, const Launch& L) {
  const int tx = (g.n + kTile - 1) / kTile, ty = (g.m + kTile - 1) / kTile;
  dim3 grid((unsigned)(tx * ty), (unsigned)(L.nact * L.ncps));
  k_edge_sweep<T, BWD, MODE><<<grid, kThreads, 0, L.st>>>(xin, xout, b, a, g, ph, mu, wide_loads(b, xin), L.slots, L.ncps, tx,
                                                         fz);
}

template <typename T, bool BWD, int MODE>
void nodal_go(View<const T> xin, View<T> xout, View<const T> b, const Geo& g, const Phase* ph, const NodalStencil& c,
              const SweepFuse<T>& fz, const Launch& L) {
  const int tx = (g.n + kTile - 1) / kTile, ty = (g.m + kTile - 1) / kTile;
  dim3 grid((unsigned)(tx * ty), (unsigned)(L.nact * L.ncps));
  k_nodal_sweep<T, BWD, MODE><<<grid, kThreads, 0, L.st>>>(xin, xout, b, g, ph, c, wide_loads(b, xin), L.slots, L.ncps, tx,
                                                          fz);
}

}  // namespace

template <typename T>
void edge_sweep(View<const T> xin, View<T> xout, View<const T> b, const double* kappa64, const float* kappa32,
                const double* sinv64, const float* sinv32, const Geo& g, const Phase* ph, const double* mu,
                bool backward, bool zero_start, const Launch& L, const SweepFuse<T>& fz) {
  if (L.nact * L.ncps == 0) return;
  const EdgeArgs a{kappa64, kappa32, sinv64, sinv32, g.s, g.mx, g.my};
  if (backward) {
    if (fz.xc.p) edge_go<T, true, kProlong>(xin, xout, b, a, g, ph, mu, fz, L);
    else edge_go<T, true, 0>(xin, xout, b, a, g, ph, mu, fz, L);
  } else if (fz.bc.p) {
    if (zero_start) edge_go<T, false, kRestrict | kZero>(xin, xout, b, a, g, ph, mu, fz, L);
    else edge_go<T, false, kRestrict>(xin, xout, b, a, g, ph, mu, fz, L);
  } else {
    if (zero_start) edge_go<T, false, kZero>(xin, xout, b, a, g, ph, mu, fz, L);
    else edge_go<T, false, 0>(xin, xout, b, a, g, ph, mu, fz, L);
  }
}

template <typename T>
void nodal_sweep(View<const T> xin, View<T> xout, View<const T> b, const Geo& g, const Phase* ph,
                 const NodalStencil& c, bool backward, bool zero_start, const Launch& L, const SweepFuse<T>& fz) {
  if (L.nact * L.ncps == 0) return;
  const int mode = (fz.bc.p ? kRestrict : 0) | (fz.xc.p ? kProlong : 0) | (fz.base.p ? kBase : 0) |
                   (fz.res.p ? kResid : 0);
  if (!backward) {
    if (mode == kRestrict && zero_start) nodal_go<T, false, kRestrict | kZero>(xin, xout, b, g, ph, c, fz, L);
    else if (mode == kRestrict) nodal_go<T, false, kRestrict>(xin, xout, b, g, ph, c, fz, L);
    else if (zero_start) nodal_go<T, false, kZero>(xin, xout, b, g, ph, c, fz, L);
    else nodal_go<T, false, 0>(xin, xout, b, g, ph, c, fz, L);
    return;
  }
  switch (mode) {
    case kProlong: nodal_go<T, true, kProlong>(xin, xout, b, g, ph, c, fz, L); break;
    case kBase: nodal_go<T, true, kBase>(xin, xout, b, g, ph, c, fz, L); break;
    case kProlong | kBase: nodal_go<T, true, kProlong | kBase>(xin, xout, b, g, ph, c, fz, L); break;
    case kProlong | kResid: nodal_go<T, true, kProlong | kResid>(xin, xout, b, g, ph, c, fz, L); break;
    case kResid: nodal_go<T, true, kResid>(xin, xout, b, g, ph, c, fz, L); break;
    default: nodal_go<T, true, 0>(xin, xout, b, g, ph, c, fz, L); break;
  }
}

template void edge_sweep<double>(View<const double>, View<double>, View<const double>, const double*, const float*, const double*, const float*, const Geo&, const Phase*, const double*, bool, bool, const Launch&, const SweepFuse<double>&);
template void edge_sweep<float>(View<const float>, View<float>, View<const float>, const double*, const float*, const double*, const float*, const Geo&, const Phase*, const double*, bool, bool, const Launch&, const SweepFuse<float>&);
template void nodal_sweep<double>(View<const double>, View<double>, View<const double>, const Geo&, const Phase*, const NodalStencil&, bool, bool, const Launch&, const SweepFuse<double>&);
template void nodal_sweep<float>(View<const float>, View<float>, View<const float>, const Geo&, const Phase*, const NodalStencil&, bool, bool, const Launch&, const SweepFuse<float>&);

}  // namespace bl

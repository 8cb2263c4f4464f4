// V-cycle legs of the large 3D levels: the stages of a leg march through the
// planes of a column of cells together (see legs.hpp for what a leg is).
//
// A block owns TX x TY cells in x-y and tz planes.  At step t the first stage
// forms plane t, every further stage (an operator application each) plane t -
// 2, t - 4, ... from the planes that the stage before finished in earlier
// steps, so a step has one barrier and no stage waits for another.  A thread
// is one (x, y) column for all stages: the values of its own column above and
// below stay in registers, and so does the divergence of the cell below; LDS
// holds the last three planes of each iterate for the neighbours in the
// plane.  The halo is recomputed in x and y only (two sites per application),
// at the ends of a chunk also in z.
//
// What a leg moves is then b read and x written (and the coarse level), where
// separate kernels read and write the iterates of every stage again.  Bound
// by the length of a step, about 2 us: a compute unit holds one block, whose
// waves go through the stages in step and meet at the barrier, so LDS reads,
// arithmetic (half of the issue slots) and waits add up; prefetching one or
// three planes ahead, or half as many waves per block, changed it by less than a
// tenth.  Where the march takes a level, and what both sides measured, stands
// at march_plan.
#include <algorithm>
#include <type_traits>

#include "legsites.hpp"

namespace gkb {
namespace {

template <typename T>
struct Tri {
  T u, v, w;
};

template <int TX_, int TY_, int NT_>
struct MTile {
  static constexpr int TX = TX_, TY = TY_, NT = NT_;
};

// What the leg reads of the grid, in the form that the loop needs: byte
// offsets and strides of the three face arrays, the pinned cell.
struct Geo {
  int n[3];
  unsigned lo, hi;  // bit a: the lower / upper side of axis a is a wall
  int off[3], row[3], pl[3];  // entries
  int pi, pj, pk;
  unsigned bytes;  // of a face array
};
inline Geo make_geo(const Grid& g, int elem) {
  Geo q{};
  for (int a = 0; a < 3; ++a) {
    q.n[a] = g.n[a];
    q.lo |= unsigned(g.bc[2 * a] == kDir) << a;
    q.hi |= unsigned(g.bc[2 * a + 1] == kDir) << a;
    q.off[a] = g.off[a];
    q.row[a] = g.ext[a][0];
    q.pl[a] = g.ext[a][0] * g.ext[a][1];
  }
  const int nxy = g.n[0] * g.n[1];
  q.pk = g.pin >= 0 ? g.pin / nxy : -9;
  q.pj = g.pin >= 0 ? (g.pin - q.pk * nxy) / g.n[0] : -9;
  q.pi = g.pin >= 0 ? g.pin - q.pk * nxy - q.pj * g.n[0] : -9;
  q.bytes = unsigned(g.m_full) * elem;
  return q;
}
__device__ __forceinline__ bool normal_on(const Geo& G, int a, int l) {
  return l >= int((G.lo >> a) & 1u) && l <= G.n[a] - int((G.hi >> a) & 1u);
}
// diagonal weight of the tangential couplings along axis a at cell l
__device__ __forceinline__ int side_weight(const Geo& G, int a, int l) {
  int v = 2;
  if (l == 0) v += (G.lo >> a) & 1u ? 1 : -1;
  if (l == G.n[a] - 1) v += (G.hi >> a) & 1u ? 1 : -1;
  return v;
}
__device__ __forceinline__ bool cell_live(const Geo& G, int i, int j, int k) {
  return unsigned(i) < unsigned(G.n[0]) && unsigned(j) < unsigned(G.n[1]) &&
         unsigned(k) < unsigned(G.n[2]) && !(i == G.pi && j == G.pj && k == G.pk);
}

// what a column knows about the grid
template <typename T>
struct Column {
  int i, j;
  bool ou, ov, oc;      // its u, v faces are unknowns along x-y; it is a column of cells
  unsigned u, v, w;     // byte offset of its faces on plane 0 (0 where none)
  T cx, cy;             // diagonal weight of the tangential couplings along x, y
  T hu, hv, nu, nv;     // half control volumes and normal couplings at do-nothing sides
};
template <typename T>
__device__ __forceinline__ Column<T> make_column(const Geo& G, bool live, int i, int j) {
  Column<T> c;
  const bool ci = unsigned(i) < unsigned(G.n[0]), cj = unsigned(j) < unsigned(G.n[1]);
  c.i = i, c.j = j;
  c.ou = live && cj && normal_on(G, 0, i);
  c.ov = live && ci && normal_on(G, 1, j);
  c.oc = live && ci && cj;
  // in the array (the boundary faces that are no unknown are stored as 0)
  const bool au = live && cj && unsigned(i) <= unsigned(G.n[0]);
  const bool av = live && ci && unsigned(j) <= unsigned(G.n[1]);
  c.u = (au ? unsigned(G.off[0] + j * G.row[0] + i) : 0u) * unsigned(sizeof(T));
  c.v = (av ? unsigned(G.off[1] + j * G.row[1] + i) : 0u) * unsigned(sizeof(T));
  c.w = (c.oc ? unsigned(G.off[2] + j * G.row[2] + i) : 0u) * unsigned(sizeof(T));
  c.cx = T(side_weight(G, 0, i));
  c.cy = T(side_weight(G, 1, j));
  const bool eu = i == 0 || i == G.n[0], ev = j == 0 || j == G.n[1];
  c.hu = eu ? T(0.5) : T(1);
  c.nu = eu ? T(1) : T(2);
  c.hv = ev ? T(0.5) : T(1);
  c.nv = ev ? T(1) : T(2);
  return c;
}

// what a plane adds: which faces exist on it, and its (uniform) byte offsets,
// clamped to the arrays
struct Plane {
  bool cell, nrm;
  unsigned u, v, w;
};
template <typename T>
__device__ __forceinline__ Plane make_plane(const Geo& G, int k) {
  const int kc = min(max(k, 0), G.n[2] - 1), kw = min(max(k, 0), G.n[2]);
  return {unsigned(k) < unsigned(G.n[2]), normal_on(G, 2, k), unsigned(kc * G.pl[0] * int(sizeof(T))),
          unsigned(kc * G.pl[1] * int(sizeof(T))), unsigned(kw * G.pl[2] * int(sizeof(T)))};
}

// values of an array at the column's faces on a plane: a uniform base, the
// column's 32-bit offset and the plane's uniform one, so no address
// arithmetic; always inside the array, masked by the user
template <typename T>
__device__ __forceinline__ Tri<T> load_faces(__amdgpu_buffer_rsrc_t a, const Column<T>& c,
                                             const Plane& p) {
  return {buf_load<T>(a, c.u, p.u), buf_load<T>(a, c.v, p.v), buf_load<T>(a, c.w, p.w)};
}
template <typename T>
__device__ __forceinline__ Tri<T> masked(const Column<T>& c, const Plane& p, T u, T v, T w) {
  return {c.ou && p.cell ? u : T(0), c.ov && p.cell ? v : T(0), c.oc && p.nrm ? w : T(0)};
}

// Constant viscosity: h^2 times the viscous diagonal (vd) and omega / D over
// h^2 (sc) of the column's faces, for any plane away from the ends of the
// grid and the pinned cell (k < 0) or for plane k.
template <typename T>
struct Diag {
  Tri<T> vd, sc;
};
template <typename T>
__device__ __forceinline__ Diag<T> make_diag(const Geo& G, const Column<T>& c, T eta, T om, int k) {
  const bool bulk = k < 0;
  const T cz = bulk ? T(2) : T(side_weight(G, 2, k));
  const bool ew = !bulk && (k == 0 || k == G.n[2]);
  Diag<T> d;
  d.vd = {c.nu + c.hu * (c.cy + cz), c.nv + c.hv * (c.cx + cz),
          (ew ? T(1) : T(2)) + (ew ? T(0.5) : T(1)) * (c.cx + c.cy)};
  // valid cells beside each face
  const int kb = bulk ? -99 : k;
  auto pin = [&](int i, int j, int l) { return i == G.pi && j == G.pj && l == G.pk; };
  const int nu = int(c.i < G.n[0] && !pin(c.i, c.j, kb)) + int(c.i > 0 && !pin(c.i - 1, c.j, kb));
  const int nv = int(c.j < G.n[1] && !pin(c.i, c.j, kb)) + int(c.j > 0 && !pin(c.i, c.j - 1, kb));
  const int nw = int((bulk || k < G.n[2]) && !pin(c.i, c.j, kb)) +
                 int((bulk || k > 0) && !pin(c.i, c.j, kb - 1));
  d.sc = {om / (d.vd.u + eta * T(nu)), om / (d.vd.v + eta * T(nv)), om / (d.vd.w + eta * T(nw))};
  return d;
}
// plane k has the bulk diagonal
__device__ __forceinline__ bool bulk_plane(const Geo& G, int k) {
  return k > 0 && k < G.n[2] - 1 && k != G.pk && k - 1 != G.pk;
}

// Rows of h^2 M x at the column's faces on plane k.  c: its entry in LDS on
// plane k (components CS apart, rows SY apart), tw: its w entry on plane k + 1;
// B, C, A: its own values on planes k - 1, k, k + 1; dB: the divergence of the
// cell below, replaced by the cell's; vd: the viscous diagonal (constant
// viscosity).  Sites that are no unknown hold 0; results there are
// meaningless.  special (uniform): a side of the grid is a do-nothing one or
// the pinned cell is near.
template <typename T, int SY, int CS>
__device__ __forceinline__ Tri<T> march_row(const Geo& G, T eta, const Column<T>& q, bool special,
                                            const T* c, const T* tw, const Tri<T>& B,
                                            const Tri<T>& C, const Tri<T>& A, T& dB, int k,
                                            const Tri<T>& vd) {
  const T *U = c, *V = c + CS, *W = c + 2 * CS;
  const T uE = U[1], uW = U[-1], uN = U[SY], uS = U[-SY], uSE = U[1 - SY];
  const T vE = V[1], vW = V[-1], vN = V[SY], vS = V[-SY], vNW = V[SY - 1];
  const T wE = W[1], wW = W[-1], wN = W[SY], wS = W[-SY], wTW = tw[-1], wTS = tw[-SY];
  T dC = (C.u - uE) + (C.v - vN) + (C.w - A.w);
  T dW = (uW - C.u) + (vW - vNW) + (wW - wTW);
  T dS = (uS - uSE) + (vS - C.v) + (wS - wTS);
  T hu = T(1), hv = T(1), hw = T(1);
  if (special) {
    dC = cell_live(G, q.i, q.j, k) ? dC : T(0);
    dW = cell_live(G, q.i - 1, q.j, k) ? dW : T(0);
    dS = cell_live(G, q.i, q.j - 1, k) ? dS : T(0);
    hu = q.hu, hv = q.hv;
    if (k == 0 || k == G.n[2]) hw = T(0.5);
  }
  Tri<T> r;
  r.u = vd.u * C.u - ((uW + uE) + hu * ((uS + uN) + (B.u + A.u)));
  r.v = vd.v * C.v - ((vS + vN) + hv * ((vW + vE) + (B.v + A.v)));
  r.w = vd.w * C.w - ((B.w + A.w) + hw * ((wW + wE) + (wS + wN)));
  r.u += eta * (dC - dW);
  r.v += eta * (dC - dS);
  r.w += eta * (dC - dB);
  dB = dC;
  return r;
}

// a side is do-nothing, or the pinned cell lies in the block's box
__device__ __forceinline__ bool special_block(const Geo& G, int i0, int i1, int j0, int j1, int k0,
                                              int k1) {
  return (G.lo & G.hi) != 7u || (G.pi >= i0 && G.pi < i1 && G.pj >= j0 && G.pj < j1 &&
                                 G.pk >= k0 && G.pk < k1);
}

// tile of a block: blocks of one XCD are neighbours, so that the halo they
// share is in its L2
struct Where {
  int x, y, z, lin;
};
__device__ __forceinline__ Where my_tile() {
  const int nb = gridDim.x * gridDim.y * gridDim.z;
  const int b = blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z);
  const int xcd = b & 7, lin = xcd * (nb >> 3) + min(xcd, nb & 7) + (b >> 3);
  const int rest = lin / gridDim.x;
  return {int(lin % gridDim.x), int(rest % gridDim.y), int(rest / gridDim.y), b};
}

// stores a plane of the leg's result at the faces that the tile owns: its own
// sites, and the boundary faces right behind it
template <class TL, typename T>
struct Owner {
  bool u, v, w;
  __device__ __forceinline__ Owner(const Geo& G, bool live, int x, int y, int i, int j) {
    const bool lo = live && x >= 0 && y >= 0;
    u = lo && x < TL::TX + int(i == G.n[0]) && y < TL::TY && i <= G.n[0] && j < G.n[1];
    v = lo && x < TL::TX && y < TL::TY + int(j == G.n[1]) && i < G.n[0] && j <= G.n[1];
    w = lo && x < TL::TX && y < TL::TY && i < G.n[0] && j < G.n[1];
  }
  __device__ __forceinline__ void store(const Geo& G, const Column<T>& c, __amdgpu_buffer_rsrc_t a,
                                        int k, int k0, int k1, const Tri<T>& r) const {
    if (k < k0 || k >= k1 + int(k1 == G.n[2])) return;  // uniform
    const Plane p = make_plane<T>(G, k);
    if (k < k1) {
      if (u) buf_store(r.u, a, c.u, p.u);
      if (v) buf_store(r.v, a, c.v, p.v);
    }
    if (w) buf_store(r.w, a, c.w, p.w);
  }
};

// ------------------------------------------------------------- way down

// restriction of component C at coarse site (I, J, K) from the planes r[0 .. 3]
// = 2K - 1 .. 2K + 2 of the residual in LDS (entry of the fine site (2I, 2J))
template <typename T, int C, int SY, bool SMOOTH>
__device__ __forceinline__ T march_restrict(const Grid& Gc, const T* const* r, int I, int J, int K) {
  T acc = T(0);
  // weights along x, y (sites 2I - 1 .. 2I + 2) and z (planes 2K - 1 .. 2K + 2)
  T w[3][4];
  const int P[3] = {I, J, K};
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    if (a == C) {
      w[a][0] = w[a][2] = T(0.5);
      w[a][1] = T(1);
      w[a][3] = T(0);
    } else if (SMOOTH) {
      w[a][0] = w[a][3] = T(0.25);
      w[a][1] = cover_weight<T>(2 * P[a], Gc.n[a], Gc.bc[2 * a], Gc.bc[2 * a + 1]);
      w[a][2] = cover_weight<T>(2 * P[a] + 1, Gc.n[a], Gc.bc[2 * a], Gc.bc[2 * a + 1]);
    } else {
      w[a][0] = w[a][3] = T(0);
      w[a][1] = w[a][2] = T(1);
    }
  }
  constexpr int lo[3] = {C == 0 ? 0 : 1, C == 1 ? 0 : 1, C == 2 ? 0 : 1};
  if constexpr (SMOOTH) {
#pragma unroll
    for (int z = 0; z < (C == 2 ? 3 : 4); ++z) {
      T t = T(0);
#pragma unroll
      for (int y = 0; y < (C == 1 ? 3 : 4); ++y) {
        T s = T(0);
#pragma unroll
        for (int x = 0; x < (C == 0 ? 3 : 4); ++x) s += w[0][x] * r[z][(y - 1) * SY + x - 1];
        t += w[1][y] * s;
      }
      acc += w[2][z] * t;
    }
  } else {
#pragma unroll
    for (int z = lo[2]; z < 3; ++z) {
      T t = T(0);
#pragma unroll
      for (int y = lo[1]; y < 3; ++y) {
        T s = T(0);
#pragma unroll
        for (int x = lo[0]; x < 3; ++x) s += w[0][x] * r[z][(y - 1) * SY + x - 1];
        t += w[1][y] * s;
      }
      acc += w[2][z] * t;
    }
  }
  return acc * T(0.125);
}

template <typename T, class TL, bool SMOOTH>
__global__ __launch_bounds__(TL::NT) void k_march_down(LegLevel<T> L, Geo G, const T* __restrict__ b,
                                                       T* __restrict__ xo, T* __restrict__ bc,
                                                       const T* __restrict__ dinv_c, T omega_c,
                                                       T* __restrict__ x0c,
                                                       const PcgState* __restrict__ st, int tz) {
  constexpr int TX = TL::TX, TY = TL::TY, NT = TL::NT;
  constexpr int EX = TX + 6, EY = TY + 6, EN = EX * EY;  // first iterate
  constexpr int WX = TX + 4, WY = TY + 4, WN = WX * WY;  // second iterate: a thread each
  // residual; the boundary faces behind the tile read one site more (0) above
  constexpr int RX = TX + 3, RY = TY + 3, RN = RX * RY;
  constexpr int F = EN - WN;  // frame of the first iterate
  static_assert(WN <= NT && F <= NT, "a thread per column");
  __shared__ T X1[3][3 * EN];
  __shared__ T X2[3][3 * WN];
  __shared__ T R[5][3 * RN];
  if (st && st->done) return;
  const Grid& Gc = L.gc;
  const int n2 = G.n[2];
  const Where tile = my_tile();
  const int ti = tile.x * TX, tj = tile.y * TY, k0 = tile.z * tz, k1 = min(k0 + tz, n2);
  const int e = threadIdx.x;
  const int y = e / WX - 2, x = e - (y + 2) * WX - 2;  // site of the tile
  const bool live = e < WN;
  const Column<T> q = make_column<T>(G, live, ti + x, tj + y);
  const Owner<TL, T> own(G, live, x, y, ti + x, tj + y);
  const bool res_on = live && x >= -1 && x <= TX && y >= -1 && y <= TY;
  const int c1 = (y + 3) * EX + x + 3, c2 = (y + 2) * WX + x + 2, cr = (y + 1) * RX + x + 1;
  // the frame site of this thread (the first waves only)
  const bool frw = __builtin_amdgcn_readfirstlane(e) < F;
  const int fe = e < 2 * EX ? e : e - 2 * EX;
  const int fx = e < EX ? e : (e < 2 * EX ? e - EX : (fe & 1 ? EX - 1 : 0));
  const int fy = e < EX ? 0 : (e < 2 * EX ? EY - 1 : 1 + (fe >> 1));
  const bool fr = e < F;
  const Column<T> qf = make_column<T>(G, fr, ti - 3 + fx, tj - 3 + fy);
  const bool special = special_block(G, ti - 4, ti + TX + 4, tj - 4, tj + TY + 4, k0 - 4, k1 + 4);
  const T om = L.omega / L.op.ih2, eta = L.op.eta, ih2 = L.op.ih2;
  const __amdgpu_buffer_rsrc_t rb = buf_rsrc(b, G.bytes), rx = buf_rsrc(xo, G.bytes);
  const Tri<T> zero{T(0), T(0), T(0)};
  const Diag<T> dq = make_diag(G, q, eta, om, -1), df = make_diag(G, qf, eta, om, -1);
  // A plane's registers and LDS slot are those of its number mod 3 (the loop is
  // unrolled by three): the first iterate on planes t - 3 .. t - 1, the second
  // on t - 5 .. t - 3, and the loads, three planes ahead of their use.
  Tri<T> xs[3] = {zero, zero, zero}, ys[3] = {zero, zero, zero};
  Tri<T> bn[3], fb[3], br[3];
  T d1 = T(0), d2 = T(0);
  const int t0 = k0 - 3;  // odd
  for (int z = e; z < 5 * 3 * RN; z += NT) (&R[0][0])[z] = T(0);
#pragma unroll
  for (int h = 0; h < 3; ++h) {
    const Plane p = make_plane<T>(G, t0 + h);
    bn[h] = load_faces(rb, q, p);
    fb[h] = load_faces(rb, qf, p);
    br[(h + 1) % 3] = load_faces(rb, q, make_plane<T>(G, k0 - 2 + h));
  }
  __syncthreads();
  int rs = 0;  // slot of the residual's plane t - 4 (mod 5)
  auto step = [&](int t, auto phase) {
    constexpr int P0 = decltype(phase)::value, P1 = (P0 + 2) % 3, P2 = (P0 + 1) % 3;
    // first sweep from a zero guess on plane t
    Tri<T> x0 = zero;
    if (t <= k1 + 2) {
      const Plane pn = make_plane<T>(G, t);
      Tri<T> s0 = dq.sc;
      if (!bulk_plane(G, t)) s0 = make_diag(G, q, eta, om, max(t, 0)).sc;
      x0 = masked(q, pn, s0.u * bn[P0].u, s0.v * bn[P0].v, s0.w * bn[P0].w);
      T* const X = X1[P0];
      if (live) X[c1] = x0.u, X[c1 + EN] = x0.v, X[c1 + 2 * EN] = x0.w;
      const Plane pl = make_plane<T>(G, t + 3);
      bn[P0] = load_faces(rb, q, pl);
      if (frw) {
        Tri<T> g0 = df.sc;
        if (!bulk_plane(G, t)) g0 = make_diag(G, qf, eta, om, max(t, 0)).sc;
        const Tri<T> f = masked(qf, pn, g0.u * fb[P0].u, g0.v * fb[P0].v, g0.w * fb[P0].w);
        const int cf = fy * EX + fx;
        if (fr) X[cf] = f.u, X[cf + EN] = f.v, X[cf + 2 * EN] = f.w;
        fb[P0] = load_faces(rb, qf, pl);
      }
    }
    // second sweep on plane t - 2 (on plane k0 - 3 only for the divergence):
    // x2 = x1 + omega / D (b - M x1), and omega / D b is x1
    Tri<T> y0 = zero;
    if (t - 2 >= k0 - 3 && t - 2 <= k1 + 1) {
      const int k = t - 2;
      Diag<T> d = dq;
      if (!bulk_plane(G, k)) d = make_diag(G, q, eta, om, max(k, 0));
      if (live) {
        const Tri<T> xC = xs[P2];
        const Tri<T> m = march_row<T, EX, EN>(G, eta, q, special, X1[P2] + c1, X1[P1] + c1 + 2 * EN,
                                              xs[P0], xC, xs[P1], d1, k, d.vd);
        y0 = masked(q, make_plane<T>(G, k), T(2) * xC.u - d.sc.u * ih2 * m.u,
                    T(2) * xC.v - d.sc.v * ih2 * m.v, T(2) * xC.w - d.sc.w * ih2 * m.w);
        T* const Q = X2[P2];
        Q[c2] = y0.u, Q[c2 + WN] = y0.v, Q[c2 + 2 * WN] = y0.w;
        own.store(G, q, rx, k, k0, k1, y0);
      }
    }
    // residual on plane t - 4 (on plane k0 - 2 only for the divergence)
    if (t - 4 >= k0 - 2) {
      const int k = t - 4;
      Tri<T> vd = dq.vd;
      if (!bulk_plane(G, k)) vd = make_diag(G, q, eta, om, max(k, 0)).vd;
      if (res_on) {
        Tri<T> r = zero;
        if (k <= k1) {  // uniform; planes above are 0 (behind the grid)
          const Tri<T> m = march_row<T, WX, WN>(G, eta, q, special, X2[P1] + c2,
                                                X2[P0] + c2 + 2 * WN, ys[P2], ys[P1], ys[P0], d2, k,
                                                vd);
          r = masked(q, make_plane<T>(G, k), br[P1].u - ih2 * m.u, br[P1].v - ih2 * m.v,
                     br[P1].w - ih2 * m.w);
        }
        T* const Q = R[rs];
        Q[cr] = r.u, Q[cr + RN] = r.v, Q[cr + 2 * RN] = r.w;
      }
      br[P1] = load_faces(rb, q, make_plane<T>(G, k + 3));
    }
    // restriction to coarse plane K from residual planes 2K - 1 .. 2K + 2 = t - 5
    if (t & 1) {
      const int K = (t - 7) >> 1;
      if (K >= k0 / 2 && (K < k1 / 2 || (k1 == n2 && K == k1 / 2))) {
        constexpr int CX = TX / 2 + 1, CY = TY / 2 + 1, CT = (CX * CY + 63) / 64 * 64;
        static_assert(3 * CT <= NT, "waves per component");
        const int c = __builtin_amdgcn_readfirstlane(e) / CT, ce = e - c * CT;
        if (c < 3 && ce < CX * CY) {
          const int cy = ce / CX, cx = ce - cy * CX;
          const int I = ti / 2 + cx, J = tj / 2 + cy;
          const bool mine = cx < TX / 2 + int(c == 0 && I == Gc.n[0]) &&
                            cy < TY / 2 + int(c == 1 && J == Gc.n[1]) &&
                            (K < k1 / 2 || c == 2) && in_array(Gc, c, I, J, K);
          if (mine) {
            const T* r[4];
#pragma unroll
            for (int z = 0; z < 4; ++z) {
              const int sl = rs + 1 + z;  // plane t - 8 + z
              r[z] = R[sl >= 5 ? sl - 5 : sl] + c * RN + (2 * cy + 1) * RX + 2 * cx + 1;
            }
            const int f = face(Gc, c, I, J, K);
            T v = T(0);
            if ((unknown_bits<3>(Gc, I, J, K) >> c) & 1u)
              v = c == 0   ? march_restrict<T, 0, RX, SMOOTH>(Gc, r, I, J, K)
                  : c == 1 ? march_restrict<T, 1, RX, SMOOTH>(Gc, r, I, J, K)
                           : march_restrict<T, 2, RX, SMOOTH>(Gc, r, I, J, K);
            bc[f] = v;
            if (x0c) x0c[f] = omega_c * dinv_c[f] * v;
          }
        }
      }
    }
    xs[P0] = x0;
    ys[P2] = y0;
    rs = rs == 4 ? 0 : rs + 1;
    __syncthreads();
  };
  // the last coarse plane wants residual planes up to 2K + 2 <= k1, and the
  // boundary plane behind the grid two more; steps beyond do nothing
  const int t1 = k1 + 5 + (k1 == n2 ? 2 : 0);
  for (int t = t0; t <= t1; t += 3) {
    step(t, std::integral_constant<int, 0>{});
    step(t + 1, std::integral_constant<int, 1>{});
    step(t + 2, std::integral_constant<int, 2>{});
  }
}

// --------------------------------------------------------------- way up

// The coarse correction at a column, interpolated along x and y on one coarse
// plane: NC values per component with fixed offsets and weights (0 where the
// coarse face is no unknown), loaded first (in flight during a step), then
// summed.
template <typename T, int NC>
struct CoarseCol {
  unsigned o[3][NC];
  T w[3][NC];
};
template <typename T, int NC>
struct CoarseRaw {
  T v[3][NC];
};
// NC = 2: constant across the fine cells (w: one value, the second unused);
// NC = 4: also the neighbouring row, weights of cover_weight
template <typename T, int NC>
__device__ __forceinline__ CoarseCol<T, NC> make_coarse_col(const Grid& Gc, bool live, int i, int j) {
  CoarseCol<T, NC> c;
  const int I = i >> 1, J = j >> 1, dx = i & 1 ? 1 : -1, dy = j & 1 ? 1 : -1;
  const T wx = cover_weight<T>(i, Gc.n[0], Gc.bc[0], Gc.bc[1]),
          wy = cover_weight<T>(j, Gc.n[1], Gc.bc[2], Gc.bc[3]);
  auto put = [&](int a, int q, int II, int JJ, T w) {
    const bool ci = unsigned(II) < unsigned(Gc.n[0]), cj = unsigned(JJ) < unsigned(Gc.n[1]);
    const int lx = Gc.bc[0] == kDir ? 1 : 0, hx = Gc.n[0] - (Gc.bc[1] == kDir ? 1 : 0);
    const int ly = Gc.bc[2] == kDir ? 1 : 0, hy = Gc.n[1] - (Gc.bc[3] == kDir ? 1 : 0);
    const bool on = live && (a == 0 ? cj && II >= lx && II <= hx
                                    : a == 1 ? ci && JJ >= ly && JJ <= hy : ci && cj) && w != T(0);
    c.o[a][q] = (on ? unsigned(face(Gc, a, II, JJ, 0)) : 0u) * unsigned(sizeof(T));
    c.w[a][q] = on ? w : T(0);
  };
  const bool oi = i & 1, oj = j & 1;
  const T n0 = oi ? T(0.5) : T(1), n1 = oi ? T(0.5) : T(0);  // along x for u
  const T m0 = oj ? T(0.5) : T(1), m1 = oj ? T(0.5) : T(0);  // along y for v
  if constexpr (NC == 2) {
    put(0, 0, I, J, n0), put(0, 1, I + 1, J, n1);
    put(1, 0, I, J, m0), put(1, 1, I, J + 1, m1);
    put(2, 0, I, J, T(1)), put(2, 1, I, J, T(0));
  } else {
    const T q = T(0.25);
    put(0, 0, I, J, n0 * wy), put(0, 1, I + 1, J, n1 * wy);
    put(0, 2, I, J + dy, n0 * q), put(0, 3, I + 1, J + dy, n1 * q);
    put(1, 0, I, J, m0 * wx), put(1, 1, I, J + 1, m1 * wx);
    put(1, 2, I + dx, J, m0 * q), put(1, 3, I + dx, J + 1, m1 * q);
    put(2, 0, I, J, wx * wy), put(2, 1, I + dx, J, q * wy);
    put(2, 2, I, J + dy, wx * q), put(2, 3, I + dx, J + dy, q * q);
  }
  return c;
}
template <typename T, int NC>
__device__ __forceinline__ void load_coarse(const Grid& Gc, __amdgpu_buffer_rsrc_t ec,
                                            const CoarseCol<T, NC>& c, int K, CoarseRaw<T, NC>& r) {
  const int Kc = min(max(K, 0), Gc.n[2] - 1), Kw = min(max(K, 0), Gc.n[2]);
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const unsigned s = unsigned((a == 2 ? Kw : Kc) * Gc.ext[a][0] * Gc.ext[a][1]) * unsigned(sizeof(T));
#pragma unroll
    for (int q = 0; q < (NC == 2 && a == 2 ? 1 : NC); ++q) r.v[a][q] = buf_load<T>(ec, c.o[a][q], s);
  }
}
template <typename T, int NC>
__device__ __forceinline__ Tri<T> sum_coarse(const Grid& Gc, const CoarseCol<T, NC>& c, int K,
                                             const CoarseRaw<T, NC>& r) {
  const bool cell = unsigned(K) < unsigned(Gc.n[2]);
  const bool nrm = K >= (Gc.bc[4] == kDir ? 1 : 0) && K <= Gc.n[2] - (Gc.bc[5] == kDir ? 1 : 0);
  T s[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    s[a] = c.w[a][0] * r.v[a][0];
#pragma unroll
    for (int q = 1; q < (NC == 2 && a == 2 ? 1 : NC); ++q) s[a] += c.w[a][q] * r.v[a][q];
  }
  return {cell ? s[0] : T(0), cell ? s[1] : T(0), nrm ? s[2] : T(0)};
}

template <typename T, class TL, bool SMOOTH>
__global__ __launch_bounds__(TL::NT) void k_march_up(LegLevel<T> L, Geo G, const T* __restrict__ ec,
                                                     const T* __restrict__ xi,
                                                     const T* __restrict__ b, T* __restrict__ xo,
                                                     double* __restrict__ partial,
                                                     const PcgState* __restrict__ st, int tz) {
  constexpr int TX = TL::TX, TY = TL::TY, NT = TL::NT, NC = SMOOTH ? 4 : 2;
  constexpr int WX = TX + 4, WY = TY + 4, WN = WX * WY;  // corrected iterate: a thread each
  constexpr int RX = TX + 3, RY = TY + 3, RN = RX * RY;  // after the first sweep
  static_assert(WN <= NT, "a thread per column");
  __shared__ T X0[3][3 * WN];
  __shared__ T Y[3][3 * RN];
  if (st && st->done) return;
  const Grid& Gc = L.gc;
  const int n2 = G.n[2];
  const Where tile = my_tile();
  const int ti = tile.x * TX, tj = tile.y * TY, k0 = tile.z * tz, k1 = min(k0 + tz, n2);
  const int e = threadIdx.x;
  const int y = e / WX - 2, x = e - (y + 2) * WX - 2;
  const bool live = e < WN;
  const Column<T> q = make_column<T>(G, live, ti + x, tj + y);
  const Owner<TL, T> own(G, live, x, y, ti + x, tj + y);
  // the boundary faces behind the tile read one site more (0) above
  const bool mid_on = live && x >= -1 && x <= TX && y >= -1 && y <= TY;
  const bool out_on = live && (own.u || own.v || own.w);
  const int c0 = (y + 2) * WX + x + 2, c1 = (y + 1) * RX + x + 1;
  const bool special = special_block(G, ti - 3, ti + TX + 3, tj - 3, tj + TY + 3, k0 - 3, k1 + 3);
  const T om = L.omega / L.op.ih2, eta = L.op.eta, ih2 = L.op.ih2;
  const __amdgpu_buffer_rsrc_t rb = buf_rsrc(b, G.bytes), rx = buf_rsrc(xi, G.bytes),
                               ro = buf_rsrc(xo, G.bytes),
                               re = buf_rsrc(ec, unsigned(Gc.m_full) * unsigned(sizeof(T)));
  const Tri<T> zero{T(0), T(0), T(0)};
  for (int z = e; z < 3 * 3 * RN; z += NT) (&Y[0][0])[z] = T(0);
  const CoarseCol<T, NC> cc = make_coarse_col<T, NC>(Gc, live, ti + x, tj + y);
  CoarseRaw<T, NC> raw;
  Tri<T> eB = zero, eC, eA = zero;  // coarse planes K - 1, K, K + 1 for fine planes 2K, 2K + 1
  const int t0 = k0 - 2;            // even
  if (SMOOTH) {
    load_coarse(Gc, re, cc, (t0 >> 1) - 1, raw);
    eB = sum_coarse(Gc, cc, (t0 >> 1) - 1, raw);
  }
  load_coarse(Gc, re, cc, t0 >> 1, raw);
  eC = sum_coarse(Gc, cc, t0 >> 1, raw);
  const Diag<T> dq = make_diag(G, q, eta, om, -1);
  // as on the way down: registers and slots by plane mod 3, the loads of a
  // step together, three planes ahead (the coarse planes one, two steps);
  // corrected iterate on planes t - 3 .. t - 1, after the first sweep on t - 5 ..
  // t - 3
  Tri<T> xs[3] = {zero, zero, zero}, ys[3] = {zero, zero, zero};
  Tri<T> xn[3], b1[3], b2[3];
  T d1 = T(0), d2 = T(0);
  load_coarse(Gc, re, cc, (t0 >> 1) + 1, raw);
#pragma unroll
  for (int h = 0; h < 3; ++h) {
    xn[h] = load_faces(rx, q, make_plane<T>(G, t0 + h));
    b1[(h + 1) % 3] = load_faces(rb, q, make_plane<T>(G, t0 - 2 + h));
    b2[(h + 2) % 3] = load_faces(rb, q, make_plane<T>(G, t0 - 4 + h));
  }
  double part = 0.0;
  __syncthreads();
  auto step = [&](int t, auto phase) {
    constexpr int H = decltype(phase)::value, P0 = H % 3, P1 = (H + 2) % 3, P2 = (H + 1) % 3;
    // x + P e on plane t
    Tri<T> p, x0 = zero;
    if constexpr (H % 2 == 0) {
      p = eC;
      if (SMOOTH) {
        const T w = cover_weight<T>(t, Gc.n[2], Gc.bc[4], Gc.bc[5]);
        p.u = w * eC.u + T(0.25) * eB.u;
        p.v = w * eC.v + T(0.25) * eB.v;
      }
      eA = sum_coarse(Gc, cc, (t >> 1) + 1, raw);
    } else {
      p = {eC.u, eC.v, T(0.5) * (eC.w + eA.w)};
      if (SMOOTH) {
        const T w = cover_weight<T>(t, Gc.n[2], Gc.bc[4], Gc.bc[5]);
        p.u = w * eC.u + T(0.25) * eA.u;
        p.v = w * eC.v + T(0.25) * eA.v;
      }
      eB = eC, eC = eA;
    }
    if (t <= k1 + 1) {
      x0 = masked(q, make_plane<T>(G, t), xn[P0].u + p.u, xn[P0].v + p.v, xn[P0].w + p.w);
      if (live) {
        T* const X = X0[P0];
        X[c0] = x0.u, X[c0 + WN] = x0.v, X[c0 + 2 * WN] = x0.w;
      }
    }
    // first sweep on plane t - 2 (on plane k0 - 2 only for the divergence)
    Tri<T> y0 = zero;
    if (t - 2 >= k0 - 2 && t - 2 <= k1) {
      const int k = t - 2;
      Diag<T> d = dq;
      if (!bulk_plane(G, k)) d = make_diag(G, q, eta, om, max(k, 0));
      if (mid_on) {
        const Tri<T> xC = xs[P2], bb = b1[P2];
        const Tri<T> m = march_row<T, WX, WN>(G, eta, q, special, X0[P2] + c0, X0[P1] + c0 + 2 * WN,
                                              xs[P0], xC, xs[P1], d1, k, d.vd);
        y0 = masked(q, make_plane<T>(G, k), xC.u + d.sc.u * (bb.u - ih2 * m.u),
                    xC.v + d.sc.v * (bb.v - ih2 * m.v), xC.w + d.sc.w * (bb.w - ih2 * m.w));
        T* const Q = Y[P2];
        Q[c1] = y0.u, Q[c1 + RN] = y0.v, Q[c1 + 2 * RN] = y0.w;
      }
    }
    // second sweep on plane t - 4 (on plane k0 - 1 only for the divergence)
    if (t - 4 >= k0 - 1 && t - 4 <= k1) {
      const int k = t - 4;
      Diag<T> d = dq;
      if (!bulk_plane(G, k)) d = make_diag(G, q, eta, om, max(k, 0));
      if (out_on) {
        const Plane pk = make_plane<T>(G, k);
        const Tri<T> yC = ys[P1], bb = masked(q, pk, b2[P1].u, b2[P1].v, b2[P1].w);
        const Tri<T> m = march_row<T, RX, RN>(G, eta, q, special, Y[P1] + c1, Y[P0] + c1 + 2 * RN,
                                              ys[P2], yC, ys[P0], d2, k, d.vd);
        const Tri<T> r = masked(q, pk, yC.u + d.sc.u * (bb.u - ih2 * m.u),
                                yC.v + d.sc.v * (bb.v - ih2 * m.v),
                                yC.w + d.sc.w * (bb.w - ih2 * m.w));
        own.store(G, q, ro, k, k0, k1, r);
        if (k >= k0 && k < k1 + int(k1 == n2)) {
          if (own.u && k < k1) part += double(bb.u) * double(r.u);
          if (own.v && k < k1) part += double(bb.v) * double(r.v);
          if (own.w) part += double(bb.w) * double(r.w);
        }
      }
    }
    xs[P0] = x0;
    ys[P2] = y0;
    if constexpr (H % 2 == 0) load_coarse(Gc, re, cc, (t >> 1) + 2, raw);
    xn[P0] = load_faces(rx, q, make_plane<T>(G, t + 3));
    b1[P2] = load_faces(rb, q, make_plane<T>(G, t + 1));
    b2[P1] = load_faces(rb, q, make_plane<T>(G, t - 1));
    __syncthreads();
  };
  const int t1 = k1 + 3 + (k1 == n2 ? 1 : 0);  // steps beyond do nothing
  for (int t = t0; t <= t1; t += 6) {
    step(t, std::integral_constant<int, 0>{});
    step(t + 1, std::integral_constant<int, 1>{});
    step(t + 2, std::integral_constant<int, 2>{});
    if (t + 3 > t1) break;  // uniform
    step(t + 3, std::integral_constant<int, 3>{});
    step(t + 4, std::integral_constant<int, 4>{});
    step(t + 5, std::integral_constant<int, 5>{});
  }
  if (partial) {
    __shared__ double sh[NT / 64];
    const double s = block_sum<NT>(part, sh);
    if (threadIdx.x == 0) partial[tile.lin] = s;
  }
}

typedef MTile<32, 16, 768> MWide;
typedef MTile<16, 16, 448> MSquare;

template <class TL>
LegPlan plan_march(const Grid& g, int id) {
  const int gx = (g.n[0] + TL::TX - 1) / TL::TX, gy = (g.n[1] + TL::TY - 1) / TL::TY;
  LegPlan p;
  p.tile = id;
  p.tz = march_planes(gx * gy, g.n[2]);
  p.grid = dim3(gx, gy, (g.n[2] + p.tz - 1) / p.tz);
  p.nblocks = p.grid.x * p.grid.y * p.grid.z;
  return p;
}

}  // namespace

// Which levels march (constant viscosity, Jacobi; those small enough for the
// box legs take these).  One V(2,2) cycle in us, separate kernels / march on
// all levels above 40^3 cells:
//                   SMOOTH FP64  SMOOTH FP32   DIV FP64   DIV FP32
//   64 x 64 x 64      133 / 131    119 / 124   119 / 123  107 / 116
//   80 x 64 x 72      177 / 150    156 / 134   163 / 138  132 / 125
//   96 x 80 x 112     237 / 214    198 / 175   215 / 192  169 / 158
//   128 x 128 x 128   346 / 318    251 / 235   278 / 284  195 / 218
//   144 x 112 x 96    333 / 274    265 / 223   270 / 248  199 / 208
//   192 x 192 x 96    556 / 507    351 / 322
//   160 x 160 x 32    216 / 219    173 / 167   205 / 199
//   32 x 160 x 160    239 / 208    183 / 171   232 / 187
//   128 x 16 x 128    134 / 130    117 / 124
//   16 x 128 x 128    167 / 131    147 / 129
//   248 x 32 x 32     141 / 129    127 / 123   123 / 121
//   240 x 64 x 64     218 / 224    182 / 171   190 / 204
//   120 x 64 x 64     160 / 167    142 / 141   149 / 151
//   160 x 160 x 160                            543 / 454
//   240 x 128 x 128                            473 / 448
// With the SMOOTH transfers, whose interpolation the tiled stencil does not
// take along, always: 0.95 to 1.28 times as fast, the more the larger the grid.
// With DIV in FP64 where the width is no multiple of the 64 cells wide tiles of
// the separate kernels, whose last one then leaves lanes idle; with few of them
// idle (120, 240, 248) the two are even on average.  In FP32 the sign
// changes with the size.
LegPlan march_plan(const Grid& g, int elem, bool smooth) {
  // 32-bit byte offsets
  if (g.dim != 3 || (long)g.m_full * elem >= (1L << 31)) return LegPlan();
  if (!smooth && (elem == 4 || g.n[0] % 64 == 0)) return LegPlan();
  return elem == 8 ? plan_march<MSquare>(g, kMarchSquare) : plan_march<MWide>(g, kMarchWide);
}

template <typename T>
void march_down(hipStream_t s, const LegPlan& p, const LegLevel<T>& L, const T* b, T* xo, T* bc,
                const T* dinv_c, T omega_c, T* x0c, const PcgState* st) {
  typedef typename std::conditional<sizeof(T) == 8, MSquare, MWide>::type TL;
  auto go = [&](auto kernel) {
    kernel<<<p.grid, TL::NT, 0, s>>>(L, make_geo(L.op.g, sizeof(T)), b, xo, bc, dinv_c, omega_c, x0c,
                                     st, p.tz);
  };
  if (L.smooth) go(k_march_down<T, TL, true>);
  else if constexpr (sizeof(T) == 8) go(k_march_down<T, TL, false>);
}

template <typename T>
void march_up(hipStream_t s, const LegPlan& p, const LegLevel<T>& L, const T* ec, const T* xi,
              const T* b, T* xo, double* partial, const PcgState* st) {
  typedef typename std::conditional<sizeof(T) == 8, MSquare, MWide>::type TL;
  auto go = [&](auto kernel) {
    kernel<<<p.grid, TL::NT, 0, s>>>(L, make_geo(L.op.g, sizeof(T)), ec, xi, b, xo, partial, st, p.tz);
  };
  if (L.smooth) go(k_march_up<T, TL, true>);
  else if constexpr (sizeof(T) == 8) go(k_march_up<T, TL, false>);
}

template void march_down<float>(hipStream_t, const LegPlan&, const LegLevel<float>&, const float*,
                                float*, float*, const float*, float, float*, const PcgState*);
template void march_down<double>(hipStream_t, const LegPlan&, const LegLevel<double>&,
                                 const double*, double*, double*, const double*, double, double*,
                                 const PcgState*);
template void march_up<float>(hipStream_t, const LegPlan&, const LegLevel<float>&, const float*,
                              const float*, const float*, float*, double*, const PcgState*);
template void march_up<double>(hipStream_t, const LegPlan&, const LegLevel<double>&, const double*,
                               const double*, const double*, double*, double*, const PcgState*);

}  // namespace gkb

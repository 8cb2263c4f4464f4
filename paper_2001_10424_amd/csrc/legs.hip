// Fused V-cycle legs (see legs.hpp).
//
// A block owns a box of fine cells and works on it plus a halo as deep as the
// chain of operators needs, recomputing the halo instead of exchanging it, so
// that a leg has no launch boundary inside.  All intermediate iterates live
// in LDS; b, 1/D and the viscosity are read from memory (the caches serve the
// repeats).  This trades arithmetic for round trips: on the levels below
// about 64^3 (3D) and on all 2D levels a single operator application is
// bound by its launch and one dependent read of memory (4-6 us whatever its
// size), while the chip has arithmetic to spare.
//
// Site s = (x, y, z) of the box is the cell (i, j, k) = origin - halo + s and
// carries its lower faces u, v[, w]; the upper boundary faces of the grid are
// sites one past the last cell.  Sites that are no unknown hold 0.
#include "legsites.hpp"

namespace gkb {
namespace {

template <int DIM_, int X, int Y, int Z, int NT_>
struct Tile {
  static constexpr int DIM = DIM_, TX = X, TY = Y, TZ = Z, NT = NT_;
};

// LDS box of a tile with halo H below and HU above
template <class TL, int H_, int HU = H_>
struct Box {
  static constexpr int H = H_, DIM = TL::DIM;
  static constexpr int EX = TL::TX + H + HU, EY = TL::TY + H + HU,
                       EZ = DIM == 3 ? TL::TZ + H + HU : 1;
  static constexpr int N = EX * EY * EZ;
  static constexpr int SY = EX, SZ = EX * EY;
};

// The sites LO <= x < EX - HI (same in y, z) of a box, spread over the
// block's threads: PER of them each, get(q) the q-th (false: none left).
// Loops over them unroll, so the loads of a thread's sites are in flight
// together.
template <class TL, class B, int LO, int HI>
struct Sites {
  static constexpr int NX = B::EX - LO - HI, NY = B::EY - LO - HI,
                       NZ = B::DIM == 3 ? B::EZ - LO - HI : 1;
  static constexpr int COUNT = NX * NY * NZ;
  static constexpr int PER = (COUNT + TL::NT - 1) / TL::NT;
  int s, x, y, z;
  __device__ __forceinline__ bool get(int q) {
    const int e = threadIdx.x + q * TL::NT;
    const int r = e / NX;
    x = e - r * NX + LO;
    y = (B::DIM == 3 ? r % NY : r) + LO;
    z = B::DIM == 3 ? r / NY + LO : 0;
    s = (z * B::EY + y) * B::EX + x;
    return e < COUNT;
  }
};

// What a block needs to know about the boundary: per axis and site the
// diagonal weight of the tangential viscous couplings for unit viscosity (a
// neighbour counts 1, a wall 2, a do-nothing side 0), and whether cells can
// need masking.  At DIRICHLET sides they cannot: every face of a cell outside
// is 0 and so is its divergence.
template <typename T, class B>
struct Edges {
  T w[3][B::EX > B::EY ? (B::EX > B::EZ ? B::EX : B::EZ) : (B::EY > B::EZ ? B::EY : B::EZ)];
};
template <typename T, class TL, class B>
__device__ __forceinline__ bool fill_edges(const Grid& G, Edges<T, B>& E, int i0, int j0, int k0) {
  const int o[3] = {i0, j0, k0};
  constexpr int ext[3] = {B::EX, B::EY, B::EZ};
#pragma unroll
  for (int a = 0; a < B::DIM; ++a)
    for (int l = threadIdx.x; l < ext[a]; l += TL::NT) {
      T v = T(2);
      if (o[a] + l == 0) v += G.bc[2 * a] == kDir ? T(1) : T(-1);
      if (o[a] + l == G.n[a] - 1) v += G.bc[2 * a + 1] == kDir ? T(1) : T(-1);
      E.w[a][l] = v;
    }
  bool special = false;  // uniform
#pragma unroll
  for (int a = 0; a < 2 * B::DIM; ++a) special |= G.bc[a] != kDir;
  if (G.pin >= 0) {
    const int nxy = G.n[0] * G.n[1], pk = G.pin / nxy, pj = (G.pin - pk * nxy) / G.n[0],
              pi = G.pin - pk * nxy - pj * G.n[0];
    special |= unsigned(pi - i0) < unsigned(B::EX) && unsigned(pj - j0) < unsigned(B::EY) &&
               (B::DIM == 2 || unsigned(pk - k0) < unsigned(B::EZ));
  }
  return special;
}

// one side of the viscous stencil along a tangential axis: the neighbour at
// index q (0 in LDS when outside), its edge viscosity kap, side type bc
template <typename T>
__device__ __forceinline__ T side(bool in, bool wall, T kap, T xc, T xn) {
  return in ? kap * (xc - xn) : (wall ? T(2) * kap * xc : T(0));
}

// rows of M x at the faces of site t = (i, j, k); x: DIM components of N
// sites in LDS, 0 where no unknown.  Results at faces that are no unknown are
// meaningless.
template <typename T, bool VARMU, class B, class S>
__device__ __forceinline__ void row_M(const Op<T>& op, const Edges<T, B>& E, bool special,
                                      const T* x, const S& t, int i, int j, int k, T* m) {
  const Grid& G = op.g;
  constexpr int DIM = B::DIM, N = B::N, SX = 1, SY = B::SY, SZ = B::SZ;
  const int s = t.s;
  const int n0 = G.n[0], n1 = G.n[1], n2 = G.n[2];
  const T* U = x;
  const T* V = x + N;
  const T* W = x + 2 * N;
  const T uC = U[s], vC = V[s];
  const T uE = U[s + SX], uW = U[s - SX], uN = U[s + SY], uS = U[s - SY];
  const T vE = V[s + SX], vW = V[s - SX], vN = V[s + SY], vS = V[s - SY];
  // divergences of the cell and of its lower neighbours
  T dC = (uC - uE) + (vC - vN);
  T dW = (uW - uC) + (vW - V[s - SX + SY]);
  T dS = (uS - U[s - SY + SX]) + (vS - vC);
  T dB = T(0), wC = T(0), wE = T(0), wW = T(0), wN = T(0), wS = T(0), wT = T(0), wB = T(0);
  T uT = T(0), uB = T(0), vT = T(0), vB = T(0);
  if constexpr (DIM == 3) {
    wC = W[s], wE = W[s + SX], wW = W[s - SX], wN = W[s + SY], wS = W[s - SY];
    wT = W[s + SZ], wB = W[s - SZ];
    uT = U[s + SZ], uB = U[s - SZ], vT = V[s + SZ], vB = V[s - SZ];
    dC += wC - wT;
    dW += wW - W[s - SX + SZ];
    dS += wS - W[s - SY + SZ];
    dB = (uB - U[s - SZ + SX]) + (vB - V[s - SZ + SY]) + (wB - wC);
  }
  T hu = T(1), hv = T(1), hw = T(1);   // half control volumes at do-nothing sides
  T nu = T(2), nv = T(2), nw = T(2);   // normal couplings
  if (special) {  // uniform
    dC = cell_on(G, i, j, k) ? dC : T(0);
    dW = cell_on(G, i - 1, j, k) ? dW : T(0);
    dS = cell_on(G, i, j - 1, k) ? dS : T(0);
    if (i == 0 || i == n0) hu = T(0.5), nu = T(1);
    if (j == 0 || j == n1) hv = T(0.5), nv = T(1);
    if constexpr (DIM == 3) {
      dB = cell_on(G, i, j, k - 1) ? dB : T(0);
      if (k == 0 || k == n2) hw = T(0.5), nw = T(1);
    }
  }
  if constexpr (!VARMU) {
    // unit viscosity: the neighbours outside are 0, so only the diagonal
    // depends on the boundary
    const T cx = E.w[0][t.x], cy = E.w[1][t.y], cz = DIM == 3 ? E.w[2][t.z] : T(0);
    m[0] = (nu + hu * (cy + cz)) * uC - ((uW + uE) + hu * ((uS + uN) + (uB + uT)));
    m[1] = (nv + hv * (cx + cz)) * vC - ((vS + vN) + hv * ((vW + vE) + (vB + vT)));
    if constexpr (DIM == 3)
      m[2] = (nw + hw * (cx + cy)) * wC - ((wB + wT) + hw * ((wW + wE) + (wS + wN)));
  } else {
    const bool lx = G.bc[0] == kDir, rx = G.bc[1] == kDir, ly = G.bc[2] == kDir,
               ry = G.bc[3] == kDir, lz = G.bc[4] == kDir, rz = G.bc[5] == kDir;
    // clamped indices keep every load inside; sites outside the grid are
    // discarded by the caller
    const int ic = min(max(i, 0), n0 - 1), jc = min(max(j, 0), n1 - 1), kc = min(max(k, 0), n2 - 1);
    const int iv = min(max(i, 0), n0), jv = min(max(j, 0), n1), kv = min(max(k, 0), n2);
    const T mC = op.mu[cidx(G, ic, jc, kc)];
    const T mW = op.mu[cidx(G, max(ic - 1, 0), jc, kc)];
    const T mS = op.mu[cidx(G, ic, max(jc - 1, 0), kc)];
    const bool iW = i > 0, iE = i < n0 - 1, jS = j > 0, jN = j < n1 - 1, kB = k > 0, kT = k < n2 - 1;
    // edge along B between the corners: vertex coordinates 0 .. n
    const T ez = edge_mu<2>(op, iv, jv, kc), ezN = edge_mu<2>(op, iv, min(jv + 1, n1), kc),
            ezE = edge_mu<2>(op, min(iv + 1, n0), jv, kc);
    T mu0 = side(jS, ly, ez, uC, uS) + side(jN, ry, ezN, uC, uN);
    T mv0 = side(iW, lx, ez, vC, vW) + side(iE, rx, ezE, vC, vE);
    // normal couplings; at a do-nothing side the face has one cell only
    T mw1 = T(0);
    if constexpr (DIM == 3) {
      const T ey = edge_mu<1>(op, iv, jc, kv), eyT = edge_mu<1>(op, iv, jc, min(kv + 1, n2)),
              eyE = edge_mu<1>(op, min(iv + 1, n0), jc, kv);
      const T ex = edge_mu<0>(op, ic, jv, kv), exT = edge_mu<0>(op, ic, jv, min(kv + 1, n2)),
              exN = edge_mu<0>(op, ic, min(jv + 1, n1), kv);
      const T mB = op.mu[cidx(G, ic, jc, max(kc - 1, 0))];
      mu0 += side(kB, lz, ey, uC, uB) + side(kT, rz, eyT, uC, uT);
      mv0 += side(kB, lz, ex, vC, vB) + side(kT, rz, exT, vC, vT);
      const T mw0 = side(iW, lx, ey, wC, wW) + side(iE, rx, eyE, wC, wE) +
                    side(jS, ly, ex, wC, wS) + side(jN, ry, exN, wC, wN);
      mw1 = k == n2 ? mC * (wC - wB)
                    : (k == 0 ? T(0) : mB * (wC - wB)) + mC * (wC - wT);
      m[2] = mw1 + hw * mw0;
    }
    m[0] = (i == n0 ? mC * (uC - uW) : (i == 0 ? T(0) : mW * (uC - uW)) + mC * (uC - uE)) + hu * mu0;
    m[1] = (j == n1 ? mC * (vC - vS) : (j == 0 ? T(0) : mS * (vC - vS)) + mC * (vC - vN)) + hv * mv0;
  }
  m[0] = (m[0] + op.eta * (dC - dW)) * op.ih2;
  m[1] = (m[1] + op.eta * (dC - dS)) * op.ih2;
  if constexpr (DIM == 3) m[2] = (m[2] + op.eta * (dC - dB)) * op.ih2;
}

// Face values of a thread's sites, loaded ahead of the stage that uses them:
// the loads are issued together at the start of the kernel (unconditional,
// from the first entry of the array where the face is no unknown), so a leg
// pays one round trip to memory instead of one per stage and site.
template <typename T, class S, int DIM>
struct Ahead {
  T v[S::PER][DIM];
  unsigned on;  // bit q * DIM + c: the face is an unknown
  __device__ __forceinline__ void mask(const Grid& G, int i0, int j0, int k0) {
    static_assert(S::PER * DIM <= 32, "mask bits");
    on = 0;
#pragma unroll
    for (int q = 0; q < S::PER; ++q) {
      S t;
      const bool in = t.get(q);
      const unsigned u = unknown_bits<DIM>(G, i0 + t.x, j0 + t.y, k0 + t.z);
      on |= (in ? u : 0u) << (q * DIM);
    }
  }
  __device__ __forceinline__ bool unk(int q, int c) const { return (on >> (q * DIM + c)) & 1u; }
  __device__ __forceinline__ void load(const Grid& G, const T* __restrict__ a, int i0, int j0,
                                       int k0, unsigned m) {
    on = m;
#pragma unroll
    for (int q = 0; q < S::PER; ++q) {
      S t;
      t.get(q);
#pragma unroll
      for (int c = 0; c < DIM; ++c)
        v[q][c] = a[unk(q, c) ? face(G, c, i0 + t.x, j0 + t.y, k0 + t.z) : 0];
    }
  }
  __device__ __forceinline__ void load(const Grid& G, const T* __restrict__ a, int i0, int j0,
                                       int k0) {
    mask(G, i0, j0, k0);
    load(G, a, i0, j0, k0, on);
  }
};

// r = b - M x on the sites S, 0 where no unknown
template <typename T, bool VARMU, class S, class B>
__device__ __forceinline__ void stage_resid(const Op<T>& op, const T* x,
                                            const Edges<T, B>& E, bool special,
                                            const Ahead<T, S, B::DIM>& b, T* r, int i0, int j0,
                                            int k0) {
#pragma unroll
  for (int q = 0; q < S::PER; ++q) {
    S t;
    if (!t.get(q)) continue;
    T m[3];
    row_M<T, VARMU, B>(op, E, special, x, t, i0 + t.x, j0 + t.y, k0 + t.z, m);
#pragma unroll
    for (int c = 0; c < B::DIM; ++c) r[c * B::N + t.s] = b.unk(q, c) ? b.v[q][c] - m[c] : T(0);
  }
}

// edge component a at (i, j, k) is on the point grid and not in a wall
template <int DIM>
__device__ __forceinline__ bool edge_on(const Grid& G, int a, int i, int j, int k) {
  if (!cell_in(G, i, j, k)) return false;
  const bool wx = i == 0 && G.bc[0] == kDir, wy = j == 0 && G.bc[2] == kDir,
             wz = DIM == 3 && k == 0 && G.bc[4] == kDir;
  if (DIM == 2) return !(wx || wy);
  return a == 0 ? !(wy || wz) : (a == 1 ? !(wx || wz) : !(wx || wy));
}

// omega_e / D_e of a thread's edge sites, loaded ahead; 0 where no edge
template <typename T, class S, int DIM>
struct AheadEdge {
  static constexpr int NE = DIM == 3 ? 3 : 1;
  T v[S::PER][NE];
  __device__ __forceinline__ void load(const LegLevel<T>& L, int i0, int j0, int k0) {
    const Grid& G = L.op.g;
#pragma unroll
    for (int q = 0; q < S::PER; ++q) {
      S t;
      const bool in = t.get(q);
      const int i = i0 + t.x, j = j0 + t.y, k = k0 + t.z;
#pragma unroll
      for (int a = 0; a < NE; ++a) {
        const bool on = in && edge_on<DIM>(G, a, i, j, k);
        const T d = L.edinv[on ? (long)a * G.n_cells + cidx(G, i, j, k) : 0];
        v[q][a] = on ? L.omega_e * d : T(0);
      }
    }
  }
};

// the edge half of the hybrid smoother, in place on x: r = b - M x on the
// sites [1, E - 1), psi = omega_e D_e^-1 C^T r on [2, E - 1), x += C psi on
// [2, E - 2)
template <typename T, bool VARMU, class TL, class B>
__device__ __forceinline__ void stage_edge(const LegLevel<T>& L, const Edges<T, B>& E, bool special,
                                           T* x,
                                           const Ahead<T, Sites<TL, B, 1, 1>, B::DIM>& b,
                                           const AheadEdge<T, Sites<TL, B, 2, 1>, B::DIM>& ed,
                                           T* r, T* psi, int i0, int j0, int k0) {
  const Grid& G = L.op.g;
  constexpr int DIM = B::DIM, N = B::N, SX = 1, SY = B::SY, SZ = B::SZ;
  stage_resid<T, VARMU, Sites<TL, B, 1, 1>, B>(L.op, x, E, special, b, r, i0, j0, k0);
  __syncthreads();
  typedef Sites<TL, B, 2, 1> S1;
#pragma unroll
  for (int q = 0; q < S1::PER; ++q) {
    S1 t;
    if (!t.get(q)) continue;
    const int s = t.s;
    const T* u = r;
    const T* v = r + N;
    T d[3];
    if constexpr (DIM == 2) {
      d[0] = u[s - SY] - u[s] - v[s - SX] + v[s];
    } else {
      const T* w = r + 2 * N;
      d[0] = v[s - SZ] - v[s] - w[s - SY] + w[s];
      d[1] = u[s] - u[s - SZ] + w[s - SX] - w[s];
      d[2] = u[s - SY] - u[s] - v[s - SX] + v[s];
    }
#pragma unroll
    for (int a = 0; a < (DIM == 3 ? 3 : 1); ++a) psi[a * N + s] = ed.v[q][a] * d[a];
  }
  __syncthreads();
  typedef Sites<TL, B, 2, 2> S2;
#pragma unroll
  for (int q = 0; q < S2::PER; ++q) {
    S2 t;
    if (!t.get(q)) continue;
    const int s = t.s, i = i0 + t.x, j = j0 + t.y, k = k0 + t.z;
    // only the lower faces of cells move
    const unsigned on = cell_in(G, i, j, k) ? unknown_bits<DIM>(G, i, j, k) : 0u;
    T d[3];
    if constexpr (DIM == 2) {
      d[0] = psi[s + SY] - psi[s];
      d[1] = psi[s] - psi[s + SX];
    } else {
      const T* px = psi;
      const T* py = psi + N;
      const T* pz = psi + 2 * N;
      d[0] = pz[s + SY] - pz[s] - py[s + SZ] + py[s];
      d[1] = px[s + SZ] - px[s] - pz[s + SX] + pz[s];
      d[2] = py[s + SX] - py[s] - px[s + SY] + px[s];
    }
#pragma unroll
    for (int c = 0; c < DIM; ++c)
      if ((on >> c) & 1u) x[c * N + s] += d[c];
  }
  __syncthreads();
}

// the tile owns the face of component c at offset (x, y, z) from its origin
// (0 <= offset): inside the tile, or the grid's upper boundary face right
// behind it
template <class TL>
__device__ __forceinline__ bool owned(const Grid& G, int c, int x, int y, int z, int i, int j,
                                      int k) {
  return x >= 0 && y >= 0 && z >= 0 && x < TL::TX + int(c == 0 && i == G.n[0]) &&
         y < TL::TY + int(c == 1 && j == G.n[1]) &&
         z < TL::TZ + int(c == 2 && k == G.n[2]) && in_array(G, c, i, j, k);
}

// restriction of component C at coarse site (I, J, K); s: the LDS site of the
// fine cell (2I, 2J, 2K)
template <typename T, class B, int C>
__device__ __forceinline__ T restrict_at(const Grid& Gc, const T* r, int s, int I, int J, int K,
                                         int smooth) {
  constexpr int DIM = B::DIM;
  constexpr int st[3] = {1, B::SY, B::SZ};
  constexpr int A1 = (C + 1) % DIM, A2 = (C + 2) % 3;
  const int P[3] = {I, J, K};
  const T* q = r + C * B::N + s;
  T acc = T(0);
  if (!smooth) {
#pragma unroll
    for (int dn = -1; dn <= 1; ++dn) {
      T t = T(0);
#pragma unroll
      for (int t1 = 0; t1 < 2; ++t1)
#pragma unroll
        for (int t2 = 0; t2 < (DIM == 3 ? 2 : 1); ++t2)
          t += q[dn * st[C] + t1 * st[A1] + (DIM == 3 ? t2 * st[A2] : 0)];
      acc += (dn == 0 ? T(1) : T(0.5)) * t;
    }
    return acc;
  }
  T w1[4], w2[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const bool cov = t == 1 || t == 2;
    w1[t] = cov ? cover_weight<T>(2 * P[A1] + t - 1, Gc.n[A1], Gc.bc[2 * A1], Gc.bc[2 * A1 + 1])
                : T(0.25);
    if (DIM == 3)
      w2[t] = cov ? cover_weight<T>(2 * P[A2] + t - 1, Gc.n[A2], Gc.bc[2 * A2], Gc.bc[2 * A2 + 1])
                  : T(0.25);
  }
#pragma unroll
  for (int dn = -1; dn <= 1; ++dn) {
    T t = T(0);
#pragma unroll
    for (int t1 = 0; t1 < 4; ++t1) {
      T u = T(0);
      if (DIM == 3) {
#pragma unroll
        for (int t2 = 0; t2 < 4; ++t2)
          u += w2[t2] * q[dn * st[C] + (t1 - 1) * st[A1] + (t2 - 1) * st[A2]];
      } else {
        u = q[dn * st[C] + (t1 - 1) * st[A1]];
      }
      t += w1[t1] * u;
    }
    acc += (dn == 0 ? T(1) : T(0.5)) * t;
  }
  return acc;
}

template <typename T, class B, class TL, int C>
__device__ __forceinline__ void restrict_store(const Grid& G, const Grid& Gc, const T* r, int s,
                                               int cx, int cy, int cz, int I, int J, int K,
                                               int smooth, T* __restrict__ bc,
                                               const T* __restrict__ dinv_c, T omega_c,
                                               T* __restrict__ x0c) {
  // owned coarse faces: the tile's, and the upper boundary face behind it
  const bool own = cx < TL::TX / 2 + int(C == 0 && I == Gc.n[0]) &&
                   cy < TL::TY / 2 + int(C == 1 && J == Gc.n[1]) &&
                   (B::DIM == 2 || cz < TL::TZ / 2 + int(C == 2 && K == Gc.n[2])) &&
                   in_array(Gc, C, I, J, K);
  if (!own) return;
  const int f = face(Gc, C, I, J, K);
  T v = T(0);
  if ((unknown_bits<B::DIM>(Gc, I, J, K) >> C) & 1u)
    v = restrict_at<T, B, C>(Gc, r, s, I, J, K, smooth) * T(B::DIM == 3 ? 0.125 : 0.25);
  bc[f] = v;
  if (x0c) x0c[f] = omega_c * dinv_c[f] * v;
}

// The way down.  HYB: Jacobi sweep + edge sweep (halo 4), else two Jacobi
// sweeps (halo 3).
template <typename T, class TL, bool VARMU, bool HYB>
__global__ __launch_bounds__(TL::NT) void k_leg_down(LegLevel<T> L, const T* __restrict__ b,
                                                     T* __restrict__ xo, T* __restrict__ bc,
                                                     const T* __restrict__ dinv_c, T omega_c,
                                                     T* __restrict__ x0c, const PcgState* st,
                                                     FoldCheck check) {
  typedef Box<TL, HYB ? 4 : 3> B;
  constexpr int DIM = B::DIM, N = B::N, H = B::H;
  __shared__ T X[DIM * N];
  __shared__ T Y[DIM * N];
  __shared__ T PSI[HYB ? (DIM == 3 ? 3 * N : N) : 1];
  __shared__ Edges<T, B> E;
  const int done = st ? st->done : 0;  // tested once the loads are in flight
  const Grid& G = L.op.g;
  const int ti = blockIdx.x * TL::TX, tj = blockIdx.y * TL::TY, tk = blockIdx.z * TL::TZ;
  const int i0 = ti - H, j0 = tj - H, k0 = DIM == 3 ? tk - H : 0;
  typedef Sites<TL, B, 0, 0> SA;                       // the whole box
  typedef Sites<TL, B, 1, 1> S1;                       // the first operator application
  typedef Sites<TL, B, HYB ? 3 : 2, HYB ? 3 : 2> SR;   // the residual that is restricted
  Ahead<T, SA, DIM> b0, d0;
  Ahead<T, S1, DIM> a1;  // HYB: b, else 1 / D
  Ahead<T, SR, DIM> br;
  AheadEdge<T, Sites<TL, B, HYB ? 2 : 0, HYB ? 1 : 0>, DIM> ed;
  b0.load(G, b, i0, j0, k0);
  d0.load(G, L.dinv, i0, j0, k0, b0.on);
  a1.load(G, HYB ? b : L.dinv, i0, j0, k0);
  if constexpr (HYB) ed.load(L, i0, j0, k0);
  br.load(G, b, i0, j0, k0);
  if (check.part) {  // uniform
    __shared__ FoldShared<TL::NT> fold;
    double rr;
    if (!fold_sum_if<TL::NT>(done, fold_share<TL::NT>(check.part, check.n), fold, rr)) return;
    const bool lead = threadIdx.x == 0 && blockIdx.x + blockIdx.y + blockIdx.z == 0;
    if (fold_check(check.st, rr, lead)) return;
  } else if (done) {
    return;
  }
  const bool special = fill_edges<T, TL, B>(G, E, i0, j0, k0);
  // first sweep from a zero guess
#pragma unroll
  for (int q = 0; q < SA::PER; ++q) {
    SA t;
    if (!t.get(q)) continue;
#pragma unroll
    for (int c = 0; c < DIM; ++c)
      X[c * N + t.s] = b0.unk(q, c) ? L.omega * d0.v[q][c] * b0.v[q][c] : T(0);
  }
  __syncthreads();
  auto store_own = [&](int c, int lx, int ly, int lz, T v) {
    const int i = i0 + lx, j = j0 + ly, k = k0 + lz;
    if (owned<TL>(G, c, lx - H, ly - H, DIM == 3 ? lz - H : 0, i, j, k)) xo[face(G, c, i, j, k)] = v;
  };
  const T* res;
  if constexpr (HYB) {
    stage_edge<T, VARMU, TL, B>(L, E, special, X, a1, ed, Y, PSI, i0, j0, k0);
    typedef Sites<TL, B, H, H - 1> SO;
#pragma unroll
    for (int q = 0; q < SO::PER; ++q) {
      SO t;
      if (!t.get(q)) continue;
#pragma unroll
      for (int c = 0; c < DIM; ++c) store_own(c, t.x, t.y, t.z, X[c * N + t.s]);
    }
    stage_resid<T, VARMU, SR, B>(L.op, X, E, special, br, Y, i0, j0, k0);
    res = Y;
  } else {
    // second sweep: x2 = x1 + omega / D (b - M x1), and omega / D b is x1
#pragma unroll
    for (int q = 0; q < S1::PER; ++q) {
      S1 t;
      if (!t.get(q)) continue;
      T m[3];
      row_M<T, VARMU, B>(L.op, E, special, X, t, i0 + t.x, j0 + t.y, k0 + t.z, m);
#pragma unroll
      for (int c = 0; c < DIM; ++c) {
        const T x1 = X[c * N + t.s];
        const T v = a1.unk(q, c) ? T(2) * x1 - L.omega * a1.v[q][c] * m[c] : T(0);
        Y[c * N + t.s] = v;
        store_own(c, t.x, t.y, t.z, v);
      }
    }
    __syncthreads();
    stage_resid<T, VARMU, SR, B>(L.op, Y, E, special, br, X, i0, j0, k0);
    res = X;
  }
  __syncthreads();
  // restriction: coarse sites of the tile and the boundary faces behind them
  constexpr int CX = TL::TX / 2 + 1, CY = TL::TY / 2 + 1, CZ = DIM == 3 ? TL::TZ / 2 + 1 : 1;
  for (int e = threadIdx.x; e < CX * CY * CZ; e += TL::NT) {
    const int q = e / CX, cx = e - q * CX, cy = DIM == 3 ? q % CY : q, cz = DIM == 3 ? q / CY : 0;
    const int I = ti / 2 + cx, J = tj / 2 + cy, K = DIM == 3 ? tk / 2 + cz : 0;
    const int s = ((DIM == 3 ? H + 2 * cz : 0) * B::EY + H + 2 * cy) * B::EX + H + 2 * cx;
    restrict_store<T, B, TL, 0>(G, L.gc, res, s, cx, cy, cz, I, J, K, L.smooth, bc, dinv_c, omega_c, x0c);
    restrict_store<T, B, TL, 1>(G, L.gc, res, s, cx, cy, cz, I, J, K, L.smooth, bc, dinv_c, omega_c, x0c);
    if constexpr (DIM == 3)
      restrict_store<T, B, TL, 2>(G, L.gc, res, s, cx, cy, cz, I, J, K, L.smooth, bc, dinv_c, omega_c, x0c);
  }
}

// prolongation of component C at fine site (i, j, k) from the coarse values
// in LDS (box of CX x CY x CZ sites from (I0, J0, K0))
template <typename T, int DIM, int C, int CX, int CY>
__device__ __forceinline__ T prolong_at(const Grid& Gc, const T* e, int I0, int J0, int K0, int i,
                                        int j, int k, int smooth) {
  constexpr int st[3] = {1, CX, CX * CY};
  constexpr int A1 = (C + 1) % DIM, A2 = (C + 2) % 3;
  const int P[3] = {i, j, k};
  const int s = ((DIM == 3 ? (k >> 1) - K0 : 0) * CY + (j >> 1) - J0) * CX + (i >> 1) - I0;
  const bool odd = P[C] & 1;
  if (!smooth) {
    const T a = e[s];
    return odd ? T(0.5) * (a + e[s + st[C]]) : a;
  }
  const int d1 = (P[A1] & 1) ? st[A1] : -st[A1];
  const T w1 = cover_weight<T>(P[A1], Gc.n[A1], Gc.bc[2 * A1], Gc.bc[2 * A1 + 1]);
  auto plane = [&](int q) {  // tangential interpolation at normal site q
    if (DIM == 2) return w1 * e[q] + T(0.25) * e[q + d1];
    const int d2 = (P[A2] & 1) ? st[A2] : -st[A2];
    const T w2 = cover_weight<T>(P[A2], Gc.n[A2], Gc.bc[2 * A2], Gc.bc[2 * A2 + 1]);
    return w1 * (w2 * e[q] + T(0.25) * e[q + d2]) +
           T(0.25) * (w2 * e[q + d1] + T(0.25) * e[q + d1 + d2]);
  };
  return odd ? T(0.5) * (plane(s) + plane(s + st[C])) : plane(s);
}

// The way up.  HYB: edge sweep + Jacobi sweep (halo 3), else two Jacobi
// sweeps (halo 2).
template <typename T, class TL, bool VARMU, bool HYB>
__global__ __launch_bounds__(TL::NT) void k_leg_up(LegLevel<T> L, const T* __restrict__ ec,
                                                   const T* __restrict__ xi,
                                                   const T* __restrict__ b, T* __restrict__ xo,
                                                   double* __restrict__ partial,
                                                   const PcgState* __restrict__ st) {
  typedef Box<TL, HYB ? 3 : 2> B;
  constexpr int DIM = B::DIM, N = B::N, H = B::H;
  // coarse box: two sites more on each side (the halo of fine sites reaches
  // one covering row further, the SMOOTH neighbours and the normal mean one
  // more)
  constexpr int CX = TL::TX / 2 + 4, CY = TL::TY / 2 + 4, CZ = DIM == 3 ? TL::TZ / 2 + 4 : 1;
  constexpr int NC = CX * CY * CZ, PC = (NC + TL::NT - 1) / TL::NT;
  __shared__ T X[DIM * N];
  __shared__ T Y[DIM * N];
  __shared__ T EC[DIM * NC];
  __shared__ T PSI[HYB ? (DIM == 3 ? 3 * N : N) : 1];
  __shared__ Edges<T, B> E;
  const int done = st ? st->done : 0;  // tested once the loads are in flight
  const Grid& G = L.op.g;
  const Grid& Gc = L.gc;
  const int ti = blockIdx.x * TL::TX, tj = blockIdx.y * TL::TY, tk = blockIdx.z * TL::TZ;
  const int i0 = ti - H, j0 = tj - H, k0 = DIM == 3 ? tk - H : 0;
  const int I0 = ti / 2 - 2, J0 = tj / 2 - 2, K0 = DIM == 3 ? tk / 2 - 2 : 0;
  typedef Sites<TL, B, 0, 0> SA;
  typedef Sites<TL, B, 1, 1> S1;
  typedef Sites<TL, B, H, H - 1> SO;  // own sites and the boundary faces behind them
  T ev[PC][DIM];
#pragma unroll
  for (int q = 0; q < PC; ++q) {
    const int e = threadIdx.x + q * TL::NT, r = e / CX, I = I0 + e - r * CX,
              J = J0 + (DIM == 3 ? r % CY : r), K = DIM == 3 ? K0 + r / CY : 0;
    const unsigned u = e < NC ? unknown_bits<DIM>(Gc, I, J, K) : 0u;
#pragma unroll
    for (int c = 0; c < DIM; ++c) {
      const bool on = (u >> c) & 1u;
      const T v = ec[on ? face(Gc, c, I, J, K) : 0];
      ev[q][c] = on ? v : T(0);
    }
  }
  Ahead<T, SA, DIM> x0;
  Ahead<T, S1, DIM> b1, d1;
  Ahead<T, SO, DIM> bo, dd;
  AheadEdge<T, Sites<TL, B, HYB ? 2 : 0, HYB ? 1 : 0>, DIM> ed;
  x0.load(G, xi, i0, j0, k0);
  b1.load(G, b, i0, j0, k0);
  if constexpr (HYB) ed.load(L, i0, j0, k0);
  else d1.load(G, L.dinv, i0, j0, k0, b1.on);
  bo.load(G, b, i0, j0, k0);
  dd.load(G, L.dinv, i0, j0, k0, bo.on);
  if (done) return;
  const bool special = fill_edges<T, TL, B>(G, E, i0, j0, k0);
#pragma unroll
  for (int q = 0; q < PC; ++q) {
    const int e = threadIdx.x + q * TL::NT;
    if (e < NC)
#pragma unroll
      for (int c = 0; c < DIM; ++c) EC[c * NC + e] = ev[q][c];
  }
  if constexpr (!HYB) {
    // the layer of Y that the first sweep leaves out is read (times nothing
    // that matters) by the upper boundary faces: it has to be 0
    for (int e = threadIdx.x; e < DIM * N; e += TL::NT) Y[e] = T(0);
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < SA::PER; ++q) {
    SA t;
    if (!t.get(q)) continue;
    const int i = i0 + t.x, j = j0 + t.y, k = k0 + t.z;
    T v[3] = {T(0), T(0), T(0)};
    if (x0.unk(q, 0))
      v[0] = x0.v[q][0] + prolong_at<T, DIM, 0, CX, CY>(Gc, EC, I0, J0, K0, i, j, k, L.smooth);
    if (x0.unk(q, 1))
      v[1] = x0.v[q][1] + prolong_at<T, DIM, 1, CX, CY>(Gc, EC + NC, I0, J0, K0, i, j, k, L.smooth);
    if constexpr (DIM == 3)
      if (x0.unk(q, 2))
        v[2] = x0.v[q][2] +
               prolong_at<T, DIM, 2, CX, CY>(Gc, EC + 2 * NC, I0, J0, K0, i, j, k, L.smooth);
#pragma unroll
    for (int c = 0; c < DIM; ++c) X[c * N + t.s] = v[c];
  }
  __syncthreads();
  const T* last = X;
  if constexpr (HYB) {
    stage_edge<T, VARMU, TL, B>(L, E, special, X, b1, ed, Y, PSI, i0, j0, k0);
  } else {
#pragma unroll
    for (int q = 0; q < S1::PER; ++q) {
      S1 t;
      if (!t.get(q)) continue;
      T m[3];
      row_M<T, VARMU, B>(L.op, E, special, X, t, i0 + t.x, j0 + t.y, k0 + t.z, m);
#pragma unroll
      for (int c = 0; c < DIM; ++c)
        if (b1.unk(q, c))
          Y[c * N + t.s] = X[c * N + t.s] + L.omega * d1.v[q][c] * (b1.v[q][c] - m[c]);
    }
    __syncthreads();
    last = Y;
  }
  double part = 0.0;
#pragma unroll
  for (int q = 0; q < SO::PER; ++q) {
    SO t;
    if (!t.get(q)) continue;
    const int i = i0 + t.x, j = j0 + t.y, k = k0 + t.z;
    T m[3];
    row_M<T, VARMU, B>(L.op, E, special, last, t, i, j, k, m);
#pragma unroll
    for (int c = 0; c < DIM; ++c) {
      if (!owned<TL>(G, c, t.x - H, t.y - H, DIM == 3 ? t.z - H : 0, i, j, k)) continue;
      T v = T(0);
      if (bo.unk(q, c)) {
        v = last[c * N + t.s] + L.omega * dd.v[q][c] * (bo.v[q][c] - m[c]);
        part += double(bo.v[q][c]) * double(v);
      }
      xo[face(G, c, i, j, k)] = v;
    }
  }
  if (partial) {
    __shared__ double sh[TL::NT / 64];
    const double t = block_sum<TL::NT>(part, sh);
    if (threadIdx.x == 0)
      partial[blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z)] = t;
  }
}

// The product of a PCG iteration with the direction update, beta folded in
// (halo 1, and one layer more above: the boundary faces behind the tile).
template <typename T, class TL, bool VARMU>
__global__ __launch_bounds__(TL::NT) void k_leg_apply(Op<T> op, const T* __restrict__ z,
                                                      const T* __restrict__ p, T* __restrict__ q,
                                                      T* __restrict__ pn,
                                                      double* __restrict__ part_pq, PcgState* st,
                                                      const double* __restrict__ part_rz, int nrz) {
  typedef Box<TL, 1, 2> B;
  constexpr int DIM = B::DIM, N = B::N, H = 1;
  __shared__ T X[DIM * N];
  __shared__ Edges<T, B> E;
  __shared__ double sh[TL::NT / 64];
  const int done = st->done;
  const Grid& G = op.g;
  const int ti = blockIdx.x * TL::TX, tj = blockIdx.y * TL::TY, tk = blockIdx.z * TL::TZ;
  const int i0 = ti - H, j0 = tj - H, k0 = DIM == 3 ? tk - H : 0;
  typedef Sites<TL, B, 0, 0> SA;
  Ahead<T, SA, DIM> za, pa;
  za.load(G, z, i0, j0, k0);
  pa.load(G, p, i0, j0, k0, za.on);
  const double share = fold_share<TL::NT>(part_rz, nrz);
  if (done) return;
  const bool special = fill_edges<T, TL, B>(G, E, i0, j0, k0);
  const double rz = fold_sum<TL::NT>(share, sh);
  const bool lead = threadIdx.x == 0 && blockIdx.x + blockIdx.y + blockIdx.z == 0;
  const T beta = T(fold_beta(st, rz, lead));
#pragma unroll
  for (int e = 0; e < SA::PER; ++e) {
    SA t;
    if (!t.get(e)) continue;
#pragma unroll
    for (int c = 0; c < DIM; ++c)
      X[c * N + t.s] = za.unk(e, c) ? za.v[e][c] + beta * pa.v[e][c] : T(0);
  }
  __syncthreads();
  double part = 0.0;
  typedef Sites<TL, B, 1, 1> SO;  // own sites and the boundary faces behind them
#pragma unroll
  for (int e = 0; e < SO::PER; ++e) {
    SO t;
    if (!t.get(e)) continue;
    const int i = i0 + t.x, j = j0 + t.y, k = k0 + t.z;
    T m[3];
    row_M<T, VARMU, B>(op, E, special, X, t, i, j, k, m);
    const unsigned on = unknown_bits<DIM>(G, i, j, k);
#pragma unroll
    for (int c = 0; c < DIM; ++c) {
      if (!owned<TL>(G, c, t.x - H, t.y - H, DIM == 3 ? t.z - H : 0, i, j, k)) continue;
      T v = T(0), w = T(0);
      if ((on >> c) & 1u) {
        w = X[c * N + t.s];
        v = m[c];
        part += double(w) * double(v);
      }
      const int f = face(G, c, i, j, k);
      q[f] = v;
      pn[f] = w;
    }
  }
  const double s = block_sum<TL::NT>(part, sh);
  if (threadIdx.x == 0)
    part_pq[blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z)] = s;
}

// tiles: 2D small and large, 3D small, medium and large
typedef Tile<2, 8, 8, 1, 256> T2S;
typedef Tile<2, 32, 16, 1, 512> T2L;
typedef Tile<3, 4, 4, 4, 512> T3S;
typedef Tile<3, 8, 8, 4, 512> T3M;
typedef Tile<3, 8, 8, 8, 512> T3L;
typedef Tile<2, 16, 8, 1, 256> T2P;  // product only (halo 1): small 2D levels

template <class TL>
LegPlan plan_of(const Grid& g, int id) {
  LegPlan p;
  p.tile = id;
  p.grid = dim3((g.n[0] + TL::TX - 1) / TL::TX, (g.n[1] + TL::TY - 1) / TL::TY,
                (g.n[2] + TL::TZ - 1) / TL::TZ);
  p.nblocks = p.grid.x * p.grid.y * p.grid.z;
  return p;
}

template <typename T, class TL, bool HYB>
void launch_down(hipStream_t s, const LegPlan& p, const LegLevel<T>& L, const T* b, T* xo, T* bc,
                 const T* dinv_c, T omega_c, T* x0c, const PcgState* st, const FoldCheck& ck) {
  if (L.op.mu)
    k_leg_down<T, TL, true, HYB><<<p.grid, TL::NT, 0, s>>>(L, b, xo, bc, dinv_c, omega_c, x0c, st, ck);
  else
    k_leg_down<T, TL, false, HYB><<<p.grid, TL::NT, 0, s>>>(L, b, xo, bc, dinv_c, omega_c, x0c, st, ck);
}

template <typename T, class TL, bool HYB>
void launch_up(hipStream_t s, const LegPlan& p, const LegLevel<T>& L, const T* ec, const T* xi,
               const T* b, T* xo, double* partial, const PcgState* st) {
  if (L.op.mu)
    k_leg_up<T, TL, true, HYB><<<p.grid, TL::NT, 0, s>>>(L, ec, xi, b, xo, partial, st);
  else
    k_leg_up<T, TL, false, HYB><<<p.grid, TL::NT, 0, s>>>(L, ec, xi, b, xo, partial, st);
}

}  // namespace

// Where the legs run.  2D: on every level; 512^2 (FP64, V(2,2), smooth
// transfers) takes 21 us for both legs against 53 us of separate kernels,
// the levels below 9-12 us against 27-34 us, whichever the smoother.  8 x 8
// tiles give the small levels enough blocks and one site per thread; from
// 2^17 cells on 32 x 16 tiles halve the recomputed halo.
// 3D: while the level is one round of blocks (256 CUs).  Both legs against
// separate kernels, FP32 with DIV transfers: 16^3 13 against 24 us, 32^3 19
// against 26 us; but 64^3, two rounds of 8^3 tiles, 39 us against 34 us: the
// recomputed halo (5.4 sites per own site) then costs more than the round
// trips it saves.  FP64 with SMOOTH transfers: 48 x 40 x 56 33 against 53 us.
// Hybrid V(1,1), FP32 with varying viscosity: 24^3 38 against 45 us, 48^3 64
// against 54 us.  A hybrid leg in FP64 needs 124 KB of LDS for the 4^3 tile,
// so larger tiles do not fit.
LegPlan leg_plan(const Grid& g, bool hybrid, int elem) {
  const long cells = g.n_cells;
  if (g.dim == 2) return cells >= (1L << 17) ? plan_of<T2L>(g, 2) : plan_of<T2S>(g, 1);
  LegPlan p;
  if (cells <= 16L * 16 * 16) p = plan_of<T3S>(g, 3);
  else if (hybrid) p = elem == 8 ? plan_of<T3S>(g, 3) : plan_of<T3M>(g, 4);
  else p = cells <= 40L * 40 * 40 ? plan_of<T3M>(g, 4) : plan_of<T3L>(g, 5);
  return p.nblocks <= 256 ? p : LegPlan();
}

LegPlan apply_plan(const Grid& g) {
  if (g.dim == 2) return g.n_cells >= (1 << 17) ? plan_of<T2L>(g, 2) : plan_of<T2P>(g, 1);
  return g.n_cells <= 32 * 32 * 32 ? plan_of<T3M>(g, 4) : plan_of<T3L>(g, 5);
}

template <typename T, class TL>
void launch_apply(hipStream_t s, const LegPlan& p, const Op<T>& op, const T* z, const T* pv, T* q,
                  T* pn, double* part_pq, PcgState* st, const double* part_rz, int nrz) {
  if (op.mu)
    k_leg_apply<T, TL, true><<<p.grid, TL::NT, 0, s>>>(op, z, pv, q, pn, part_pq, st, part_rz, nrz);
  else
    k_leg_apply<T, TL, false><<<p.grid, TL::NT, 0, s>>>(op, z, pv, q, pn, part_pq, st, part_rz, nrz);
}

template <typename T>
void leg_apply(hipStream_t s, const LegPlan& p, const Op<T>& op, const T* z, const T* pv, T* q,
               T* pn, double* part_pq, PcgState* st, const double* part_rz, int nrz) {
  switch (p.tile) {
    case 1: launch_apply<T, T2P>(s, p, op, z, pv, q, pn, part_pq, st, part_rz, nrz); break;
    case 2: launch_apply<T, T2L>(s, p, op, z, pv, q, pn, part_pq, st, part_rz, nrz); break;
    case 4: launch_apply<T, T3M>(s, p, op, z, pv, q, pn, part_pq, st, part_rz, nrz); break;
    case 5: launch_apply<T, T3L>(s, p, op, z, pv, q, pn, part_pq, st, part_rz, nrz); break;
  }
}

template <typename T>
void leg_down(hipStream_t s, const LegPlan& p, const LegLevel<T>& L, const T* b, T* xo, T* bc,
              const T* dinv_c, T omega_c, T* x0c, const PcgState* st,
              const FoldCheck& ck) {
  const bool hyb = L.edinv != nullptr;
  switch (p.tile) {
    case 1:
      if (hyb) launch_down<T, T2S, true>(s, p, L, b, xo, bc, dinv_c, omega_c, x0c, st, ck);
      else launch_down<T, T2S, false>(s, p, L, b, xo, bc, dinv_c, omega_c, x0c, st, ck);
      break;
    case 2:
      if (hyb) launch_down<T, T2L, true>(s, p, L, b, xo, bc, dinv_c, omega_c, x0c, st, ck);
      else launch_down<T, T2L, false>(s, p, L, b, xo, bc, dinv_c, omega_c, x0c, st, ck);
      break;
    case 3:
      if (hyb) launch_down<T, T3S, true>(s, p, L, b, xo, bc, dinv_c, omega_c, x0c, st, ck);
      else launch_down<T, T3S, false>(s, p, L, b, xo, bc, dinv_c, omega_c, x0c, st, ck);
      break;
    case 4:
      if (!hyb) launch_down<T, T3M, false>(s, p, L, b, xo, bc, dinv_c, omega_c, x0c, st, ck);
      else if constexpr (sizeof(T) == 4)  // FP64 needs more LDS than a CU has
        launch_down<T, T3M, true>(s, p, L, b, xo, bc, dinv_c, omega_c, x0c, st, ck);
      break;
    case 5:
      launch_down<T, T3L, false>(s, p, L, b, xo, bc, dinv_c, omega_c, x0c, st, ck);
      break;
  }
}

template <typename T>
void leg_up(hipStream_t s, const LegPlan& p, const LegLevel<T>& L, const T* ec, const T* xi,
            const T* b, T* xo, double* partial, const PcgState* st) {
  const bool hyb = L.edinv != nullptr;
  switch (p.tile) {
    case 1:
      if (hyb) launch_up<T, T2S, true>(s, p, L, ec, xi, b, xo, partial, st);
      else launch_up<T, T2S, false>(s, p, L, ec, xi, b, xo, partial, st);
      break;
    case 2:
      if (hyb) launch_up<T, T2L, true>(s, p, L, ec, xi, b, xo, partial, st);
      else launch_up<T, T2L, false>(s, p, L, ec, xi, b, xo, partial, st);
      break;
    case 3:
      if (hyb) launch_up<T, T3S, true>(s, p, L, ec, xi, b, xo, partial, st);
      else launch_up<T, T3S, false>(s, p, L, ec, xi, b, xo, partial, st);
      break;
    case 4:
      if (!hyb) launch_up<T, T3M, false>(s, p, L, ec, xi, b, xo, partial, st);
      else if constexpr (sizeof(T) == 4)
        launch_up<T, T3M, true>(s, p, L, ec, xi, b, xo, partial, st);
      break;
    case 5:
      launch_up<T, T3L, false>(s, p, L, ec, xi, b, xo, partial, st);
      break;
  }
}

template void leg_apply<float>(hipStream_t, const LegPlan&, const Op<float>&, const float*,
                               const float*, float*, float*, double*, PcgState*, const double*,
                               int);
template void leg_apply<double>(hipStream_t, const LegPlan&, const Op<double>&, const double*,
                                const double*, double*, double*, double*, PcgState*,
                                const double*, int);
template void leg_down<float>(hipStream_t, const LegPlan&, const LegLevel<float>&, const float*,
                              float*, float*, const float*, float, float*, const PcgState*,
                              const FoldCheck&);
template void leg_down<double>(hipStream_t, const LegPlan&, const LegLevel<double>&, const double*,
                               double*, double*, const double*, double, double*, const PcgState*,
                               const FoldCheck&);
template void leg_up<float>(hipStream_t, const LegPlan&, const LegLevel<float>&, const float*,
                            const float*, const float*, float*, double*, const PcgState*);
template void leg_up<double>(hipStream_t, const LegPlan&, const LegLevel<double>&, const double*,
                             const double*, const double*, double*, double*, const PcgState*);

}  // namespace gkb

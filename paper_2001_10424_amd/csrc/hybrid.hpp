// Edge-space (vector potential) smoothing for M = W + eta A A^T.
//
// Point-Jacobi on M cannot damp the oscillatory divergence-free error of a
// level once eta >> mu: those fields see only W, a thousandth of the diagonal
// that scales the sweep.  Every discretely divergence-free face field of the
// MAC grid is a discrete curl C psi of an edge field psi (a stream function
// on the vertices in 2D), and A^T C = 0, so M C = W C.  The hybrid smoother
// follows each weighted-Jacobi sweep on M by a weighted-Jacobi sweep on the
// edge operator C^T W C,
//     x += C omega_e D_e^-1 C^T (b - M x),   D_e = diag(C^T W C),
// which acts on exactly the fields the face sweep misses (Hiptmair's hybrid
// smoother for H(div) problems, here with Jacobi in both spaces).  Applied
// as (face, edge) before and (edge, face) after the coarse correction, the
// V-cycle stays symmetric.
//
// Edge storage: the point grid of the cells, component-major.  3D point
// (i, j, k) carries the x-edge (i+1/2, j, k), the y-edge (i, j+1/2, k) and
// the z-edge (i, j, k+1/2), i.e. the edges through the lowest corner of cell
// (i, j, k); 2D point (i, j) carries the vertex (i, j).  Edges beyond the
// point grid are 0, and so is every edge lying in a DIRICHLET wall, which
// keeps C psi zero on the faces that are not unknowns.  With these
// conventions
//     u(p) = psi_z(p + e_y) - psi_z(p) - psi_y(p + e_z) + psi_y(p)
//     v(p) = psi_x(p + e_z) - psi_x(p) - psi_z(p + e_x) + psi_z(p)
//     w(p) = psi_y(p + e_x) - psi_y(p) - psi_x(p + e_y) + psi_x(p)
// (2D: u(p) = psi(p + e_y) - psi(p), v(p) = psi(p) - psi(p + e_x)) on the
// lower faces of cell p, and C^T is the exact transpose.  The 1/h of the
// curl is left out: D_e absorbs the scale.
#pragma once
#include <hip/hip_runtime.h>

#include "kernels.hpp"

namespace gkb {

template <int DIM>
constexpr int edge_comps() { return DIM == 3 ? 3 : 1; }

// edge component a at point (i, j, k) lies in a DIRICHLET wall
template <int DIM>
__device__ __forceinline__ bool edge_in_wall(const Grid& G, int a, int i, int j, int k) {
  const bool wx = i == 0 && G.bc[0] == kDir;
  const bool wy = j == 0 && G.bc[2] == kDir;
  const bool wz = DIM == 3 && k == 0 && G.bc[4] == kDir;
  if (DIM == 2) return wx || wy;
  if (a == 0) return wy || wz;  // x-edge: planes y = j and z = k
  if (a == 1) return wx || wz;
  return wx || wy;
}

// value of face component C at point (i, j, k) of the lower-face lattice;
// 0 outside the point grid
template <int C, typename T>
__device__ __forceinline__ T face_at(const Grid& G, const T* __restrict__ r, int i, int j, int k) {
  if (i < 0 || j < 0 || k < 0) return T(0);
  return r[fidx<C>(G, i, j, k)];
}

// psi = omega dinv (C^T r) on every edge (dinv == nullptr: unscaled C^T r);
// edges in a DIRICHLET wall get 0.  Grid: cell planes (x fastest).
template <typename T, int DIM>
__global__ __launch_bounds__(kBlock) void k_edge_ct(Grid G, const T* __restrict__ r,
                                                    const T* __restrict__ dinv, T omega,
                                                    T* __restrict__ psi, const PcgState* st) {
  if (st && st->done) return;
  const int k = blockIdx.z;
  const int idx = blockIdx.x * kBlock + threadIdx.x;
  if (idx >= G.n[0] * G.n[1]) return;
  const int j = idx / G.n[0], i = idx - j * G.n[0];
  const long nc = G.n_cells;
  const long p = (long)k * G.n[0] * G.n[1] + idx;
  if (DIM == 2) {
    T t = face_at<0>(G, r, i, j - 1, 0) - face_at<0>(G, r, i, j, 0) -
          face_at<1>(G, r, i - 1, j, 0) + face_at<1>(G, r, i, j, 0);
    if (edge_in_wall<2>(G, 0, i, j, 0)) t = T(0);
    else t *= dinv ? omega * dinv[p] : omega;
    psi[p] = t;
    return;
  }
  const T du = face_at<0>(G, r, i, j, k), dv = face_at<1>(G, r, i, j, k),
          dw = face_at<2>(G, r, i, j, k);
  T tx = face_at<1>(G, r, i, j, k - 1) - dv - face_at<2>(G, r, i, j - 1, k) + dw;
  T ty = du - face_at<0>(G, r, i, j, k - 1) + face_at<2>(G, r, i - 1, j, k) - dw;
  T tz = face_at<0>(G, r, i, j - 1, k) - du - face_at<1>(G, r, i - 1, j, k) + dv;
  tx = edge_in_wall<3>(G, 0, i, j, k) ? T(0) : tx * (dinv ? omega * dinv[p] : omega);
  ty = edge_in_wall<3>(G, 1, i, j, k) ? T(0) : ty * (dinv ? omega * dinv[nc + p] : omega);
  tz = edge_in_wall<3>(G, 2, i, j, k) ? T(0) : tz * (dinv ? omega * dinv[2 * nc + p] : omega);
  psi[p] = tx;
  psi[nc + p] = ty;
  psi[2 * nc + p] = tz;
}

template <typename T>
__device__ __forceinline__ T pt(const Grid& G, const T* __restrict__ a, int i, int j, int k) {
  if (i >= G.n[0] || j >= G.n[1] || k >= G.n[2]) return T(0);
  return a[((long)k * G.n[1] + j) * G.n[0] + i];
}

// x += C psi on the unknown faces (the lower faces of each cell; C psi is 0
// on the upper boundary faces)
template <typename T, int DIM>
__global__ __launch_bounds__(kBlock) void k_curl_add(Grid G, const T* __restrict__ psi,
                                                     T* __restrict__ x, const PcgState* st) {
  if (st && st->done) return;
  const int k = blockIdx.z;
  const int idx = blockIdx.x * kBlock + threadIdx.x;
  if (idx >= G.n[0] * G.n[1]) return;
  const int j = idx / G.n[0], i = idx - j * G.n[0];
  const long nc = G.n_cells;
  if (DIM == 2) {
    const T s = pt(G, psi, i, j, 0);
    if (unk<0>(G, i)) x[fidx<0>(G, i, j, 0)] += pt(G, psi, i, j + 1, 0) - s;
    if (unk<1>(G, j)) x[fidx<1>(G, i, j, 0)] += s - pt(G, psi, i + 1, j, 0);
    return;
  }
  const T* px = psi;
  const T* py = psi + nc;
  const T* pz = psi + 2 * nc;
  const T sx = pt(G, px, i, j, k), sy = pt(G, py, i, j, k), sz = pt(G, pz, i, j, k);
  if (unk<0>(G, i))
    x[fidx<0>(G, i, j, k)] += pt(G, pz, i, j + 1, k) - sz - pt(G, py, i, j, k + 1) + sy;
  if (unk<1>(G, j))
    x[fidx<1>(G, i, j, k)] += pt(G, px, i, j, k + 1) - sx - pt(G, pz, i + 1, j, k) + sz;
  if (unk<2>(G, k))
    x[fidx<2>(G, i, j, k)] += pt(G, py, i + 1, j, k) - sy - pt(G, px, i, j + 1, k) + sx;
}

// psi = omega dinv (C^T r) at the vertex (i, j) >= 0; 0 beyond the point grid
// or in a DIRICHLET wall
template <typename T>
__device__ __forceinline__ T vertex_psi(const Grid& G, const T* __restrict__ r,
                                        const T* __restrict__ dinv, T omega, int i, int j) {
  if (i >= G.n[0] || j >= G.n[1] || edge_in_wall<2>(G, 0, i, j, 0)) return T(0);
  const T t = face_at<0>(G, r, i, j - 1, 0) - face_at<0>(G, r, i, j, 0) -
              face_at<1>(G, r, i - 1, j, 0) + face_at<1>(G, r, i, j, 0);
  return omega * dinv[j * G.n[0] + i] * t;
}

// The edge half of the hybrid smoother in one pass, x += C omega D_e^-1 C^T r on
// the lower faces of every cell; the edge field is never stored.  2D: each
// point evaluates the three vertex values that its two faces need.
template <typename T>
__global__ __launch_bounds__(kBlock) void k_edge_smooth2(Grid G, const T* __restrict__ r,
                                                         const T* __restrict__ dinv, T omega,
                                                         T* __restrict__ x, const PcgState* st) {
  if (st && st->done) return;
  const int idx = blockIdx.x * kBlock + threadIdx.x;
  if (idx >= G.n[0] * G.n[1]) return;
  const int j = idx / G.n[0], i = idx - j * G.n[0];
  const T s = vertex_psi<T>(G, r, dinv, omega, i, j);
  if (unk<0>(G, i)) x[fidx<0>(G, i, j, 0)] += vertex_psi<T>(G, r, dinv, omega, i, j + 1) - s;
  if (unk<1>(G, j)) x[fidx<1>(G, i, j, 0)] += s - vertex_psi<T>(G, r, dinv, omega, i + 1, j);
}

// 3D: a block of 33 x 15 points forms each edge value of a plane once and
// marches kz planes up; its own values of the plane above stay in registers,
// the neighbours' come from LDS, so 32 x 14 points move their faces (extents are mostly multiples of 8).  Loads are
// unconditional (clamped) and one plane ahead.
// Bound by memory: r and 1/D_e read, x read and written.  192^3 FP32: 87 us
// (343 MB); every point evaluating the nine edge values of its faces from r
// took 130 us.
constexpr int kEdgeX = 33, kEdgeY = 15, kEdgeThreads = 512;
template <typename T>
__global__ __launch_bounds__(kEdgeThreads) void k_edge_smooth3(Grid G, const T* __restrict__ r,
                                                                 const T* __restrict__ dinv,
                                                                 T omega, T* __restrict__ x,
                                                                 const PcgState* st, int kz) {
  if (st && st->done) return;
  __shared__ T P[2][3][kEdgeY][kEdgeX];
  const int nx = G.n[0], ny = G.n[1], nz = G.n[2];
  // blocks of one XCD are neighbours
  const int nb = gridDim.x * gridDim.y * gridDim.z;
  const int b = blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z);
  const int xcd = b & 7, lin = xcd * (nb >> 3) + min(xcd, nb & 7) + (b >> 3);
  const int bx = lin % gridDim.x, rest = lin / gridDim.x;
  const int lx = threadIdx.x % kEdgeX, ly = threadIdx.x / kEdgeX;
  const int i = bx * (kEdgeX - 1) + lx, j = int(rest % gridDim.y) * (kEdgeY - 1) + ly;
  const int k0 = int(rest / gridDim.y) * kz, k1 = min(k0 + kz, nz);
  const bool slot = ly < kEdgeY, in = slot && i < nx && j < ny;
  const bool own = in && lx < kEdgeX - 1 && ly < kEdgeY - 1;
  const bool wx = i == 0 && G.bc[0] == kDir, wy = j == 0 && G.bc[2] == kDir;
  const int ic = min(i, nx - 1), jc = min(j, ny - 1), iw = max(ic - 1, 0), js = max(jc - 1, 0);
  const int e0 = G.ext[0][0];
  const int pu = e0 * G.ext[0][1], pv = nx * G.ext[1][1], pw = nx * ny;
  const int ou = G.off[0] + jc * e0 + ic, ous = G.off[0] + js * e0 + ic;
  const int ov = G.off[1] + jc * nx + ic, ovw = G.off[1] + jc * nx + iw;
  const int ow = G.off[2] + jc * nx + ic, oww = G.off[2] + jc * nx + iw, ows = G.off[2] + js * nx + ic;
  const int od = jc * nx + ic;
  const long nc = G.n_cells;
  struct Raw {
    T u, us, v, vw, w, ww, ws, dx, dy, dz;
  };
  auto load = [&](int k) {
    const int kk = min(max(k, 0), nz - 1);
    const T *ru = r + kk * pu, *rv = r + kk * pv, *rw = r + kk * pw, *d = dinv + (long)kk * pw;
    return Raw{ru[ou], ru[ous], rv[ov],  rv[ovw],      rw[ow],
               rw[oww], rw[ows], d[od], (d + nc)[od], (d + 2 * nc)[od]};
  };
  struct Tri3 {
    T a, b, c;
  };
  auto load_x = [&](int k) {
    const int kk = min(k, nz - 1);
    return Tri3{(x + kk * pu)[ou], (x + kk * pv)[ov], (x + kk * pw)[ow]};
  };
  T uB = T(0), vB = T(0);  // r on the plane below
  auto psi = [&](int k, const Raw& q) {
    const bool on = in && k < nz, wz = k == 0 && G.bc[4] == kDir;
    const T us = j > 0 ? q.us : T(0), vw = i > 0 ? q.vw : T(0), ww = i > 0 ? q.ww : T(0),
            ws = j > 0 ? q.ws : T(0);
    const T tx = vB - q.v - ws + q.w, ty = q.u - uB + ww - q.w, tz = us - q.u - vw + q.v;
    uB = q.u;
    vB = q.v;
    return Tri3{on && !(wy || wz) ? omega * q.dx * tx : T(0),
                on && !(wx || wz) ? omega * q.dy * ty : T(0),
                on && !(wx || wy) ? omega * q.dz * tz : T(0)};
  };
  if (k0 > 0) {  // uniform
    uB = (r + (k0 - 1) * pu)[ou];
    vB = (r + (k0 - 1) * pv)[ov];
  }
  Raw q = load(k0);
  Tri3 p = psi(k0, q);
  q = load(k0 + 1);
  Tri3 xv = load_x(k0);
  int s = 0;
  if (slot) P[s][0][ly][lx] = p.a, P[s][1][ly][lx] = p.b, P[s][2][ly][lx] = p.c;
  __syncthreads();
  for (int k = k0; k < k1; ++k) {
    const Tri3 n = psi(k + 1, q);
    const Tri3 xc = xv;
    q = load(k + 2);
    xv = load_x(k + 1);
    if (own) {
      const T zE = P[s][2][ly][lx + 1], zN = P[s][2][ly + 1][lx], yE = P[s][1][ly][lx + 1],
              xN = P[s][0][ly + 1][lx];
      if (unk<0>(G, i)) (x + k * pu)[ou] = xc.a + (zN - p.c - n.b + p.b);
      if (unk<1>(G, j)) (x + k * pv)[ov] = xc.b + (n.a - p.a - zE + p.c);
      if (unk<2>(G, k)) (x + k * pw)[ow] = xc.c + (yE - p.b - xN + p.a);
    }
    s ^= 1;
    if (slot) P[s][0][ly][lx] = n.a, P[s][1][ly][lx] = n.b, P[s][2][ly][lx] = n.c;
    p = n;
    __syncthreads();
  }
}

// planes per block: as many as leave about two rounds of blocks
inline dim3 edge_grid(const Grid& g, int* kz) {
  const int gx = (g.n[0] + kEdgeX - 2) / (kEdgeX - 1), gy = (g.n[1] + kEdgeY - 2) / (kEdgeY - 1);
  *kz = 16;
  while (*kz > 2 && gx * gy * ((g.n[2] + *kz - 1) / *kz) < 1024) *kz /= 2;
  return dim3(gx, gy, (g.n[2] + *kz - 1) / *kz);
}

// probe for diag(C^T W C): psi = 1 on the edges of component a whose point is
// congruent to (cx, cy, cz) modulo 3 and not in a wall, 0 elsewhere.  Two
// such edges are three points apart along some axis, so their curls touch
// faces that W does not couple.
template <int DIM>
__global__ __launch_bounds__(kBlock) void k_edge_probe(Grid G, int a, int cx, int cy, int cz,
                                                       double* __restrict__ psi) {
  const int k = blockIdx.z;
  const int idx = blockIdx.x * kBlock + threadIdx.x;
  if (idx >= G.n[0] * G.n[1]) return;
  const int j = idx / G.n[0], i = idx - j * G.n[0];
  const long nc = G.n_cells;
  const long p = (long)k * G.n[0] * G.n[1] + idx;
  for (int b = 0; b < edge_comps<DIM>(); ++b) {
    const bool on = b == a && i % 3 == cx && j % 3 == cy && (DIM == 2 || k % 3 == cz) &&
                    !edge_in_wall<DIM>(G, b, i, j, k);
    psi[b * nc + p] = on ? 1.0 : 0.0;
  }
}

// diag[e] = t[e] on the probed edges (psi[e] != 0)
__global__ __launch_bounds__(kBlock) void k_edge_collect(long n, const double* __restrict__ psi,
                                                         const double* __restrict__ t,
                                                         double* __restrict__ diag) {
  for (long e = (long)blockIdx.x * kBlock + threadIdx.x; e < n; e += (long)gridDim.x * kBlock)
    if (psi[e] != 0.0) diag[e] = t[e];
}

}  // namespace gkb

// What the fused V-cycle legs (legs.hip, march.hip) share on the device.
//
// Site (i, j, k) is the cell with its lower faces u, v, w; the upper boundary
// faces of the grid are sites one past the last cell.
#pragma once
#include "legs.hpp"

namespace gkb {

// component c has a face at (i, j, k), and it is an unknown
__device__ __forceinline__ bool in_array(const Grid& G, int c, int i, int j, int k) {
  return unsigned(i) < unsigned(G.ext[c][0]) && unsigned(j) < unsigned(G.ext[c][1]) &&
         unsigned(k) < unsigned(G.ext[c][2]);
}
// bits 0 .. 2: the face of that component at (i, j, k) is an unknown (in the
// array, and not normal to a DIRICHLET side it lies on)
template <int DIM>
__device__ __forceinline__ unsigned unknown_bits(const Grid& G, int i, int j, int k) {
  const int P[3] = {i, j, k};
  bool cell[3], nrm[3];
#pragma unroll
  for (int a = 0; a < DIM; ++a) {
    const int lo = G.bc[2 * a] == kDir ? 1 : 0, hi = G.n[a] + (G.bc[2 * a + 1] == kDir ? 0 : 1);
    cell[a] = unsigned(P[a]) < unsigned(G.n[a]);
    nrm[a] = unsigned(P[a] - lo) < unsigned(hi - lo);
  }
  if (DIM == 2) return unsigned(nrm[0] && cell[1]) | unsigned(cell[0] && nrm[1]) << 1;
  return unsigned(nrm[0] && cell[1] && cell[2]) | unsigned(cell[0] && nrm[1] && cell[2]) << 1 |
         unsigned(cell[0] && cell[1] && nrm[2]) << 2;
}
__device__ __forceinline__ int face(const Grid& G, int c, int i, int j, int k) {
  return G.off[c] + (k * G.ext[c][1] + j) * G.ext[c][0] + i;
}
__device__ __forceinline__ bool cell_in(const Grid& G, int i, int j, int k) {
  return unsigned(i) < unsigned(G.n[0]) && unsigned(j) < unsigned(G.n[1]) &&
         unsigned(k) < unsigned(G.n[2]);
}
__device__ __forceinline__ bool cell_on(const Grid& G, int i, int j, int k) {
  return cell_in(G, i, j, k) && cidx(G, i, j, k) != G.pin;
}

// SMOOTH: weight of the covering coarse row of fine row t: 3/4, with the
// mirror ghost of the missing neighbour folded in at a side
template <typename T>
__device__ __forceinline__ T cover_weight(int t, int nc, int lo, int hi) {
  T w = T(0.75);
  if (t == 0) w += lo == kDir ? T(-0.25) : T(0.25);
  if (t == 2 * nc - 1) w += hi == kDir ? T(-0.25) : T(0.25);
  return w;
}

}  // namespace gkb

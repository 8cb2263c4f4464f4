// Fused V-cycle legs: everything a level does on the way down (pre-smoothing
// from a zero guess, residual, restriction) in one kernel, and everything on
// the way up (prolongation, post-smoothing) in another.  Launch interface of
// legs.hip.
#pragma once
#include "common.hpp"

namespace gkb {

// how a level's legs are launched; tile 0: not fused
struct LegPlan {
  int tile = 0;
  dim3 grid;
  int nblocks = 0;  // partials of the dot product that the way up can form
  int tz = 0;       // planes per block of the marching legs
};

// plan of a level: size of an element in bytes, hybrid or Jacobi smoother
LegPlan leg_plan(const Grid& g, bool hybrid, int elem);

// The marching legs (march.hip) of large 3D levels with the Jacobi smoother and
// constant viscosity; they take no folded convergence test
constexpr int kMarchWide = 16, kMarchSquare = 17;
inline bool marches(const LegPlan& p) { return p.tile >= kMarchWide; }
LegPlan march_plan(const Grid& g, int elem, bool smooth);

// Planes per block of a march over nz planes by `columns` blocks per plane
// (even: a chunk starts on a coarse plane).  A block has a compute unit for
// itself, and a chunk costs about 9 planes more than it has, so the shortest sum
// of rounds is taken; four planes are the least, also where a grid has fewer.
inline int march_planes(int columns, int nz) {
  int best_tz = 4;
  long best = -1;
  for (int tz = 4; tz < nz + 2; tz += 2) {
    const int chunks = (nz + tz - 1) / tz;
    const long cost = ((long)columns * chunks + 255) / 256 * (tz + 9);
    if (best < 0 || cost < best) {
      best = cost;
      best_tz = tz;
    }
  }
  return best_tz;
}

// what both legs read of a level
template <typename T>
struct LegLevel {
  Op<T> op;
  Grid gc;            // next coarser grid
  const T* dinv;      // 1 / diag(M), 0 at faces that are not unknowns
  const T* edinv;     // 1 / diag(C^T W C) of the edge sweeps (hybrid)
  T omega, omega_e;
  int smooth;         // SMOOTH transfers (else DIV)
};

// the product of a PCG iteration whose scalar steps are folded (common.hpp):
// p' = z + beta p with beta from the nrz partials of r.z, q = M p', partials
// of p'.q; p and pn must not overlap
LegPlan apply_plan(const Grid& g);
template <typename T>
void leg_apply(hipStream_t s, const LegPlan& plan, const Op<T>& op, const T* z, const T* p, T* q,
               T* pn, double* part_pq, PcgState* st, const double* part_rz, int nrz);

// partials of r.r whose convergence test is folded into the way down
struct FoldCheck {
  PcgState* st = nullptr;
  const double* part = nullptr;
  int n = 0;
};

// xo = the pre-smoothed iterate from a zero guess (two Jacobi sweeps, or one
// with an edge sweep), bc = R (b - M xo); x0c (optional): the first sweep
// from a zero guess on the coarse level, omega_c dinv_c bc
template <typename T>
void leg_down(hipStream_t s, const LegPlan& plan, const LegLevel<T>& L, const T* b, T* xo, T* bc,
              const T* dinv_c, T omega_c, T* x0c, const PcgState* st,
              const FoldCheck& check = FoldCheck());

// xo = the post-smoothed iterate from xi + P ec; partial (optional): block
// partials of b . xo.  xi and xo must not overlap.
template <typename T>
void leg_up(hipStream_t s, const LegPlan& plan, const LegLevel<T>& L, const T* ec, const T* xi,
            const T* b, T* xo, double* partial, const PcgState* st);

template <typename T>
void march_down(hipStream_t s, const LegPlan& plan, const LegLevel<T>& L, const T* b, T* xo, T* bc,
                const T* dinv_c, T omega_c, T* x0c, const PcgState* st);
template <typename T>
void march_up(hipStream_t s, const LegPlan& plan, const LegLevel<T>& L, const T* ec, const T* xi,
              const T* b, T* xo, double* partial, const PcgState* st);

}  // namespace gkb

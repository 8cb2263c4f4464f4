// Restarted flexible GMRES for the inner systems M x = f (right
// preconditioned: the Krylov basis V is built from M z_j with z_j = P(v_j),
// and the correction is formed from the stored z_j, so P may be any fixed or
// varying preconditioner; Saad's flexible variant of GMRES).  The paper
// leaves the inner Krylov method open (Section 3) and compares CG with
// fgmres (Section 4.1.3).
//
// GPU design: the basis is orthogonalised by classical Gram-Schmidt applied
// twice (every coefficient of one pass comes from one multi-vector dot
// kernel, so a step costs a fixed number of launches however long the basis
// is, and the second pass restores the orthogonality one pass loses).  The
// Hessenberg matrix, the Givens rotations and the least-squares right-hand
// side live on the device in FP64, so a whole restart cycle is captured in
// one HIP graph and the host looks at the state once per cycle.  Two flags
// steer the early exits: the solve's PcgState (done for good) and a cycle
// state whose `done` ends the Arnoldi steps of the current cycle (converged,
// breakdown, iteration cap, or the cycle is full).
//
// A step on systems of up to about 200k unknowns is bound by its launches and
// by the trips to memory inside each, so it is four kernels: the next basis
// vector with its preconditioned form (and A^T of it on an assembled system),
// the product with the first pass's dots, the first pass with the second
// pass's dots, the second pass with the norm.  No scalar kernel stands
// between them: every block sums the (at most kGmFold) partials of the
// kernel before, in the same order, and block 0 keeps the coefficients and
// turns the rotations.  On 24^3 cells (40k rows, Jacobi, restart 30) an inner
// solve takes 4.2 ms; as eleven kernels per step, the coefficient sums
// one after the other in a one-block kernel (13 us) and four rows per thread,
// it took 17.4 ms.
#pragma once
#include "csr.hpp"

namespace gkb {

constexpr int kGmMaxRestart = 64;  // Krylov vectors per cycle (bound of the option)
// Partials that every block of the next kernel sums by itself.  At most four
// rows per thread keep the blocks of a folded step short; above that a step
// streams the basis from memory, the blocks are more, and one extra kernel
// sums their partials (k_gm_sums).
constexpr int kGmFold = 192;
constexpr int kGmFoldRows = 4 * kGmFold * kBlock;
inline bool gm_folded(int n) { return n <= kGmFoldRows; }
inline int gm_blocks(int n) {
  const int rows = gm_folded(n) ? kBlock : 4 * kBlock, cap = gm_folded(n) ? kGmFold : 4096;
  const int b = (n - 1) / rows + 1;
  return n < 1 ? 1 : b < cap ? b : cap;
}

struct FgmState {
  // R[j][i]: row i of rotated column j; before that, of the first pass's
  // coefficients
  double R[kGmMaxRestart][kGmMaxRestart];
  double cs[kGmMaxRestart], sn[kGmMaxRestart];  // Givens rotations
  double g[kGmMaxRestart];                      // rotated least-squares rhs, then the
                                                // solution y of the triangular system
  double gam[kGmMaxRestart + 1];                // its last entry after j steps
  double h[kGmMaxRestart];                      // coefficients of the second pass
  double beta;                                  // ||r|| at the start of the cycle
  int it0;                                      // steps before this cycle
  int k;                                        // completed Arnoldi steps of the cycle
  int conv;                                     // residual estimate met the tolerance
};

// ------------------------------------------------------ coefficients

// Wave sums of Q values (a power of two, 2 .. 16) at once: in each step a
// lane keeps half of its values and hands the other half over, so 64 lanes
// take Q - 1 + log2(64 / Q) exchanges instead of 6 Q.  The sum of value q ends
// in the lanes with lane / (64 / Q) == q.
template <int Q>
__device__ __forceinline__ double wave_sums(double* s) {
  const int lane = threadIdx.x & 63;
  int o = 32;
#pragma unroll
  for (int n = Q / 2; n >= 1; n /= 2) {
    const bool up = lane & o;
#pragma unroll
    for (int q = 0; q < n; ++q) {
      const double keep = up ? s[q + n] : s[q], give = up ? s[q] : s[q + n];
      s[q] = keep + __shfl_xor(give, o, 64);
    }
    o >>= 1;
  }
  for (; o > 0; o >>= 1) s[0] += __shfl_xor(s[0], o, 64);
  return s[0];
}

// block partials of the nv <= Q sums s[] to part[k * gridDim.x + block]:
// through LDS, kBlock / Q threads per sum (lane exchanges alone, 31 of two
// words at Q = 32, took 5.5 us of a 10.9 us kernel)
template <int Q>
__device__ __forceinline__ void put_sums(const double* s, int nv, double* __restrict__ part) {
  constexpr int kT = kBlock / Q;
  __shared__ double sh[Q][kBlock + 8];
#pragma unroll
  for (int q = 0; q < Q; ++q)
    if (q < nv) sh[q][threadIdx.x] = s[q];
  __syncthreads();
  const int k = threadIdx.x / kT, e = threadIdx.x % kT;
  double v = 0.0;
  if (k < nv)
#pragma unroll
    for (int m = 0; m < Q; ++m) v += sh[k][e + kT * m];
#pragma unroll
  for (int o = kT / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  if (k < nv && e == 0) part[(long)k * gridDim.x + blockIdx.x] = v;
}

// the nv <= Q sums of nb <= kGmFold partials each, to hs in LDS, the same
// bits in every block: Q / 4 sums per wave, all their loads in flight together
// (one sum after the other paid a trip to memory for each: 14.9 us per pass
// kernel at nv = 17 .. 30 against 10.9)
template <int Q>
__device__ __forceinline__ void get_sums(const double* __restrict__ part, int nb, int nv,
                                         double* hs) {
  constexpr int kPer = Q / (kBlock / 64), kLanes = 64 / kPer;
  const int lane = threadIdx.x & 63, k0 = (threadIdx.x >> 6) * kPer;
  double v[kPer][kGmFold / 64];
#pragma unroll
  for (int q = 0; q < kPer; ++q)
#pragma unroll
    for (int b = 0; b < kGmFold / 64; ++b) {
      const bool in = k0 + q < nv && lane + 64 * b < nb;
      v[q][b] = in ? part[(long)(k0 + q) * nb + lane + 64 * b] : 0.0;
    }
  double s[kPer];
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    s[q] = v[q][0];
#pragma unroll
    for (int b = 1; b < kGmFold / 64; ++b) s[q] += v[q][b];
  }
  const double t = wave_sums<kPer>(s);
  if (lane % kLanes == 0) hs[k0 + lane / kLanes] = t;
  __syncthreads();
}

// sums of more than kGmFold partials each, one block per sum: they take the
// place of the partials (one per sum)
__global__ __launch_bounds__(kFinal) void k_gm_sums(const PcgState* cyc, double* sums,
                                                    const double* part, int nb) {
  if (cyc->done) return;
  __shared__ double sh[kFinal / 64];
  const double v = sum_partials(part + (long)blockIdx.x * nb, nb, sh);
  if (threadIdx.x == 0) sums[blockIdx.x] = v;
}

// ------------------------------------------------------- Arnoldi steps

// End of Arnoldi step j (one block): column j of the Hessenberg matrix from
// the two passes, hn = H[j+1][j] = ||w||, the earlier rotations applied to
// it, a new rotation that zeroes hn, the rotated right-hand side and its last
// entry |gam[j+1]| = the residual norm of the least-squares solution; the
// cycle ends on convergence, breakdown, the iteration cap or a full basis
__device__ __forceinline__ void gm_step_end(PcgState* st, PcgState* cyc, FgmState* fs, double hn,
                                            int j, bool last) {
  __shared__ double col[kGmMaxRestart], cs[kGmMaxRestart], sn[kGmMaxRestart];
  if (threadIdx.x <= j) {
    col[threadIdx.x] = fs->R[j][threadIdx.x] + fs->h[threadIdx.x];
    cs[threadIdx.x] = fs->cs[threadIdx.x];
    sn[threadIdx.x] = fs->sn[threadIdx.x];
  }
  __syncthreads();
  if (threadIdx.x != 0) return;
  double a = col[0];
  for (int i = 0; i < j; ++i) {
    const double b = col[i + 1];
    fs->R[j][i] = cs[i] * a + sn[i] * b;
    a = -sn[i] * a + cs[i] * b;
  }
  const double rr = sqrt(a * a + hn * hn);
  st->it += 1;
  if (rr == 0.0) {
    // M z_j adds nothing to the basis: the step is dropped, the cycle ends
    // and the next one restarts from the true residual
    fs->k = j;
    cyc->done = 1;
    return;
  }
  const double c = a / rr, s = hn / rr, gam = fs->gam[j], res = -s * gam;
  fs->cs[j] = c;
  fs->sn[j] = s;
  fs->R[j][j] = rr;
  fs->g[j] = c * gam;
  fs->gam[j + 1] = res;
  fs->k = j + 1;
  const double res2 = res * res;
  if (!isfinite(res2) || !isfinite(rr)) {
    st->nonfinite = 1;
    st->status = -4;
    cyc->done = 1;
    return;
  }
  if (res2 <= st->tol2 * st->rr0 || hn == 0.0) {
    fs->conv = 1;
    cyc->done = 1;
  } else if (fs->it0 + j + 1 >= st->maxit || last) {
    cyc->done = 1;
  }
}

// Start of step j: step j - 1 ends (block 0), v_j = w / ||w|| (w: the second
// pass's result with nb partials of w.w; j = 0: w = r and ||w|| = beta).  With
// dinv also z_j = D^-1 v_j, and with t (assembled system) t = A'^T z_j, formed
// from w, so that the product needs no kernel in between.  Blocks that
// start after block 0 ended the cycle leave their part of v_j unwritten (all
// waves of a block or none); no kernel reads it then.
template <typename T>
__global__ __launch_bounds__(kBlock) void k_gm_next(int n, PcgState* st, PcgState* cyc,
                                                    FgmState* fs, const double* __restrict__ part,
                                                    int nb, int j, const T* __restrict__ w,
                                                    T* __restrict__ v, const T* __restrict__ dinv,
                                                    T* __restrict__ z, CsrOps<T> o,
                                                    T* __restrict__ t) {
  __shared__ FoldShared<kBlock> fold;
  const int done = cyc->done;
  if (done && j == 0) return;
  const int i0 = blockIdx.x * kBlock + threadIdx.x, step = gridDim.x * kBlock;
  auto at = [&](int k) { return csr_at_row(o, k, [&](int i) { return dinv[i] * w[i]; }); };
  T wi = T(0), di = T(0), ti = T(0);
  double share = 0.0;
  if (!done) {
    // the first entries are fetched beside the partials
    if (i0 < n) wi = w[i0];
    if (dinv && i0 < n) di = dinv[i0];
    if (t && i0 < o.n) ti = at(i0);
    if (j > 0) share = fold_share<kBlock>(part, nb);
  }
  double hn = fs->beta;
  if (j > 0) {
    double ww;
    if (!fold_sum_if<kBlock>(done, share, fold, ww)) return;
    hn = sqrt(ww);
    if (blockIdx.x == 0) gm_step_end(st, cyc, fs, hn, j - 1, false);
  }
  const T s = T(1.0 / hn);
  for (int i = i0; i < n; i += step) {
    if (i != i0) {
      wi = w[i];
      if (dinv) di = dinv[i];
    }
    const T vi = wi * s;
    v[i] = vi;
    if (dinv) z[i] = di * vi;
  }
  if (t)
    for (int k = i0; k < o.n; k += step) t[k] = s * (k == i0 ? ti : at(k));
}

// partials of V_k . w for the nv <= Q basis vectors, layout
// part[k * gridDim.x + block]
template <typename T, int Q>
__global__ __launch_bounds__(kBlock) void k_gm_dots(int n, const PcgState* __restrict__ cyc,
                                                    const T* __restrict__ V, long ldv, int nv,
                                                    const T* __restrict__ w,
                                                    double* __restrict__ part) {
  if (cyc->done) return;
  double s[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q) s[q] = 0.0;
  for (int i = blockIdx.x * kBlock + threadIdx.x; i < n; i += gridDim.x * kBlock) {
    const double wi = double(w[i]);
#pragma unroll
    for (int q = 0; q < Q; ++q)
      if (q < nv) s[q] += double(V[q * ldv + i]) * wi;
  }
  put_sums<Q>(s, nv, part);
}

// the same with the product of an assembled system: w = M z (t = A'^T z
// given)
template <typename T, int Q>
__global__ __launch_bounds__(kBlock) void k_gm_csr_dots(CsrOps<T> o, T eta,
                                                        const PcgState* __restrict__ cyc,
                                                        const T* __restrict__ z,
                                                        const T* __restrict__ t,
                                                        const T* __restrict__ V, long ldv, int nv,
                                                        T* __restrict__ w,
                                                        double* __restrict__ part) {
  if (cyc->done) return;
  double s[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q) s[q] = 0.0;
  for (int i = blockIdx.x * kBlock + threadIdx.x; i < o.m; i += gridDim.x * kBlock) {
    T v[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) v[q] = q < nv ? V[q * ldv + i] : T(0);
    const T wt = csr_M_row<T>(o, eta, z, t, i);
    w[i] = wt;
    const double wi = double(wt);
#pragma unroll
    for (int q = 0; q < Q; ++q)
      if (q < nv) s[q] += double(v[q]) * wi;
  }
  put_sums<Q>(s, nv, part);
}

// One Gram-Schmidt pass over the nv <= Q basis vectors: h from the nb
// partials per vector, wo = w - sum_k h_k V_k; partials of V_k . wo (pass 0, wo
// may be w) or of wo.wo (pass 1) to part_out
template <typename T, int Q, int PASS>
__global__ __launch_bounds__(kBlock) void k_gm_pass(int n, const PcgState* __restrict__ cyc,
                                                    FgmState* fs, const T* __restrict__ V,
                                                    long ldv, int nv,
                                                    const double* __restrict__ part, int nb,
                                                    const T* w, T* wo,
                                                    double* __restrict__ part_out) {
  if (cyc->done) return;
  __shared__ double hs[Q];
  double s[PASS == 0 ? Q : 1];
#pragma unroll
  for (int q = 0; q < (PASS == 0 ? Q : 1); ++q) s[q] = 0.0;
  const int i0 = blockIdx.x * kBlock + threadIdx.x;
  T v[Q];
  T wi = T(0);
  auto fetch = [&](int i) {
    wi = w[i];
#pragma unroll
    for (int q = 0; q < Q; ++q) v[q] = q < nv ? V[q * ldv + i] : T(0);
  };
  if (i0 < n) fetch(i0);  // in flight beside the partials
  get_sums<Q>(part, nb, nv, hs);
  if (blockIdx.x == 0 && threadIdx.x < nv)
    (PASS == 0 ? fs->R[nv - 1] : fs->h)[threadIdx.x] = hs[threadIdx.x];
  for (int i = i0; i < n; i += gridDim.x * kBlock) {
    if (i != i0) fetch(i);
    double x = double(wi);
#pragma unroll
    for (int q = 0; q < Q; ++q)
      if (q < nv) x -= hs[q] * double(v[q]);
    const T xt = T(x);
    wo[i] = xt;
    x = double(xt);
    if (PASS == 0) {
#pragma unroll
      for (int q = 0; q < Q; ++q)
        if (q < nv) s[q] += double(v[q]) * x;
    } else {
      s[0] += x * x;
    }
  }
  if constexpr (PASS == 0) {
    put_sums<Q>(s, nv, part_out);
  } else {
    __shared__ double sh[kBlock / 64];
    const double ww = block_sum<kBlock>(s[0], sh);
    if (threadIdx.x == 0) part_out[blockIdx.x] = ww;
  }
}

// ------------------------------------------------------ cycle end, start

// End of a cycle (one block): a full basis's last step ends, then R y = g by
// back substitution over the k steps of the cycle, a lane per row
__global__ __launch_bounds__(kBlock) void k_gm_finish(PcgState* st, PcgState* cyc, FgmState* fs,
                                                      const double* part, int nb, int restart) {
  if (st->done) return;
  __shared__ double R[kGmMaxRestart * (kGmMaxRestart + 1)], sh[kBlock / 64];
  if (!cyc->done) {
    const double hn = sqrt(fold_sum<kBlock>(fold_share<kBlock>(part, nb), sh));
    gm_step_end(st, cyc, fs, hn, restart - 1, true);
  }
  __syncthreads();
  const int k = fs->k;
  for (int e = threadIdx.x; e < k * k; e += kBlock) {
    const int c = e / k, r = e - c * k;
    if (r <= c) R[c * (kGmMaxRestart + 1) + r] = fs->R[c][r];
  }
  __syncthreads();
  const int lane = threadIdx.x;
  if (lane >= 64) return;
  double g = lane < k ? fs->g[lane] : 0.0;
  for (int c = k - 1; c >= 0; --c) {
    const double* Rc = R + c * (kGmMaxRestart + 1);
    const double y = __shfl(g, c, 64) / Rc[c];
    if (lane == c) g = y;
    else if (lane < c) g -= Rc[lane] * y;
  }
  if (lane < k) fs->g[lane] = g;
}

// x += sum_{i<k} y_i z_i
template <typename T>
__global__ __launch_bounds__(kBlock) void k_gm_update_x(int n, const PcgState* __restrict__ st,
                                                        const FgmState* __restrict__ fs,
                                                        const T* __restrict__ Z, long ldz,
                                                        T* __restrict__ x) {
  if (st->done) return;
  const int k = fs->k;
  for (int i = blockIdx.x * kBlock + threadIdx.x; i < n; i += gridDim.x * kBlock) {
    double xi = double(x[i]);
#pragma unroll 8
    for (int l = 0; l < k; ++l) xi += fs->g[l] * double(Z[l * ldz + i]);
    x[i] = T(xi);
  }
}

// start of a cycle from r (partials of r.r): beta = ||r||, g = beta e_1.
// first = 1 also initialises the solve's state (rr0 = f.f, tolerance,
// iteration cap).  At a restart the recomputed residual decides: done when
// it meets the tolerance (also where the least-squares estimate of the last
// cycle already did: near rounding level the two part), else done with
// status -5 once the iteration cap is reached.  accept_estimate = 1 (FP32
// inner solves) also ends the solve when the last cycle's least-squares
// estimate met the tolerance: that estimate plays the part of CG's
// recursive residual, while f - M x formed in FP32 has a rounding floor
// of about eps_32 |M| |x| / |f|, which on grad-div dominated M (eta >> mu)
// lies above the loose inner tolerances of the mixed-precision solver; the
// FP64 defect correction around the inner solves removes what is left
__global__ __launch_bounds__(kFinal) void k_gm_start(PcgState* st, PcgState* cyc, FgmState* fs,
                                                     const double* part_rr, int nrr, double tol,
                                                     int maxit, int first, int accept_estimate) {
  if (!first && st->done) return;
  __shared__ double sh[kFinal / 64];
  const double rr = sum_partials(part_rr, nrr, sh);
  if (threadIdx.x != 0) return;
  if (first) {
    st->rr0 = rr;
    st->tol2 = tol * tol;
    st->it = 0;
    st->maxit = maxit;
    st->nonfinite = 0;
    st->status = 0;
    st->done = rr == 0.0 ? 1 : 0;
  } else if (st->nonfinite || !isfinite(rr)) {
    st->nonfinite = 1;
    st->status = -4;
    st->done = 1;
  } else if (rr <= st->tol2 * st->rr0 || (accept_estimate && fs->conv)) {
    st->done = 1;
    st->status = 0;
  } else if (st->it >= st->maxit) {
    st->done = 1;
    st->status = -5;
  }
  st->rr = rr;
  fs->beta = sqrt(rr);
  fs->gam[0] = fs->beta;
  fs->it0 = st->it;
  fs->k = 0;
  fs->conv = 0;
  cyc->done = st->done;
}

}  // namespace gkb

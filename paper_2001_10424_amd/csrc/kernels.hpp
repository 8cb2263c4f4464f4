// HIP kernels for gfx950: MAC operators with fused reductions, BLAS-1
// updates of the GKB recurrence and of PCG, multigrid transfers and the dense
// FP64 coarsest-grid solve.
#pragma once
#include <hip/hip_runtime.h>

#include "common.hpp"

namespace gkb {

__global__ __launch_bounds__(kFinal) void k_sum_partials(const double* part, int n, double* out) {
  __shared__ double sh[kFinal / 64];
  double s = sum_partials(part, n, sh);
  if (threadIdx.x == 0) *out = s;
}

// ------------------------------------------------- face-operator kernels

enum MMode {
  kApply = 0,      // y = M x
  kApplyDot = 1,   // y = M x, partial x.y
  kJacobi = 2,     // y = x + omega (b - M x) / D
  kJacobiDot = 3,  // y = x + omega (b - M x) / D, partial b.y
  kResid = 4,      // y = b - M x
  kDinvM = 5,      // y = (M x) / D, partial y.y
  kJacobi0 = 6,    // y = omega b / D   (first sweep from a zero guess)
  kDiag = 7,       // y = D
  kResidDot = 8,   // y = b - M x, partial y.y
  kJacobiZ = 9,    // two sweeps from a zero guess: y = x1 + omega (b - M x1) / D
                   // with x1 = omega b / D (x1 formed while staging; tiled
                   // kernel, constant viscosity only; x = b)
  kJacobiP = 10,   // sweep after the coarse-grid correction: y = x' + omega
                   // (b - M x') / D with x' = x + P e (prolongation of the
                   // coarse correction e added while staging; tiled kernel)
  kApplyDotP = 11  // CG direction update and product in one pass: p' = x + beta
                   // p (x = z, b = p, beta from the PCG state) formed while
                   // staging, y = M p', p' written to y2, partial p'.y
};

// Thread mapping: blockIdx.z = component * zchunks + z-chunk; each block
// covers kBlock consecutive (x fastest) faces of one z-plane of that
// component's array and loops over kz consecutive planes.
template <typename T, int DIM, bool VARMU, int MODE, int C>
__device__ __forceinline__ double face_op(const Op<T>& op, const T* __restrict__ x,
                                          const T* __restrict__ b, T* __restrict__ y, T omega,
                                          int idx, int k0, int kz) {
  const Grid& G = op.g;
  const int e0 = G.ext[C][0], e1 = G.ext[C][1], e2 = G.ext[C][2];
  double part = 0.0;
  if (idx >= e0 * e1) return part;
  const int j = idx / e0, i = idx - j * e0;
  const int ic_fixed = C == 0 ? i : (C == 1 ? j : -1);
  for (int k = k0; k < k0 + kz && k < e2; ++k) {
    const int ic = C == 2 ? k : ic_fixed;
    const int f = fidx<C>(G, i, j, k);
    if (!unk<C>(G, ic)) {
      y[f] = T(0);
      continue;
    }
    if (MODE == kJacobi0 || MODE == kDiag) {
      const T d = diag_M<T, DIM, VARMU, C>(op, i, j, k);
      y[f] = MODE == kDiag ? d : omega * b[f] / d;
      continue;
    }
    T mx, d;
    stencil_M<T, DIM, VARMU, C>(op, x, i, j, k, mx, d);
    T out;
    if (MODE == kApply || MODE == kApplyDot) {
      out = mx;
      if (MODE == kApplyDot) part += double(x[f]) * double(out);
    } else if (MODE == kJacobi || MODE == kJacobiDot) {
      const T bf = b[f];
      out = x[f] + omega * (bf - mx) / d;
      if (MODE == kJacobiDot) part += double(bf) * double(out);
    } else if (MODE == kResid || MODE == kResidDot) {
      out = b[f] - mx;
      if (MODE == kResidDot) part += double(out) * double(out);
    } else {  // kDinvM
      out = mx / d;
      part += double(out) * double(out);
    }
    y[f] = out;
  }
  return part;
}

template <typename T, int DIM, bool VARMU, int MODE>
__global__ __launch_bounds__(kBlock) void k_face_op(Op<T> op, const T* __restrict__ x,
                                                    const T* __restrict__ b, T* __restrict__ y,
                                                    T omega, int kz, int zchunks,
                                                    double* __restrict__ partial,
                                                    const PcgState* __restrict__ st) {
  if (st && st->done) return;
  const int c = blockIdx.z / zchunks;
  const int k0 = (blockIdx.z - c * zchunks) * kz;
  const int idx = blockIdx.x * kBlock + threadIdx.x;
  double part = 0.0;
  if (c == 0) part = face_op<T, DIM, VARMU, MODE, 0>(op, x, b, y, omega, idx, k0, kz);
  else if (c == 1) part = face_op<T, DIM, VARMU, MODE, 1>(op, x, b, y, omega, idx, k0, kz);
  else if (DIM == 3) part = face_op<T, DIM, VARMU, MODE, 2>(op, x, b, y, omega, idx, k0, kz);
  constexpr bool kRed = MODE == kApplyDot || MODE == kJacobiDot || MODE == kDinvM || MODE == kResidDot;
  if (kRed) {
    __shared__ double sh[kBlock / 64];
    double s = block_sum<kBlock>(part, sh);
    if (threadIdx.x == 0) partial[blockIdx.z * gridDim.x + blockIdx.x] = s;
  }
}

// out = s1 * (A q) + s2 * yv on unknown faces (yv may be null), 0 elsewhere
template <typename T, int C>
__device__ __forceinline__ void grad_face(const Grid& G, const T* __restrict__ q,
                                          const double* __restrict__ yv, double s1, double s2,
                                          double ih, double* __restrict__ out, int idx, int k0,
                                          int kz) {
  const int e0 = G.ext[C][0], e1 = G.ext[C][1], e2 = G.ext[C][2];
  if (idx >= e0 * e1) return;
  const int j = idx / e0, i = idx - j * e0;
  for (int k = k0; k < k0 + kz && k < e2; ++k) {
    const int ic = C == 0 ? i : (C == 1 ? j : k);
    const int f = fidx<C>(G, i, j, k);
    if (!unk<C>(G, ic)) {
      out[f] = 0.0;
      continue;
    }
    double v = s1 * double(grad_f<C>(G, q, i, j, k)) * ih;
    if (yv) v += s2 * yv[f];
    out[f] = v;
  }
}

template <int DIM>
__global__ __launch_bounds__(kBlock) void k_grad_axpy(Grid G, const double* __restrict__ q,
                                                      const double* __restrict__ yv, double s1,
                                                      double s2, double* __restrict__ out, int kz,
                                                      int zchunks) {
  const int c = blockIdx.z / zchunks;
  const int k0 = (blockIdx.z - c * zchunks) * kz;
  const int idx = blockIdx.x * kBlock + threadIdx.x;
  const double ih = 1.0 / G.h;
  if (c == 0) grad_face<double, 0>(G, q, yv, s1, s2, ih, out, idx, k0, kz);
  else if (c == 1) grad_face<double, 1>(G, q, yv, s1, s2, ih, out, idx, k0, kz);
  else if (DIM == 3) grad_face<double, 2>(G, q, yv, s1, s2, ih, out, idx, k0, kz);
}

// t = s1 * (A^T x) + s2 * z on unpinned cells (z may be null), 0 at the pin;
// partial t.t and, if zz_partial, z.z over unpinned cells
template <typename T, int DIM>
__global__ __launch_bounds__(kBlock) void k_div_axpy(Grid G, const T* __restrict__ x,
                                                     const T* __restrict__ z, double s1, double s2,
                                                     T* __restrict__ t, double* __restrict__ partial,
                                                     double* __restrict__ zz_partial) {
  const int nxy = G.n[0] * G.n[1];
  const int k = blockIdx.z;
  const int idx = blockIdx.x * kBlock + threadIdx.x;
  double a = 0.0, bz = 0.0;
  if (idx < nxy) {
    const int j = idx / G.n[0], i = idx - j * G.n[0];
    const int cc = cidx(G, i, j, k);
    double v = 0.0;
    if (cc != G.pin) {
      v = s1 * double(cdiv<DIM>(G, x, i, j, k)) / G.h;
      if (z) {
        const double zv = double(z[cc]);
        v += s2 * zv;
        bz = zv * zv;
      }
    }
    t[cc] = T(v);
    a = v * v;
  }
  __shared__ double sh[kBlock / 64];
  double s = block_sum<kBlock>(a, sh);
  if (threadIdx.x == 0 && partial) partial[blockIdx.z * gridDim.x + blockIdx.x] = s;
  if (zz_partial) {
    __syncthreads();
    double s2v = block_sum<kBlock>(bz, sh);
    if (threadIdx.x == 0) zz_partial[blockIdx.z * gridDim.x + blockIdx.x] = s2v;
  }
}

// ------------------------------------------------------ saddle residual

// one neighbour of the viscous stencil: inside the array kap (xf - xn), across
// a wall the mirror ghost 2 kap xf, else (do-nothing side) 0
__device__ __forceinline__ double visc_side(bool in, bool wall, double kap, double xf, double xn) {
  return in ? kap * (xf - xn) : (wall ? 2.0 * kap * xf : 0.0);
}

constexpr int kSaddleBlock = 512;

// FP64 saddle residual in one pass: res_w = g - W w - A p on the unknown faces
// (0 elsewhere, may be null), res_r = r - A^T w on the cells (0 at the pin; may
// be null);
// partials of res_w.res_w, g.g (unknown faces), res_r.res_r, r.r (unpinned
// cells) to part[0 .. 3][block].
//
// Bound by memory: at least g, w, p, r read and both results written.  A
// thread owns the column (i, j) of lower faces and cells and marches kz planes
// up, the plane below and the next one in registers; a block is a run of the
// flattened (nx + 1) x (ny + 1) plane, so every extent fills its waves, and
// blocks of one XCD are neighbours (rows and planes they share stay in its
// L2).  Every load is unconditional from a clamped address, so a plane's loads
// are in flight together.  128^3: 52 us (203 MB); one kernel per component
// with branches around its loads and one for the cells took 64.5 + 18.7 us.
template <int DIM, bool VARMU>
__global__ __launch_bounds__(kSaddleBlock) void k_saddle(Op<double> op,
                                                         const double* __restrict__ g,
                                                         const double* __restrict__ r,
                                                         const double* __restrict__ w,
                                                         const double* __restrict__ p,
                                                         double* __restrict__ res_w,
                                                         double* __restrict__ res_r, int kz, int bx,
                                                         double* __restrict__ p_rr,
                                                         double* __restrict__ p_gg,
                                                         double* __restrict__ p_tt,
                                                         double* __restrict__ p_zz) {
  const Grid& G = op.g;
  const int nx = G.n[0], ny = G.n[1], nz = G.n[2];
  const int nb = gridDim.x, xcd = blockIdx.x & 7;
  const int lin = xcd * (nb >> 3) + min(xcd, nb & 7) + int(blockIdx.x >> 3);
  const int k0 = (lin / bx) * kz;
  const int e = (lin % bx) * kSaddleBlock + threadIdx.x;
  const int j = e / (nx + 1), i = e - j * (nx + 1);
  const bool col = j <= ny;
  const bool cx = col && i < nx, cy = col && j < ny;  // a cell along x, along y
  auto normal = [&](int c, int q) {  // faces at index q along their normal are unknowns
    return q >= (G.bc[2 * c] == kDir ? 1 : 0) && q <= G.n[c] - (G.bc[2 * c + 1] == kDir ? 1 : 0);
  };
  const bool ux = normal(0, i), vy = normal(1, j);
  const bool lx = G.bc[0] == kDir, hx = G.bc[1] == kDir, ly = G.bc[2] == kDir, hy = G.bc[3] == kDir,
             lz = G.bc[4] == kDir, hz = G.bc[5] == kDir;
  // w at a face, 0 where it is no unknown of the array
  auto fu = [&](bool in, int ii, int jj, int kk) {
    const double v = w[in ? fidx<0>(G, ii, jj, kk) : 0];
    return in ? v : 0.0;
  };
  auto fv = [&](bool in, int ii, int jj, int kk) {
    const double v = w[in ? fidx<1>(G, ii, jj, kk) : 0];
    return in ? v : 0.0;
  };
  auto fw = [&](bool in, int ii, int jj, int kk) {
    const double v = w[in ? fidx<2>(G, ii, jj, kk) : 0];
    return in ? v : 0.0;
  };
  auto fp = [&](bool in, int ii, int jj, int kk) {
    const int q = in ? cidx(G, ii, jj, kk) : 0;
    const double v = p[q];
    return in && q != G.pin ? v : 0.0;
  };
  const double gu = (i == 0 || i == nx) ? 0.5 : 1.0, gv = (j == 0 || j == ny) ? 0.5 : 1.0;
  double rr = 0.0, gg = 0.0, tt = 0.0, zz = 0.0;
  double uB = 0.0, vB = 0.0, wB = 0.0, pB = 0.0;
  if (DIM == 3) {
    const bool in = k0 > 0;
    uB = fu(in && cy && ux, i, j, k0 - 1);
    vB = fv(in && cx && vy, i, j, k0 - 1);
    wB = fw(in && cx && cy && normal(2, k0 - 1), i, j, k0 - 1);
    pB = fp(in && cx && cy, i, j, k0 - 1);
  }
  double uC = fu(cy && ux && k0 < nz, i, j, k0), vC = fv(cx && vy && k0 < nz, i, j, k0);
  double wC = DIM == 3 ? fw(cx && cy && normal(2, k0), i, j, k0) : 0.0;
  const int k1 = min(k0 + kz, DIM == 3 ? nz + 1 : 1);
  for (int k = k0; k < k1; ++k) {
    const bool cz = k < nz, cell = cx && cy && cz;
    const bool onu = cy && cz && ux, onv = cx && cz && vy, onw = DIM == 3 && cx && cy && normal(2, k);
    const int iu = onu ? fidx<0>(G, i, j, k) : 0, iv = onv ? fidx<1>(G, i, j, k) : 0,
              iw = onw ? fidx<2>(G, i, j, k) : 0, ic = cell ? cidx(G, i, j, k) : 0;
    // the face at i + 1 counts in the divergence also where i is a wall
    const double uE = fu(cell && normal(0, i + 1), i + 1, j, k), uW = fu(onu && i > 0 && normal(0, i - 1), i - 1, j, k);
    const double vN = fv(cell && normal(1, j + 1), i, j + 1, k), vS = fv(onv && j > 0 && normal(1, j - 1), i, j - 1, k);
    const double uN = fu(onu && j < ny - 1, i, j + 1, k), uS = fu(onu && j > 0, i, j - 1, k);
    const double vE = fv(onv && i < nx - 1, i + 1, j, k), vW = fv(onv && i > 0, i - 1, j, k);
    const double pC = fp(cell, i, j, k), pW = fp(onu && i > 0, i - 1, j, k),
                 pS = fp(onv && j > 0, i, j - 1, k);
    const double gfu = g[iu], gfv = g[iv], rc = r[ic];
    double uT = 0.0, vT = 0.0, wT = 0.0, wN = 0.0, wS = 0.0, wE = 0.0, wW = 0.0, gfw = 0.0;
    if (DIM == 3) {
      uT = fu(cy && ux && k < nz - 1, i, j, k + 1);
      vT = fv(cx && vy && k < nz - 1, i, j, k + 1);
      wT = fw(cell && normal(2, k + 1), i, j, k + 1);
      wN = fw(onw && j < ny - 1, i, j + 1, k), wS = fw(onw && j > 0, i, j - 1, k);
      wE = fw(onw && i < nx - 1, i + 1, j, k), wW = fw(onw && i > 0, i - 1, j, k);
      gfw = g[iw];
    }
    // viscosities: cells C, W, S, B and the edges around the three faces
    double mC = 1.0, mW = 1.0, mS = 1.0, mB = 1.0, ez = 1.0, ezN = 1.0, ezE = 1.0, ey = 1.0,
           eyT = 1.0, eyE = 1.0, ex = 1.0, exT = 1.0, exN = 1.0;
    if (VARMU) {
      const int a = min(i, nx - 1), b = min(j, ny - 1), c = min(k, nz - 1);
      const int jv = min(j, ny);
      mC = op.mu[cidx(G, a, b, c)];
      mW = op.mu[cidx(G, max(i - 1, 0), b, c)];
      mS = op.mu[cidx(G, a, min(max(j - 1, 0), ny - 1), c)];
      ez = edge_mu<2>(op, i, jv, c), ezN = edge_mu<2>(op, i, min(j + 1, ny), c);
      ezE = edge_mu<2>(op, min(i + 1, nx), jv, c);
      if (DIM == 3) {
        mB = op.mu[cidx(G, a, b, max(k - 1, 0))];
        ey = edge_mu<1>(op, i, b, k), eyT = edge_mu<1>(op, i, b, min(k + 1, nz));
        eyE = edge_mu<1>(op, min(i + 1, nx), b, k);
        ex = edge_mu<0>(op, a, jv, k), exT = edge_mu<0>(op, a, jv, min(k + 1, nz));
        exN = edge_mu<0>(op, a, min(j + 1, ny), k);
      }
    }
    if (cy && cz) {
      double v = 0.0;
      if (ux) {
        double m = 0.0, t = 0.0;
        if (i > 0) m += mW * (uC - uW);
        if (i < nx) m += mC * (uC - uE);
        t += visc_side(j > 0, ly, ez, uC, uS);
        t += visc_side(j < ny - 1, hy, ezN, uC, uN);
        if (DIM == 3) {
          t += visc_side(k > 0, lz, ey, uC, uB);
          t += visc_side(k < nz - 1, hz, eyT, uC, uT);
        }
        v = gfu - (m + gu * t) * op.ih2 - (pC - pW) * op.ih;
        rr += v * v;
        gg += gfu * gfu;
      }
      if (res_w) res_w[fidx<0>(G, i, j, k)] = v;
    }
    if (cx && cz) {
      double v = 0.0;
      if (vy) {
        double m = 0.0, t = 0.0;
        if (j > 0) m += mS * (vC - vS);
        if (j < ny) m += mC * (vC - vN);
        t += visc_side(i > 0, lx, ez, vC, vW);
        t += visc_side(i < nx - 1, hx, ezE, vC, vE);
        if (DIM == 3) {
          t += visc_side(k > 0, lz, ex, vC, vB);
          t += visc_side(k < nz - 1, hz, exT, vC, vT);
        }
        v = gfv - (m + gv * t) * op.ih2 - (pC - pS) * op.ih;
        rr += v * v;
        gg += gfv * gfv;
      }
      if (res_w) res_w[fidx<1>(G, i, j, k)] = v;
    }
    if (DIM == 3 && cx && cy) {
      double v = 0.0;
      if (onw) {
        const double gw = (k == 0 || k == nz) ? 0.5 : 1.0;
        double m = 0.0, t = 0.0;
        if (k > 0) m += mB * (wC - wB);
        if (k < nz) m += mC * (wC - wT);
        t += visc_side(i > 0, lx, ey, wC, wW);
        t += visc_side(i < nx - 1, hx, eyE, wC, wE);
        t += visc_side(j > 0, ly, ex, wC, wS);
        t += visc_side(j < ny - 1, hy, exN, wC, wN);
        v = gfw - (m + gw * t) * op.ih2 - (pC - pB) * op.ih;
        rr += v * v;
        gg += gfw * gfw;
      }
      if (res_w) res_w[fidx<2>(G, i, j, k)] = v;
    }
    if (cell) {
      double v = 0.0;
      if (ic != G.pin) {
        double d = uC - uE;
        d += vC - vN;
        if (DIM == 3) d += wC - wT;
        v = rc - d / G.h;
        tt += v * v;
        zz += rc * rc;
      }
      if (res_r) res_r[ic] = v;
    }
    uB = uC, vB = vC, wB = wC, pB = pC;
    uC = uT, vC = vT, wC = wT;
  }
  __shared__ double sh[4][kSaddleBlock / 64];
  const double v[4] = {wave_sum(rr), wave_sum(gg), wave_sum(tt), wave_sum(zz)};
  if ((threadIdx.x & 63) == 0)
#pragma unroll
    for (int q = 0; q < 4; ++q) sh[q][threadIdx.x >> 6] = v[q];
  __syncthreads();
  if (threadIdx.x < 4) {
    double s = 0.0;
    for (int q = 0; q < kSaddleBlock / 64; ++q) s += sh[threadIdx.x][q];
    double* const out = threadIdx.x == 0 ? p_rr : threadIdx.x == 1 ? p_gg : threadIdx.x == 2 ? p_tt : p_zz;
    out[blockIdx.x] = s;
  }
}

// planes per thread and blocks of k_saddle: four planes amortise the columns'
// first loads, two where that leaves fewer than about 1000 blocks of waves;
// never more partials than the face kernels' launches have
struct SaddleLaunch {
  int kz, bx, blocks;
};
inline SaddleLaunch saddle_launch(const Grid& g) {
  const int bx = ((g.n[0] + 1) * (g.n[1] + 1) + kSaddleBlock - 1) / kSaddleBlock;
  const int kz = g.dim == 2 ? 1 : (bx * ((g.nze + 3) / 4) >= 1000 ? 4 : 2);
  return {kz, bx, bx * ((g.nze + kz - 1) / kz)};
}

// sums of four partial arrays, one block each
__global__ __launch_bounds__(kFinal) void k_sum_four(const double* a, const double* b,
                                                     const double* c, const double* d, int n,
                                                     int n2, double* out) {
  __shared__ double sh[kFinal / 64];
  const double* const src = blockIdx.x == 0 ? a : blockIdx.x == 1 ? b : blockIdx.x == 2 ? c : d;
  const double s = sum_partials(src, blockIdx.x < 2 ? n : n2, sh);
  if (threadIdx.x == 0) out[blockIdx.x] = s;
}

// --------------------------------------------------------- vector kernels

template <typename T>
__global__ __launch_bounds__(kBlock) void k_fill(int n, T v, T* __restrict__ y) {
  for (int i = blockIdx.x * kBlock + threadIdx.x; i < n; i += gridDim.x * kBlock) y[i] = v;
}

// y = a x + b y
__global__ __launch_bounds__(kBlock) void k_axpby(int n, double a, const double* __restrict__ x,
                                                  double b, double* __restrict__ y) {
  for (int i = blockIdx.x * kBlock + threadIdx.x; i < n; i += gridDim.x * kBlock)
    y[i] = a * x[i] + b * y[i];
}

// partial x.y
template <typename T>
__global__ __launch_bounds__(kBlock) void k_dot(int n, const T* __restrict__ x,
                                                const T* __restrict__ y, double* __restrict__ partial) {
  double s = 0.0;
  for (int i = blockIdx.x * kBlock + threadIdx.x; i < n; i += gridDim.x * kBlock)
    s += double(x[i]) * double(y[i]);
  __shared__ double sh[kBlock / 64];
  s = block_sum<kBlock>(s, sh);
  if (threadIdx.x == 0) partial[blockIdx.x] = s;
}

template <typename TI, typename TO>
__global__ __launch_bounds__(kBlock) void k_cast(int n, const TI* __restrict__ x, TO* __restrict__ y) {
  for (int i = blockIdx.x * kBlock + threadIdx.x; i < n; i += gridDim.x * kBlock) y[i] = TO(x[i]);
}

// GKB face update: v = s/alpha, Mv = y/alpha, u += zeta v
__global__ __launch_bounds__(kBlock) void k_gkb_faces(int n, double ialpha, double zeta,
                                                      const double* __restrict__ s,
                                                      const double* __restrict__ yv,
                                                      double* __restrict__ v, double* __restrict__ Mv,
                                                      double* __restrict__ u) {
  for (int i = blockIdx.x * kBlock + threadIdx.x; i < n; i += gridDim.x * kBlock) {
    const double vi = s[i] * ialpha;
    v[i] = vi;
    Mv[i] = yv[i] * ialpha;
    u[i] += zeta * vi;
  }
}

// GKB cell update: d = (q - beta d)/alpha, p -= zeta d
__global__ __launch_bounds__(kBlock) void k_gkb_cells(int n, double ialpha, double beta, double zeta,
                                                      const double* __restrict__ q,
                                                      double* __restrict__ d, double* __restrict__ p) {
  for (int i = blockIdx.x * kBlock + threadIdx.x; i < n; i += gridDim.x * kBlock) {
    const double di = (q[i] - beta * d[i]) * ialpha;
    d[i] = di;
    p[i] -= zeta * di;
  }
}

// --------------------------------------------------------------- PCG

// x = 0, r = f (cast), partial f.f
template <typename TI, typename T>
__global__ __launch_bounds__(kBlock) void k_pcg_init(int n, const TI* __restrict__ f,
                                                     T* __restrict__ x, T* __restrict__ r,
                                                     double* __restrict__ part_ff) {
  double s = 0.0;
  for (int i = blockIdx.x * kBlock + threadIdx.x; i < n; i += gridDim.x * kBlock) {
    const T fi = T(f[i]);
    x[i] = T(0);
    r[i] = fi;
    s += double(fi) * double(fi);
  }
  __shared__ double sh[kBlock / 64];
  s = block_sum<kBlock>(s, sh);
  if (threadIdx.x == 0) part_ff[blockIdx.x] = s;
}

// z = dinv r (Jacobi) when dinv != null; p = z; partial r.z
template <typename T>
__global__ __launch_bounds__(kBlock) void k_pcg_p0(int n, const T* __restrict__ dinv,
                                                   const T* __restrict__ r, T* __restrict__ z,
                                                   T* __restrict__ p, double* __restrict__ part_rz) {
  double s = 0.0;
  for (int i = blockIdx.x * kBlock + threadIdx.x; i < n; i += gridDim.x * kBlock) {
    const T ri = r[i];
    const T zi = dinv ? dinv[i] * ri : z[i];
    if (dinv) z[i] = zi;
    p[i] = zi;
    s += double(ri) * double(zi);
  }
  __shared__ double sh[kBlock / 64];
  s = block_sum<kBlock>(s, sh);
  if (threadIdx.x == 0) part_rz[blockIdx.x] = s;
}

__global__ __launch_bounds__(kFinal) void k_pcg_start(PcgState* st, const double* part_ff, int nff,
                                                      const double* part_rz, int nrz, double tol,
                                                      int maxit) {
  __shared__ double sh[kFinal / 64];
  const double ff = sum_partials(part_ff, nff, sh);
  __syncthreads();
  const double rz = sum_partials(part_rz, nrz, sh);
  if (threadIdx.x == 0) {
    st->rr0 = ff;
    st->rr = ff;
    st->rz = rz;
    st->tol2 = tol * tol;
    st->it = 0;
    st->maxit = maxit;
    st->alpha = st->beta = st->pq = 0.0;
    st->rz_prev = rz;
    st->rz_x = rz;
    st->it_x = 0;
    st->fresh = 1;
    st->nonfinite = 0;
    st->done = (ff == 0.0) ? 1 : 0;
    st->status = 0;
    st->fallback = st->stagnant = st->use_zv = st->fallbacks = 0;
    st->fb_it = st->fb_reason = 0;
    st->theta = st->gain = st->gain_sum = 0.0;
    st->gain_n = 0;
    for (int i = 0; i < 10; ++i) st->ring[i] = 0.0;
  }
}

// The one-block scalar kernels below read the done flag together with the
// partials (the flag is tested once both loads are in flight).
__global__ __launch_bounds__(kFinal) void k_pcg_alpha(PcgState* st, const double* part_pq, int n) {
  const int done = st->done;
  const double v = thread_partials(part_pq, n);
  if (done) return;
  __shared__ double sh[kFinal / 64];
  const double pq = block_sum<kFinal>(v, sh);
  if (threadIdx.x == 0) pcg_set_alpha(st, pq);
}

// x += alpha p, r -= alpha q; partial r.r; Jacobi (dinv != null): z = dinv r
// and partial r.z
template <typename T>
__global__ __launch_bounds__(kBlock) void k_pcg_xr(int n, const PcgState* __restrict__ st,
                                                   const T* __restrict__ p, const T* __restrict__ q,
                                                   T* __restrict__ x, T* __restrict__ r,
                                                   const T* __restrict__ dinv, T* __restrict__ z,
                                                   double* __restrict__ part_rr,
                                                   double* __restrict__ part_rz) {
  // the flag and alpha are tested / used once this thread's first loads are
  // in flight
  const int done = st->done;
  const T a = T(st->alpha);
  double s = 0.0, t = 0.0;
  for (int i = blockIdx.x * kBlock + threadIdx.x; i < n; i += gridDim.x * kBlock) {
    const T xi = x[i], pi = p[i], r0 = r[i], qi = q[i];
    if (done) break;
    x[i] = xi + a * pi;
    const T ri = r0 - a * qi;
    r[i] = ri;
    s += double(ri) * double(ri);
    if (dinv) {
      const T zi = dinv[i] * ri;
      z[i] = zi;
      t += double(ri) * double(zi);
    }
  }
  if (done) return;  // uniform: every thread of the block leaves
  __shared__ double sh[kBlock / 64];
  double v = block_sum<kBlock>(s, sh);
  if (threadIdx.x == 0) part_rr[blockIdx.x] = v;
  if (dinv) {
    __syncthreads();
    v = block_sum<kBlock>(t, sh);
    if (threadIdx.x == 0) part_rz[blockIdx.x] = v;
  }
}

// The same update with alpha folded in: every block sums the npq partials of
// p.q (folded scalar steps, common.hpp).  Its blocks are small (one entry per
// thread up to 2^18 entries), so the loads, the partials among them, are one
// round trip.
template <typename T>
__global__ __launch_bounds__(kBlock) void k_pcg_xr_fold(int n, PcgState* st,
                                                        const double* __restrict__ part_pq, int npq,
                                                        const T* __restrict__ p,
                                                        const T* __restrict__ q,
                                                        T* __restrict__ x, T* __restrict__ r,
                                                        double* __restrict__ part_rr) {
  __shared__ FoldShared<kBlock> fold;
  __shared__ double sh[kBlock / 64];
  const int done = st->done;
  int i = blockIdx.x * kBlock + threadIdx.x;
  const int e = i < n ? i : 0;
  T xi = x[e], pi = p[e], ri = r[e], qi = q[e];
  double pq;
  if (!fold_sum_if<kBlock>(done, fold_share<kBlock>(part_pq, npq), fold, pq)) return;
  double alpha;
  if (!fold_alpha(st, pq, blockIdx.x == 0 && threadIdx.x == 0, alpha)) return;
  const T a = T(alpha);
  double s = 0.0;
  while (i < n) {
    x[i] = xi + a * pi;
    ri = ri - a * qi;
    r[i] = ri;
    s += double(ri) * double(ri);
    i += gridDim.x * kBlock;
    if (i < n) xi = x[i], pi = p[i], ri = r[i], qi = q[i];
  }
  const double v = block_sum<kBlock>(s, sh);
  if (threadIdx.x == 0) part_rr[blockIdx.x] = v;
}

// convergence test on r.r; with part_rz also the CG beta (Jacobi path)
__global__ __launch_bounds__(kFinal) void k_pcg_check(PcgState* st, const double* part_rr, int nrr,
                                                      const double* part_rz, int nrz) {
  const int done = st->done;
  const double vrr = thread_partials(part_rr, nrr);
  const double vrz = part_rz ? thread_partials(part_rz, nrz) : 0.0;
  if (done) return;
  __shared__ double sh[kFinal / 64];
  const double rr = block_sum<kFinal>(vrr, sh);
  double rz = 0.0;
  if (part_rz) {
    __syncthreads();
    rz = block_sum<kFinal>(vrz, sh);
  }
  if (threadIdx.x == 0) pcg_set_check(st, rr, part_rz != nullptr, rz);
}

// preconditioned path: rz_new from the partials of the last V-cycle kernel
__global__ __launch_bounds__(kFinal) void k_pcg_beta(PcgState* st, const double* part_rz, int n) {
  const int done = st->done;
  const double v = thread_partials(part_rz, n);
  if (done) return;
  __shared__ double sh[kFinal / 64];
  const double rz = block_sum<kFinal>(v, sh);
  if (threadIdx.x == 0) pcg_set_beta(st, rz);
}

// p = z + beta p
template <typename T>
__global__ __launch_bounds__(kBlock) void k_pcg_p(int n, const PcgState* __restrict__ st,
                                                  const T* __restrict__ z, T* __restrict__ p) {
  if (st->done) return;
  const T b = T(st->beta);
  for (int i = blockIdx.x * kBlock + threadIdx.x; i < n; i += gridDim.x * kBlock)
    p[i] = z[i] + b * p[i];
}

// ------------------------------------------------------------ multigrid

// Tangential weights of the two transfer pairs.  DIV (divergence
// compatible): a fine face takes the value of the coarse face whose cell
// pair covers it, constant across the two fine cells in each tangential
// direction.  SMOOTH: linear in each tangential direction between the
// centres of the coarse rows, 3/4 from the row that covers the fine row and
// 1/4 from the next row on the fine row's side; beyond a side that next row
// is a mirror ghost, -1 times the covering row at a DIRICHLET wall (zero
// tangential velocity on the wall) and +1 times it at a NATURAL side.
// Weight of coarse row T in the value of fine row t along a tangential axis
// with nc coarse rows and side types lo / hi:
__device__ __forceinline__ double tan_weight(int t, int T, int nc, int lo, int hi) {
  const int Tc = t >> 1, Tn = (t & 1) ? Tc + 1 : Tc - 1;
  double w = 0.0;
  if (Tc == T) {
    w = 0.75;
    if (Tn < 0) w += lo == kDir ? -0.25 : 0.25;
    if (Tn >= nc) w += hi == kDir ? -0.25 : 0.25;
  } else if (Tn == T) {
    w = 0.25;
  }
  return w;
}

// Restriction of face residuals, full weighting: coarse face = (1/2^d) *
// sum over the fine faces it covers, normal neighbours weighted 1/2
// (transpose of the prolongation below divided by 2^d); SMOOTH also takes
// the fine rows next to the covered ones in each tangential direction, with
// the transposed weights.
// x0c (optional): the coarse level's first smoothing sweep from a zero
// guess, x0c = omega_c dinv_c bc, written in the same pass
template <typename T>
struct Pair2;
template <>
struct Pair2<float> {
  typedef float2 type;
};
template <>
struct Pair2<double> {
  typedef double2 type;
};

// pair: the fine v and w faces 2i, 2i+1 of a row sit at an even (aligned)
// index (x extent and array offsets even), so the DIV transfer in 3D loads
// them as one pair (they share the mask of their normal index); the sum
// keeps the order of the general loop below, so both give the same bits
template <typename T, int DIM, int C, bool SM>
__device__ __forceinline__ void restrict_face(const Grid& Gf, const Grid& Gc,
                                              const T* __restrict__ rf, T* __restrict__ bc,
                                              const T* __restrict__ dinv_c, T omega_c,
                                              T* __restrict__ x0c, int idx, int k, int done,
                                              int pair) {
  const int e0 = Gc.ext[C][0], e1 = Gc.ext[C][1];
  if (idx >= e0 * e1 || k >= Gc.ext[C][2]) return;
  const int j = idx / e0, i = idx - j * e0;
  const int P[3] = {i, j, k};
  const int f = fidx<C>(Gc, i, j, k);
  if (!unk<C>(Gc, P[C])) {
    if (done) return;
    bc[f] = T(0);
    if (x0c) x0c[f] = T(0);
    return;
  }
  T acc = T(0);
  const int nfC = Gf.n[C];
  const int A1 = (C + 1) % DIM;
  const int A2 = (C + 2) % 3;
  // fine rows per tangential axis: the two covered ones (DIV), with one
  // more on each side (SMOOTH)
  constexpr int kT = SM ? 4 : 2, kT0 = SM ? -1 : 0;
  if constexpr (!SM && DIM == 3 && C != 0) {
    if (pair) {  // uniform
      // x is a tangential axis; B the other one (z for v, y for w).  The
      // general loop runs (dn, A1, A2): for v A1 = z, A2 = x, for w A1 = x,
      // A2 = y
      constexpr int B = C == 1 ? 2 : 1;
      typedef typename Pair2<T>::type T2;
#pragma unroll
      for (int dn = -1; dn <= 1; ++dn) {
        const int fn = 2 * P[C] + dn;
        if (fn < 0 || fn > nfC) continue;
        const T wn = dn == 0 ? T(1) : T(0.5);
        const bool on = unk<C>(Gf, fn);
        T2 pb[2];
#pragma unroll
        for (int tb = 0; tb < 2; ++tb) {
          int Q[3];
          Q[C] = fn;
          Q[0] = 2 * P[0];
          Q[B] = 2 * P[B] + tb;
          pb[tb] = on ? *reinterpret_cast<const T2*>(rf + fidx<C>(Gf, Q[0], Q[1], Q[2]))
                      : T2{T(0), T(0)};
        }
        if (C == 1) {  // (z, x) order
          acc += wn * pb[0].x;
          acc += wn * pb[0].y;
          acc += wn * pb[1].x;
          acc += wn * pb[1].y;
        } else {  // (x, y) order
          acc += wn * pb[0].x;
          acc += wn * pb[1].x;
          acc += wn * pb[0].y;
          acc += wn * pb[1].y;
        }
      }
      const T dc = x0c ? dinv_c[f] : T(0);
      if (done) return;
      const T v = acc * T(0.125);
      bc[f] = v;
      if (x0c) x0c[f] = omega_c * dc * v;
      return;
    }
  }
#pragma unroll
  for (int dn = -1; dn <= 1; ++dn) {
    const int fn = 2 * P[C] + dn;
    if (fn < 0 || fn > nfC) continue;
    const T wn = dn == 0 ? T(1) : T(0.5);
#pragma unroll
    for (int t1 = 0; t1 < kT; ++t1)
#pragma unroll
      for (int t2 = 0; t2 < (DIM == 3 ? kT : 1); ++t2) {
        int Q[3];
        Q[C] = fn;
        Q[A1] = 2 * P[A1] + kT0 + t1;
        if (DIM == 3) Q[A2] = 2 * P[A2] + kT0 + t2;
        else Q[2] = 0;
        T w = wn;
        if (SM) {
          if (Q[A1] < 0 || Q[A1] >= Gf.n[A1]) continue;
          w *= T(tan_weight(Q[A1], P[A1], Gc.n[A1], Gc.bc[2 * A1], Gc.bc[2 * A1 + 1]));
          if (DIM == 3) {
            if (Q[A2] < 0 || Q[A2] >= Gf.n[A2]) continue;
            w *= T(tan_weight(Q[A2], P[A2], Gc.n[A2], Gc.bc[2 * A2], Gc.bc[2 * A2 + 1]));
          }
        }
        acc += w * ldm<C>(Gf, rf, Q[0], Q[1], Q[2]);
      }
  }
  const T dc = x0c ? dinv_c[f] : T(0);
  if (done) return;
  const T v = acc * T(DIM == 3 ? 0.125 : 0.25);
  bc[f] = v;
  if (x0c) x0c[f] = omega_c * dc * v;
}

template <typename T, int DIM, bool SM>
__global__ __launch_bounds__(kBlock) void k_restrict(Grid Gf, Grid Gc, const T* __restrict__ rf,
                                                     T* __restrict__ bc, const PcgState* st,
                                                     const T* __restrict__ dinv_c = nullptr,
                                                     T omega_c = T(0), T* __restrict__ x0c = nullptr,
                                                     int pair = 0) {
  // the flag is tested after the fine values are loaded
  const int done = st ? st->done : 0;
  const int c = blockIdx.z / Gc.nze;
  const int k = blockIdx.z - c * Gc.nze;
  const int idx = blockIdx.x * kBlock + threadIdx.x;
  if (c == 0) restrict_face<T, DIM, 0, SM>(Gf, Gc, rf, bc, dinv_c, omega_c, x0c, idx, k, done, pair);
  else if (c == 1) restrict_face<T, DIM, 1, SM>(Gf, Gc, rf, bc, dinv_c, omega_c, x0c, idx, k, done, pair);
  else if (DIM == 3) restrict_face<T, DIM, 2, SM>(Gf, Gc, rf, bc, dinv_c, omega_c, x0c, idx, k, done, pair);
}

// Prolongation + correction: fine faces coinciding with a coarse face take
// its value, fine faces between two coarse faces the mean (linear in the
// normal direction); across the two fine cells in tangential directions
// constant (DIV) or linear between coarse row centres (SMOOTH, weights of
// tan_weight).
// A thread takes kProPlanes planes of one (x, y): the index arithmetic is done
// once, and the coarse values of all its planes, loaded unconditionally
// (clamped to a valid face, weight 0), are in flight together.  192^3 FP32 DIV:
// 40 us (183 MB), one plane per thread 78 us.
constexpr int kProPlanes = 4;
__host__ __device__ inline int prolong_chunks(const Grid& g) { return (g.nze + kProPlanes - 1) / kProPlanes; }

template <typename T, int DIM, int C, bool SM>
__device__ __forceinline__ T prolong_value(const Grid& Gf, const Grid& Gc,
                                           const T* __restrict__ ec, int i, int j, int k) {
  const int P[3] = {i, j, k};
  const int Q[3] = {P[0] >> 1, P[1] >> 1, P[2] >> 1};
  const bool odd = P[C] & 1;
  // a coarse face, 0 where it is no unknown
  auto at = [&](const int* R) {
    const T v = ec[fidx<C>(Gc, R[0], R[1], R[2])];
    return unk<C>(Gc, R[C]) ? v : T(0);
  };
  int N[3] = {Q[0], Q[1], Q[2]};
  N[C] += odd ? 1 : 0;
  if (!SM) {
    const T a = at(Q), b = at(N);
    return odd ? T(0.5) * (a + b) : a;
  }
  constexpr int A1 = (C + 1) % DIM, A2 = (C + 2) % 3;
  T v = T(0);
#pragma unroll
  for (int dn = 0; dn < 2; ++dn) {
    const T wn = dn == 0 ? (odd ? T(0.5) : T(1)) : (odd ? T(0.5) : T(0));
#pragma unroll
    for (int a1 = 0; a1 < 2; ++a1)
#pragma unroll
      for (int a2 = 0; a2 < (DIM == 3 ? 2 : 1); ++a2) {
        int R[3] = {dn ? N[0] : Q[0], dn ? N[1] : Q[1], dn ? N[2] : Q[2]};
        T w = wn;
        if (a1 == 1) R[A1] += (P[A1] & 1) ? 1 : -1;
        if (DIM == 3 && a2 == 1) R[A2] += (P[A2] & 1) ? 1 : -1;
        // rows beyond a side are folded into the covering one
        const bool in1 = unsigned(R[A1]) < unsigned(Gc.n[A1]);
        R[A1] = in1 ? R[A1] : Q[A1];
        w *= in1 ? T(tan_weight(P[A1], R[A1], Gc.n[A1], Gc.bc[2 * A1], Gc.bc[2 * A1 + 1])) : T(0);
        if (DIM == 3) {
          const bool in2 = unsigned(R[A2]) < unsigned(Gc.n[A2]);
          R[A2] = in2 ? R[A2] : Q[A2];
          w *= in2 ? T(tan_weight(P[A2], R[A2], Gc.n[A2], Gc.bc[2 * A2], Gc.bc[2 * A2 + 1])) : T(0);
        }
        v += w * at(R);
      }
  }
  return v;
}

template <typename T, int DIM, int C, bool SM>
__device__ __forceinline__ void prolong_face(const Grid& Gf, const Grid& Gc,
                                             const T* __restrict__ ec, T* __restrict__ xf, int idx,
                                             int k0) {
  const int e0 = Gf.ext[C][0], e1 = Gf.ext[C][1], e2 = Gf.ext[C][2];
  if (idx >= e0 * e1) return;
  const int j = idx / e0, i = idx - j * e0;
  constexpr int N = DIM == 3 ? kProPlanes : 1;
  T x[N], v[N];
#pragma unroll
  for (int q = 0; q < N; ++q) {
    const int k = min(k0 + q, e2 - 1);
    x[q] = xf[fidx<C>(Gf, i, j, k)];
    v[q] = prolong_value<T, DIM, C, SM>(Gf, Gc, ec, i, j, k);
  }
#pragma unroll
  for (int q = 0; q < N; ++q) {
    const int k = k0 + q;
    if (k < e2 && unk<C>(Gf, C == 0 ? i : (C == 1 ? j : k)))
      xf[fidx<C>(Gf, i, j, k)] = x[q] + v[q];
  }
}

template <typename T, int DIM, bool SM>
__global__ __launch_bounds__(kBlock) void k_prolong_add(Grid Gf, Grid Gc, const T* __restrict__ ec,
                                                        T* __restrict__ xf, const PcgState* st) {
  if (st && st->done) return;
  const int chunks = prolong_chunks(Gf);
  const int c = blockIdx.z / chunks;
  const int k = (blockIdx.z - c * chunks) * kProPlanes;
  const int idx = blockIdx.x * kBlock + threadIdx.x;
  if (c == 0) prolong_face<T, DIM, 0, SM>(Gf, Gc, ec, xf, idx, k);
  else if (c == 1) prolong_face<T, DIM, 1, SM>(Gf, Gc, ec, xf, idx, k);
  else if (DIM == 3) prolong_face<T, DIM, 2, SM>(Gf, Gc, ec, xf, idx, k);
}

// x = Minv b on the coarsest grid: FP64 dense inverse (full-face layout,
// zero rows/columns at non-unknown faces); one wave64 per row, b staged in LDS
template <typename T>
__global__ __launch_bounds__(kBlock) void k_coarse_gemv(int m, const double* __restrict__ Minv,
                                                        const T* __restrict__ b, T* __restrict__ x,
                                                        const PcgState* st) {
  const int done = st ? st->done : 0;
  extern __shared__ __align__(16) double sb[];
  for (int i = threadIdx.x; i < m; i += kBlock) sb[i] = double(b[i]);
  if (done) return;  // uniform, before the barrier
  __syncthreads();
  const int lane = threadIdx.x & 63;
  const int row = blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6);
  if (row >= m) return;
  const double* a = Minv + (size_t)row * m;
  double s = 0.0;
  if ((m & 1) == 0) {
    // 16-byte loads, four independent partial sums: more loads in flight
    const double2* a2 = reinterpret_cast<const double2*>(a);
    const double2* b2 = reinterpret_cast<const double2*>(sb);
    const int h = m >> 1;
    double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
    int c = lane;
    for (; c + 64 < h; c += 128) {
      const double2 u = a2[c], v = a2[c + 64], bu = b2[c], bv = b2[c + 64];
      s0 += u.x * bu.x;
      s1 += u.y * bu.y;
      s2 += v.x * bv.x;
      s3 += v.y * bv.y;
    }
    for (; c < h; c += 64) {
      const double2 u = a2[c], bu = b2[c];
      s0 += u.x * bu.x;
      s1 += u.y * bu.y;
    }
    s = (s0 + s1) + (s2 + s3);
  } else {
    for (int c = lane; c < m; c += 64) s += a[c] * sb[c];
  }
  s = wave_sum(s);
  if (lane == 0) x[row] = T(s);
}

}  // namespace gkb

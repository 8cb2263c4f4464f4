// What every kernel source shares: block sizes, the deterministic reductions
// and the device-side state of the inner Krylov solves.
//
// Reductions are deterministic: each block reduces its values with a fixed
// wave-shuffle tree and a fixed-order pass over the waves, writes one FP64
// partial, and a one-block kernel sums the partials in a fixed order.
#pragma once
#include <hip/hip_runtime.h>

#include <cstddef>

#include "mac.hpp"

namespace gkb {

constexpr int kBlock = 256;   // threads per block (4 wave64)
constexpr int kFinal = 1024;  // threads of the one-block finalisers

// two buffers of the caller share memory
inline bool overlap(const void* a, size_t bytes_a, const void* b, size_t bytes_b) {
  const char *p = static_cast<const char*>(a), *q = static_cast<const char*>(b);
  return p < q + bytes_b && q < p + bytes_a;
}

// ------------------------------------------------------------- reductions

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// block-wide sum, result valid in thread 0; fixed order
template <int BS>
__device__ __forceinline__ double block_sum(double v, double* sh) {
  v = wave_sum(v);
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  if (lane == 0) sh[wid] = v;
  __syncthreads();
  double s = 0.0;
  if (threadIdx.x == 0) {
#pragma unroll
    for (int w = 0; w < BS / 64; ++w) s += sh[w];
  }
  return s;
}

// Sum of n partials in a fixed order (one block of kFinal threads): each
// thread's strided share, then the block sum.
__device__ __forceinline__ double thread_partials(const double* __restrict__ part, int n) {
  double v = 0.0;
  for (int i = threadIdx.x; i < n; i += kFinal) v += part[i];
  return v;
}
__device__ __forceinline__ double sum_partials(const double* __restrict__ part, int n, double* sh) {
  return block_sum<kFinal>(thread_partials(part, n), sh);  // valid in thread 0
}

// ------------------------------------------------------------ PCG state

struct PcgState {
  double rz, pq, alpha, beta, rr, rr0, tol2;
  double rz_prev;   // flexible CG
  double rt2;       // squared norm of the post-V-cycle residual (learned path)
  double theta;     // energy-optimal weight of the network correction
  double gain;      // error energy removed by that step, (c.rt)^2 / (c.Mc)
  double gain_sum;  // sum over network applications of gain / (r.V(r))
  double rz_x;      // folded steps: r.z of the current direction, kept for beta
  double ring[10];  // r.r sampled every 5 iterations (stagnation test)
  int it, maxit, done, status, nonfinite;
  int fallback;     // learned preconditioner switched off for this solve
  int stagnant;     // no decrease of r.r over the last 50 iterations
  int use_zv;       // direction from the V-cycle alone
  int fallbacks;
  int fb_it;        // iteration and cause of the fallback (1 descent,
  int fb_reason;    // 2 stagnation, 3 gain below the threshold)
  int gain_n;       // network applications counted in gain_sum
  int it_x;         // folded steps: iterations before the current one
  int fresh;        // folded steps: no direction update yet in this solve
};

// Sum of n partials by every thread of a block of BS threads, in a fixed
// order, so that all blocks get the same bits: a thread's share (its loads
// can be in flight with others), then the block's; sh: BS / 64 doubles.
template <int BS>
__device__ __forceinline__ double fold_share(const double* __restrict__ part, int n) {
  double v = 0.0;
  for (int i = threadIdx.x; i < n; i += BS) v += part[i];
  return v;
}
template <int BS>
__device__ __forceinline__ double fold_sum(double v, double* sh) {
  v = wave_sum(v);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  double s = 0.0;
#pragma unroll
  for (int w = 0; w < BS / 64; ++w) s += sh[w];
  __syncthreads();  // sh may be used again
  return s;
}
// The same sum in a kernel whose block 0 may set the flag that its blocks test:
// a late block's waves can read the flag on either side of that store, so each
// brings what it read (off) and the block goes by all of them.  Returns
// false, in every thread, if any wave saw the flag set; else s is the sum.
template <int BS>
struct FoldShared {
  double s[BS / 64];
  int off[BS / 64];
};
template <int BS>
__device__ __forceinline__ bool fold_sum_if(int off, double v, FoldShared<BS>& sh, double& s) {
  v = wave_sum(v);
  off = __any(off);
  if ((threadIdx.x & 63) == 0) {
    sh.s[threadIdx.x >> 6] = v;
    sh.off[threadIdx.x >> 6] = off;
  }
  __syncthreads();
  s = 0.0;
  int any = 0;
#pragma unroll
  for (int w = 0; w < BS / 64; ++w) {
    s += sh.s[w];
    any |= sh.off[w];
  }
  __syncthreads();  // sh may be used again
  return any == 0;
}

// Scalar steps of PCG on the device state (one thread): alpha from p.q;
// the convergence test on r.r (with rz: also beta, Jacobi path); beta from
// the new r.z.
__device__ __forceinline__ void pcg_set_alpha(PcgState* st, double pq) {
  st->pq = pq;
  const double a = st->rz / pq;
  if (!(pq > 0.0) || !isfinite(a)) {
    st->alpha = 0.0;
    st->nonfinite = 1;
    st->status = -4;
    st->done = 1;
  } else {
    st->alpha = a;
  }
}
__device__ __forceinline__ void pcg_set_check(PcgState* st, double rr, bool has_rz, double rz) {
  st->rr = rr;
  st->it += 1;
  // r.r sampled every 5 iterations: stagnant when no decrease over 50
  // (CG minimises the energy norm, so r.r may rise over shorter spans)
  if (st->it % 5 == 0) {
    const int slot = (st->it / 5) % 10;
    if (st->it > 50 && rr >= st->ring[slot]) st->stagnant = 1;
    st->ring[slot] = rr;
  }
  if (!isfinite(rr)) {
    st->nonfinite = 1;
    st->status = -4;
    st->done = 1;
  } else if (rr <= st->tol2 * st->rr0) {
    st->done = 1;
    st->status = 0;
  } else if (st->it >= st->maxit) {
    st->done = 1;
    st->status = -5;
  } else if (has_rz) {
    st->beta = rz / st->rz;
    st->rz = rz;
  }
}
__device__ __forceinline__ void pcg_set_beta(PcgState* st, double rz) {
  st->beta = rz / st->rz;
  st->rz = rz;
}

// Folded scalar steps.  Where a PCG iteration is bound by its launches, the
// scalar steps are not kernels of their own: every block of the kernel that
// needs the scalar sums the (few) partials itself, in the same order, and
// block 0 records it.  No kernel reads a field that it writes itself: the
// product (A) reads rz_x and fresh and writes rz and beta; the update (X)
// reads rz and it and writes alpha, rz_x, it_x and fresh; the first V-cycle
// kernel (C) reads it_x and writes it and the outcome.  done alone is read and
// written by X and C, where every block comes to the same end by itself; a
// block that starts late may see it set, and then all of its waves have to
// (fold_sum_if).
__device__ __forceinline__ double fold_beta(PcgState* st, double rz_new, bool lead) {
  if (st->fresh) return 0.0;  // p = z: rz is that of the start
  const double b = rz_new / st->rz_x;
  if (lead) {
    st->rz = rz_new;
    st->beta = b;
  }
  return b;
}
// false: breakdown, the iterate stays as it is and the solve ends
__device__ __forceinline__ bool fold_alpha(PcgState* st, double pq, bool lead, double& alpha) {
  const double rz = st->rz, a = rz / pq;
  if (lead) {
    pcg_set_alpha(st, pq);
    st->rz_x = rz;
    st->it_x = st->it;
    st->fresh = 0;
  }
  alpha = a;
  return pq > 0.0 && isfinite(a);
}
// true: the iteration ends here
__device__ __forceinline__ bool fold_check(PcgState* st, double rr, bool lead) {
  const bool end = !isfinite(rr) || rr <= st->tol2 * st->rr0 || st->it_x + 1 >= st->maxit;
  if (lead) pcg_set_check(st, rr, false, 0.0);
  return end;
}

// ---------------------------------------------------------- buffer access

// Raw buffer access: a scalar base (buffer resource) plus a per-lane 32-bit
// byte offset and a uniform scalar byte offset, so an access costs no 64-bit
// address arithmetic.  Its users take only face arrays below 2 GiB, which keeps
// every offset in 31 bits.
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buf_rsrc(const void* p, unsigned bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, (int)bytes, 0x00020000);
}
template <typename T>
__device__ __forceinline__ T buf_load(__amdgpu_buffer_rsrc_t r, unsigned voff, unsigned soff);
template <>
__device__ __forceinline__ float buf_load<float>(__amdgpu_buffer_rsrc_t r, unsigned voff,
                                                 unsigned soff) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0));
}
template <>
__device__ __forceinline__ double buf_load<double>(__amdgpu_buffer_rsrc_t r, unsigned voff,
                                                   unsigned soff) {
  return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0));
}
__device__ __forceinline__ void buf_store(float v, __amdgpu_buffer_rsrc_t r, unsigned voff,
                                          unsigned soff) {
  __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), r, voff, soff, 0);
}
__device__ __forceinline__ void buf_store(double v, __amdgpu_buffer_rsrc_t r, unsigned voff,
                                          unsigned soff) {
  __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), r, voff, soff, 0);
}

}  // namespace gkb

// What every kernel source shares: block sizes, the deterministic reductions
// and the device-side state of the inner Krylov solves.
//
// Reductions are deterministic: each block reduces its values with a fixed
// wave-shuffle tree and a fixed-order pass over the waves, writes one FP64
// partial, and a one-block kernel sums the partials in a fixed order.
#pragma once
#include <hip/hip_runtime.h>

#include "mac.hpp"

namespace gkb {

constexpr int kBlock = 256;   // threads per block (4 wave64)
constexpr int kFinal = 1024;  // threads of the one-block finalisers

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
  double ring[10];  // r.r sampled every 5 iterations (stagnation test)
  int it, maxit, done, status, nonfinite;
  int fallback;     // learned preconditioner switched off for this solve
  int stagnant;     // no decrease of r.r over the last 50 iterations
  int use_zv;       // direction from the V-cycle alone
  int fallbacks;
  int fb_it;        // iteration and cause of the fallback (1 descent,
  int fb_reason;    // 2 stagnation, 3 gain below the threshold)
  int gain_n;       // network applications counted in gain_sum
};

}  // namespace gkb

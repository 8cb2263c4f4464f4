// A stand-in for the HIP headers that lets a host compiler take the device
// headers: a block runs as host threads, one per GPU thread, with a real
// barrier and lane exchanges inside each wave of 64.  A thread that leaves the
// kernel leaves the barrier, as a wave does on the GPU.
#pragma once
#include <algorithm>
#include <cmath>
#include <condition_variable>
#include <cstdint>
#include <mutex>

#define __host__
#define __device__
#define __global__
#define __forceinline__ inline
#define __launch_bounds__(...)
#define __shared__ static
#define __align__(n) __attribute__((aligned(n)))
#define __amdgpu_buffer_rsrc_t int
#define __builtin_amdgcn_make_buffer_rsrc(p, a, b, c) (0)
#define __builtin_amdgcn_raw_buffer_load_b32(...) (0u)
#define __builtin_amdgcn_raw_buffer_load_b64(...) (u32x2{0u, 0u})
#define __builtin_amdgcn_raw_buffer_store_b32(...) ((void)0)
#define __builtin_amdgcn_raw_buffer_store_b64(...) ((void)0)

typedef void* hipStream_t;
typedef float float2 __attribute__((ext_vector_type(2)));
typedef double double2 __attribute__((ext_vector_type(2)));
struct dim3 {
  unsigned x, y, z;
  dim3(unsigned a = 1, unsigned b = 1, unsigned c = 1) : x(a), y(b), z(c) {}
};
inline thread_local dim3 threadIdx(0, 0, 0), blockIdx(0, 0, 0);
inline dim3 gridDim, blockDim;

using std::isfinite;
using std::max;
using std::min;

namespace hostsim {

// barrier over the members that are still running
class Barrier {
  std::mutex m;
  std::condition_variable cv;
  int members = 0, waiting = 0;
  long turn = 0;
  void open() {
    waiting = 0;
    ++turn;
    cv.notify_all();
  }

 public:
  void reset(int n) { members = n, waiting = 0; }
  void wait() {
    std::unique_lock<std::mutex> l(m);
    const long t = turn;
    if (++waiting == members) return open();
    cv.wait(l, [&] { return turn != t; });
  }
  void leave() {
    std::unique_lock<std::mutex> l(m);
    if (--members == waiting && waiting > 0) open();
  }
  int stopped() {  // members at the barrier
    std::unique_lock<std::mutex> l(m);
    return waiting;
  }
};
inline Barrier block, wave[16];
inline double lanes[16][64];

}  // namespace hostsim

inline void __syncthreads() { hostsim::block.wait(); }
inline double __shfl(double v, int lane, int) {
  const int w = threadIdx.x >> 6;
  hostsim::lanes[w][threadIdx.x & 63] = v;
  hostsim::wave[w].wait();
  const double r = hostsim::lanes[w][lane & 63];
  hostsim::wave[w].wait();
  return r;
}
inline double __shfl_xor(double v, int mask, int width) {
  return __shfl(v, (threadIdx.x & 63) ^ mask, width);
}
inline int __any(int v) {
  double any = 0.0;
  for (int lane = 0; lane < 64; ++lane) any += __shfl(double(v != 0), lane, 64);
  return any != 0.0;
}

// Convolution and weight-gradient launches of the preconditioner network
// (kernels in conv.hip; 3x3 / 3x3x3 taps, zero padding, at most 16 channels).
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstring>

namespace gkb {

constexpr int kCP = 16;  // most channels of a layer; rows of the packed weights

// channels that an activation of c channels is stored with (the padded ones
// are 0)
__host__ __device__ inline int chan_group(int c) { return c <= 4 ? 4 : (c <= 8 ? 8 : 16); }

__host__ __device__ inline uint16_t f2bf(float f) {
  uint32_t u;
  std::memcpy(&u, &f, 4);
  u += 0x7FFFu + ((u >> 16) & 1u);  // round to nearest even
  return uint16_t(u >> 16);
}

constexpr int kMaxLayers = 8;

struct CnnGeom {
  int nx, ny, nz, batch;
  long P;  // nx * ny * nz * batch
};

// a layer input: BF16 activations [P][chan_group(c)], or FP32 [P][c] rounded
// to BF16 as it is read
struct ConvIn {
  const void* p;
  int c;
  bool f32;
};

enum ConvOut {
  kOutReluBf16 = 0,  // ReLU, BF16 [P][chan_group(cout)]
  kOutF32 = 1,       // FP32 [P][cout]
  kOutMaskBf16 = 2   // 0 where mask <= 0, BF16 [P][chan_group(cout)] (mask alike)
};

// out[p][n] = bias[n] + sum_tap sum_c in[p + off(tap)][c] * w[tap][n][c] with
// w BF16 [taps][16][16]; skip1, skip2: device flags that turn the launch into
// a no-op
void conv_layer(hipStream_t s, int dim, const CnnGeom& g, const ConvIn& in, const uint16_t* w,
                const float* bias, ConvOut mode, void* out, int cout, const uint16_t* mask,
                const int* skip1 = nullptr, const int* skip2 = nullptr);

// weight gradient of the layers in the flat parameter layout:
// flat[tap][ci][co] = sum_p act[p + off(tap)][ci] dz[p][co], then
// flat[..][co] = sum_p dz[p][co].  wgrad_layer leaves a layer's block partials
// in part (wgrad_part_floats() floats for cin input channels, kept until
// wgrad_finish) and notes it in sum; wgrad_finish adds up all layers at once.
struct WgradLayer {
  const float* part;
  float* flat;
  int nt, cg, cin, cout;
};
struct WgradSum {
  int layers = 0, nblk = 0;
  int first[kMaxLayers + 1] = {0};  // first block of each layer's reduction
  WgradLayer l[kMaxLayers];
};
int wgrad_blocks(int dim, const CnnGeom& g);
size_t wgrad_part_floats(int dim, const CnnGeom& g, int cin);
void wgrad_layer(hipStream_t s, int dim, const CnnGeom& g, const ConvIn& act, const ConvIn& dz,
                 float* part, float* flat, WgradSum& sum);
void wgrad_finish(hipStream_t s, int dim, const WgradSum& sum);

}  // namespace gkb

// Convolutional preconditioner network on gfx950 (see include/gkb_cnn.h):
// layers, loss, Adam and checkpoints; the convolution and weight-gradient
// kernels are in conv.hip.
//
// Activations are channels-last BF16, stored with 4, 8 or 16 channels per
// point (the smallest that holds the layer's); the network's FP32 input and
// the FP32 output gradient are rounded to BF16 as they are read.  All
// reductions are deterministic.
#pragma once
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <vector>

#include "../../include/gkb_cnn.h"
#include "conv.hpp"

namespace gkb {

// flat FP32 layer parameters -> BF16 forward weights wf[t][co][ci], dgrad
// weights wd[t][ci][co] taken from the mirrored tap, FP32 bias[16]
__global__ __launch_bounds__(256) void k_pack_weights(const float* __restrict__ flat, int taps,
                                                      int cin, int cout, uint16_t* __restrict__ wf,
                                                      uint16_t* __restrict__ wd,
                                                      float* __restrict__ bias) {
  for (int e = blockIdx.x * 256 + threadIdx.x; e < taps * 256; e += gridDim.x * 256) {
    const int t = e / 256, a = (e / 16) % 16, c = e % 16;
    // wf[t][a = co][c = ci]
    float vf = (a < cout && c < cin) ? flat[(t * cin + c) * cout + a] : 0.f;
    wf[e] = f2bf(vf);
    // wd[t][a = ci (output of the adjoint)][c = co] = W[taps-1-t][ci][co]
    const int tm = taps - 1 - t;
    float vd = (a < cin && c < cout) ? flat[(tm * cin + a) * cout + c] : 0.f;
    wd[e] = f2bf(vd);
  }
  if (blockIdx.x == 0 && threadIdx.x < 16)
    bias[threadIdx.x] = threadIdx.x < cout ? flat[taps * cin * cout + threadIdx.x] : 0.f;
}

// per-sample partial sums of ||y - e||^2 and ||e||^2 (grid: (blocks, batch))
__global__ __launch_bounds__(256) void k_loss_part(long Pb, int c, const float* __restrict__ y,
                                                   const float* __restrict__ e,
                                                   double* __restrict__ num,
                                                   double* __restrict__ den) {
  const int s = blockIdx.y;
  double a = 0.0, b = 0.0;
  for (long q = (long)blockIdx.x * 256 + threadIdx.x; q < Pb * c; q += (long)gridDim.x * 256) {
    const double ev = e[(size_t)s * Pb * c + q];
    const double d = double(y[(size_t)s * Pb * c + q]) - ev;
    a += d * d;
    b += ev * ev;
  }
  __shared__ double sh[4];
  double t = block_sum<256>(a, sh);
  if (threadIdx.x == 0) num[s * gridDim.x + blockIdx.x] = t;
  __syncthreads();
  t = block_sum<256>(b, sh);
  if (threadIdx.x == 0) den[s * gridDim.x + blockIdx.x] = t;
}

// mean squared error over all batch entries (scalar[0]) and the per-sample
// weight 1 / (points * channels) (scalar[1 + s]) from the partials (one
// block of 256 threads, fixed order); inputs and targets are already
// normalised by the residual scale
__global__ __launch_bounds__(256) void k_loss_final(int batch, int nblk, long per_sample,
                                                    const double* num, double* scal) {
  __shared__ double sh[4];
  double L = 0.0;
  const double inv = 1.0 / double(per_sample);
  for (int s = 0; s < batch; ++s) {
    double a = 0.0;
    for (int k = threadIdx.x; k < nblk; k += 256) a += num[s * nblk + k];
    a = block_sum<256>(a, sh);  // valid in thread 0
    __syncthreads();            // sh is reused by the next sample
    if (threadIdx.x == 0) {
      scal[1 + s] = inv;
      L += a * inv;
    }
  }
  if (threadIdx.x == 0) scal[0] = L / batch;
}

// dz = 2 (y - e) / (points * channels * batch), BF16 [P][chan_group(c)]
__global__ __launch_bounds__(256) void k_loss_grad(long Pb, int c, int batch,
                                                   const float* __restrict__ y,
                                                   const float* __restrict__ e,
                                                   const double* __restrict__ scal,
                                                   uint16_t* __restrict__ dz) {
  const int cg = chan_group(c);
  const long P = Pb * batch;
  for (long q = (long)blockIdx.x * 256 + threadIdx.x; q < P * cg; q += (long)gridDim.x * 256) {
    const long p = q / cg;
    const int ch = int(q % cg);
    float v = 0.f;
    if (ch < c) {
      const int s = int(p / Pb);
      const double ev = e[p * c + ch];
      v = float(2.0 * (double(y[p * c + ch]) - ev) * scal[1 + s] / batch);
    }
    dz[q] = f2bf(v);
  }
}

__global__ __launch_bounds__(256) void k_adam(int n, float* __restrict__ w,
                                              const float* __restrict__ g, float* __restrict__ m,
                                              float* __restrict__ v, float lr, float b1, float b2,
                                              float eps, float c1, float c2) {
  for (int e = blockIdx.x * 256 + threadIdx.x; e < n; e += gridDim.x * 256) {
    const float gi = g[e];
    const float mi = b1 * m[e] + (1.f - b1) * gi;
    const float vi = b2 * v[e] + (1.f - b2) * gi * gi;
    m[e] = mi;
    v[e] = vi;
    w[e] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
  }
}

// gather crops: inputs [pairs][P][cin] -> act BF16 [B][crop^d][chan_group(cin)],
// targets [pairs][P][cout] -> e FP32 [B][crop^d][cout]; desc[s] = {pair, ox, oy, oz}
__global__ __launch_bounds__(256) void k_gather(int nx, int ny, int nz, int dim, int crop, int cin,
                                                int cout, const float* __restrict__ inputs,
                                                const float* __restrict__ targets,
                                                const int* __restrict__ desc,
                                                uint16_t* __restrict__ act, float* __restrict__ e) {
  const int s = blockIdx.y;
  const int cz = dim == 3 ? crop : 1;
  const long Pc = (long)crop * crop * cz;
  const long P = (long)nx * ny * nz;
  const int pair = desc[4 * s], ox = desc[4 * s + 1], oy = desc[4 * s + 2], oz = desc[4 * s + 3];
  for (long q = (long)blockIdx.x * 256 + threadIdx.x; q < Pc; q += (long)gridDim.x * 256) {
    const int i = int(q % crop), j = int((q / crop) % crop), k = int(q / ((long)crop * crop));
    const long src = ((long)(k + oz) * ny + (j + oy)) * nx + (i + ox);
    const float* xi = inputs + ((size_t)pair * P + src) * cin;
    const int cg = chan_group(cin);
    uint16_t* a = act + ((size_t)s * Pc + q) * cg;
    for (int ch = 0; ch < cg; ++ch) a[ch] = f2bf(ch < cin ? xi[ch] : 0.f);
    const float* ti = targets + ((size_t)pair * P + src) * cout;
    float* eo = e + ((size_t)s * Pc + q) * cout;
    for (int ch = 0; ch < cout; ++ch) eo[ch] = ti[ch];
  }
}

}  // namespace gkb

// --------------------------------------------------------------- network

struct gkb_cnn {
  int dim = 3, L = 0, taps = 27;
  int ch[gkb::kMaxLayers + 1] = {0};
  long np = 0;
  long off[gkb::kMaxLayers + 1] = {0};  // flat offset of each layer
  float *params = nullptr, *grad = nullptr, *m = nullptr, *v = nullptr;
  uint16_t *wf = nullptr, *wd = nullptr;  // [L][taps][256]
  float* bias = nullptr;                  // [L][16]
  int adam_t = 0;
  // workspace (grown on demand; a graph that holds its buffers is valid while
  // buffers is what it was at the capture)
  long cap = 0;
  long buffers = 0;
  uint16_t* act[gkb::kMaxLayers] = {nullptr};  // layer inputs, [P][chan_group]
  uint16_t *dz0 = nullptr, *dz1 = nullptr;
  float* y = nullptr;      // output [P][c_L]
  float* wpart = nullptr;  // wgrad block partials
  size_t wcap = 0;
  double* lscal = nullptr;  // loss scalars
  double *lnum = nullptr, *lden = nullptr;
  int lcap = 0;
  float* ebuf = nullptr;  // training targets
  long ecap = 0;
  int* desc = nullptr;
  int dcap = 0;
  hipStream_t s = nullptr;
  bool weights_dirty = true;
};

namespace {

#define CNNCK(expr)                                                              \
  do {                                                                           \
    hipError_t e_ = (expr);                                                      \
    if (e_ != hipSuccess) {                                                      \
      std::fprintf(stderr, "gkb_cnn: HIP error %s at %s:%d\n", hipGetErrorString(e_), \
                   __FILE__, __LINE__);                                          \
      return GKB_EHIP;                                                           \
    }                                                                            \
  } while (0)

// Host <-> device copy ordered on the network's (non-blocking) stream and
// complete on return
hipError_t cnn_copy(gkb_cnn* n, void* dst, const void* src, size_t bytes, hipMemcpyKind kind) {
  hipError_t e = hipMemcpyAsync(dst, src, bytes, kind, n->s);
  return e != hipSuccess ? e : hipStreamSynchronize(n->s);
}

int cnn_grid(long n) { return (int)std::max<long>(1, std::min<long>((n + 255) / 256, 8192)); }

int cnn_prepare_weights(gkb_cnn* n) {
  if (!n->weights_dirty) return GKB_OK;
  for (int l = 0; l < n->L; ++l)
    gkb::k_pack_weights<<<cnn_grid(n->taps * 256), 256, 0, n->s>>>(
        n->params + n->off[l], n->taps, n->ch[l], n->ch[l + 1], n->wf + (size_t)l * n->taps * 256,
        n->wd + (size_t)l * n->taps * 256, n->bias + 16 * l);
  CNNCK(hipGetLastError());
  n->weights_dirty = false;
  return GKB_OK;
}

int cnn_reserve(gkb_cnn* n, long P) {
  // tiles of points are counted in 32 bits
  if (P <= 0 || P > 0x7fffffffL) return GKB_EINVAL;
  if (P <= n->cap) return GKB_OK;
  n->cap = 0;
  n->buffers += 1;
  auto grow = [&](auto*& p, size_t bytes) {
    if (p) (void)hipFree(p);
    p = nullptr;
    return hipMalloc(&p, bytes);
  };
  int cmax = 1;
  for (int l = 0; l <= n->L; ++l) cmax = std::max(cmax, n->ch[l]);
  for (int l = 0; l < n->L; ++l)
    CNNCK(grow(n->act[l], P * gkb::chan_group(n->ch[l]) * sizeof(uint16_t)));
  CNNCK(grow(n->dz0, P * gkb::chan_group(cmax) * sizeof(uint16_t)));
  CNNCK(grow(n->dz1, P * gkb::chan_group(cmax) * sizeof(uint16_t)));
  CNNCK(grow(n->y, P * n->ch[n->L] * sizeof(float)));
  n->cap = P;
  return GKB_OK;
}

// the BF16 input of the network that a caller filled
gkb::ConvIn cnn_act0(const gkb_cnn* n) { return gkb::ConvIn{n->act[0], n->ch[0], false}; }

// hidden layers from the input x, then (y != null) the output layer into y
// (FP32 [P][c_L]); skip1, skip2 as conv_layer
void cnn_layers(hipStream_t s, const gkb_cnn* n, const gkb::CnnGeom& g, const gkb::ConvIn& x,
                float* y, const int* skip1 = nullptr, const int* skip2 = nullptr) {
  gkb::ConvIn in = x;
  for (int l = 0; l < n->L; ++l) {
    const uint16_t* w = n->wf + (size_t)l * n->taps * 256;
    const float* b = n->bias + 16 * l;
    const int cout = n->ch[l + 1];
    if (l < n->L - 1) {
      gkb::conv_layer(s, n->dim, g, in, w, b, gkb::kOutReluBf16, n->act[l + 1], cout, nullptr,
                      skip1, skip2);
      in = gkb::ConvIn{n->act[l + 1], cout, false};
    } else if (y) {
      gkb::conv_layer(s, n->dim, g, in, w, b, gkb::kOutF32, y, cout, nullptr, skip1, skip2);
    }
  }
}

int cnn_forward(gkb_cnn* n, const gkb::CnnGeom& g, const gkb::ConvIn& x, float* y) {
  int rc = cnn_prepare_weights(n);
  if (rc) return rc;
  cnn_layers(n->s, n, g, x, y);
  CNNCK(hipGetLastError());
  return GKB_OK;
}

// parameter gradient into n->grad and (dx != null) the input gradient, from
// the hidden activations of cnn_forward, its input x and the output gradient
int cnn_backward(gkb_cnn* n, const gkb::CnnGeom& g, const gkb::ConvIn& x, const gkb::ConvIn& dy,
                 float* dx) {
  int rc = cnn_prepare_weights(n);
  if (rc) return rc;
  size_t need = 0;
  for (int l = 0; l < n->L; ++l) need += gkb::wgrad_part_floats(n->dim, g, n->ch[l]);
  if (need > n->wcap) {
    if (n->wpart) (void)hipFree(n->wpart);
    n->wpart = nullptr;
    n->wcap = 0;
    CNNCK(hipMalloc(&n->wpart, need * sizeof(float)));
    n->wcap = need;
  }
  gkb::ConvIn dz = dy;
  // dz0 may hold the output gradient: the hidden ones start in dz1
  uint16_t *cur = n->dz1, *other = n->dz0;
  gkb::WgradSum sum;
  float* part = n->wpart;
  for (int l = n->L - 1; l >= 0; --l) {
    const gkb::ConvIn a = l == 0 ? x : gkb::ConvIn{n->act[l], n->ch[l], false};
    gkb::wgrad_layer(n->s, n->dim, g, a, dz, part, n->grad + n->off[l], sum);
    part += gkb::wgrad_part_floats(n->dim, g, n->ch[l]);
    const uint16_t* wd = n->wd + (size_t)l * n->taps * 256;
    // the adjoint convolution reads the layer's output channels
    if (l > 0) {
      gkb::conv_layer(n->s, n->dim, g, dz, wd, nullptr, gkb::kOutMaskBf16, cur, n->ch[l],
                      n->act[l]);
      dz = gkb::ConvIn{cur, n->ch[l], false};
      std::swap(cur, other);
    } else if (dx) {
      gkb::conv_layer(n->s, n->dim, g, dz, wd, nullptr, gkb::kOutF32, dx, n->ch[0], nullptr);
    }
  }
  gkb::wgrad_finish(n->s, n->dim, sum);
  CNNCK(hipGetLastError());
  return GKB_OK;
}

int cnn_adam(gkb_cnn* n, double lr, double b1, double b2, double eps) {
  n->adam_t += 1;
  const float c1 = float(1.0 - std::pow(b1, n->adam_t)), c2 = float(1.0 - std::pow(b2, n->adam_t));
  gkb::k_adam<<<cnn_grid(n->np), 256, 0, n->s>>>((int)n->np, n->params, n->grad, n->m, n->v,
                                                  float(lr), float(b1), float(b2), float(eps), c1,
                                                  c2);
  n->weights_dirty = true;
  CNNCK(hipGetLastError());
  return GKB_OK;
}

int cnn_loss_buffers(gkb_cnn* n, int batch, int nblk) {
  if (batch * nblk > n->lcap) {
    if (n->lnum) (void)hipFree(n->lnum);
    if (n->lden) (void)hipFree(n->lden);
    CNNCK(hipMalloc(&n->lnum, (size_t)batch * nblk * sizeof(double)));
    CNNCK(hipMalloc(&n->lden, (size_t)batch * nblk * sizeof(double)));
    n->lcap = batch * nblk;
  }
  if (!n->lscal) CNNCK(hipMalloc(&n->lscal, 1025 * sizeof(double)));
  return GKB_OK;
}

}  // namespace

extern "C" {

int gkb_cnn_create(int dim, int n_layers, const int* channels, unsigned seed, gkb_cnn** out) {
  if (!out || !channels || (dim != 2 && dim != 3) || n_layers < 1 || n_layers > gkb::kMaxLayers)
    return GKB_EINVAL;
  for (int l = 0; l <= n_layers; ++l)
    if (channels[l] < 1 || channels[l] > gkb::kCP) return GKB_EINVAL;
  gkb_cnn* n = new gkb_cnn();
  n->dim = dim;
  n->L = n_layers;
  n->taps = dim == 2 ? 9 : 27;
  long o = 0;
  for (int l = 0; l <= n_layers; ++l) n->ch[l] = channels[l];
  for (int l = 0; l < n_layers; ++l) {
    n->off[l] = o;
    o += (long)n->taps * channels[l] * channels[l + 1] + channels[l + 1];
  }
  n->np = o;
  auto fail = [&](int rc) {
    gkb_cnn_destroy(n);
    return rc;
  };
  if (hipStreamCreateWithFlags(&n->s, hipStreamNonBlocking) != hipSuccess) return fail(GKB_EHIP);
  float** fp[] = {&n->params, &n->grad, &n->m, &n->v};
  for (auto p : fp) {
    if (hipMalloc(p, n->np * sizeof(float)) != hipSuccess) return fail(GKB_ENOMEM);
    if (hipMemsetAsync(*p, 0, n->np * sizeof(float), n->s) != hipSuccess) return fail(GKB_EHIP);
  }
  if (hipMalloc(&n->wf, (size_t)n_layers * n->taps * 256 * 2) != hipSuccess ||
      hipMalloc(&n->wd, (size_t)n_layers * n->taps * 256 * 2) != hipSuccess ||
      hipMalloc(&n->bias, (size_t)n_layers * 16 * 4) != hipSuccess)
    return fail(GKB_ENOMEM);
  // seeded He-uniform initialisation (64-bit LCG), zero biases
  std::vector<float> h(n->np, 0.f);
  uint64_t st = 0x9E3779B97F4A7C15ull ^ seed;
  for (int l = 0; l < n_layers; ++l) {
    const int fan_in = n->taps * channels[l];
    const float lim = std::sqrt(6.0f / fan_in);
    const long nw = (long)n->taps * channels[l] * channels[l + 1];
    for (long e = 0; e < nw; ++e) {
      st = st * 6364136223846793005ull + 1442695040888963407ull;
      const double u = double(st >> 11) * (1.0 / 9007199254740992.0);
      h[n->off[l] + e] = float((2.0 * u - 1.0) * lim);
    }
  }
  if (cnn_copy(n, n->params, h.data(), n->np * 4, hipMemcpyHostToDevice) != hipSuccess)
    return fail(GKB_EHIP);
  *out = n;
  return GKB_OK;
}

void gkb_cnn_destroy(gkb_cnn* n) {
  if (!n) return;
  if (n->s) (void)hipStreamSynchronize(n->s);
  void* ptrs[] = {n->params, n->grad, n->m,    n->v,    n->wf,    n->wd,   n->bias,
                  n->dz0,    n->dz1,  n->y,    n->wpart, n->lscal, n->lnum, n->lden,
                  n->ebuf,   n->desc};
  for (void* p : ptrs)
    if (p) (void)hipFree(p);
  for (int l = 0; l < gkb::kMaxLayers; ++l)
    if (n->act[l]) (void)hipFree(n->act[l]);
  if (n->s) (void)hipStreamDestroy(n->s);
  delete n;
}

long gkb_cnn_param_count(const gkb_cnn* n) { return n ? n->np : -1; }

int gkb_cnn_set_params(gkb_cnn* n, const float* hp) {
  if (!n || !hp) return GKB_EINVAL;
  CNNCK(cnn_copy(n, n->params, hp, n->np * 4, hipMemcpyHostToDevice));
  n->weights_dirty = true;
  return GKB_OK;
}

int gkb_cnn_get_params(const gkb_cnn* n, float* hp) {
  if (!n || !hp) return GKB_EINVAL;
  CNNCK(cnn_copy(const_cast<gkb_cnn*>(n), hp, n->params, n->np * 4, hipMemcpyDeviceToHost));
  return GKB_OK;
}

int gkb_cnn_forward(gkb_cnn* n, int nx, int ny, int nz, int batch, const float* x, float* y) {
  // inputs may come from any stream: wait for all submitted device work
  CNNCK(hipDeviceSynchronize());
  if (!n || !x || !y || nx < 1 || ny < 1 || nz < 1 || batch < 1 || (n->dim == 2 && nz != 1))
    return GKB_EINVAL;
  gkb::CnnGeom g{nx, ny, nz, batch, (long)nx * ny * nz * batch};
  int rc = cnn_reserve(n, g.P);
  if (rc) return rc;
  // a single layer reads x while it writes y: where they overlap, y is formed
  // in the network's own buffer
  const size_t bx = g.P * n->ch[0] * sizeof(float), by = g.P * n->ch[n->L] * sizeof(float);
  const bool own = n->L == 1 && gkb::overlap(x, bx, y, by);
  rc = cnn_forward(n, g, gkb::ConvIn{x, n->ch[0], true}, own ? n->y : y);
  if (rc) return rc;
  if (own) CNNCK(hipMemcpyAsync(y, n->y, by, hipMemcpyDeviceToDevice, n->s));
  CNNCK(hipStreamSynchronize(n->s));
  return GKB_OK;
}

int gkb_cnn_backward(gkb_cnn* n, int nx, int ny, int nz, int batch, const float* x,
                     const float* dy, float* dx, float* grad_host) {
  // inputs may come from any stream: wait for all submitted device work
  CNNCK(hipDeviceSynchronize());
  if (!n || !x || !dy || nx < 1 || ny < 1 || nz < 1 || batch < 1 || (n->dim == 2 && nz != 1))
    return GKB_EINVAL;
  gkb::CnnGeom g{nx, ny, nz, batch, (long)nx * ny * nz * batch};
  int rc = cnn_reserve(n, g.P);
  if (rc) return rc;
  const gkb::ConvIn in{x, n->ch[0], true};
  rc = cnn_forward(n, g, in, nullptr);  // the output itself is not needed
  if (rc) return rc;
  // a single layer reads dy while it writes dx: where they overlap, it reads a
  // copy (the network's output buffer is free)
  const size_t bx = g.P * n->ch[0] * sizeof(float), by = g.P * n->ch[n->L] * sizeof(float);
  if (n->L == 1 && dx && gkb::overlap(dx, bx, dy, by)) {
    CNNCK(hipMemcpyAsync(n->y, dy, by, hipMemcpyDeviceToDevice, n->s));
    dy = n->y;
  }
  rc = cnn_backward(n, g, in, gkb::ConvIn{dy, n->ch[n->L], true}, dx);
  if (rc) return rc;
  if (grad_host) CNNCK(hipMemcpyAsync(grad_host, n->grad, n->np * 4, hipMemcpyDeviceToHost, n->s));
  CNNCK(hipStreamSynchronize(n->s));
  return GKB_OK;
}

int gkb_cnn_adam_step(gkb_cnn* n, const float* grad_host, double lr, double b1, double b2,
                      double eps) {
  if (!n) return GKB_EINVAL;
  if (grad_host) CNNCK(cnn_copy(n, n->grad, grad_host, n->np * 4, hipMemcpyHostToDevice));
  int rc = cnn_adam(n, lr, b1, b2, eps);
  if (rc) return rc;
  CNNCK(hipStreamSynchronize(n->s));
  return GKB_OK;
}

int gkb_cnn_train(gkb_cnn* n, const float* inputs, const float* targets, int n_pairs, int nx,
                  int ny, int nz, int crop, int batch, int steps, double lr, unsigned seed,
                  float* loss_host) {
  // inputs may come from any stream: wait for all submitted device work
  CNNCK(hipDeviceSynchronize());
  if (!n || !inputs || !targets || n_pairs < 1 || batch < 1 || batch > 1024 || steps < 0 ||
      crop < 3 || crop > nx || crop > ny || (n->dim == 3 && crop > nz) || (n->dim == 2 && nz != 1))
    return GKB_EINVAL;
  const int dim = n->dim, cin = n->ch[0], cout = n->ch[n->L];
  const long Pc = (long)crop * crop * (dim == 3 ? crop : 1);
  gkb::CnnGeom g{crop, crop, dim == 3 ? crop : 1, batch, Pc * batch};
  int rc = cnn_reserve(n, g.P);
  if (rc) return rc;
  if (g.P * cout > n->ecap) {
    if (n->ebuf) (void)hipFree(n->ebuf);
    CNNCK(hipMalloc(&n->ebuf, g.P * cout * sizeof(float)));
    n->ecap = g.P * cout;
  }
  if (batch > n->dcap) {
    if (n->desc) (void)hipFree(n->desc);
    CNNCK(hipMalloc(&n->desc, batch * 4 * sizeof(int)));
    n->dcap = batch;
  }
  const int lblk = (int)std::max<long>(1, std::min<long>((Pc * cout + 255) / 256, 256));
  rc = cnn_loss_buffers(n, batch, lblk);
  if (rc) return rc;
  std::vector<int> desc(4 * batch);
  uint64_t st = 0xD1B54A32D192ED03ull ^ ((uint64_t)seed << 1);
  auto rnd = [&](int mod) {
    st = st * 6364136223846793005ull + 1442695040888963407ull;
    return int((st >> 33) % (uint64_t)mod);
  };
  double hl[1];
  for (int it = 0; it < steps; ++it) {
    for (int s = 0; s < batch; ++s) {
      desc[4 * s] = rnd(n_pairs);
      desc[4 * s + 1] = rnd(nx - crop + 1);
      desc[4 * s + 2] = rnd(ny - crop + 1);
      desc[4 * s + 3] = dim == 3 ? rnd(nz - crop + 1) : 0;
    }
    CNNCK(hipMemcpyAsync(n->desc, desc.data(), 4 * batch * sizeof(int), hipMemcpyHostToDevice, n->s));
    gkb::k_gather<<<dim3(cnn_grid(Pc), batch), 256, 0, n->s>>>(
        nx, ny, nz, dim, crop, cin, cout, inputs, targets, n->desc, n->act[0], n->ebuf);
    rc = cnn_forward(n, g, cnn_act0(n), n->y);
    if (rc) return rc;
    gkb::k_loss_part<<<dim3(lblk, batch), 256, 0, n->s>>>(Pc, cout, n->y, n->ebuf, n->lnum,
                                                          n->lden);
    gkb::k_loss_final<<<1, 256, 0, n->s>>>(batch, lblk, Pc * cout, n->lnum, n->lscal);
    gkb::k_loss_grad<<<cnn_grid(g.P * 4), 256, 0, n->s>>>(Pc, cout, batch, n->y, n->ebuf,
                                                           n->lscal, n->dz0);
    rc = cnn_backward(n, g, cnn_act0(n), gkb::ConvIn{n->dz0, cout, false}, nullptr);
    if (rc) return rc;
    rc = cnn_adam(n, lr, 0.9, 0.999, 1e-8);
    if (rc) return rc;
    if (loss_host) {
      CNNCK(hipMemcpyAsync(hl, n->lscal, sizeof(double), hipMemcpyDeviceToHost, n->s));
      CNNCK(hipStreamSynchronize(n->s));
      loss_host[it] = float(hl[0]);
    }
  }
  CNNCK(hipStreamSynchronize(n->s));
  return GKB_OK;
}

int gkb_cnn_eval(gkb_cnn* n, const float* inputs, const float* targets, int n_pairs, int nx,
                 int ny, int nz, double* loss) {
  // inputs may come from any stream: wait for all submitted device work
  CNNCK(hipDeviceSynchronize());
  if (!n || !inputs || !targets || !loss || n_pairs < 1 || (n->dim == 2 && nz != 1))
    return GKB_EINVAL;
  const int cin = n->ch[0], cout = n->ch[n->L];
  const long P = (long)nx * ny * nz;
  gkb::CnnGeom g{nx, ny, nz, 1, P};
  int rc = cnn_reserve(n, P);
  if (rc) return rc;
  const int lblk = (int)std::max<long>(1, std::min<long>((P * cout + 255) / 256, 256));
  rc = cnn_loss_buffers(n, 1, lblk);
  if (rc) return rc;
  double total = 0.0, hl[1];
  for (int k = 0; k < n_pairs; ++k) {
    rc = cnn_forward(n, g, gkb::ConvIn{inputs + (size_t)k * P * cin, cin, true}, n->y);
    if (rc) return rc;
    gkb::k_loss_part<<<dim3(lblk, 1), 256, 0, n->s>>>(P, cout, n->y,
                                                      targets + (size_t)k * P * cout, n->lnum,
                                                      n->lden);
    gkb::k_loss_final<<<1, 256, 0, n->s>>>(1, lblk, P * cout, n->lnum, n->lscal);
    CNNCK(hipMemcpyAsync(hl, n->lscal, sizeof(double), hipMemcpyDeviceToHost, n->s));
    CNNCK(hipStreamSynchronize(n->s));
    total += hl[0];
  }
  *loss = total / n_pairs;
  return GKB_OK;
}

int gkb_cnn_save(const gkb_cnn* n, const char* path) {
  if (!n || !path) return GKB_EINVAL;
  std::vector<float> p(n->np), m(n->np), v(n->np);
  gkb_cnn* nn = const_cast<gkb_cnn*>(n);
  CNNCK(cnn_copy(nn, p.data(), n->params, n->np * 4, hipMemcpyDeviceToHost));
  CNNCK(cnn_copy(nn, m.data(), n->m, n->np * 4, hipMemcpyDeviceToHost));
  CNNCK(cnn_copy(nn, v.data(), n->v, n->np * 4, hipMemcpyDeviceToHost));
  FILE* f = std::fopen(path, "wb");
  if (!f) return GKB_EINVAL;
  const char magic[8] = {'G', 'K', 'B', 'C', 'N', 'N', '0', '1'};
  int hdr[4 + gkb::kMaxLayers + 1] = {1, n->dim, n->L, n->adam_t};
  for (int l = 0; l <= n->L; ++l) hdr[4 + l] = n->ch[l];
  bool ok = std::fwrite(magic, 1, 8, f) == 8 && std::fwrite(hdr, sizeof(hdr), 1, f) == 1 &&
            std::fwrite(p.data(), 4, n->np, f) == (size_t)n->np &&
            std::fwrite(m.data(), 4, n->np, f) == (size_t)n->np &&
            std::fwrite(v.data(), 4, n->np, f) == (size_t)n->np;
  ok = (std::fclose(f) == 0) && ok;
  return ok ? GKB_OK : GKB_EINVAL;
}

int gkb_cnn_load(const char* path, gkb_cnn** out) {
  if (!path || !out) return GKB_EINVAL;
  FILE* f = std::fopen(path, "rb");
  if (!f) return GKB_EINVAL;
  char magic[8];
  int hdr[4 + gkb::kMaxLayers + 1];
  if (std::fread(magic, 1, 8, f) != 8 || std::memcmp(magic, "GKBCNN01", 8) != 0 ||
      std::fread(hdr, sizeof(hdr), 1, f) != 1 || hdr[0] != 1 || hdr[2] < 1 ||
      hdr[2] > gkb::kMaxLayers) {
    std::fclose(f);
    return GKB_EINVAL;
  }
  gkb_cnn* n = nullptr;
  int rc = gkb_cnn_create(hdr[1], hdr[2], hdr + 4, 0, &n);
  if (rc) {
    std::fclose(f);
    return rc;
  }
  std::vector<float> p(n->np), m(n->np), v(n->np);
  bool ok = std::fread(p.data(), 4, n->np, f) == (size_t)n->np &&
            std::fread(m.data(), 4, n->np, f) == (size_t)n->np &&
            std::fread(v.data(), 4, n->np, f) == (size_t)n->np;
  std::fclose(f);
  if (!ok) {
    gkb_cnn_destroy(n);
    return GKB_EINVAL;
  }
  n->adam_t = hdr[3];
  if (cnn_copy(n, n->params, p.data(), n->np * 4, hipMemcpyHostToDevice) != hipSuccess ||
      cnn_copy(n, n->m, m.data(), n->np * 4, hipMemcpyHostToDevice) != hipSuccess ||
      cnn_copy(n, n->v, v.data(), n->np * 4, hipMemcpyHostToDevice) != hipSuccess) {
    gkb_cnn_destroy(n);
    return GKB_EHIP;
  }
  *out = n;
  return GKB_OK;
}

}  // extern "C"

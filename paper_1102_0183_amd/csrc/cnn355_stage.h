// What the stage kernels share: the context of an image's step, the activation function, sums over a wavefront.
#pragma once
#include <hip/hip_runtime.h>

#if defined(__HIP_DEVICE_COMPILE__)
#define CNN_GLOBAL __attribute__((address_space(1)))
#endif
#include "cnn355_dev.h"

namespace cnn355 {

typedef CNN_GLOBAL float gfloat;  // a float in device (global) memory

// Scaled hyperbolic tangent of Sec. 4, constants as printed.
#define ACT_A 1.7159f
#define ACT_B 0.6666f
__device__ __forceinline__ float act_f(float a) { return ACT_A * tanhf(ACT_B * a); }
// Its derivative A B (1 - tanh^2(B a)) = 4 A B z / (1 + z)^2 with z = e^{-2B|a|}, from the sum a the unit
// received (the forward pass stores it wherever a delta can arrive: at the pooling winners and at the hidden
// fully connected units).  Written in terms of the output, A B - (B/A) y^2, the two terms cancel to 1e-3 of
// themselves at a saturated unit and fp32 keeps only 1e-4 of the result; here nothing cancels.
__device__ __forceinline__ float dact_pre_f(float a) {
  const float z = expf(-2.0f * ACT_B * fabsf(a));
  const float r = 1.0f / (1.0f + z);
  return (4.0f * ACT_A * ACT_B) * z * r * r;
}

struct Ctx {
  const gfloat* image;
  gfloat* probs_out;
  gfloat* grad_out;
  int label;
  int train;  // this image is trained on (0 for forward-only calls and for rejected labels)
  float lr;
};

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

__device__ __forceinline__ Ctx make_ctx(const ProgramDev& P, const RunArgs& a, long long t,
                                        StatusDev* status) {
  Ctx c;
  if (a.call) {   // a node of a replayed graph: the call's arguments lie in device memory
    const CNN_GLOBAL CallArgs& q = *a.call;
    const long long tq = q.t0 + a.t_local;
    c.image = q.images + tq * q.image_stride;
    c.probs_out = q.probs_out ? q.probs_out + tq * P.n_classes : nullptr;
    c.grad_out = nullptr;
    c.label = q.labels[tq];
    c.lr = q.lr;
    c.train = q.train;
  } else {
  c.image = a.images + t * a.image_stride;
  c.probs_out = a.probs_out ? a.probs_out + t * P.n_classes : nullptr;
  c.grad_out = a.grad_out;
  c.label = a.labels ? a.labels[t] : a.label_imm;
  c.lr = a.lr;
  c.train = a.train;
  }
  if (a.train && (c.label < 0 || c.label >= P.n_classes)) {
    // a label outside the classes: the image is skipped and the host is told
    c.train = 0;
    if (blockIdx.x == 0 && threadIdx.x == 0) status->bad_label = 1u;
  }
  return c;
}

// Work item of workgroup b of n when neighbouring items are to share an L2: workgroups go round the eight XCDs, so
// XCD x takes a run of consecutive items.
__device__ __forceinline__ int xcd_item(int b, int n) {
  const int x = b & 7, q = n >> 3, r = n & 7;
  return x * q + min(x, r) + (b >> 3);
}

}  // namespace cnn355

// Device code that the feed-forward kernels share: activations and bf16 packing.
#pragma once
#include "mfma_common.h"

namespace ssa {
namespace {

constexpr float GELU_C0 = 0.7978845608028654f, GELU_C1 = 0.044715f;
constexpr uint32_t OUTSIDE = 0x7ffffff0u;  // a lane offset past every descriptor's extent: the load returns zeros
constexpr int DEVICE_SCOPE = 16;           // cache policy of a buffer access (sc1): coherent between the XCDs

// gelu(z) = z (1 - r), r = 1 / (1 + exp(2u)), u = C0 (z + C1 z^3)   [0.5 (1 + tanh u) = 1 - r]
// gelu'(z) = (1 - r) (1 + 2 z r u'(z)), u'(z) = C0 (1 + 3 C1 z^2)      [1 - tanh^2 u = 4 r (1 - r)]
template <bool GRAD, int N>
__device__ inline void gelu_n(const float (&z)[N], float (&h)[N], float (&d)[N]) {
  constexpr float K0 = 2.f * LOG2E * GELU_C0, K1 = K0 * GELU_C1;
#pragma unroll
  for (int e = 0; e < N; ++e) {
    const float z2 = z[e] * z[e];
    const float r = __builtin_amdgcn_rcpf(1.f + fast_exp2(z[e] * fmaf(z2, K1, K0)));
    const float s = 1.f - r;
    h[e] = z[e] * s;
    if (GRAD) d[e] = s * fmaf(2.f * z[e] * r, fmaf(z2, 3.f * GELU_C0 * GELU_C1, GELU_C0), 1.f);
  }
}
template <bool GRAD, int N>
__device__ inline void relu_n(const float (&z)[N], float (&h)[N], float (&d)[N]) {
#pragma unroll
  for (int e = 0; e < N; ++e) {
    h[e] = fmaxf(z[e], 0.f);
    if (GRAD) d[e] = z[e] > 0.f ? 1.f : 0.f;
  }
}
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
// two / four fp32 -> bf16 (round to nearest even, the hardware conversion)
__device__ inline uint32_t pack2(float x, float y) {
  union { bf16x2 v; uint32_t u; } a;
  a.v = __builtin_convertvector(f32x2{x, y}, bf16x2);
  return a.u;
}
__device__ inline uint2 pack4(const float (&y)[4]) { return uint2{pack2(y[0], y[1]), pack2(y[2], y[3])}; }
__device__ inline void unpack4(uint2 u, float (&y)[4]) {
  y[0] = __uint_as_float(u.x << 16); y[1] = __uint_as_float(u.x & 0xffff0000u);
  y[2] = __uint_as_float(u.y << 16); y[3] = __uint_as_float(u.y & 0xffff0000u);
}

}  // namespace
}  // namespace ssa

// What the kernels of windows of 17 to 160 tokens share (win_fwd.hip, win_bwd.hip): a wavefront per block of 16 tokens, tensors of 32 columns in LDS.
#pragma once
#include "mfma_common.h"

namespace ssa {
namespace {

constexpr int WB_TOKEN = 64;  // bytes of a token of a tensor in LDS: four chunks of 16

typedef __attribute__((address_space(3))) void wb_lds_void;
typedef __attribute__((address_space(1))) void wb_glb_void;
typedef __attribute__((address_space(3))) s16x4 wb_lds_s16x4;

// Chunk c of token i sits at position c ^ wb_place(i): 16 consecutive tokens put a chunk at 16 different places of 256 bytes (reads along
// the head), and eight consecutive ones two neighbouring chunks at eight different places (transposed reads).
__device__ inline int wb_place(int i) { return ((i >> 1) & 2) | ((i >> 3) & 1); }

__device__ inline f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); }

// over the four 16-lane groups
__device__ inline float groups_max(float x) {
  auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return half_max(fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1])));
}
__device__ inline float groups_sum(float x) {
  auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return half_sum(__uint_as_float(r[0]) + __uint_as_float(r[1]));
}
// A lane's columns 16 db + 4 g .. + 3 of 32 (g = its 16-lane group) as 16 bytes of memory order, for column 8 * store_chunk(g) on: neighbouring
// groups exchange pieces.
__device__ inline u32x4 gather16(const uint2 (&x)[2]) {
  auto a = __builtin_amdgcn_permlane16_swap(x[0].x, x[1].x, false, false);
  auto c = __builtin_amdgcn_permlane16_swap(x[0].y, x[1].y, false, false);
  return u32x4{a[0], c[0], a[1], c[1]};
}
__device__ inline int store_chunk(int g) { return 2 * (g & 1) + (g >> 1); }

// does the row's region mask mask anything at all?  (uniform; most rows do not)
template <int NB>
__device__ inline bool ids_differ(const int* rid, int lane) {
  const int first = rid[0];
  int other = 0;
#pragma unroll
  for (int c = 0; c < (NB + 3) / 4; ++c) other |= rid[min(lane + 64 * c, 16 * NB - 1)] ^ first;
  return __builtin_amdgcn_ballot_w64(other != 0) != 0;
}

// Where a lane (r = lane % 16, g = lane / 16) reads: along the head, token r of a block, chunk g;
__device__ inline uint32_t wb_along(int r, int g) { return (uint32_t)(r * WB_TOKEN + ((g ^ wb_place(r)) << 4)); }
// transposed, token 4 g + r / 4 and the four columns 16 db + 4 (r % 4) on, for db = 0 (1: ^ 32).
__device__ inline uint32_t wb_across(int r, int g) {
  const int token = 4 * g + (r >> 2);
  return (uint32_t)(token * WB_TOKEN + ((((r & 3) >> 1) ^ wb_place(token)) << 4) + 8 * (r & 1));
}
__device__ inline bf16x8 wb_tr_pair(const char* at, int step, bool both) {
  union { s16x4 h[2]; bf16x8 v; } o;
  o.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((wb_lds_s16x4*)at);
  o.h[1] = s16x4{0, 0, 0, 0};
  if (both) o.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((wb_lds_s16x4*)(at + step));
  return o.v;
}
// columns 16 db .. of tokens 32 t + {0 .. 3, 16 .. 19} + 4 g of a tensor of NB blocks, transposed (zeros for a block past the last)
template <int NB>
__device__ inline bf16x8 wb_read_across(const char* tensor, uint32_t across, int t, int db) {
  return wb_tr_pair(tensor + (across ^ (uint32_t)(32 * db)) + 32 * WB_TOKEN * t, 16 * WB_TOKEN, 2 * t + 1 < NB);
}
__device__ inline void wb_barrier() {  // a bare one: __syncthreads() would wait for every load and store in flight
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// Packed bf16: the bias of query 16 w + lane % 16 (past S - 1: the last one again) and keys 16 c + 4 (lane / 16) .. + 3; -inf past the last key.  From a copy
// in this order (win_bias_pack_kernel), or gathered; `buffer`: LDS of 128 NB x 16 bytes that nothing has been put into.  Called by the whole work-group.
template <int NB>
__device__ inline void win_bias(const KP& p, const uint2* copy, char* buffer, int h, int w, int lane, uint32_t (&bz)[NB][2]) {
  const int g = lane >> 4, mc = min(16 * w + (lane & 15), p.S - 1), tid = 64 * w + lane;
  if (copy) {
#pragma unroll
    for (int c = 0; c < NB; ++c) {
      const uint2 x = copy[(((int64_t)(h - p.bc_h0) * NB + w) * NB + c) * 64 + lane];
      bz[c][0] = x.x;
      bz[c][1] = x.y;
    }
    return;
  }
  const uint16_t* m = (const uint16_t*)p.bias;
  uint32_t x[NB][4];
  if (p.bias_kind == 2) {
    uint16_t* table = (uint16_t*)buffer;
    int* place = (int*)(buffer + MAX_RELPOS_R * 2);
    static_assert(MAX_RELPOS_R * 2 + 64 * NB <= 2 * 16 * NB * WB_TOKEN, "the table fits the buffer");
    const int rowlen = 2 * p.win_w - 1, R = (2 * p.win_h - 1) * rowlen;
    if (tid < 16 * NB) {
      const int i = min(tid, p.S - 1);
      place[tid] = (i / p.win_w) * rowlen + i % p.win_w;
    }
    for (int i = tid; i < R; i += 64 * NB) table[i] = m[(int64_t)h * R + i];
    __syncthreads();
    const int c0 = (p.win_h - 1) * rowlen + p.win_w - 1 + place[mc];
#pragma unroll
    for (int c = 0; c < NB; ++c) {
      const int4 k = *(const int4*)(place + 16 * c + 4 * g);
      x[c][0] = table[c0 - k.x]; x[c][1] = table[c0 - k.y]; x[c][2] = table[c0 - k.z]; x[c][3] = table[c0 - k.w];
    }
    __syncthreads();  // the buffer is free again
  } else {
    // four entries at a time, at any alignment; the last block's one by one: they may end with the matrix
    typedef __attribute__((ext_vector_type(2))) uint32_t u32x2_any __attribute__((aligned(2)));
    m += ((int64_t)h * p.S + mc) * p.S + 4 * g;
#pragma unroll
    for (int c = 0; c < NB - 1; ++c) {
      const u32x2_any y = *(const u32x2_any*)(m + 16 * c);
      x[c][0] = y[0] & 0xffffu; x[c][1] = y[0] >> 16; x[c][2] = y[1] & 0xffffu; x[c][3] = y[1] >> 16;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) x[NB - 1][e] = m[min(16 * (NB - 1) + e, p.S - 1 - 4 * g)];
  }
#pragma unroll
  for (int c = 0; c < NB; ++c) {
    if (c == NB - 1)
#pragma unroll
      for (int e = 0; e < 4; ++e) x[c][e] = 16 * c + 4 * g + e < p.S ? x[c][e] : 0xff80u;
    bz[c][0] = x[c][0] | x[c][1] << 16;
    bz[c][1] = x[c][2] | x[c][3] << 16;
  }
}

}  // namespace
}  // namespace ssa

// The copies of a dense bias that the kernels of head size 32 start their scores from (BiasCopy in mfma_common.h): who
// takes them, and the kernel that makes them.
#pragma once
#include "mfma_common.h"

namespace ssa {
namespace {

// Bytes of a copy of the bias of `heads` heads, if the forward (by query) or the backward (by key) of `rows` rows is faster
// with it, else 0.  For head size 32 without a causal mask on the large-share shapes, slices within 32-bit offsets, and
// where the scores are enough to pay for the launch (some 6 us with the library's buffer) and for the pass over the bias.
// Forward without | with the copy, us: 128 rows x 8 heads x 384: 65.6 | 66.5, 256 rows 127.3 | 120.6; 128 x 4 x 1024: 188 | 176,
// 256 rows 373 | 329; odd lengths, whose parked tiles are loaded unaligned: 64 x 8 x 501: 58.0 | 58.3, 512 x 4 x 301: 107 | 92.
// Backward: dK / dV 9 % shorter (1024 x 4 x 1024: 2037 -> 1850 us), and the copy replaces the transposed bf16 one; the
// recompute + dQ kernel gains nothing from a copy of its own (2469 | 2510).
// Windows (win_fwd.hip, win_bwd.hip: packed bf16): a dense bias only.  Without a copy a work-group gathers it from the matrix; without | with, us, 12 x 12 tokens with
// regions, 64 x 8 and 512 x 8 rows x heads: forward 27.3 | 18.4, 65.9 | 54.8, backward 44.3 | 40.5, 128 | 126 (11 x 11, 512 x 8: 90 | 92).  From a table, which a
// work-group gathers in LDS, the copy's launch costs more than it saves: forward, 64 x 8 11.0 | 16.7, 512 x 8 49.7 | 53.7,
// 256 x 24 59.3 | 65.0, 1024 x 16 162.8 | 167.3, 512 x 8 of 10 x 16 40.6 | 45.7; backward 3 us.
inline int64_t win_packed_bytes(int S, int heads) { return (int64_t)heads * ((S + 15) / 16) * ((S + 15) / 16) * 512; }
inline size_t bias_copy_bytes_for(const KP& p, bool backward, int64_t rows, int heads) {
  if (win_ok(p)) {
    if (p.bias_kind != 1 || (!backward && p.S <= 128) || rows * heads < (backward ? (p.S <= 128 ? 1024 : 64) : 512)) return 0;
    return (size_t)win_packed_bytes(p.S, heads);
  }
  if (row_ok(p, !backward) || !pair_fwd_ok(p) || p.S > 16384) return 0;
  const int64_t row_stride = p.ss > (int64_t)p.H * p.D ? p.ss : (int64_t)p.H * p.D;
  if (((int64_t)(p.S - 1) * row_stride + p.D) * 2 >= (1ll << 31)) return 0;
  const int64_t entries = (int64_t)heads * p.S * p.S;
  const int64_t enough = backward ? 1ll << 28 : p.S & 1 ? (1ll << 26) + 32 * entries : (1ll << 27) + 64 * entries;
  return rows * entries < enough ? 0 : (size_t)bias_copy_bytes(p.S, heads);
}

// BiasCopy: four wavefronts, a 32 x 32 block each.  1024 x 1024 x 4 heads: 8 MiB in, 16 out.
__global__ __launch_bounds__(256) void bias_copy_kernel(const uint16_t* src, float* dst, int S, int h0, int by_key, float inv_scale) {
  const int lane = threadIdx.x & 63, block = blockIdx.x * 4 + (threadIdx.x >> 6), strip = blockIdx.y;
  if (block >= bias_copy_blocks(S)) return;
  const uint16_t* m = src + (int64_t)(h0 + blockIdx.z) * S * S;
  f32x4* out = (f32x4*)dst + ((blockIdx.z * bias_copy_strips(S) + strip) * bias_copy_blocks(S) + block) * 256 + lane;
  const int row = 32 * strip + (lane & 31), col = 32 * block + 4 * (lane >> 5);
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    f32x4 x;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int c = col + 8 * g + e, r = min(row, S - 1), cc = min(c, S - 1);
      const float b = bf2f(m[by_key ? (int64_t)cc * S + r : (int64_t)r * S + cc]);
      x[e] = row < S && c < S ? b * inv_scale : -INFINITY;
    }
    out[64 * g] = x;
  }
}
// What the kernels of windows read (win_common.h): bf16, blocks of 16 queries x 16 keys, lane l the query l % 16 and four keys from 4 (l / 16) on; -inf
// past the last key.  x = block of keys, y = block of queries, z = head.
__global__ __launch_bounds__(64) void win_bias_pack_kernel(KP p, uint2* dst) {
  const int lane = threadIdx.x, i = min(16 * (int)blockIdx.y + (lane & 15), p.S - 1), j0 = 16 * blockIdx.x + 4 * (lane >> 4);
  const uint16_t* row = (const uint16_t*)p.bias + ((int64_t)(p.bc_h0 + blockIdx.z) * p.S + i) * p.S;
  uint32_t x[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) x[e] = j0 + e < p.S ? row[min(j0 + e, p.S - 1)] : 0xff80u;
  dst[((blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x) * 64 + lane] = uint2{x[0] | x[1] << 16, x[2] | x[3] << 16};
}
// Makes the copy that bias_copy_bytes_for asks for, of the heads [h0, h1), and points `p` at it.
inline hipError_t launch_bias_copies(KP& p, float* copy, bool backward, int h0, int h1, hipStream_t st) {
  const int heads = h1 - h0;
  p.bc_h0 = h0;
  const dim3 g((unsigned)((bias_copy_blocks(p.S) + 3) / 4), (unsigned)bias_copy_strips(p.S), heads);
  if (win_ok(p)) win_bias_pack_kernel<<<dim3((p.S + 15) / 16, (p.S + 15) / 16, heads), 64, 0, st>>>(p, (uint2*)copy);
  else bias_copy_kernel<<<g, 256, 0, st>>>((const uint16_t*)p.bias, copy, p.S, h0, backward ? 1 : 0, p.inv_scale);
  if (backward) p.bias_k = copy;
  else p.bias_q = copy;
  return hipGetLastError();
}

}  // namespace
}  // namespace ssa

// The gradient of a relative-position table from the partial sums of dS that groups of rows left (short rows and windows).
#pragma once
#include "mfma_common.h"

namespace ssa {
namespace {

// Two steps: the groups of a slice (consecutive, which ones depends on the share only) are summed in ascending order, entry by entry, and the
// S x S sum is reduced to the table; then the slices' tables are summed in ascending order.  The additions are the same for every k.
//
// Bound by reading the partial sums: a work-group takes some S / Z queries of a slice and head, sums them into LDS and leaves their part of the table where they were.
// Reducing the slices to one S x S sum and that to the table took three kernels, of which the second read the slices' sums again and the third had two
// wavefronts a compute unit: backward of 64 windows of 12 x 12 tokens x 8 heads 40.1 -> 38.4 us, 512 131.6 -> 128.4, 128 of 7 x 7 32.2 -> 27.8,
// 4096 x 16 469 -> 466.  The second step alone, with one read under way instead of 16: 7.4 against 4.0.
typedef f32x4 f32x4_at4 __attribute__((aligned(4)));

constexpr int FOLD_ELEMS = 40 * 160;  // S <= 64: 32 x 64; S <= 160: 40 x 160
inline int fold_parts(int S) { return S > 64 ? 4 : S >= 16 ? 2 : 1; }  // a part's table fits its place: (2 a - 1) (2 b - 1) < 4 S <= S / Z * S from 4 tokens on; 1, 2 and 3 have 1, 3 and 5 entries of S * S

// Q runs of four entries a thread
template <int Q>
__global__ __launch_bounds__(256) void slice_table_kernel(float* partial, int ring, int hs, int S, int slice, int s0, int ngroups, int win_h, int win_w) {
  __shared__ __attribute__((aligned(16))) float sum[FOLD_ELEMS];
  const int tid = threadIdx.x, Z = gridDim.z, i0 = S * blockIdx.z / Z, i1 = S * (blockIdx.z + 1) / Z, n = (i1 - i0) * S;
  const int g0 = (s0 + blockIdx.x) * slice, g1 = min(g0 + slice, ngroups);
  const int64_t gs = (int64_t)hs * S * S, at = (int64_t)blockIdx.y * S * S + i0 * S;
  if (n >= 4) {
    int from[Q];  // the last run ends with the part, what it shares with the one before is the same sum
    f32x4 a[Q];
#pragma unroll
    for (int i = 0; i < Q; ++i) {
      from[i] = min(4 * (tid + 256 * i), n - 4);
      a[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    int slot = g0 % ring;
#pragma unroll 4
    for (int g = g0; g < g1; ++g) {
      const float* x = partial + slot * gs + at;
#pragma unroll
      for (int i = 0; i < Q; ++i) {
        const f32x4 v = *(const f32x4_at4*)(x + from[i]);
#pragma unroll
        for (int e = 0; e < 4; ++e) a[i][e] += v[e];
      }
      slot = slot + 1 == ring ? 0 : slot + 1;
    }
#pragma unroll
    for (int i = 0; i < Q; ++i) *(f32x4_at4*)(sum + from[i]) = a[i];
  } else if (tid < n) {
    float a = 0.f;
    for (int g = g0; g < g1; ++g) a += partial[(g % ring) * gs + at + tid];
    sum[tid] = a;
  }
  __syncthreads();
  float* table = partial + (g0 % ring) * gs + at;
  const int rowlen = 2 * win_w - 1, R = (2 * win_h - 1) * rowlen, l = tid & 3;
  const int y0 = i0 / win_w, y1 = (i1 - 1) / win_w + 1;
  const float per_row = 1.f / rowlen;
  for (int r = tid >> 2; r < R; r += 64) {  // four lanes an entry
    const int row = (int)((r + 0.5f) * per_row);  // r / rowlen: half a step is far more than the product's rounding
    const int dy = row - (win_h - 1), dx = r - row * rowlen - (win_w - 1);
    // queries (y, x) with a partner inside the window, those of this part
    const int ylo = max(max(dy, 0), y0), yhi = min(min(win_h + dy, win_h), y1), xlo = max(dx, 0), xhi = min(win_w + dx, win_w);
    const int back = dy * win_w + dx;
    float v = 0.f;
    for (int y = ylo + l; y < yhi; y += 4) {
      const int lo = max(y * win_w + xlo, i0), hi = min(y * win_w + xhi, i1);
      for (int i = lo; i < hi; i += 6) {  // six reads under way
        float x[6];
#pragma unroll
        for (int e = 0; e < 6; ++e) x[e] = sum[(min(i + e, hi - 1) - i0) * S + min(i + e, hi - 1) - back];
#pragma unroll
        for (int e = 0; e < 6; ++e) v += i + e < hi ? x[e] : 0.f;
      }
    }
    v += __shfl_xor(v, 1, 64);
    v += __shfl_xor(v, 2, 64);
    if (l == 0) table[r] = v;
  }
}
// four lanes an entry, one part each
__global__ __launch_bounds__(64) void table_sum_kernel(const float* partial, float* table, int ring, int hs, int hd0, int nh, int S, int R, int slice, int s0, int s1,
                                                       int Z, int first) {
  const int t = blockIdx.x * 16 + (threadIdx.x >> 2), z = threadIdx.x & 3;
  const int hh = t / R, r = t - hh * R;
  const bool live = t < nh * R;
  const bool has = live && z < Z;
  const float* from = partial + (has ? (int64_t)hh * S * S + S * z / Z * S + r : 0);
  const int64_t gs = (int64_t)hs * S * S;
  float* out = table + (live ? (int64_t)(hd0 + hh) * R + r : 0);
  float v = first || !live ? 0.f : *out;
  int slot = s0 * slice % ring;
  constexpr int N = 16;  // loads under way
  for (int s = s0; s < s1; s += N) {
    float x[N];
#pragma unroll
    for (int e = 0; e < N; ++e) {
      x[e] = has && s + e < s1 ? from[slot * gs] : 0.f;
      slot += slice;
      while (slot >= ring) slot -= ring;
    }
#pragma unroll
    for (int e = 0; e < N; ++e) {  // slice after slice, whatever the chunk that it came from
      x[e] += __shfl_xor(x[e], 1, 64);
      x[e] += __shfl_xor(x[e], 2, 64);
      v += x[e];
    }
  }
  if (live && z == 0) *out = v;
}

// Adds the complete slices [s0, s1) of heads hd0 .. hd0 + nh - 1 to the table (which starts from zero when `first`); arguments as of launch_group_fold.
inline hipError_t launch_table_slices(float* partial, int ring, int hs, int nh, int S, int slice, int s0, int s1, int ngroups, int win_h, int win_w, hipStream_t st) {
  const dim3 grid(s1 - s0, nh, fold_parts(S));
  const int most = (S + (int)grid.z - 1) / (int)grid.z * S;  // entries of a part
  auto go = [&](auto q) { slice_table_kernel<q()><<<grid, 256, 0, st>>>(partial, ring, hs, S, slice, s0, ngroups, win_h, win_w); };
  if (most <= 2048) go(std::integral_constant<int, 2>{});
  else if (most <= 4096) go(std::integral_constant<int, 4>{});
  else go(std::integral_constant<int, 7>{});
  return hipGetLastError();
}
inline hipError_t launch_table_sum(const float* partial, float* table, int ring, int hs, int hd0, int nh, int S, int slice, int s0, int s1, int win_h, int win_w,
                                   bool first, hipStream_t st) {
  const int R = (2 * win_h - 1) * (2 * win_w - 1);
  table_sum_kernel<<<(nh * R + 15) / 16, 64, 0, st>>>(partial, table, ring, hs, hd0, nh, S, R, slice, s0, s1, fold_parts(S), first ? 1 : 0);
  return hipGetLastError();
}

}  // namespace
}  // namespace ssa

// C[M,N] = A[M,K] B[K,N] for a few rows of A (M <= 64): the products of a feed-forward share that
// serves a few tokens at a time.
#include "ffn_kernels.h"

#include "ffn_common.h"

namespace ssa {
namespace {

// What bounds it: reading B once, and for small B the time to start.  A work-group takes 16 NW columns and
// its WV wavefronts deal a part of the contraction out among themselves, 32 rows of B at a time, so that
// every wavefront has DEPTH steps of loads in flight; their sums meet in LDS in wavefront order, and the
// sums of a tile's g.split parts (work-groups of their own) in g.parts.  A compute unit gets only
// some 35 GB/s out of 128-byte pieces this way, so the parts have to cover all of them.  Forward of 16
// tokens x 12288 x 6144 (302 MB of weights): 162 -> 75 us, 4.0 TB/s; 16 x 1760 x 1624: 32 -> 14 us; 1 x 768 x
// 768: 18 -> 9 us (before: one tile of the tiled kernel per 128 columns).
//
// B goes from memory to registers without LDS: lane (c = lane % 16, g = lane / 16) loads NW columns of
// 8 consecutive rows, turns them in place into NW fragments of 8 contraction indexes (v_perm, 4 per
// fragment) and feeds each to v_mfma_f32_16x16x32_bf16 as the row operand of column NW c + j.  A lane
// ends up with the token lane % 16 and 4 NW consecutive columns.
template <int NW> struct BRow;
template <> struct BRow<4> { typedef u32x2 type; };
template <> struct BRow<2> { typedef uint32_t type; };

template <int NW>
__device__ inline typename BRow<NW>::type load_b(__amdgpu_buffer_rsrc_t rs, uint32_t off) {
  if constexpr (NW == 4) return __builtin_amdgcn_raw_buffer_load_b64(rs, off, 0, 0);
  else return __builtin_amdgcn_raw_buffer_load_b32(rs, off, 0, 0);
}

template <int TB, int NW, int WV, int DEPTH, int EPI>
__global__ __launch_bounds__(64 * WV) void skinny_kernel(GemmArgs g) {
  typedef typename BRow<NW>::type brow;
  constexpr int COLS = 16 * NW, LD = COLS + 4;
  __shared__ __attribute__((aligned(16))) float part_sum[WV * 16 * LD];
  const int tid = threadIdx.x, lane = tid & 63, c = lane & 15, q = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  // neighbouring tiles share cache lines of B: keep them on one XCD (work-groups go round the 8 XCDs)
  const int tiles = (g.N + COLS - 1) / COLS, b = (int)blockIdx.x % tiles, xcd = b % 8;
  const int tile = xcd * (tiles / 8) + min(xcd, tiles % 8) + b / 8, n0 = tile * COLS;

  // Lane offsets inside a step are the same for every step: a step is a descriptor that starts at its
  // first row of B / column of A and ends with the matrix, so rows of B past the contraction read as
  // zeros; the columns of A past it are left out by the lane.
  const uint32_t ldb2 = (uint32_t)g.ldb * 2u, lda2 = (uint32_t)g.lda * 2u;
  const int64_t bbytes = ((int64_t)(g.K - 1) * g.ldb + g.N) * 2, abytes = ((int64_t)(g.M - 1) * g.lda + g.K) * 2;
  uint32_t boff[8], aoff[TB];
#pragma unroll
  for (int e = 0; e < 8; ++e) boff[e] = (uint32_t)(8 * q + e) * ldb2 + (uint32_t)(n0 + NW * c) * 2u;
#pragma unroll
  for (int t = 0; t < TB; ++t) aoff[t] = 16 * t + c < g.M ? (uint32_t)(16 * t + c) * lda2 + 16u * q : OUTSIDE;
  const int klast = g.K - 8 * q - 8;  // the lane's columns of A are inside while 32 s <= klast

  brow rowb[DEPTH][8];
  u32x4 rowa[DEPTH][TB];
  // step s: contraction indexes 32 s .. 32 s + 31, this lane those from 32 s + 8 q on
  auto fetch = [&](int s, brow (&fb)[8], u32x4 (&fa)[TB]) {
    const int64_t bo = (int64_t)s * 32 * ldb2, ao = (int64_t)s * 64;
    const __amdgpu_buffer_rsrc_t rb =
        __builtin_amdgcn_make_buffer_rsrc((char*)g.B + bo, 0, bo < bbytes ? (int)(bbytes - bo) : 0, 0x00020000);
    const __amdgpu_buffer_rsrc_t ra =
        __builtin_amdgcn_make_buffer_rsrc((char*)g.A + ao, 0, ao < abytes ? (int)(abytes - ao) : 0, 0x00020000);
    const bool in = 32 * s <= klast;
#pragma unroll
    for (int t = 0; t < TB; ++t) fa[t] = __builtin_amdgcn_raw_buffer_load_b128(ra, in ? aoff[t] : OUTSIDE, 0, 0);
#pragma unroll
    for (int e = 0; e < 8; ++e) fb[e] = load_b<NW>(rb, boff[e]);
  };
  f32x4 acc[NW][TB];
  auto multiply = [&](brow (&fb)[8], u32x4 (&fa)[TB]) {
#pragma unroll
    for (int j = 0; j < NW; ++j) {
      union { uint32_t u[4]; bf16x8 v; } bf;
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        uint32_t lo, hi;
        if constexpr (NW == 4) { lo = fb[2 * p][j >> 1]; hi = fb[2 * p + 1][j >> 1]; }
        else { lo = fb[2 * p]; hi = fb[2 * p + 1]; }
        bf.u[p] = __builtin_amdgcn_perm(hi, lo, (j & 1) ? 0x07060302u : 0x05040100u);
      }
#pragma unroll
      for (int t = 0; t < TB; ++t) {
        union { u32x4 u; bf16x8 v; } af;
        af.u = fa[t];
        acc[j][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bf.v, af.v, acc[j][t], 0, 0, 0);
      }
    }
  };
  // what a thread sums up over the wavefronts: columns col, col + 1 of row `row` of every block of tokens
  constexpr int PAIRS = 16 * COLS / 2;
  static_assert(PAIRS <= 64 * WV, "one pair of columns per thread");
  const bool sums = tid < PAIRS;
  const int row = tid / (COLS / 2), col = 2 * (tid % (COLS / 2));
  f32x2 total[TB];

  const int parts = g.split, steps = (g.K + 31) / 32;
  const bool alone = parts > 1 && g.parts;  // one part per work-group; otherwise all of them in turn
  const int first = alone ? (int)blockIdx.x / tiles : 0, last = alone ? first + 1 : parts;
  const __amdgpu_buffer_rsrc_t rp = __builtin_amdgcn_make_buffer_rsrc(
      alone ? (char*)g.parts + (int64_t)tile * parts * (TB * PAIRS * 8) : nullptr, 0, alone ? parts * (TB * PAIRS * 8) : 0, 0x00020000);
  for (int part = first; part < last; ++part) {
#pragma unroll
    for (int j = 0; j < NW; ++j)
#pragma unroll
      for (int t = 0; t < TB; ++t) acc[j][t] = f32x4{0.f, 0.f, 0.f, 0.f};
    // the part's steps s0 .. s1 - 1, this wavefront's s0 + w, s0 + w + WV, ...
    const int s0 = (int)((int64_t)steps * part / parts), s1 = (int)((int64_t)steps * (part + 1) / parts);
    const int mine = (s1 - s0 - w + WV - 1) / WV;
    // steps past the end of the part: of no matrix, zeros
    auto step = [&](int i) { return i < mine ? s0 + w + i * WV : steps; };
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) {
      fetch(step(d), rowb[d], rowa[d]);
      __builtin_amdgcn_sched_barrier(0);
    }
    for (int i = 0; i < mine; i += DEPTH)
#pragma unroll
      for (int d = 0; d < DEPTH; ++d) {
        multiply(rowb[d], rowa[d]);
        fetch(step(i + d + DEPTH), rowb[d], rowa[d]);
        __builtin_amdgcn_sched_barrier(0);  // or the compiler gathers the loads of all DEPTH steps at the end
      }
#pragma unroll
    for (int t = 0; t < TB; ++t) {
      if (t || part > first) __syncthreads();
      float* mp = part_sum + (w * 16 + c) * LD + 4 * NW * q;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        if constexpr (NW == 4) *(f32x4*)(mp + 4 * v) = f32x4{acc[0][t][v], acc[1][t][v], acc[2][t][v], acc[3][t][v]};
        else *(f32x2*)(mp + 2 * v) = f32x2{acc[0][t][v], acc[1][t][v]};
      }
      __syncthreads();
      if (sums) {
        union { f32x2 f; u32x2 u; } s;
        s.f = *(const f32x2*)(part_sum + row * LD + col);
#pragma unroll
        for (int x = 1; x < WV; ++x) {
          const f32x2 y = *(const f32x2*)(part_sum + (x * 16 + row) * LD + col);
          s.f[0] += y[0];
          s.f[1] += y[1];
        }
        if (alone) __builtin_amdgcn_raw_buffer_store_b64(s.u, rp, (t * PAIRS + tid) * 8, first * (TB * PAIRS * 8), DEVICE_SCOPE);
        else if (part == first) total[t] = s.f;
        else { total[t][0] += s.f[0]; total[t][1] += s.f[1]; }
      }
    }
  }
  if (alone) {
    // the last part of a tile to finish adds the sums up, in the order of the parts (see gemm_kernel)
    __shared__ int is_last;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (tid == 0) {
      is_last = __hip_atomic_fetch_add(g.counters + tile, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (unsigned)parts - 1u;
      if (is_last) __hip_atomic_store(g.counters + tile, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    if (!is_last) return;
    if (sums)
      for (int part = 0; part < parts; ++part)
#pragma unroll
        for (int t = 0; t < TB; ++t) {
          union { u32x2 u; f32x2 f; } s;
          s.u = __builtin_amdgcn_raw_buffer_load_b64(rp, (t * PAIRS + tid) * 8, part * (TB * PAIRS * 8), DEVICE_SCOPE);
          if (part == 0) total[t] = s.f;
          else { total[t][0] += s.f[0]; total[t][1] += s.f[1]; }
        }
  }
  if (!sums) return;
#pragma unroll
  for (int t = 0; t < TB; ++t) {
    const int m = 16 * t + row, n = n0 + col;
    if (m >= g.M || n >= g.N) continue;
    float z[2] = {total[t][0], total[t][1]};
    uint32_t* out = (uint32_t*)(g.out + (int64_t)m * g.ldo + n);
    if (g.bias) {
      const uint32_t u = *(const uint32_t*)(g.bias + n);
      z[0] += __uint_as_float(u << 16);
      z[1] += __uint_as_float(u & 0xffff0000u);
    }
    if (EPI == EPI_ACC16 && g.accumulate) {
      z[0] += __uint_as_float(*out << 16);
      z[1] += __uint_as_float(*out & 0xffff0000u);
    }
    if (EPI == EPI_ACT) {
      float h[2], d[2];
      if (g.out2) {
        if (g.act == 0) relu_n<true>(z, h, d); else gelu_n<true>(z, h, d);
        *(uint32_t*)(g.out2 + (int64_t)m * g.ldo + n) = pack2(d[0], d[1]);
      } else {
        if (g.act == 0) relu_n<false>(z, h, d); else gelu_n<false>(z, h, d);
      }
      *out = pack2(h[0], h[1]);
    } else {
      *out = pack2(z[0], z[1]);
    }
  }
}

#define SS_SKINNY_INST(tb, nw, depth) \
  template __global__ void skinny_kernel<tb, nw, 8, depth, EPI_ACT>(GemmArgs); \
  template __global__ void skinny_kernel<tb, nw, 8, depth, EPI_ACC16>(GemmArgs);
SS_SKINNY_INST(1, 4, 3) SS_SKINNY_INST(1, 2, 4)
SS_SKINNY_INST(2, 4, 3) SS_SKINNY_INST(2, 2, 4)
SS_SKINNY_INST(4, 4, 2) SS_SKINNY_INST(4, 2, 3)
#undef SS_SKINNY_INST

template <int TB, int NW, int DEPTH>
hipError_t launch_one(const GemmArgs& g, int epi, hipStream_t st) {
  const int tiles = (g.N + 16 * NW - 1) / (16 * NW), grid = g.split > 1 && g.parts ? tiles * g.split : tiles;
  if (epi == EPI_ACT) skinny_kernel<TB, NW, 8, DEPTH, EPI_ACT><<<grid, 512, 0, st>>>(g);
  else skinny_kernel<TB, NW, 8, DEPTH, EPI_ACC16><<<grid, 512, 0, st>>>(g);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_skinny(const GemmArgs& g, int epi, hipStream_t st) {
  if (g.M > 64 || (epi != EPI_ACT && epi != EPI_ACC16)) return hipErrorInvalidValue;
  if (g.cols == 64) {
    if (g.M <= 16) return launch_one<1, 4, 3>(g, epi, st);
    return g.M <= 32 ? launch_one<2, 4, 3>(g, epi, st) : launch_one<4, 4, 2>(g, epi, st);
  }
  if (g.M <= 16) return launch_one<1, 2, 4>(g, epi, st);
  return g.M <= 32 ? launch_one<2, 2, 4>(g, epi, st) : launch_one<4, 2, 3>(g, epi, st);
}

}  // namespace ssa

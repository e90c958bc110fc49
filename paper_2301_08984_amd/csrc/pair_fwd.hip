// Forward at head size 32 with a dense bias (pair attention): NR rows b of one head per wavefront.
//
// A score costs two matrix steps for 32 x 32 of them but a bias entry each, and the bias is most of what a compute unit
// loads.  Where the share is large (bias_copy.h) the bias comes from a copy in accumulator layout: the scores start from
// it, so unpacking and adding it cost no vector instruction, and it passes no LDS.  That is 4 bytes an entry, and
// with one row per wavefront the launch was bound by what the L2s deliver (17 - 19 TB/s: 1290 us for 1024 rows x 4 heads x
// 1024); two rows share every entry.  1024 x 4 x 1024: 1312 -> 1050 us, 901 x 4 x 901: 1549 -> 845, 512 x 8 x 384: 245 -> 216
// (before: the general forward kernel, a parked bf16 tile per wavefront, a comparison per score for the maximum).
// Without the copy a wavefront takes one row and parks its bias tile in LDS, with the same arithmetic, bit for bit.
//
// Work-group: four wavefronts of 32 queries share the rows' 64-key K / V tiles (two buffers, one barrier per tile); a
// tile is two 32-key blocks, each a complete online-softmax step.  168 registers: three wavefronts per SIMD.
#include "mfma_common.h"

namespace ssa {
namespace {

constexpr int PD = 32, PLK = PD + 8, PLV = PD + 16;  // row pads chosen for conflict-free b128 / transpose reads
constexpr int PTILE = BN * (PLK + PLV);               // K and V of one row, 64 keys

template <int BIAS, int NR>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(BIAS == BIAS_COPY ? 3 : 4, BIAS == BIAS_COPY ? 3 : 4))) void pair_fwd_kernel(KP p, int together) {
#pragma clang fp contract(off)  // the variants are to give the same bits
  constexpr bool PARKED = BIAS != BIAS_COPY;
  constexpr int BLOCK_UNROLL = PARKED ? 1 : 2;
  __shared__ __attribute__((aligned(16))) uint16_t smem[2][NR][PTILE];  // buffer, row
  __shared__ __attribute__((aligned(16))) uint16_t parked[PARKED ? 4 * BIAS_TILE_ELEMS : 8];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, r = lane & 31, hl = lane >> 5;
  const BlockId blk = xcd_block_id(together);
  const int h = p.h0 + blk.y, q0 = blk.x * 128 + 32 * w, q = q0 + r, qc = min(q, p.S - 1);
  int64_t base[NR];
#pragma unroll
  for (int n = 0; n < NR; ++n) base[n] = (int64_t)min(p.b0 + NR * blk.z + n, p.b1 - 1) * p.sb + (int64_t)h * p.sh;
  BiasCopy bc;
  BiasTile<BIAS == BIAS_ODD> bt;
  f32x16 cz;  // bias / scale of the block, then of the next one
  if (PARKED) bt.init((const uint16_t*)p.bias + (int64_t)h * p.S * p.S, q0, p.S, parked + w * BIAS_TILE_ELEMS, lane);
  else bc.init(p.bias_q, h - p.bc_h0, q0, p.S, lane);
  const float inv_scale = in_vgpr(p.inv_scale);
  bf16x8 qf[NR][2];
#pragma unroll
  for (int n = 0; n < NR; ++n)
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
      qf[n][ks] = *(const bf16x8*)((const uint16_t*)p.Q + base[n] + (int64_t)qc * p.ss + 16 * ks + 8 * hl);
  f32x16 oacc[NR];
  float nm[NR], l[NR];  // the negated running maximum, the row sum
  RowMaxima<NR> maxima;
#pragma unroll
  for (int n = 0; n < NR; ++n) {
#pragma unroll
    for (int v = 0; v < 16; ++v) oacc[n][v] = 0.f;
    nm[n] = 1e30f;
    maxima.looks[n] = ~0ull;
    l[n] = 0.f;
  }
  const float c1 = in_vgpr(p.scale * LOG2E);
  const int ntiles = (p.S + BN - 1) / BN;

  // a thread's 16-byte chunk of a tile; rows past S - 1 arrive as zeros
  const uint32_t ss2 = (uint32_t)p.ss * 2u, slice = (uint32_t)(((int64_t)(p.S - 1) * p.ss + PD) * 2);
  const uint32_t goff = (uint32_t)(tid >> 2) * ss2 + (uint32_t)(tid & 3) * 16u;
  u32x4 pk[NR], pv[NR];
  auto gload = [&](int kt) {
    const uint32_t boff = (uint32_t)(kt * BN) * ss2;  // kt * BN < S
#pragma unroll
    for (int n = 0; n < NR; ++n) {
      const __amdgpu_buffer_rsrc_t rk = __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)p.K + 2 * base[n] + boff), 0, (int)(slice - boff), 0x00020000);
      const __amdgpu_buffer_rsrc_t rv = __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)p.V + 2 * base[n] + boff), 0, (int)(slice - boff), 0x00020000);
      pk[n] = __builtin_amdgcn_raw_buffer_load_b128(rk, goff, 0, 0);
      pv[n] = __builtin_amdgcn_raw_buffer_load_b128(rv, goff, 0, 0);
    }
  };
  auto stage = [&](int buf) {
#pragma unroll
    for (int n = 0; n < NR; ++n) {
      *(u32x4*)(smem[buf][n] + (tid >> 2) * PLK + (tid & 3) * 8) = pk[n];
      *(u32x4*)(smem[buf][n] + BN * PLK + (tid >> 2) * PLV + (tid & 3) * 8) = pv[n];
    }
  };
  // 32 keys; the running maximum as RowMaxima says
  auto block = [&](int buf, int kb, int at) __attribute__((always_inline)) {
    f32x16 s[NR];
    float sum[NR];
    for (bool again = false;; again = true) {
      // without this the compiler keeps a block's K fragments for a second time and loads the next block's early, beyond 128 registers: 24 and 16
      // bytes of scratch, and 1024 rows x 8 heads x 100 took 73 us (63 with it; 67 in the general forward), x 128 95 (87; 88), 1024 x 4 x 1024 1385 (1347; 1372)
      if (PARKED) asm volatile("" ::: "memory");
      if (PARKED) parked_bias(bt, r, kb, hl, inv_scale, cz);
#pragma unroll
      for (int n = 0; n < NR; ++n) {
        s[n] = cz;
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) s[n] = mfma(lds_nat<PLK>(smem[buf][n], 32 * kb + r, ks, hl), qf[n][ks], s[n]);
      }
      if (!PARKED) {
        bc.load(cz, min(at + 1, 2 * ntiles - 1));
      } else if (32 * at + 32 > p.S) {  // (the copy masks what lies past the end)
#pragma unroll
        for (int n = 0; n < NR; ++n)
#pragma unroll
          for (int v = 0; v < 16; ++v) s[n][v] = 32 * at + key_of(v, hl) >= p.S ? -INFINITY : s[n][v];
      }
      if (again || maxima.any()) {
#pragma unroll
        for (int n = 0; n < NR; ++n) {
          const float alpha = maxima.raise(n, s[n], c1, nm[n], at == 0, again, sum[n]);
          l[n] *= alpha;
#pragma unroll
          for (int v = 0; v < 16; ++v) oacc[n][v] *= alpha;
        }
      }
#pragma unroll
      for (int n = 0; n < NR; ++n) {
        float x[16];
#pragma unroll
        for (int v = 0; v < 16; ++v) x[v] = s[n][v] = fast_exp2(fmaf(s[n][v], c1, nm[n]));
        sum[n] = sum16(x);
      }
      const float top = fmaxf(sum[0], sum[NR - 1]);
      if (__builtin_amdgcn_ballot_w64(top > maxima.SCALE) == 0) break;
      if (again || __builtin_amdgcn_ballot_w64(top > maxima.RAISE) == 0) {
#pragma unroll
        for (int n = 0; n < NR; ++n) {
          const float f = maxima.scale(n, nm[n], sum[n]);
          sum[n] *= f;
          l[n] *= f;
#pragma unroll
          for (int v = 0; v < 16; ++v) { s[n][v] *= f; oacc[n][v] *= f; }
        }
        break;
      }
      if (!PARKED) bc.load(cz, at);
    }
#pragma unroll
    for (int n = 0; n < NR; ++n) {
      l[n] += sum[n];
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        float x[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] = s[n][8 * j + e];
        oacc[n] = mfma(lds_tr<PLV>(smem[buf][n] + BN * PLK, 32 * kb + 16 * j, 0, lane), pack8(x), oacc[n]);
      }
    }
  };

  gload(0);
  if (PARKED) bt.load(0);
  else bc.load(cz, 0);
  stage(0);
  if (PARKED) bt.park(lane);
  if (1 < ntiles) {
    gload(1);
    if (PARKED) bt.load(1);
  }
  __syncthreads();
  for (int kt = 0; kt < ntiles; ++kt) {
    if (q0 < p.S) {
#pragma unroll BLOCK_UNROLL
      for (int kb = 0; kb < 2; ++kb) block(kt & 1, kb, 2 * kt + kb);
    }
    if (kt + 1 < ntiles) {
      stage((kt + 1) & 1);
      if (PARKED) bt.park(lane);
      if (kt + 2 < ntiles) {
        gload(kt + 2);
        if (PARKED) bt.load(kt + 2);
      }
    }
    __syncthreads();
  }
#pragma unroll
  for (int n = 0; n < NR; ++n) {
    const int b = p.b0 + NR * blk.z + n;
    f32x16 o[1] = {oacc[n]};
    if (b < p.b1) fwd_epilogue<1, false>(p, o, -nm[n], l[n], b, h, q, hl, base[n]);
  }
}

}  // namespace

hipError_t launch_pair_fwd(const KP& p, hipStream_t st) {
  const int together = heads_together(p.h1 - p.h0, p.S, p.bias_q ? 4 : 2), rows = p.b1 - p.b0;
  auto grid = [&](int nr) { return dim3((p.S + 127) / 128, p.h1 - p.h0, (rows + nr - 1) / nr); };
  if (p.bias_q) pair_fwd_kernel<BIAS_COPY, 2><<<grid(2), 256, 0, st>>>(p, together);
  else if (p.S & 1) pair_fwd_kernel<BIAS_ODD, 1><<<grid(1), 256, 0, st>>>(p, together);
  else pair_fwd_kernel<BIAS_EVEN, 1><<<grid(1), 256, 0, st>>>(p, together);
  return hipGetLastError();
}

}  // namespace ssa

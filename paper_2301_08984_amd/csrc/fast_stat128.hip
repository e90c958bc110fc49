// The statistics of the backward for large shares at head size 128 without a bias or a gate: Delta_i = sum_j P_ij dP_ij, and the LSE unless the caller
// kept it.
//
// The recompute pass of fast_fwd128.hip forms O for Delta = dO . O; without a gate nobody else needs O.  Scores and dP give Delta as well, with both
// operands read along the rows (no transposed fragments, which cost LDS twice the time), no accumulators to keep, and so room for 64 queries a wavefront:
// a K or V fragment serves two query blocks, half of the LDS reads per matrix instruction.  And Delta is a sum of unrounded probabilities.
// A work-group of four wavefronts owns 128 queries and the tile buffers of fast_fwd128.hip; wavefronts 0 and 1 take the first 32 keys of every tile for the
// queries' halves, 2 and 3 the last 32, and hand maximum, sum and Delta over at the end.  Recompute pass | this, us: 12 heads x 12288, causal, 447 | 397; 12 x 4000
// 76.3 | 65.5; 40 x 1100 27.9 | 24.5; 64 x 400 14.7 | 14.0 (16.7 with Q and dO fragments straight from memory); no mask, 8 x 7000 203 | 176.  dQ of 48 heads x 4000
// against fp64: 2.378e-3 | 2.356e-3.
#include "wave_dma.h"

#include <type_traits>

namespace ssa {
namespace {

constexpr int S_STAGE_B = 4 * W_TILE_B;  // K rows 0..31, K rows 32..63, V rows 0..31, V rows 32..63

// four of the eight operand fragments (4 half ..) of the tile OFF bytes after the one the addresses were made for
template <int OFF, int HALF>
__device__ __forceinline__ void nat4_issue(u32x4 (&f)[4], const uint32_t (&ka)[8]) {
  asm volatile("ds_read_b128 %0, %4 offset:%8\n\tds_read_b128 %1, %5 offset:%8\n\tds_read_b128 %2, %6 offset:%8\n\tds_read_b128 %3, %7 offset:%8"
               : "=&v"(f[0]), "=&v"(f[1]), "=&v"(f[2]), "=&v"(f[3])
               : "v"(ka[4 * HALF]), "v"(ka[4 * HALF + 1]), "v"(ka[4 * HALF + 2]), "v"(ka[4 * HALF + 3]), "n"(OFF)
               : "memory");
}
__device__ __forceinline__ void nat4_wait(u32x4 (&f)[4]) {
  asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(f[0]), "+v"(f[1]), "+v"(f[2]), "+v"(f[3]) : : "memory");
}

// KEPT: the caller's LSE
template <bool CAUSAL, bool KEPT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void stat_fast128_kernel(KP p) {
  constexpr int D = 128, KS = D / 16, BM = 128, BN = 64;
  __shared__ __attribute__((aligned(1024))) char smem[2 * S_STAGE_B];
  const int lane = threadIdx.x & 63, r = lane & 31, hl = lane >> 5;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), qw = w & 1, kg = w >> 1;
  const BlockId blk = CAUSAL ? causal_block_id(true) : xcd_block_id();
  const int h = p.h0 + blk.y, b = p.b0 + blk.z;
  const int qblk = (gridDim.x - 1 - blk.x) * BM;  // long (late) causal blocks first
  const int q0 = qblk + 64 * qw;
  const int64_t base = (int64_t)b * p.sb + (int64_t)h * p.sh;
  const uint16_t* Kb = (const uint16_t*)p.K + base;
  const uint16_t* Vb = (const uint16_t*)p.V + base;
  const uint16_t* dOb = (const uint16_t*)p.dO + (int64_t)(b - p.do_b0) * p.do_sb + (int64_t)(h - p.do_h0) * p.do_sh;
  const float c1 = in_vgpr(p.scale * LOG2E);

  int ntiles = (p.S + BN - 1) / BN;
  if (CAUSAL) ntiles = min(ntiles, (min(qblk + BM, p.S) + BN - 1) / BN);

  // this wavefront's share of a tile: load instructions 2w and 2w+1 of each of its four sub-tiles
  const uint32_t ss2 = (uint32_t)p.ss * 2u;
  const uint32_t slice = (uint32_t)(((int64_t)(p.S - 1) * p.ss + D) * 2);  // < 2 GiB, checked on the host
  uint32_t goff[2];
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int rho = 4 * (2 * w + u) + (lane >> 4);
    goff[u] = (uint32_t)rho * ss2 + 16u * (uint32_t)((lane & 15) ^ w_sw(rho));
  }
  // 64 rows of two tensors from row0 and row1 on (a sub-tile past the last row: an empty descriptor, zeros arrive)
  auto fetch = [&](char* stage, const uint16_t* t0, int row0, const uint16_t* t1, int row1, uint32_t stride, uint32_t bytes, const uint32_t (&off)[2]) {
#pragma unroll
    for (int sub = 0; sub < 4; ++sub) {
      const int row = (sub < 2 ? row0 : row1) + 32 * (sub & 1);
      const uint32_t boff = row < p.S ? (uint32_t)row * stride : bytes;
      const __amdgpu_buffer_rsrc_t rs =
          __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)(sub < 2 ? t0 : t1) + boff), 0, (int)(bytes - boff), 0x00020000);
#pragma unroll
      for (int u = 0; u < 2; ++u)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (w_lds_void*)(stage + sub * W_TILE_B + (2 * w + u) * 1024), 16, off[u], 0, 0, 0);
    }
  };
  auto fetch_tile = [&](char* stage, int kt) { fetch(stage, Kb, kt * BN, Vb, kt * BN, ss2, slice, goff); };

  // Q and dO fragments, through the two buffers (straight from memory in operand layout an instruction touches 32 lines)
  u32x4 qf[2][KS], gf[2][KS];
  {
    const uint32_t dss2 = (uint32_t)p.do_ss * 2u, dslice = (uint32_t)(((int64_t)(p.S - 1) * p.do_ss + D) * 2);
    uint32_t goff_g[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) goff_g[u] = goff[u] + (uint32_t)(4 * (2 * w + u) + (lane >> 4)) * (dss2 - ss2);
    const uint16_t* Qb = (const uint16_t*)p.Q + base;
    fetch(smem, Qb, qblk, Qb, qblk + 64, ss2, slice, goff);
    fetch(smem + S_STAGE_B, dOb, qblk, dOb, qblk + 64, dss2, dslice, goff_g);
    uint32_t qa[8];
    w_nat_addr(qa, smem + 2 * qw * W_TILE_B, r, hl);
    W_VMCNT(0);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    w_nat_issue<0>(qf[0], qa);
    w_nat_issue<W_TILE_B>(qf[1], qa);
    w_nat_issue<S_STAGE_B>(gf[0], qa);
    w_nat_issue<S_STAGE_B + W_TILE_B>(gf[1], qa);
    w_nat_wait(qf[0]);
    w_nat_wait(qf[1]);
    w_nat_wait(gf[0]);
    w_nat_wait(gf[1]);
    __builtin_amdgcn_s_barrier();  // everybody's fragments are read
    asm volatile("" ::: "memory");
  }
  fetch_tile(smem, 0);
  uint32_t ka[8];
  w_nat_addr(ka, smem + kg * W_TILE_B, r, hl);
  float nm[2], l[2] = {0.f, 0.f}, d[2] = {0.f, 0.f};  // negated maximum (KEPT: LSE) in base-2 units; this half-wave's sums of p and p dP
#pragma unroll
  for (int i = 0; i < 2; ++i)
    nm[i] = KEPT ? -p.lse[(int64_t)(b - p.lse_b0) * p.lse_sb + (int64_t)(h - p.lse_h0) * p.lse_sh + min(q0 + 32 * i + r, p.S - 1)] * LOG2E : 1e30f;

  // this wavefront's 32 keys, from k0 on, of the tile in the stage buffer SB bytes into LDS
  auto tile = [&](auto sb, int k0) {
    constexpr int SB = decltype(sb)::value;
    f32x16 s[2], t[2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int v = 0; v < 16; ++v) { s[i][v] = 0.f; t[i][v] = 0.f; }
    u32x4 fa[4], fb[4];
    auto product = [&](f32x16 (&x)[2], const u32x4 (&f)[4], const u32x4 (&y)[2][KS], int half) {
#pragma unroll
      for (int ks = 0; ks < 4; ++ks)
#pragma unroll
        for (int i = 0; i < 2; ++i) x[i] = mfma(w_frag(f[ks]), w_frag(y[i][4 * half + ks]), x[i]);
    };
    nat4_issue<SB, 0>(fa, ka);
    nat4_wait(fa);
    nat4_issue<SB, 1>(fb, ka);
    __builtin_amdgcn_sched_barrier(0);  // (the reads stay in front of the products that cover them)
    product(s, fa, qf, 0);
    __builtin_amdgcn_sched_barrier(0);
    nat4_wait(fb);
    nat4_issue<SB + 2 * W_TILE_B, 0>(fa, ka);
    __builtin_amdgcn_sched_barrier(0);
    product(s, fb, qf, 1);
    __builtin_amdgcn_sched_barrier(0);
    nat4_wait(fa);
    nat4_issue<SB + 2 * W_TILE_B, 1>(fb, ka);
    __builtin_amdgcn_sched_barrier(0);
    product(t, fa, gf, 0);
    // the probabilities are formed under the products with V
    if ((k0 + 32 > p.S) || (CAUSAL && k0 + 31 > q0)) {
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int key = k0 + key_of(v, hl);
          const bool dead = key >= p.S || (CAUSAL && key > q0 + 32 * i + r);
          s[i][v] = dead ? -INFINITY : s[i][v];
        }
    }
    if (!KEPT) {
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        float rmax = -INFINITY;
#pragma unroll
        for (int v = 0; v < 16; ++v) rmax = fmaxf(rmax, s[i][v]);
        const float nn = fminf(nm[i], -half_max(rmax * c1)), alpha = fast_exp2(nn - nm[i]);  // scale > 0 on this path
        nm[i] = nn;
        l[i] *= alpha;
        d[i] *= alpha;
      }
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      float sum[2] = {0.f, 0.f};
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        s[i][v] = fast_exp2(fmaf(s[i][v], c1, nm[i]));
        if (!KEPT) sum[v & 1] += s[i][v];
      }
      if (!KEPT) l[i] += sum[0] + sum[1];
    }
    nat4_wait(fb);
    product(t, fb, gf, 1);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      float sum[2] = {0.f, 0.f};
#pragma unroll
      for (int v = 0; v < 16; ++v) sum[v & 1] = fmaf(s[i][v], t[i][v], sum[v & 1]);
      d[i] += sum[0] + sum[1];
    }
  };
  // step kt: tile kt is on its way into buffer kt % 2
  auto step = [&](auto sb, int kt) {
    constexpr int SB = decltype(sb)::value;
    W_VMCNT(0);  // this wavefront's part of tile kt has landed
    __builtin_amdgcn_s_barrier();  // ... everybody's; and everybody is done with the other buffer
    asm volatile("" ::: "memory");
    if (kt + 1 < ntiles) fetch_tile(smem + (S_STAGE_B - SB), kt + 1);
    const int k0 = kt * BN + 32 * kg;
    if (q0 < p.S && k0 < p.S && !(CAUSAL && k0 > q0 + 63)) tile(sb, k0);  // else no visible pair for this wavefront
  };
  int kt = 0;
  for (; kt + 1 < ntiles; kt += 2) {
    step(std::integral_constant<int, 0>{}, kt);
    step(std::integral_constant<int, S_STAGE_B>{}, kt + 1);
  }
  if (kt < ntiles) step(std::integral_constant<int, 0>{}, kt);

  // the two key groups' parts: [query half][block][maximum, sum, Delta][32]
  float* part = (float*)smem + qw * 192;
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    l[i] = half_sum(l[i]);
    d[i] = half_sum(d[i]);
    if (kg == 1 && hl == 0) {
      part[96 * i + r] = nm[i];
      part[96 * i + 32 + r] = l[i];
      part[96 * i + 64 + r] = d[i];
    }
  }
  __syncthreads();
  if (kg == 1 || hl == 1) return;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int q = q0 + 32 * i + r;
    if (q >= p.S) continue;
    const float nm1 = part[96 * i + r], l1 = part[96 * i + 32 + r], d1 = part[96 * i + 64 + r];
    float delta;
    if (KEPT) {
      delta = d[i] + d1;
    } else {
      const float nn = fminf(nm[i], nm1), a0 = fast_exp2(nn - nm[i]), a1 = fast_exp2(nn - nm1);
      const float sum = fmaf(a1, l1, a0 * l[i]);
      delta = fmaf(a1, d1, a0 * d[i]) / sum;
      p.lse_out[(int64_t)(b - p.lse_b0) * p.lse_sb + (int64_t)(h - p.lse_h0) * p.lse_sh + q] = (log2f(sum) - nn) * LN2;
    }
    p.delta[(int64_t)(b - p.dl_b0) * p.dl_sb + (int64_t)(h - p.dl_h0) * p.dl_sh + q] = delta;
  }
}

}  // namespace

hipError_t launch_fast_stat128(const KP& p, hipStream_t st) {
  const dim3 g((p.S + 127) / 128, p.h1 - p.h0, p.b1 - p.b0);
  auto with = [&](auto causal) {
    if (p.lse_out) stat_fast128_kernel<causal(), false><<<g, 256, 0, st>>>(p);
    else stat_fast128_kernel<causal(), true><<<g, 256, 0, st>>>(p);
  };
  if (p.mask_kind == 1) with(std::true_type{});
  else with(std::false_type{});
  return hipGetLastError();
}

}  // namespace ssa

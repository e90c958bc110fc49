// dK and dV for large shares at head size 128 without a bias: a wavefront for each gradient, the probabilities handed over through LDS.
//
// A key-stationary wavefront with both accumulators (128 registers) and the K and V fragments of its 32 keys needs more than 400 registers and
// runs alone on its SIMD; with one gradient per work-group, as this kernel was before, the scores and their exponentials are formed
// twice.  Here a work-group of eight wavefronts owns 128 keys.  Of the two wavefronts of a 32-key block the first forms S = Q K^T and P, hands
// P over in fp32 (accumulator layout, 4 KB) and adds dO^T P to dV; the second forms dP = dO V^T, takes P a step
// later, forms dS and adds Q^T dS to dK: four contractions in all instead of five, half of the exponentials, each wavefront within 256 registers.
// The queries go by in steps of 32: their Q and dO sub-tiles (wave_dma.h) travel straight into a ring of four LDS slots, two steps ahead, with one
// barrier a step; the second wavefronts are a step behind the first ones.  One gradient per work-group | this, us: 12 heads x 12288, causal, 1138 | 889;
// 12 x 4000 150 | 119; 40 x 1100 48.6 | 40.0; 64 x 400 22.6 | 20.5; no mask, 8 x 7000 595 | 397, 18 x 1531 76 | 53.
#include "wave_dma.h"

#include <type_traits>

namespace ssa {
namespace {

constexpr int KV_SLOTS = 4, KV_SLOT_B = 2 * W_TILE_B;   // Q and dO rows of a step
constexpr int KV_P = KV_SLOTS * KV_SLOT_B;              // two slots of P: a block of 32 x 32 fp32 for each of the four key blocks
constexpr int KV_STAT = KV_P + 2 * 4 * 4096;            // -LSE (base 2) [32] and Delta [32] of a step, a ring too
constexpr int KV_LDS = KV_STAT + KV_SLOTS * 256;

template <bool CAUSAL, bool DK>  // DK: the second wavefront of a key block
__device__ __forceinline__ void kv_fast128_wave(const KP& p, char* smem, int rank, int by, int bz_) {
  constexpr int D = 128, KS = D / 16, DB = D / 32, BK = 128;
  const int lane = threadIdx.x & 63, r = lane & 31, hl = lane >> 5;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), kblock = w & 3;
  const int h = p.h0 + by, b = p.b0 + bz_;
  const int k0 = rank * BK + 32 * kblock, key = k0 + r;
  const int kc = min(key, p.S - 1);
  const int64_t base = (int64_t)b * p.sb + (int64_t)h * p.sh;
  const uint16_t* Qb = (const uint16_t*)p.Q + base;
  const uint16_t* own = (const uint16_t*)(DK ? p.V : p.K) + base + (int64_t)kc * p.ss;
  const uint16_t* dOb = (const uint16_t*)p.dO + (int64_t)(b - p.do_b0) * p.do_sb + (int64_t)(h - p.do_h0) * p.do_sh;
  const float* stat = DK ? p.delta + (int64_t)(b - p.dl_b0) * p.dl_sb + (int64_t)(h - p.dl_h0) * p.dl_sh
                         : p.lse + (int64_t)(b - p.lse_b0) * p.lse_sb + (int64_t)(h - p.lse_h0) * p.lse_sh;
  const float c1 = p.scale * LOG2E;
  const int first = CAUSAL ? rank * (BK / 32) : 0;  // queries before the block's first key see none of it
  const int n = (p.S + 31) / 32 - first;            // steps

  // this wavefront's share of a step: rows 4w .. 4w + 3 of Q and of dO
  const uint32_t ss2 = (uint32_t)p.ss * 2u, dss2 = (uint32_t)p.do_ss * 2u;
  const uint32_t slice = (uint32_t)(((int64_t)(p.S - 1) * p.ss + D) * 2);  // < 2 GiB, checked on the host
  const uint32_t dslice = (uint32_t)(((int64_t)(p.S - 1) * p.do_ss + D) * 2);
  const int rho = 4 * w + (lane >> 4);
  const uint32_t c16 = 16u * (uint32_t)((lane & 15) ^ w_sw(rho));
  const uint32_t goff = (uint32_t)rho * ss2 + c16, goff_g = (uint32_t)rho * dss2 + c16;
  float pstat = 0.f;
  // step t into its slot (past the last step: empty descriptors, zeros arrive); the statistics travel through a register of one wavefront of
  // each kind, asked for before the sub-tiles so that waiting for them leaves those under way
  auto fetch = [&](char* slot, int t) {
    const int row0 = 32 * (first + t);
    const bool live = t < n;
    if (kblock == 0) pstat = stat[min(row0 + r, p.S - 1)];
    const uint32_t bq = live ? (uint32_t)row0 * ss2 : slice, bg = live ? (uint32_t)row0 * dss2 : dslice;
    const __amdgpu_buffer_rsrc_t rq = __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)Qb + bq), 0, (int)(slice - bq), 0x00020000);
    const __amdgpu_buffer_rsrc_t rg = __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)dOb + bg), 0, (int)(dslice - bg), 0x00020000);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rq, (w_lds_void*)(slot + w * 1024), 16, goff, 0, 0, 0);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rg, (w_lds_void*)(slot + W_TILE_B + w * 1024), 16, goff_g, 0, 0, 0);
  };
  const uint32_t lds0 = (uint32_t)(size_t)(w_lds_void*)smem;
  uint32_t ka[8], va[2][4];
  w_nat_addr(ka, smem, r, hl);
  w_tr_addr(va, smem, lane);
  const uint32_t pa_ = lds0 + KV_P + 4096u * kblock + 16u * lane;
  const uint32_t st_w = lds0 + KV_STAT + (DK ? 128u : 0u) + 4u * r, st_r = lds0 + KV_STAT + (DK ? 128u : 0u) + 16u * hl;
  auto put_stat = [&](auto slot) {
    const uint32_t to = st_w;
    const float x = DK ? pstat : -pstat * LOG2E;
    if (kblock == 0)
      asm volatile("ds_write_b32 %0, %1 offset:%2" ::"v"(to), "v"(x), "n"(256 * decltype(slot)::value) : "memory");
  };

  u32x4 kr[KS];  // of K, of V
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) kr[ks] = *(const u32x4*)(own + 16 * ks + 8 * hl);
  fetch(smem, 0);
  put_stat(std::integral_constant<int, 0>{});
  fetch(smem + KV_SLOT_B, 1);
  // (used here, so that the loop holds no wait for them)
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+v"(kr[ks]));
  f32x16 acc[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[db][v] = 0.f;

  // step t: S and dV, or dP and dK of the step before
  auto work = [&](auto slot, int t) {
    constexpr int SL = decltype(slot)::value, SO = SL * KV_SLOT_B, PO = 16384 * (SL & 1), TO = 256 * SL;
    const int i0 = 32 * (first + t);
    const uint32_t sr = st_r, pp = pa_;
    if (k0 >= p.S || (CAUSAL && i0 + 31 < k0)) return;  // no visible pair for this key block
    f32x16 x;
#pragma unroll
    for (int v = 0; v < 16; ++v) x[v] = 0.f;
    u32x4 l4[4], pr[4];
    {
      u32x4 fr[KS];
      w_nat_issue<SO + (DK ? W_TILE_B : 0)>(fr, ka);
      asm volatile("ds_read_b128 %0, %4 offset:%5\n\tds_read_b128 %1, %4 offset:%6\n\tds_read_b128 %2, %4 offset:%7\n\t"
                   "ds_read_b128 %3, %4 offset:%8"
                   : "=&v"(l4[0]), "=&v"(l4[1]), "=&v"(l4[2]), "=&v"(l4[3])
                   : "v"(sr), "n"(TO), "n"(TO + 32), "n"(TO + 64), "n"(TO + 96)
                   : "memory");
      if (DK)
        asm volatile("ds_read_b128 %0, %4 offset:%5\n\tds_read_b128 %1, %4 offset:%6\n\tds_read_b128 %2, %4 offset:%7\n\t"
                     "ds_read_b128 %3, %4 offset:%8"
                     : "=&v"(pr[0]), "=&v"(pr[1]), "=&v"(pr[2]), "=&v"(pr[3])
                     : "v"(pp), "n"(PO), "n"(PO + 1024), "n"(PO + 2048), "n"(PO + 3072)
                     : "memory");
      w_nat_wait(fr);
      asm volatile("" : "+v"(l4[0]), "+v"(l4[1]), "+v"(l4[2]), "+v"(l4[3]));
      if (DK) asm volatile("" : "+v"(pr[0]), "+v"(pr[1]), "+v"(pr[2]), "+v"(pr[3]));
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) x = mfma(w_frag(fr[ks]), w_frag(kr[ks]), x);
    }
    // the transposed fragments of the second product arrive under the arithmetic
    u32x2 tf[2][2 * DB];
    w_tr_issue<SO + (DK ? 0 : W_TILE_B)>(tf, va);
    bf16x8 of[2];  // P or dS as packed operands
    float y[16];
    if (DK) {
#pragma unroll
      for (int v = 0; v < 16; ++v) y[v] = __uint_as_float(pr[v >> 2][v & 3]) * (x[v] - __uint_as_float(l4[v >> 2][v & 3]));
    } else {
      if ((i0 + 32 > p.S) || (k0 + 32 > p.S) || (CAUSAL && i0 < k0 + 31)) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int qi = i0 + key_of(v, hl);
          const bool dead = qi >= p.S || key >= p.S || (CAUSAL && key > qi);
          x[v] = dead ? -INFINITY : x[v];
        }
      }
#pragma unroll
      for (int v = 0; v < 16; ++v) y[v] = fast_exp2(fmaf(x[v], c1, __uint_as_float(l4[v >> 2][v & 3])));
#pragma unroll
      for (int g = 0; g < 4; ++g) pr[g] = u32x4{__float_as_uint(y[4 * g]), __float_as_uint(y[4 * g + 1]), __float_as_uint(y[4 * g + 2]), __float_as_uint(y[4 * g + 3])};
      asm volatile("ds_write_b128 %4, %0 offset:%5\n\tds_write_b128 %4, %1 offset:%6\n\tds_write_b128 %4, %2 offset:%7\n\t"
                   "ds_write_b128 %4, %3 offset:%8"
                   : : "v"(pr[0]), "v"(pr[1]), "v"(pr[2]), "v"(pr[3]), "v"(pp), "n"(PO), "n"(PO + 1024), "n"(PO + 2048), "n"(PO + 3072)
                   : "memory");
    }
    of[0] = pack8(&y[0]);
    of[1] = pack8(&y[8]);
    w_tr_wait(tf);
#pragma unroll
    for (int hb = 0; hb < 2; ++hb)
#pragma unroll
      for (int db = 0; db < DB; ++db) acc[db] = mfma(w_frag2(tf[hb][2 * db], tf[hb][2 * db + 1]), of[hb], acc[db]);
  };
  // step t of the work-group: sub-tiles t have landed for everybody, P of step t - 1 is there, and slot t + 2 and P's slot t are free
  auto step = [&](auto slot, int t) {
    constexpr int SL = decltype(slot)::value;
    asm volatile("s_waitcnt vmcnt(2) lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    put_stat(std::integral_constant<int, (SL + 1) & 3>{});
    fetch(smem + ((SL + 2) & 3) * KV_SLOT_B, t + 2);
    if (DK) {
      if (t > 0) work(std::integral_constant<int, (SL + 3) & 3>{}, t - 1);
    } else {
      if (t < n) work(slot, t);
    }
  };
  for (int t = 0; t <= n; t += 4) {
    step(std::integral_constant<int, 0>{}, t);
    if (t + 1 <= n) step(std::integral_constant<int, 1>{}, t + 1);
    if (t + 2 <= n) step(std::integral_constant<int, 2>{}, t + 2);
    if (t + 3 <= n) step(std::integral_constant<int, 3>{}, t + 3);
  }
  W_VMCNT(0);  // nothing may still be on its way into LDS when the work-group ends
  if (key >= p.S) return;
  uint16_t* out = (uint16_t*)(DK ? p.dK : p.dV) + base + (int64_t)key * p.ss;
#pragma unroll
  for (int db = 0; db < DB; ++db) {
    uint2 o[4];
#pragma unroll
    for (int g = 0; g < 4; ++g)
      o[g] = pack4_bf16(acc[db][4 * g], acc[db][4 * g + 1], acc[db][4 * g + 2], acc[db][4 * g + 3], DK ? p.scale : 1.f);
    store_row32(out + 32 * db, o, hl, true);
  }
}

template <bool CAUSAL>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void kv_fast128_kernel(KP p) {
  __shared__ __attribute__((aligned(1024))) char smem[KV_LDS];
  const BlockId blk = CAUSAL ? causal_block_id(false) : xcd_block_id();
  if (__builtin_amdgcn_readfirstlane(threadIdx.x >> 8)) kv_fast128_wave<CAUSAL, true>(p, smem, blk.x, blk.y, blk.z);
  else kv_fast128_wave<CAUSAL, false>(p, smem, blk.x, blk.y, blk.z);
}

}  // namespace

hipError_t launch_fast_kv128(const KP& p, hipStream_t st) {
  const dim3 g((p.S + 127) / 128, p.h1 - p.h0, p.b1 - p.b0);
  if (p.mask_kind == 1) kv_fast128_kernel<true><<<g, 512, 0, st>>>(p);
  else kv_fast128_kernel<false><<<g, 512, 0, st>>>(p);
  return hipGetLastError();
}

}  // namespace ssa

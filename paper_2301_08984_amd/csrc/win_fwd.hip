// Forward of attention over windows of 17 to 160 tokens with head size 32, bf16: a whole row (b, h) is small
// enough to share one work-group (the backward is win_bwd.hip).
//
// A work-group takes a run of rows of one head, a wavefront 16 queries (NB = 2 to 10 wavefronts), lane = query.  K and V of a row travel straight into
// one of two LDS buffers, a row ahead; the scores with all keys are held in registers, so that the maximum is known before the first exponential, and
// the probabilities are the operand of the second product as they are.  One barrier a row.  The bias is fetched or gathered once per work-group.
//
// Before, a wavefront took 32 queries and walked the keys with a running maximum, K and V went through registers, and work-groups of more than 128 tokens took
// one row each.  Us, 8 heads, regions: 512 windows of 12 x 12 tokens 67.7 -> 55.0, without a bias 58.2 -> 43.1, 11 x 11 39.6 -> 33.7, 10 x 10 38.1 -> 29.5,
// 9 x 9 22.9 -> 21.7; 256 x 24 heads of 12 x 12 99 -> 77; 1024 x 16 of 9 x 9 (memory: 69) 87.5 -> 82.3.
// What bounds it: 12 x 12: some 450 vector instructions a wavefront and row, half of them arithmetic on the scores, and reading and writing 64-byte pieces at 3 TB/s.
#include "win_common.h"

namespace ssa {
namespace {

// work-groups on a compute unit, wavefronts on a SIMD that this takes; the bias in LDS where the registers of that many do not hold it
template <int NB> constexpr int WF_GROUPS = NB == 2 ? 12 : NB == 3 ? 8 : NB == 4 ? 6 : NB == 5 ? 4 : NB == 6 ? 4 : NB == 10 ? 1 : 2;
template <int NB> constexpr int WF_WAVES = (WF_GROUPS<NB> * NB + 3) / 4;
template <int NB> constexpr bool WF_LDS_BIAS = NB == 9;
// Region ids straight into LDS where a register for them is one too many (what is spilled is waited for when it is read back, and with it the row that was just
// asked for): 81 to 96 tokens with a bias and regions, us: 1024 x 16 heads of 9 x 9 90.5 -> 82.3, 4096 x 8 173 -> 160, 512 x 8 23.6 -> 21.7.  Elsewhere a load and a
// store more cost more than a register (1024 x 16 of 8 x 10 79.6 -> 83.3).
template <int NB, bool BIAS> constexpr bool WF_ID_DMA = NB == 6 || (NB == 9 && BIAS);
// The gate asked for ahead of the next row, where there are registers for it and the wait for that row was felt, us: 1024 x 16 heads, regions, 9 x 9 without a bias
// 111.9 -> 106.9, 10 x 10 with one 144.8 -> 137.9; 800 x 8 of 5 x 14 with regions and no bias 33.9 -> 31.6 (32.6 with the kernels before these), of 5 x 16 36.2 -> 34.0
// (34.2), of 9 x 9 with a bias and no regions 39.8 -> 38.1 (38.2), of 6 x 16 42.8 -> 40.2 (40.0).
template <int NB, bool REGION, bool BIAS> constexpr bool WF_EARLY_GATE = NB == 5 || NB == 7 || (NB == 6 && !(REGION && BIAS));

template <int NB, bool REGION, bool BIAS, bool LSE>
__global__ __launch_bounds__(64 * NB) __attribute__((amdgpu_waves_per_eu(WF_WAVES<NB>, WF_WAVES<NB>))) void win_fwd_kernel(KP p, int rows_per_wg) {
#pragma clang fp contract(off)
  constexpr int T = 16 * NB, STEPS = (NB + 1) / 2, TENSOR = T * WB_TOKEN;
  constexpr bool LB = BIAS && WF_LDS_BIAS<NB>, ID_DMA = REGION && WF_ID_DMA<NB, BIAS>, EARLY_GATE = WF_EARLY_GATE<NB, REGION, BIAS>;
  // arrays of their own: the compiler then knows that a load into one does not feed a read of the other
  __shared__ __attribute__((aligned(1024))) char kv0[2 * TENSOR];
  __shared__ __attribute__((aligned(1024))) char kv1[2 * TENSOR];
  __shared__ uint2 bias_lds[LB ? NB * NB * 64 : 1];
  __shared__ __attribute__((aligned(16))) int rids[2][REGION ? (ID_DMA ? (T + 63) / 64 * 64 : T) : 4];
  const int tid = threadIdx.x, lane = tid & 63, r = lane & 15, g = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const BlockId blk = xcd_block_id();  // heads of a row next to each other: they share cache lines
  const int h = p.h0 + blk.x;
  const int bfirst = p.b0 + blk.z * rows_per_wg, blast = min(bfirst + rows_per_wg, p.b1);

  // Queries past the end are the last one again, from the loads to the stores: the same values to the same place, and no store that some lanes skip.
  const int me = min(16 * w + r, p.S - 1);
  const int64_t mine = (int64_t)me * p.ss + (int64_t)h * p.sh;
  const int64_t piece = (int64_t)min(16 * w + (lane >> 2), p.S - 1) * p.ss + (int64_t)h * p.sh + 8 * ((lane & 3) ^ wb_place(lane >> 2));
  auto load_keys = [&](char* to, int b) {
    const int64_t at = (int64_t)b * p.sb + piece;
    asm volatile("" ::: "memory");  // stays where it is: the waits count what is younger
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_global_load_lds((wb_glb_void*)((const uint16_t*)p.K + at), (wb_lds_void*)(to + 1024 * w), 16, 0, 0);
    __builtin_amdgcn_global_load_lds((wb_glb_void*)((const uint16_t*)p.V + at), (wb_lds_void*)(to + TENSOR + 1024 * w), 16, 0, 0);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  int id = 0;
  bf16x8 qn;
  auto load_query = [&](int b) {
    qn = *(const bf16x8*)((const uint16_t*)p.Q + (int64_t)b * p.sb + mine + 8 * g);
  };
  auto load_ids = [&](int* to, int b) {
    if (!REGION) return;
    const int32_t* at = p.region + (int64_t)(b % p.mask_period) * p.S + min(tid, p.S - 1);
    if (!ID_DMA) id = *at;
    else if (64 * w < T) __builtin_amdgcn_global_load_lds((wb_glb_void*)at, (wb_lds_void*)(to + 64 * w), 4, 0, 0);
  };
  auto gate_at = [&](int b, int db) { return *(const uint2*)((const uint16_t*)p.G + (int64_t)b * p.sb + mine + 16 * db + 4 * g); };
  load_keys(kv0, bfirst);
  load_query(bfirst);
  load_ids(rids[0], bfirst);
  uint32_t bz[BIAS ? NB : 1][2];
  if constexpr (BIAS) win_bias<NB>(p, (const uint2*)p.bias_q, kv1, h, w, lane, bz);
  // Waited for here: else the waits, for every load, come in every row.
  __builtin_amdgcn_s_waitcnt(0xf70);  // vmcnt(0)
  asm volatile("" ::: "memory");
#pragma unroll
  for (int c = 0; c < (BIAS ? NB : 1); ++c) {
    if (BIAS) asm volatile("" : "+v"(bz[c][0]), "+v"(bz[c][1]));
    if (LB) bias_lds[(w * NB + c) * 64 + lane] = uint2{bz[c][0], bz[c][1]};  // the lane itself reads it
  }
  const float scale = in_vgpr(p.scale), c1 = in_vgpr(BIAS ? LOG2E : p.scale * LOG2E);  // score to logit, then to exponent of two
  uint32_t nat = wb_along(r, g), tr = wb_across(r, g);

  auto row = [&](int b, char* kv, char* kv_next, int* rid, int* rid_next) __attribute__((always_inline)) {
    asm volatile("" : "+v"(nat), "+v"(tr));  // sums with the buffers' places are not kept from row to row
    // This row is in LDS: the stores of O and of the statistics are younger than its last piece.  (As a builtin: a wait that the compiler does not know of
    // it repeats before the first read, on every load in flight by then.)
    __builtin_amdgcn_s_waitcnt(LSE ? 0xf72 : 0xf71);  // vmcnt(2), vmcnt(1)
    asm volatile("" ::: "memory");
    if (REGION && !ID_DMA && tid < T) rid[tid] = id;
    const bf16x8 qf = qn;
    wb_barrier();
    uint2 gate[2];
    if (EARLY_GATE && p.gated) gate[0] = gate_at(b, 0), gate[1] = gate_at(b, 1);
    if (b + 1 < blast) {
      load_keys(kv_next, b + 1);
      load_query(b + 1);
      load_ids(rid_next, b + 1);
    }
    constexpr int AHEAD = 2;  // blocks of keys whose operands are under way
    bf16x8 kf[AHEAD];
    uint2 bn[AHEAD];
    auto read_keys = [&](int c) __attribute__((always_inline)) {
      kf[c % AHEAD] = *(const bf16x8*)(kv + nat + 1024 * c);
      if (LB) bn[c % AHEAD] = bias_lds[(w * NB + c) * 64 + lane];
    };
#pragma unroll
    for (int c = 0; c < AHEAD; ++c) read_keys(c);
    f32x4 s[NB];
#pragma unroll
    for (int c = 0; c < NB; ++c) {
#pragma unroll
      for (int v = 0; v < 4; ++v) s[c][v] = BIAS || c < NB - 1 || 16 * c + 4 * g + v < p.S ? 0.f : -INFINITY;
      s[c] = mfma16(kf[c % AHEAD], qf, s[c]);
      if (BIAS) {  // logits
        uint32_t lo = bz[BIAS ? c : 0][0], hi = bz[BIAS ? c : 0][1];
        if (LB) {
          lo = bn[c % AHEAD].x;
          hi = bn[c % AHEAD].y;
        } else {
          asm volatile("" : "+v"(lo), "+v"(hi));  // stays packed from row to row
        }
        s[c][0] = fmaf(s[c][0], scale, __uint_as_float(lo << 16));
        s[c][1] = fmaf(s[c][1], scale, __uint_as_float(lo & 0xffff0000u));
        s[c][2] = fmaf(s[c][2], scale, __uint_as_float(hi << 16));
        s[c][3] = fmaf(s[c][3], scale, __uint_as_float(hi & 0xffff0000u));
      }
      if (c + AHEAD < NB) read_keys(c + AHEAD);
    }
    if (REGION && ids_differ<NB>(rid, lane)) {
      const int my_rid = rid[16 * w + r];
#pragma unroll
      for (int c = 0; c < NB; ++c) {
        const int4 k = *(const int4*)(rid + 16 * c + 4 * g);
        s[c][0] = k.x != my_rid ? -INFINITY : s[c][0];
        s[c][1] = k.y != my_rid ? -INFINITY : s[c][1];
        s[c][2] = k.z != my_rid ? -INFINITY : s[c][2];
        s[c][3] = k.w != my_rid ? -INFINITY : s[c][3];
      }
    }
    float top[4] = {-1e30f, -1e30f, -1e30f, -1e30f};
#pragma unroll
    for (int c = 0; c < NB; ++c)
#pragma unroll
      for (int v = 0; v < 4; ++v) top[v] = fmaxf(top[v], s[c][v]);
    const float nm = -groups_max(fmaxf(fmaxf(top[0], top[1]), fmaxf(top[2], top[3]))) * c1;
    float sum[4] = {0.f, 0.f, 0.f, 0.f};
    f32x4 o[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
    for (int t = 0; t < STEPS; ++t) {
      float e[8];
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          e[4 * u + v] = 2 * t + u < NB ? fast_exp2(fmaf(s[min(2 * t + u, NB - 1)][v], c1, nm)) : 0.f;
          if (2 * t + u < NB) sum[v] += e[4 * u + v];
        }
      const bf16x8 pf = pack8(e);
#pragma unroll
      for (int db = 0; db < 2; ++db) o[db] = mfma16(wb_read_across<NB>(kv + TENSOR, tr, t, db), pf, o[db]);
    }
    const float l = groups_sum((sum[0] + sum[1]) + (sum[2] + sum[3])), inv = 1.f / l;
    const int64_t at = (int64_t)b * p.sb + mine;
#pragma unroll
    for (int db = 0; db < 2; ++db) {
#pragma unroll
      for (int v = 0; v < 4; ++v) o[db][v] *= inv;
      if (p.gated) {
        const uint2 u = EARLY_GATE ? gate[db] : gate_at(b, db);
        const float z[4] = {__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xffff0000u), __uint_as_float(u.y << 16), __uint_as_float(u.y & 0xffff0000u)};
#pragma unroll
        for (int v = 0; v < 4; ++v) o[db][v] *= fast_rcp(1.f + fast_exp2(-z[v] * LOG2E));
      }
    }
    const uint2 y[2] = {pack4_bf16(o[0][0], o[0][1], o[0][2], o[0][3], 1.f), pack4_bf16(o[1][0], o[1][1], o[1][2], o[1][3], 1.f)};
    const u32x4 z = gather16(y);
    asm volatile("" ::: "memory");
    *(u32x4*)((uint16_t*)p.Y + at + 8 * store_chunk(g)) = z;
    if (LSE) {
      int x = lane;
      asm volatile("" : "+v"(x));  // (an address formed here, not kept from row to row)
      p.lse_out[(int64_t)(b - p.lse_b0) * p.lse_sb + (int64_t)(h - p.lse_h0) * p.lse_sh + min(16 * w + (x & 15), p.S - 1)] = (log2f(l) - nm) * LN2;
    }
    asm volatile("" ::: "memory");
  };
  for (int b = bfirst;; b += 2) {
    row(b, kv0, kv1, rids[0], rids[1]);
    if (b + 1 >= blast) break;
    row(b + 1, kv1, kv0, rids[1], rids[0]);
    if (b + 2 >= blast) break;
  }
}

template <int NB>
void launch_blocks(const KP& p, hipStream_t st) {
  // A run of rows for as many work-groups as the chip holds at a time, in several rounds where that would be a long one: the heads of a row, which share its
  // cache lines, drift apart.  Of up to 96 tokens rounds of at most 6 rows from 9 on (4096 x 16 heads of 7 x 7: 177 us, rounds of 4 the same, of 12 187).  Of up to
  // 112, of 16 rows and more (one round | so, regions: 1024 x 16 heads of 10 x 10 124 | 113, 1024 x 32 252 | 213; 1536 x 12, where rounds would be of 18, 122 | 121); of up to
  // 128, of 8 and more from 24 on (11 x 11: 768 x 16 114 | 96, 1024 x 16 157 | 127, 1024 x 32 322 | 239, 4096 x 8 285 | 243; 768 x 12, 18 rows, 68 | 70).  Of more tokens
  // one (256 x 24 of 12 x 12: 85 in rounds, 77 in one; 4096 x 8 349 | 328).
  // Of 65 to 96 without a bias, which a work-group would have to gather first, and six heads or more (of up to 80 eight): rounds of at most 4 rows (as above | so, with the kernels before
  // these; regions: 900 x 8 heads of 6 x 16 35.2 | 30.5, 31.5; 512 x 16 39.7 | 35.0, 35.7; gated 48.5 | 43.3, 41.8; 900 x 8 of 5 x 16 29.2 | 25.6, 30.4; 700 x 8 of 9 x 9
  // 25.0 | 24.7, 26.5; 1024 x 6 of 6 x 16 30.2 | 28.5, 27.7; of fewer heads 2048 x 6 of 5 x 13 37.4 | 38.4, 45.3, 2000 x 3 of 9 x 9 25.8 | 26.7, 28.2, 1600 x 4 of 6 x 16 30.0 | 28.5, 28.9).
  const int64_t rows = p.b1 - p.b0, heads = p.h1 - p.h0, slots = 256 * WF_GROUPS<NB>;
  const int64_t once = (rows * heads + slots - 1) / slots;
  const int64_t rounds = NB > 8 ? 1 : NB == 8 ? (once < 24 ? 1 : once / 8) : NB == 7 ? (once < 16 ? 1 : once / 16) :
                         NB > 4 && p.bias_kind == 0 && heads >= (NB == 5 ? 8 : 6) ? (once + 3) / 4 : once <= 8 ? 1 : (once + 5) / 6;
  const int64_t of_head = slots * rounds / heads > 1 ? slots * rounds / heads : 1;
  const int run = (int)((rows + of_head - 1) / of_head);
  const dim3 grid((unsigned)heads, 1, (unsigned)((rows + run - 1) / run));
  auto go = [&](auto region, auto bias, auto lse) { win_fwd_kernel<NB, region(), bias(), lse()><<<grid, 64 * NB, 0, st>>>(p, run); };
  auto with_bias = [&](auto region, auto bias) {
    if (p.lse_out) go(region, bias, std::true_type{});
    else go(region, bias, std::false_type{});
  };
  auto with_mask = [&](auto region) {
    if (p.bias_kind) with_bias(region, std::true_type{});
    else with_bias(region, std::false_type{});
  };
  if (p.mask_kind == 2) with_mask(std::true_type{});
  else with_mask(std::false_type{});
}

}  // namespace

hipError_t launch_win_fwd(const KP& p, hipStream_t st) {
  switch ((p.S + 15) / 16) {
    case 2: launch_blocks<2>(p, st); break;
    case 3: launch_blocks<3>(p, st); break;
    case 4: launch_blocks<4>(p, st); break;
    case 5: launch_blocks<5>(p, st); break;
    case 6: launch_blocks<6>(p, st); break;
    case 7: launch_blocks<7>(p, st); break;
    case 8: launch_blocks<8>(p, st); break;
    case 9: launch_blocks<9>(p, st); break;
    case 10: launch_blocks<10>(p, st); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace ssa

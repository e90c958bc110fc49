// Backward of windows of 17 to 160 tokens with head size 32, bf16, in one kernel: dQ, dK, dV, dG and the bias gradient.
//
// A work-group takes one head and one group of p.sm_gw consecutive global rows (or the chunk's part of it), a wavefront 16 tokens
// (NB = 2 to 10 wavefronts).  For a row, a wavefront holds the scores and dP of its 16 queries with all keys in registers (lane = query), so
// that the softmax needs no second look at them: maximum, sum and Delta, then P and dS, dQ, and the sum of dS over the rows, which stays in
// registers and is stored as the group's partial sum, resumed when a chunk boundary cuts the group.  P and dS are handed over through LDS,
// rounded to bf16, to the wavefronts of the keys (lane = key), which sum dV and dK.  The row's Q, dO, K and V travel straight into
// LDS, a row ahead.
//
// Before, recompute + dQ and dK / dV + bias gradient were two kernels of 32-token blocks, which read the tensors twice, formed the scores and their
// exponentials twice and left one work-group of five wavefronts on a compute unit.  Backward, us, 8 heads: 512 windows of 12 x 12 tokens with regions 227 -> 137
// (this kernel 116 of it, 92 + 130 before), 64 windows 61 -> 43; 512 of 9 x 9 98 -> 78, of 11 x 11 137 -> 95, of 10 x 10 116 -> 86; 1024 x 16 heads of
// 9 x 9 354 -> 235; without a bias 512 of 12 x 12 196 -> 101.  Errors of dQ and of the table's gradient against 64 bits 2.32 -> 2.28e-3, 3.4 -> 1.4e-7.
//
// What bounds it (12 x 12): nine wavefronts on four SIMDs, of which one runs three: its vector arithmetic, some 20 instructions a score
// with what goes round it, takes 60 % of the time; sums of S x S and a row's S and dP (108 registers) leave no room for a second work-group.  LDS 25 %.
// 4096 x 16 heads of 7 x 7 (memory: 248): 387 with a work-group for every 8 rows, 462 with as many as the chip holds and several groups each, whose heads drift
// apart and no longer share cache lines; two buffers of K and V, three work-groups a compute unit instead of four, 406.
// Timed on the way there: waits for loads that the compiler inserted (see `store`) 280 -> 228 (1024 x 16 x 9 x 9), nine spilled registers 147 -> 137.
#include "win_common.h"

namespace ssa {
namespace {

// LDS of a work-group.  Two buffers of a row's tensors, but one of K and V where that makes room for a second work-group on the compute unit; P and
// dS next to each other, or one after the other in one place (and two barriers more a row).  KiB from NB = 2 on: 14, 23, 33, 65, 74, 69, 129, 155, 132.
template <int NB> constexpr bool TWO_KV = NB > 4 && NB != 6 && NB != 7;
template <int NB> constexpr bool ONE_PLACE = NB <= 4 || NB == 7 || NB == 9 || NB == 10;
// wavefronts on a SIMD that LDS then allows
template <int NB> constexpr int WB_WAVES = NB <= 4 ? 4 : NB == 8 ? 2 : 3;
// the bias in LDS where the registers do not hold it (of ten wavefronts LDS does not, either)
template <int NB> constexpr bool LDS_BIAS = NB == 9;
// What is spilled is waited for when it is read back, and with it the row that was just asked for.  Left to itself the compiler adds dS to the sums over
// rows, and packs P and dS, at the row's end: it keeps all of them in fp32 until then.  Where the registers do not hold that: each block of keys is finished
// before the next, and O is formed as soon as the exponentials are there (elsewhere that costs 2 %).  Gated windows with regions and a bias, 512 x 8, us:
// 9 x 9 101 -> 82.5, 10 x 10 120 -> 110, 12 x 12 232 -> 157 (without regions 201 -> 147); with the kernels before these 113, 154, 316 (280).
template <int NB, bool REGION, bool BIAS, bool GATED> constexpr bool AT_ONCE = BIAS && (NB == 10 || (GATED && (NB == 9 || (REGION && (NB == 6 || NB == 7)))));
// Ten wavefronts with a bias: dP of a block is formed again where it is used, from the same operands, instead of kept from the mean on (40 registers).  512 x 8 of
// 10 x 16 with regions 227 -> 139, gated 589 -> 329 (424 with the kernels before these), 300 x 8 x 160 with a dense bias 135 -> 85.
template <int NB, bool BIAS> constexpr bool DP_AGAIN = BIAS && NB == 10;

template <int NB, bool REGION, bool BIAS, bool GATED>
__global__ __launch_bounds__(64 * NB) __attribute__((amdgpu_waves_per_eu(WB_WAVES<NB> - (GATED && (NB == 3 || NB == 4)), WB_WAVES<NB> - (GATED && (NB == 3 || NB == 4))))) void win_bwd_kernel(KP p) {
#pragma clang fp contract(off)
  constexpr int T = 16 * NB, STEPS = (NB + 1) / 2, TENSOR = T * WB_TOKEN, BLOCK = T * 32;
  constexpr bool KV2 = TWO_KV<NB>, ONE = ONE_PLACE<NB>, LB = BIAS && LDS_BIAS<NB>, TIGHT = NB == 7 || NB > 8;
  constexpr bool NOW = AT_ONCE<NB, REGION, BIAS, GATED>, AGAIN = DP_AGAIN<NB, BIAS>, ID_DMA = REGION && GATED && AGAIN;  // (region ids: straight into LDS)
  // arrays of their own: the compiler then knows that a load into one does not feed a read of another
  __shared__ __attribute__((aligned(1024))) char qg0[2 * TENSOR];
  __shared__ __attribute__((aligned(1024))) char qg1[2 * TENSOR];
  __shared__ __attribute__((aligned(1024))) char kv0[2 * TENSOR];
  __shared__ __attribute__((aligned(1024))) char kv1[KV2 ? 2 * TENSOR : 16];
  __shared__ __attribute__((aligned(1024))) char hand[(ONE ? 1 : 2) * NB * BLOCK];  // P, dS: per block of 16 keys a row of 32 bytes per query
  __shared__ uint2 bias_lds[LB ? NB * NB * 64 : 1];
  __shared__ __attribute__((aligned(16))) int rids[2][REGION ? (ID_DMA ? (T + 63) / 64 * 64 : T) : 4];
  const int tid = threadIdx.x, lane = tid & 63, r = lane & 15, g = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const BlockId blk = xcd_block_id();  // heads of a row next to each other: they share cache lines
  const int h = p.h0 + blk.x, me = 16 * w + r, mc = min(me, p.S - 1);
  const int group = p.b0 / p.sm_gw + blk.y;  // global
  const int bfirst = max(group * p.sm_gw, p.b0), blast = min((group + 1) * p.sm_gw, p.b1);

  // this lane's piece of a row: token 16 w + lane / 4 (past S - 1: the last one again), the chunk that belongs at position lane % 4
  // (lane addresses are formed anew in every row where the registers hold no more than they must)
  auto anew = [&] {
    int x = lane;
    if (TIGHT) asm volatile("" : "+v"(x));
    return x;
  };
  auto piece_at = [&] {
    const int l = anew();
    return (int64_t)min(16 * w + (l >> 2), p.S - 1) * p.ss + 8 * ((l & 3) ^ wb_place(l >> 2));
  };
  auto row_at = [&](int b) { return (int64_t)b * p.sb + (int64_t)h * p.sh; };
  auto load_pair = [&](char* to, const void* x, const void* y, int b) {
    const int64_t at = row_at(b) + piece_at();
    asm volatile("" ::: "memory");  // stays where it is: the waits count what is younger
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_global_load_lds((wb_glb_void*)((const uint16_t*)x + at), (wb_lds_void*)(to + 1024 * w), 16, 0, 0);
    __builtin_amdgcn_global_load_lds((wb_glb_void*)((const uint16_t*)y + at), (wb_lds_void*)(to + TENSOR + 1024 * w), 16, 0, 0);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  int id = 0;
  auto load_id = [&](int* to, int b) {
    if (!REGION) return;
    const int32_t* at = p.region + (int64_t)(b % p.mask_period) * p.S + min(64 * w + anew(), p.S - 1);
    if (!ID_DMA) id = *at;
    else if (64 * w < T) __builtin_amdgcn_global_load_lds((wb_glb_void*)at, (wb_lds_void*)(to + 64 * w), 4, 0, 0);
  };
  u32x4 gate = {0, 0, 0, 0};  // of the lane's piece of dY
  auto load_gate = [&](int b) {
    if (GATED) gate = *(const u32x4*)((const uint16_t*)p.G + row_at(b) + piece_at());
  };
  load_pair(kv0, p.K, p.V, bfirst);
  load_pair(qg0, p.Q, p.dY, bfirst);
  load_id(rids[0], bfirst);
  load_gate(bfirst);

  uint32_t bz[BIAS ? NB : 1][2];
  if constexpr (BIAS) win_bias<NB>(p, (const uint2*)p.bias_k, qg1, h, w, lane, bz);
  f32x4 acc[BIAS ? NB : 1];
#pragma unroll
  for (int c = 0; c < (BIAS ? NB : 1); ++c) acc[c] = f32x4{0.f, 0.f, 0.f, 0.f};
  float* part = nullptr;
  if (BIAS && p.sm_partial) {
    part = p.sm_partial + ((int64_t)((group - p.sm_g0) % p.sm_ring) * p.sm_hs + (h - p.sm_h0)) * p.S * p.S;
    const bool resume = max(group * p.sm_gw, p.share_b0) < p.b0;  // an earlier chunk started this group
    if (resume)
#pragma unroll
      for (int c = 0; c < NB; ++c)
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[BIAS ? c : 0][v] = part[mc * p.S + min(16 * c + 4 * g + v, p.S - 1)];
  }
  // Waited for here, as the first row's loads are: else the waits, for every load, come in every row.
  __builtin_amdgcn_s_waitcnt(0xf70);  // vmcnt(0)
  asm volatile("" ::: "memory");
#pragma unroll
  for (int c = 0; c < (BIAS ? NB : 1); ++c) {
    asm volatile("" : "+v"(acc[c]));
    if (BIAS) asm volatile("" : "+v"(bz[c][0]), "+v"(bz[c][1]));
    if (LB) bias_lds[(w * NB + c) * 64 + lane] = uint2{bz[c][0], bz[c][1]};  // the lane itself reads it
  }
  const float scale = in_vgpr(p.scale), c1 = in_vgpr(BIAS ? LOG2E : p.scale * LOG2E);  // score to logit, then to exponent of two
  uint32_t nat = wb_along(r, g), tr = wb_across(r, g);
  // in a block of P or dS, keys 4 j on of query i are at position j ^ (i / 4) of its row of 32 bytes (as above): as this lane writes them, as it reads
  uint32_t give = (uint32_t)(32 * r + 8 * (g ^ (r >> 2))), take = (uint32_t)(w * BLOCK + 32 * (4 * g + (r >> 2)) + 8 * ((r & 3) ^ g));
  auto read_tr = [&](const char* tensor, int t, int db) { return wb_read_across<NB>(tensor, tr, t, db); };
  // keys 16 w .. of the same queries of P or dS
  auto read_hand = [&](const char* from, int t) { return wb_tr_pair(from + take + 1024 * t, 512, 2 * t + 1 < NB); };

  auto row = [&](int b, char* qg, char* kv, char* qg_next, char* kv_next, int* rid, int* rid_next) __attribute__((always_inline)) {
    if (TIGHT) asm volatile("" : "+v"(nat), "+v"(tr), "+v"(give), "+v"(take));  // sums with the buffers' places are not kept from row to row
    // This row is in LDS: three stores (dQ, dK, dV) are younger than its last piece, or two where K and V come after dQ.
    // (As a builtin: a wait that the compiler does not know of it repeats before the first read, on every load in flight by then.)
    __builtin_amdgcn_s_waitcnt(KV2 ? 0xf73 : 0xf72);  // vmcnt(3), vmcnt(2)
    asm volatile("" ::: "memory");
    if (REGION && !ID_DMA && tid < T) rid[tid] = id;
    if (GATED) {  // dO = dY * gate, of the lane's own piece
      u32x4* at = (u32x4*)(qg + TENSOR + 1024 * w + 16 * lane);
      u32x4 o = *at;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float g0 = __uint_as_float(gate[e] << 16), g1 = __uint_as_float(gate[e] & 0xffff0000u);
        o[e] = pack2_bf16(__uint_as_float(o[e] << 16) * fast_rcp(1.f + fast_exp2(-g0 * LOG2E)),
                          __uint_as_float(o[e] & 0xffff0000u) * fast_rcp(1.f + fast_exp2(-g1 * LOG2E)));
      }
      *at = o;
    }
    wb_barrier();
    const bool more = b + 1 < blast;
    if (more) {
      if (KV2) load_pair(kv_next, p.K, p.V, b + 1);
      load_pair(qg_next, p.Q, p.dY, b + 1);
      load_id(rid_next, b + 1);
      load_gate(b + 1);
    }
    uint2 pw[NB], dw[NB], ew[GATED && !NOW ? NB : 1];  // P, dS and, for O, P before it is divided by the sum, of this lane's query, packed
    auto pack = [](const f32x4& x) { return uint2{pack2_bf16(x[0], x[1]), pack2_bf16(x[2], x[3])}; };
    auto operand = [](uint2 lo, uint2 hi) {
      union { u32x4 u; bf16x8 v; } o;
      o.u = u32x4{lo.x, lo.y, hi.x, hi.y};
      return o.v;
    };
    auto ones = [] {
      union { u32x4 u; bf16x8 v; } o;
      o.u = u32x4{0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u};
      return o.v;
    };
    // O from the probabilities before they are divided by their sum (error of dG 2.21e-3 if after: the largest are exact), and the sum of those, rounded as they are
    f32x4 o[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}}, esum = o[0];
    auto add_to_o = [&](int t, uint2 lo, uint2 hi) __attribute__((always_inline)) {
      const bf16x8 ef = operand(lo, hi);
      esum = mfma16(ones(), ef, esum);
#pragma unroll
      for (int db = 0; db < 2; ++db) o[db] = mfma16(read_tr(kv + TENSOR, t, db), ef, o[db]);
    };
    {
      const bf16x8 qf = *(const bf16x8*)(qg + nat + 1024 * w), gf = *(const bf16x8*)(qg + TENSOR + nat + 1024 * w);
      f32x4 s[NB], dp[NB];
      constexpr int AHEAD = 2;  // blocks of keys whose operands are under way
      bf16x8 kf[AHEAD], vf[AHEAD];
      uint2 bn[AHEAD];
      auto read_keys = [&](int c) __attribute__((always_inline)) {
        kf[c % AHEAD] = *(const bf16x8*)(kv + nat + 1024 * c);
        if (!AGAIN) vf[c % AHEAD] = *(const bf16x8*)(kv + TENSOR + nat + 1024 * c);
        if (LB) bn[c % AHEAD] = bias_lds[(w * NB + c) * 64 + lane];
      };
#pragma unroll
      for (int c = 0; c < AHEAD; ++c) read_keys(c);
#pragma unroll
      for (int c = 0; c < NB; ++c) {
#pragma unroll
        for (int v = 0; v < 4; ++v) s[c][v] = BIAS || c < NB - 1 || 16 * c + 4 * g + v < p.S ? 0.f : -INFINITY;
        s[c] = mfma16(kf[c % AHEAD], qf, s[c]);
        if (!AGAIN) dp[c] = mfma16(vf[c % AHEAD], gf, f32x4{0.f, 0.f, 0.f, 0.f});
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
      const bool masked = REGION && ids_differ<NB>(rid, AGAIN ? anew() : lane);
      const int my_rid = masked ? rid[me] : 0;
      if (masked) {
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
      float sum[4] = {0.f, 0.f, 0.f, 0.f}, mean[4] = {0.f, 0.f, 0.f, 0.f};
      uint32_t vat = nat;
      auto read_values = [&](int c) __attribute__((always_inline)) { vf[c % AHEAD] = *(const bf16x8*)(kv + TENSOR + vat + 1024 * c); };
      auto values_anew = [&] {
        asm volatile("" : "+v"(vat));
#pragma unroll
        for (int c = 0; c < AHEAD; ++c) read_values(c);
      };
      if (AGAIN) values_anew();  // (opaque: not the same reads as before)
#pragma unroll
      for (int c = 0; c < NB; ++c) {
        const f32x4 d = AGAIN ? mfma16(vf[c % AHEAD], gf, f32x4{0.f, 0.f, 0.f, 0.f}) : dp[c];
        if (AGAIN && c + AHEAD < NB) read_values(c + AHEAD);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          s[c][v] = fast_exp2(fmaf(s[c][v], c1, nm));
          sum[v] += s[c][v];
          mean[v] = fmaf(s[c][v], d[v], mean[v]);
        }
        if (AGAIN) asm volatile("" : "+v"(mean[0]), "+v"(mean[1]), "+v"(mean[2]), "+v"(mean[3]), "+v"(sum[0]), "+v"(sum[1]), "+v"(sum[2]), "+v"(sum[3]));
      }
      if (GATED && NOW) {
#pragma unroll
        for (int t = 0; t < STEPS; ++t) {
          const uint2 e[2] = {pack(s[2 * t]), 2 * t + 1 < NB ? pack(s[min(2 * t + 1, NB - 1)]) : uint2{0, 0}};
          add_to_o(t, e[0], e[1]);
          if (AGAIN) __builtin_amdgcn_sched_barrier(0);
        }
      }
      if (AGAIN) values_anew();
      // queries past the end (the last one again) contribute nothing
      const float inv = me < p.S ? 1.f / groups_sum((sum[0] + sum[1]) + (sum[2] + sum[3])) : 0.f;
      const float delta = groups_sum((mean[0] + mean[1]) + (mean[2] + mean[3])) * inv;
      // masked pairs contribute nothing also where a query has infinite or NaN statistics
      const int unsound = REGION ? __builtin_amdgcn_readfirstlane(masked && __builtin_amdgcn_ballot_w64(!(fmaf(inv, 0.f, delta * 0.f) == 0.f)) != 0) : 0;
#pragma unroll
      for (int c = 0; c < NB; ++c) {
        float pr[4], ds[4];
        if (GATED && !NOW) ew[GATED && !NOW ? c : 0] = pack(s[c]);
        const f32x4 d = AGAIN ? mfma16(vf[c % AHEAD], gf, f32x4{0.f, 0.f, 0.f, 0.f}) : dp[c];
        if (AGAIN && c + AHEAD < NB) read_values(c + AHEAD);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          pr[v] = s[c][v] * inv;
          ds[v] = pr[v] * (d[v] - delta);
        }
        if (REGION) {
          int cut = unsound;  // opaque: one version of the loop
          asm volatile("" : "+s"(cut));
          if (cut) {
            const int4 k = *(const int4*)(rid + 16 * c + 4 * g);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
              const bool dead = (v == 0 ? k.x : v == 1 ? k.y : v == 2 ? k.z : k.w) != my_rid;
              pr[v] = dead ? 0.f : pr[v];
              ds[v] = dead ? 0.f : ds[v];
            }
          }
        }
        if (BIAS) {
#pragma unroll
          for (int v = 0; v < 4; ++v) acc[BIAS ? c : 0][v] += ds[v];
          if (NOW) asm volatile("" : "+v"(acc[BIAS ? c : 0]));
        }
        pw[c] = uint2{pack2_bf16(pr[0], pr[1]), pack2_bf16(pr[2], pr[3])};
        dw[c] = uint2{pack2_bf16(ds[0], ds[1]), pack2_bf16(ds[2], ds[3])};
        if (NOW) asm volatile("" : "+v"(pw[c].x), "+v"(pw[c].y), "+v"(dw[c].x), "+v"(dw[c].y));
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    auto put = [&](char* to, const uint2 (&x)[NB]) {
#pragma unroll
      for (int c = 0; c < NB; ++c) *(uint2*)(to + c * BLOCK + 512 * w + give) = x[c];
    };
    auto both = [](const auto& x, int t) {
      union { u32x4 u; bf16x8 v; } o;
      const uint2 hi = 2 * t + 1 < NB ? x[min(2 * t + 1, NB - 1)] : uint2{0, 0};
      o.u = u32x4{x[2 * t].x, x[2 * t].y, hi.x, hi.y};
      return o.v;
    };
    put(hand, pw);
    if (!ONE) put(hand + NB * BLOCK, dw);
    // dQ: a row of dS sums to zero, rounded to bf16 it does not, and keys with something in common would show the difference: it is
    // taken off along the mean key of the rounded probabilities.
    f32x4 a[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}}, k1[2] = {a[0], a[1]};
    f32x4 psum = a[0], dsum = a[0];
#pragma unroll
    for (int t = 0; t < STEPS; ++t) {
      const bf16x8 pf = both(pw, t), df = both(dw, t);
      psum = mfma16(ones(), pf, psum);
      dsum = mfma16(ones(), df, dsum);
#pragma unroll
      for (int db = 0; db < 2; ++db) {
        const bf16x8 kt = read_tr(kv, t, db);
        a[db] = mfma16(kt, df, a[db]);
        k1[db] = mfma16(kt, pf, k1[db]);
      }
    }
    const float excess = -dsum[0] / psum[0];
#pragma unroll
    for (int db = 0; db < 2; ++db)
#pragma unroll
      for (int v = 0; v < 4; ++v) a[db][v] = fmaf(excess, k1[db][v], a[db][v]);
    auto store = [&](void* to, const f32x4 (&x)[2], float factor) {
      const uint2 y[2] = {pack4_bf16(x[0][0], x[0][1], x[0][2], x[0][3], factor), pack4_bf16(x[1][0], x[1][1], x[1][2], x[1][3], factor)};
      const u32x4 z = gather16(y);
      const int l = anew(), token = 16 * w + (l & 15);
      uint16_t* at = (uint16_t*)to + row_at(b) + (int64_t)token * p.ss + 8 * store_chunk(l >> 4);
      // Tokens past the end go to scratch that nobody reads: around a store that some lanes skip there is a branch, and the compiler then counts on
      // it not having been issued, here and in its waits for the loads before it.
      *(u32x4*)(token < p.S ? at : (uint16_t*)p.delta) = z;
    };
    if (GATED) {
      if (!NOW) {
#pragma unroll
        for (int t = 0; t < STEPS; ++t) add_to_o(t, ew[2 * t], 2 * t + 1 < NB ? ew[min(2 * t + 1, NB - 1)] : uint2{0, 0});
      }
      const float inv = 1.f / esum[0];  // dG = dY O g (1 - g)
#pragma unroll
      for (int db = 0; db < 2; ++db) {
        const int64_t at = row_at(b) + (int64_t)min(16 * w + (anew() & 15), p.S - 1) * p.ss + 16 * db + 4 * (NOW && REGION ? anew() >> 4 : g);
        const uint2 ux = *(const uint2*)((const uint16_t*)p.dY + at), ug = *(const uint2*)((const uint16_t*)p.G + at);
        const float y[4] = {__uint_as_float(ux.x << 16), __uint_as_float(ux.x & 0xffff0000u), __uint_as_float(ux.y << 16), __uint_as_float(ux.y & 0xffff0000u)};
        const float z[4] = {__uint_as_float(ug.x << 16), __uint_as_float(ug.x & 0xffff0000u), __uint_as_float(ug.y << 16), __uint_as_float(ug.y & 0xffff0000u)};
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const float gt = fast_rcp(1.f + fast_exp2(-z[v] * LOG2E));
          o[db][v] = y[v] * (o[db][v] * inv) * gt * (1.f - gt);
        }
      }
      store(p.dG, o, 1.f);
      asm volatile("" ::: "memory");  // older than the three stores that the next row's wait leaves in flight
    }
    store(p.dQ, a, p.scale);
    wb_barrier();
    if (!KV2 && more) load_pair(kv, p.K, p.V, b + 1);
#pragma unroll
    for (int db = 0; db < 2; ++db) a[db] = f32x4{0.f, 0.f, 0.f, 0.f};
    f32x4 dv[2] = {a[0], a[1]};
#pragma unroll
    for (int t = 0; t < STEPS; ++t) {
      const bf16x8 x = read_hand(hand, t);
#pragma unroll
      for (int db = 0; db < 2; ++db) dv[db] = mfma16(read_tr(qg + TENSOR, t, db), x, dv[db]);
    }
    store(p.dV, dv, 1.f);
    if (ONE) {
      wb_barrier();
      put(hand, dw);
      wb_barrier();
    }
#pragma unroll
    for (int t = 0; t < STEPS; ++t) {
      const bf16x8 x = read_hand(ONE ? hand : hand + NB * BLOCK, t);
#pragma unroll
      for (int db = 0; db < 2; ++db) a[db] = mfma16(read_tr(qg, t, db), x, a[db]);
    }
    store(p.dK, a, p.scale);
  };
  for (int b = bfirst;; b += 2) {
    row(b, qg0, kv0, qg1, KV2 ? kv1 : kv0, rids[0], rids[1]);
    if (b + 1 >= blast) break;
    row(b + 1, qg1, KV2 ? kv1 : kv0, qg0, kv0, rids[1], rids[0]);
    if (b + 2 >= blast) break;
  }
  int l = lane;  // opaque: the addresses are not to be kept in registers from the load of the partial sum on
  asm volatile("" : "+v"(l));
  if (BIAS && part && 16 * w + (l & 15) < p.S) {
    const int at = (16 * w + (l & 15)) * p.S + 4 * (l >> 4);
#pragma unroll
    for (int c = 0; c < NB; ++c)
#pragma unroll
      for (int v = 0; v < 4; ++v)
        if (c < NB - 1 || 16 * c + 4 * (l >> 4) + v < p.S) part[at + 16 * c + v] = acc[BIAS ? c : 0][v];
  }
}

template <int NB>
void launch_blocks(const KP& args, hipStream_t st) {
  KP p = args;
  if (!p.sm_partial) {  // nothing summed over rows: as few in a work-group as let the launch fit the chip in one round, at most 8 (64 rows x 4 heads x 128: 36 us with 8, 9.9 so)
    const int64_t slots = 256 * (4 * WB_WAVES<NB> / NB), once = ((int64_t)(p.b1 - p.b0) * (p.h1 - p.h0) + slots - 1) / slots;
    p.sm_gw = once < 8 ? (int)once : 8;
  }
  const dim3 grid(p.h1 - p.h0, (p.b1 - 1) / p.sm_gw - p.b0 / p.sm_gw + 1);
  auto go = [&](auto region, auto bias, auto gated) { win_bwd_kernel<NB, region(), bias(), gated()><<<grid, 64 * NB, 0, st>>>(p); };
  auto with_bias = [&](auto region, auto bias) {
    if (p.gated) go(region, bias, std::true_type{});
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

hipError_t launch_win_bwd(const KP& args, hipStream_t st) {
  KP p = args;
  if (p.dbias_acc && !p.sm_partial) {  // no partial sums: all rows are one group, which sums in the result itself
    p.sm_partial = p.dbias_acc;
    p.sm_gw = p.B;
    p.sm_g0 = 0; p.sm_ring = 1; p.sm_hs = p.H; p.sm_h0 = 0;
  }
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

// Attention over windows of 65 to 160 tokens with head size 32, bf16: a whole row (b, h) is small
// enough to share one work-group, too large for one wavefront (small_kernels.hip ends at 64 tokens).
//
// A work-group has one wavefront per 32-token block (NB = 3, 4 or 5) and walks several rows b of one
// head.  Each wavefront keeps the bias of its 32 queries (or keys) against every token in registers,
// packed bf16, 8 per 32 x 32 block, gathered once per work-group (from the relative-position table or
// the dense matrix; -inf where a pair lies outside the window), so that a row costs no bias traffic and
// no index arithmetic.  K and V (or Q and dO) of the row are staged in LDS once for all
// wavefronts, the next row's travel global -> registers meanwhile.
//
// What bounds it: the vector arithmetic per score element (bias unpack and addition, exp2 at a quarter of
// the rate, maximum, sums, conversions) against two to five matrix steps.  The all-feature kernels that
// served these shapes spent most of their time on a table lookup, an integer subtraction and a mask
// comparison per element and gave the bias gradient a wavefront per 32 x 32 tile that read the operands
// in 16-byte pieces.  512 windows of 12 x 12 tokens, 8 heads: 3.57 ms per step with them, 0.52 with these (one
// chunk: forward 99 us, recompute + dQ 252, dK / dV and the bias gradient 151, folds and table 19).
#include "mfma_common.h"

namespace ssa {
namespace {

constexpr int WD = 32;        // head size
constexpr int WLD = WD + 24;  // LDS row stride of the staged tiles (elements): conflict-free for b128 and transposed reads
constexpr uint32_t NEG_INF_BF16 = 0xff80u;

typedef uint2 uint2_u __attribute__((aligned(2)));

// The blocks of a row are unrolled (the bias and the gradient sums are registers) but meant to run one
// after the other, other wavefronts fill the gaps; and the bias, which does not change from row to
// row, is meant to stay packed: the compiler would unpack it once, outside the row loop, into twice the
// registers (measured: 200 spilled in the dK/dV kernel at NB = 5).
__device__ inline void block_boundary(uint32_t (&bz)[8]) {
#pragma unroll
  for (int i = 0; i < 8; ++i) asm volatile("" : "+v"(bz[i]));
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// Registers of a 32-row strip of the score matrix against NB column blocks: element v of block c is the
// pair (row, 32 c + key_of(v, hl)).  ROW_IS_QUERY: lane = query, registers = keys; else transposed.
// -inf outside the window on the register axis, and everywhere for a row with `row_dead`; other rows past
// the end repeat the last one (their results are never stored).  Table and cidx in LDS.
template <int NB, bool ROW_IS_QUERY>
__device__ inline void gather_bias(const KP& p, const uint16_t* table, const int* cidx, int h, int row, int hl, bool row_dead,
                                   uint32_t (&bz)[NB][8]) {
  const int rc = min(row, p.S - 1);
  auto fill = [&](auto raw) {  // raw(k): bf16 bits of the pair of this row with register index k < S
#pragma unroll
    for (int c = 0; c < NB; ++c) {
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int k = 32 * c + 8 * (j >> 1) + 4 * hl + 2 * (j & 1);
        const uint32_t x = raw(min(k, p.S - 1)), y = raw(min(k + 1, p.S - 1));
        bz[c][j] = (row_dead || k >= p.S ? NEG_INF_BF16 : x) | ((row_dead || k + 1 >= p.S ? NEG_INF_BF16 : y) << 16);
      }
      block_boundary(bz[c]);
    }
  };
  if (p.bias_kind == 2) {
    const int c0 = (p.win_h - 1) * (2 * p.win_w - 1) + (p.win_w - 1), cr = cidx[rc] + (ROW_IS_QUERY ? c0 : -c0);
    fill([&](int k) -> uint32_t { return table[ROW_IS_QUERY ? cr - cidx[k] : cidx[k] - cr]; });
  } else if (p.bias_kind == 1) {
    const uint16_t* m = (const uint16_t*)p.bias + (int64_t)h * p.S * p.S;
    fill([&](int k) -> uint32_t { return m[ROW_IS_QUERY ? rc * p.S + k : k * p.S + rc]; });
  } else {
    fill([&](int) -> uint32_t { return 0; });
  }
}
// element v of a block
__device__ inline float bias_of(const uint32_t (&b)[8], int v) {
  return (v & 1) ? __uint_as_float(b[v >> 1] & 0xffff0000u) : __uint_as_float(b[v >> 1] << 16);
}

template <int NB>
struct WinLds {
  uint16_t t0[32 * NB * WLD];  // forward, dQ: K; dK/dV: Q
  uint16_t t1[32 * NB * WLD];  // forward, dQ: V; dK/dV: dO
  float lse2[32 * NB], delta[32 * NB];
  int rid[32 * NB];
  int cidx[32 * NB];
  uint16_t table[MAX_RELPOS_R];
};

// relative-position table and token coordinates into LDS; the caller synchronises
template <int NB>
__device__ inline void table_setup(const KP& p, int h, WinLds<NB>& L, int tid) {
  if (p.bias_kind != 2) return;
  const int R = (2 * p.win_h - 1) * (2 * p.win_w - 1);
  for (int i = tid; i < p.S; i += 64 * NB) L.cidx[i] = (i / p.win_w) * (2 * p.win_w - 1) + (i % p.win_w);
  for (int i = tid; i < R; i += 64 * NB) L.table[i] = ((const uint16_t*)p.bias)[(int64_t)h * R + i];
}

// a row's two tensors, two 16-byte chunks of each per thread (rows past S - 1 repeat the last one)
template <int NB>
struct RowStage {
  u32x4 a[2], c[2];
  __device__ void load(const uint16_t* A, int64_t sa, const uint16_t* C, int64_t sc, int S, int tid) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int idx = tid + i * 64 * NB, row = min(idx >> 2, S - 1), col = (idx & 3) * 8;
      a[i] = *(const u32x4*)(A + (int64_t)row * sa + col);
      c[i] = *(const u32x4*)(C + (int64_t)row * sc + col);
    }
  }
  __device__ void store(WinLds<NB>& L, int tid) const {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int idx = tid + i * 64 * NB, at = (idx >> 2) * WLD + (idx & 3) * 8;
      *(u32x4*)(L.t0 + at) = a[i];
      *(u32x4*)(L.t1 + at) = c[i];
    }
  }
};

// does the row's region mask mask anything at all?  Most windows of a shifted map lie inside one region;
// their rows take the code without the comparison (uniform)
template <int NB>
__device__ inline bool row_is_masked(const int* ids, int S, int lane) {
  const int first = ids[0];
  int other = 0;  // all loads in flight together
#pragma unroll
  for (int c = 0; c < (NB + 1) / 2; ++c) other |= ids[min(lane + 64 * c, S - 1)] ^ first;
  return __builtin_amdgcn_ballot_w64(other != 0) != 0;
}

// adds the bias to a block of scores (natural units) and masks pairs of different regions
__device__ inline void bias_and_mask(f32x16& s, const uint32_t (&bz)[8], float scale, bool masked, const int* rid, int my_rid,
                                     int k0, int hl) {
#pragma unroll
  for (int v = 0; v < 16; ++v) s[v] = fmaf(s[v], scale, bias_of(bz, v));
  if (masked) {
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int4 rk = *(const int4*)(rid + k0 + 8 * g + 4 * hl);
      s[4 * g + 0] = rk.x != my_rid ? -INFINITY : s[4 * g + 0];
      s[4 * g + 1] = rk.y != my_rid ? -INFINITY : s[4 * g + 1];
      s[4 * g + 2] = rk.z != my_rid ? -INFINITY : s[4 * g + 2];
      s[4 * g + 3] = rk.w != my_rid ? -INFINITY : s[4 * g + 3];
    }
  }
}

// ---------------------------------------------------------------------------
// forward: grid (row groups, heads); lane = query
// ---------------------------------------------------------------------------
template <int NB, bool REGION>
__global__ __launch_bounds__(64 * NB) __attribute__((amdgpu_waves_per_eu(3, 3))) void win_fwd_kernel(KP p, int rows_per_wg) {
  __shared__ __attribute__((aligned(16))) WinLds<NB> L;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, r = lane & 31, hl = lane >> 5;
  const int h = p.h0 + blockIdx.y, q = 32 * w + r, qc = min(q, p.S - 1);
  const int bfirst = p.b0 + blockIdx.x * rows_per_wg, blast = min(bfirst + rows_per_wg, p.b1);
  RowStage<NB> next;
  bf16x8 qn[2];
  auto fetch = [&](int b) {
    const int64_t base = (int64_t)b * p.sb + (int64_t)h * p.sh;
    next.load((const uint16_t*)p.K + base, p.ss, (const uint16_t*)p.V + base, p.ss, p.S, tid);
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) qn[ks] = *(const bf16x8*)((const uint16_t*)p.Q + base + (int64_t)qc * p.ss + 16 * ks + 8 * hl);
  };
  fetch(bfirst);
  table_setup(p, h, L, tid);
  __syncthreads();
  uint32_t bz[NB][8];
  gather_bias<NB, true>(p, L.table, L.cidx, h, q, hl, false, bz);
  for (int b = bfirst; b < blast; ++b) {
    const int64_t base = (int64_t)b * p.sb + (int64_t)h * p.sh;
    const bf16x8 qf[2] = {qn[0], qn[1]};
    __syncthreads();
    next.store(L, tid);
    bool masked = false;
    int my_rid = 0;
    if (REGION) {
      const int* ids = p.region + (int64_t)(b % p.mask_period) * p.S;
      masked = row_is_masked<NB>(ids, p.S, lane);
      my_rid = ids[qc];
      if (tid < 32 * NB) L.rid[tid] = ids[min(tid, p.S - 1)];
    }
    __syncthreads();
    if (b + 1 < blast) fetch(b + 1);
    f32x16 oacc;
#pragma unroll
    for (int v = 0; v < 16; ++v) oacc[v] = 0.f;
    float m = -1e30f, l = 0.f;
    f32x16 oacc1[1];
#pragma unroll
    for (int c = 0; c < NB; ++c) {
      block_boundary(bz[c]);
      f32x16 s;
#pragma unroll
      for (int v = 0; v < 16; ++v) s[v] = 0.f;
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) s = mfma(lds_nat<WLD>(L.t0, 32 * c + r, ks, hl), qf[ks], s);
      bias_and_mask(s, bz[c], p.scale, masked, L.rid, my_rid, 32 * c, hl);
      float rmax = s[0];
#pragma unroll
      for (int v = 1; v < 16; ++v) rmax = fmaxf(rmax, s[v]);
      rmax = half_max(rmax * LOG2E);
      if (__builtin_amdgcn_ballot_w64(rmax > m + 8.f) != 0) {  // raised only when exceeded by 2^8
        const float mn = fmaxf(m, rmax);
        const float alpha = fast_exp2(m - mn);
        m = mn;
        l *= alpha;
#pragma unroll
        for (int v = 0; v < 16; ++v) oacc[v] *= alpha;
      }
      float pr[16];
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        pr[v] = fast_exp2(fmaf(s[v], LOG2E, -m));
        l += pr[v];
      }
#pragma unroll
      for (int j = 0; j < 2; ++j) oacc = mfma(lds_tr<WLD>(L.t1, 32 * c + 16 * j, 0, lane), pack8(&pr[8 * j]), oacc);
    }
    oacc1[0] = oacc;
    fwd_epilogue<1, false>(p, oacc1, m, l, b, h, q, hl, base);
  }
}

// ---------------------------------------------------------------------------
// recompute pass and dQ in one walk over the keys (the two-product form of fast_rdq.hip): statistics,
// Delta, dG, the pre-gated dO and dQ; lane = query
// ---------------------------------------------------------------------------
template <int NB, bool REGION>
__global__ __launch_bounds__(64 * NB) __attribute__((amdgpu_waves_per_eu(3, 3))) void win_rdq_kernel(KP p, int rows_per_wg) {
  __shared__ __attribute__((aligned(16))) WinLds<NB> L;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, r = lane & 31, hl = lane >> 5;
  const int h = p.h0 + blockIdx.y, q = 32 * w + r, qc = min(q, p.S - 1);
  const int bfirst = p.b0 + blockIdx.x * rows_per_wg, blast = min(bfirst + rows_per_wg, p.b1);
  RowStage<NB> next;
  bf16x8 qn[2];
  u32x4 dyn[2];
  auto fetch = [&](int b) {
    const int64_t base = (int64_t)b * p.sb + (int64_t)h * p.sh;
    next.load((const uint16_t*)p.K + base, p.ss, (const uint16_t*)p.V + base, p.ss, p.S, tid);
  };
  auto fetch_q = [&](int b) {
    const int64_t at = (int64_t)b * p.sb + (int64_t)h * p.sh + (int64_t)qc * p.ss + 8 * hl;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      qn[ks] = *(const bf16x8*)((const uint16_t*)p.Q + at + 16 * ks);
      dyn[ks] = *(const u32x4*)((const uint16_t*)p.dY + at + 16 * ks);
    }
  };
  fetch(bfirst);
  fetch_q(bfirst);
  table_setup(p, h, L, tid);
  __syncthreads();
  uint32_t bz[NB][8];
  gather_bias<NB, true>(p, L.table, L.cidx, h, q, hl, false, bz);
  union { uint32_t u; bf16x2 v; } one_pair;
  one_pair.u = 0x3f803f80u;
  const bf16x2 ones2 = one_pair.v;
  for (int b = bfirst; b < blast; ++b) {
    const int64_t base = (int64_t)b * p.sb + (int64_t)h * p.sh;
    const bf16x8 qf[2] = {qn[0], qn[1]};
    bf16x8 gf[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      union { u32x4 u; uint16_t s[8]; bf16x8 v; } o;
      o.u = dyn[ks];
      if (p.gated) {  // dO = dY * gate, rounded as the epilogue rounds the copy that the later kernel reads
        const u32x4 gg = *(const u32x4*)((const uint16_t*)p.G + base + (int64_t)qc * p.ss + 16 * ks + 8 * hl);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float go = (e & 1) ? __uint_as_float(dyn[ks][e >> 1] & 0xffff0000u) : __uint_as_float(dyn[ks][e >> 1] << 16);
          const float gl = (e & 1) ? __uint_as_float(gg[e >> 1] & 0xffff0000u) : __uint_as_float(gg[e >> 1] << 16);
          o.s[e] = f2bf(go * fast_rcp(1.f + fast_exp2(-gl * LOG2E)));
        }
      }
      gf[ks] = o.v;
    }
    __syncthreads();
    next.store(L, tid);
    bool masked = false;
    int my_rid = 0;
    if (REGION) {
      const int* ids = p.region + (int64_t)(b % p.mask_period) * p.S;
      masked = row_is_masked<NB>(ids, p.S, lane);
      my_rid = ids[qc];
      if (tid < 32 * NB) L.rid[tid] = ids[min(tid, p.S - 1)];
    }
    __syncthreads();
    if (b + 1 < blast) fetch(b + 1);
    f32x16 oacc[1], a1, a2;
#pragma unroll
    for (int v = 0; v < 16; ++v) { oacc[0][v] = 0.f; a1[v] = 0.f; a2[v] = 0.f; }
    float m = -1e30f, lsum = 0.f, dsum = 0.f, l32 = 0.f;
    DpShift shift;
#pragma unroll
    for (int c = 0; c < NB; ++c) {
      block_boundary(bz[c]);
      f32x16 s, pa;
#pragma unroll
      for (int v = 0; v < 16; ++v) { s[v] = 0.f; pa[v] = 0.f; }
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        s = mfma(lds_nat<WLD>(L.t0, 32 * c + r, ks, hl), qf[ks], s);
        pa = mfma(lds_nat<WLD>(L.t1, 32 * c + r, ks, hl), gf[ks], pa);
      }
      bias_and_mask(s, bz[c], p.scale, masked, L.rid, my_rid, 32 * c, hl);
      float rmax = s[0];
#pragma unroll
      for (int v = 1; v < 16; ++v) rmax = fmaxf(rmax, s[v]);
      rmax = half_max(rmax * LOG2E);
      if (__builtin_amdgcn_ballot_w64(rmax > m + 8.f) != 0) {
        const float mn = fmaxf(m, rmax);
        const float alpha = fast_exp2(m - mn);
        m = mn;
        shift.rescaled(alpha);
        lsum *= alpha;
        dsum *= alpha;
        l32 *= alpha;
#pragma unroll
        for (int v = 0; v < 16; ++v) { oacc[0][v] *= alpha; a1[v] *= alpha; a2[v] *= alpha; }
      }
      float pr[16], dp[16];
#pragma unroll
      for (int v = 0; v < 16; ++v) pr[v] = fast_exp2(fmaf(s[v], LOG2E, -m));
      if (p.lse_out) {
#pragma unroll
        for (int v = 0; v < 16; ++v) l32 += pr[v];
      }
      shift.choose(pr, pa);
#pragma unroll
      for (int v = 0; v < 16; ++v) dp[v] = pr[v] * (pa[v] - shift.c);
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        union { bf16x8 v; bf16x2 h[4]; } pf, df;
        pf.v = pack8(&pr[8 * j]);
        df.v = pack8(&dp[8 * j]);
#pragma unroll
        for (int e = 0; e < 4; ++e) {  // the sums run over the rounded operands
          lsum = __builtin_amdgcn_fdot2_f32_bf16(pf.h[e], ones2, lsum, false);
          dsum = __builtin_amdgcn_fdot2_f32_bf16(df.h[e], ones2, dsum, false);
        }
        const bf16x8 vt = lds_tr<WLD>(L.t1, 32 * c + 16 * j, 0, lane), kt = lds_tr<WLD>(L.t0, 32 * c + 16 * j, 0, lane);
        oacc[0] = mfma(vt, pf.v, oacc[0]);
        a2 = mfma(kt, pf.v, a2);
        a1 = mfma(kt, df.v, a1);
      }
    }
    if (b + 1 < blast) fetch_q(b + 1);
    if (q < p.S) {
      const float l = half_sum(lsum), inv = 1.f / l, dmean = half_sum(dsum) * inv;
      uint2 o[4];
#pragma unroll
      for (int g = 0; g < 4; ++g)
        o[g] = pack4_bf16(fmaf(-dmean, a2[4 * g], a1[4 * g]), fmaf(-dmean, a2[4 * g + 1], a1[4 * g + 1]),
                          fmaf(-dmean, a2[4 * g + 2], a1[4 * g + 2]), fmaf(-dmean, a2[4 * g + 3], a1[4 * g + 3]), p.scale * inv);
      store_row32((uint16_t*)p.dQ + base + (int64_t)q * p.ss, o, hl, true);
      fwd_epilogue_rowsum<1, true>(p, oacc, m, l, half_sum(l32), b, h, q, hl, base);
    }
  }
}

// ---------------------------------------------------------------------------
// dK, dV and the bias gradient in one walk over the queries; lane = key.  A work-group takes one group
// of p.sm_gw consecutive global rows (or the chunk's part of it); dS is added in registers, row after
// row, and stored as the group's partial sum, resumed when a chunk boundary cuts the group.
// ---------------------------------------------------------------------------
template <int NB, bool REGION>
__global__ __launch_bounds__(64 * NB) __attribute__((amdgpu_waves_per_eu(2, 2))) void win_kv_kernel(KP p) {
  __shared__ __attribute__((aligned(16))) WinLds<NB> L;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, r = lane & 31, hl = lane >> 5;
  const int h = p.h0 + blockIdx.y, key = 32 * w + r, kc = min(key, p.S - 1);
  const int g = p.b0 / p.sm_gw + blockIdx.x;  // global group
  const int bfirst = max(g * p.sm_gw, p.b0), blast = min((g + 1) * p.sm_gw, p.b1);
  RowStage<NB> next;
  float stat = 0.f;
  auto fetch = [&](int b) {
    const int64_t base = (int64_t)b * p.sb + (int64_t)h * p.sh;
    next.load((const uint16_t*)p.Q + base, p.ss,
              (const uint16_t*)p.dO + (int64_t)(b - p.do_b0) * p.do_sb + (int64_t)(h - p.do_h0) * p.do_sh, p.do_ss, p.S, tid);
    // 64 NB threads, two statistics for 32 NB queries
    const int i = min(tid < 32 * NB ? tid : tid - 32 * NB, p.S - 1);
    stat = tid < 32 * NB ? p.lse[(int64_t)(b - p.lse_b0) * p.lse_sb + (int64_t)(h - p.lse_h0) * p.lse_sh + i]
                         : p.delta[(int64_t)(b - p.dl_b0) * p.dl_sb + (int64_t)(h - p.dl_h0) * p.dl_sh + i];
  };
  fetch(bfirst);
  table_setup(p, h, L, tid);
  __syncthreads();
  uint32_t bz[NB][8];
  gather_bias<NB, false>(p, L.table, L.cidx, h, key, hl, key >= p.S, bz);
  float acc[NB][16];
  float* part = nullptr;
  if (p.sm_partial) {
    part = p.sm_partial + ((int64_t)((g - p.sm_g0) % p.sm_ring) * p.sm_hs + (h - p.sm_h0)) * p.S * p.S;
    const bool resume = max(g * p.sm_gw, p.share_b0) < p.b0;  // an earlier chunk started this group
#pragma unroll
    for (int c = 0; c < NB; ++c)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        if ((v & 7) == 0) block_boundary(bz[c]);
        const int i = 32 * c + key_of(v, hl);
        acc[c][v] = resume && i < p.S && key < p.S ? part[i * p.S + key] : 0.f;
      }
  }
  for (int b = bfirst; b < blast; ++b) {
    const int64_t base = (int64_t)b * p.sb + (int64_t)h * p.sh;
    bf16x8 kf[2], vf[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      const int64_t at = base + (int64_t)kc * p.ss + 16 * ks + 8 * hl;
      kf[ks] = *(const bf16x8*)((const uint16_t*)p.K + at);
      vf[ks] = *(const bf16x8*)((const uint16_t*)p.V + at);
    }
    __syncthreads();
    next.store(L, tid);
    if (tid < 32 * NB) L.lse2[tid] = -stat * LOG2E;  // negated: one fused multiply-add per score
    else L.delta[tid - 32 * NB] = stat;
    bool masked = false;
    int my_rid = 0;
    if (REGION) {
      const int* ids = p.region + (int64_t)(b % p.mask_period) * p.S;
      masked = row_is_masked<NB>(ids, p.S, lane);
      my_rid = ids[kc];
      if (tid < 32 * NB) L.rid[tid] = ids[min(tid, p.S - 1)];
    }
    __syncthreads();
    if (b + 1 < blast) fetch(b + 1);
    f32x16 dk, dv;
#pragma unroll
    for (int v = 0; v < 16; ++v) { dk[v] = 0.f; dv[v] = 0.f; }
#pragma unroll
    for (int c = 0; c < NB; ++c) {
      block_boundary(bz[c]);
      f32x16 s, pa;
#pragma unroll
      for (int v = 0; v < 16; ++v) { s[v] = 0.f; pa[v] = 0.f; }
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        s = mfma(lds_nat<WLD>(L.t0, 32 * c + r, ks, hl), kf[ks], s);
        pa = mfma(lds_nat<WLD>(L.t1, 32 * c + r, ks, hl), vf[ks], pa);
      }
      // exponents and dP - Delta; masked pairs get -inf and 0 here, after the statistics went in, so that they contribute
      // nothing also where a query has NaN statistics
#pragma unroll
      for (int gq = 0; gq < 4; ++gq) {
        const f32x4 l4 = *(const f32x4*)(L.lse2 + 32 * c + 8 * gq + 4 * hl);
        const f32x4 d4 = *(const f32x4*)(L.delta + 32 * c + 8 * gq + 4 * hl);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int v = 4 * gq + e;
          s[v] = fmaf(fmaf(s[v], p.scale, bias_of(bz[c], v)), LOG2E, l4[e]);
          pa[v] -= d4[e];
        }
      }
      if (REGION && masked) {
#pragma unroll
        for (int gq = 0; gq < 4; ++gq) {
          const int4 rk = *(const int4*)(L.rid + 32 * c + 8 * gq + 4 * hl);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const bool dead = (e == 0 ? rk.x : e == 1 ? rk.y : e == 2 ? rk.z : rk.w) != my_rid;
            s[4 * gq + e] = dead ? -INFINITY : s[4 * gq + e];
            pa[4 * gq + e] = dead ? 0.f : pa[4 * gq + e];
          }
        }
      }
      float pr[16], ds[16];
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        pr[v] = fast_exp2(s[v]);
        ds[v] = pr[v] * pa[v];
      }
      if (part) {
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[c][v] += ds[v];
      }
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        dv = mfma(lds_tr<WLD>(L.t1, 32 * c + 16 * j, 0, lane), pack8(&pr[8 * j]), dv);
        dk = mfma(lds_tr<WLD>(L.t0, 32 * c + 16 * j, 0, lane), pack8(&ds[8 * j]), dk);
      }
    }
    if (key < p.S) {
      uint2 a[4], c[4];
#pragma unroll
      for (int gd = 0; gd < 4; ++gd) {
        a[gd] = pack4_bf16(dk[4 * gd], dk[4 * gd + 1], dk[4 * gd + 2], dk[4 * gd + 3], p.scale);
        c[gd] = pack4_bf16(dv[4 * gd], dv[4 * gd + 1], dv[4 * gd + 2], dv[4 * gd + 3], 1.f);
      }
      store_row32((uint16_t*)p.dK + base + (int64_t)key * p.ss, a, hl, true);
      store_row32((uint16_t*)p.dV + base + (int64_t)key * p.ss, c, hl, true);
    }
  }
  if (part && key < p.S) {
    int at = key;  // opaque: the addresses are not to be kept in registers from the load of the partial sum on
    asm volatile("" : "+v"(at));
#pragma unroll
    for (int c = 0; c < NB; ++c)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        if ((v & 7) == 0) block_boundary(bz[c]);
        const int i = 32 * c + key_of(v, hl);
        if (i < p.S) part[i * p.S + at] = acc[c][v];
      }
  }
}

// Rows per work-group of the kernels that may choose freely (a row's results do not depend on it): the
// bias gather costs about half a row, so as many rows as still leave `per_cu` work-groups per
// compute unit, at most 8.
inline int rows_per_wg(const KP& p, int per_cu) {
  const int64_t units = (int64_t)(p.b1 - p.b0) * (p.h1 - p.h0), r = units / (256 * per_cu);
  return (int)(r < 1 ? 1 : r > 8 ? 8 : r);
}

template <class F>
hipError_t with_shape(const KP& p, F f) {
  auto mask = [&](auto nb) {
    if (p.mask_kind == 2) f(nb, std::true_type{});
    else f(nb, std::false_type{});
  };
  if (p.S <= 96) mask(std::integral_constant<int, 3>{});
  else if (p.S <= 128) mask(std::integral_constant<int, 4>{});
  else mask(std::integral_constant<int, 5>{});
  return hipGetLastError();
}

}  // namespace

hipError_t launch_win_fwd(const KP& p, hipStream_t st) {
  const int rows = rows_per_wg(p, 3);
  const dim3 g((p.b1 - p.b0 + rows - 1) / rows, p.h1 - p.h0);
  return with_shape(p, [&](auto nb, auto region) { win_fwd_kernel<nb(), region()><<<g, 64 * nb(), 0, st>>>(p, rows); });
}
hipError_t launch_win_recompute_dq(const KP& p, hipStream_t st) {
  const int rows = rows_per_wg(p, 2);
  const dim3 g((p.b1 - p.b0 + rows - 1) / rows, p.h1 - p.h0);
  return with_shape(p, [&](auto nb, auto region) { win_rdq_kernel<nb(), region()><<<g, 64 * nb(), 0, st>>>(p, rows); });
}
hipError_t launch_win_kv(const KP& args, hipStream_t st) {
  KP p = args;
  if (p.dbias_acc && !p.sm_partial) {  // no partial sums: all rows are one group, which sums in the result itself
    p.sm_partial = p.dbias_acc;
    p.sm_gw = p.B;
    p.sm_g0 = 0; p.sm_ring = 1; p.sm_hs = p.H; p.sm_h0 = 0;
  }
  const dim3 g((p.b1 - 1) / p.sm_gw - p.b0 / p.sm_gw + 1, p.h1 - p.h0);
  return with_shape(p, [&](auto nb, auto region) { win_kv_kernel<nb(), region()><<<g, 64 * nb(), 0, st>>>(p); });
}

}  // namespace ssa

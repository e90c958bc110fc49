// Forward of attention over windows of 65 to 160 tokens with head size 32, bf16: a whole row (b, h) is small
// enough to share one work-group, too large for one wavefront (small_kernels.hip ends at 64 tokens; the backward is win_bwd.hip).
//
// A work-group has one wavefront per 32-token block (NB = 3, 4 or 5); K and V of the row are staged in LDS
// once for all of them.  The scores start from the bias (BiasCopy in mfma_common.h): of more than 128 tokens large shares read it in accumulator
// layout, expanded from the relative-position table once per call into the library's buffer; others and captured calls
// gather it once per work-group and keep it in registers, packed bf16, with the same values.
//
// What bounds it: the chain of loads, matrix steps and vector arithmetic of the few wavefronts that fit a compute unit.
// The bias held in registers by every wavefront (40 of them at NB = 5) left one or two work-groups per compute unit.
// 512 windows of 12 x 12 tokens, 8 heads: 100 -> 71 us.
#include "mfma_common.h"

namespace ssa {
namespace {

constexpr int WD = 32;        // head size
constexpr int WLD = WD + 24;  // LDS row stride of the staged tiles (elements): conflict-free for b128 and transposed reads

// where a block's bias comes from
enum { WB_NONE = 0, WB_COPY = 1, WB_REGS = 2 };

template <int NB>
struct WinLds {
  uint16_t t0[32 * NB * WLD];  // K
  uint16_t t1[32 * NB * WLD];  // V
  alignas(16) int rid[32 * NB];
  alignas(16) int cidx[32 * NB];
  uint16_t table[MAX_RELPOS_R];
};

// relative-position table and token coordinates into LDS; the caller synchronises
template <int NB>
__device__ inline void table_setup(const KP& p, int h, WinLds<NB>& L, int tid) {
  if (p.bias_kind != 2) return;
  const int R = (2 * p.win_h - 1) * (2 * p.win_w - 1);
  if (tid < 32 * NB) {
    const int i = min(tid, p.S - 1);
    L.cidx[tid] = (i / p.win_w) * (2 * p.win_w - 1) + (i % p.win_w);
  }
  for (int i = tid; i < R; i += 64 * NB) L.table[i] = ((const uint16_t*)p.bias)[(int64_t)h * R + i];
}

// What the scores of a block start from: element v is the pair (lane's row, column 32 c + key_of(v, hl)), bias / scale,
// -inf where either lies outside the window.
//  WB_COPY: loaded from the copy in accumulator layout;
//  WB_REGS: gathered once per work-group and kept in registers, packed bf16, 8 per block (the caller unrolls the blocks).
template <int NB, int WB>
struct WinBias {
  BiasCopy bc;
  uint32_t bz[WB == WB_REGS ? NB : 1][8];
  // WB_REGS: the table and the coordinates are in LDS and visible
  __device__ void init(const KP& p, const WinLds<NB>& L, int h, int w, int lane) {
    if (WB == WB_COPY) bc.init(p.bias_q, h - p.bc_h0, 32 * w, p.S, lane);
    if (WB != WB_REGS) return;
    const int row = 32 * w + (lane & 31), hl = lane >> 5, rc = min(row, p.S - 1);
    const int c0 = (p.win_h - 1) * (2 * p.win_w - 1) + (p.win_w - 1);
    const uint16_t* m = (const uint16_t*)p.bias + (int64_t)h * p.S * p.S;
    const int cr = p.bias_kind == 2 ? L.cidx[rc] + c0 : 0;
#pragma unroll
    for (int c = 0; c < NB; ++c) {
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int k = 32 * c + 8 * g + 4 * hl;
        uint32_t x[4];
        if (p.bias_kind == 2) {
          const int4 ck = *(const int4*)(L.cidx + k);
          x[0] = L.table[cr - ck.x];
          x[1] = L.table[cr - ck.y];
          x[2] = L.table[cr - ck.z];
          x[3] = L.table[cr - ck.w];
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e) x[e] = m[rc * p.S + min(k + e, p.S - 1)];
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = row < p.S && k + e < p.S ? x[e] : 0xff80u;  // -inf
        bz[c][2 * g] = x[0] | (x[1] << 16);
        bz[c][2 * g + 1] = x[2] | (x[3] << 16);
      }
#pragma unroll
      for (int i = 0; i < 8; ++i) asm volatile("" : "+v"(bz[c][i]));
    }
  }
  __device__ void get(const KP& p, int w, int c, int lane, f32x16& x) {
    if (WB == WB_COPY) {
      bc.load(x, c);
      return;
    }
    if (WB == WB_REGS) {
      // the bias, which does not change from row to row, is meant to stay packed: the compiler would unpack it once, outside
      // the row loop, into twice the registers
#pragma unroll
      for (int i = 0; i < 8; ++i) asm volatile("" : "+v"(bz[c][i]));
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const uint32_t u = bz[c][v >> 1];
        x[v] = __uint_as_float((v & 1) ? u & 0xffff0000u : u << 16) * p.inv_scale;
      }
      return;
    }
    int row = 32 * w + (lane & 31);  // opaque: nothing of this is to be kept in registers from one row b to the next
    asm volatile("" : "+v"(row));
#pragma unroll
    for (int v = 0; v < 16; ++v) x[v] = row < p.S && 32 * c + key_of(v, lane >> 5) < p.S ? 0.f : -INFINITY;
  }
};

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

// pairs of different regions: -inf
__device__ inline void mask_regions(f32x16& s, const int* rid, int my_rid, int k0, int hl) {
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const int4 rk = *(const int4*)(rid + k0 + 8 * g + 4 * hl);
    s[4 * g + 0] = rk.x != my_rid ? -INFINITY : s[4 * g + 0];
    s[4 * g + 1] = rk.y != my_rid ? -INFINITY : s[4 * g + 1];
    s[4 * g + 2] = rk.z != my_rid ? -INFINITY : s[4 * g + 2];
    s[4 * g + 3] = rk.w != my_rid ? -INFINITY : s[4 * g + 3];
  }
}

// ---------------------------------------------------------------------------
// forward: a run of rows of one head per work-group, heads of a row next to each other; lane = query.  WB_REGS: the next row's
// operands travel global -> registers meanwhile.  WB_COPY: one row, 4 wavefronts per SIMD instead (71 us against 74 for 512
// windows of 12 x 12 tokens x 8 heads).
// ---------------------------------------------------------------------------
template <int NB, bool REGION, int WB>
__global__ __launch_bounds__(64 * NB) __attribute__((amdgpu_waves_per_eu(WB == WB_REGS ? 3 : 4, WB == WB_REGS ? 3 : 4))) void win_fwd_kernel(KP p, int rows_per_wg) {
#pragma clang fp contract(off)  // the variants are to give the same bits
  __shared__ __attribute__((aligned(16))) WinLds<NB> L;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, r = lane & 31, hl = lane >> 5;
  constexpr int BLOCK_UNROLL = WB == WB_REGS ? NB : 1;
  constexpr bool RUN = WB != WB_COPY;
  // the next block's bias is at hand before a block's arithmetic (five blocks in registers: no room for a second one)
  constexpr bool AHEAD = WB == WB_COPY || (WB == WB_REGS && NB < 5);
  const BlockId blk = xcd_block_id();
  const int h = p.h0 + blk.x, q = 32 * w + r, qc = min(q, p.S - 1);
  const int bfirst = p.b0 + blk.z * rows_per_wg, blast = RUN ? min(bfirst + rows_per_wg, p.b1) : bfirst + 1;
  RowStage<NB> next;
  bf16x8 qn[2];
  int id0 = 0, ids_n[(NB + 1) / 2] = {};
  auto fetch = [&](int b) {
    const int64_t base = (int64_t)b * p.sb + (int64_t)h * p.sh;
    next.load((const uint16_t*)p.K + base, p.ss, (const uint16_t*)p.V + base, p.ss, p.S, tid);
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) qn[ks] = *(const bf16x8*)((const uint16_t*)p.Q + base + (int64_t)qc * p.ss + 16 * ks + 8 * hl);
    if (REGION) {
      const int* ids = p.region + (int64_t)(b % p.mask_period) * p.S;
      id0 = ids[0];
#pragma unroll
      for (int c = 0; c < (NB + 1) / 2; ++c) ids_n[c] = ids[min(lane + 64 * c, p.S - 1)];
    }
  };
  fetch(bfirst);
  if (WB == WB_REGS) {
    table_setup(p, h, L, tid);
    __syncthreads();
  }
  WinBias<NB, WB> bias;
  bias.init(p, L, h, w, lane);
  f32x16 cz;  // of the block, then of the next one
  if (AHEAD) bias.get(p, w, 0, lane, cz);
  const float c1 = in_vgpr(p.scale * LOG2E);
  for (int b = bfirst; b < blast; ++b) {
    const int64_t base = (int64_t)b * p.sb + (int64_t)h * p.sh;
    const bf16x8 qf[2] = {qn[0], qn[1]};
    if (b > bfirst) __syncthreads();
    next.store(L, tid);
    bool masked = false;
    int my_rid = 0;
    if (REGION) {
      int other = 0;
#pragma unroll
      for (int c = 0; c < (NB + 1) / 2; ++c) other |= ids_n[c] ^ id0;
      masked = __builtin_amdgcn_ballot_w64(other != 0) != 0;
      if (masked && w == 0) {  // every wavefront has all ids; loading them here instead would be a wait of its own
#pragma unroll
        for (int c = 0; c < (NB + 1) / 2; ++c)
          if (lane + 64 * c < 32 * NB) L.rid[lane + 64 * c] = ids_n[c];
      }
    }
    __syncthreads();
    if (masked) my_rid = L.rid[q];
    if (RUN && b + 1 < blast) fetch(b + 1);
    f32x16 oacc[1];
#pragma unroll
    for (int v = 0; v < 16; ++v) oacc[0][v] = 0.f;
    float nm = 1e30f, l = 0.f;  // the negated running maximum, the row sum
#pragma unroll BLOCK_UNROLL
    for (int c = 0; c < NB; ++c) {
      // The maximum is taken on the first block, and where a half-wave's sum of 16 probabilities says that it has grown by a lot: above
      // 2^8 (infinite ones included) for any query the block is formed again, with the maxima of those queries raised; the
      // others go through the same arithmetic as before.
      f32x16 s;
      float sum = INFINITY;
      for (bool look = c == 0 || masked;; look = true) {
        if (!AHEAD) bias.get(p, w, c, lane, cz);
        s = cz;
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) s = mfma(lds_nat<WLD>(L.t0, 32 * c + r, ks, hl), qf[ks], s);
        if (AHEAD) bias.get(p, w, c + 1 < NB ? c + 1 : 0, lane, cz);
        if (masked) mask_regions(s, L.rid, my_rid, 32 * c, hl);
        if (look) {
          float rmax = s[0];
#pragma unroll
          for (int v = 1; v < 16; ++v) rmax = fmaxf(rmax, s[v]);
          rmax = half_max(rmax * c1);
          const float mn = half_max(sum) > 256.f ? fmaxf(-nm, rmax) : -nm, alpha = fast_exp2(-nm - mn);
          nm = -mn;
          l *= alpha;
#pragma unroll
          for (int v = 0; v < 16; ++v) oacc[0][v] *= alpha;
        }
        float x[16];
#pragma unroll
        for (int v = 0; v < 16; ++v) x[v] = s[v] = fast_exp2(fmaf(s[v], c1, nm));
        sum = sum16(x);
        if (look || __builtin_amdgcn_ballot_w64(sum > 256.f) == 0) break;
        if (AHEAD) bias.get(p, w, c, lane, cz);
      }
      l += sum;
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        float x[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] = s[8 * j + e];
        oacc[0] = mfma(lds_tr<WLD>(L.t1, 32 * c + 16 * j, 0, lane), pack8(x), oacc[0]);
      }
    }
    fwd_epilogue<1, false>(p, oacc, -nm, l, b, h, q, hl, base);
  }
}

template <class F>
hipError_t with_shape(const KP& p, bool copy, F f) {
  auto mask = [&](auto nb) {
    auto source = [&](auto region) {
      if (p.bias_kind == 0) f(nb, region, std::integral_constant<int, WB_NONE>{});
      else if (copy) f(nb, region, std::integral_constant<int, WB_COPY>{});
      else f(nb, region, std::integral_constant<int, WB_REGS>{});
    };
    if (p.mask_kind == 2) source(std::true_type{});
    else source(std::false_type{});
  };
  if (p.S <= 96) mask(std::integral_constant<int, 3>{});
  else if (p.S <= 128) mask(std::integral_constant<int, 4>{});
  else mask(std::integral_constant<int, 5>{});
  return hipGetLastError();
}

}  // namespace

hipError_t launch_win_fwd(const KP& p, hipStream_t st) {
  // Rows per work-group.  With the bias in registers, gathered once per work-group: as many as let the launch fit the chip in one round (4, 3 and 1
  // work-groups of 3, 4 and 5 wavefronts per compute unit: two of 5 take as long as one after the other), at most 8; beyond that rounds of at most 6, or 8 of
  // 5 wavefronts.  8 heads, region mask, us, rows x heads of 1536, 2048, 3072, 4096, 6144, 8192, with one row | a row for every 1536 of them | this rule:
  // 9 x 9 tokens 14.4 | 14.4 | 12.0, 19.2 | 19.2 | 14.1, 25.3 | 21.7 | 18.4, 31.1 | 27.2 | 22.8, 42.6 | 33.2 | 30.5, 54.1 | 41.9 | 39.6; 11 x 11: 19.8 | 19.8 | 16.7,
  // 25.7 | 25.8 | 21.9, 34.6 | 29.2 | 26.1, 43.5 | 36.5 | 35.5, 61.4 | 46.1 | 46.0, 78.7 | 61.2 | 61.5; 12 x 12 without the copy (captured): 47.3 | 47.3 | 30.2,
  // 63.8 | 63.8 | 43.6, 92.8 | 71.7 | 60.4, 121 | 93.3 | 77.7, 179 | 116 | 111, 255 | 162 | 168.  One row where there is nothing to gather (no bias, 9 x 9: 2048
  // 12.4 us, two rows 13.2, 8192 33.0 | 35.1; 11 x 11: 17.1 | 19.2, 50.5 | 51.6; 12 x 12: 30.2 | 35.5, 110 | 111) or to hold (the copy).
  // (Work-groups of one head, not rows x heads through rows: 24 heads x 128 rows of 9 x 9 tokens are 1032 work-groups of three rows, 20.7 us, or 768 of four, 17.9.)
  const int per_cu = p.S <= 96 ? 4 : p.S <= 128 ? 3 : 1;
  const int64_t slots = 256 * per_cu, nrows = p.b1 - p.b0, heads = p.h1 - p.h0, once = (nrows * heads + slots - 1) / slots;
  const int64_t most = per_cu == 1 ? 8 : 6, rounds = once <= 8 ? 1 : (once + most - 1) / most;
  const int64_t of_head = slots * rounds / heads > 1 ? slots * rounds / heads : 1;
  const int rows = p.bias_q || p.bias_kind == 0 ? 1 : (int)((nrows + of_head - 1) / of_head);
  const dim3 g(p.h1 - p.h0, 1, (p.b1 - p.b0 + rows - 1) / rows);
  return with_shape(p, p.bias_q != nullptr, [&](auto nb, auto region, auto wb) {
    constexpr int WB = wb() == WB_COPY && nb() < 5 ? WB_REGS : wb();  // no copy up to 128 tokens (bias_copy_bytes_for)
    win_fwd_kernel<nb(), region(), WB><<<g, 64 * nb(), 0, st>>>(p, rows);
  });
}
}  // namespace ssa

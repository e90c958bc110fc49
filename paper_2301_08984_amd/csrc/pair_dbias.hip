// Bias gradient of pair attention, head size 32, heads side by side in memory: dBias[h][i][j] = sum over rows b of P (dP - Delta).
//
// A work-group owns 64 queries x 64 keys of two neighbouring heads and walks rows b; each of its four wavefronts owns 32 x 64 of one head, lane = query,
// so that a row's Q and dO fragments serve two key blocks.  A row's Q, dO, K and V pieces (128 bytes a token: both heads) travel straight into
// one of two LDS buffers, a row ahead, with one barrier a row; two work-groups share a compute unit.
//
// What bounds it: 1024 rows x 4 heads x 1024, an eighth of the rows a launch, all launches, us: 1180 (1620 with a wavefront per 32 x 32 block, operands stored to
// LDS from registers and Delta subtracted).  Timing builds of the first version, 64 x 128 keys and eight wavefronts, three buffers (1300; without a row step at all 180: the
// start and end of eight launches): the vector arithmetic alone 550 more, of which the exponentials 350, the matrix instructions 360, these
// two 740, with the LDS reads 840, the loads alone 520 (24 TB/s from L2).  Loads dealt out over the arithmetic instead of in one piece after the barrier,
// and all start-up loads in flight together: 1200; half the keys and two work-groups on a compute unit 1180, and 512 x 8 x 384 (288 work-groups a launch instead of
// 144) 285 -> 260.  Not better: the heads' wavefronts half a row apart (1300 -> 1330), key tiles in bands of 4 or 2 (the same).
#include "wave_dma.h"

namespace ssa {
namespace {

constexpr int PB_T = 64;                              // queries, and keys, of a work-group
constexpr int PB_NST = 2;                             // buffers
typedef f32x4 f32x4_any __attribute__((aligned(4)));  // rows of S entries start anywhere
typedef u32x2 u32x2_any __attribute__((aligned(2)));

template <bool CAUSAL>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void dbias_pair_kernel(KP p) {
  constexpr int D = 32, NW = 4;                               // wavefronts
  constexpr int AREA_G = 128 * PB_T, AREA_K = 2 * AREA_G, AREA_V = 3 * AREA_G, AREA_S = 4 * AREA_G;
  constexpr int STAGE = AREA_S + 16 * PB_T;                   // Q, dO, K, V; LSE, Delta of head 0, of head 1
  constexpr int RQ = PB_T / (8 * NW), LOADS = 4 * RQ + 1;     // load instructions of 8 rows per wavefront and tensor; all
  __shared__ __attribute__((aligned(1024))) char smem[PB_NST * STAGE];
  const int lane = threadIdx.x & 63, r = lane & 31, hl = lane >> 5;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int hsel = w >> 1, wq = w & 1;
  const int pairs = (p.h1 - p.h0) / 2;
  const BlockId blk = xcd_block_id();
  const int hA = p.h0 + (blk.z % pairs) * 2, h = hA + hsel;
  const int q0t = blk.y * PB_T, k0 = blk.x * PB_T, q0 = q0t + 32 * wq;
  const int q = q0 + r, qc = min(q, p.S - 1);
  // rows of this work-group: the chunk, or the part of one row group inside the chunk
  int bfirst = p.b0, blast = p.b1;
  float* dst;
  bool resume;
  if (p.sm_partial) {
    const int g = p.b0 / p.sm_gw + blk.z / pairs;
    bfirst = max(g * p.sm_gw, p.b0);
    blast = min((g + 1) * p.sm_gw, p.b1);
    dst = p.sm_partial + ((int64_t)((g - p.sm_g0) % p.sm_ring) * p.sm_hs + (h - p.sm_h0)) * p.S * p.S + (int64_t)qc * p.S;
    resume = max(g * p.sm_gw, p.share_b0) < p.b0;
  } else {
    dst = p.dbias_acc + ((int64_t)h * p.S + qc) * p.S;
    resume = p.dbias_accumulate != 0;
  }
  if (bfirst >= blast) return;
  const bool skip = CAUSAL && k0 > q0t + PB_T - 1;  // whole tile above the diagonal: gradient is zero

  // A load instruction fills 1 KB, 8 rows of both heads: lane l the position l % 8 of row l / 8, where chunk c (16 bytes) of row i
  // sits at position c ^ (i / 2 % 8): 16 consecutive rows put one chunk index at 16 different bank groups.  Wavefront w fetches
  // rows 8w .. 8w + 7 and those 32 on of a tensor, and one of the four runs of statistics.
  // Rows past S - 1 arrive as zeros or belong to somebody else: their results are not stored.
  const uint32_t ss2 = (uint32_t)p.ss * 2u, dss2 = (uint32_t)p.do_ss * 2u;
  const int slice = (int)(((int64_t)(p.S - 1) * p.ss + 2 * D) * 2), dslice = (int)(((int64_t)(p.S - 1) * p.do_ss + 2 * D) * 2);  // < 1 GiB
  const int row = 8 * w + (lane >> 3);
  const uint32_t chunk = 16u * (uint32_t)((lane & 7) ^ ((row >> 1) & 7));
  const uint32_t oq = (uint32_t)(q0t + row) * ss2 + chunk, og = (uint32_t)(q0t + row) * dss2 + chunk, ok = (uint32_t)(k0 + row) * ss2 + chunk;
  const bool second = (w & 1) != 0;
  const int hs = hA + (w >> 1);
  const float* stats = second ? p.delta + (int64_t)(hs - p.dl_h0) * p.dl_sh : p.lse + (int64_t)(hs - p.lse_h0) * p.lse_sh;
  const int64_t stats_sb = second ? p.dl_sb : p.lse_sb;
  const int stats_b0 = second ? p.dl_b0 : p.lse_b0;
  const uint32_t os = 4u * (uint32_t)(q0t + lane);
  struct Row {  // where a row's tensors are
    __amdgpu_buffer_rsrc_t q, g, k, v, s;
  };
  auto row_of = [&](int b) {
    const bool live = b < blast;  // past the last row: empty descriptors, zeros arrive
    b = min(b, blast - 1);
    auto rsrc = [&](const void* x, int bytes) { return __builtin_amdgcn_make_buffer_rsrc((void*)x, 0, live ? bytes : 0, 0x00020000); };
    const int64_t base = (int64_t)b * p.sb + (int64_t)hA * p.sh;
    return Row{rsrc((const uint16_t*)p.Q + base, slice),
               rsrc((const uint16_t*)p.dO + (int64_t)(b - p.do_b0) * p.do_sb + (int64_t)(hA - p.do_h0) * p.do_sh, dslice),
               rsrc((const uint16_t*)p.K + base, slice), rsrc((const uint16_t*)p.V + base, slice),
               rsrc(stats + (int64_t)(b - stats_b0) * stats_sb, p.S * 4)};
  };
  auto load = [&](int at, const Row& x, int i) {  // the i-th load instruction of a row
    char* to = smem + at + w * 1024;
    auto piece = [&](const __amdgpu_buffer_rsrc_t& from, int area, uint32_t off, int n, uint32_t step) {
      __builtin_amdgcn_raw_ptr_buffer_load_lds(from, (w_lds_void*)(to + area + n * NW * 1024), 16, off + (uint32_t)n * (8u * NW) * step, 0, 0, 0);
    };
    if (i < RQ) piece(x.q, 0, oq, i, ss2);
    else if (i < 2 * RQ) piece(x.g, AREA_G, og, i - RQ, dss2);
    else if (i < 3 * RQ) piece(x.k, AREA_K, ok, i - 2 * RQ, ss2);
    else if (i < 4 * RQ) piece(x.v, AREA_V, ok, i - 3 * RQ, ss2);
    else __builtin_amdgcn_raw_ptr_buffer_load_lds(x.s, (w_lds_void*)(smem + at + AREA_S + 256 * w), 4, os, 0, 0, 0);
  };
  if (!skip) {
#pragma unroll
    for (int n = 0; n < PB_NST; ++n) {
      const Row x = row_of(bfirst + n);
#pragma unroll
      for (int i = 0; i < LOADS; ++i) load(n * STAGE, x, i);
    }
  }
  f32x16 bz[2], acc[2];  // bias / scale, from which the scores start; the sums
  {
    const uint16_t* brow = (const uint16_t*)p.bias + ((int64_t)h * p.S + qc) * p.S;
    const bool inside = k0 + PB_T <= p.S, from = resume && !skip;
    u32x2 u[2][4];
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[c][v] = 0.f;
    if (inside) {
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int g = 0; g < 4; ++g) u[c][g] = *(const u32x2_any*)(brow + k0 + 32 * c + 8 * g + 4 * hl);
      if (from) {
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            const f32x4 a = *(const f32x4_any*)(dst + k0 + 32 * c + 8 * g + 4 * hl);
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[c][4 * g + e] = a[e];
          }
      }
    } else {
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          uint32_t x[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) x[e] = brow[min(k0 + 32 * c + 8 * g + 4 * hl + e, p.S - 1)];
          u[c][g] = u32x2{x[0] | x[1] << 16, x[2] | x[3] << 16};
        }
      if (from) {
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
          for (int v = 0; v < 16; ++v) acc[c][v] = dst[min(k0 + 32 * c + key_of(v, hl), p.S - 1)];
      }
    }
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const uint32_t x = u[c][v >> 2][(v >> 1) & 1];
        bz[c][v] = __uint_as_float(v & 1 ? x & 0xffff0000u : x << 16) * p.inv_scale;
      }
  }
  if (!skip) {
    // the lane's fragments: chunk 4 hsel + 2 ks + hl of its rows; its query's statistics
    const uint32_t lds0 = (uint32_t)(size_t)(w_lds_void*)smem;
    const uint32_t pos = (uint32_t)(((4 * hsel + hl) ^ ((r >> 1) & 7)) << 4);
    const uint32_t aq = lds0 + (uint32_t)(32 * wq + r) * 128u + pos, ak = lds0 + AREA_K + (uint32_t)r * 128u + pos;
    const uint32_t as = lds0 + AREA_S + 512u * hsel + 4u * (uint32_t)(32 * wq + r);
    const float c1 = in_vgpr(p.scale * LOG2E);
    struct Frags {
      float lse, delta;
      u32x4 q[2], g[2], k[2][2], v[2][2];
    } f;
    // A row's fragments are read under the arithmetic on the row before.
    auto issue = [&](int at) {
      const uint32_t q0a = aq + at, q1a = q0a ^ 32u, k0a = ak + at, k1a = k0a ^ 32u, sta = as + at;
      asm volatile("ds_read_b32 %0, %2\n\tds_read_b32 %1, %2 offset:256" : "=&v"(f.lse), "=&v"(f.delta) : "v"(sta) : "memory");
      asm volatile(
          "ds_read_b128 %0, %8\n\tds_read_b128 %1, %9\n\tds_read_b128 %4, %10\n\tds_read_b128 %5, %11\n\t"
          "ds_read_b128 %2, %8 offset:%12\n\tds_read_b128 %3, %9 offset:%12\n\tds_read_b128 %6, %10 offset:%13\n\tds_read_b128 %7, %11 offset:%13"
          : "=&v"(f.q[0]), "=&v"(f.q[1]), "=&v"(f.g[0]), "=&v"(f.g[1]), "=&v"(f.k[0][0]), "=&v"(f.k[0][1]), "=&v"(f.v[0][0]), "=&v"(f.v[0][1])
          : "v"(q0a), "v"(q1a), "v"(k0a), "v"(k1a), "n"(AREA_G), "n"(AREA_V - AREA_K)
          : "memory");
      asm volatile(
          "ds_read_b128 %0, %4 offset:%6\n\tds_read_b128 %1, %5 offset:%6\n\tds_read_b128 %2, %4 offset:%7\n\tds_read_b128 %3, %5 offset:%7"
          : "=&v"(f.k[1][0]), "=&v"(f.k[1][1]), "=&v"(f.v[1][0]), "=&v"(f.v[1][1])
          : "v"(k0a), "v"(k1a), "n"(4096), "n"(4096 + AREA_V - AREA_K)
          : "memory");
    };
    auto wait = [&] {
      asm volatile("s_waitcnt lgkmcnt(0)"
                   : "+v"(f.lse), "+v"(f.delta), "+v"(f.q[0]), "+v"(f.q[1]), "+v"(f.g[0]), "+v"(f.g[1]), "+v"(f.k[0][0]), "+v"(f.k[0][1]),
                     "+v"(f.v[0][0]), "+v"(f.v[0][1]), "+v"(f.k[1][0]), "+v"(f.k[1][1]), "+v"(f.v[1][0]), "+v"(f.v[1][1])
                   :
                   : "memory");
    };
    auto barrier = [] {
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
    };
    int at = 0;  // of row b
    W_VMCNT((PB_NST - 1) * LOADS);  // (whatever else is under way is younger or done)
    barrier();
    issue(0);
    wait();
    for (int b = bfirst; b < blast; ++b) {
      W_VMCNT((PB_NST - 2) * LOADS);  // this wavefront's part of row b + 1 has landed
      barrier();                   // ... everybody's; and everybody has read row b
      const Row far = row_of(b + PB_NST);
      const int here = at;
      at = at == (PB_NST - 1) * STAGE ? 0 : at + STAGE;
      const float nlse2 = -f.lse * LOG2E;
      f32x16 nd, s[2], t[2];
#pragma unroll
      for (int v = 0; v < 16; ++v) nd[v] = -f.delta;
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        s[c] = mfma(w_frag(f.k[c][0]), w_frag(f.q[0]), bz[c]);
        t[c] = mfma(w_frag(f.v[c][0]), w_frag(f.g[0]), nd);
        s[c] = mfma(w_frag(f.k[c][1]), w_frag(f.q[1]), s[c]);
        t[c] = mfma(w_frag(f.v[c][1]), w_frag(f.g[1]), t[c]);
      }
      __builtin_amdgcn_sched_barrier(0);
      issue(at);  // (past the last row: of a buffer of zeros)
      // the loads of row b + PB_NST, which takes row b's buffer, one by one: a compute unit takes one in 16 cycles or more
#pragma unroll
      for (int x = 0; x < 8; ++x) {
#pragma unroll
        for (int i = x * LOADS / 8; i < (x + 1) * LOADS / 8; ++i) load(here, far, i);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int v = 4 * (x & 3); v < 4 * (x & 3) + 4; ++v) {
          const int c = x >> 2;
          const float e = fast_exp2(fmaf(s[c][v], c1, nlse2));
          const float sum = __builtin_fmaf(e, t[c][v], acc[c][v]);
          // (a masked pair's exponential has no bound: its logit is not part of the LSE)
          acc[c][v] = CAUSAL && k0 + 32 * c + key_of(v, hl) > q ? acc[c][v] : sum;
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      wait();
    }
    W_VMCNT(0);  // nothing may still be on its way into LDS when the work-group ends
  }
  if (q < p.S && !(skip && resume)) {
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int kb = k0 + 32 * c + 8 * g + 4 * hl;
        if (kb + 3 < p.S) *(f32x4_any*)(dst + kb) = f32x4{acc[c][4 * g], acc[c][4 * g + 1], acc[c][4 * g + 2], acc[c][4 * g + 3]};
        else for (int e = 0; e < 4; ++e) if (kb + e < p.S) dst[kb + e] = acc[c][4 * g + e];
      }
  }
}

}  // namespace

hipError_t launch_pair_dbias(const KP& p, hipStream_t st) {
  const int ng = p.sm_partial ? (p.b1 - 1) / p.sm_gw - p.b0 / p.sm_gw + 1 : 1;
  const dim3 g((p.S + PB_T - 1) / PB_T, (p.S + PB_T - 1) / PB_T, (p.h1 - p.h0) / 2 * ng);
  if (p.mask_kind == 1) dbias_pair_kernel<true><<<g, 256, 0, st>>>(p);
  else dbias_pair_kernel<false><<<g, 256, 0, st>>>(p);
  return hipGetLastError();
}

}  // namespace ssa

// Kernels of the co-sharded feed-forward operator: one bf16 MFMA GEMM with fused epilogues, and a
// fixed-order column sum for the bias gradients.
#include "ffn_kernels.h"

#include "ffn_common.h"

namespace ssa {
namespace {

constexpr int GBK = 32;  // contraction depth of one stage
// Work-group -> tile.  Work-groups go to the 8 XCDs round-robin in launch order and each XCD has its
// own L2: work-group b becomes logical index (b % 8) * (tiles / 8) + b / 8, so an XCD works on a
// contiguous range of logical indices, and logical indices walk the tile grid in bands of four
// tile rows, down the band's rows first: the tiles an XCD runs at a time share a few row panels of
// A and column panels of B.
struct TilePos { int mt, nt; };
__device__ inline TilePos tile_pos(int b, int mtiles, int ntiles) {
  const int tiles = mtiles * ntiles;
  const int xcd = b % 8, idx = b / 8;
  const int id = xcd * (tiles / 8) + min(xcd, tiles % 8) + idx;
  constexpr int BAND = 4;
  const int per_band = BAND * ntiles, band = id / per_band, in_band = id % per_band;
  const int rows = min(BAND, mtiles - band * BAND);
  TilePos t;
  t.mt = band * BAND + in_band % rows;
  t.nt = in_band / rows;
  return t;
}

typedef __attribute__((address_space(3))) void lds_void;
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

// One operand of a 16 KS deep contraction stage (KS = 16-wide contraction steps per stage), 64 F
// rows (of A) or columns (of B) -- "rho" below; F = 32-wide fragments per wavefront -- fetched from
// global memory straight into LDS, 16 bytes per lane, 1 KB per wavefront instruction, F KS / 2
// instructions per wavefront.  Bounds-checked buffer loads (the whole offset is the lane offset,
// the only part the hardware range-checks): everything outside the matrix lands as zeros.  The LDS
// image is swizzled at 16-byte granularity by choosing WHICH global chunk a lane fetches for its
// fixed LDS slot, so that the fragment reads below are free of bank conflicts:
//   TR = false (contraction index contiguous in memory): LDS row = rho, 32 KS bytes = 2 KS chunks;
//        chunk c of row rho sits at slot c ^ ((rho >> 2) & 3) (KS = 2), c ^ ((rho >> 1) & 7) (KS = 4)
//   TR = true  (rho contiguous in memory): LDS row = k, 128 F bytes = 8 F chunks; chunk c of row k
//        sits at slot c ^ (4 * (k & 3)) (F = 3: see swizzle)
// With KS = 2 a row of a contraction-contiguous operand is half a cache line per stage, and the
// compute unit's load path then moves whole lines for half the bytes: KS = 4 for such operands.
// place of 64-byte block `blk` of row k of a TR operand (k3 = k & 3), and back; three fragments (six blocks)
// rotate instead
template <int F>
__device__ inline int swizzle(int blk, int k3) { return (F & (F - 1)) == 0 ? blk ^ k3 : (blk + k3) % (2 * F); }
template <int F>
__device__ inline int unswizzle(int blk, int k3) { return (F & (F - 1)) == 0 ? blk ^ k3 : (blk + 2 * F - k3) % (2 * F); }

template <bool TR, int F, int KS>
struct Stager {
  static constexpr int BYTES = 2048 * F * KS, NI = F * KS / 2, BK = 16 * KS;
  const char* base;      // start of the next stage to fetch
  int64_t step;          // bytes from one stage to the next
  int left;              // bytes from `base` to the end of the matrix (meaningful while k0 < kend)
  int k0, kcur, kend;
  uint32_t lane_off[NI]; // lane offset of instruction t inside a stage (OUTSIDE if its rho are not in the matrix)
  int klimit[2];         // !TR: the lane's chunk (even / odd instruction) is inside the contraction range while k0 <= klimit
  __amdgpu_buffer_rsrc_t rs;
  __device__ void init(const uint16_t* base_, int64_t ld, int rho_tot, int ktot_, int rho0, int lane, int w) {
    base = (const char*)base_;
    const uint32_t ld2 = (uint32_t)ld * 2u;
    kend = ktot_;
    k0 = kcur = 0;
    klimit[0] = klimit[1] = 0;
    if (!TR) {
      constexpr int CPR = 2 * KS, RPI = 64 / CPR;  // chunks per LDS row, rows per instruction
      step = 2 * BK;
      left = (int)(((int64_t)(rho_tot - 1) * ld + ktot_) * 2);
#pragma unroll
      for (int t = 0; t < NI; ++t) {
        const int row = RPI * (w * NI + t) + lane / CPR;
        const int c = (lane % CPR) ^ (KS == 2 ? (row >> 2) & 3 : (row >> 1) & 7);
        lane_off[t] = (uint32_t)(rho0 + row) * ld2 + 16u * c;
        if (t < 2) klimit[t] = ktot_ - 8 * c - 8;  // the chunk depends on the parity of t only
      }
    } else {
      constexpr int LPR = 8 * F;  // 16-byte chunks per LDS row
      step = (int64_t)BK * ld * 2;
      left = (int)(((int64_t)(ktot_ - 1) * ld + rho_tot) * 2);
#pragma unroll
      for (int t = 0; t < NI; ++t) {
        const int slot = 64 * (w * NI + t) + lane, krow = slot / LPR, s = slot % LPR;
        const int c = 4 * unswizzle<F>(s >> 2, krow & 3) + (s & 3);
        lane_off[t] = rho0 + 8 * c + 8 <= rho_tot ? (uint32_t)krow * ld2 + (uint32_t)(rho0 + 8 * c) * 2u : OUTSIDE;
      }
    }
  }
  // start at stage s0 and stop before stage s1
  __device__ void range(int s0, int s1) {
    base += s0 * step;
    left -= (int)(s0 * step);
    k0 = s0 * BK;
    kend = min(kend, s1 * BK);
  }
  // Scalar work once per stage, stages in ascending order: a descriptor that starts at the stage's
  // first contraction index and ends with the matrix, so the lane offsets are the same for every
  // stage, and is empty for stages past the end of the contraction (they load zeros).
  __device__ void begin_stage() {
    rs = __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, k0 < kend ? left : 0, 0x00020000);
    kcur = k0;
    base += step;
    left -= (int)step;
    k0 += BK;
  }
  // instruction t (0..NI-1) of the stage -> LDS at `dst` (this operand's part of a stage buffer)
  __device__ void issue(char* dst, int w, int t) const {
    const bool ok = TR || kcur <= klimit[t & 1];
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void*)(dst + (w * NI + t) * 1024), 16, ok ? lane_off[t] : OUTSIDE, 0, 0, 0);
  }
};

// Fragment addresses of one operand for one wavefront (`wr` = which half of the tile's rho).
// A fragment is 32 rho x 16 k, lane (r = lane % 32, hl = lane / 32) holding rho = r, k = 8 hl .. 8 hl + 7.
template <bool TR, int F, int KS>
struct FragReader {
  uint32_t a0;
  uint32_t blk[TR ? F : 1];
  __device__ void init(int lane, int wr) {
    const int r = lane & 31, hl = lane >> 5;
    if (!TR) {
      const int sw = KS == 2 ? (r >> 2) & 3 : (r >> 1) & 7;
      a0 = (uint32_t)(32 * F * wr + r) * (32u * KS) + (uint32_t)((hl ^ sw) << 4);
      blk[0] = 0;
    } else {
      const int i = lane & 15, bk = lane >> 4, kk = 8 * (bk >> 1) + (i >> 2);
      a0 = (uint32_t)kk * (128u * F) + 32u * (bk & 1) + 8u * (i & 3);
#pragma unroll
      for (int f = 0; f < F; ++f) blk[f] = (uint32_t)swizzle<F>(F * wr + f, (i >> 2) & 3) << 6;
    }
  }
  // fragment f (rho = 32 F wr + 32 f ..) of contraction step ks of the stage at `op`
  __device__ bf16x8 read(const char* op, int f, int ks) const {
    if (!TR) {
      return *(const bf16x8*)(op + ((a0 ^ (uint32_t)(ks << 5)) + (uint32_t)f * (1024u * KS)));
    } else {
      const char* p = op + (a0 + blk[f] + (uint32_t)ks * (2048u * F));
      union { s16x4 h[2]; bf16x8 v; } o;
      o.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)p);
      o.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p + 512 * F));
      return o.v;
    }
  }
};

// slot of item `i` when `n` items are dealt out evenly over `slots` slots; how many come before `slot`
constexpr int slot_of(int i, int n, int slots) { return i * slots / n; }
constexpr int items_before(int slot, int n, int slots) {
  int c = 0;
  for (int i = 0; i < n; ++i) c += slot_of(i, n, slots) < slot ? 1 : 0;
  return c;
}

// ---------------------------------------------------------------------------
// C[M,N] = A B with bf16 operands and fp32 accumulation on v_mfma_f32_32x32x16_bf16.
//   AT = false: A[m][k] at A + m*lda + k      AT = true: A[k][m] at A + k*lda + m
//   BT = false: B[k][n] at B + k*ldb + n      BT = true: B[n][k] at B + n*ldb + k
// Four wavefronts, 2 x 2, each with 32 FI x 32 FJ of the result in accumulation registers; a stage
// is KS contraction steps of 16 deep; NS stage buffers form a ring:
//   FI = 4, FJ = 2, KS = 2, NS = 3: 256 x 128 tile, 72 KB of LDS and 128 accumulation registers:
//        two work-groups per compute unit, which overlap each other's prologue, epilogue and
//        barriers.  For products whose operands are both read transposed.
//   FI = 4, FJ = 2, KS = 4, NS = 3: 144 KB of LDS, one work-group per compute unit, half as many
//        barriers per MFMA.  For products with a contraction-contiguous operand (see Stager).
//   FI = FJ = 2, KS = 4, NS = 3: 128 x 128 tile, for products with few tiles; the contraction may be cut into
//        g.split parts (gemm_plan_tiled).  Forward of 127 tokens x 12288 x 6144: 185 -> 92 us.
//   FI = 1, FJ = 2, KS = 4, NS = 5: 64 x 128 tile, for few rows of A and a B too large for the few-rows kernel: bound by what a compute unit
//        has under way, 64 KB of B (three buffers of 128 x 128: 32).  Forward of 16 tokens x 12288 x 6144 (302 MB of weights): 75.3 -> 68.2 us, 4.4 TB/s;
//        64 81.5 -> 77.6, 50 x 12288 x 2000 45.1 -> 40.8.  Not better: three buffers, two work-groups and twice the parts (73.6); 128 x 128
//        with four buffers for every product (71.2, and 700 x 1600 x 2400, a step, 159 -> 166: stages past the end of a part).
//   FI = 2, FJ = 3, KS = 4, NS = 3 and FI = 4, FJ = 3, KS = 2, NS = 4: 128 x 192 and 256 x 192 tiles, for
//        sizes of which the others leave the last round of work-groups nearly empty (gemm_shape).
// Stages travel global -> LDS directly, NS - 1 stages ahead of the multiplication, the load
// instructions spread evenly between the MFMAs (the compute unit's load path moves 64 bytes per
// cycle, of which the kernel needs 32 to 48), and one barrier per stage, issued with half a step of
// MFMAs still to go so the matrix cores keep busy across it.  Operands whose contraction index is
// not contiguous in memory are read from LDS with the transposed read.
// The matrix cores are fed B fragments as their row operand and A fragments as their column
// operand, so a lane ends up with one row m and runs of four consecutive columns n.
// The contraction runs in ascending k, 16 at a time, whatever the tile position or shape: with
// EPI_ACC the accumulator starts from the fp32 partial result of the previous chunks, so a sum
// cut into chunks at multiples of 16 is the same sum.
// ---------------------------------------------------------------------------
template <bool AT, bool BT, int EPI, int FI, int FJ, int KS, int NS>
__global__ __launch_bounds__(256, (FI * FJ <= 8 && KS == 2) ? 2 : 1) void gemm_kernel(GemmArgs g) {
  constexpr bool SPLIT = FI <= 2 && FJ == 2 && EPI != EPI_ACC;  // g.split parts
  constexpr int GBM = 64 * FI, GBN = 64 * FJ;
  using StageA = Stager<AT, FI, KS>;
  using StageB = Stager<!BT, FJ, KS>;
  constexpr int A_BYTES = StageA::BYTES, STAGE_BYTES = StageA::BYTES + StageB::BYTES;
  constexpr int NM = FI * FJ, SLOTS = KS * NM;             // MFMAs per contraction step / per stage
  constexpr int LA = StageA::NI, NL = LA + StageB::NI;     // loads per stage (per wavefront): A first
  constexpr int NR = FI + FJ;                              // fragment reads per step
  constexpr int BAR = SLOTS - NM / 2;                      // the barrier sits before this slot
  // the stage buffers are separate arrays: the compiler then knows that a load into one does not
  // feed a read of another, and does not wait for it
  __shared__ __attribute__((aligned(1024))) char stage0[STAGE_BYTES];
  __shared__ __attribute__((aligned(1024))) char stage1[STAGE_BYTES];
  __shared__ __attribute__((aligned(1024))) char stage2[STAGE_BYTES];
  __shared__ __attribute__((aligned(1024))) char stage3[NS >= 4 ? STAGE_BYTES : 16];
  __shared__ __attribute__((aligned(1024))) char stage4[NS >= 5 ? STAGE_BYTES : 16];
  const int tid = threadIdx.x, lane = tid & 63, r = lane & 31, hl = lane >> 5;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = w >> 1, wn = w & 1;
  const int mtiles = (g.M + GBM - 1) / GBM, ntiles = (g.N + GBN - 1) / GBN;
  const int tiles = mtiles * ntiles;
  const int tile = SPLIT ? (int)blockIdx.x % tiles : (int)blockIdx.x;
  const TilePos tp = tile_pos(tile, mtiles, ntiles);
  const int m0 = tp.mt * GBM, n0 = tp.nt * GBN;

  StageA sa;
  StageB sb;
  FragReader<AT, FI, KS> ra;
  FragReader<!BT, FJ, KS> rb;
  ra.init(lane, wm);
  rb.init(lane, wn);

  // acc[j][i]: row m0 + 32 FI wm + 32 i + r, columns n0 + 32 FJ wn + 32 j + key_of(v, hl).
  // The fp32 partial result between chunks lives in the workspace in the order the registers hold
  // it (tile, wavefront, (j, i, quad), lane): 1 KB per wavefront instruction, fully coalesced.
  f32x16 acc[FJ][FI];
  f32x4* frag32 = nullptr;
  if (EPI == EPI_ACC) frag32 = (f32x4*)g.acc32 + ((int64_t)(tp.mt * ntiles + tp.nt) * 4 + w) * (NM * 4 * 64) + lane;

  const int nk = (g.K + 16 * KS - 1) / (16 * KS);
  // Column sums of B (the bias gradients: B is dY or dZ, on its way through the registers anyway), by the
  // wavefronts of the first tile row: packed pairs against (1, 1), two instructions per MFMA and under it.
  // A kernel of their own read B once more (8192 tokens x 12288: 59 us).  The sums of each turn of the ring are
  // added up apart: chains of 24 to 48 additions and one of K / 192 to K / 96, not one of K / 4.
  constexpr bool SUMS = EPI == EPI_STORE;
  const bf16x2 ones2 = {(__bf16)1.f, (__bf16)1.f};
  const bool sums = SUMS && g.colsum && m0 == 0 && wm == 0;
  float csum[SUMS ? FJ : 1], turn[SUMS ? FJ : 1];
  if (SUMS) {
#pragma unroll
    for (int j = 0; j < FJ; ++j) csum[SUMS ? j : 0] = turn[SUMS ? j : 0] = 0.f;
  }
  bf16x8 fa[2][FI], fb[2][FJ];  // fragments of the contraction step being multiplied and of the next one
  // fragment reads of one contraction step in the order of their first use: B 0, A 0 .. FI-1, B 1 .. FJ-1
  auto read_item = [&](const char* st, int item, int ks, int set) {
    if (item == 0) fb[set][0] = rb.read(st + A_BYTES, 0, ks);
    else if (item <= FI) fa[set][item - 1] = ra.read(st, item - 1, ks);
    else fb[set][item - FI] = rb.read(st + A_BYTES, item - FI, ks);
  };
  // One stage: multiply `cur` (the fragments of its first step are in registers), fetch the stage
  // NS - 1 ahead into `ldst` (the buffer of the stage before `cur`, free since the last barrier),
  // and, once the stage after `cur` has landed for every wavefront, read the fragments of its
  // first step from `nxt`.  KS NM slots of one MFMA each; the other instructions are dealt out over
  // the slots (loads evenly over the stage, the fragments of the next step over a step, in the
  // order of their first use) and the scheduler is told to keep every slot together: the matrix
  // cores stall as soon as the instructions between two MFMAs take longer to issue than one MFMA
  // takes to run.
  auto stage = [&](auto with_sums, const char* cur, const char* nxt, char* ldst) __attribute__((always_inline)) {
    sa.begin_stage();
    sb.begin_stage();
#pragma unroll
    for (int s = 0; s < SLOTS; ++s) {
      const int ks = s / NM, x = s % NM, j = x / FI, i = x % FI;
      if (s == BAR) {
        // all but the youngest loads are done: the next stage is in LDS (this wavefront's part), and
        // so are this wavefront's reads of `cur`.  A bare barrier: __syncthreads() would wait for
        // every load in flight.
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((NS - 3) * NL + items_before(BAR, NL, SLOTS)) : "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
      }
      acc[j][i] = mfma(fb[ks & 1][j], fa[ks & 1][i], acc[j][i]);
      if (decltype(with_sums)::value && i == FI - 1) {
        if (wm == 0) {
          union { bf16x8 v; bf16x2 h[4]; } b;
          b.v = fb[ks & 1][j];
#pragma unroll
          for (int e = 0; e < 4; ++e) turn[SUMS ? j : 0] = __builtin_amdgcn_fdot2_f32_bf16(b.h[e], ones2, turn[SUMS ? j : 0], false);
        }
      }
#pragma unroll
      for (int l = 0; l < NL; ++l)
        if (s == slot_of(l, NL, SLOTS)) {
          if (l < LA) sa.issue(ldst, w, l);
          else sb.issue(ldst + A_BYTES, w, l - LA);
        }
      if (ks + 1 < KS) {  // fragments of the next step of this stage
#pragma unroll
        for (int item = 0; item < NR; ++item)
          if (x == 1 + slot_of(item, NR, NM - 2)) read_item(cur, item, ks + 1, (ks + 1) & 1);
      } else if (s >= BAR) {  // fragments of the first step of the next stage
#pragma unroll
        for (int item = 0; item < NR; ++item)
          if (s - BAR == slot_of(item, NR, NM / 2)) read_item(nxt, item, 0, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  auto fetch_all = [&](char* dst) {
    sa.begin_stage();
    sb.begin_stage();
#pragma unroll
    for (int t = 0; t < LA; ++t) sa.issue(dst, w, t);
#pragma unroll
    for (int t = 0; t < NL - LA; ++t) sb.issue(dst + A_BYTES, w, t);
  };
  const int parts = SPLIT ? g.split : 1;
  const bool alone = SPLIT && parts > 1 && g.parts;  // one part per work-group; otherwise all of them in turn
  const int first = alone ? (int)blockIdx.x / tiles : 0, last = alone ? first + 1 : parts;
  f32x16 sum[SPLIT ? FJ : 1][SPLIT ? FI : 1];
  for (int part = first; part < last; ++part) {
    // stages s0 .. s1 - 1, their count rounded up to a multiple of the ring: stages past the end load zeros
    // and add nothing
    const int s0 = (int)((int64_t)nk * part / parts), s1 = (int)((int64_t)nk * (part + 1) / parts);
    sa.init(g.A, g.lda, g.M, g.K, m0, lane, w);
    sb.init(g.B, g.ldb, g.N, g.K, n0, lane, w);
    if (SPLIT) {
      sa.range(s0, s1);
      sb.range(s0, s1);
    }
    if (EPI == EPI_ACC && g.accumulate) {
#pragma unroll
      for (int j = 0; j < FJ; ++j)
#pragma unroll
        for (int i = 0; i < FI; ++i)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const f32x4 v = frag32[((j * FI + i) * 4 + q) * 64];
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[j][i][4 * q + e] = v[e];
          }
    } else {
#pragma unroll
      for (int j = 0; j < FJ; ++j)
#pragma unroll
        for (int i = 0; i < FI; ++i)
#pragma unroll
          for (int v = 0; v < 16; ++v) acc[j][i][v] = 0.f;
    }
    fetch_all(stage0);
    fetch_all(stage1);
    if (NS >= 4) fetch_all(stage2);
    if (NS >= 5) fetch_all(stage3);
    if constexpr (EPI == EPI_ACC16 && FJ != 3 && FI != 1) {  // (these tiles do not continue sums)
     if (g.accumulate && part == 0) {
      // The partial sum of the earlier chunks is the output itself (bf16): read as whole rows (64 FJ
      // contiguous bytes per row), widened, and turned into the register layout through a piece of
      // LDS of the wavefront's own -- the epilogue's path backwards.  The pieces lie in the last stage
      // buffer, which no load targets before the barrier that ends the prologue; 16-byte pieces are swizzled
      // by row, conflict-free both ways.
      constexpr int TLD = 128 * FJ, LPR = 8 * FJ, RPI = 64 / LPR;
      static_assert(4 * 32 * TLD <= STAGE_BYTES, "accumulator staging does not fit");
      char* tb = (NS == 4 ? stage3 : stage2) + w * (32 * TLD);
      const int c4 = 4 * (lane % LPR), rsub = lane / LPR;
      const int n = n0 + wn * 32 * FJ + c4;
#pragma unroll
      for (int i = 0; i < FI; ++i) {
#pragma unroll
        for (int it = 0; it < 32 / RPI; ++it) {
          const int row = RPI * it + rsub, m = m0 + wm * 32 * FI + 32 * i + row;
          float x[4] = {0.f, 0.f, 0.f, 0.f};
          if (m < g.M && n < g.N) unpack4(*(const uint2*)(g.out + (int64_t)m * g.ldo + n), x);
          *(f32x4*)(tb + row * TLD + ((c4 * 4) ^ ((row & 15) << 4))) = f32x4{x[0], x[1], x[2], x[3]};
        }
#pragma unroll
        for (int j = 0; j < FJ; ++j)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const f32x4 v = *(const f32x4*)(tb + r * TLD + (((32 * j + 8 * q + 4 * hl) * 4) ^ ((r & 15) << 4)));
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[j][i][4 * q + e] = v[e];
          }
      }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
     }
    }
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NS - 2) * NL) : "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
#pragma unroll
    for (int item = 0; item < NR; ++item) read_item(stage0, item, 0, 0);
    bool plain = true;
    if constexpr (SUMS) {
      if (g.colsum && m0 == 0) {
        plain = false;
        for (int kt = s0; kt < s1; kt += NS) {
          if (NS == 4) {
            stage(std::true_type{}, stage0, stage1, stage3);
            stage(std::true_type{}, stage1, stage2, stage0);
            stage(std::true_type{}, stage2, stage3, stage1);
            stage(std::true_type{}, stage3, stage0, stage2);
          } else {
            stage(std::true_type{}, stage0, stage1, stage2);
            stage(std::true_type{}, stage1, stage2, stage0);
            stage(std::true_type{}, stage2, stage0, stage1);
          }
#pragma unroll
          for (int j = 0; j < FJ; ++j) {
            csum[SUMS ? j : 0] += turn[SUMS ? j : 0];
            turn[SUMS ? j : 0] = 0.f;
          }
        }
      }
    }
    if (plain) {
      for (int kt = s0; kt < s1; kt += NS) {
        if (NS == 5) {
          stage(std::false_type{}, stage0, stage1, stage4);
          stage(std::false_type{}, stage1, stage2, stage0);
          stage(std::false_type{}, stage2, stage3, stage1);
          stage(std::false_type{}, stage3, stage4, stage2);
          stage(std::false_type{}, stage4, stage0, stage3);
        } else if (NS == 4) {
          stage(std::false_type{}, stage0, stage1, stage3);
          stage(std::false_type{}, stage1, stage2, stage0);
          stage(std::false_type{}, stage2, stage3, stage1);
          stage(std::false_type{}, stage3, stage0, stage2);
        } else {
          stage(std::false_type{}, stage0, stage1, stage2);
          stage(std::false_type{}, stage1, stage2, stage0);
          stage(std::false_type{}, stage2, stage0, stage1);
        }
      }
    }
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    if constexpr (SPLIT) {
      if (last - first > 1) {
        __builtin_amdgcn_s_barrier();  // everybody has left the stage buffers
        asm volatile("" ::: "memory");
#pragma unroll
        for (int j = 0; j < FJ; ++j)
#pragma unroll
          for (int i = 0; i < FI; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) sum[j][i][v] = part == first ? acc[j][i][v] : sum[j][i][v] + acc[j][i][v];
      }
    }
  }
  if (sums) {
#pragma unroll
    for (int j = 0; j < FJ; ++j) {
      const float t = half_sum(csum[SUMS ? j : 0]);
      const int n = n0 + wn * 32 * FJ + 32 * j + r;
      if (hl == 0 && n < g.N) g.colsum[n] = f2bf(t);
    }
  }
  if constexpr (SPLIT) {
    if (alone) {
      // Partial sums go to the scratch in the order the registers hold them; the work-group that finishes
      // a tile last adds them in the order of the parts (so the result does not depend on who that is)
      // and runs the epilogue.  Blocks of 32 rows past the end of the matrix are left out.  The sums
      // are stored and loaded at device scope (past the L2s, which the XCDs do not share), so no fence
      // has to write a whole L2 back: with fences a product of 16 x 1624 x 1760 took 25 us.
      __shared__ int is_last;
      const __amdgpu_buffer_rsrc_t rp = __builtin_amdgcn_make_buffer_rsrc(
          (char*)g.parts + (int64_t)tile * parts * (NM * 16384), 0, parts * (NM * 16384), 0x00020000);
      const int at = (w * (NM * 4 * 64) + lane) * 16;
#pragma unroll
      for (int i = 0; i < FI; ++i)
        if (m0 + wm * 32 * FI + 32 * i < g.M)
#pragma unroll
          for (int j = 0; j < FJ; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              union { f32x4 f; u32x4 u; } v;
              v.f = f32x4{acc[j][i][4 * q], acc[j][i][4 * q + 1], acc[j][i][4 * q + 2], acc[j][i][4 * q + 3]};
              __builtin_amdgcn_raw_buffer_store_b128(v.u, rp, at + ((j * FI + i) * 4 + q) * 1024, first * (NM * 16384), DEVICE_SCOPE);
            }
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // in memory, before the barrier that the count follows
      __syncthreads();
      if (tid == 0) {
        is_last = __hip_atomic_fetch_add(g.counters + tile, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (unsigned)parts - 1u;
        if (is_last) __hip_atomic_store(g.counters + tile, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // nobody else comes
      }
      __syncthreads();
      if (!is_last) return;
#pragma unroll
      for (int i = 0; i < FI; ++i)
        if (m0 + wm * 32 * FI + 32 * i < g.M)
          for (int part = 0; part < parts; part += 4) {  // the loads of four parts at a time (past the last: zeros)
            union { u32x4 u; f32x4 f; } v[4][FJ][4];
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
              for (int j = 0; j < FJ; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                  v[u][j][q].u = __builtin_amdgcn_raw_buffer_load_b128(
                      rp, at + ((part + u) * NM * 16 + (j * FI + i) * 4 + q) * 1024, 0, DEVICE_SCOPE);
#pragma unroll
            for (int u = 0; u < 4; ++u)
              if (part + u < parts)
#pragma unroll
                for (int j = 0; j < FJ; ++j)
#pragma unroll
                  for (int q = 0; q < 4; ++q)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                      acc[j][i][4 * q + e] = part + u ? acc[j][i][4 * q + e] + v[u][j][q].f[e] : v[u][j][q].f[e];
          }
    } else if (parts > 1) {
#pragma unroll
      for (int j = 0; j < FJ; ++j)
#pragma unroll
        for (int i = 0; i < FI; ++i) acc[j][i] = sum[j][i];
    }
  }

  if (EPI == EPI_ACC && !g.last) {
#pragma unroll
    for (int j = 0; j < FJ; ++j)
#pragma unroll
      for (int i = 0; i < FI; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          frag32[((j * FI + i) * 4 + q) * 64] =
              f32x4{acc[j][i][4 * q], acc[j][i][4 * q + 1], acc[j][i][4 * q + 2], acc[j][i][4 * q + 3]};
  } else {
    // Epilogue through LDS, one 32-row block of the wavefront's part at a time: the registers hold
    // one row and scattered column quads per lane; written to a piece of stage buffer of the
    // wavefront's own (rows padded by 16 bytes: conflict-free both ways) and read back as whole
    // rows, 8 FJ lanes x 4 columns, so that every global access of the epilogue is 64 FJ
    // contiguous bytes per row.  Everybody's loads have landed and everybody has left the main loop
    // before a buffer is reused.
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    constexpr int TLD = 128 * FJ + 16, LPR = 8 * FJ;
    constexpr int CY = FJ == 3 ? 3 : 1, RPC = 64 * CY / LPR;  // passes of 64 lanes until the columns repeat, rows they cover
    static_assert(32 * TLD <= (NS >= 4 ? STAGE_BYTES : STAGE_BYTES / 2), "epilogue staging does not fit");
    char* tb = NS >= 4 ? (w == 0 ? stage0 : w == 1 ? stage1 : w == 2 ? stage2 : stage3)
                       : (w == 0 ? stage0 : w == 1 ? stage1 : w == 2 ? stage2 : stage0 + STAGE_BYTES / 2);
    int col[CY], rsub[CY];
    float bias[CY][4];
#pragma unroll
    for (int y = 0; y < CY; ++y) {
      col[y] = 4 * ((64 * y + lane) % LPR);
      rsub[y] = (64 * y + lane) / LPR;
      const int n = n0 + wn * 32 * FJ + col[y];
      bias[y][0] = bias[y][1] = bias[y][2] = bias[y][3] = 0.f;
      if ((EPI == EPI_ACT || EPI == EPI_ACC || EPI == EPI_ACC16) && g.bias && n < g.N) unpack4(*(const uint2*)(g.bias + n), bias[y]);
    }
#pragma unroll
    for (int i = 0; i < FI; ++i) {
#pragma unroll
      for (int j = 0; j < FJ; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          *(f32x4*)(tb + r * TLD + (32 * j + 8 * q + 4 * hl) * 4) =
              f32x4{acc[j][i][4 * q], acc[j][i][4 * q + 1], acc[j][i][4 * q + 2], acc[j][i][4 * q + 3]};
#pragma unroll
      for (int it = 0; it < 32 / RPC * CY; ++it) {
        const int y = it % CY, row = RPC * (it / CY) + rsub[y], m = m0 + wm * 32 * FI + 32 * i + row, n = n0 + wn * 32 * FJ + col[y];
        const f32x4 v = *(const f32x4*)(tb + row * TLD + col[y] * 4);
        if (m >= g.M || n >= g.N) continue;
        float x[4] = {v[0] + bias[y][0], v[1] + bias[y][1], v[2] + bias[y][2], v[3] + bias[y][3]};
        uint16_t* orow = g.out + (int64_t)m * g.ldo + n;
        if (EPI == EPI_ACT) {
          float h[4], d[4];
          if (g.out2) {
            if (g.act == 0) relu_n<true>(x, h, d); else gelu_n<true>(x, h, d);
            *(uint2*)(g.out2 + (int64_t)m * g.ldo + n) = pack4(d);
          } else {
            if (g.act == 0) relu_n<false>(x, h, d); else gelu_n<false>(x, h, d);
          }
          *(uint2*)orow = pack4(h);
        } else if (EPI == EPI_MUL) {
          float mu[4];
          unpack4(*(const uint2*)(g.mul + (int64_t)m * g.ldm + n), mu);
#pragma unroll
          for (int e = 0; e < 4; ++e) x[e] *= mu[e];
          *(uint2*)orow = pack4(x);
        } else {
          *(uint2*)orow = pack4(x);
        }
      }
    }
  }
}

// out[n] = sum over m of A[m][n], fp32, fixed order: a work-group takes 64 columns; 32 row groups
// per column (rows g, g+32, .. summed in ascending order, 16-byte loads of 8 columns), then the 32
// partial sums in ascending g.  N is a multiple of 8 and A + n 16-byte aligned for n % 8 == 0.
__global__ __launch_bounds__(256) void colsum_kernel(const uint16_t* A, int64_t lda, int M, int N, uint16_t* out) {
  __shared__ float part[32][65];
  const int cl = threadIdx.x & 7, rg = threadIdx.x >> 3;
  const int n = blockIdx.x * 64 + cl * 8;
  float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (n < N) {
    const uint16_t* col = A + n;
#pragma unroll 4
    for (int m = rg; m < M; m += 32) {
      const u32x4 v = *(const u32x4*)(col + (int64_t)m * lda);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        s[2 * e] += __uint_as_float(v[e] << 16);
        s[2 * e + 1] += __uint_as_float(v[e] & 0xffff0000u);
      }
    }
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) part[rg][cl * 8 + e] = s[e];
  __syncthreads();
  const int c = threadIdx.x;
  if (c < 64 && blockIdx.x * 64 + c < N) {
    float t = part[0][c];
#pragma unroll
    for (int g = 1; g < 32; ++g) t += part[g][c];
    out[blockIdx.x * 64 + c] = f2bf(t);
  }
}

// Explicit instantiations: the host compiler emits the launch stub of the first implicit
// instantiation only.
#define SS_GEMM_INST(a, b, e, fi, fj, ks) template __global__ void gemm_kernel<a, b, e, fi, fj, ks, fi * fj == 2 ? 5 : fi * fj <= 8 ? 3 : 4>(GemmArgs);
SS_GEMM_INST(false, false, 0, 4, 2, 4) SS_GEMM_INST(false, false, 2, 4, 2, 4) SS_GEMM_INST(false, false, 4, 4, 2, 4)
SS_GEMM_INST(false, true, 1, 4, 2, 4) SS_GEMM_INST(false, true, 2, 4, 2, 4) SS_GEMM_INST(false, true, 4, 4, 2, 4)
SS_GEMM_INST(true, false, 3, 4, 2, 2)
SS_GEMM_INST(false, false, 0, 2, 3, 4) SS_GEMM_INST(false, false, 4, 2, 3, 4) SS_GEMM_INST(false, true, 1, 2, 3, 4) SS_GEMM_INST(false, true, 4, 2, 3, 4) SS_GEMM_INST(true, false, 3, 2, 3, 4) 
SS_GEMM_INST(false, false, 0, 4, 3, 2) SS_GEMM_INST(false, false, 4, 4, 3, 2) SS_GEMM_INST(false, true, 1, 4, 3, 2) SS_GEMM_INST(false, true, 4, 4, 3, 2) SS_GEMM_INST(true, false, 3, 4, 3, 2) 

// 128 x 128 tiles for products with few of the large ones
SS_GEMM_INST(false, false, 0, 2, 2, 4) SS_GEMM_INST(false, false, 2, 2, 2, 4) SS_GEMM_INST(false, false, 4, 2, 2, 4)
SS_GEMM_INST(false, true, 1, 2, 2, 4) SS_GEMM_INST(false, true, 2, 2, 2, 4) SS_GEMM_INST(false, true, 4, 2, 2, 4)
SS_GEMM_INST(true, false, 3, 2, 2, 4)
// 64 x 128 for few rows of A and a large B
SS_GEMM_INST(false, false, 0, 1, 2, 4) SS_GEMM_INST(false, false, 4, 1, 2, 4)
#undef SS_GEMM_INST

template <bool AT, bool BT, int EPI, int FI, int FJ, int KS>
hipError_t launch_one(const GemmArgs& g, hipStream_t st) {
  const int tiles = ((g.M + 64 * FI - 1) / (64 * FI)) * ((g.N + 64 * FJ - 1) / (64 * FJ));
  const bool split = FI <= 2 && EPI != EPI_ACC && g.split > 1 && g.parts;
  gemm_kernel<AT, BT, EPI, FI, FJ, KS, FI * FJ == 2 ? 5 : FI * FJ <= 8 ? 3 : 4><<<split ? tiles * g.split : tiles, 256, 0, st>>>(g);
  return hipGetLastError();
}

template <bool AT, bool BT, int EPI>
hipError_t launch_shape(const GemmArgs& g, hipStream_t st) {
  const bool narrow = g.narrow || EPI == EPI_ACC || (EPI == EPI_ACC16 && g.accumulate);
  const GemmTile t = gemm_shape(g.M, g.N, g.K, g.split, narrow).tile;
  // few rows of A: the tile that has most of B under way (see gemm_kernel); the same bits
  if constexpr (!AT && !BT && EPI != EPI_ACC)
    if (t == TILE_128x128 && g.M <= 64 && !(EPI == EPI_ACC16 && g.accumulate)) return launch_one<AT, BT, EPI, 1, 2, 4>(g, st);
  if (t == TILE_128x128) return launch_one<AT, BT, EPI, 2, 2, 4>(g, st);
  if (t == TILE_256x128) return launch_one<AT, BT, EPI, 4, 2, AT ? 2 : 4>(g, st);
  if constexpr (EPI != EPI_ACC) return t == TILE_128x192 ? launch_one<AT, BT, EPI, 2, 3, 4>(g, st) : launch_one<AT, BT, EPI, 4, 3, 2>(g, st);
  return hipErrorInvalidValue;
}

}  // namespace

size_t gemm_acc_bytes(int M, int N) {
  // whole tiles; no tile is larger than 256 x 256
  return (size_t)((M + 255) / 256) * ((N + 255) / 256) * 256 * 256 * sizeof(float);
}

hipError_t launch_gemm(const GemmArgs& args, bool at, bool bt, int epi, hipStream_t st) {
  if (args.M <= 0 || args.N <= 0 || args.K <= 0) return hipErrorInvalidValue;
  GemmArgs g = args;
  if (g.split < 1) g.split = 1;
  // each operand layout comes with the epilogues that the feed-forward operator has for it
  if (!at && !bt) {
    if (g.cols) return launch_skinny(g, epi, st);
    switch (epi) {
      case EPI_ACT: return launch_shape<false, false, EPI_ACT>(g, st);
      case EPI_ACC: return launch_shape<false, false, EPI_ACC>(g, st);
      case EPI_ACC16: return launch_shape<false, false, EPI_ACC16>(g, st);
    }
  } else if (!at && bt) {
    switch (epi) {
      case EPI_MUL: return launch_shape<false, true, EPI_MUL>(g, st);
      case EPI_ACC: return launch_shape<false, true, EPI_ACC>(g, st);
      case EPI_ACC16: return launch_shape<false, true, EPI_ACC16>(g, st);
    }
  } else if (at && !bt && epi == EPI_STORE) {
    return launch_shape<true, false, EPI_STORE>(g, st);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_colsum(const void* A, int64_t lda, int M, int N, void* out, hipStream_t st) {
  colsum_kernel<<<(N + 63) / 64, 256, 0, st>>>((const uint16_t*)A, lda, M, N, (uint16_t*)out);
  return hipGetLastError();
}

}  // namespace ssa

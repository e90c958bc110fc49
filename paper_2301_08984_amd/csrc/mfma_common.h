// Shared device helpers of the MFMA kernels (gfx950).
//
// MFMA v_mfma_f32_32x32x16_bf16 layouts (lane l, r = l%32, hl = l/32):
//   A[m][k]: lane holds m = r,  k = 8*hl + 0..7      B[k][n]: lane holds n = r, k = 8*hl + 0..7
//   C[m][n]: lane holds n = r,  register v holds m = 8*(v/4) + 4*hl + v%4
// An accumulator block is reused as the B operand of the next product with its
// registers 8t..8t+7 as the eight k-slots; the matching A operand is read from a
// row-major LDS tile with ds_read_b64_tr_b16 (transpose read) in the same row order.
#pragma once
#include "kparams.h"

#include <type_traits>

namespace ssa {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(4))) float f32x4;

constexpr float LOG2E = 1.4426950408889634f;
constexpr float LN2 = 0.6931471805599453f;
constexpr int BN = 64;            // rows of a staged LDS tile
constexpr int MAX_RELPOS_S = 256;
constexpr int MAX_RELPOS_R = 1024;

__device__ inline float bf2f(uint16_t u) { return __uint_as_float(((uint32_t)u) << 16); }
// Round to nearest even in hardware (v_cvt_pk_bf16_f32): one instruction for two values.  With integer arithmetic it
// took four for one, which in the epilogues of short rows was a fifth of a kernel's vector instructions.
__device__ inline uint16_t f2bf(float f) {
  union { __bf16 b; uint16_t u; } o;
  o.b = (__bf16)f;
  return o.u;
}
__device__ inline uint32_t pack2_bf16(float lo, float hi) {
  union { bf16x2 v; uint32_t u; } o;
  o.v[0] = (__bf16)lo;
  o.v[1] = (__bf16)hi;
  return o.u;
}
// A uniform factor of the inner loops, in a vector register.  A vector instruction on vector registers and literals issues
// in 2.3 - 3.4 cycles per wavefront (fma, mul, add, and), one that reads a scalar register in 4.2; the compiler prefers
// the scalar register.
__device__ inline float in_vgpr(float x) {
  asm("" : "+v"(x));
  return x;
}
__device__ inline float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }  // v_exp_f32
// v_rcp_f32 (1 ulp): the gate 1 / (1 + e^-g) is rounded to bf16 right after, and a full division
// costs ten instructions per element
__device__ inline float fast_rcp(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ inline float half_max(float x) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ inline float half_sum(float x) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
// Stores one row of 32 bf16 columns held as "lane = row, group g = columns 8g + 4*hl .. +3" (the
// layout of a 32x32 accumulator block, packed to 8 bytes per group): the two half-waves exchange
// pieces so that every lane writes 16 contiguous bytes twice (columns 8*(2j + hl) .. +7) instead of
// 8 bytes four times, which halves the cache-line lookups of the store.  Both lanes of a row (l and
// l + 32) must be active; `live` masks the stores only.
__device__ inline void store_row32(uint16_t* row_ptr, const uint2 (&a)[4], int hl, bool live) {
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    auto s = __builtin_amdgcn_permlane32_swap(a[2 * j].x, a[2 * j + 1].x, false, false);
    auto t = __builtin_amdgcn_permlane32_swap(a[2 * j].y, a[2 * j + 1].y, false, false);
    if (live) *(u32x4*)(row_ptr + 8 * (2 * j + hl)) = u32x4{s[0], t[0], s[1], t[1]};
  }
}
// four scaled values as packed bf16
__device__ inline uint2 pack4_bf16(float a, float b, float c, float d, float s) {
  uint2 o;
  o.x = pack2_bf16(a * s, b * s);
  o.y = pack2_bf16(c * s, d * s);
  return o;
}
// The matching load: every lane fetches 16 contiguous bytes twice and the half-waves exchange pieces,
// so that a[g] ends up holding columns 8g + 4*hl .. +3 of the lane's row.  Both lanes of a row (l and
// l + 32) must be active.
__device__ inline void load_row32(const uint16_t* row_ptr, uint2 (&a)[4], int hl) {
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const u32x4 v = *(const u32x4*)(row_ptr + 8 * (2 * j + hl));
    auto s = __builtin_amdgcn_permlane32_swap(v[0], v[2], false, false);
    auto t = __builtin_amdgcn_permlane32_swap(v[1], v[3], false, false);
    a[2 * j].x = s[0]; a[2 * j].y = t[0];
    a[2 * j + 1].x = s[1]; a[2 * j + 1].y = t[1];
  }
}
// in four sums: a single one would be a chain of dependent additions
__device__ inline float sum16(const float (&x)[16]) {
  float s[4] = {x[0], x[1], x[2], x[3]};
#pragma unroll
  for (int v = 4; v < 16; ++v) s[v & 3] += x[v];
  return (s[0] + s[1]) + (s[2] + s[3]);
}
// A value as the sum of three bf16 (exact: 24 bits), packed for contraction indexes 0 to 2 of a matrix instruction: with
// `three_ones` as the other operand it adds the value to a whole row or column of an accumulator block, which costs one
// matrix instruction instead of sixteen subtractions where the vector instructions are the scarcer ones.
__device__ inline uint2 split3(float x) {
  const float hi = (float)(__bf16)x, r = x - hi, mid = (float)(__bf16)r;
  return uint2{pack2_bf16(hi, mid), pack2_bf16(r - mid, 0.f)};
}
__device__ inline bf16x8 split3_operand(uint2 s) {
  union { u32x4 u; bf16x8 v; } o;
  o.u = u32x4{s.x, s.y, 0, 0};
  return o.v;
}
__device__ inline bf16x8 three_ones(int hl) {  // zeros for the half-wave of indexes 8 to 15
  union { u32x4 u; bf16x8 v; } o;
  o.u = u32x4{hl ? 0u : 0x3f803f80u, hl ? 0u : 0x3f80u, 0, 0};
  return o.v;
}
// continues a sum over packed operands as they were rounded
__device__ __forceinline__ float sum_rounded(bf16x8 x, float sum) {
  union { uint32_t u; bf16x2 v; } ones;
  ones.u = 0x3f803f80u;
  union { bf16x8 v; bf16x2 h[4]; } o;
  o.v = x;
#pragma unroll
  for (int e = 0; e < 4; ++e) sum = __builtin_amdgcn_fdot2_f32_bf16(o.h[e], ones.v, sum, false);
  return sum;
}
__device__ inline f32x16 mfma(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
__device__ inline bf16x8 zero8() {
  union { u32x4 u; bf16x8 v; } z;
  z.u = u32x4{0, 0, 0, 0};
  return z.v;
}
// eight fp32 -> one bf16x8 operand (round to nearest even)
__device__ inline bf16x8 pack8(const float* x) {
  bf16x8 o;
#pragma unroll
  for (int e = 0; e < 8; ++e) o[e] = (__bf16)x[e];
  return o;
}

// Row-major bf16 tile in LDS, `LD` elements per row.
// natural operand: row = r, eight consecutive columns starting at 16*ks + 8*hl
template <int LD>
__device__ inline bf16x8 lds_nat(const uint16_t* t, int row, int ks, int hl) {
  return *(const bf16x8*)(t + row * LD + 16 * ks + 8 * hl);
}
// transposed operand for the product whose k-slots are accumulator registers 8t..8t+7 of a
// 32-row block: lane gets column (cbase + l%32) of rows rbase + {0..3, 8..11} + 4*hl
template <int LD>
__device__ inline bf16x8 lds_tr(const uint16_t* t, int rbase, int cbase, int lane) {
  const int i = lane & 15, bk = lane >> 4;
  const int row = rbase + 4 * (bk >> 1) + (i >> 2);
  const int col = cbase + 16 * (bk & 1) + 4 * (i & 3);
  typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
  union { s16x4 h[2]; bf16x8 v; } o;
  o.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(t + row * LD + col));
  o.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(t + (row + 8) * LD + col));
  return o.v;
}

// Work-groups are handed to the 8 XCDs round-robin in launch order, and each XCD has its own L2.
// This maps the hardware block id to a logical (x, y, z) such that blocks with consecutive
// logical ids (same head and row, neighbouring tiles: the ones that re-read the same K/V or
// Q/dO) run on the same XCD.  A bijection on [0, gridDim.x*gridDim.y*gridDim.z).
// `together`: heads are taken in groups of that many (a divisor of gridDim.y), a group's rows one after the other.  For
// kernels with a dense bias: the work-groups that an XCD runs at one time then belong to as many heads as its L2
// holds the bias of (heads_together below), instead of fetching every head's bias again for every row, while a row's K / V
// (or Q / dO) are still shared by neighbouring tiles.  As many heads as fit, because neighbouring heads' slices of 64
// bytes share cache lines: forward of 512 rows x 8 heads x 384, one head at a time 230 us,
// four 216.
struct BlockId { int x, y, z; };
__device__ inline BlockId xcd_block_id(int together = 0) {
  constexpr int NX = 8;
  const int gx = gridDim.x, gy = together > 0 ? together : gridDim.y, gz = gridDim.z;
  const int n = gx * gridDim.y * gz;
  const int lin = blockIdx.x + gx * (blockIdx.y + gridDim.y * blockIdx.z);
  const int xcd = lin % NX, idx = lin / NX;
  const int v = xcd * (n / NX) + min(xcd, n % NX) + idx;
  BlockId b;
  b.x = v % gx;
  const int yz = v / gx;
  b.y = yz % gy;
  b.z = yz / gy;
  if (gy < (int)gridDim.y) {
    b.y += gy * (b.z / gz);
    b.z %= gz;
  }
  return b;
}
// the most heads, dividing `heads`, whose bias of `entry` bytes an entry fits the 4 MiB of an XCD's L2 (1 if none does)
inline int heads_together(int heads, int S, int entry) {
  int g = heads;
  while (g > 1 && (heads % g || (int64_t)g * S * S * entry > (4 << 20))) --g;
  return g;
}

// Dense bias tile of one wavefront: 32 rows (queries, or keys of the transposed copy) by 64 columns.
// A lane of the score tile owns one row and needs 4 consecutive columns at a time, so direct loads
// would touch 64 rows per instruction.  Instead 8 lanes fetch 128 contiguous bytes of one row, 16
// bytes each (8 rows per instruction, 4 instructions per tile, issued one tile ahead: 8-byte loads
// move half as many bytes per cycle through a compute unit's load path, and the bias is two thirds
// of these kernels' load traffic), the tile is parked in a wavefront-private LDS area and read back
// in the layout of the accumulator.  LDS rows are padded to 136 bytes so that the 8-byte reads of 32
// rows fall into distinct banks.  The loads are buffer loads over the head's S x S matrix: a row past
// S - 1 lies past the end and reads as zeros, columns past S - 1 read the next row; both belong to
// scores that are masked or never stored.  S * S * 2 is at most 2 GiB.
// Any S: rows start at multiples of 2 S bytes, so with S % 8 != 0 the 16-byte loads are unaligned
// (down to 2 bytes), which the hardware takes; only the bytes of a row then touch one cache line
// more.  With S odd the matrix ends inside a dword: the descriptor stops before it and the one entry
// that lies there, (S - 1, S - 1), is put into the parked tile by hand.
// (ODD: a variant of its own, the registers of that step cost the others a spill.)
constexpr int BIAS_LD = 68, BIAS_TILE_ELEMS = 32 * BIAS_LD;
enum { BIAS_OFF = 0, BIAS_EVEN = 1, BIAS_ODD = 2, BIAS_COPY = 3 };  // no dense bias; S even, S odd; BiasCopy below
template <bool ODD>
struct BiasTile {
  __amdgpu_buffer_rsrc_t rs;  // the head's matrix
  uint16_t* lds;              // the wavefront's area, BIAS_TILE_ELEMS elements
  uint32_t off, rstep;        // byte offset of this lane's chunk in tile 0; bytes between its rows
  u32x4 nxt[4];
  const uint16_t* last;       // S odd: the entry added by hand, the tile that holds it (-1: not in these rows), its place
  int last_tile, last_at, in_flight;  // ... and the tile in the registers; all uniform
  __device__ void init(const uint16_t* head, int row0, int S, uint16_t* area, int lane) {
    rs = __builtin_amdgcn_make_buffer_rsrc((void*)head, 0, (int)((int64_t)S * S * 2) & ~3, 0x00020000);
    const int first = __builtin_amdgcn_readfirstlane(min(row0, S - 1));
    off = ((uint32_t)(first + (lane >> 3)) * (uint32_t)S + 8u * (lane & 7)) * 2u;
    rstep = 16u * (uint32_t)S;  // 8 rows
    lds = area;
    last = head + ((int64_t)S * S - 1);
    last_tile = first + 32 >= S ? (S - 1) >> 6 : -1;
    last_at = (S - 1 - first) * BIAS_LD + ((S - 1) & 63);
    in_flight = -1;
  }
  __device__ void load(int tile) {
#pragma unroll
    for (int c = 0; c < 4; ++c) nxt[c] = __builtin_amdgcn_raw_buffer_load_b128(rs, off + tile * 128 + c * rstep, 0, 0);
    in_flight = tile;
  }
  __device__ void park(int lane) {
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      uint16_t* d = lds + ((lane >> 3) + 8 * c) * BIAS_LD + 8 * (lane & 7);
      *(uint2*)d = uint2{nxt[c][0], nxt[c][1]};
      *(uint2*)(d + 4) = uint2{nxt[c][2], nxt[c][3]};
    }
    if (ODD && in_flight == last_tile) lds[last_at] = *last;
  }
  // columns col .. col + 3 (col a multiple of 4) of row r of the parked tile
  __device__ uint2 read(int r, int col) const { return *(const uint2*)(lds + r * BIAS_LD + col); }
};

// Dense bias in the form in which the matrix instructions take it: the accumulator that the scores start from.
// A scale * score + bias is scale * (score + bias / scale), so the quotient, in fp32 and in accumulator layout, is the C
// operand of a block's first matrix instruction, and a score costs neither the unpacking of a bf16 bias nor an addition.
// `bias_copy_kernel` lays the heads' matrices out that way once per call, in scratch: blocks of 32 x 32 (strip of 32
// rows, then column block), a block as four runs of 64 lanes x 16 bytes, so that every load is 1 KB in one piece; entries
// outside S x S are -inf, which masks them.  Twice the bytes of the parked tile above, but no LDS traffic, no
// alignment to observe and half the registers in flight.  Both give the same bits (bf16 to fp32 times 1 / scale).
constexpr int64_t bias_copy_strips(int S) { return (S + 31) / 32; }
constexpr int64_t bias_copy_blocks(int S) { return 2 * ((S + 63) / 64); }  // of a strip
constexpr int64_t bias_copy_bytes(int S, int heads) { return heads * bias_copy_strips(S) * bias_copy_blocks(S) * 4096; }
struct BiasCopy {
  __amdgpu_buffer_rsrc_t rs;  // the strip
  uint32_t at;                // of the lane
  __device__ void init(const float* copy, int head, int row0, int S, int lane) {  // head counts from the copy's first
    const int64_t strip = head * bias_copy_strips(S) + min(row0 >> 5, (int)bias_copy_strips(S) - 1);
    const uint32_t bytes = (uint32_t)bias_copy_blocks(S) * 4096u;
    const uint64_t from = (uint64_t)copy + (uint64_t)strip * bytes;
    // (the builtin returns an int: unsigned before it is widened)
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)from), hi = __builtin_amdgcn_readfirstlane((uint32_t)(from >> 32));
    const uint64_t uniform = (uint64_t)hi << 32 | lo;
    rs = __builtin_amdgcn_make_buffer_rsrc((void*)uniform, 0, (int)bytes, 0x00020000);
    at = 16u * lane;
  }
  __device__ void load(f32x16& x, int block) const {
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rs, at + 1024u * g, block * 4096, 0);
#pragma unroll
      for (int e = 0; e < 4; ++e) x[4 * g + e] = __uint_as_float(v[e]);
    }
  }
};
// the same of a parked tile: columns 32 kb .. + 31 of the lane's row
template <bool ODD>
__device__ inline void parked_bias(const BiasTile<ODD>& bt, int r, int kb, int hl, float inv_scale, f32x16& x) {
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const uint2 u = bt.read(r, 32 * kb + 8 * g + 4 * hl);
    x[4 * g + 0] = __uint_as_float(u.x << 16) * inv_scale;
    x[4 * g + 1] = __uint_as_float(u.x & 0xffff0000u) * inv_scale;
    x[4 * g + 2] = __uint_as_float(u.y << 16) * inv_scale;
    x[4 * g + 3] = __uint_as_float(u.y & 0xffff0000u) * inv_scale;
  }
}

// Block order of launches whose blocks of a (row, head) unit differ in work (causal), x counting from the
// heaviest.  The XCDs are dealt the work-groups round-robin, and inside an XCD the dispatcher deals the
// first 32 out one per compute unit and then starts over, so both the share of an XCD and the company
// a work-group gets on its compute unit follow from the launch position:
//  - every XCD gets units / 8 whole units, whose K / V (or Q / dO) stay in its L2; the blocks of the units
//    left over are dealt round-robin, 4, 2 and 1 of those units at a time, so that a unit is spread over
//    2, 4 or 8 XCDs in equal parts (contiguous pieces gave one XCD the heavy half of a unit and the next
//    one the light half);
//  - an XCD takes its blocks heaviest first, the units' blocks of one rank next to each other;
//  - with 32 to 64 blocks, and two to a compute unit (`pairs`), the heaviest stay alone and the others are
//    paired medium with light.
// Any order gives the same results.  Causal forward of 12 heads x 12288 x 128: 568 -> 457 us, backward 2.69 ->
// 2.23 ms; 12 x 4000 x 128: 102 -> 77 us (before: heaviest first in contiguous pieces, xcd_block_id).
__device__ inline BlockId causal_block_id(bool pairs) {
  constexpr int NX = 8, NCU = 32;
  const int gx = gridDim.x, units = gridDim.y * gridDim.z, n = gx * units;
  const int lin = blockIdx.x + gx * (blockIdx.y + gridDim.y * blockIdx.z), xcd = lin % NX, idx = lin / NX;
  const int count = (n - xcd + NX - 1) / NX;
  int at = idx;  // rank in the XCD's order
  if (pairs && count > NCU && count <= 2 * NCU) {
    const int m = count - NCU;
    at = idx < m ? NCU - m + idx : idx < NCU ? idx - m : count - 1 - (idx - NCU);
  }
  // the whole units' blocks and the dealt ones, mixed in proportion; then the dealt ones by group
  const int own = units / NX;
  int over = count - own * gx, unit, x;
  // (a 64-bit division costs a good hundred instructions before the first load: only for launches that need it)
  const bool wide = (int64_t)(count + 1) * over >= (1ll << 31);
  auto before = [&](int pos, int part, int all) {
    return wide ? (int)((int64_t)pos * part / all) : (int)((uint32_t)(pos * part) / (uint32_t)all);
  };
  int lo = over ? before(at, over, count) : 0;
  if (!over || before(at + 1, over, count) == lo) {
    const int f = at - lo;
    x = f / own;
    unit = xcd * own + f % own;
  } else {
    int first = own * NX, start = 0;  // first unit of the group, XCD at which its dealing starts
    unit = first;
    x = 0;
    for (int g = 4; g >= 1; g >>= 1) {
      if (!(units & g)) continue;
      const int place = (xcd - start + NX) % NX, here = (g * gx - place + NX - 1) / NX;  // blocks of the group on this XCD
      const int taken = before(lo, here, over);
      if (here == over || before(lo + 1, here, over) != taken) {
        unit = first + place % g;
        x = taken * (NX / g) + place / g;
        break;
      }
      lo -= taken;
      over -= here;
      first += g;
      start = (start + g * gx) % NX;
    }
  }
  BlockId b;
  b.x = x;
  b.y = unit % (int)gridDim.y;
  b.z = unit / (int)gridDim.y;
  return b;
}

// The two-product form of dQ (fast_rdq.hip) rounds p dP to bf16 before the mean of dP is taken off,
// so what dP has in common over a query's keys (as activations and gradients with a mean of their own give
// it) would cost its size times 2^-9.  dS does not change if a constant per query is subtracted from every dP: the mean
// of dP so far, weighted with the probabilities, the block at hand included.  It is taken anew on the first block in which a
// query sees a key and whenever the weight seen has grown fourfold, for all queries of the wavefront as soon as one asks for
// it, and the sums formed with the old constant are moved to the new one.  The bound: between two changes, a weight w < 3 W
// of keys whose mean is off by x is rounded at the size of x, and adds at least w W / (W + w) x^2 > w x^2 / 4 to
// the variance of dP; so the products' rounding is at most twice that of dS formed directly, however the means and the weights
// of the keys are spread.  Relative error of dQ, 384 tokens, dO offset by 1, the products' arithmetic with no constant | with the
// unweighted mean of the first 32 keys, kept | with this one | dS formed directly, x 1e-3: no offset in V 1.7 | 1.7 | 1.7 | 1.7; V offset by 2
// throughout 23 | 1.7 | 1.6 | 1.7; V of the first 32 keys by 4: 2.0 | 8.2 | 3.0 | 1.8, these keys with a bias of -8 too: 1.7 | 40 | 1.6 | 1.8;
// V and bias rising by 8 and 40 along the keys: 70 | 65 | 1.4 | 1.7.  (Twofold instead of fourfold: 2.1 instead of 3.0, and twice as many
// changes: six instead of three of 12 blocks of normal scores, seven instead of four of 32.)
struct DpShift {
  float c = 0.f;    // of the lane's query
  float due = 0.f;  // weight of this half-wave's keys above which c is taken anew
  // after the row maximum was raised
  __device__ void rescaled(float alpha) { due *= alpha; }
  // On every block, in order, `lnew` being this half-wave's sum of p with the block's: whether the constant is taken anew ...
  __device__ bool is_due(float lnew) const { return __builtin_amdgcn_ballot_w64(lnew > due) != 0; }
  // ... which returns what, times the sums of p, is to be added to the sums formed with the old one.  `lsum`, `dsum`: the sums of p and
  // p (dP - c) over the earlier blocks, rounded operands or not.
  __device__ float take(const float (&p)[16], const f32x16& dp, float lsum, float lnew, float dsum) {
#pragma clang fp contract(off)  // the same bits wherever this is inlined
    float x = __builtin_fmaf(lsum - lnew, c, dsum);
#pragma unroll
    for (int v = 0; v < 16; ++v) x = __builtin_fmaf(p[v], dp[v], x);
    const float w = half_sum(lnew);  // 0 if no key was seen, else at least 2^-8
    const float d = -half_sum(x) * fast_rcp(fmaxf(w, 1e-30f));
    c -= d;
    due = 4.f * lnew;
    return d;
  }
};

// The running maxima of a kernel that forms a block's probabilities with the maximum so far and looks at the block's own only where
// that is needed (pair_fwd.hip), NR rows per wavefront.  What tells is a half-wave's sum of 16 probabilities:
//  up to 2^8: nothing to be done, and a score has cost no comparison;
//  up to 2^26: the probabilities and the sums so far are scaled down by the sum's power of two (an exponent below 26 is exact to
//    2^-20, the result's LSE is rounded to no less);
//  beyond, infinite ones included: the block is formed again with the maxima of those queries raised.
// After a block formed again, or scaled by 2^19 or more, these queries look first, as all do on a row's first block, until their maximum
// grows by no more than 2^6.  A block formed again costs nearly as much as two, a scaled one or a look a quarter of one.  The lines: 2^6, 2^19 and 2^26 are
// far enough apart for a steady growth to find its one way, and all queries of a wavefront the same (a scaled block that has a look too costs half a block; with 2^16
// in place of 2^26 a growth of 9 or 14 bits a block took 1.4 times as long).  256 rows x 4 heads x 1024, bias less 0 | 0.03 | 0.1 | 0.2 | 0.3 | 0.5 | 1 times |i - j|,
// us: 300 | 333 | 338 | 377 | 371 | 332 | 327, queries four times larger 329; every such block formed again 295 | 421 | 431 | 430 | 429 | 426 | 425, 396; the
// general forward, a maximum on every block: 343 | 347 | 348 | 345 | 344 | 342 | 341, 348.
// What a query does depends on its own scores alone, not on its company.
template <int NR>
struct RowMaxima {
  static constexpr float SCALE = 1 << 8, RAISE = 1 << 26;
  uint64_t looks[NR];  // lane masks
  __device__ bool any() const { return (looks[0] | looks[NR - 1]) != 0; }
  // Raises the negated maximum `nm` of row n (again: where the half-wave's `sum` asks for it); returns the factor of the sums so far.
  __device__ __forceinline__ float raise(int n, const f32x16& s, float c1, float& nm, bool first, bool again, float sum) {
    float rmax = -INFINITY;
#pragma unroll
    for (int v = 0; v < 16; ++v) rmax = fmaxf(rmax, s[v]);
    rmax = half_max(rmax * c1);
    const bool mine = again ? half_max(sum) > RAISE : __builtin_amdgcn_inverse_ballot_w64(looks[n]);
    const float by = mine ? fmaxf(rmax + nm, 0.f) : 0.f;
    const uint64_t more = __builtin_amdgcn_ballot_w64(by > 6.f && !first);
    looks[n] = again ? looks[n] | more : more;
    const float mn = by > 0.f ? rmax : -nm, alpha = fast_exp2(-nm - mn);
    nm = -mn;
    return alpha;
  }
  // the factor of row n where the sum exceeds 2^8, with `nm` set to it; else 1
  __device__ __forceinline__ float scale(int n, float& nm, float sum) {
    sum = half_max(sum);
    const float by = sum > SCALE && sum < INFINITY ? (float)((int)(__float_as_uint(sum) >> 23) - 127) : 0.f;
    looks[n] |= __builtin_amdgcn_ballot_w64(by >= 19.f);
    const float old = nm;
    nm -= by;
    return fast_exp2(nm - old);  // of the difference that was taken: the subtraction may have rounded
  }
};

__device__ inline int key_of(int v, int hl) { return 8 * (v >> 2) + 4 * hl + (v & 3); }

// Forward epilogue for one 32-column block `db` of a query's output (lane = query, registers =
// columns 8g + 4*hl + e, not yet normalised): normalise by `inv`, gate, store Y; recompute
// mode: gate gradient and pre-gated dO copy, and `part` continues this lane's part of
// Delta = rowsum(dO * O).  Rows are read and written 16 bytes per lane (load_row32 / store_row32).
// Both lanes of the row must be active.
template <bool RECOMP>
__device__ inline float fwd_epilogue_block(const KP& p, const f32x16& o16, int db, float inv, int b, int h, int q, int hl,
                                           int64_t base, float part) {
  const int64_t row = base + (int64_t)q * p.ss + 32 * db;
  float o[16], gt[16];
#pragma unroll
  for (int v = 0; v < 16; ++v) o[v] = o16[v] * inv;
  if (p.gated) {
    uint2 gu[4];
    load_row32((const uint16_t*)p.G + row, gu, hl);
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const float gl[4] = {__uint_as_float(gu[g].x << 16), __uint_as_float(gu[g].x & 0xffff0000u),
                           __uint_as_float(gu[g].y << 16), __uint_as_float(gu[g].y & 0xffff0000u)};
#pragma unroll
      for (int e = 0; e < 4; ++e) gt[4 * g + e] = fast_rcp(1.f + fast_exp2(-gl[e] * LOG2E));
    }
  }
  if (!RECOMP) {
    if (p.gated) {
#pragma unroll
      for (int v = 0; v < 16; ++v) o[v] *= gt[v];
    }
    uint2 out[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      out[g].x = pack2_bf16(o[4 * g], o[4 * g + 1]);
      out[g].y = pack2_bf16(o[4 * g + 2], o[4 * g + 3]);
    }
    store_row32((uint16_t*)p.Y + row, out, hl, true);
  } else {
    uint2 du[4];
    load_row32((const uint16_t*)p.dY + row, du, hl);
    float go[16];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      go[4 * g] = __uint_as_float(du[g].x << 16); go[4 * g + 1] = __uint_as_float(du[g].x & 0xffff0000u);
      go[4 * g + 2] = __uint_as_float(du[g].y << 16); go[4 * g + 3] = __uint_as_float(du[g].y & 0xffff0000u);
    }
    if (p.gated) {
      uint2 o1[4], o2[4];
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        float dg[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int v = 4 * g + e;
          dg[e] = go[v] * o[v] * gt[v] * (1.f - gt[v]);
          go[v] *= gt[v];
        }
        o1[g] = uint2{pack2_bf16(dg[0], dg[1]), pack2_bf16(dg[2], dg[3])};
        o2[g] = uint2{pack2_bf16(go[4 * g], go[4 * g + 1]), pack2_bf16(go[4 * g + 2], go[4 * g + 3])};
        // the later kernels read the rounded copy
        go[4 * g] = __uint_as_float(o2[g].x << 16); go[4 * g + 1] = __uint_as_float(o2[g].x & 0xffff0000u);
        go[4 * g + 2] = __uint_as_float(o2[g].y << 16); go[4 * g + 3] = __uint_as_float(o2[g].y & 0xffff0000u);
      }
      store_row32((uint16_t*)p.dG + row, o1, hl, true);
      store_row32((uint16_t*)p.dO_out + (int64_t)(b - p.do_b0) * p.do_sb + (int64_t)q * p.do_ss + (int64_t)(h - p.do_h0) * p.do_sh + 32 * db, o2, hl,
                  true);
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) part = fmaf(go[v], o[v], part);
  }
  return part;
}

// forward epilogue: normalise, gate, store Y (and LSE); recompute mode: gate gradient,
// pre-gated dO copy, Delta = rowsum(dO*O) and LSE into the workspace.  `l` is the complete row sum that O
// is divided by, `lse_l` the one that the LSE is taken of.
template <int DB, bool RECOMP>
__device__ inline void fwd_epilogue_rowsum(const KP& p, f32x16 (&oacc)[DB], float m, float l, float lse_l, int b, int h, int q,
                                           int hl, int64_t base) {
  if (q >= p.S) return;
  const float inv = 1.f / l;
  const float lse = (m + log2f(lse_l)) * LN2;
  float part = 0.f;
#pragma unroll
  for (int db = 0; db < DB; ++db) part = fwd_epilogue_block<RECOMP>(p, oacc[db], db, inv, b, h, q, hl, base, part);
  if (!RECOMP) {
    if (p.lse_out && hl == 0) p.lse_out[(int64_t)(b - p.lse_b0) * p.lse_sb + (int64_t)(h - p.lse_h0) * p.lse_sh + q] = lse;
  } else {
    part = half_sum(part);
    if (hl == 0) {
      p.delta[(int64_t)(b - p.dl_b0) * p.dl_sb + (int64_t)(h - p.dl_h0) * p.dl_sh + q] = part;
      if (p.lse_out) p.lse_out[(int64_t)(b - p.lse_b0) * p.lse_sb + (int64_t)(h - p.lse_h0) * p.lse_sh + q] = lse;
    }
  }
}
// the same with `l` = each half-wave's part of the row sum
template <int DB, bool RECOMP>
__device__ inline void fwd_epilogue(const KP& p, f32x16 (&oacc)[DB], float m, float l, int b, int h, int q,
                                    int hl, int64_t base) {
  if (q >= p.S) return;
  const float rowsum = half_sum(l);
  fwd_epilogue_rowsum<DB, RECOMP>(p, oacc, m, rowsum, rowsum, b, h, q, hl, base);
}

// the specialised kernels serve: no bias or a dense bf16 bias; no mask or the causal mask; a
// positive scale; more than one 64-key tile's worth of rows
inline bool fast_ok(const KP& p) {
  if (p.S <= 64 || !(p.scale > 0.f) || p.mask_kind == 2 || p.bias_kind == 2) return false;
  // the bias is divided by the scale: not where that could leave the range of fp32
  if (p.bias_kind == 1 && !(p.scale > 1e-9f && p.scale < 1e9f)) return false;
  if (p.bias_kind == 1 && (!p.bias_bf16 || p.S > 32768)) return false;
  return true;
}

// the window kernels (win_fwd.hip, win_bwd.hip) serve, beside what row_ok adds: head size 32, 65 to 160 tokens, a relative-position bias or a
// region mask (a bf16 bias of either kind, or none; no causal mask), a positive scale
inline bool win_ok(const KP& p) {
  if (p.D != 32 || p.S <= 64 || p.S > 160 || !(p.scale > 0.f) || p.mask_kind == 1) return false;
  // (scales outside these go to the all-feature kernels as those of fast_ok do, which form bias / scale; nothing here does)
  if (p.bias_kind != 0 && (!p.bias_bf16 || !(p.scale > 1e-9f && p.scale < 1e9f))) return false;
  return p.bias_kind == 2 || p.mask_kind == 2;
}
// Rows of pair attention take the same kernels, head size 32, no mask, a dense bf16 bias or none: the backward of 65 to 160 tokens, with a gate up to 144 (that line
// is from when ten wavefronts with a gate spilled; they no longer do and would be the faster ones: backward, tiled kernels | these, dense bias, 1000 rows x 8 heads x 160
// 638 | 552 us, 300 x 8 x 160 192 | 112, 100 x 60 x 160 513 | 492, 16 x 4 x 150 33.8 | 22.8, no bias 1000 x 8 x 160 408 | 264); the forward of 129 to 160, of up to 128 (row, head)
// pairs only without a bias, which a work-group gathers before its first row.  Us, gated, dense bias, tiled
// kernels | these: backward, 16 x 4 x 100 30.4 | 16.5, 100 x 4 x 128 40.9 | 34.2, 64 x 8 x 128 41.1 | 34.6, 1000 x 8 x 112 339 | 221; without a bias 64 x 4 x 128
// 16.2 | 9.9, 1000 x 8 x 144 407 | 245; without a gate 300 x 8 x 160 177 | 112.  Forward, 60 x 8 x 155 14.4 | 12.3, 120 x 8 x 140 23.6 | 18.9, 1000 x 8 x 160
// 163 | 121; 4 x 129 6.5 | 7.7, 128 x 160 6.5 | 7.1 (without a bias 5.1 | 4.4), 136 x 129 8.2 | 7.9, 144 x 160 7.8 | 7.1; 100 x 8 x 128 11.7 | 15.0, 500 x 4 x 128 20.2 | 23.9, 150 x 8 x 100 14.4 | 15.1, 200 x 4 x 96 10.4 | 11.9.
// Gated rows of 17 to 64 tokens with any bf16 bias, without a causal mask, too (without a gate: small_kernels.hip); the all-feature kernels | these, step: 512 rows x 8 heads x 64,
// dense bias, 1607 | 72, no bias 200 x 8 x 64 69 | 27, 300 windows of 7 x 7 x 8 heads with regions 1278 | 47; backward 20 x 4 x 50 90 | 14; forward 512 x 8 x 64 36.7 | 21.7 (of small shares the launch, 8 - 10).
inline bool row_ok(const KP& p, bool forward) {
  if (win_ok(p)) return true;
  if (p.D == 32 && p.gated && p.S > 16 && p.S <= 64 && p.scale > 0.f && p.mask_kind != 1 && (p.bias_kind == 0 || p.bias_bf16)) return true;
  return p.D == 32 && p.S > 64 && p.S <= 160 && p.scale > 0.f && p.mask_kind == 0 && (p.bias_kind == 0 || (p.bias_kind == 1 && p.bias_bf16)) &&
         (forward ? p.S > 128 && (p.bias_kind == 0 || p.share_units > 128) : !p.gated || p.S <= 144);
}

// Work-group shape of the forward / dQ kernels: query wavefronts x key-tile groups.  Large shares
// use 4x1 (many independent work-groups per compute unit); when the whole share offers fewer than
// two 128-query work-groups per compute unit the key tiles are split over groups inside the
// work-group (4x2); below one per compute unit (2x4) separate kernels take over whose work-groups
// own 32 queries (forward, dQ) or 32 keys (dK/dV) and whose four wavefronts split the other axis.
// Decided from the share, never from the chunk.
// Rows per group of the tiled bias-gradient kernel: 0 = one group (the sum continues in the output);
// otherwise the share's rows are cut into groups so that about two work-groups per compute unit exist.
inline int tiled_group_rows(const KP& p) {
  if (p.bias_kind != 1 || !fast_ok(p)) return 0;
  const int64_t tiles = (int64_t)((p.S + 63) / 64) * ((p.S + 63) / 64);
  if (tiles * p.H >= 512) return 0;
  // A work-group walks its group's rows one after the other: shorter groups while the launch has fewer than
  // some 480 work-groups, down to 8 rows (the sums of a group cost a pass over H x S x S).  Backward of 108 rows x
  // 4 heads x 284: 121 -> 106 us; 46 x 4 x 295: 82 -> 69; 247 x 8 x 77: 105 -> 87.
  int gw = 64;
  while (gw > 8 && tiles * p.share_units < 480 * (int64_t)gw) gw >>= 1;
  return gw;
}

inline int dbias_group_rows(const KP& p) {
  if (!row_ok(p, false)) return tiled_group_rows(p);
  // one work-group per group and head, all of them at one time: two on a compute unit of up to 112 tokens, one of more (win_bwd.hip)
  const int most = p.S > 112 ? 256 : 512;
  int rows = (p.share_units + most - 1) / most;
  if (p.bias_kind == 0 || win_ok(p) || p.S <= 64) return p.bias_kind == 0 ? 0 : rows;
  // (a dense bias: two or three rows are not worth sums beyond what a workspace is made larger for)
  while (rows > 1 && rows < 4 && (int64_t)(p.share_units / rows) * p.S * p.S * 4 > (12 << 20)) ++rows;
  return rows < 64 ? rows : 64;
}

// the longest such groups (0: one group): 64 rows, but for shapes whose sums can go on in the output
inline int dbias_longest_group(const KP& p) {
  return win_ok(p) || (p.S & 3) || tiled_group_rows(p) == 0 ? 0 : 64;
}

// calls f with the compile-time bias variant and causal flag of the launch
template <class F>
inline void dispatch_bias(const KP& p, F f) {
  const int bias = p.bias_kind == 1 ? ((p.S & 1) ? BIAS_ODD : BIAS_EVEN) : BIAS_OFF;
  auto with = [&](auto causal) {
    if (bias == BIAS_ODD) f(std::integral_constant<int, BIAS_ODD>{}, causal);
    else if (bias == BIAS_EVEN) f(std::integral_constant<int, BIAS_EVEN>{}, causal);
    else f(std::integral_constant<int, BIAS_OFF>{}, causal);
  };
  if (p.mask_kind == 1) with(std::true_type{});
  else with(std::false_type{});
}

enum WgShape { WG_4x1, WG_4x2, WG_2x4 };
inline WgShape wg_shape(const KP& p) {
  const int64_t wgs = (int64_t)((p.S + 127) / 128) * p.share_units;
  const bool causal = p.mask_kind == 1;
  if (p.bias_kind == 0 && p.D >= 64) {
    // Where the lines lie (measured on 40 shapes each, forward and backward): at head size 128 the 4x1
    // kernels are a family of their own (fast_fwd128.hip) that beats 4x2 at any fill (12 x 4000: 325 us
    // backward against 389), and without a mask already below one work-group per compute unit (8 x 3500: 68
    // against 77 us forward); short rows leave the chip to fewer, longer work-groups unless the smallest
    // shape is used (4 x 10 x 400: 53 -> 35 us backward, 12 heads x 450: 49 -> 20), which loses its edge
    // near 160 work-groups, 128 without a mask.
    if (p.S < 512) {
      if (wgs >= (causal ? 168 : 128)) return WG_4x1;
    } else {
      if (wgs >= (p.D == 128 ? (causal ? 304 : 192) : 512)) return WG_4x1;
      // 4x2 holds one work-group per compute unit: without a mask a second round pays only when it is filled
      // (15 heads x 2300 x 64, 270 work-groups: 259 us backward against 206)
      if (p.D == 64 && (causal ? wgs >= 256 : (wgs >= 192 && wgs <= 256) || wgs >= 352)) return WG_4x2;
    }
  } else {
    if (wgs >= 512 || p.S < 512) return WG_4x1;
    if (wgs >= 256) return WG_4x2;
  }
  // the kernels of the smallest shape read the bias four aligned columns at a time
  if (p.bias_kind == 1 && (p.S & 3)) return WG_4x2;
  // the kernels of the smallest shape address one (row, head) slice with 32-bit buffer offsets
  const int64_t row_stride = p.ss > (int64_t)p.H * p.D ? p.ss : (int64_t)p.H * p.D;
  if (((int64_t)(p.S - 1) * row_stride + p.D) * 2 >= (1ll << 31)) return WG_4x2;
  return WG_2x4;
}

// Large shares at head size 128 without a bias: the kernels whose tiles go straight into LDS (fast_fwd128.hip, fast_stat128.hip, fast_dq128.hip, fast_kv128.hip).
// They address a (row, head) slice with 32-bit offsets; longer ones (transposed storage) go to the kernels with 64-bit addresses.
inline bool direct128_ok(const KP& p) {
  if (p.D != 128 || p.bias_kind != 0 || wg_shape(p) != WG_4x1) return false;
  const int64_t row_stride = p.ss > (int64_t)p.H * p.D ? p.ss : (int64_t)p.H * p.D;  // also of dO's scratch
  return ((int64_t)(p.S - 1) * row_stride + p.D) * 2 < (1ll << 31);
}

// The forward of the smallest shape at head size 128, causal: two query blocks per work-group of eight wavefronts where
// that leaves blocks enough for more than one per compute unit (12 heads x 2048, 384 of them: 27.5 -> 23.9 us; 8 x 3000, 376:
// 33.6 -> 30.3; 3 x 8000, 375: 77.6 -> 72.2; 16 x 1024, 256: 12.2 -> 13.9; 4 x 4096, 256: 29.2 -> 37.6) and no more than two (16 x 2048, 512:
// 30.1 -> 26.9; 50 x 617, 500: 17.4 -> 17.3; but 40 x 800, 520: 18.7 -> 22.0, 52 x 617, 520: 19.6 -> 21.4, 27 x 1400, 594: 29.7 -> 31.5, 60 x 617, 600: 20.7 -> 22.3).
// Without a mask all blocks are as long as the longest and the work-groups of four do better (10 x 2000: 37.0 -> 41.7).
inline bool wave_pairs(const KP& p) {
  const int64_t blocks = (int64_t)((p.S + 31) / 32) * p.share_units, pairs = (int64_t)((p.S + 63) / 64) * p.share_units;
  return p.mask_kind == 1 && blocks >= 704 && pairs <= 512;
}
// The backward of that shape, two blocks per work-group of four wavefronts (bwd_pair128_kernel), with the work-groups of the
// whole share.  Causal: from a little over one round of the 512 that the chip holds (384: 28.6 -> 29.5 us; 480: 33.6 -> 32.3
// and 56.6 -> 60.0; 576: 37.8 -> 34.8; 768: 116 -> 108; 1152: 101.8 -> 84.5, all with the recompute pass).  Without a mask
// all work-groups are equally long: where the last round is at least half full (240: 16.3 -> 16.8; 384: 40.4 -> 35.6;
// 480: 49.6 -> 43.9; 564: 484 -> 501; 600: 117.5 -> 127.2; 768: 66.1 -> 64.2; 960: 146 -> 138).
inline bool wave_bwd_pairs(const KP& p) {
  const int64_t n = 3 * (int64_t)((p.S + 63) / 64) * p.share_units;
  return p.mask_kind == 1 ? n >= 544 : (n - 1) % 512 >= 255 && n >= 384;
}
// the forward of pair_fwd.hip: head size 32 with a dense bias, no causal mask, the large-share shape, 32-bit offsets
inline bool pair_fwd_ok(const KP& p) {
  return fast_ok(p) && p.D == 32 && p.bias_kind == 1 && p.mask_kind == 0 && wg_shape(p) == WG_4x1 &&
         ((int64_t)(p.S - 1) * p.ss + p.D) * 2 < (1ll << 31);
}
// head size 32 on the large-share work-group shape: the vector arithmetic per score element binds, and
// the recompute pass and dQ share all of it (fast_rdq.hip)
inline bool rdq_ok(const KP& p) {
  if (!fast_ok(p) || p.D != 32 || wg_shape(p) != WG_4x1) return false;
  return ((int64_t)(p.S - 1) * p.ss + p.D) * 2 < (1ll << 31);  // the kernel addresses a (row, head) slice with 32-bit offsets
}

}  // namespace

// specialised kernels, one translation unit each
hipError_t launch_fast_fwd(const KP& p, bool recompute, hipStream_t st);
hipError_t launch_pair_fwd(const KP& p, hipStream_t st);
hipError_t launch_fast_fwd128(const KP& p, bool recompute, hipStream_t st);
hipError_t launch_fast_stat128(const KP& p, hipStream_t st);  // the recompute pass without a gate
hipError_t launch_fast_dq(const KP& p, hipStream_t st);
hipError_t launch_fast_dq128(const KP& p, hipStream_t st);
hipError_t launch_fast_recompute_dq(const KP& p, hipStream_t st);
hipError_t launch_fast_dkdv(const KP& p, hipStream_t st);
hipError_t launch_fast_kv128(const KP& p, hipStream_t st);
hipError_t launch_fast_fwd_wave(const KP& p, bool recompute, hipStream_t st);
hipError_t launch_fast_fwd_wave128(const KP& p, bool recompute, hipStream_t st);
hipError_t launch_fast_bwd_wave(const KP& p, hipStream_t st);
hipError_t launch_fast_bwd_wave3(const KP& p, hipStream_t st);
hipError_t launch_fast_dbias(const KP& p, hipStream_t st);
hipError_t launch_pair_dbias(const KP& p, hipStream_t st);
hipError_t launch_win_fwd(const KP& p, hipStream_t st);
hipError_t launch_win_bwd(const KP& p, hipStream_t st);  // all gradients, the bias gradient's group partials among them

}  // namespace ssa

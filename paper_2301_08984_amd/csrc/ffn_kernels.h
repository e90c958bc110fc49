// Launchers of the feed-forward kernels (bf16 MFMA GEMM with fused epilogues, column sums).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ssa {

enum { EPI_ACT = 0, EPI_MUL = 1, EPI_ACC = 2, EPI_STORE = 3, EPI_ACC16 = 4 };

// C[M,N] = A B (see gemm_kernel for the operand layouts); what happens to C:
//   EPI_ACT   out = act(C + bias[n]) (bf16); out2, if given, = act'(C + bias[n])
//   EPI_MUL   out = C * mul[m][n] (bf16; out may be mul)
//   EPI_ACC   the accumulator starts from acc32 if `accumulate`; then `last` ? out = C + bias[n] (bf16,
//             bias may be NULL) : acc32 = C (fp32, whole tiles in the kernel's own order; see gemm_acc_bytes)
//   EPI_STORE out = C (bf16)
//   EPI_ACC16 the accumulator starts from `out` (bf16, widened) if `accumulate`; out = C + bias[n] (bf16,
//             bias may be NULL): the partial sum between chunks lives in the output itself
struct GemmArgs {
  const uint16_t* A;
  const uint16_t* B;
  int64_t lda, ldb;
  int M, N, K;
  const uint16_t* bias;
  uint16_t* out;
  int64_t ldo;
  uint16_t* out2;
  const uint16_t* mul;
  int64_t ldm;
  float* acc32;  // ceil(M/256) * ceil(N/256) tiles of 256 x 256 fp32, in the kernel's own order
  int accumulate, last, act;
  uint16_t* colsum;  // EPI_STORE: if given (split = 1 only), colsum[n] (bf16) = sum over k of B[k][n]
  // how the product is cut up (gemm_plan)
  int narrow;          // tiled kernel: no 192-wide tiles
  int cols;            // 0: the tiled kernel; 64 or 32: the few-rows kernel, that many columns per work-group
  int split;           // parts of the contraction
  float* parts;        // fp32 partial sums, SPLIT_BYTES, and
  unsigned* counters;  // SPLIT_TILES zeros (left zero); NULL: one work-group takes a tile's parts in turn
};

// A product with few tiles leaves most of the chip idle while each tile walks the whole contraction, so
// its contraction is cut into parts that work-groups of their own sum up.  `M` and `N` are the extents
// of the whole share, so that an element's sum does not depend on the chunk it falls into.
struct GemmPlan { int cols, split; };
constexpr int SPLIT_TILES = 256;
constexpr size_t SPLIT_BYTES = (size_t)SPLIT_TILES * 128 * 128 * sizeof(float);
// The tiled kernel: as many parts as keep one 128 x 128 tile per compute unit (256), none shorter than 8
// stages of 64 (a part's sum takes some 4 us to hand over).
inline GemmPlan gemm_plan_tiled(int M, int N, int K) {
  const int64_t tiles = (int64_t)((M + 127) / 128) * ((N + 127) / 128);
  const int by_tiles = tiles > SPLIT_TILES ? 1 : (int)(SPLIT_TILES / tiles), by_depth = K / 512;
  const int p = by_tiles < by_depth ? by_tiles : by_depth;
  return {0, p < 2 ? 1 : p > 16 ? 16 : p};
}
// Tile shape of a product.  An output element is the same chain of MFMA steps whatever tile it falls into, so
// the shape goes by the sizes: the one that needs the least time for its rounds of one work-group per
// compute unit (256), a round of 256 x 128 tiles being 100 (168 us at a depth of 12288, measured; per
// element 128 x 128 takes 1.33, 128 x 192 1.13 and 256 x 192 1.07 times as long, the last two longer on short
// contractions).  Products cut into parts use 128 x 128.  `narrow`: no 192-wide tiles (a sum that continues
// from chunk to chunk has no such variant).  2048 x 6144 x 12288 (384 tiles of 256 x 128, one and a half
// rounds): 304 -> 259 us; 3000 x 3000 x 3000: 105 -> 77.
enum GemmTile { TILE_256x128, TILE_128x128, TILE_128x192, TILE_256x192 };
struct GemmShape {
  GemmTile tile;
  int cost;      // time in hundredths of a round of 256 x 128 tiles
  int64_t rounds;
  double idle;   // part of the chip that the last round leaves idle
  double round;  // us of a round
};
inline GemmShape gemm_shape(int M, int N, int K, int split, bool narrow) {
  constexpr int COST[4] = {100, 66, 85, 160}, BM[4] = {256, 128, 128, 256}, BN[4] = {128, 128, 192, 192};
  GemmShape best{TILE_256x128, 0, 0, 0., 0.};
  for (int t = 0; t < 4; ++t) {
    if ((split > 1 && t != TILE_128x128) || (narrow && BN[t] == 192)) continue;
    const int64_t n = (int64_t)((M + BM[t] - 1) / BM[t]) * ((N + BN[t] - 1) / BN[t]) * split, rounds = (n + 255) / 256;
    const int64_t cost = rounds * COST[t] * (BN[t] == 192 ? K + 160 : K) / K;
    if (best.cost && cost >= best.cost) continue;
    best = {(GemmTile)t, (int)(cost < 1000000 ? cost : 1000000), rounds, 1. - n / (256. * rounds), 0.0075 * COST[t] * K / (64. * split)};
  }
  return best;
}
// A of at most 64 rows, neither operand transposed.  The few-rows kernel starts faster (1 x 768 x 768: 5 us
// against 9), the tiled kernel streams a large B faster (64 x 6144 x 12288: 41 us against 57, one row 36
// against 37; 64 x 3000 x 2168: 20 against 12; the line lies near 16 million elements).  Narrow column tiles,
// up to one work-group per compute unit, no part with less than 3 steps of 32 for each of the 8 wavefronts;
// wide tiles where the narrow ones are more than the compute units (16 x 12288 x 768: 9.1 us against 11.3).
inline GemmPlan gemm_plan(int M, int N, int K) {
  if (M > 64 || (int64_t)N * K > (1 << 24)) return gemm_plan_tiled(M, N, K);
  const int tiles = (N + 31) / 32, deepest = K / (32 * 8 * 3);
  if (tiles > SPLIT_TILES) return {64, 1};
  const int p = SPLIT_TILES / tiles < deepest ? SPLIT_TILES / tiles : deepest;
  return {32, p < 1 ? 1 : p > 16 ? 16 : p};
}

// bytes of the fp32 partial-result buffer of an M x N product
size_t gemm_acc_bytes(int M, int N);
hipError_t launch_gemm(const GemmArgs& g, bool a_transposed, bool b_transposed, int epilogue, hipStream_t st);
// the few-rows kernel (g.cols != 0): A and B untransposed, EPI_ACT or EPI_ACC16
hipError_t launch_skinny(const GemmArgs& g, int epilogue, hipStream_t st);
// out[n] (bf16) = sum over m of A[m][n] (bf16 in, fp32 sum, fixed order)
hipError_t launch_colsum(const void* A, int64_t lda, int M, int N, void* out, hipStream_t st);

}  // namespace ssa

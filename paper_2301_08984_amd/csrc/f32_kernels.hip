// fp32 attention, head sizes up to 64, on v_mfma_f32_16x16x4_f32 (fp32 operands, products and sums).
//
// What bounds it: fp32 operators come small (a few heads of some hundred tokens), so the time is that of
// one work-group's chain of dependent loads and of the launches.  A work-group therefore takes only
// 16 queries (or keys), and its 8 wavefronts deal the other axis out among themselves in blocks of 16,
// every wavefront with a softmax (or sum) of its own; the 8 results meet in LDS.  The recompute pass and
// dQ share a launch, and so do dK/dV and the bias gradient: 3 launches for forward and backward.
// Operands go from memory (L2: the tensors are small) to registers, no LDS.  Step of 4 heads x 128 x
// 32: 85 -> 21 us; 4 x 8 heads x 508 x 16 with bias: 986 -> 156 us (plain vector kernels before).
//
// v_mfma_f32_16x16x4_f32 (lane l, i = l % 16, g = l / 16): A[m][k]: m = i, k = g;  B[k][n]: n = i, k = g;
// C[m][n]: n = i, register v holds m = 4g + v.  Which index a k-slot stands for is free as long as A and B
// agree:
//  - contractions over the head size: slot g of step (c, e) is d = 16c + 4g + e, so both operands are
//    16-byte loads of a row ("natural");
//  - contractions over the 16 rows of a block: slot g of step v is row 4g + v, so the registers of a C block
//    are the B operand of the next product as they stand; the A operand is column DC i + e of row 4g + v,
//    DC consecutive columns per lane ("transposed"), and the result holds columns DC (4g + v) + e.
#include "f32_kernels.h"

namespace ssa {
namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(2))) float f32x2;
constexpr int W = 8;  // wavefronts per work-group

__device__ inline f32x4 mfma4(float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

// e^x for x <= a few units above 0, relative error of about 1e-7: 2^(x log2 e) with the product's rounding
// error put back in; below e^-150 (also for -inf) zero; NaN stays NaN
__device__ inline float exp_f32(float x) {
  constexpr float L2E = 1.44269502e+00f, L2E_LO = 1.92596299e-08f, LN2 = 6.93147182e-01f;  // log2(e) = L2E + L2E_LO
  x = __builtin_elementwise_maximum(x, -150.f);
  const float t = x * L2E, r = fmaf(x, L2E_LO, fmaf(x, L2E, -t));
  const float y = __builtin_amdgcn_exp2f(t);
  return fmaf(y, r * LN2, y);
}

// what is subtracted from scores (and earlier maxima) under a maximum m: not -inf (no key yet), so that they
// get a weight of 0
__device__ inline float base_of(float m) { return m == -INFINITY ? 0.f : m; }

template <int DC>
struct Nat { f32x4 x[DC]; };
// natural operand: 16 floats of every 64 bytes of a row
template <int DC>
__device__ inline Nat<DC> load_nat(const float* row, int g, int D) {
  Nat<DC> f;
#pragma unroll
  for (int c = 0; c < DC; ++c) {
    f.x[c] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (16 * c + 4 * g < D) f.x[c] = *(const f32x4*)(row + 16 * c + 4 * g);
  }
  return f;
}
// transposed operand: DC columns of a row
template <int DC>
__device__ inline void load_tr(const float* row, int i, int D, float (&x)[DC]) {
  if constexpr (DC == 1) {
    x[0] = i < D ? row[i] : 0.f;
  } else if constexpr (DC == 2) {
    f32x2 v = f32x2{0.f, 0.f};
    if (2 * i < D) v = *(const f32x2*)(row + 2 * i);
    x[0] = v[0]; x[1] = v[1];
  } else {
    f32x4 v = f32x4{0.f, 0.f, 0.f, 0.f};
    if (4 * i < D) v = *(const f32x4*)(row + 4 * i);
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] = v[e];
  }
}
template <int DC>
__device__ inline f32x4 dot(const Nat<DC>& a, const Nat<DC>& b) {
  f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int c = 0; c < DC; ++c)
#pragma unroll
    for (int e = 0; e < 4; ++e) acc = mfma4(a.x[c][e], b.x[c][e], acc);
  return acc;
}
// sum of the products of the 16 rows of a block with the block's C registers, columns DC (4g + v) + e
template <int DC>
__device__ inline void accumulate(const float* base, int64_t stride, int row0, int S, int i, int g, int D, const f32x4& w,
                                  f32x4 (&acc)[DC]) {
  float x[4][DC];
#pragma unroll
  for (int v = 0; v < 4; ++v) load_tr<DC>(base + (int64_t)min(row0 + 4 * g + v, S - 1) * stride, i, D, x[v]);
#pragma unroll
  for (int v = 0; v < 4; ++v)
#pragma unroll
    for (int e = 0; e < DC; ++e) acc[e] = mfma4(x[v][e], w[v], acc[e]);
}
__device__ inline float over_groups_max(float x) {
  x = fmaxf(x, __shfl_xor(x, 16, 64));
  return fmaxf(x, __shfl_xor(x, 32, 64));
}
__device__ inline float over_groups_sum(float x) {
  x += __shfl_xor(x, 16, 64);
  return x + __shfl_xor(x, 32, 64);
}

// additive bias of pair (i, j)
__device__ inline float bias_f32(const KP& p, int h, int i, int j) {
  int64_t off;
  if (p.bias_kind == 1) {
    off = ((int64_t)h * p.S + i) * p.S + j;
  } else {
    const int yi = i / p.win_w, xi = i - yi * p.win_w, yj = j / p.win_w, xj = j - yj * p.win_w;
    off = (int64_t)h * ((2 * p.win_h - 1) * (2 * p.win_w - 1)) + (yi - yj + p.win_h - 1) * (2 * p.win_w - 1) + (xi - xj + p.win_w - 1);
  }
  return p.bias_bf16 ? __uint_as_float((uint32_t)((const uint16_t*)p.bias)[off] << 16) : ((const float*)p.bias)[off];
}
// may any pair of the block of 16 queries from q0 and 16 keys from k0 be masked (or lie past the end)?  Uniform.
__device__ inline bool has_edge(const KP& p, const int32_t* rid, int q0, int k0) {
  return rid || q0 + 16 > p.S || k0 + 16 > p.S || (p.mask_kind == 1 && k0 + 15 > q0);
}
// scores of a block in C registers -> scale s + bias, -inf where the pair is masked.  Register v is the
// pair (q, k + v) if KEYS_RUN, else (q + v, k).  `dead` (of a block with an edge): the masked registers.
template <bool KEYS_RUN>
__device__ inline void finish_scores(const KP& p, int h, const int32_t* rid, int q, int k, bool edge, f32x4& s, bool (&dead)[4]) {
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    if (p.bias_kind) s[v] = fmaf(p.scale, s[v], bias_f32(p, h, min(KEYS_RUN ? q : q + v, p.S - 1), min(KEYS_RUN ? k + v : k, p.S - 1)));
    else s[v] *= p.scale;
    dead[v] = false;
  }
  if (edge) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int i = KEYS_RUN ? q : q + v, j = KEYS_RUN ? k + v : k;
      dead[v] = i >= p.S || j >= p.S || (p.mask_kind == 1 && j > i);
      if (rid) dead[v] = dead[v] || rid[min(i, p.S - 1)] != rid[min(j, p.S - 1)];
      s[v] = dead[v] ? -INFINITY : s[v];
    }
  }
}
// masked pairs contribute exactly 0 to the gradients, whatever the statistics are (a query that sees a NaN has NaN
// statistics)
__device__ inline void kill(bool edge, const bool (&dead)[4], f32x4& x) {
  if (edge) {
#pragma unroll
    for (int v = 0; v < 4; ++v) x[v] = dead[v] ? 0.f : x[v];
  }
}

struct Stats { float m[W][16], l[W][16], lse[16], delta[16]; };

// A wavefront's partial result -> LDS; the caller synchronises.
template <int DC>
__device__ inline void put_part(float* buf, int w, int i, int g, const f32x4 (&acc)[DC]) {
  constexpr int LD = 16 * DC + 4;
  float* row = buf + (w * 16 + i) * LD + 4 * DC * g;
  float y[4 * DC];
#pragma unroll
  for (int v = 0; v < 4; ++v)
#pragma unroll
    for (int e = 0; e < DC; ++e) y[DC * v + e] = acc[e][v];
#pragma unroll
  for (int x = 0; x < DC; ++x) *(f32x4*)(row + 4 * x) = f32x4{y[4 * x], y[4 * x + 1], y[4 * x + 2], y[4 * x + 3]};
}

// ---------------------------------------------------------------------------
// Forward (BWD = false), or the backward's recompute pass and dQ.  C blocks: lane = query, registers = keys.
// NB key blocks per wavefront at a time; with one such round (S <= 128 NB) the backward keeps the scores.
// ---------------------------------------------------------------------------
template <int DC, int NB, bool BWD>
__global__ __launch_bounds__(64 * W) void f32_query_kernel(KP p) {
  constexpr int LD = 16 * DC + 4;
  __shared__ __attribute__((aligned(16))) float buf[W * 16 * LD];
  __shared__ __attribute__((aligned(16))) float sdo[BWD ? 16 * LD : 4];
  __shared__ Stats st;
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6), i = lane & 15, g = lane >> 4;
  const int q0 = blockIdx.x * 16, h = p.h0 + blockIdx.y, b = p.b0 + blockIdx.z, q = q0 + i, qc = min(q, p.S - 1);
  const int D = p.D;
  const int64_t base = (int64_t)b * p.sb + (int64_t)h * p.sh;
  const float *K = (const float*)p.K + base, *V = (const float*)p.V + base;
  const int32_t* rid = p.mask_kind == 2 ? p.region + (int64_t)(b % p.mask_period) * p.S : nullptr;
  const int visible = p.mask_kind == 1 ? min(p.S, q0 + 16) : p.S;  // keys that some query of the block sees
  const Nat<DC> qf = load_nat<DC>((const float*)p.Q + base + (int64_t)qc * p.ss, g, D);

  f32x4 s[NB], acc[DC];
  bool dead[NB][4];
  auto scores = [&](int k0) {
#pragma unroll
    for (int t = 0; t < NB; ++t) {
      const int kb = k0 + 16 * (w + W * t);
      s[t] = f32x4{-INFINITY, -INFINITY, -INFINITY, -INFINITY};
      if (kb < visible) {
        s[t] = dot<DC>(load_nat<DC>(K + (int64_t)min(kb + i, p.S - 1) * p.ss, g, D), qf);
        finish_scores<true>(p, h, rid, q, kb + 4 * g, has_edge(p, rid, q0, kb), s[t], dead[t]);
      }
    }
  };
#pragma unroll
  for (int e = 0; e < DC; ++e) acc[e] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m = -INFINITY, l = 0.f;
  for (int k0 = 0; k0 < visible; k0 += 16 * W * NB) {
    scores(k0);
    float mn = -INFINITY;
#pragma unroll
    for (int t = 0; t < NB; ++t)
#pragma unroll
      for (int v = 0; v < 4; ++v) mn = fmaxf(mn, s[t][v]);
    mn = fmaxf(m, over_groups_max(mn));
    const float ref = base_of(mn), alpha = exp_f32(m - ref);
    m = mn;
    l *= alpha;
#pragma unroll
    for (int e = 0; e < DC; ++e) acc[e] *= alpha;
#pragma unroll
    for (int t = 0; t < NB; ++t) {
      const int kb = k0 + 16 * (w + W * t);
      if (kb < visible) {
        f32x4 pr;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          pr[v] = exp_f32(s[t][v] - ref);
          l += pr[v];
        }
        accumulate<DC>(V, p.ss, kb, p.S, i, g, D, pr, acc);
      }
    }
  }
  l = over_groups_sum(l);
  put_part<DC>(buf, w, i, g, acc);
  if (g == 0) { st.m[w][i] = m; st.l[w][i] = l; }
  __syncthreads();

  // merge: 32 threads per query, each columns dl and dl + 32
  const int mq = tid >> 5, dl = tid & 31, row = q0 + mq;
  const bool live = row < p.S;
  const int rc = min(row, p.S - 1);
  float M = st.m[0][mq];
#pragma unroll
  for (int x = 1; x < W; ++x) M = fmaxf(M, st.m[x][mq]);
  float wt[W], L = 0.f;
#pragma unroll
  for (int x = 0; x < W; ++x) {
    wt[x] = exp_f32(st.m[x][mq] - base_of(M));
    L = fmaf(wt[x], st.l[x][mq], L);
  }
  const float inv = 1.f / L, lse = M + logf(L);
  const int64_t at = base + (int64_t)rc * p.ss, lse_at = (int64_t)(b - p.lse_b0) * p.lse_sb + (int64_t)(h - p.lse_h0) * p.lse_sh + rc;
  float part = 0.f;
#pragma unroll
  for (int u = 0; u < (DC + 1) / 2; ++u) {
    const int d = dl + 32 * u;
    if (BWD && d < 16 * DC) sdo[mq * LD + d] = 0.f;
    if (d < D) {
      float o = 0.f;
#pragma unroll
      for (int x = 0; x < W; ++x) o = fmaf(wt[x], buf[(x * 16 + mq) * LD + d], o);
      o *= inv;
      const float gate = p.gated ? 1.f / (1.f + expf(-((const float*)p.G)[at + d])) : 1.f;
      if (!BWD) {
        if (live) ((float*)p.Y)[at + d] = o * gate;
      } else {
        float go = ((const float*)p.dY)[at + d];
        if (p.gated) {
          if (live) ((float*)p.dG)[at + d] = go * o * gate * (1.f - gate);
          go *= gate;
          if (live)
            ((float*)p.dO_out)[(int64_t)(b - p.do_b0) * p.do_sb + (int64_t)rc * p.do_ss + (int64_t)(h - p.do_h0) * p.do_sh + d] = go;
        }
        sdo[mq * LD + d] = go;
        part = fmaf(go, o, part);
      }
    }
  }
  if (!BWD) {
    if (live && dl == 0 && p.lse_out) p.lse_out[lse_at] = lse;
    return;
  }
#pragma unroll
  for (int x = 1; x < 32; x <<= 1) part += __shfl_xor(part, x, 64);
  if (dl == 0) {
    st.lse[mq] = p.lse_out ? lse : p.lse[lse_at];
    st.delta[mq] = part;
    if (live) {
      if (p.lse_out) p.lse_out[lse_at] = lse;
      p.delta[(int64_t)(b - p.dl_b0) * p.dl_sb + (int64_t)(h - p.dl_h0) * p.dl_sh + rc] = part;
    }
  }
  __syncthreads();
  Nat<DC> gf;
#pragma unroll
  for (int c = 0; c < DC; ++c) gf.x[c] = *(const f32x4*)(sdo + i * LD + 16 * c + 4 * g);
  const float my_lse = st.lse[i], my_delta = st.delta[i];
#pragma unroll
  for (int e = 0; e < DC; ++e) acc[e] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int k0 = 0; k0 < visible; k0 += 16 * W * NB) {
    if (visible > 16 * W * NB) scores(k0);
#pragma unroll
    for (int t = 0; t < NB; ++t) {
      const int kb = k0 + 16 * (w + W * t);
      if (kb < visible) {
        f32x4 ds = dot<DC>(load_nat<DC>(V + (int64_t)min(kb + i, p.S - 1) * p.ss, g, D), gf);
#pragma unroll
        for (int v = 0; v < 4; ++v) ds[v] = exp_f32(s[t][v] - my_lse) * (ds[v] - my_delta);
        kill(has_edge(p, rid, q0, kb), dead[t], ds);
        accumulate<DC>(K, p.ss, kb, p.S, i, g, D, ds, acc);
      }
    }
  }
  put_part<DC>(buf, w, i, g, acc);  // the merge above is behind a barrier
  __syncthreads();
#pragma unroll
  for (int u = 0; u < (DC + 1) / 2; ++u) {
    const int d = dl + 32 * u;
    if (live && d < D) {
      float o = 0.f;
#pragma unroll
      for (int x = 0; x < W; ++x) o += buf[(x * 16 + mq) * LD + d];
      ((float*)p.dQ)[at + d] = p.scale * o;
    }
  }
}

// ---------------------------------------------------------------------------
// dK and dV of 16 keys (C blocks: lane = key, registers = queries), and, in the work-groups after those, the
// bias gradient of 16 queries of a head (lane = query, registers = keys), summed over the rows in order.
// ---------------------------------------------------------------------------
template <int DC, int NB>
__global__ __launch_bounds__(64 * W) void f32_key_kernel(KP p) {
  constexpr int LD = 16 * DC + 4;
  __shared__ __attribute__((aligned(16))) float buf[W * 16 * LD];
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6), i = lane & 15, g = lane >> 4;
  const int D = p.D, nblk = (p.S + 15) / 16, Hc = p.h1 - p.h0, nkv = nblk * Hc * (p.b1 - p.b0);
  const int id = blockIdx.x < nkv ? blockIdx.x : blockIdx.x - nkv;
  const int x0 = id % nblk * 16, h = p.h0 + id / nblk % Hc;
  const bool causal = p.mask_kind == 1;

  if (blockIdx.x >= nkv) {
    const int q = x0 + i, qc = min(q, p.S - 1);
    for (int k0 = 0; k0 < p.S; k0 += 16 * W * NB) {
      f32x4 acc[NB];
#pragma unroll
      for (int t = 0; t < NB; ++t)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int k = k0 + 16 * (w + W * t) + 4 * g + v;
          acc[t][v] = p.dbias_accumulate && q < p.S && k < p.S ? p.dbias_acc[((int64_t)h * p.S + q) * p.S + k] : 0.f;
        }
      for (int b = p.b0; b < p.b1; ++b) {
        const int64_t base = (int64_t)b * p.sb + (int64_t)h * p.sh;
        const int32_t* rid = p.mask_kind == 2 ? p.region + (int64_t)(b % p.mask_period) * p.S : nullptr;
        const Nat<DC> qf = load_nat<DC>((const float*)p.Q + base + (int64_t)qc * p.ss, g, D);
        const Nat<DC> gf = load_nat<DC>((const float*)p.dO + (int64_t)(b - p.do_b0) * p.do_sb + (int64_t)qc * p.do_ss +
                                            (int64_t)(h - p.do_h0) * p.do_sh, g, D);
        const float lse = p.lse[(int64_t)(b - p.lse_b0) * p.lse_sb + (int64_t)(h - p.lse_h0) * p.lse_sh + qc];
        const float delta = p.delta[(int64_t)(b - p.dl_b0) * p.dl_sb + (int64_t)(h - p.dl_h0) * p.dl_sh + qc];
#pragma unroll
        for (int t = 0; t < NB; ++t) {
          const int kb = k0 + 16 * (w + W * t);
          if (kb >= p.S || (causal && kb > x0 + 15)) continue;
          const int64_t at = base + (int64_t)min(kb + i, p.S - 1) * p.ss;
          f32x4 s = dot<DC>(load_nat<DC>((const float*)p.K + at, g, D), qf);
          const f32x4 dp = dot<DC>(load_nat<DC>((const float*)p.V + at, g, D), gf);
          const bool edge = has_edge(p, rid, x0, kb);
          bool dead[4];
          finish_scores<true>(p, h, rid, q, kb + 4 * g, edge, s, dead);
#pragma unroll
          for (int v = 0; v < 4; ++v) s[v] = exp_f32(s[v] - lse) * (dp[v] - delta);
          kill(edge, dead, s);
          acc[t] += s;
        }
      }
#pragma unroll
      for (int t = 0; t < NB; ++t)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int k = k0 + 16 * (w + W * t) + 4 * g + v;
          if (q < p.S && k < p.S) p.dbias_acc[((int64_t)h * p.S + q) * p.S + k] = acc[t][v];
        }
    }
    return;
  }

  const int b = p.b0 + id / (nblk * Hc), key = x0 + i, kc = min(key, p.S - 1);
  const int64_t base = (int64_t)b * p.sb + (int64_t)h * p.sh;
  const float* Q = (const float*)p.Q + base;
  const float* G = (const float*)p.dO + (int64_t)(b - p.do_b0) * p.do_sb + (int64_t)(h - p.do_h0) * p.do_sh;
  const float* lse = p.lse + (int64_t)(b - p.lse_b0) * p.lse_sb + (int64_t)(h - p.lse_h0) * p.lse_sh;
  const float* delta = p.delta + (int64_t)(b - p.dl_b0) * p.dl_sb + (int64_t)(h - p.dl_h0) * p.dl_sh;
  const int32_t* rid = p.mask_kind == 2 ? p.region + (int64_t)(b % p.mask_period) * p.S : nullptr;
  const Nat<DC> kf = load_nat<DC>((const float*)p.K + base + (int64_t)kc * p.ss, g, D);
  const Nat<DC> vf = load_nat<DC>((const float*)p.V + base + (int64_t)kc * p.ss, g, D);
  f32x4 dk[DC], dv[DC];
#pragma unroll
  for (int e = 0; e < DC; ++e) dk[e] = dv[e] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int first = causal ? x0 : 0;  // earlier queries see none of these keys
  for (int q0 = first; q0 < p.S; q0 += 16 * W * NB)
#pragma unroll
    for (int t = 0; t < NB; ++t) {
      const int qb = q0 + 16 * (w + W * t), row = min(qb + i, p.S - 1);
      if (qb >= p.S) continue;
      f32x4 s = dot<DC>(load_nat<DC>(Q + (int64_t)row * p.ss, g, D), kf);
      const f32x4 dp = dot<DC>(load_nat<DC>(G + (int64_t)row * p.do_ss, g, D), vf);
      const bool edge = has_edge(p, rid, qb, x0);
      bool dead[4];
      finish_scores<false>(p, h, rid, qb + 4 * g, key, edge, s, dead);
      f32x4 ds;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int r = min(qb + 4 * g + v, p.S - 1);
        s[v] = exp_f32(s[v] - lse[r]);
        ds[v] = s[v] * (dp[v] - delta[r]);
      }
      kill(edge, dead, s);
      kill(edge, dead, ds);
      accumulate<DC>(G, p.do_ss, qb, p.S, i, g, D, s, dv);
      accumulate<DC>(Q, p.ss, qb, p.S, i, g, D, ds, dk);
    }
  const int mk = tid >> 5, dl = tid & 31, out_row = x0 + mk;
#pragma unroll
  for (int which = 0; which < 2; ++which) {
    if (which) __syncthreads();
    put_part<DC>(buf, w, i, g, which ? dk : dv);
    __syncthreads();
    float* out = (float*)(which ? p.dK : p.dV) + base + (int64_t)out_row * p.ss;
#pragma unroll
    for (int u = 0; u < (DC + 1) / 2; ++u) {
      const int d = dl + 32 * u;
      if (out_row < p.S && d < D) {
        float o = 0.f;
#pragma unroll
        for (int x = 0; x < W; ++x) o += buf[(x * 16 + mk) * LD + d];
        out[d] = which ? p.scale * o : o;
      }
    }
  }
}

template <int DC, int NB>
hipError_t run(const KP& p, int what, hipStream_t st) {
  const int nblk = (p.S + 15) / 16, Hc = p.h1 - p.h0, Bc = p.b1 - p.b0;
  if (what == 2) f32_key_kernel<DC, NB><<<nblk * Hc * (Bc + (p.dbias_acc ? 1 : 0)), 64 * W, 0, st>>>(p);
  else if (what == 1) f32_query_kernel<DC, NB, true><<<dim3(nblk, Hc, Bc), 64 * W, 0, st>>>(p);
  else f32_query_kernel<DC, NB, false><<<dim3(nblk, Hc, Bc), 64 * W, 0, st>>>(p);
  return hipGetLastError();
}
template <int DC>
hipError_t run_nb(const KP& p, int what, hipStream_t st) {
  return p.S <= 16 * W ? run<DC, 1>(p, what, st) : p.S <= 32 * W ? run<DC, 2>(p, what, st) : run<DC, 4>(p, what, st);
}
hipError_t run_dc(const KP& p, int what, hipStream_t st) {
  return p.D <= 16 ? run_nb<1>(p, what, st) : p.D <= 32 ? run_nb<2>(p, what, st) : run_nb<4>(p, what, st);
}

}  // namespace

hipError_t launch_f32_fwd(const KP& p, hipStream_t st) { return run_dc(p, 0, st); }
hipError_t launch_f32_recompute_dq(const KP& p, hipStream_t st) { return run_dc(p, 1, st); }
hipError_t launch_f32_dkdv_dbias(const KP& p, hipStream_t st) { return run_dc(p, 2, st); }

}  // namespace ssa

// fade_dev.h — types shared by the HIP translation units of libfade (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "fade_rules.h"

typedef __bf16 bf16_t;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;

// ---------------------------------------------------------------------------------------------------
// exchanges inside a wavefront on the vector ALU (DPP and gfx950's row swaps) instead of through LDS: a ds_bpermute
// butterfly over 64 lanes is six dependent LDS round trips of 60 to 100 cycles, these are one or two instructions a level
// ---------------------------------------------------------------------------------------------------
template <int CTRL, int ROWS = 0xf> __device__ __forceinline__ uint32_t fade_dpp(uint32_t v) {  // lanes without a source give 0
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xf, false);
}
__device__ __forceinline__ uint32_t fade_bits(uint32_t v) { return v; }
__device__ __forceinline__ uint32_t fade_bits(int v) { return (uint32_t)v; }
__device__ __forceinline__ uint32_t fade_bits(float v) { return __builtin_bit_cast(uint32_t, v); }
// One level of a butterfly that starts at the widest distance: op(value of this lane, value of lane ^ D), D = 32 ... 1, for a
// commutative op. Below 16 the value already repeats with period 2 D inside a row of 16 lanes (the wider levels have been
// done), or D is 8, so a rotation of the row by D fetches lane ^ D. Levels of 16 and 32 hold for any value.
template <int D, typename T, typename OP> __device__ __forceinline__ T fade_level(T v, OP op) {
  const uint32_t u = fade_bits(v);
  if constexpr (D >= 16) {
    const auto r = D == 32 ? __builtin_amdgcn_permlane32_swap(u, u, false, false) : __builtin_amdgcn_permlane16_swap(u, u, false, false);
    return op(__builtin_bit_cast(T, (uint32_t)r[0]), __builtin_bit_cast(T, (uint32_t)r[1]));
  } else {
    return op(v, __builtin_bit_cast(T, fade_dpp<0x120 + D>(u)));
  }
}
template <int W = 64, typename T, typename OP> __device__ __forceinline__ T fade_butterfly(T v, OP op) {  // over aligned groups of W lanes
  if constexpr (W >= 64) v = fade_level<32>(v, op);
  if constexpr (W >= 32) v = fade_level<16>(v, op);
  if constexpr (W >= 16) v = fade_level<8>(v, op);
  static_assert(W >= 16, "the levels below a row's 8 rely on it");
  v = fade_level<4>(v, op);
  v = fade_level<2>(v, op);
  return fade_level<1>(v, op);
}
template <int W = 64, typename T> __device__ __forceinline__ T fade_lanes_sum(T v) { return fade_butterfly<W>(v, [](T a, T b) { return a + b; }); }
__device__ __forceinline__ float fade_lanes_max(float v) { return fade_butterfly(v, [](float a, float b) { return fmaxf(a, b); }); }
// Sum over aligned groups of 16 lanes from the nearest neighbours outwards (lane ^ 1, 2, 4, 8): quads first, then mirrored halves of
// the row and the mirrored row, whose groups already hold one value.
__device__ __forceinline__ float fade_row_sum_up(float v) {
  v += __builtin_bit_cast(float, fade_dpp<0xB1>(fade_bits(v)));
  v += __builtin_bit_cast(float, fade_dpp<0x4E>(fade_bits(v)));
  v += __builtin_bit_cast(float, fade_dpp<0x141>(fade_bits(v)));
  return v + __builtin_bit_cast(float, fade_dpp<0x140>(fade_bits(v)));
}
// inclusive prefix sum over the 64 lanes
__device__ __forceinline__ uint32_t fade_lanes_scan(uint32_t v) {
  v += fade_dpp<0x111>(v);  // row_shr 1, 2, 4, 8
  v += fade_dpp<0x112>(v);
  v += fade_dpp<0x114>(v);
  v += fade_dpp<0x118>(v);
  v += fade_dpp<0x142, 0xa>(v);  // last lane of rows 0 and 2 into rows 1 and 3
  v += fade_dpp<0x143, 0xc>(v);  // lane 31 into rows 2 and 3
  return v;
}

// Where the context windows come from: stream b's window is the T bytes ending just before symbol i,
// i.e. base + b * stride + (i - T). n is the total byte count (streams past the end are inactive).
struct WinSrc {
  const uint8_t *base;
  long long stride;        // bytes between consecutive streams
  long long n;             // total bytes (stream b is active at step i iff b * stride + i < n and i < stride)
  const uint8_t *active;   // optional explicit mask [B]; overrides the rule above when non-NULL
  long long i;             // index of the symbol being coded in every stream
};

__device__ __forceinline__ bool stream_active(const WinSrc &w, int b) {
  if (w.active) return w.active[b] != 0;
  const long long i = w.i;
  return i < w.stride && (long long)b * w.stride + i < w.n;
}
__device__ __forceinline__ const uint8_t *stream_window(const WinSrc &w, int b, int T) {
  return w.base + (long long)b * w.stride + (w.i - T);
}

// ---------------------------------------------------------------------------------------------------
// prologue (how the A operand of a product is formed) and epilogue (what happens to the accumulator)
// ---------------------------------------------------------------------------------------------------
enum {
  PRO_PLAIN = 0,   // A[m][k]
  PRO_LN,          // (A[m][k] - mean_m) * rstd_m * gamma[k] + beta[k]          (LN of Eq. 7 / Eq. 9)
  PRO_FINAL,       // psi(LN(A)[m][k]) + lam * A2[m][k]                          (Eq. 10, feeding the head)
  PRO_CONV,        // row (b, j): concat over taps r of XL[b][j-(k-1)+r][:], zero where the index is negative (Eq. 4)
  PRO_CONVT,       // backward of Eq. 4 w.r.t. its input: row (b, j): concat over taps r of dY[b][j+(k-1)-r][:], zero past T-1
};
enum {
  EPI_STORE = 0,   // C = acc                                   (+ optional row statistics for a following LN)
  EPI_STORE_F32,   // C (fp32) = acc + bias
  EPI_GLOBAL,      // C = psi(acc) + lam * S1                   (Eq. 3; S1 = X)
  EPI_MIX,         // a = sigma(acc); C = a*S1 + (1-a)*S2       (Eq. 5-6; S1 = H_global, S2 = H_local)
  EPI_GATE,        // s = sigma(acc); C = S1*s + lam*S2         (Eq. 8; S1 = H_a, S2 = H_mix)
  EPI_GEGLU,       // C = psi(acc_gate) * acc_value             (Eq. 9; gate/value interleaved per 128 columns)
  EPI_CONV,        // C = psi(acc + bias[n])                    (Eq. 4)
  EPI_PARTIAL,     // C (fp32)[split][M][N] = acc of this block's K range (summed later in split order)
  EPI_GRAD,        // C (fp32) = acc: a weight gradient; with C3 set, columns interleaved per 128 go to the pair (C, C3)
  EPI_GEGLU_FOLD,  // EPI_GEGLU on a product of raw activations: the LayerNorm folded into W is finished here, per row
                   // (statistics of A) and per column (fold_s, fold_t), then C = psi(gate) * value; C2 / C3 = gate / value
};

// LN(h) W = rstd * (h W' - mean * s) + t for one output element (raw = h W'); one spelling for every kernel that finishes
// a folded LayerNorm, so that they agree to the bit.
__device__ __forceinline__ float fade_fold_ln(float raw, float mean, float rstd, float s, float t) {
  return fmaf(rstd, fmaf(-mean, s, raw), t);
}

struct GemmArgs {
  int M, N, K;            // C[M][N] = A'[M][K] * W[K][N]
  int splits;             // EPI_PARTIAL: number of K ranges (grid.y); 0 or 1 otherwise
  int sum_splits;         // EPI_PARTIAL, pipelined kernel: one workgroup takes all ranges in turn and writes the sum of their
                          // sums (added in range order) as the only partial
  // A operand
  const void *A;  int lda;
  int a_rows;             // row-major weight-gradient product: rows of A that exist (rows up to K are clamped to the last one)
  const void *A2;         // PRO_FINAL: residual source (same leading dimension)
  const float *stats;     // PRO_LN / PRO_FINAL: [M][stats_n][2] partial (sum, sum of squares) of A's rows
  int stats_n;
  const float *gamma, *beta;
  const float *lam;       // device scalar used by PRO_FINAL / EPI_GLOBAL / EPI_GATE
  int T, D, taps;         // PRO_CONV geometry
  // B operand: bf16 fragments in MFMA order (bf16 path) or plain fp32 [K][N] (fp32 path)
  const void *W;
  int ldb;                // pipelined kernel with a row-major B operand ([N][ldb], K contiguous); fp32 kernel with wt != 0
  int wt;                 // fp32 kernel: W is given transposed ([N][ldb]) instead of [K][N]
  // output
  void *C;  int ldc;
  void *C2, *C3;          // optional copies of pre-activation values for the backward pass
  const void *S1, *S2;    // side inputs [M][N] (leading dimension ldc)
  const float *bias;
  float *stats_out;       // optional [M][N / BN][2]
  const float *fold_s, *fold_t;  // EPI_GEGLU_FOLD: the folded LayerNorm's column vectors [N] (stats / stats_n: rows of A)
  int weight;             // weight gradient: index of the parameter + 1 (0: not one)
  int col_groups;         // pipelined kernel: column ranges of the XCD split of the tile grid (1, 2, 4, 8; 0 = chosen by the launcher)
};

// A grouped launch: up to 4 independent products, each with the kernel body named by kind[]; blocks [first_block[p],
// first_block[p + 1]) work on problem p (tiles[p] output tiles x splits[p] ranges of K).
enum { GK_STORE_64x128 = 0, GK_STORE_64x64, GK_STORE_128x128, GK_PARTIAL_64x64, GK_PARTIAL_128x128, GK_TN_64x128, GK_TN_128x128, GK_TN_64x64 };
struct GemmGroup {
  int count;
  int kind[4], tiles[4], splits[4], first_block[5];
  GemmArgs g[4];
};

// Weight gradients on 256 x 256 tiles of several matrices in ONE launch (gemm_tn2_kernel). A weight gradient feeds nothing but the
// optimiser, so the products of a whole backward pass can wait for its end. order[i]: the i-th piece, one of `ranges` equal
// ranges of the batch for one tile; the plan (whose tiles are these pieces) says which workgroup works on which rows of which.
struct Tn2Piece {
  uint32_t at;     // product << 28 | range << 24 | row tile << 12 | column tile
  uint32_t slice;  // of the product's partial sums: the piece's first one
};
struct Tn2Group {
  int count, pieces, ranges;
  FadeTilePlan plan;
  const Tn2Piece *order;
  GemmArgs g[8];
};

// 16 bytes that are not worth a place in the caches (nt loads and stores): what is read for the last time, or written and not
// read again before more has passed than the 256 MB Infinity Cache holds. An adapting step at B = 1024 moves 360 MB of weights and
// moments between any two uses of an operand; kept out of the cache they leave the step's 45 MB of bf16 operand copies and its
// activations there. Step of configurations B = 1024 / 4096 (D_cache 4096, D_e 8192) / 16384: 438 / 1168 / 2766 us with plain
// accesses, 422 / 1148 / 2724 with nt on the optimiser's state, 394-413 / 1126 / 2677 with the backward pass's operands too.
// The optimiser's state follows a rule on sizes (fade_streamed). What only the backward pass reads is nt in the bf16 path at every
// batch, one instance of each kernel: where everything fits it costs half a percent (step in us with plain accesses and with nt:
// D_h = 256, B = 16 / 128 / 512 150.4 -> 151.6, 162.9 -> 164.3, 181.3 -> 183.5; D_h = 512, B = 128 / 512 185.7 -> 186.9, 209.1 -> 210.3;
// D_h = 2048, B = 128 / 512 275.3 -> 277.4, 329.2 -> 330.0) against 3 to 5 % gained from there on (D_h = 2048, B = 768 / 1024
// 377 -> 361, 419 -> 400; D_h = 1024, B = 2048 384 -> 374). The fp32 path's accesses are plain: 300 streams of D_h = 2048 lost 2 %.
__device__ __forceinline__ f32x4 fade_nt_load(const void *p) { return __builtin_nontemporal_load(static_cast<const f32x4 *>(p)); }
__device__ __forceinline__ void fade_nt_store(void *p, f32x4 v) { __builtin_nontemporal_store(v, static_cast<f32x4 *>(p)); }
template <bool NT> __device__ __forceinline__ f32x4 fade_load4(const float *p) {
  if constexpr (NT) return fade_nt_load(p);
  else return *reinterpret_cast<const f32x4 *>(p);
}
template <bool NT> __device__ __forceinline__ void fade_store4(float *p, f32x4 v) {
  if constexpr (NT) fade_nt_store(p, v);
  else *reinterpret_cast<f32x4 *>(p) = v;
}
// Row statistics are accumulated per block tile of BN columns; consumers add the partials in index order.
#define FADE_STATS_BN 128

// Sum and sum of squares of a row of `width` -> mean and 1 / sigma (biased variance, eps 1e-5). Explicit product and fused
// multiply-add: this is inlined into many kernels whose results must agree bit for bit, which must not depend on which of the
// two products the compiler fuses with the subtraction.
__device__ __forceinline__ void fade_moments_of(float s, float q, int width, float &mean, float &rstd) {
  const float inv = 1.0f / (float)width;
  mean = s * inv;
  rstd = 1.0f / sqrtf(fmaxf(fmaf(q, inv, -__fmul_rn(mean, mean)), 0.0f) + 1e-5f);
}
// The same from a row's (sum, sum of squares) partials. The pairs are fetched 16 at
// a time with no add between the loads (a loop of load-add-load-add would pay the memory latency once per pair); the adds
// run in index order, slots past stats_n add an exact zero.
__device__ __forceinline__ void fade_row_moments(const float *stats, int stats_n, int width, float &mean, float &rstd) {
  const float2 *p = reinterpret_cast<const float2 *>(stats);
  float s = 0.0f, q = 0.0f;
  for (int j0 = 0; j0 < stats_n; j0 += 16) {
    float2 v[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const int idx = j0 + j;
      v[j] = p[idx < stats_n ? idx : stats_n - 1];
    }
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const bool in = j0 + j < stats_n;
      s += in ? v[j].x : 0.0f;
      q += in ? v[j].y : 0.0f;
    }
  }
  fade_moments_of(s, q, width, mean, rstd);
}

// The same, bit for bit, for W = 8 or 16 neighbouring lanes that work on one row: the pairs come with 16 / W loads per lane
// (every lane used to fetch all 16, beside the 3 to 12 loads of a row kernel's data), and are added in index order as
// broadcasts inside the row of 16 lanes.
template <int J> __device__ __forceinline__ float fade_row_bcast(float v, int half) {  // lane J of the row; half 0 / 1: into lanes 0-7 / 8-15 only (zero elsewhere)
  const int u = (int)fade_bits(v);
  if (half < 0) return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, u, 0x150 + J, 0xf, 0xf, false));
  return half == 0 ? __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, u, 0x150 + J, 0xf, 0x3, false))
                   : __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, u, 0x150 + J, 0xf, 0xc, false));
}
template <int W, int J, int END> __device__ __forceinline__ void fade_add_pairs(const float2 &v, float &s, float &q) {
  if constexpr (J < END) {
    if constexpr (W == 16) {
      s += fade_row_bcast<J>(v.x, -1);
      q += fade_row_bcast<J>(v.y, -1);
    } else {
      s = (s + fade_row_bcast<J>(v.x, 0)) + fade_row_bcast<8 + J>(v.x, 1);
      q = (q + fade_row_bcast<J>(v.y, 0)) + fade_row_bcast<8 + J>(v.y, 1);
    }
    fade_add_pairs<W, J + 1, END>(v, s, q);
  }
}
template <int W> __device__ __forceinline__ void fade_row_moments_lanes(const float *stats, int stats_n, int width, float &mean, float &rstd) {
  static_assert(W == 8 || W == 16, "lanes per row");
  const float2 *p = reinterpret_cast<const float2 *>(stats);
  const int l = threadIdx.x & (W - 1);
  float s = 0.0f, q = 0.0f;
  for (int j0 = 0; j0 < stats_n; j0 += 16) {
    float2 v[16 / W];
#pragma unroll
    for (int i = 0; i < 16 / W; ++i) {
      const int j = j0 + i * W + l;
      v[i] = p[j < stats_n ? j : 0];
      if (j >= stats_n) v[i] = make_float2(0.0f, 0.0f);
    }
    const int left = stats_n - j0;  // pairs past the last are zeros; a short row skips most of them
    if constexpr (W == 16) {
      fade_add_pairs<16, 0, 4>(v[0], s, q);
      if (left > 4) fade_add_pairs<16, 4, 16>(v[0], s, q);
    } else {
      fade_add_pairs<8, 0, 4>(v[0], s, q);
      if (left > 4) fade_add_pairs<8, 4, 8>(v[0], s, q);
      if (left > 8) fade_add_pairs<8, 0, 8>(v[1], s, q);
    }
  }
  fade_moments_of(s, q, width, mean, rstd);
}

// Row-wise element kernels: thread t = blockIdx.x * 256 + tid owns the 8-wide chunk t % chunks of the RPT rows of row
// group t / chunks (RPT = 4 for tall inputs: one fetch of the per-column vectors serves 4 rows, whose loads are in flight
// together; RPT = 1 when there are too few rows to fill the chip that way). The moments of the rows a workgroup covers
// are formed once per row and shared through LDS instead of once per thread. mom must hold RPT * (256 / chunks + 2)
// rows (chunks >= 8: at most FADE_GROUP_ROWS_MAX). Returns the workgroup's first row; ends with a barrier.
#define FADE_GROUP_ROWS_MAX 136
template <int RPT>
__device__ __forceinline__ int fade_group_moments(const float *stats, int stats_n, int width, int chunks, int rows, float (*mom)[2]) {
  const long long t0 = (long long)blockIdx.x * 256;
  const int g0 = (int)(t0 / chunks), g1 = (int)((t0 + 255) / chunks);
  const int r0 = g0 * RPT, nr = (g1 - g0 + 1) * RPT;
  for (int r = threadIdx.x >> 4; r < nr; r += 16)
    if (r0 + r < rows) {
      float mean, rstd;
      fade_row_moments_lanes<16>(stats + (size_t)(r0 + r) * stats_n * 2, stats_n, width, mean, rstd);
      if ((threadIdx.x & 15) == 0) { mom[r][0] = mean; mom[r][1] = rstd; }
    }
  __syncthreads();
  return r0;
}
// rows per thread for `rows` rows of `chunks` chunks: 4 once that still leaves four workgroups for every compute unit
inline int fade_rows_per_thread(long long rows, int chunks) { return (rows / 4) * chunks / 256 >= 1024 ? 4 : 1; }

// ---------------------------------------------------------------------------------------------------
// activation arithmetic shared by every kernel (encoder and decoder run the same code, so they agree bit for bit)
// ---------------------------------------------------------------------------------------------------
// erf by the rational-times-Gaussian formula 7.1.26 of Abramowitz & Stegun (|error| <= 1.5e-7 absolute): the row kernels
// run one wavefront per SIMD and were bound by the library erff + expf (over a hundred instructions per element).
// The Gaussian e = exp(-x^2) is passed in because GeLU's derivative needs the same exponential.
__device__ __forceinline__ float fade_exp(float x) { return __builtin_amdgcn_exp2f(x * 1.4426950408889634f); }
__device__ __forceinline__ float fade_erf_pos(float ax, float e) {  // ax >= 0, e = exp(-ax^2)
  const float t = __builtin_amdgcn_rcpf(fmaf(0.3275911f, ax, 1.0f));
  float p = fmaf(1.061405429f, t, -1.453152027f);
  p = fmaf(p, t, 1.421413741f);
  p = fmaf(p, t, -0.284496736f);
  p = fmaf(p, t, 0.254829592f);
  return fmaf(-p * t, e, 1.0f);
}
// Phi(x) = (1 + erf(x / sqrt 2)) / 2 and the Gaussian g = exp(-x^2 / 2)
__device__ __forceinline__ float fade_norm_cdf(float x, float &g) {
  const float ax = fabsf(x) * 0.70710678118654752f;
  g = fade_exp(-ax * ax);
  const float er = fade_erf_pos(ax, g);
  return 0.5f * (1.0f + copysignf(er, x));
}
__device__ __forceinline__ float fade_gelu(float x) {  // psi(x) = x Phi(x) (exact-erf GeLU)
  float g;
  return x * fade_norm_cdf(x, g);
}
__device__ __forceinline__ float fade_gelu_grad(float x) {  // psi'(x) = Phi(x) + x phi(x)
  float g;
  const float cdf = fade_norm_cdf(x, g);
  return fmaf(x * 0.3989422804014327f, g, cdf);
}
// psi(x) and psi'(x) from one evaluation of Phi and the Gaussian
__device__ __forceinline__ float fade_gelu_both(float x, float &grad) {
  float g;
  const float cdf = fade_norm_cdf(x, g);
  grad = fmaf(x * 0.3989422804014327f, g, cdf);
  return x * cdf;
}
__device__ __forceinline__ float fade_sigmoid(float x) { return __builtin_amdgcn_rcpf(1.0f + fade_exp(-x)); }

// fade_rows.hip — the fp32 path at small batches (up to 256 streams, D_h, D_cache, D_e <= 2048; `rows16` contexts).
//
// At 16 streams every product of the step is a chain of latencies: a launch, one round trip for the operands, a sum, the
// epilogue. Bytes and flops are nothing (4 MB of weights, 17 Mflop). What these kernels do about it:
//   * products on the matrix cores in fp32 (v_mfma_f32_16x16x4_f32, exact fp32 multiply-add): a workgroup is one 16 x 16
//     tile, its eight wavefronts split K in blocks of 16, everything a wavefront reads (operand rows, weights, LayerNorm
//     vectors, row statistics) is requested in one go, and the eight partial tiles are added in wavefront order through LDS.
//     Within a block of 16 the k index is permuted (lane group g takes k = 4 g .. 4 g + 3 over the four instructions) so that
//     rows are read in 16-byte pieces.
//   * products that meet in one epilogue share a launch: Eq. 3 with Eq. 5-6, Up with Eq. 8; the loss gradient is formed
//     in the operand load of the head's activation gradient, GeGLU's backward in the epilogue of its product; independent
//     work of one stage is tiles of one grid.
//   * weight gradients and Adam are one launch for all matrices: a wavefront contracts the batch for a 16 x 64 strip from the
//     row-major activations (no transposed copies) and steps the weights it just formed the gradient of.
// A step at 16 streams (T = 32, D = 16, H = 128), kernel time: forward 12 launches, 79 us -> 9 launches, 41 us; with the update
// 46 launches, 300 us -> 24 launches, 117 us.
// Row statistics are left per 16 columns (stats_n = N / 16). Every sum has a fixed order.
#include "fade_dev.h"
#include "fade_kernels.h"
#include "fade_rules.h"

namespace {

constexpr int NW = 8, NTH = NW * 64;
enum { A_PLAIN, A_LN, A_FINAL, A_LOSS, A_CONV, A_CONVT };                                       // how operand rows are formed
enum { W_KN, W_NK, W_NK_PAIR, W_NK_CONV };                                                      // how the weights lie
enum { E_STORE, E_BIAS, E_GLOBAL, E_MIX, E_GATE, E_GEGLU, E_CONV, E_DGEGLU };                  // what happens to the sums

__device__ __forceinline__ f32x4 ld4(const float *p) { return *reinterpret_cast<const f32x4 *>(p); }
__device__ __forceinline__ void st4(float *p, const f32x4 &v) { *reinterpret_cast<f32x4 *>(p) = v; }
__device__ __forceinline__ int wave_id() { return __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)); }

// LayerNorm of the operand rows: gains, shifts and the tile's moments in LDS. What a compute unit issues to memory is what
// bounds these kernels (a wavefront's load instruction takes some 16 cycles whatever it fetches), and per lane and wavefront
// the vectors and the partial statistics would be 16 of 36 instructions; here they are 3. Wavefront w sums rows 2 w, 2 w + 1.
struct NormShared {
  float ga[2048], be[2048];  // D_h <= 2048
  float2 mom[16];
};
struct NormLoad {
  float2 v;
  float g[4], b[4];
  __device__ __forceinline__ void load(const RowsArgs &a, int m0) {
    const int tid = threadIdx.x, lane = tid & 63, row = m0 + wave_id() * 2 + (lane >> 5);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (i * NTH < a.width) {  // uniform
        const int k = i * NTH + tid < a.width ? i * NTH + tid : 0;
        g[i] = a.gamma[k]; b[i] = a.beta[k];
      }
    }
    v = pair(a, row, lane & 31);
  }
  static __device__ __forceinline__ float2 pair(const RowsArgs &a, int row, int j) {
    float2 x = reinterpret_cast<const float2 *>(a.stats)[(size_t)(row < a.M ? row : a.M - 1) * a.stats_n + (j < a.stats_n ? j : 0)];
    if (j >= a.stats_n) x = make_float2(0.0f, 0.0f);
    return x;
  }
  __device__ __forceinline__ void finish(const RowsArgs &a, int m0, bool first, NormShared &sh) {
    const int tid = threadIdx.x, lane = tid & 63, r = wave_id() * 2 + (lane >> 5);
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (i * NTH + tid < a.width) { sh.ga[i * NTH + tid] = g[i]; sh.be[i * NTH + tid] = b[i]; }
    float s = v.x, q = v.y;
    for (int j = 32 + (lane & 31); j - (lane & 31) < a.stats_n; j += 32) {  // rows of more than 512
      const float2 x = pair(a, m0 + r, j);
      s += x.x; q += x.y;
    }
    s = fade_lanes_sum<32>(s);
    q = fade_lanes_sum<32>(q);
    float2 m;
    fade_moments_of(s, q, a.width, m.x, m.y);
    if ((lane & 31) == 0) {
      sh.mom[r] = m;
      if (first && a.mom_out && m0 + r < a.M) reinterpret_cast<float2 *>(a.mom_out)[m0 + r] = m;
    }
    __syncthreads();
  }
};

struct RowCtx {
  int m;              // this lane's operand row, clamped into the matrix
  bool live;          // it exists
  float mean, rstd;   // A_LN, A_FINAL
  const NormShared *norm;
  float sc;           // A_LOSS: 1 / active streams
  int x;              // A_LOSS: target of the row, -1: inactive
  bool first;         // this workgroup also writes what is formed on the fly
};

// Requested pieces of one 16-wide k block: lane group g holds k = 16 kb + 4 g .. + 3 of its row and the weights of those k.
template <int PRO> struct Piece {
  f32x4 a, a2, w;
};
template <int PRO, int WL>
__device__ __forceinline__ void request(const RowsArgs &a, const RowsOp &o, const RowCtx &rc, int col, int k, Piece<PRO> &p) {
  if constexpr (PRO == A_CONV) {  // row (b, j): the taps' tokens of the window, from the per-symbol table
    const int b = rc.m / a.T, j = rc.m - b * a.T, tap = k / a.D, i = k - tap * a.D, tok = j - (a.taps - 1) + tap;
    const int s = stream_active(a.ws, b) ? (int)stream_window(a.ws, b, a.T)[tok >= 0 ? tok : 0] : 0;  // the window of a stream that has ended may not exist
    p.a = ld4(a.tabXl + (size_t)s * a.D + i);
    if (tok < 0) p.a = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  } else if constexpr (PRO == A_CONVT) {  // row (b, j): dY[j + (taps - 1) - tap], zero past the window
    const int b = rc.m / a.T, j = rc.m - b * a.T, tap = k / a.D, i = k - tap * a.D, tok = j + (a.taps - 1) - tap;
    p.a = ld4(o.A + ((size_t)b * a.T + (tok < a.T ? tok : j)) * a.D + i);
    if (tok >= a.T) p.a = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  } else {
    p.a = ld4(o.A + (size_t)rc.m * o.lda + k);
  }
  if constexpr (PRO == A_FINAL) p.a2 = ld4(o.A2 + (size_t)rc.m * o.lda + k);
  if constexpr (WL == W_KN) {
#pragma unroll
    for (int j = 0; j < 4; ++j) p.w[j] = o.W[(size_t)(k + j) * o.ldw + col];
  } else if constexpr (WL == W_NK) {
    p.w = ld4(o.W + (size_t)col * o.ldw + k);
  } else if constexpr (WL == W_NK_PAIR) {  // the contraction runs through W's columns, then W2's
    p.w = ld4(k < o.ldw ? o.W + (size_t)col * o.ldw + k : o.W2 + (size_t)col * o.ldw + (k - o.ldw));
  } else {  // W_conv [taps][D][D] with k = (tap, output channel)
    const int tap = k / a.D, c = k - tap * a.D;
    p.w = ld4(o.W + ((size_t)tap * a.D + col) * a.D + c);
  }
}
template <int PRO>
__device__ __forceinline__ f32x4 form(const RowsArgs &a, const RowsOp &o, const RowCtx &rc, int k, const Piece<PRO> &p, float lam) {
  f32x4 v = p.a;
  if constexpr (PRO == A_LN || PRO == A_FINAL) {
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = fmaf(__fmul_rn(v[j] - rc.mean, rc.rstd), rc.norm->ga[k + j], rc.norm->be[k + j]);
  }
  if constexpr (PRO == A_FINAL) {
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = fmaf(lam, p.a2[j], fade_gelu(v[j]));
    if (rc.first && a.keep && rc.live) st4(a.keep + (size_t)rc.m * o.lda + k, v);
  }
  if constexpr (PRO == A_LOSS) {
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = rc.x >= 0 ? rc.sc * (v[j] - (k + j == rc.x ? 1.0f : 0.0f)) : 0.0f;
    if (rc.first) {
      if (rc.live) st4(a.keep + (size_t)rc.m * o.lda + k, v);
      f32x4 c;
#pragma unroll
      for (int j = 0; j < 4; ++j) c[j] = fade_lanes_sum<16>(v[j]);
      if ((threadIdx.x & 15) == 0) st4(a.col_part + k, c);
    }
  }
  return v;
}
// This wavefront's share of sum_k A[row][k] W[k][col] over the tile: K blocks wave, wave + 8, ... in batches of U. start() requests
// the first batch (all of it up to K = 512), finish() works through it and the rest.
template <int PRO, int WL> struct Contraction {
  static constexpr int U = 4;
  Piece<PRO> p[U];
  __device__ __forceinline__ void batch(const RowsArgs &a, const RowsOp &o, const RowCtx &rc, int col, int kb0) {
    const int nkb = o.K / 16, g4 = ((threadIdx.x >> 4) & 3) * 4;
    if (kb0 < nkb) {
#pragma unroll
      for (int u = 0; u < U; ++u) request<PRO, WL>(a, o, rc, col, (kb0 + u * NW < nkb ? kb0 + u * NW : kb0) * 16 + g4, p[u]);
    }
  }
  __device__ __forceinline__ void start(const RowsArgs &a, const RowsOp &o, const RowCtx &rc, int col) { batch(a, o, rc, col, wave_id()); }
  __device__ __forceinline__ f32x4 finish(const RowsArgs &a, const RowsOp &o, const RowCtx &rc, int col) {
    const int nkb = o.K / 16, g4 = ((threadIdx.x >> 4) & 3) * 4, w = wave_id();
    float lam = 0.0f;
    if (PRO == A_FINAL) lam = a.lam[0];
    f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int kb0 = w; kb0 < nkb; kb0 += NW * U) {
      if (kb0 != w) batch(a, o, rc, col, kb0);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (kb0 + u * NW < nkb) {
          const f32x4 v = form<PRO>(a, o, rc, (kb0 + u * NW) * 16 + g4, p[u], lam);
#pragma unroll
          for (int j = 0; j < 4; ++j) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(v[j], p[u].w[j], acc, 0, 0, 0);
        }
      }
    }
    return acc;
  }
};

// One 16 x 16 tile of C. TWO: a second product (op1) over the same tile, which the epilogue combines with the first.
template <int PRO, int WL, int EPI, bool TWO = false>
__device__ __forceinline__ void tile(RowsArgs a, int mt, int nt, float *red /*[(TWO ? 2 : 1) * NW * 256]*/) {
  const int tid = threadIdx.x, lane = tid & 63, wave = wave_id(), r = lane & 15;
  const int m0 = mt * 16;
  // columns of the tile: 16 neighbours; for GeGLU 8 of the gate and the same 8 of the value matrix
  int col = nt * 16 + r;
  RowsOp o0 = a.op0;
  if constexpr (EPI == E_GEGLU) {
    col = nt * 8 + (r & 7);
    if (r >= 8) o0.W = o0.W2;
  }
  const int colc = col < a.N ? col : a.N - 1;
  RowCtx rc{};
  rc.live = m0 + r < a.M;
  rc.m = rc.live ? m0 + r : a.M - 1;
  rc.first = nt == 0;
  // one round trip: row statistics, side inputs of the epilogue (thread = one output), operands of both products
  constexpr bool kNorm = PRO == A_LN || PRO == A_FINAL;
  NormLoad nl;
  if constexpr (kNorm) nl.load(a, m0);
  const int em = m0 + (tid >> 4), ec = (EPI == E_GEGLU ? nt * 8 + (tid & 7) : nt * 16 + (tid & 15));
  const bool mine = tid < 256 && em < a.M && ec < a.N;
  const size_t eo = (size_t)(mine ? em : 0) * a.ldc + (mine ? ec : 0), es = (size_t)(mine ? em : 0) * a.lds + (mine ? ec : 0);
  float s1 = 0.0f, s2 = 0.0f, bi = 0.0f, lam = 0.0f;
  if constexpr (EPI == E_GLOBAL || EPI == E_MIX || EPI == E_DGEGLU) s1 = a.S1[es];
  if constexpr (EPI == E_MIX || EPI == E_GATE || EPI == E_DGEGLU) s2 = a.S2[es];
  if constexpr (EPI == E_BIAS || EPI == E_CONV) bi = a.bias[mine ? ec : 0];
  if constexpr (EPI == E_GLOBAL || EPI == E_MIX || EPI == E_GATE) lam = a.lam[0];
  Contraction<PRO, WL> c0;
  Contraction<A_PLAIN, W_KN> c1;
  c0.start(a, o0, rc, colc);
  if constexpr (TWO) c1.start(a, a.op1, rc, colc);
  if constexpr (kNorm) {
    __shared__ NormShared norm;
    nl.finish(a, m0, rc.first, norm);
    rc.mean = norm.mom[r].x; rc.rstd = norm.mom[r].y; rc.norm = &norm;
  }
  if constexpr (PRO == A_LOSS) {
    const int na = __syncthreads_count(tid < a.M && stream_active(a.ws, tid));
    rc.sc = na > 0 ? 1.0f / (float)na : 0.0f;
    rc.x = rc.live && stream_active(a.ws, rc.m) ? (int)a.targets[(long long)rc.m * a.tstride] : -1;
    a.col_part += (size_t)mt * 256;
    if (rc.first && mt == 0 && tid == 0) {  // Adam's step count and bias corrections, for the kernels that follow
      a.u->na = na;
      if (na > 0) {
        a.u->t += 1;
        a.u->c1 = 1.0f - powf(a.beta1, (float)a.u->t);
        a.u->c2 = 1.0f - powf(a.beta2, (float)a.u->t);
        a.u->inv_na = rc.sc;
      }
    }
  }
  {  // lane l holds column l & 15, rows 4 (l >> 4) + e
    const f32x4 acc = c0.finish(a, o0, rc, colc);
#pragma unroll
    for (int e = 0; e < 4; ++e) red[wave * 256 + ((lane >> 4) * 4 + e) * 16 + r] = acc[e];
  }
  if constexpr (TWO) {
    const f32x4 acc = c1.finish(a, a.op1, rc, colc);
#pragma unroll
    for (int e = 0; e < 4; ++e) red[(NW + wave) * 256 + ((lane >> 4) * 4 + e) * 16 + r] = acc[e];
  }
  __syncthreads();
  if (tid >= 256) return;
  float x = red[tid], y = 0.0f;
#pragma unroll
  for (int w = 1; w < NW; ++w) x += red[w * 256 + tid];
  if constexpr (TWO) {
    y = red[NW * 256 + tid];
#pragma unroll
    for (int w = 1; w < NW; ++w) y += red[(NW + w) * 256 + tid];
  }
  float out = x;
  if constexpr (EPI == E_BIAS) out = x + bi;
  if constexpr (EPI == E_GLOBAL || EPI == E_MIX) out = fmaf(lam, s1, fade_gelu(x));  // H_global
  if constexpr (EPI == E_GLOBAL) {
    if (mine && a.C3) a.C3[eo] = x;
  }
  if constexpr (EPI == E_MIX) {
    const float al = fade_sigmoid(y), hg = out;
    out = fmaf(al, hg, __fmul_rn(1.0f - al, s2));
    if (mine) {
      a.C4[eo] = hg;
      if (a.C2) { a.C2[eo] = al; a.C3[eo] = x; }
    }
  }
  if constexpr (EPI == E_GATE) {
    const float sg = fade_sigmoid(y);
    out = fmaf(lam, s2, __fmul_rn(x, sg));
    if (mine) {
      a.C4[eo] = x;  // H_a
      if (a.C2) a.C2[eo] = sg;
    }
  }
  if constexpr (EPI == E_GEGLU) {
    const float v = __builtin_bit_cast(float, fade_dpp<0x128>(fade_bits(x)));  // value column: eight lanes on
    out = fade_gelu(x) * v;
    if ((tid & 15) >= 8) return;
    if (mine && a.C2) { a.C2[eo] = x; a.C3[eo] = v; }
  }
  if constexpr (EPI == E_CONV) {
    const float pre = x + bi;
    out = fade_gelu(pre);
    if (mine && a.C2) a.C2[eo] = pre;
  }
  if constexpr (EPI == E_DGEGLU) {  // s1 gate, s2 value: [gradient of the gate | of the value]
    float grad;
    const float psi = fade_gelu_both(s1, grad);
    if (mine) { a.C[eo] = x * s2 * grad; a.C[eo + a.N] = x * psi; }
    return;
  }
  if (mine) a.C[eo] = out;
  if constexpr (EPI == E_STORE || EPI == E_MIX || EPI == E_GATE) {
    if (a.stats_out) {
      const float sv = mine ? out : 0.0f;
      const float s = fade_lanes_sum<16>(sv), q = fade_lanes_sum<16>(sv * sv);
      if ((tid & 15) == 0 && em < a.M) *reinterpret_cast<float2 *>(a.stats_out + ((size_t)em * (a.N / 16) + nt) * 2) = make_float2(s, q);
    }
  }
}
template <int PRO, int WL, int EPI, bool TWO>
__global__ __launch_bounds__(NTH) void rows_kernel(RowsArgs a) {
  __shared__ float red[(TWO ? 2 : 1) * NW * 256];
  tile<PRO, WL, EPI, TWO>(a, blockIdx.y, blockIdx.x, red);
}

// ---------------------------------------------------------------------------------------------------
// The window of one step: X, X_l, the rolled cache and its new slot (one workgroup per stream), and Eq. 4 as tiles of the
// [B T][D] product whose operand comes from the window and the per-symbol table: independent, one grid.
// ---------------------------------------------------------------------------------------------------
__device__ __forceinline__ void window_stream(const RowsWindowArgs &a, int b) {
  const int tid = threadIdx.x;
  const uint8_t *win = stream_window(a.ws, b, a.T);
  if (a.win_copy && tid < a.T) a.win_copy[(size_t)b * a.T + tid] = win[tid];
  if (!stream_active(a.ws, b)) return;
  float *X = a.X + (size_t)b * a.Dh, *XL = a.XL ? a.XL + (size_t)b * a.Dh : nullptr, *M = a.M + (size_t)b * a.Dc;
  const int s = win[a.T - 1], q = tid < a.c ? tid : 0;
  const float gg = a.gg_tab[(size_t)s * a.c + q], gv = a.gv_tab[(size_t)s * a.c + q];
  float keep[4];  // D_cache <= 2048
#pragma unroll
  for (int i = 0; i < 4; ++i) keep[i] = M[i * NTH + tid < a.Dc ? i * NTH + tid : 0];
  for (int e = tid * 4; e < a.Dh; e += NTH * 4) {
    const int j = e / a.D, i = e - j * a.D, sy = win[j];
    st4(X + e, ld4(a.tabXe + (size_t)sy * a.D + i));
    if (XL) st4(XL + e, ld4(a.tabXl + (size_t)sy * a.D + i));
  }
  __syncthreads();  // the row is in registers: shift it left by one slot (Eq. 2) and append Eq. 1's GeGLU of the newest symbol
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int idx = i * NTH + tid;
    if (idx < a.Dc && idx >= a.c) M[idx - a.c] = keep[i];
  }
  if (tid < a.c) {
    M[a.Dc - a.c + tid] = fade_gelu(gg) * gv;
    if (a.GG) { a.GG[(size_t)b * a.c + tid] = gg; a.GV[(size_t)b * a.c + tid] = gv; }
  }
}
__global__ __launch_bounds__(NTH) void rows_window_kernel(RowsWindowArgs a, RowsArgs conv) {
  __shared__ float red[NW * 256];
  const int b = blockIdx.x, ntn = conv.N / 16;
  if (b < a.B) window_stream(a, b);
  else tile<A_CONV, W_KN, E_CONV>(conv, (b - a.B) / ntn, (b - a.B) % ntn, red);
}

// Eq. 7's per-stream memory: z[b] = y[b] W_U[b], one workgroup per stream, a quarter of W_U's rows per wavefront, all of it requested
// at once. (Down as a part of it, four streams per workgroup, took 13 us: each of the few workgroups then pulls all of W_down
// through one compute unit. Apart they take 3.6 + 2.5.)
__global__ __launch_bounds__(256) void rows_memory_kernel(const float *y, const float *WU, float *z) {
  __shared__ float part[4][64];
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = wave_id();
  const float *W = WU + (size_t)b * 4096 + wave * 1024 + lane;
  float wu[16], yk[16];
#pragma unroll
  for (int k = 0; k < 16; ++k) wu[k] = W[k * 64];
#pragma unroll
  for (int k = 0; k < 16; ++k) yk[k] = y[(size_t)b * 64 + wave * 16 + k];
  float s = 0.0f;
#pragma unroll
  for (int k = 0; k < 16; ++k) s = fmaf(yk[k], wu[k], s);
  part[wave][lane] = s;
  __syncthreads();
  if (wave == 0) z[(size_t)b * 64 + lane] = ((part[0][lane] + part[1][lane]) + part[2][lane]) + part[3][lane];
}

// ---------------------------------------------------------------------------------------------------
// update: products of one stage in one grid
// ---------------------------------------------------------------------------------------------------
// two products dX = dY W^T: first[0] workgroups are tiles of the first, the rest of the second
__global__ __launch_bounds__(NTH) void rows_dx2_kernel(RowsArgs a, RowsArgs b, int first) {
  __shared__ float red[NW * 256];
  const int q = blockIdx.x;
  if (q < first) { const int ntn = a.N / 16; tile<A_PLAIN, W_NK, E_STORE>(a, q / ntn, q % ntn, red); }
  else { const int ntn = b.N / 16; tile<A_PLAIN, W_NK, E_STORE>(b, (q - first) / ntn, (q - first) % ntn, red); }
}
// Newest cache slot, 16 streams per workgroup (Eq. 1-3 backward): dg = d(hm) W_m[last slot]^T as tiles, then per element
// d gg = dg gv psi'(gg), d gv = dg psi(gg), and dxt = W_g d gg + W_v d gv; x_t is left for the weight gradients of W_g, W_v.
__device__ __forceinline__ void slot_streams(const RowsSlotArgs &a, int mt, float *red) {
  __shared__ float dg_s[2][16][257];
  __shared__ int sym_s[16];
  const int tid = threadIdx.x, lane = tid & 63, wave = wave_id(), r = lane & 15;
  RowsArgs ra{};
  RowsOp o{a.dhm, nullptr, a.Dh, a.Wslot, nullptr, a.Dh, a.Dh};
  RowCtx rc{};
  rc.m = mt * 16 + r < a.B ? mt * 16 + r : a.B - 1;
  if (tid < 16) {
    const int b = mt * 16 + tid;
    sym_s[tid] = b < a.B && stream_active(a.ws, b) ? (int)stream_window(a.ws, b, a.T)[a.T - 1] : -1;
  }
  for (int q0 = 0; q0 < a.c; q0 += 16) {
    Contraction<A_PLAIN, W_NK> c;
    const int col = q0 + r < a.c ? q0 + r : a.c - 1;
    c.start(ra, o, rc, col);
    const f32x4 acc = c.finish(ra, o, rc, col);
    __syncthreads();  // the previous tile's sums have been read
#pragma unroll
    for (int e = 0; e < 4; ++e) red[wave * 256 + ((lane >> 4) * 4 + e) * 16 + r] = acc[e];
    __syncthreads();
    const int row = tid >> 4, q = q0 + (tid & 15), b = mt * 16 + row;
    if (tid < 256 && q < a.c) {
      float dg = red[tid];
#pragma unroll
      for (int w = 1; w < NW; ++w) dg += red[w * 256 + tid];
      float dgg = 0.0f, dgv = 0.0f;
      if (b < a.B) {
        const float gg = a.GG[(size_t)b * a.c + q], gv = a.GV[(size_t)b * a.c + q];
        float grad;
        const float psi = fade_gelu_both(gg, grad);
        dgg = dg * gv * grad;
        dgv = dg * psi;
        a.dgg[(size_t)b * a.c + q] = dgg;
        a.dgv[(size_t)b * a.c + q] = dgv;
      }
      dg_s[0][row][q] = dgg;
      dg_s[1][row][q] = dgv;
    }
  }
  __syncthreads();
  for (int t = tid; t < 16 * a.D; t += NTH) {
    const int row = t / a.D, i = t - row * a.D, b = mt * 16 + row;
    if (b >= a.B) continue;
    float s = 0.0f;
    for (int q0 = 0; q0 < a.c; q0 += 4) {
      float wg[4], wv[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) { const int q = q0 + j < a.c ? q0 + j : a.c - 1; wg[j] = a.Wg[i * a.c + q]; wv[j] = a.Wv[i * a.c + q]; }
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (q0 + j < a.c) s = fmaf(wg[j], dg_s[0][row][q0 + j], fmaf(wv[j], dg_s[1][row][q0 + j], s));
    }
    a.dxt[(size_t)b * a.D + i] = s;
    a.xt[(size_t)b * a.D + i] = sym_s[row] >= 0 ? a.tabXe32[(size_t)sym_s[row] * a.D + i] : 0.0f;  // an inactive stream adds nothing
  }
}
// Eq. 4's weight gradient, first stage: dW[(tap, i)][o] over 128 tokens (b, j), sum of xl[b][j - (taps - 1) + tap][i] dY[b][j][o], as one
// strip of 16 (tap, i) rows, sixteen tokens a wavefront; the strips of tap rows 0 .. 15 also leave the tokens' sum for the bias.
__device__ __forceinline__ void conv_strip(const RowsConvArgs &a, int chunk, int m0, float *red) {
  __shared__ float bred[NW][64];
  const int tid = threadIdx.x, lane = tid & 63, wave = wave_id(), r = lane & 15, g = lane >> 4, rows = a.taps * a.D;
  const int m = m0 + r < rows ? m0 + r : rows - 1, tap = m / a.D, ci = m - tap * a.D, back = a.taps - 1 - tap;
  float *out = a.part + (size_t)chunk * (rows + 1) * a.D;
  for (int n0 = 0; n0 < a.D; n0 += 16) {
    float l[4], v[4], bs = 0.0f;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int k = chunk * 128 + wave * 16 + 4 * u + g, kc = k < a.tokens ? k : a.tokens - 1, j = kc & (a.T - 1);  // T: a power of two
      l[u] = a.XL[(size_t)(j >= back ? kc - back : kc) * a.D + ci];
      v[u] = a.dcv[(size_t)kc * a.D + n0 + r];
      if (j < back) l[u] = 0.0f;  // in front of the window
      if (k >= a.tokens) v[u] = 0.0f;
    }
    f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int u = 0; u < 4; ++u) { acc = __builtin_amdgcn_mfma_f32_16x16x4f32(l[u], v[u], acc, 0, 0, 0); bs += v[u]; }
    __syncthreads();  // the previous columns' sums have been read
#pragma unroll
    for (int e = 0; e < 4; ++e) red[wave * 256 + (g * 4 + e) * 16 + r] = acc[e];
    bred[wave][lane] = bs;
    __syncthreads();
    if (tid < 256) {
      float x = red[tid];
#pragma unroll
      for (int w = 1; w < NW; ++w) x += red[w * 256 + tid];
      if (m0 + (tid >> 4) < rows) out[(size_t)(m0 + (tid >> 4)) * a.D + n0 + (tid & 15)] = x;
    } else if (m0 == 0 && tid < 272) {
      float x = 0.0f;
      for (int w = 0; w < NW; ++w) x += (bred[w][r] + bred[w][16 + r]) + (bred[w][32 + r] + bred[w][48 + r]);
      out[(size_t)rows * a.D + n0 + r] = x;
    }
  }
}
__global__ __launch_bounds__(NTH) void rows_last_kernel(RowsArgs rt, int n_rt, RowsArgs ct, int n_ct, RowsSlotArgs sl, RowsConvArgs cv, int n_cv) {
  __shared__ float red[NW * 256];
  int q = blockIdx.x;
  const int n_sl = (sl.B + 15) / 16;
  if (q < n_sl) { slot_streams(sl, q, red); return; }  // the longest chain first
  q -= n_sl;
  if (q < n_rt) { const int ntn = rt.N / 16; tile<A_PLAIN, W_NK, E_STORE>(rt, q / ntn, q % ntn, red); return; }
  q -= n_rt;
  if (q < n_cv) { const int nm = (cv.taps * cv.D + 15) / 16; conv_strip(cv, q / nm, q % nm * 16, red); return; }
  q -= n_cv;
  const int ntn = ct.N / 16;
  tile<A_CONVT, W_NK_CONV, E_STORE>(ct, q / ntn, q % ntn, red);
}

// ---------------------------------------------------------------------------------------------------
// Weight gradients of every matrix and their Adam step, one launch. A wavefront owns a strip of 16 rows x 64 columns of one
// matrix: dW[m][n] = sum over rows b of L[b][m] R[b][n], four tiles of 16 x 16 with tile t holding columns n0 + 4 (l & 15) + t, so
// that a lane's outputs, R's operands and the optimiser state all move in 16-byte pieces. 24 bytes of state per weight are
// what bounds it. L may be a LayerNorm (moments per row) formed on the way.
// ---------------------------------------------------------------------------------------------------
struct Adam4 {  // optimiser state of n <= 4 neighbouring weights, requested ahead of the gradient; vec: as one 16-byte piece
  f32x4 m, v, w;
  __device__ __forceinline__ void load(const AdamArrays &o, size_t idx, int n, bool vec) {
    if (vec) { m = ld4(o.m + idx); v = ld4(o.v + idx); w = ld4(o.master + idx); }
    else
#pragma unroll
      for (int i = 0; i < 4; ++i) { const size_t k = idx + (i < n ? i : 0); m[i] = o.m[k]; v[i] = o.v[k]; w[i] = o.master[k]; }
  }
  __device__ __forceinline__ void step(const AdamArrays &o, const UpdateState &us, size_t idx, const f32x4 &g, int n, bool vec) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      m[i] = o.beta1 * m[i] + (1.0f - o.beta1) * g[i];
      v[i] = o.beta2 * v[i] + (1.0f - o.beta2) * g[i] * g[i];
      w[i] = w[i] - o.lr * (m[i] / us.c1) / (sqrtf(v[i] / us.c2) + o.eps);
    }
    float *grad = const_cast<float *>(o.grad_base);
    const bool live = us.na != 0;  // no active stream: a gradient of zero, and no update
    if (vec) {
      st4(grad + idx, g);
      if (live) { st4(o.m + idx, m); st4(o.v + idx, v); st4(o.master + idx, w); }
    } else
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (i < n) {
          grad[idx + i] = g[i];
          if (live) { o.m[idx + i] = m[i]; o.v[idx + i] = v[i]; o.master[idx + i] = w[i]; }
        }
  }
};
// the contraction for one strip, four rows (lane group g: row k + g) a matrix instruction
__device__ __forceinline__ void strip(const RowsDw &d, int m0, int n0, f32x4 (&acc)[4]) {
  constexpr int U = 4;
  const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
  const int m = m0 + r < d.M ? m0 + r : d.M - 1, n = n0 + 4 * r < d.N ? n0 + 4 * r : 0;
  const bool vec = (d.N & 3) == 0 && (d.ldr & 3) == 0;
  float ga = 1.0f, be = 0.0f;
  if (d.gamma) { ga = d.gamma[m]; be = d.beta[m]; }
  for (int k = 0; k < d.K; k += U * 4) {
    float l[U];
    f32x4 rv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int kk = k + 4 * u + g, kc = kk < d.K ? kk : d.K - 1;
      l[u] = d.L[(size_t)kc * d.ldl + m];
      if (d.gamma) {
        const float2 mo = *reinterpret_cast<const float2 *>(d.mom + 2 * kc);
        l[u] = fmaf(__fmul_rn(l[u] - mo.x, mo.y), ga, be);
      }
      if (vec) rv[u] = ld4(d.R + (size_t)kc * d.ldr + n);
      else
#pragma unroll
        for (int t = 0; t < 4; ++t) rv[u][t] = d.R[(size_t)kc * d.ldr + (n + t < d.N ? n + t : n)];
      if (kk >= d.K) rv[u] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (k + 4 * u < d.K) {
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(l[u], rv[u][t], acc[t], 0, 0, 0);
      }
  }
}
struct StripState {  // lane l: rows m0 + 4 (l >> 4) + e, columns n0 + 4 (l & 15) .. + 3
  Adam4 st[4];
  int m;
  FadeStripLane at;
  __device__ __forceinline__ void load(const RowsDwArgs &a, const RowsDw &d, int m0, int n0) {
    const int lane = threadIdx.x & 63;
    m = m0 + (lane >> 4) * 4;
    at = fade_strip_lane(d.off, d.N, n0, m, lane & 15);
#pragma unroll
    for (int e = 0; e < 4; ++e) st[e].load(a.opt, at.left > 0 && m + e < d.M ? at.idx + (size_t)e * d.N : d.off, at.left > 0 ? at.left : 1, at.vec);
  }
  __device__ __forceinline__ void step(const RowsDwArgs &a, const RowsDw &d, const UpdateState &us, const f32x4 (&acc)[4]) {
    if (at.left <= 0) return;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (m + e < d.M) st[e].step(a.opt, us, at.idx + (size_t)e * d.N, f32x4{acc[0][e], acc[1][e], acc[2][e], acc[3][e]}, at.left, at.vec);
  }
};
__global__ __launch_bounds__(256) void rows_dw_adam_kernel(RowsDwArgs a) {
  const UpdateState us = *a.opt.u;
  // four strips a workgroup: 960 strips at D_h = 512 then spread over all compute units
  int unit = (int)blockIdx.x * 4 + wave_id(), p = 0, at = 0;
#pragma unroll
  for (int i = 1; i < 12; ++i)  // every bound in one load (a search that stops early is a chain of them)
    if (i < a.count && unit >= a.first[i]) { p = i; at = a.first[i]; }
  unit -= at;
  const RowsDw d = a.d[p];
  const int ns = (d.N + 63) / 64, m0 = unit / ns * 16, n0 = unit % ns * 64;
  if (m0 >= d.M) return;  // the last workgroup's spare wavefronts
  StripState ss;
  ss.load(a, d, m0, n0);
  f32x4 acc[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) acc[t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  strip(d, m0, n0, acc);
  ss.step(a, d, us, acc);
}

template <int PRO, int WL, int EPI, bool TWO = false> hipError_t launch(const RowsArgs &a, hipStream_t s, bool geglu = false) {
  if (a.M <= 0 || a.op0.K % 16 || a.N % (geglu ? 8 : 16) || (TWO && a.op1.K % 16)) return hipErrorInvalidValue;
  hipLaunchKernelGGL((rows_kernel<PRO, WL, EPI, TWO>), dim3(a.N / (geglu ? 8 : 16), (a.M + 15) / 16), dim3(NTH), 0, s, a);
  return hipGetLastError();
}

}  // namespace

hipError_t fade_rows(int op, const RowsArgs &a, hipStream_t s) {
  switch (op) {
    case ROWS_GLOBAL:     return launch<A_PLAIN, W_KN, E_GLOBAL>(a, s);
    case ROWS_MIX:        return launch<A_PLAIN, W_KN, E_MIX, true>(a, s);
    case ROWS_STORE:      return launch<A_PLAIN, W_KN, E_STORE>(a, s);
    case ROWS_DOWN:       return launch<A_LN, W_KN, E_STORE>(a, s);
    case ROWS_GATE:       return launch<A_PLAIN, W_KN, E_GATE, true>(a, s);
    case ROWS_FNR_IN:     return launch<A_LN, W_KN, E_GEGLU>(a, s, true);
    case ROWS_HEAD:       return launch<A_FINAL, W_KN, E_BIAS>(a, s);
    case ROWS_HEAD_PLAIN: return launch<A_PLAIN, W_KN, E_BIAS>(a, s);
    case ROWS_DHEAD:      return a.M <= NTH ? launch<A_LOSS, W_NK, E_STORE>(a, s) : hipErrorInvalidValue;
    case ROWS_DX:         return launch<A_PLAIN, W_NK, E_STORE>(a, s);
    case ROWS_DGEGLU:     return launch<A_PLAIN, W_NK, E_DGEGLU>(a, s);
    case ROWS_DX_PAIR:    return launch<A_PLAIN, W_NK_PAIR, E_STORE>(a, s);
    default: return hipErrorInvalidValue;
  }
}
hipError_t fade_rows_window(const RowsWindowArgs &a, const RowsArgs &conv, hipStream_t s) {
  if (a.Dc > 4 * NTH || a.c > NTH || a.T > NTH || a.D % 4 || (conv.M > 0 && (conv.op0.K % 16 || conv.N % 16 || conv.D % 16))) return hipErrorInvalidValue;
  const int tiles = conv.M > 0 ? (conv.M + 15) / 16 * (conv.N / 16) : 0;
  hipLaunchKernelGGL(rows_window_kernel, dim3(a.B + tiles), dim3(NTH), 0, s, a, conv);
  return hipGetLastError();
}
hipError_t fade_rows_memory(const float *y, const float *WU, float *z, int B, hipStream_t s) {
  hipLaunchKernelGGL(rows_memory_kernel, dim3(B), dim3(256), 0, s, y, WU, z);
  return hipGetLastError();
}
hipError_t fade_rows_dx2(const RowsArgs &a, const RowsArgs &b, hipStream_t s) {
  if (a.M <= 0 || b.M <= 0 || a.N % 16 || b.N % 16 || a.op0.K % 16 || b.op0.K % 16) return hipErrorInvalidValue;
  const int na = (a.M + 15) / 16 * (a.N / 16), nb = (b.M + 15) / 16 * (b.N / 16);
  hipLaunchKernelGGL(rows_dx2_kernel, dim3(na + nb), dim3(NTH), 0, s, a, b, na);
  return hipGetLastError();
}
hipError_t fade_rows_last(const RowsArgs &router, const RowsArgs &convt, const RowsConvArgs &conv, const RowsSlotArgs &slot, hipStream_t s) {
  if (slot.B <= 0 || slot.c > 256 || slot.Dh % 16 || (router.M > 0 && (router.N % 16 || router.op0.K % 16)) ||
      (convt.M > 0 && (convt.N % 16 || convt.D % 16 || conv.D % 16 || (conv.T & (conv.T - 1)))))
    return hipErrorInvalidValue;
  const int nr = router.M > 0 ? (router.M + 15) / 16 * (router.N / 16) : 0, nc = convt.M > 0 ? (convt.M + 15) / 16 * (convt.N / 16) : 0;
  const int nv = convt.M > 0 ? fade_rows_conv_parts(conv.tokens) * ((conv.taps * conv.D + 15) / 16) : 0;
  hipLaunchKernelGGL(rows_last_kernel, dim3((slot.B + 15) / 16 + nr + nv + nc), dim3(NTH), 0, s, router, nr, convt, nc, slot, conv, nv);
  return hipGetLastError();
}
int fade_rows_conv_parts(int tokens) { return (tokens + 127) / 128; }
hipError_t fade_rows_dw_adam(RowsDwArgs &a, hipStream_t s) {
  a.first[0] = 0;
  for (int i = 0; i < a.count; ++i) {
    const RowsDw &d = a.d[i];
    if (d.M <= 0 || d.N <= 0 || d.K <= 0 || d.off % 4) return hipErrorInvalidValue;
    a.first[i + 1] = a.first[i] + (d.M + 15) / 16 * ((d.N + 63) / 64);
  }
  hipLaunchKernelGGL(rows_dw_adam_kernel, dim3((a.first[a.count] + 3) / 4), dim3(256), 0, s, a);
  return hipGetLastError();
}

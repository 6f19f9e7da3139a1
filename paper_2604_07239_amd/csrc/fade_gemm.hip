// fade_gemm.hip — the dense products of the model step with fused prologues and epilogues (gfx950).
//
// bf16 path: C[M][N] = A[M][K] * W[K][N] on the matrix cores (v_mfma_f32_32x32x16_bf16, fp32 accumulate).
//   * Both operands stream global -> LDS by LDS-DMA through rings of units of 64 along K, synchronised by hand (s_waitcnt vmcnt +
//     a bare s_barrier); A is row-major with its 16-byte pieces XOR-permuted in LDS, W was rearranged at load time into MFMA
//     fragment order (1 KiB per 32 columns x 16 k, contiguous along K). Fragment reads go through inline assembly with
//     hand-placed lgkmcnt waits, a k-step or more ahead of the matrix instructions they feed.
//     pipe_body: 4 wavefronts, tiles of 64 / 128 rows x 64 / 128 columns (small and medium batches, grouped launches, split-K
//     partials). gemm_fnr_kernel: 32 / 64 x 128 on two groups of 4 wavefronts that share the ranges of K (the refiner's input
//     with few tiles). pipe2_body: 8 wavefronts on a 256 x 256 tile (large batches, tall split-K partials).
//   * gemm_bf16_kernel forms A on the fly instead (the causal-conv row gather; Eq. 10's tail for the head product) and
//     stages it through LDS from registers; its W fragments go straight from L2 into registers.
//   * Weight gradients dW = L^T R contract over the batch: tn_body stages both row-major operands as they lie in memory
//     and turns them on the way out of LDS with the transposing read (ds_read_b64_tr_b16); 4 wavefronts on up to
//     128 x 128 inside grouped launches. gemm_tn2_kernel: 256 x 256 tiles on 8 wavefronts, all matrices in one launch that shares the
//     k-steps out to the compute units in equal pieces (large batches).
//   * The accumulators are parked in LDS (fp32; the 256-row tiles a wavefront's rows at a time) and re-read row-wise, so that every
//     side input and every output moves in 16-byte pieces and per-row statistics for the next LayerNorm fall out of a
//     16-lane butterfly. Partial statistics are stored per 128-column tile and summed by the consumer in index order: no
//     atomics, so the result is reproducible bit for bit, and the same for every tile shape.
//   * blockIdx -> tile: the chip dispatches consecutive workgroups round-robin over its 8 XCDs, each with a private L2;
//     tile_of_block gives an XCD a range of column tiles (its share of W stays in its L2) and walks its tiles row by row.
// fp32 path above 256 rows, and at any batch with D_h, D_cache or D_e above 2048: the same prologues / epilogues around a plain
// FMA core (gemm_f32_kernel); the other batches have kernels of their own (fade_rows.hip).
#include <cstdlib>
#include <type_traits>

#include "fade_dev.h"
#include "fade_kernels.h"

int fade_gemm_tune();

namespace {

__device__ __forceinline__ float gelu_f(float x) { return fade_gelu(x); }
__device__ __forceinline__ float sigmoid_f(float x) { return fade_sigmoid(x); }

// 8 consecutive activations <-> registers
__device__ __forceinline__ void load8(const bf16_t *p, float v[8]) {
  const bf16x8 r = *reinterpret_cast<const bf16x8 *>(p);
#pragma unroll
  for (int i = 0; i < 8; ++i) v[i] = (float)r[i];
}
__device__ __forceinline__ void load8(const float *p, float v[8]) {
  const f32x4 a = *reinterpret_cast<const f32x4 *>(p), b = *reinterpret_cast<const f32x4 *>(p + 4);
#pragma unroll
  for (int i = 0; i < 4; ++i) { v[i] = a[i]; v[4 + i] = b[i]; }
}
__device__ __forceinline__ void store8(bf16_t *p, const float v[8]) {
  bf16x8 r;
#pragma unroll
  for (int i = 0; i < 8; ++i) r[i] = (bf16_t)v[i];
  *reinterpret_cast<bf16x8 *>(p) = r;
}
// outputs that only the backward pass reads (bf16)
__device__ __forceinline__ void store8_nt(bf16_t *p, const float v[8]) {
  bf16x8 r;
#pragma unroll
  for (int i = 0; i < 8; ++i) r[i] = (bf16_t)v[i];
  fade_nt_store(p, __builtin_bit_cast(f32x4, r));
}
__device__ __forceinline__ void store8(float *p, const float v[8]) {
  f32x4 a, b;
#pragma unroll
  for (int i = 0; i < 4; ++i) { a[i] = v[i]; b[i] = v[4 + i]; }
  *reinterpret_cast<f32x4 *>(p) = a;
  *reinterpret_cast<f32x4 *>(p + 4) = b;
}
__device__ __forceinline__ void store8_nt(float *p, const float v[8]) { store8(p, v); }  // read again with plain loads

// ---------------------------------------------------------------------------------------------------
// A-operand staging: one thread owns one 8-wide chunk of one row per pass.
// ---------------------------------------------------------------------------------------------------
template <typename AT> struct Raw8 { float v[8]; };
template <> struct Raw8<bf16_t> { bf16x8 v; };

template <typename AT> __device__ __forceinline__ void raw_zero(Raw8<AT> &r);
template <> __device__ __forceinline__ void raw_zero<bf16_t>(Raw8<bf16_t> &r) {
#pragma unroll
  for (int i = 0; i < 8; ++i) r.v[i] = (bf16_t)0.0f;
}
template <> __device__ __forceinline__ void raw_zero<float>(Raw8<float> &r) {
#pragma unroll
  for (int i = 0; i < 8; ++i) r.v[i] = 0.0f;
}
__device__ __forceinline__ void raw_load(Raw8<bf16_t> &r, const bf16_t *p) { r.v = *reinterpret_cast<const bf16x8 *>(p); }
__device__ __forceinline__ void raw_load(Raw8<float> &r, const float *p) { load8(p, r.v); }
__device__ __forceinline__ void raw_to_float(const Raw8<bf16_t> &r, float v[8]) {
#pragma unroll
  for (int i = 0; i < 8; ++i) v[i] = (float)r.v[i];
}
__device__ __forceinline__ void raw_to_float(const Raw8<float> &r, float v[8]) {
#pragma unroll
  for (int i = 0; i < 8; ++i) v[i] = r.v[i];
}

// Issue the global loads for chunk (row m, columns k..k+7) of the A operand.
template <int PRO, typename AT>
__device__ __forceinline__ void stage_load(const GemmArgs &g, int m, int k, Raw8<AT> &a, Raw8<AT> &a2) {
  const AT *A = static_cast<const AT *>(g.A);
  if (m >= g.M) { raw_zero(a); if (PRO == PRO_FINAL) raw_zero(a2); return; }
  if (PRO == PRO_CONV) {
    const int b = m / g.T, j = m - b * g.T;
    const int tap = k / g.D, i = k - tap * g.D;
    const int tok = j - (g.taps - 1) + tap;
    if (tap < g.taps && tok >= 0) raw_load(a, A + ((size_t)b * g.T + tok) * g.D + i);
    else raw_zero(a);
  } else if (PRO == PRO_CONVT) {
    const int b = m / g.T, j = m - b * g.T;
    const int tap = k / g.D, i = k - tap * g.D;
    const int tok = j + (g.taps - 1) - tap;
    if (tap < g.taps && tok < g.T) raw_load(a, A + ((size_t)b * g.T + tok) * g.D + i);
    else raw_zero(a);
  } else {
    raw_load(a, A + (size_t)m * g.lda + k);
    if (PRO == PRO_FINAL) raw_load(a2, static_cast<const AT *>(g.A2) + (size_t)m * g.lda + k);
  }
}

// Turn the loaded chunk into operand values.
template <int PRO, typename AT>
__device__ __forceinline__ void stage_transform(const GemmArgs &g, int k, const Raw8<AT> &a, const Raw8<AT> &a2,
                                                float mean, float rstd, float lam, float v[8]) {
  raw_to_float(a, v);
  if (PRO == PRO_LN || PRO == PRO_FINAL) {
    float ga[8], be[8];
    load8(g.gamma + k, ga);
    load8(g.beta + k, be);
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = fmaf(__fmul_rn(v[i] - mean, rstd), ga[i], be[i]);
    if (PRO == PRO_FINAL) {
      float r[8];
      raw_to_float(a2, r);
#pragma unroll
      for (int i = 0; i < 8; ++i) v[i] = fmaf(lam, r[i], gelu_f(v[i]));
    }
  }
}

// The same with the LayerNorm gain / shift of the chunk already in registers (requested together with the chunk itself).
template <int PRO, typename AT>
__device__ __forceinline__ void stage_transform_gb(const Raw8<AT> &a, const Raw8<AT> &a2, float mean, float rstd, float lam,
                                                   const float ga[8], const float be[8], float v[8]) {
  raw_to_float(a, v);
  if (PRO == PRO_LN || PRO == PRO_FINAL) {
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = fmaf(__fmul_rn(v[i] - mean, rstd), ga[i], be[i]);
    if (PRO == PRO_FINAL) {
      float r[8];
      raw_to_float(a2, r);
#pragma unroll
      for (int i = 0; i < 8; ++i) v[i] = fmaf(lam, r[i], gelu_f(v[i]));
    }
  }
}

// mean / rstd of row m from the partial sums its producer left behind (fixed summation order).
__device__ __forceinline__ void row_moments(const GemmArgs &g, int m, float &mean, float &rstd) {
  mean = 0.0f; rstd = 1.0f;
  if (m >= g.M) return;
  fade_row_moments(g.stats + (size_t)m * g.stats_n * 2, g.stats_n, g.K, mean, rstd);
}

// the same where eight neighbouring lanes share row m
__device__ __forceinline__ void row_moments_lanes(const GemmArgs &g, int m, float &mean, float &rstd) {
  fade_row_moments_lanes<8>(g.stats + (size_t)(m < g.M ? m : g.M - 1) * g.stats_n * 2, g.stats_n, g.K, mean, rstd);
}

// ---------------------------------------------------------------------------------------------------
// epilogue: the accumulator tile sits in LDS as fp32 [BM][BN + 4]; threads walk it in 8-wide row chunks
// ---------------------------------------------------------------------------------------------------
// Side inputs an epilogue reads beside the accumulator: 2 for the mix and gate forms, 1 for the global projection.
template <int EPI> struct EpiSides { static constexpr int n = (EPI == EPI_MIX || EPI == EPI_GATE) ? 2 : (EPI == EPI_GLOBAL ? 1 : 0); };

// Issue the global loads of one 8-wide chunk of the side inputs (element offset o); the values stay raw until used.
template <int EPI, typename AT>
__device__ __forceinline__ void epi_side_load(const GemmArgs &g, size_t o, bool live, Raw8<AT> *sd) {
  if (!live) return;
  if (EpiSides<EPI>::n >= 1) raw_load(sd[0], static_cast<const AT *>(g.S1) + o);
  if (EpiSides<EPI>::n >= 2) raw_load(sd[1], static_cast<const AT *>(g.S2) + o);
}

// What happens to one 8-wide chunk of finished sums x at element offset o, for the epilogues that more than one kernel body has.
// The arithmetic is written with explicit fused multiply-adds and unfusable products (fmaf, __fmul_rn): instances for
// different tile shapes must give the same bits (a pass over many steps and a single step use different ones), which must not
// depend on where the compiler chooses to contract a * b + c.
// KEEP: whether the copies for the backward pass (C2, C3) are written; KEEP_ASK looks at the pointer here.
enum { KEEP_NO = 0, KEEP_YES = 1, KEEP_ASK = 2 };
template <int KEEP> __device__ __forceinline__ bool keeps(const void *p) { return KEEP == KEEP_ASK ? p != nullptr : KEEP == KEEP_YES; }
template <int EPI, typename AT, int KEEP = KEEP_ASK>
__device__ __forceinline__ void epi_finish(const GemmArgs &g, size_t o, float lam, const Raw8<AT> *sd, const float x[8], float out[8]) {
  static_assert(EPI == EPI_STORE || EPI == EPI_GLOBAL || EPI == EPI_MIX || EPI == EPI_GATE, "epilogue");
  if constexpr (EPI == EPI_STORE) {
#pragma unroll
    for (int i = 0; i < 8; ++i) out[i] = x[i];
    store8(static_cast<AT *>(g.C) + o, out);
  } else if constexpr (EPI == EPI_GLOBAL) {
    float s1[8];
    raw_to_float(sd[0], s1);
#pragma unroll
    for (int i = 0; i < 8; ++i) out[i] = fmaf(lam, s1[i], gelu_f(x[i]));
    store8(static_cast<AT *>(g.C) + o, out);
    if (keeps<KEEP>(g.C2)) store8_nt(static_cast<AT *>(g.C2) + o, x);
  } else if constexpr (EPI == EPI_MIX) {
    float s1[8], s2[8], al[8];
    raw_to_float(sd[0], s1);
    raw_to_float(sd[1], s2);
#pragma unroll
    for (int i = 0; i < 8; ++i) { al[i] = sigmoid_f(x[i]); out[i] = fmaf(al[i], s1[i], __fmul_rn(1.0f - al[i], s2[i])); }
    store8(static_cast<AT *>(g.C) + o, out);
    if (keeps<KEEP>(g.C2)) store8_nt(static_cast<AT *>(g.C2) + o, al);
  } else {
    float s1[8], s2[8], sgm[8];
    raw_to_float(sd[0], s1);
    raw_to_float(sd[1], s2);
#pragma unroll
    for (int i = 0; i < 8; ++i) { sgm[i] = sigmoid_f(x[i]); out[i] = fmaf(lam, s2[i], __fmul_rn(s1[i], sgm[i])); }
    store8(static_cast<AT *>(g.C) + o, out);
    if (keeps<KEEP>(g.C2)) store8_nt(static_cast<AT *>(g.C2) + o, sgm);
  }
}
struct FoldCols { float sg[8], tg[8], sv[8], tv[8]; };  // the folded LayerNorm's column vectors of a gate chunk and its value chunk
template <typename AT, int KEEP = KEEP_ASK>
__device__ __forceinline__ void epi_finish_geglu_fold(const GemmArgs &g, size_t o, float mean, float rstd, const FoldCols &f, const float x[8], const float xv[8]) {
  float eg[8], ev[8], out[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    eg[i] = fade_fold_ln(x[i], mean, rstd, f.sg[i], f.tg[i]);
    ev[i] = fade_fold_ln(xv[i], mean, rstd, f.sv[i], f.tv[i]);
    out[i] = gelu_f(eg[i]) * ev[i];
  }
  store8(static_cast<AT *>(g.C) + o, out);
  if (keeps<KEEP>(g.C2)) store8_nt(static_cast<AT *>(g.C2) + o, eg);
  if (keeps<KEEP>(g.C3)) store8_nt(static_cast<AT *>(g.C3) + o, ev);
}

// A thread walks rows r0, r0 + RP, ... of its 8-wide column chunk. The side inputs (and the row moments of the folded
// form) of U consecutive passes are requested together before the first of them is used, so that one memory latency
// covers U rows.
template <int EPI, typename AT, int BM, int BN, int LDC = BN + 4, int NT = 256>
__device__ __forceinline__ void epilogue(const GemmArgs &g, const float *Cs, int m0, int n0, int nt, int tid, int split = 0) {
  constexpr bool kGeglu = EPI == EPI_GEGLU || EPI == EPI_GEGLU_FOLD;
  constexpr int BNO = kGeglu ? BN / 2 : BN;  // output columns of this tile
  constexpr int CH = BNO / 8;                            // chunks (threads) per row
  constexpr int RP = NT / CH;                            // rows per pass
  constexpr int PASSES = (BM + RP - 1) / RP;
  constexpr int NS = EpiSides<EPI>::n;
  constexpr bool kAhead = NS > 0 || EPI == EPI_GEGLU_FOLD;
  constexpr int U = kAhead ? (PASSES < 4 ? PASSES : 4) : 1;
  constexpr bool kRagged = BM % (RP * U) != 0;  // a tile shorter than one round of passes: some threads own no row
  static_assert(PASSES % U == 0, "row passes");
  const int c8 = (tid % CH) * 8, r0 = tid / CH;
  const int nout0 = kGeglu ? nt * BNO : n0;  // first output column of the tile
  float lam = 0.0f;
  if (EPI == EPI_GLOBAL || EPI == EPI_GATE) lam = g.lam[0];
  FoldCols fc;
  if (EPI == EPI_GEGLU_FOLD) {
    load8(g.fold_s + n0 + c8, fc.sg); load8(g.fold_t + n0 + c8, fc.tg);
    load8(g.fold_s + n0 + BNO + c8, fc.sv); load8(g.fold_t + n0 + BNO + c8, fc.tv);
  }
#pragma unroll 1
  for (int rb = r0; rb < BM; rb += RP * U) {
    Raw8<AT> own[U][2];
    float mean[U], rstd[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int m = m0 + rb + u * RP;
      if (kRagged && rb + u * RP >= BM) continue;
      // past the last row: any row (dropped below); a branch around the loads would cost the exact vmcnt waits
      epi_side_load<EPI, AT>(g, (size_t)(m < g.M ? m : g.M - 1) * g.ldc + nout0 + c8, true, own[u]);
      if (EPI == EPI_GEGLU_FOLD) row_moments_lanes(g, m, mean[u], rstd[u]);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
    const Raw8<AT> *sd = own[u];
    const int r = rb + u * RP;
    if (kRagged && r >= BM) continue;
    const int m = m0 + r;
    const bool live = m < g.M;
    float x[8], out[8];
    load8(Cs + r * LDC + c8, x);
    const size_t o = (size_t)m * g.ldc + nout0 + c8;
    if (live) {
      if constexpr (EPI == EPI_STORE || EPI == EPI_GLOBAL || EPI == EPI_MIX || EPI == EPI_GATE) {
        epi_finish<EPI, AT>(g, o, lam, sd, x, out);
      } else if (EPI == EPI_STORE_F32) {
        float bi[8];
        if (g.bias) load8(g.bias + n0 + c8, bi);
#pragma unroll
        for (int i = 0; i < 8; ++i) out[i] = g.bias ? x[i] + bi[i] : x[i];
        store8(static_cast<float *>(g.C) + o, out);
      } else if (EPI == EPI_GEGLU) {
        float xv[8];
        load8(Cs + r * LDC + BNO + c8, xv);
#pragma unroll
        for (int i = 0; i < 8; ++i) out[i] = gelu_f(x[i]) * xv[i];
        store8(static_cast<AT *>(g.C) + o, out);
        if (g.C2) store8_nt(static_cast<AT *>(g.C2) + o, x);
        if (g.C3) store8_nt(static_cast<AT *>(g.C3) + o, xv);
      } else if (EPI == EPI_GEGLU_FOLD) {
        float xv[8];
        load8(Cs + r * LDC + BNO + c8, xv);
        epi_finish_geglu_fold<AT>(g, o, mean[u], rstd[u], fc, x, xv);
      } else if (EPI == EPI_GRAD) {  // split: partial sum over one range of the batch, slices [split][M][width] behind each other
        if (g.C3) {
          const int v = n0 + c8;
          float *dstp = ((v & 127) < 64) ? static_cast<float *>(g.C) : static_cast<float *>(g.C3);
          store8(dstp + ((size_t)split * g.M + m) * (g.N / 2) + (v / 128) * 64 + (v & 63), x);
        } else {
          store8(static_cast<float *>(g.C) + (size_t)split * g.M * g.ldc + o, x);
        }
      } else if (EPI == EPI_PARTIAL) {
        store8(static_cast<float *>(g.C) + ((size_t)split * g.M + m) * g.ldc + n0 + c8, x);
      } else if (EPI == EPI_CONV) {
        float bi[8], pre_act[8];
        load8(g.bias + n0 + c8, bi);
#pragma unroll
        for (int i = 0; i < 8; ++i) { pre_act[i] = x[i] + bi[i]; out[i] = gelu_f(pre_act[i]); }
        store8(static_cast<AT *>(g.C) + o, out);
        if (g.C2) store8_nt(static_cast<AT *>(g.C2) + o, pre_act);
      }
    } else {
#pragma unroll
      for (int i = 0; i < 8; ++i) out[i] = 0.0f;
    }
    if (g.stats_out && (EPI == EPI_STORE || EPI == EPI_MIX || EPI == EPI_GATE)) {
      float s = 0.0f, q = 0.0f;
#pragma unroll
      for (int i = 0; i < 8; ++i) { s += out[i]; q = fmaf(out[i], out[i], q); }
      if constexpr (CH == 16) {
        s = fade_lanes_sum<16>(s);
        q = fade_lanes_sum<16>(q);
      } else {
#pragma unroll
        for (int off = CH / 2; off > 0; off >>= 1) { s += __shfl_xor(s, off, 64); q += __shfl_xor(q, off, 64); }
      }
      if (live && (tid % CH) == 0) {
        float *p = g.stats_out + ((size_t)m * (g.N / BN) + nt) * 2;
        p[0] = s; p[1] = q;
      }
    }
    }
  }
}

// Block -> tile. Workgroups are dealt to the 8 XCDs round-robin (bid % 8), and each XCD has its own L2: the XCDs split
// the tile grid into cg column ranges x (8 / cg) interleaved row sets, and one XCD walks its tiles row by row, so the
// tiles that run together share their A rows and the XCD's slice of W stays in its L2. cg = 8 suits a small A (every
// XCD streams all of A past its own eighth of W); a tall A wants fewer column ranges so that it is fetched cg times
// instead of 8. Returns false for the padding blocks of a grid rounded up to whole row sets.
__device__ __forceinline__ bool tile_of_block(int bid, int ntm, int ntn, int cg, int &mt, int &nt) {
  if (cg <= 0) cg = 8;
  if (ntn % cg == 0) {
    const int rg = 8 / cg, x = bid & 7, r = bid >> 3, per = ntn / cg;
    nt = (x % cg) * per + r % per;
    mt = (r / per) * rg + x / cg;
  } else {
    nt = bid % ntn;
    mt = bid / ntn;
  }
  return mt < ntm;
}

// ---------------------------------------------------------------------------------------------------
// bf16 MFMA core
// ---------------------------------------------------------------------------------------------------
// KEEP (PRO_FINAL, M a multiple of the tile height): the operand formed on the fly, H of Eq. 10, is also written to C2
// ([M][lda], the update needs it for the head's weight gradient). Its stores are unconditional and sit behind the request
// for the block after next, so that no load ever waits for them (the memory counter is in order and covers stores).
template <int WM, int WN, int TM, int TN, int PRO, int EPI, bool KEEP = false>
__global__ __launch_bounds__(256) void gemm_bf16_kernel(GemmArgs g) {
  typedef bf16_t AT;
  constexpr int BM = WM * TM * 32, BN = WN * TN * 32, BK = 64, LDA = BK + 8, PASSES = BM / 32, LDC = BN + 4;
  static_assert(WM * WN == 4, "four wavefronts per workgroup");
  extern __shared__ __align__(16) unsigned char smem[];
  bf16_t *As = reinterpret_cast<bf16_t *>(smem);  // [2][BM][LDA]
  float *Cs = reinterpret_cast<float *>(smem);    // [BM][LDC], reuses the space after the K loop

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WN, wn = wave % WN;
  const int ntn = g.N / BN, ntm = (g.M + BM - 1) / BM;
  int mt, nt;
  if (!tile_of_block(blockIdx.x, ntm, ntn, 8, mt, nt)) return;
  const int m0 = mt * BM, n0 = nt * BN;

  const int srow = tid >> 3, skc = (tid & 7) * 8;
  float mean[PASSES], rstd[PASSES];
  float lam = 0.0f;
  if (PRO == PRO_LN || PRO == PRO_FINAL) {
#pragma unroll
    for (int p = 0; p < PASSES; ++p) row_moments_lanes(g, m0 + p * 32 + srow, mean[p], rstd[p]);
    if (PRO == PRO_FINAL) lam = g.lam[0];
  }

  // EPI_PARTIAL: the contraction in ranges (grid.y), each leaving its own partial, or, with sum_splits, every range in
  // turn inside this workgroup with their sums added in range order: the same bits as separate partials added later
  const bool fuse = EPI == EPI_PARTIAL && g.sum_splits != 0;
  const int nsplit = EPI == EPI_PARTIAL ? (fuse ? g.splits : (int)gridDim.y) : 1;
  const int sp_first = fuse ? 0 : (int)blockIdx.y, sp_end = fuse ? nsplit : (int)blockIdx.y + 1;
  const int nkb = g.K / BK / nsplit, ksteps = g.K / 16;
  // fragment stream of this wavefront's first column tile
  const bf16x8 *Wf = static_cast<const bf16x8 *>(g.W) + ((size_t)((n0 + wn * TN * 32) / 32) * ksteps) * 64 + lane;

  f32x16 acc[TM][TN], tot[EPI == EPI_PARTIAL ? TM : 1][EPI == EPI_PARTIAL ? TN : 1];
  for (int sp = sp_first; sp < sp_end; ++sp) {
  const int kb0 = sp * nkb;
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;

  Raw8<AT> ra[PASSES], ra2[PASSES];
  bf16x8 bcur[4][TN], bnext[4][TN];
  bf16x8 hkeep[KEEP ? PASSES : 1];  // KEEP: the block's transformed values as they went to LDS
  // LayerNorm gain / shift of this thread's 8 columns of the block: requested with the block's rows, not when they are used
  constexpr bool kGB = PRO == PRO_LN || PRO == PRO_FINAL;
  float ga[kGB ? 8 : 1], be[kGB ? 8 : 1];
  auto load_gb = [&](int k) {
    if constexpr (kGB) { load8(g.gamma + k, ga); load8(g.beta + k, be); }
  };

  // preamble: the range's first K block
#pragma unroll
  for (int p = 0; p < PASSES; ++p) stage_load<PRO, AT>(g, m0 + p * 32 + srow, kb0 * BK + skc, ra[p], ra2[p]);
  load_gb(kb0 * BK + skc);
#pragma unroll
  for (int ks = 0; ks < 4; ++ks)
#pragma unroll
    for (int j = 0; j < TN; ++j) bcur[ks][j] = Wf[((size_t)j * ksteps + kb0 * 4 + ks) * 64];
  if (sp != sp_first) __syncthreads();  // the previous range's last block has been read
#pragma unroll
  for (int p = 0; p < PASSES; ++p) {
    bf16_t *dst = As + (p * 32 + srow) * LDA + skc;
    if (PRO == PRO_PLAIN || PRO == PRO_CONV || PRO == PRO_CONVT) {
      *reinterpret_cast<bf16x8 *>(dst) = ra[p].v;
    } else {
      float v[8];
      if constexpr (kGB) stage_transform_gb<PRO, AT>(ra[p], ra2[p], mean[p], rstd[p], lam, ga, be, v);
      else stage_transform<PRO, AT>(g, kb0 * BK + skc, ra[p], ra2[p], mean[p], rstd[p], lam, v);
      store8(dst, v);
      if constexpr (KEEP) {
#pragma unroll
        for (int q = 0; q < 8; ++q) hkeep[p][q] = (bf16_t)v[q];
      }
    }
  }
  auto request = [&](int kb_abs) {  // rows, gain / shift and W fragments of K block kb_abs
    const int k1 = kb_abs * BK;
#pragma unroll
    for (int p = 0; p < PASSES; ++p) stage_load<PRO, AT>(g, m0 + p * 32 + srow, k1 + skc, ra[p], ra2[p]);
    load_gb(k1 + skc);
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
#pragma unroll
      for (int j = 0; j < TN; ++j) bnext[ks][j] = Wf[((size_t)j * ksteps + kb_abs * 4 + ks) * 64];
  };
  auto keep_store = [&](int kb_abs) {
    if constexpr (KEEP) {
#pragma unroll
      for (int p = 0; p < PASSES; ++p)
        *reinterpret_cast<bf16x8 *>(static_cast<AT *>(g.C2) + (size_t)(m0 + p * 32 + srow) * g.lda + kb_abs * BK + skc) = hkeep[p];
    }
  };
  if constexpr (KEEP) {
    if (nkb > 1) request(kb0 + 1);
    keep_store(kb0);
  }

  for (int kb = 0; kb < nkb; ++kb) {
    const bool more = kb + 1 < nkb;
    if (more && !KEEP) {
      const int k1 = (kb0 + kb + 1) * BK;
#pragma unroll
      for (int p = 0; p < PASSES; ++p) stage_load<PRO, AT>(g, m0 + p * 32 + srow, k1 + skc, ra[p], ra2[p]);
      load_gb(k1 + skc);
#pragma unroll
      for (int ks = 0; ks < 4; ++ks)
#pragma unroll
        for (int j = 0; j < TN; ++j) bnext[ks][j] = Wf[((size_t)j * ksteps + (kb0 + kb + 1) * 4 + ks) * 64];
    }
    __syncthreads();
    const bf16_t *Ab = As + (kb & 1) * BM * LDA;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      bf16x8 af[TM];
#pragma unroll
      for (int i = 0; i < TM; ++i)
        af[i] = *reinterpret_cast<const bf16x8 *>(Ab + ((wm * TM + i) * 32 + (lane & 31)) * LDA + ks * 16 + (lane >> 5) * 8);
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[i], bcur[ks][j], acc[i][j], 0, 0, 0);
    }
    if (more) {
      bf16_t *An = As + ((kb + 1) & 1) * BM * LDA;
      const int k1 = (kb0 + kb + 1) * BK;
#pragma unroll
      for (int p = 0; p < PASSES; ++p) {
        bf16_t *dst = An + (p * 32 + srow) * LDA + skc;
        if (PRO == PRO_PLAIN || PRO == PRO_CONV || PRO == PRO_CONVT) {
          *reinterpret_cast<bf16x8 *>(dst) = ra[p].v;
        } else {
          float v[8];
          if constexpr (kGB) stage_transform_gb<PRO, AT>(ra[p], ra2[p], mean[p], rstd[p], lam, ga, be, v);
          else stage_transform<PRO, AT>(g, k1 + skc, ra[p], ra2[p], mean[p], rstd[p], lam, v);
          store8(dst, v);
          if constexpr (KEEP) {
#pragma unroll
        for (int q = 0; q < 8; ++q) hkeep[p][q] = (bf16_t)v[q];
      }
        }
      }
#pragma unroll
      for (int ks = 0; ks < 4; ++ks)
#pragma unroll
        for (int j = 0; j < TN; ++j) bcur[ks][j] = bnext[ks][j];
      if constexpr (KEEP) {
        if (kb + 2 < nkb) request(kb0 + kb + 2);
        keep_store(kb0 + kb + 1);
      }
    }
  }
  if constexpr (EPI == EPI_PARTIAL) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        if (sp == sp_first) tot[i][j] = acc[i][j];
        else tot[i][j] += acc[i][j];
      }
  }
  }

  // park the accumulators: lane l of a 32x32 tile holds column l % 32, rows (e / 4) * 8 + (l / 32) * 4 + e % 4
  __syncthreads();
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int row = (wm * TM + i) * 32 + (e >> 2) * 8 + (lane >> 5) * 4 + (e & 3);
        const int col = (wn * TN + j) * 32 + (lane & 31);
        if constexpr (EPI == EPI_PARTIAL) Cs[row * LDC + col] = tot[i][j][e];
        else Cs[row * LDC + col] = acc[i][j][e];
      }
  __syncthreads();
  epilogue<EPI, AT, BM, BN>(g, Cs, m0, n0, nt, tid, fuse ? 0 : (int)blockIdx.y);
}

// ---------------------------------------------------------------------------------------------------
// bf16 MFMA core, pipelined: both operands stream global -> LDS with the asynchronous LDS-DMA loads (16 bytes per lane land at
// M0-base + lane * 16, no registers involved) through a ring of STAGES units of 64 along K. A: plain row-major bf16 [M][lda] (rows
// past M are clamped to row M - 1 and never stored), W: bf16 fragments as written by the weight preparation.
// Synchronisation is by hand: s_waitcnt vmcnt(n) for this wavefront's own DMAs, then a bare s_barrier (a __syncthreads() would
// drain every outstanding load and with it the pipeline).
// Four wavefronts, one or two per SIMD, so nothing hides a wavefront's own waits and the loop has to (unit_loop): the fragments of
// the next half unit are read from LDS under the matrix instructions of this one, into a second set of registers. A unit's hand-over
// (DMA wait, barrier) sits between its halves: its reads are complete by then, so behind the barrier its slot is free for
// the unit STAGES further on, whose requests go between the matrix instructions. Their addresses are a buffer resource, lane
// offsets and a scalar offset: no vector instructions.
// M = 1024, N = K = 2048, 64 x 128 tiles with the mix / gate epilogue: 18.7 / 18.4 us with the first fragments of a unit waited
// for behind its barrier and the requests in one burst in front of them, 17.0 / 16.4 now (kernel traces of whole steps), where what a compute unit is
// fed with from the L2 (24 KiB per unit) bounds it.
// grid.y > 1: split K, each block leaves an fp32 partial tile (EPI_PARTIAL)
// ---------------------------------------------------------------------------------------------------
template <int N> __device__ __forceinline__ void wait_vmcnt() {
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}
__device__ __forceinline__ void bare_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}
// The LDS-DMA of one KiB: lane offset + scalar offset from the resource's base, to lds + lane * 16.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t dma_rsrc(const void *base) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, 0x7fffffff, 0x00020000);
}
__device__ __forceinline__ void dma16(__amdgpu_buffer_rsrc_t r, uint32_t lane_off, uint32_t off, unsigned char *lds) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void *)lds, 16, lane_off, off, 0, 0);
}

// LDS fragment reads whose completion is waited for by hand: the compiler would wait for every outstanding read before the
// first matrix instruction of a group (s_waitcnt lgkmcnt(0)), also for the reads just issued for the next group. Reads issued
// through lds_read16 are invisible to it; lds_wait<N> lets the N youngest stay in flight (LDS returns in order) and
// lds_landed ties the value to the wait, so that no use can move above it.
template <int OFF> __device__ __forceinline__ bf16x8 lds_read16(uint32_t addr) {
  typedef __attribute__((ext_vector_type(4))) int i32x4;
  i32x4 v;
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF) : "memory");
  return __builtin_bit_cast(bf16x8, v);
}
template <int N> __device__ __forceinline__ void lds_wait() { asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(N) : "memory"); }
__device__ __forceinline__ void lds_landed(bf16x8 &v) {
  typedef __attribute__((ext_vector_type(4))) int i32x4;
  i32x4 t = __builtin_bit_cast(i32x4, v);
  asm volatile("" : "+v"(t));
  v = __builtin_bit_cast(bf16x8, t);
}
// The same for gfx950's transposing read of four 16-bit values per lane (ds_read_b64_tr_b16); two of them make one operand.
typedef __attribute__((ext_vector_type(2))) int i32x2;
template <int OFF> __device__ __forceinline__ i32x2 tr_read8(uint32_t addr) {
  i32x2 v;
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF) : "memory");
  return v;
}
__device__ __forceinline__ void tr_landed(i32x2 &v) { asm volatile("" : "+v"(v)); }
__device__ __forceinline__ bf16x8 tr_pair(i32x2 lo, i32x2 hi) {
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3));
}

template <int I> using Int = std::integral_constant<int, I>;
template <int N, typename F> __device__ __forceinline__ void static_for(F &&f) {  // f(Int<0>) ... f(Int<N - 1>)
  if constexpr (N > 0) {
    static_for<N - 1>(f);
    f(Int<N - 1>{});
  }
}
// NM matrix instructions mm(i); in front of them, evenly spread and in this order, NR reads rd(i) and ND requests dma(i)
template <int NM, int NR, int ND, typename MM, typename RD, typename DMA>
__device__ __forceinline__ void woven(MM &&mm, RD &&rd, DMA &&dma) {
  static_for<NM>([&](auto i_c) {
    constexpr int i = decltype(i_c)::value, r0 = (i * NR + NM - 1) / NM, r1 = ((i + 1) * NR + NM - 1) / NM, d0 = i * ND / NM, d1 = (i + 1) * ND / NM;
    static_for<r1 - r0>([&](auto k) { rd(Int<r0 + decltype(k)::value>{}); });
    static_for<d1 - d0>([&](auto k) { dma(Int<d0 + decltype(k)::value>{}); });
    __builtin_amdgcn_sched_barrier(0);
    mm(i_c);
    __builtin_amdgcn_sched_barrier(0);
  });
}
// wait until at most min(units, MAX) units of ND requests each are in flight
template <int MAX, int ND> __device__ __forceinline__ void wait_units(int units) {
  if constexpr (MAX == 0) wait_vmcnt<0>();
  else if (units >= MAX) wait_vmcnt<MAX * ND>();
  else wait_units<MAX - 1, ND>(units);
}
// The loop of pipe_body and tn_body over U units of four k-steps in two groups. read(buf, h, i, slot): read i < NR of group h of the unit in
// `slot` into register set buf; landed(buf): they have; mm(buf, i): matrix instruction i < NM of the group in that set;
// request(i, u, slot): request i < ND of unit u; unit_done().
template <int STAGES, int NM, int NR, int ND, typename READ, typename LANDED, typename MM, typename REQ, typename DONE>
__device__ __forceinline__ void unit_loop(int U, READ &&read, LANDED &&landed, MM &&mm, REQ &&request, DONE &&unit_done) {
  static_assert(STAGES >= 2 && (STAGES - 1) * ND <= 63, "vmcnt range");
  for (int s = 0; s < STAGES && s < U; ++s) static_for<ND>([&](auto i) { request(i, s, s); });
  wait_units<STAGES - 1, ND>(U - 1);
  bare_barrier();  // unit 0 is in LDS for everyone
  static_for<NR>([&](auto i) { read(Int<0>{}, Int<0>{}, i, 0); });
  int slot = 0;
  // In the tail (the last STAGES units) nothing is left to request and the wait asks how many units are in flight; reads behind the last unit fetch old bytes of the
  // ring and are dropped. One copy of the matrix instructions per loop: with several, the compiler moves the sums between
  // register sets where the paths meet.
  auto unit = [&](int u, auto tail_c) {
    constexpr bool tail = decltype(tail_c)::value;
    landed(Int<0>{});
    woven<NM, NR, 0>([&](auto i) { mm(Int<0>{}, i); }, [&](auto i) { read(Int<1>{}, Int<1>{}, i, slot); }, [](auto) {});
    landed(Int<1>{});  // every read of unit u
    if constexpr (tail) wait_units<STAGES - 2, ND>(U - 2 - u);
    else wait_vmcnt<(STAGES - 2) * ND>();  // unit u + 1 has landed, younger ones may be in flight
    __builtin_amdgcn_sched_barrier(0);
    bare_barrier();  // unit u + 1 is in LDS for everyone, and everyone is done reading unit u
    __builtin_amdgcn_sched_barrier(0);
    const int free_slot = slot;
    slot = slot + 1 == STAGES ? 0 : slot + 1;
    woven<NM, NR, tail ? 0 : ND>([&](auto i) { mm(Int<1>{}, i); }, [&](auto i) { read(Int<0>{}, Int<0>{}, i, slot); },
                                 [&](auto i) { request(i, u + STAGES, free_slot); });
    unit_done();
  };
  int u = 0;
  for (; u + STAGES < U; ++u) unit(u, std::false_type{});
  for (; u < U; ++u) unit(u, std::true_type{});
  landed(Int<0>{});  // the reads behind the last unit too: their registers are free from here on
}

// SUMS: several ranges of K may be walked in turn (sum_splits; EPI_PARTIAL outside grouped launches)
template <int BM, int BN, int STAGES, int EPI, bool SUMS = EPI == EPI_PARTIAL>
__device__ __forceinline__ void pipe_body(const GemmArgs &g, int bid, int split, int nsplit) {
  typedef bf16_t AT;
  constexpr int BK = 64, KS = 4, NW = 4;
  constexpr int TM = BM / 64, TN = BN / 64;          // 32x32 tiles per wavefront, 2 x 2 wavefronts
  constexpr int GK = 2;                              // k-steps per group of reads
  constexpr int BFR = BN / 32;
  constexpr int A_BYTES = BM * 128;                  // A stage: BM rows of 64 k (128 bytes), 16-byte pieces XOR-swizzled
  constexpr int ACH = BM / 8 / NW;                   // A DMAs per wavefront and stage (one DMA = 8 rows x 128 bytes)
  constexpr int BCH = BFR * KS / NW;                 // W DMAs per wavefront and stage (one fragment)
  constexpr int STAGE_BYTES = A_BYTES + BFR * KS * 1024, LDC = BN + 4;
  static_assert((BM / 8) % NW == 0 && (BFR * KS) % NW == 0, "chunk split");
  extern __shared__ __align__(16) unsigned char smem[];
  float *Cs = reinterpret_cast<float *>(smem);

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / 2, wn = wave % 2;
  const int ntn = g.N / BN, ntm = (g.M + BM - 1) / BM;
  int mt, nt;
  if (!tile_of_block(bid, ntm, ntn, g.col_groups, mt, nt)) return;
  const int m0 = mt * BM, n0 = nt * BN;
  // sum_splits: this workgroup walks all K ranges itself and adds their sums in range order, which is
  // bit for bit what the reducing kernels make of separate partials; otherwise it owns the one range `split`.
  const bool fuse = SUMS && g.sum_splits != 0;
  const int range = g.K / nsplit / BK, kb0 = fuse ? 0 : split * range, units = fuse ? g.K / BK : range;

  // DMA sources of this wavefront for one stage.
  // A: DMA c covers rows 8c .. 8c+7; lane i fetches row r = 8c + i/8, 16-byte piece (i % 8) ^ ((r / 2) % 8): eight lanes
  //    read one 128-byte run of a row, and the XOR spreads the pieces that a later fragment read touches (16 rows
  //    x one piece per quarter-wavefront) over all 64 LDS banks.
  // W: DMA c is fragment c / 4 (32 columns), k-step c % 4, already contiguous.
  const auto rsrc_a = dma_rsrc(static_cast<const bf16_t *>(g.A) + (size_t)m0 * g.lda + kb0 * BK);
  const auto rsrc_w = dma_rsrc(static_cast<const bf16_t *>(g.W) + (size_t)n0 * g.K + (size_t)kb0 * KS * 512);
  uint32_t a_vo[ACH], w_so[BCH];
#pragma unroll
  for (int q = 0; q < ACH; ++q) {
    const int r = (wave + NW * q) * 8 + (lane >> 3), rc = m0 + r < g.M ? r : g.M - 1 - m0;
    a_vo[q] = (uint32_t)(rc * g.lda * 2 + (((lane & 7) ^ ((r >> 1) & 7)) << 4));
  }
#pragma unroll
  for (int q = 0; q < BCH; ++q) {
    const int c = wave + NW * q;
    w_so[q] = (uint32_t)(((c / KS) * (g.K / 16) + c % KS) * 1024);
  }
  auto request = [&](auto i_c, int u, int slot) {  // request i of unit u
    constexpr int i = decltype(i_c)::value;
    unsigned char *base = smem + slot * STAGE_BYTES;
    if constexpr (i < ACH) dma16(rsrc_a, a_vo[i], u * (BK * 2), base + (wave + NW * i) * 1024);
    else dma16(rsrc_w, (uint32_t)lane * 16, w_so[i - ACH] + u * (KS * 1024), base + A_BYTES + (wave + NW * (i - ACH)) * 1024);
  };

  // fragment read offsets inside a stage: row r, k-step ks, half h -> r * 128 + (((2 ks + h) ^ ((r / 2) & 7)) * 16), i.e. k-step 0's
  // with 32 ks XORed in (A tile i of the wavefront 4096 bytes = 32 rows further on; W fragment j KS KiB further on)
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)smem;
  const uint32_t a_first = lds0 + (wm * TM * 32 + (lane & 31)) * 128 + (((lane >> 5) ^ ((lane >> 1) & 7)) << 4);
  const uint32_t w_first = lds0 + A_BYTES + wn * TN * KS * 1024 + lane * 16;
  bf16x8 af[2][GK][TM], bf[2][GK][TN];
  auto read = [&](auto buf_c, auto h_c, auto i_c, int slot) {  // read i of group h of the unit in `slot`
    constexpr int buf = decltype(buf_c)::value, i = decltype(i_c)::value, k = i / (TM + TN), x = i % (TM + TN), ks = decltype(h_c)::value * GK + k;
    if constexpr (x < TN) bf[buf][k][x] = lds_read16<ks * 1024 + x * KS * 1024>(w_first + slot * STAGE_BYTES);
    else af[buf][k][x - TN] = lds_read16<(x - TN) * 4096>((a_first + slot * STAGE_BYTES) ^ (ks * 32));
  };
  auto landed = [&](auto buf_c) {
    constexpr int buf = decltype(buf_c)::value;
    lds_wait<0>();
#pragma unroll
    for (int k = 0; k < GK; ++k) {
#pragma unroll
      for (int i = 0; i < TM; ++i) lds_landed(af[buf][k][i]);
#pragma unroll
      for (int j = 0; j < TN; ++j) lds_landed(bf[buf][k][j]);
    }
  };
  f32x16 acc[TM][TN], tot[SUMS ? TM : 1][SUMS ? TN : 1];
  auto clear = [&] {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;
  };
  clear();
  auto mm = [&](auto buf_c, auto x_c) {
    constexpr int buf = decltype(buf_c)::value, x = decltype(x_c)::value, k = x / (TM * TN), i = x % (TM * TN) / TN, j = x % TN;
    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[buf][k][i], bf[buf][k][j], acc[i][j], 0, 0, 0);
  };
  int in_range = 0;
  bool first = true;
  auto unit_done = [&] {
    if constexpr (SUMS) {
      if (++in_range == range) {
        in_range = 0;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j) {
            if (first) tot[i][j] = acc[i][j];
            else tot[i][j] += acc[i][j];
          }
        first = false;
        clear();
      }
    }
  };
  unit_loop<STAGES, TM * TN * GK, (TM + TN) * GK, ACH + BCH>(units, read, landed, mm, request, unit_done);

  wait_vmcnt<0>();
  __syncthreads();
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int row = (wm * TM + i) * 32 + (e >> 2) * 8 + (lane >> 5) * 4 + (e & 3);
        const int col = (wn * TN + j) * 32 + (lane & 31);
        if constexpr (SUMS) Cs[row * LDC + col] = tot[i][j][e];
        else Cs[row * LDC + col] = acc[i][j][e];
      }
  __syncthreads();
  epilogue<EPI, AT, BM, BN>(g, Cs, m0, n0, nt, tid, fuse ? 0 : split);
}
template <int BM, int BN, int STAGES, int EPI>
__global__ __launch_bounds__(256, STAGES == 2 ? 2 : 1) void gemm_pipe_kernel(GemmArgs g) {
  pipe_body<BM, BN, STAGES, EPI>(g, (int)blockIdx.x, (int)blockIdx.y, g.sum_splits ? g.splits : (int)gridDim.y);
}


// ---------------------------------------------------------------------------------------------------
// Eq. 9's gate | value product where its tiles are too few to fill the chip (M = 1024, N = 512: 64 of 64 x 128): folded LayerNorm and GeGLU
// in the epilogue all the same, K = 2048 walked by two groups of four wavefronts, each with its own ring, side by side. The sum is
// that of g.splits ranges of K added in range order, as a pass over many steps adds them (GEMM_PARTIAL with sum_splits, then
// geglu_kernel) and to the same bits: group 0 adds the first half of the ranges as it goes, group 1 keeps its ranges' sums apart,
// and they are added to group 0's one by one at the end.
// In place of fp32 partials of 128 x 128 tiles (64 KiB written by every workgroup and read back by the GeGLU kernel), us for the two
// launches and for the one: M = 1024, N = 512, K = 2048, 8 ranges 12.9 + 6.3 -> 12.9; M = 1500, N = 384, K = 1024
// 14.5 + 6.2 -> 9.8; M = 128, N = 1024, K = 512 7.2 + 4.1 -> 8.0. Tiles of 32 rows (with 64, on half the compute units, 16.5 / 12.7 / 11.8) up to 256 of them.
// ---------------------------------------------------------------------------------------------------
template <int BM> struct FnrRing {
  static constexpr int stages = BM == 32 ? 4 : 3, unit = BM * 128 + 128 * 128, bytes = 2 * stages * unit;
};
template <int BM>  // 32 or 64 rows x 128 columns
__global__ __launch_bounds__(512, 1) void gemm_fnr_kernel(GemmArgs g) {
  typedef bf16_t AT;
  constexpr int BN = 128, KS = 4, NW = 4, WN = BM == 32 ? 4 : 2, TN = 4 / WN, GK = 2, UNIT = FnrRing<BM>::unit, A_BYTES = BM * 128, ACH = BM / 8 / NW, BCH = BN / 32 * KS / NW, LDC = BN + 4;
  constexpr int OWN = 4;  // ranges a group can keep
  static_assert(FnrRing<BM>::bytes <= 160 * 1024 && OWN * BM * BN * 4 <= FnrRing<BM>::bytes && BM * LDC * 4 <= FnrRing<BM>::bytes, "LDS");
  extern __shared__ __align__(16) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63, wave8 = __builtin_amdgcn_readfirstlane(tid >> 6), grp = wave8 >> 2, wave = wave8 & 3;
  const int wm = wave / WN, wn = wave % WN;
  const int ntn = g.N / BN, ntm = (g.M + BM - 1) / BM;
  int mt, nt;
  if (!tile_of_block((int)blockIdx.x, ntm, ntn, g.col_groups, mt, nt)) return;
  const int m0 = mt * BM, n0 = nt * BN;
  const int range = g.K / 64 / g.splits, own = g.splits / 2, units = own * range, kb0 = grp * units;
  unsigned char *ring = smem + grp * (FnrRing<BM>::bytes / 2);

  // requests and reads as in pipe_body
  const auto rsrc_a = dma_rsrc(static_cast<const bf16_t *>(g.A) + (size_t)m0 * g.lda + kb0 * 64);
  const auto rsrc_w = dma_rsrc(static_cast<const bf16_t *>(g.W) + (size_t)n0 * g.K + (size_t)kb0 * KS * 512);
  uint32_t a_vo[ACH], w_so[BCH];
#pragma unroll
  for (int q = 0; q < ACH; ++q) {
    const int r = (wave + NW * q) * 8 + (lane >> 3), rc = m0 + r < g.M ? r : g.M - 1 - m0;
    a_vo[q] = (uint32_t)(rc * g.lda * 2 + (((lane & 7) ^ ((r >> 1) & 7)) << 4));
  }
#pragma unroll
  for (int q = 0; q < BCH; ++q) {
    const int c = wave + NW * q;
    w_so[q] = (uint32_t)(((c / KS) * (g.K / 16) + c % KS) * 1024);
  }
  auto request = [&](auto i_c, int u, int slot) {
    constexpr int i = decltype(i_c)::value;
    unsigned char *base = ring + slot * UNIT;
    if constexpr (i < ACH) dma16(rsrc_a, a_vo[i], u * 128, base + (wave + NW * i) * 1024);
    else dma16(rsrc_w, (uint32_t)lane * 16, w_so[i - ACH] + u * (KS * 1024), base + A_BYTES + (wave + NW * (i - ACH)) * 1024);
  };
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)ring;
  const uint32_t a_first = lds0 + (wm * 32 + (lane & 31)) * 128 + (((lane >> 5) ^ ((lane >> 1) & 7)) << 4);
  const uint32_t w_first = lds0 + A_BYTES + wn * TN * KS * 1024 + lane * 16;
  bf16x8 af[2][GK], bf[2][GK][TN];
  auto read = [&](auto buf_c, auto h_c, auto i_c, int slot) {
    constexpr int buf = decltype(buf_c)::value, i = decltype(i_c)::value, k = i / (1 + TN), x = i % (1 + TN), ks = decltype(h_c)::value * GK + k;
    if constexpr (x < TN) bf[buf][k][x] = lds_read16<ks * 1024 + x * KS * 1024>(w_first + slot * UNIT);
    else af[buf][k] = lds_read16<0>((a_first + slot * UNIT) ^ (ks * 32));
  };
  auto landed = [&](auto buf_c) {
    constexpr int buf = decltype(buf_c)::value;
    lds_wait<0>();
#pragma unroll
    for (int k = 0; k < GK; ++k) {
      lds_landed(af[buf][k]);
#pragma unroll
      for (int j = 0; j < TN; ++j) lds_landed(bf[buf][k][j]);
    }
  };
  f32x16 acc[TN], keep[OWN][TN];  // group 0: keep[0] is the sum of its ranges
  auto clear = [&] {
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[j][e] = 0.0f;
  };
  clear();
#pragma unroll
  for (int r = 0; r < OWN; ++r)
#pragma unroll
    for (int j = 0; j < TN; ++j) keep[r][j] = acc[j];
  auto mm = [&](auto buf_c, auto x_c) {
    constexpr int buf = decltype(buf_c)::value, x = decltype(x_c)::value, k = x / TN, j = x % TN;
    acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[buf][k], bf[buf][k][j], acc[j], 0, 0, 0);
  };
  int in_range = 0, slot_of_range = 0;  // group 0 adds into the one place, group 1 takes the next
  auto unit_done = [&] {
    if (++in_range < range) return;
    in_range = 0;
    static_for<OWN>([&](auto q_c) {
      constexpr int q = decltype(q_c)::value;
      if (slot_of_range == q) {
        asm volatile("");  // a branch: as selects every set of sums would be rewritten
#pragma unroll
        for (int j = 0; j < TN; ++j) keep[q][j] += acc[j];
      }
    });
    slot_of_range += grp;
    clear();
  };
  unit_loop<FnrRing<BM>::stages, TN * GK, (1 + TN) * GK, ACH + BCH>(units, read, landed, mm, request, unit_done);

  wait_vmcnt<0>();
  __syncthreads();  // the rings are no longer being read
  float *part = reinterpret_cast<float *>(smem), *Cs = part;
  const int at = wave * 64 * 16 * TN + lane;  // [range][wavefront][element][lane]: as the registers lie
  if (grp) {
    static_for<OWN>([&](auto q_c) {
      constexpr int q = decltype(q_c)::value;
      if (q < own) {
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int e = 0; e < 16; ++e) part[q * (BM * BN) + at + (j * 16 + e) * 64] = keep[q][j][e];
      }
    });
  }
  __syncthreads();
  if (!grp) {
    for (int q = 0; q < own; ++q)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) keep[0][j][e] += part[q * (BM * BN) + at + (j * 16 + e) * 64];
  }
  __syncthreads();
  if (!grp) {
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e)
        Cs[(wm * 32 + (e >> 2) * 8 + (lane >> 5) * 4 + (e & 3)) * LDC + (wn * TN + j) * 32 + (lane & 31)] = keep[0][j][e];
  }
  __syncthreads();
  epilogue<EPI_GEGLU_FOLD, AT, BM, BN, LDC, 512>(g, Cs, m0, n0, nt, tid);
}

// ---------------------------------------------------------------------------------------------------
// The same product on 256 x 256 tiles, eight wavefronts (2 x 4, 128 x 64 each), one workgroup per compute unit, for batches that
// give every unit a tile. Both operands come in units of 64 along K (32 KiB each: A as rows of 128 bytes, whole cache lines,
// swizzled as in pipe_body; W as ready-made fragments), A through a ring of three, W through a ring of two: 160 KiB of LDS.
// One hand-over (DMA wait, barrier) per unit, between its third and fourth k-step: the fragments of the fourth are in
// registers by then, so behind the barrier the unit's slots are free, and the reads of the next unit's first k-step run under
// the fourth's matrix instructions. unit u requests A of unit u + 2 during its first two k-steps and W of unit u + 2 behind
// its barrier; unit u + 1's barrier waits for both (all but the youngest CH requests).
// What bounds it is the power the matrix cores draw on real data: M = 16384, K = N = 2048 plain 107-109 us (1.27 PFLOP/s) on
// random operands, 79.5 (1.73) on zeros; the ring of 32-wide W stages with a barrier each that this replaces took 117-120 and
// 95, a plain library product 115.7. M = N = K = 8192: 757 us (1.45 PFLOP/s) against 827. What made the difference, each
// on its own (16384 x 2048 x 2048): requests spread between the matrix instructions instead of in front of them 118 -> 115;
// their addresses as a buffer resource with scalar offsets, so that a request needs no vector instruction, 115 -> 112; one
// barrier per 64 of K instead of two 112 -> 109. Four wavefronts of 128 x 128 (a third fewer LDS reads, one wavefront per SIMD):
// 113; two groups of four that alternate between reading and multiplying: 146.
// Every output element sees the same sequence of k-steps as in pipe_body, so both give the same bits.
//
// The epilogue keeps to the wavefront: the operands enter the matrix instructions exchanged (columns of W as rows), so a lane
// holds four consecutive columns of one row, which it parks in its wavefront's own 32 x 64 LDS slab in 16-byte pieces and reads
// back row-wise; no barrier until the row statistics, whose chunk sums meet in LDS at the end. The side inputs of a
// pass are requested a whole slab ahead, those of the first slab before the last unit. A GeGLU tile is gate | value per 128 columns: the
// wavefront then takes 32 gate columns and their 32 value columns.
// ---------------------------------------------------------------------------------------------------
constexpr int PIPE2_LDS = 160 * 1024;
template <int EPI>
__device__ __forceinline__ void pipe2_body(const GemmArgs &g, int bid) {
  typedef bf16_t AT;
  static_assert(EPI == EPI_STORE || EPI == EPI_GLOBAL || EPI == EPI_MIX || EPI == EPI_GATE || EPI == EPI_GEGLU_FOLD || EPI == EPI_PARTIAL, "epilogue");
  constexpr bool kPair = EPI == EPI_GEGLU_FOLD;
  constexpr int BM = 256, BN = 256, NW = 8, KS = 4, AUNITS = 3, WUNITS = 2;
  constexpr int WN = NW / 2;                         // wavefronts 2 (rows) x WN (columns)
  constexpr int TM = BM / 64, TN = BN / (32 * WN), NRD = TM + TN;  // 32x32 tiles per wavefront; fragment reads per k-step
  constexpr int UNIT = BM * 128, A_RING = AUNITS * UNIT;
  constexpr int CH = UNIT / 1024 / NW;               // DMAs per wavefront, operand and unit
  constexpr int FS = kPair ? 2 : 1;                  // distance of the wavefront's two W fragments
  static_assert((AUNITS + WUNITS) * UNIT == PIPE2_LDS && BM == BN && TM == 4 && TN == 2, "LDS, tile");
  extern __shared__ __align__(16) unsigned char smem[];

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const int ntn = g.N / BN, ntm = g.M / BM;
  // EPI_PARTIAL: ranges of K innermost, so that with eight of them an XCD streams one range of both operands
  constexpr bool kPart = EPI == EPI_PARTIAL;
  const int splits = kPart ? g.splits : 1, split = kPart ? bid % splits : 0;
  int mt, nt;
  if (kPart) { mt = bid / splits / ntn; nt = bid / splits % ntn; }
  else if (!tile_of_block(bid, ntm, ntn, g.col_groups, mt, nt)) return;
  const int m0 = mt * BM, n0 = nt * BN;
  const int nku = g.K / 64 / splits;

  // DMA sources: a resource at the tile's first row / fragment, one lane offset each, and scalar offsets per request
  const auto rsrc_a = dma_rsrc(static_cast<const bf16_t *>(g.A) + (size_t)m0 * g.lda + (size_t)split * nku * 64);
  const auto rsrc_w = dma_rsrc(static_cast<const bf16_t *>(g.W) + (size_t)n0 * g.K + (size_t)split * nku * (KS * 512));
  // A: DMA c = wave + NW q covers rows 8c .. 8c + 7, lane i piece (i % 8) ^ ((r / 2) % 8) of row r = 8c + i / 8; as NW is even,
  // (r / 2) % 8 is 4 (wave % 2) + i / 16 for every q
  const uint32_t a_vo = (uint32_t)((lane >> 3) * g.lda * 2 + (((lane & 7) ^ (((wave & 1) << 2) + (lane >> 4))) << 4)), w_vo = (uint32_t)lane * 16;
  const uint32_t a_so = (uint32_t)(wave * 8 * g.lda * 2), a_q = (uint32_t)(NW * 8 * g.lda * 2);
  uint32_t w_so[CH];
#pragma unroll
  for (int q = 0; q < CH; ++q) {
    const int c = wave + NW * q;  // fragment c / 4 (32 columns), k-step c % 4
    w_so[q] = (uint32_t)(((c / KS) * (g.K / 16) + c % KS) * 1024);
  }
  auto dma_a = [&](int q, int u, int slot) {
    dma16(rsrc_a, a_vo, a_so + q * a_q + u * 128, smem + slot * UNIT + (wave + NW * q) * 1024);
  };
  auto dma_w = [&](int q, int u, int slot) {
    dma16(rsrc_w, w_vo, w_so[q] + u * (KS * 1024), smem + A_RING + slot * UNIT + (wave + NW * q) * 1024);
  };
  // fragment reads: row r, piece p of a unit at r * 128 + ((p ^ ((r / 2) % 8)) * 16); k-step ks, half h reads piece 2 ks + h, i.e.
  // the address of k-step 0 with 32 ks XORed in (slots start at multiples of 128)
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)smem;
  const uint32_t a_first = lds0 + (wm * TM * 32 + (lane & 31)) * 128 + (((lane >> 5) ^ ((lane >> 1) & 7)) << 4);
  const uint32_t w_first = lds0 + A_RING + (kPair ? (wn >> 1) * 4 + (wn & 1) : wn * TN) * (KS * 1024) + lane * 16;
  uint32_t a_cur = a_first, w_cur = w_first;

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;
  typedef std::integral_constant<int, 0> I0;
  typedef std::integral_constant<int, 1> I1;
  typedef std::integral_constant<int, 2> I2;
  typedef std::integral_constant<int, 3> I3;
  typedef std::integral_constant<int, 4> I4;
  typedef std::integral_constant<int, 5> I5;
#pragma unroll
  for (int q = 0; q < CH; ++q) dma_a(q, 0, 0);
#pragma unroll
  for (int q = 0; q < CH; ++q) dma_w(q, 0, 0);
  if (nku > 1) {
#pragma unroll
    for (int q = 0; q < CH; ++q) dma_a(q, 1, 1);
#pragma unroll
    for (int q = 0; q < CH; ++q) dma_w(q, 1, 1);
    wait_vmcnt<2 * CH>();
  } else {
    wait_vmcnt<0>();
  }
  bare_barrier();  // unit 0 is in LDS for everyone

  bf16x8 af[2][TM], bf[2][TN];
  auto read = [&](auto buf_c, auto ks_c, auto x_c, uint32_t sa, uint32_t sb) {  // read x of the k-step's NRD
    constexpr int buf = decltype(buf_c)::value, ks = decltype(ks_c)::value, x = decltype(x_c)::value;
    if constexpr (x < TN) bf[buf][x] = lds_read16<ks * 1024 + x * FS * KS * 1024>(sb);
    else af[buf][x - TN] = lds_read16<(x - TN) * 4096>(sa);
  };
  auto landed = [&](auto buf_c) {
    constexpr int buf = decltype(buf_c)::value;
    lds_wait<0>();
#pragma unroll
    for (int i = 0; i < TM; ++i) lds_landed(af[buf][i]);
#pragma unroll
    for (int j = 0; j < TN; ++j) lds_landed(bf[buf][j]);
  };
  // One k-step: the matrix instructions of register buffer `buf` in four pairs, in front of each pair two reads of the next k-step
  // into the other buffer and its share of the k-step's ND requests. The order is fixed (sched_barrier): left alone the
  // compiler gathers the requests behind the barrier, where eight wavefronts' worth of them hold up the matrix instructions.
  auto kstep = [&](auto buf_c, auto nks_c, uint32_t sa, uint32_t sb, auto reads_c, auto nd_c, auto dma) {
    constexpr int buf = decltype(buf_c)::value, ND = decltype(nd_c)::value;
    static_assert(ND <= 4, "one request per pair");
    auto pair = [&](auto i_c, auto x0_c, auto x1_c) {
      constexpr int i = decltype(i_c)::value;
      typedef std::integral_constant<int, 1 - buf> NB;
      if constexpr (decltype(reads_c)::value) {
        if constexpr (decltype(x0_c)::value < NRD) read(NB{}, nks_c, x0_c, sa, sb);
        if constexpr (decltype(x1_c)::value < NRD) read(NB{}, nks_c, x1_c, sa, sb);
      }
      if constexpr (i < ND) dma(i);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bf[buf][j], af[buf][i], acc[i][j], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    };
    typedef std::integral_constant<int, NRD> None;
    pair(I0{}, I0{}, I1{});
    pair(I1{}, I2{}, I3{});
    pair(I2{}, I4{}, I5{});
    pair(I3{}, None{}, None{});
  };
  {
    auto first = [&](auto x_c) { read(I0{}, I0{}, x_c, a_cur, w_cur); };
    first(I0{}); first(I1{}); first(I2{}); first(I3{}); first(I4{}); first(I5{});
  }
  int aslot = 0, afill = 2;  // A slot of this unit and of the unit two further on
  auto none = [](int) {};
  // mode 2: unit u + 2 is requested; 1: nothing is left to request; 0: the last unit
  auto unit = [&](int u, auto mode_c) {
    constexpr int mode = decltype(mode_c)::value;
    typedef std::integral_constant<int, mode == 2 ? CH / 2 : 0> NDA;
    typedef std::integral_constant<int, mode == 2 ? CH : 0> NDW;
    landed(I0{});
    kstep(I0{}, I1{}, a_cur ^ 32, w_cur, std::true_type{}, NDA{}, [&](int q) { dma_a(q, u + 2, afill); });
    landed(I1{});
    kstep(I1{}, I2{}, a_cur ^ 64, w_cur, std::true_type{}, NDA{}, [&](int q) { dma_a(CH / 2 + q, u + 2, afill); });
    landed(I0{});
    kstep(I0{}, I3{}, a_cur ^ 96, w_cur, std::true_type{}, I0{}, none);
    landed(I1{});  // every read of this unit
    if constexpr (mode != 0) {
      if constexpr (mode == 2) wait_vmcnt<CH>();  // unit u + 1 has landed, A of unit u + 2 may be in flight
      else wait_vmcnt<0>();
      __builtin_amdgcn_sched_barrier(0);
      bare_barrier();
      __builtin_amdgcn_sched_barrier(0);
      aslot = aslot == AUNITS - 1 ? 0 : aslot + 1;
      afill = afill == AUNITS - 1 ? 0 : afill + 1;
      a_cur = a_first + aslot * UNIT;
      w_cur = w_first + ((u + 1) & 1) * UNIT;
      kstep(I1{}, I0{}, a_cur, w_cur, std::true_type{}, NDW{}, [&](int q) { dma_w(q, u + 2, u & 1); });
    } else {
      kstep(I1{}, I0{}, a_cur, w_cur, std::false_type{}, I0{}, none);
    }
  };
  int u = 0;
  for (; u + 2 < nku; ++u) unit(u, I2{});
  if (u + 1 < nku) {
    unit(u, I1{});
    ++u;
  }

  constexpr int LDC = 68;                                    // slab row: 64 columns; 68 keeps writes and reads free of bank conflicts
  constexpr int OCH = kPair ? 4 : 8, RP = 64 / OCH, PASSES = 32 / RP;  // 8-wide output chunks per row, rows per pass, passes per slab
  constexpr int CSP = 17;                                    // pitch of the chunk sums of a row's 128-column piece
  constexpr int SLABS = NW * 32 * LDC * 4, NS = EpiSides<EPI>::n;
  static_assert(SLABS + 2 * BM * CSP * 8 <= PIPE2_LDS, "LDS");
  const int c8 = (lane % OCH) * 8, r0 = lane / OCH;
  const size_t nout = kPair ? (size_t)nt * (BN / 2) + wn * 32 + c8 : (size_t)n0 + wn * 64 + c8;  // first output column of this lane's chunk
  Raw8<AT> sd[NS ? PASSES : 1][2];  // side inputs of the next PASSES passes
  auto side = [&](int i, int p) {
    if constexpr (NS != 0) epi_side_load<EPI, AT>(g, (size_t)(m0 + wm * 128 + i * 32 + p * RP + r0) * g.ldc + nout, true, sd[p]);
  };
  float lam = 0.0f, mean0 = 0.0f, rstd0 = 1.0f;
  if constexpr (EPI == EPI_GLOBAL || EPI == EPI_GATE) lam = g.lam[0];
  FoldCols fc;
  if constexpr (kPair) {
    const int v = n0 + (wn >> 1) * 128 + (wn & 1) * 32 + c8;
    load8(g.fold_s + v, fc.sg); load8(g.fold_t + v, fc.tg);
    load8(g.fold_s + v + 64, fc.sv); load8(g.fold_t + v + 64, fc.tv);
    row_moments(g, m0 + (tid & (BM - 1)), mean0, rstd0);
  }
#pragma unroll
  for (int p = 0; p < PASSES; ++p) side(0, p);
  unit(u, I0{});

  __syncthreads();  // the rings are no longer being read
  float *slab = reinterpret_cast<float *>(smem) + wave * 32 * LDC;
  float2 *sums = reinterpret_cast<float2 *>(smem + SLABS);  // [2 pieces][256 rows][16 chunks]; of a pair: the rows' moments
  if constexpr (kPair) {
    if (tid < BM) sums[tid] = make_float2(mean0, rstd0);
    __syncthreads();
  }
  // keep_c: whether C2 / C3 are written, decided once. The counter of outstanding memory operations is in order and covers stores;
  // for a load older than stores that sit in branches the compiler's wait count assumes the branches not taken, so the wait
  // for the next slab's side inputs would also wait for this slab's stores to be acknowledged.
  auto slabs = [&](auto keep_c) {
  constexpr int KEEP = decltype(keep_c)::value;
#pragma unroll
  for (int i = 0; i < TM; ++i) {
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        *reinterpret_cast<f32x4 *>(slab + (lane & 31) * LDC + j * 32 + q * 8 + (lane >> 5) * 4) = f32x4{acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
    // the wavefront's lanes exchange through its own slab: LDS serves one wavefront's accesses in order
    asm volatile("" ::: "memory");
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int p = 0; p < PASSES; ++p) {
      const int r = p * RP + r0, row = wm * 128 + i * 32 + r;
      const size_t o = (size_t)(m0 + row) * g.ldc + nout;
      float x[8];
      load8(slab + r * LDC + c8, x);
      if constexpr (kPart) {
        store8(static_cast<float *>(g.C) + (size_t)split * g.M * g.ldc + o, x);
      } else if constexpr (kPair) {
        float xv[8];
        load8(slab + r * LDC + 32 + c8, xv);
        const float2 mr = sums[row];
        epi_finish_geglu_fold<AT, KEEP>(g, o, mr.x, mr.y, fc, x, xv);
      } else {
        float out[8];
        epi_finish<EPI, AT, KEEP>(g, o, lam, sd[NS ? p : 0], x, out);
        if (i + 1 < TM) side(i + 1, p);
        if constexpr (EPI != EPI_GLOBAL) {
          if (g.stats_out) {
            float s = 0.0f, q = 0.0f;
#pragma unroll
            for (int k = 0; k < 8; ++k) { s += out[k]; q = fmaf(out[k], out[k], q); }
            sums[((wn >> 1) * BM + row) * CSP + (wn & 1) * 8 + lane % OCH] = make_float2(s, q);
          }
        }
      }
    }
    asm volatile("" ::: "memory");
    __builtin_amdgcn_wave_barrier();
  }
  };
  if (EPI != EPI_STORE && !kPart && g.C2) slabs(std::integral_constant<int, KEEP_YES>{});
  else slabs(std::integral_constant<int, KEEP_NO>{});
  if constexpr (EPI == EPI_STORE || EPI == EPI_MIX || EPI == EPI_GATE) {
    if (g.stats_out) {  // a row's 16 chunk sums per 128 columns, added as the 16-lane butterfly of the smaller tiles adds them
      __syncthreads();
      const int row = tid >> 1, piece = tid & 1;
      const float2 *p = sums + (piece * BM + row) * CSP;
      float2 v[16];
#pragma unroll
      for (int k = 0; k < 16; ++k) v[k] = p[k];
#pragma unroll
      for (int w = 8; w > 0; w >>= 1)
#pragma unroll
        for (int k = 0; k < w; ++k) { v[k].x += v[k + w].x; v[k].y += v[k + w].y; }
      *reinterpret_cast<float2 *>(g.stats_out + ((size_t)(m0 + row) * (g.N / 128) + nt * 2 + piece) * 2) = v[0];
    }
  }
}
template <int EPI> __global__ __launch_bounds__(512, 1) void gemm_pipe2_kernel(GemmArgs g) { pipe2_body<EPI>(g, (int)blockIdx.x); }

// ---------------------------------------------------------------------------------------------------
// Weight gradients from ROW-MAJOR operands: C[M][N] = sum over rows b < K of A[b][m] * W[b][n]  (dW = L^T R over the batch;
// A = a forward activation [a_rows][lda], W = a gradient [K][ldb] whose rows past the batch are zero).
// The contraction index is the row index, which the matrix cores want contiguous per lane; instead of keeping transposed
// copies of all sixteen operands in HBM, the turn happens on the way out of LDS. A stage holds 64 rows of BM (BN) columns
// as they are in memory (LDS-DMA, 1 KiB = 8 rows x 128 bytes or 4 rows x 256 bytes per instruction), and fragments are
// read with gfx950's transposing LDS load (ds_read_b64_tr_b16): within each group of 16 lanes, lane s supplies the
// address of 4 consecutive 16-bit values, and lane i receives value (i % 4) of the lanes i / 4, i / 4 + 4, i / 4 + 8,
// i / 4 + 12 (layout checked on the hardware). Pointing lane s at row s / 4, columns 4 (s % 4) .. + 3 of a 4 x 16 block
// therefore hands lane i column i of the block with its 4 rows in order: two such loads give a lane the 8 contraction
// rows of its column, which is the operand layout of v_mfma_f32_32x32x16_bf16.
// Bank conflicts: one load touches 4 rows x 64 contiguous bytes per 32 lanes; with a row pitch of 128 (256) bytes those
// rows would share banks, so the 16-byte pieces of a row are XOR-permuted by a function of the row (below) such that
// 4 consecutive rows land in 4 different quarter-ranges of the 64 banks.
// ---------------------------------------------------------------------------------------------------
typedef __attribute__((ext_vector_type(4))) short i16x4;
typedef __attribute__((ext_vector_type(8))) short i16x8;
// piece permutation of row r in a stage whose rows are PITCH bytes long
template <int PITCH> __device__ __forceinline__ int tn_swizzle(int r) {
  static_assert(PITCH == 128 || PITCH == 256, "row pitch");
  return PITCH == 256 ? ((r & 3) << 2) : (((r >> 1) & 1) << 2);
}

template <int BM, int BN, int STAGES>
__device__ __forceinline__ void tn_body(const GemmArgs &g, int bid, int split = 0, int nsplit = 1) {
  typedef bf16_t AT;
  constexpr int BK = 64, NW = 4;
  constexpr int TM = BM / 64, TN = BN / 64;
  constexpr int GK = 2;                            // k-steps per group of reads
  constexpr int PA = BM / 8, PB = BN / 8;          // 16-byte pieces per row
  constexpr int RA = 64 / PA, RB = 64 / PB;        // rows per DMA
  constexpr int A_BYTES = BK * BM * 2, B_BYTES = BK * BN * 2;
  constexpr int ACH = BK / RA / NW, BCH = BK / RB / NW;  // DMAs per wavefront and stage
  constexpr int STAGE_BYTES = A_BYTES + B_BYTES, LDC = BN + 4;
  static_assert(PA >= 8 && PB >= 8 && (BK / RA) % NW == 0 && (BK / RB) % NW == 0, "tile shape");
  extern __shared__ __align__(16) unsigned char smem[];
  float *Cs = reinterpret_cast<float *>(smem);

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / 2, wn = wave % 2;
  const int ntn = g.N / BN, ntm = g.M / BM;
  int mt, nt;
  if (!tile_of_block(bid, ntm, ntn, 8, mt, nt)) return;
  const int m0 = mt * BM, n0 = nt * BN;
  const int units = g.K / BK / nsplit, kb0 = split * units;  // this workgroup's range of the contraction (the batch)

  // DMA c of an operand covers rows c * R .. c * R + R - 1 of the stage; lane i lands at byte 16 i of that KiB, i.e. at
  // (row, piece) = (c * R + i / P, i % P), and fetches the piece whose index is XORed as described above.
  int a_row[ACH], a_piece[ACH];
  uint32_t b_vo[BCH];
#pragma unroll
  for (int q = 0; q < ACH; ++q) {
    a_row[q] = (wave + NW * q) * RA + lane / PA;
    a_piece[q] = ((lane % PA) ^ tn_swizzle<BM * 2>(a_row[q])) * 16;
  }
#pragma unroll
  for (int q = 0; q < BCH; ++q) {
    const int row = (wave + NW * q) * RB + lane / PB;
    b_vo[q] = (uint32_t)(row * g.ldb * 2 + ((lane % PB) ^ tn_swizzle<BN * 2>(row)) * 16);
  }
  uint32_t a_vo[ACH];
#pragma unroll
  for (int q = 0; q < ACH; ++q) a_vo[q] = (uint32_t)(a_row[q] * g.lda * 2 + a_piece[q]);
  const bf16_t *a_src = static_cast<const bf16_t *>(g.A) + (size_t)kb0 * BK * g.lda + m0, *b_src = static_cast<const bf16_t *>(g.W) + (size_t)kb0 * BK * g.ldb + n0;
  auto request = [&](auto i_c, int u, int slot) {  // request i of unit u
    constexpr int i = decltype(i_c)::value;
    unsigned char *base = smem + slot * STAGE_BYTES;
    if constexpr (i < ACH) {
      const int rows = g.a_rows - (kb0 + u) * BK;  // that exist from the unit's first row on
      const auto rs = dma_rsrc(a_src + (size_t)u * BK * g.lda);
      if (rows >= BK) {
        dma16(rs, a_vo[i], 0, base + (wave + NW * i) * 1024);
      } else {  // past the batch: any finite row, its partner row of W is zero
        const int r = a_row[i] < rows ? a_row[i] : rows - 1;
        dma16(rs, r * g.lda * 2 + a_piece[i], 0, base + (wave + NW * i) * 1024);
      }
    } else {
      dma16(dma_rsrc(b_src + (size_t)u * BK * g.ldb), b_vo[i - ACH], 0, base + A_BYTES + (wave + NW * (i - ACH)) * 1024);
    }
  };

  // address this lane supplies to the transposing loads of k-step 0 (first of the two loads; the second is 4 rows on):
  // row 8 * (lane / 32) + (lane % 16) / 4, columns tile * 32 + 16 * ((lane / 16) % 2) + 4 * (lane % 4) .. + 3
  const int s16 = lane & 15, r0 = (lane >> 5) * 8 + (s16 >> 2), mh = (lane >> 4) & 1;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)smem;
  uint32_t a_off[TM], b_off[TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
    a_off[i] = lds0 + r0 * (BM * 2) + ((((wm * TM + i) * 4 + 2 * mh + ((s16 & 3) >> 1)) ^ tn_swizzle<BM * 2>(r0)) << 4) + (s16 & 1) * 8;
#pragma unroll
  for (int j = 0; j < TN; ++j)
    b_off[j] = lds0 + A_BYTES + r0 * (BN * 2) + ((((wn * TN + j) * 4 + 2 * mh + ((s16 & 3) >> 1)) ^ tn_swizzle<BN * 2>(r0)) << 4) + (s16 & 1) * 8;
  // rows 4 and 16 further on have the same (r & 3) and the same ((r >> 1) & 1): the permutation term does not change

  // The transposing reads go through inline assembly with hand-placed waits (tr_read8 / lds_wait / tr_landed): issued through
  // the builtin, the compiler orders every one of them behind the LDS-DMA just requested for a later stage
  // (s_waitcnt vmcnt(0) in front of the first read), which exposes a full memory latency per stage.
  i32x2 alo[2][GK][TM], ahi[2][GK][TM], blo[2][GK][TN], bhi[2][GK][TN];
  auto read = [&](auto buf_c, auto h_c, auto i_c, int slot) {  // pair i of group h of the unit in `slot`
    constexpr int buf = decltype(buf_c)::value, i = decltype(i_c)::value, k = i / (TM + TN), x = i % (TM + TN), ks = decltype(h_c)::value * GK + k;
    if constexpr (x < TN) {
      blo[buf][k][x] = tr_read8<ks * 16 * (BN * 2)>(b_off[x] + slot * STAGE_BYTES);
      bhi[buf][k][x] = tr_read8<ks * 16 * (BN * 2) + 4 * (BN * 2)>(b_off[x] + slot * STAGE_BYTES);
    } else {
      alo[buf][k][x - TN] = tr_read8<ks * 16 * (BM * 2)>(a_off[x - TN] + slot * STAGE_BYTES);
      ahi[buf][k][x - TN] = tr_read8<ks * 16 * (BM * 2) + 4 * (BM * 2)>(a_off[x - TN] + slot * STAGE_BYTES);
    }
  };
  bf16x8 af[GK][TM], bf[GK][TN];
  auto landed = [&](auto buf_c) {
    constexpr int buf = decltype(buf_c)::value;
    lds_wait<0>();
#pragma unroll
    for (int k = 0; k < GK; ++k) {
#pragma unroll
      for (int i = 0; i < TM; ++i) { tr_landed(alo[buf][k][i]); tr_landed(ahi[buf][k][i]); af[k][i] = tr_pair(alo[buf][k][i], ahi[buf][k][i]); }
#pragma unroll
      for (int j = 0; j < TN; ++j) { tr_landed(blo[buf][k][j]); tr_landed(bhi[buf][k][j]); bf[k][j] = tr_pair(blo[buf][k][j], bhi[buf][k][j]); }
    }
  };
  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;
  auto mm = [&](auto, auto x_c) {
    constexpr int x = decltype(x_c)::value, k = x / (TM * TN), i = x % (TM * TN) / TN, j = x % TN;
    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[k][i], bf[k][j], acc[i][j], 0, 0, 0);
  };
  unit_loop<STAGES, TM * TN * GK, (TM + TN) * GK, ACH + BCH>(units, read, landed, mm, request, [] {});

  wait_vmcnt<0>();
  __syncthreads();
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int row = (wm * TM + i) * 32 + (e >> 2) * 8 + (lane >> 5) * 4 + (e & 3);
        const int col = (wn * TN + j) * 32 + (lane & 31);
        Cs[row * LDC + col] = acc[i][j][e];
      }
  __syncthreads();
  epilogue<EPI_GRAD, AT, BM, BN>(g, Cs, m0, n0, nt, tid, split);
}
// ---------------------------------------------------------------------------------------------------
// The same on 256 x 256 tiles, eight wavefronts (2 x 4, 128 x 64 each), for large batches: all such matrices of a backward pass in
// one launch, one workgroup per compute unit (Tn2Group). Every tile's contraction is summed in a few equal ranges of the batch
// (fade_tile_ranges), as slices that the Adam pass adds in order; these pieces are laid end to end and cut into 256 equal shares
// (fade_tile_plan), so no round of the chip is left half full whatever their number. D_h = 2048, D_cache = D_e = 512, 16384 rows: 192
// tiles in 4 ranges, three whole pieces per workgroup; 4096 rows: 2 ranges, a share is one and a half pieces.
// An XCD's workgroups are on neighbouring tiles (blocks of 2 x 4) of one range at a time, so six operand panels in its L2 serve eight.
// The K loop is pipe2_body's: units of 64 rows of the batch (32 KiB per operand, rows of 512 bytes as they lie in memory), L through a
// ring of three, R through a ring of two, one hand-over per unit, requests with scalar offsets spread between the matrix
// instructions. It does not stop at the end of a piece: the requests run two units ahead into the next one while the sums
// leave as they lie in the registers (a lane holds a column: 128-byte runs).
// B = 16384 (411 Gflop): 336 us (1.22 PFLOP/s) against 375 for a launch of 768 workgroups; with shares that cut whole tiles, half the
// slices and chains of up to 12288 rows 325, and 87 us in the Adam pass against 104.
// ---------------------------------------------------------------------------------------------------
constexpr int TN2_LDS = 160 * 1024;
__global__ __launch_bounds__(512, 1) void gemm_tn2_kernel(Tn2Group tg) {
  constexpr int NW = 8, TM = 4, TN = 2, AUNITS = 3, UNIT = 64 * 512, R_RING = AUNITS * UNIT, CH = UNIT / 1024 / NW;
  extern __shared__ __align__(16) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 2, wn = wave & 3;
  const FadeTilePlan pl = tg.plan;
  const int xcd = (int)blockIdx.x & 7, slot = (int)blockIdx.x >> 3, grp = slot / pl.wgs, member = slot - grp * pl.wgs;
  if (grp >= pl.groups) return;
  const int begin = member * pl.per_wg, end = fade_tile_end(pl, tg.pieces, xcd, grp, member);
  if (begin >= end) return;

  // requests: one cursor two units ahead of the arithmetic. j: piece (position in the group), k: unit of it
  struct Cursor { int j, k; } f{begin / pl.units, begin % pl.units}, c = f;
  const bf16_t *pa = nullptr, *pb = nullptr;  // first row of the unit the cursor stands at, first column of the tile
  int lda = 0, ldb = 0, rows = 0;             // rows of L that exist from that row on
  auto open = [&](const Cursor &t) {
    const uint32_t e = (uint32_t)__builtin_amdgcn_readfirstlane((int)tg.order[fade_tile_seq(pl, xcd, grp, t.j)].at);
    const GemmArgs &g = tg.g[e >> 28];
    const int first = ((int)((e >> 24) & 15) * pl.units + t.k) * 64;
    lda = g.lda; ldb = g.ldb;
    pa = static_cast<const bf16_t *>(g.A) + (size_t)first * lda + (size_t)((e >> 12) & 0xfff) * 256;
    pb = static_cast<const bf16_t *>(g.W) + (size_t)first * ldb + (size_t)(e & 0xfff) * 256;
    rows = g.a_rows - first;
  };
  open(f);
  auto advance = [&](int u) {  // to the unit behind u (counted like begin); nothing past the end
    if (u + 1 >= end) return;
    if (++f.k == pl.units) { f.k = 0; ++f.j; open(f); }
    else { pa += (size_t)64 * lda; pb += (size_t)64 * ldb; rows -= 64; }
  };
  // DMA c = wave + NW q covers rows 2c, 2c + 1 of the unit; lane i lands at byte 16 i of that KiB, i.e. at row 2c + i / 32, piece i % 32,
  // and fetches the piece whose index is XORed with 4 (row % 4); as NW is even, row % 4 is 2 (wave % 2) + i / 32 for every q
  const int lrow = lane >> 5, lpiece = ((lane & 31) ^ ((((wave & 1) << 1) + lrow) << 2)) << 4;
  auto request_l = [&](int q, int s) {
    const int r = 2 * (wave + NW * q);
    unsigned char *dst = smem + s * UNIT + (wave + NW * q) * 1024;
    if (rows >= 64) {
      dma16(dma_rsrc(pa), lrow * lda * 2 + lpiece, r * lda * 2, dst);
    } else {  // past the batch: any finite row, its partner row of R is zero
      const int rr = r + lrow < rows ? r + lrow : rows - 1;
      dma16(dma_rsrc(pa), rr * lda * 2 + lpiece, 0, dst);
    }
  };
  auto request_r = [&](int q, int s) {
    dma16(dma_rsrc(pb), lrow * ldb * 2 + lpiece, 2 * (wave + NW * q) * ldb * 2, smem + R_RING + s * UNIT + (wave + NW * q) * 1024);
  };

  // addresses this lane supplies to the transposing reads of k-step 0 (see tn_body); tile i's differ in two bits that no row changes
  const int s16 = lane & 15, r0 = (lane >> 5) * 8 + (s16 >> 2), mh = (lane >> 4) & 1;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)smem;
  const uint32_t col = (uint32_t)(r0 * 512 + ((2 * mh + ((s16 & 3) >> 1)) << 4) + (s16 & 1) * 8);
  uint32_t l_off[TM], r_off[TN];
#pragma unroll
  for (int i = 0; i < TM; ++i) l_off[i] = lds0 + col + ((((wm * TM + i) ^ (r0 & 3)) & 7) << 6);
#pragma unroll
  for (int j = 0; j < TN; ++j) r_off[j] = lds0 + R_RING + col + ((((wn * TN + j) ^ (r0 & 3)) & 7) << 6);

  f32x16 acc[TM][TN];
  auto clear = [&] {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;
  };
  clear();
  typedef std::integral_constant<int, 0> I0;
  typedef std::integral_constant<int, 1> I1;
  typedef std::integral_constant<int, 2> I2;
  typedef std::integral_constant<int, 3> I3;
#pragma unroll
  for (int q = 0; q < CH; ++q) request_l(q, 0);
#pragma unroll
  for (int q = 0; q < CH; ++q) request_r(q, 0);
  if (begin + 1 < end) {
    advance(begin);
#pragma unroll
    for (int q = 0; q < CH; ++q) request_l(q, 1);
#pragma unroll
    for (int q = 0; q < CH; ++q) request_r(q, 1);
    advance(begin + 1);
    wait_vmcnt<2 * CH>();
  } else {
    wait_vmcnt<0>();
  }
  bare_barrier();

  i32x2 llo[2][TM], lhi[2][TM], rlo[2][TN], rhi[2][TN];
  auto read_l = [&](auto buf_c, auto ks_c, auto i_c, uint32_t base) {
    constexpr int buf = decltype(buf_c)::value, ks = decltype(ks_c)::value, i = decltype(i_c)::value;
    llo[buf][i] = tr_read8<ks * 16 * 512>(base + l_off[i]);
    lhi[buf][i] = tr_read8<ks * 16 * 512 + 4 * 512>(base + l_off[i]);
  };
  auto read_r = [&](auto buf_c, auto ks_c, auto j_c, uint32_t base) {
    constexpr int buf = decltype(buf_c)::value, ks = decltype(ks_c)::value, j = decltype(j_c)::value;
    rlo[buf][j] = tr_read8<ks * 16 * 512>(base + r_off[j]);
    rhi[buf][j] = tr_read8<ks * 16 * 512 + 4 * 512>(base + r_off[j]);
  };
  bf16x8 lf[TM], rf[TN];
  auto landed = [&](auto buf_c) {
    constexpr int buf = decltype(buf_c)::value;
    lds_wait<0>();
#pragma unroll
    for (int i = 0; i < TM; ++i) { tr_landed(llo[buf][i]); tr_landed(lhi[buf][i]); lf[i] = tr_pair(llo[buf][i], lhi[buf][i]); }
#pragma unroll
    for (int j = 0; j < TN; ++j) { tr_landed(rlo[buf][j]); tr_landed(rhi[buf][j]); rf[j] = tr_pair(rlo[buf][j], rhi[buf][j]); }
  };
  // one k-step as in pipe2_body: the reads of the next one and the requests in front of the pairs of matrix instructions
  auto kstep = [&](auto buf_c, auto nks_c, uint32_t lbase, uint32_t rbase, auto reads_c, auto req) {
    typedef std::integral_constant<int, 1 - decltype(buf_c)::value> NB;
    constexpr bool reads = decltype(reads_c)::value;
    auto pair = [&](auto i_c) {
      constexpr int i = decltype(i_c)::value;
      if constexpr (reads) {
        if constexpr (i < TN) { read_r(NB{}, nks_c, i_c, rbase); read_l(NB{}, nks_c, i_c, lbase); }
        else read_l(NB{}, nks_c, i_c, lbase);
      }
      req(i);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lf[i], rf[j], acc[i][j], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    };
    pair(I0{}); pair(I1{}); pair(I2{}); pair(I3{});
  };
  // the sums of the piece the arithmetic has finished, or of the part of it that is this workgroup's
  auto store = [&] {
    const Tn2Piece *piece = tg.order + fade_tile_seq(pl, xcd, grp, c.j);
    const uint32_t e = (uint32_t)__builtin_amdgcn_readfirstlane((int)piece->at);
    const GemmArgs &g = tg.g[e >> 28];
    const int slice = __builtin_amdgcn_readfirstlane((int)piece->slice) + member - fade_tile_first(pl, c.j);
    const int m = (int)((e >> 12) & 0xfff) * 256 + wm * 128 + (lane >> 5) * 4, n = (int)(e & 0xfff) * 256 + wn * 64;
    // a pair of matrices, columns interleaved per 64: the wavefront's 64 columns belong to one of them
    float *dst = static_cast<float *>(g.C3 && (n & 64) ? g.C3 : g.C);
    const int width = g.C3 ? g.N / 2 : g.N, n1 = g.C3 ? (n >> 7) * 64 : n;
    dst += (size_t)slice * g.M * width + (size_t)m * width + n1 + (lane & 31);
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int e16 = 0; e16 < 16; ++e16)
#pragma unroll
        for (int j = 0; j < TN; ++j) dst[(size_t)(i * 32 + (e16 >> 2) * 8 + (e16 & 3)) * width + j * 32] = acc[i][j][e16];
    clear();
  };
#pragma unroll
  for (int j = 0; j < 1; ++j) {
    read_r(I0{}, I0{}, I0{}, 0); read_r(I0{}, I0{}, I1{}, 0);
    read_l(I0{}, I0{}, I0{}, 0); read_l(I0{}, I0{}, I1{}, 0); read_l(I0{}, I0{}, I2{}, 0); read_l(I0{}, I0{}, I3{}, 0);
  }
  int aslot = 0, afill = 2;
  auto none = [](int) {};
  // mode 2: unit u + 2 is requested; 1: nothing is left to request; 0: the last unit
  auto unit = [&](int u, auto mode_c) {
    constexpr int mode = decltype(mode_c)::value;
    const uint32_t lb = aslot * UNIT, rb = ((u - begin) & 1) * UNIT;
    auto req_l0 = [&](int i) { if constexpr (mode == 2) { if (i < CH / 2) request_l(i, afill); } };
    auto req_l1 = [&](int i) { if constexpr (mode == 2) { if (i < CH / 2) request_l(CH / 2 + i, afill); } };
    auto req_r = [&](int i) { if constexpr (mode == 2) request_r(i, (u - begin) & 1); };
    landed(I0{});
    kstep(I0{}, I1{}, lb, rb, std::true_type{}, req_l0);
    landed(I1{});
    kstep(I1{}, I2{}, lb, rb, std::true_type{}, req_l1);
    landed(I0{});
    kstep(I0{}, I3{}, lb, rb, std::true_type{}, none);
    landed(I1{});
    if constexpr (mode != 0) {
      if constexpr (mode == 2) wait_vmcnt<CH>();  // unit u + 1 has landed, L of unit u + 2 may be in flight
      else wait_vmcnt<0>();
      __builtin_amdgcn_sched_barrier(0);
      bare_barrier();
      __builtin_amdgcn_sched_barrier(0);
      aslot = aslot == AUNITS - 1 ? 0 : aslot + 1;
      afill = afill == AUNITS - 1 ? 0 : afill + 1;
      kstep(I1{}, I0{}, aslot * UNIT, rb ^ UNIT, std::true_type{}, req_r);
      if constexpr (mode == 2) advance(u + 2);
    } else {
      kstep(I1{}, I0{}, lb, rb, std::false_type{}, none);
    }
    if (++c.k == pl.units || mode == 0) {
      store();
      c.k = 0; ++c.j;
    }
  };
  int u = begin;
  for (; u + 2 < end; ++u) unit(u, I2{});
  if (u + 1 < end) {
    unit(u, I1{});
    ++u;
  }
  unit(u, I0{});
}

// Several independent products in ONE launch (a block-uniform switch picks the problem and its kernel body): the products
// of one backward phase (dX = dY W^T, dW = L^T dY, ...) consume the same gradient and do not depend on each other, and at
// B = 1024 none of them fills the chip alone.
template <int STAGES>
__device__ __forceinline__ void group_body(const GemmGroup &gg) {
  int p = 0;
  while (p + 1 < gg.count && (int)blockIdx.x >= gg.first_block[p + 1]) ++p;
  const int local = (int)blockIdx.x - gg.first_block[p], tiles = gg.tiles[p];
  const GemmArgs &g = gg.g[p];
  switch (gg.kind[p]) {
    case GK_STORE_64x128:   pipe_body<64, 128, STAGES, EPI_STORE>(g, local, 0, 1); break;
    case GK_STORE_128x128:  pipe_body<128, 128, STAGES, EPI_STORE>(g, local, 0, 1); break;
    case GK_STORE_64x64:    pipe_body<64, 64, STAGES, EPI_STORE>(g, local, 0, 1); break;
    case GK_PARTIAL_64x64:  pipe_body<64, 64, STAGES, EPI_PARTIAL, false>(g, local % tiles, local / tiles, gg.splits[p]); break;
    case GK_PARTIAL_128x128: pipe_body<128, 128, STAGES, EPI_PARTIAL, false>(g, local % tiles, local / tiles, gg.splits[p]); break;
    case GK_TN_64x128:      tn_body<64, 128, STAGES>(g, local % tiles, local / tiles, gg.splits[p]); break;
    case GK_TN_128x128:     tn_body<128, 128, STAGES>(g, local % tiles, local / tiles, gg.splits[p]); break;
    case GK_TN_64x64:       tn_body<64, 64, STAGES>(g, local % tiles, local / tiles, gg.splits[p]); break;
    default: break;
  }
}
__global__ __launch_bounds__(256) void gemm_group_kernel(GemmGroup gg) { group_body<4>(gg); }
// The same with two-stage rings and at most 256 registers: two workgroups share a compute unit, so one's pipeline fill and
// epilogue run under the other's products. For groups with workgroups enough to use that (large batches).
__global__ __launch_bounds__(256, 2) void gemm_group2_kernel(GemmGroup gg) { group_body<2>(gg); }


// ---------------------------------------------------------------------------------------------------
// fp32 FMA core: 256 threads, each owning 8 consecutive columns of one row; tile (2048 / BN) x BN,
// K blocks of 32; W is plain [K][N] fp32
// ---------------------------------------------------------------------------------------------------
template <int BN, int PRO, int EPI>
__global__ __launch_bounds__(256) void gemm_f32_kernel(GemmArgs g) {
  typedef float AT;
  constexpr int CHN = BN / 8, BM = 256 / CHN, BK = 32, LDC = BN + 4;
  constexpr int NCH = (BM * 4 + 255) / 256;  // A chunks staged per thread
  __shared__ __align__(16) float As[BM][BK + 4];
  __shared__ __align__(16) float Ws[BK][BN];
  __shared__ __align__(16) float Cs[BM * LDC];
  const int tid = threadIdx.x;
  const int ntn = g.N / BN;
  const int nt = blockIdx.x % ntn, mt = blockIdx.x / ntn;
  const int m0 = mt * BM, n0 = nt * BN;
  const int r = tid / CHN, cg = (tid % CHN) * 8;  // this thread's output row and first column
  float mean[NCH], rstd[NCH], lam = 0.0f;
#pragma unroll
  for (int q = 0; q < NCH; ++q) {
    mean[q] = 0.0f; rstd[q] = 1.0f;
    const int c = q * 256 + tid;
    if ((PRO == PRO_LN || PRO == PRO_FINAL) && c < BM * 4) row_moments(g, m0 + (c >> 2), mean[q], rstd[q]);
  }
  if (PRO == PRO_FINAL) lam = g.lam[0];
  float acc[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) acc[i] = 0.0f;
  const float *W = static_cast<const float *>(g.W);
  for (int k0 = 0; k0 < g.K; k0 += BK) {
#pragma unroll
    for (int q = 0; q < NCH; ++q) {
      const int c = q * 256 + tid;
      if (c < BM * 4) {
        const int srow = c >> 2, skc = (c & 3) * 8;
        Raw8<AT> a, a2;
        stage_load<PRO, AT>(g, m0 + srow, k0 + skc, a, a2);
        float v[8];
        stage_transform<PRO, AT>(g, k0 + skc, a, a2, mean[q], rstd[q], lam, v);
#pragma unroll
        for (int i = 0; i < 8; ++i) As[srow][skc + i] = v[i];
      }
    }
    if (g.wt) {  // W given as [N][ldb]: rows are output columns, K contiguous
      for (int idx = tid; idx < BK * BN; idx += 256) {
        const int c = idx / BK, kk = idx % BK;
        Ws[kk][c] = W[(size_t)(n0 + c) * g.ldb + k0 + kk];
      }
    } else {
      for (int idx = tid; idx < BK * BN / 4; idx += 256) {
        const int kk = idx / (BN / 4), c4 = (idx % (BN / 4)) * 4;
        *reinterpret_cast<f32x4 *>(&Ws[kk][c4]) = *reinterpret_cast<const f32x4 *>(W + (size_t)(k0 + kk) * g.N + n0 + c4);
      }
    }
    __syncthreads();
#pragma unroll 8
    for (int kk = 0; kk < BK; ++kk) {
      const float a = As[r][kk];
      const f32x4 w0 = *reinterpret_cast<const f32x4 *>(&Ws[kk][cg]), w1 = *reinterpret_cast<const f32x4 *>(&Ws[kk][cg + 4]);
#pragma unroll
      for (int i = 0; i < 4; ++i) { acc[i] = fmaf(a, w0[i], acc[i]); acc[4 + i] = fmaf(a, w1[i], acc[4 + i]); }
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < 8; ++i) Cs[r * LDC + cg + i] = acc[i];
  __syncthreads();
  epilogue<EPI, AT, BM, BN>(g, Cs, m0, n0, nt, tid);
}

template <int WM, int WN, int TM, int TN, int PRO, int EPI, bool KEEP = false>
hipError_t launch_bf16(const GemmArgs &g, hipStream_t s) {
  constexpr int BM = WM * TM * 32, BN = WN * TN * 32;
  constexpr size_t lds_a = 2 * BM * (64 + 8) * sizeof(bf16_t), lds_c = (size_t)BM * (BN + 4) * sizeof(float);
  constexpr size_t lds = lds_a > lds_c ? lds_a : lds_c;
  static bool attr_done = false;
  auto kern = gemm_bf16_kernel<WM, WN, TM, TN, PRO, EPI, KEEP>;
  if (KEEP && (g.M % BM || !g.C2)) return hipErrorInvalidValue;
  if (!attr_done) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    attr_done = true;
  }
  const int splits = (EPI == EPI_PARTIAL && g.splits > 1) ? g.splits : 1;
  if (g.N % BN || g.K % (64 * splits) || g.M <= 0 || (EPI != EPI_PARTIAL && (g.splits > 1 || g.sum_splits))) return hipErrorInvalidValue;
  const int grid = ((g.M + BM - 1) / BM) * (g.N / BN);
  hipLaunchKernelGGL(kern, dim3(grid, g.sum_splits ? 1 : splits), dim3(256), lds, s, g);
  return hipGetLastError();
}

// Column ranges of the XCD split (see tile_of_block) by the size of the A operand; FADE_GEMM_XCD overrides for sweeps.
int fade_gemm_col_groups(int M, int K, int N, size_t w_slice = (size_t)2 << 20) {
  static int v = -1;
  if (v < 0) { const char *e = getenv("FADE_GEMM_XCD"); v = e ? atoi(e) : 0; }
  if (v > 0) return v;
  // Router product, M = 16384, N = K = 2048 (A 64 MiB, 200 MiB algorithmic reads): 8 ranges fetch 678 MiB from memory,
  // 4 fetch 467, 2 fetch 433, 1 (rows only; W then streams through every L2) 453, at equal run time within 3 %.
  // Tall A: as few ranges as keep an XCD's slice of W (K x N / ranges, bf16) within 2 MiB, half of its L2.
  if ((size_t)M * K < ((size_t)4 << 20)) return 8;
  int cg = 1;
  while (cg < 8 && (size_t)K * N * 2 / cg > w_slice) cg *= 2;
  return cg;
}

template <int BM, int BN, int STAGES, int EPI>
hipError_t launch_pipe(const GemmArgs &g, hipStream_t s) {
  constexpr int BK = 64;
  constexpr size_t lds_ring = (size_t)STAGES * (BM * 128 + (BN / 32) * 4 * 1024), lds_c = (size_t)BM * (BN + 4) * sizeof(float);
  constexpr size_t lds = lds_ring > lds_c ? lds_ring : lds_c;
  static bool attr_done = false;
  auto kern = gemm_pipe_kernel<BM, BN, STAGES, EPI>;
  if (!attr_done) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    attr_done = true;
  }
  const int splits = g.splits > 1 ? g.splits : 1;
  if (g.N % BN || g.M <= 0 || g.K % (splits * BK) || (EPI != EPI_PARTIAL && splits != 1) || g.lda % 8) return hipErrorInvalidValue;
  GemmArgs ga = g;
  const int ntm = (g.M + BM - 1) / BM, ntn = g.N / BN;
  if (ga.col_groups == 0) ga.col_groups = fade_gemm_col_groups(g.M, g.K, g.N);
  if ((ga.col_groups != 1 && ga.col_groups != 2 && ga.col_groups != 4) || ntn % ga.col_groups) ga.col_groups = 8;
  const int rg = 8 / ga.col_groups;
  if (ga.sum_splits && EPI != EPI_PARTIAL) return hipErrorInvalidValue;
  const dim3 grid((ntn % ga.col_groups == 0 ? (ntm + rg - 1) / rg * rg : ntm) * ntn, ga.sum_splits ? 1 : splits);
  hipLaunchKernelGGL(kern, grid, dim3(256), lds, s, ga);
  return hipGetLastError();
}

}  // namespace
// tg.plan, tg.order, tg.pieces and tg.ranges belong to the context; product p of the group is matrix p of the plan's order.
hipError_t fade_gemm_tn2_launch(const Tn2Group &tg, hipStream_t s) {
  static bool attr_done = false;
  if (!attr_done) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(gemm_tn2_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, TN2_LDS);
    if (e != hipSuccess) return e;
    attr_done = true;
  }
  int tiles = 0;
  for (int p = 0; p < tg.count; ++p) {
    const GemmArgs &g = tg.g[p];
    if (!g.A || !g.W || !g.C || !fade_gemm_tn2_ok(g.M, g.N, g.K) || g.K != tg.ranges * tg.plan.units * 64 || g.a_rows <= 0 || g.a_rows > g.K || g.K - g.a_rows >= 64 ||
        g.lda % 8 || g.ldb % 8 || g.lda < g.M || g.ldb < g.N || g.lda > (1 << 20) || g.ldb > (1 << 20))
      return hipErrorInvalidValue;
    tiles += (g.M / 256) * (g.N / 256);
  }
  if (tg.count <= 0 || tg.count > 8 || tg.ranges < 1 || tg.ranges > 16 || tiles * tg.ranges != tg.pieces || !tg.order) return hipErrorInvalidValue;
  hipLaunchKernelGGL(gemm_tn2_kernel, dim3(256), dim3(512), TN2_LDS, s, tg);
  return hipGetLastError();
}
namespace {

template <int EPI>
hipError_t launch_pipe2(const GemmArgs &g, hipStream_t s) {
  static bool attr_done = false;
  auto kern = gemm_pipe2_kernel<EPI>;
  if (!attr_done) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, PIPE2_LDS);
    if (e != hipSuccess) return e;
    attr_done = true;
  }
  if (g.M <= 0 || g.N <= 0 || g.K <= 0 || g.M % 256 || g.N % 256 || g.sum_splits || g.lda % 8) return hipErrorInvalidValue;
  const int splits = EPI == EPI_PARTIAL && g.splits > 1 ? g.splits : 1;
  if (g.K % (64 * splits) || (EPI != EPI_PARTIAL && g.splits > 1)) return hipErrorInvalidValue;
  if ((size_t)256 * g.lda * 2 + (size_t)g.K * 2 > 0x7fffffff || (EPI == EPI_GEGLU_FOLD && (g.C2 == nullptr) != (g.C3 == nullptr))) return hipErrorInvalidValue;
  GemmArgs ga = g;
  const int ntm = g.M / 256, ntn = g.N / 256;
  if (ga.col_groups == 0) ga.col_groups = fade_gemm_col_groups(g.M, g.K, g.N, (size_t)4 << 20);
  if ((ga.col_groups != 1 && ga.col_groups != 2 && ga.col_groups != 4) || ntn % ga.col_groups) ga.col_groups = 8;
  ga.splits = splits;
  const int rg = 8 / ga.col_groups, tiles = EPI == EPI_PARTIAL ? ntm * ntn * splits : (ntn % ga.col_groups == 0 ? (ntm + rg - 1) / rg * rg : ntm) * ntn;
  hipLaunchKernelGGL(kern, dim3(tiles), dim3(512), PIPE2_LDS, s, ga);
  return hipGetLastError();
}

template <int BM>
hipError_t launch_fnr(const GemmArgs &g, hipStream_t s) {
  static bool attr_done = false;
  if (!attr_done) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(gemm_fnr_kernel<BM>), hipFuncAttributeMaxDynamicSharedMemorySize, FnrRing<BM>::bytes);
    if (e != hipSuccess) return e;
    attr_done = true;
  }
  if (g.M <= 0 || g.N % 128 || (g.splits != 2 && g.splits != 4 && g.splits != 8) || g.K % (64 * g.splits) || g.lda % 8 || !g.stats || !g.fold_s || !g.fold_t) return hipErrorInvalidValue;
  GemmArgs ga = g;
  const int ntm = (g.M + BM - 1) / BM, ntn = g.N / 128;
  ga.col_groups = fade_gemm_col_groups(g.M, g.K, g.N);
  if ((ga.col_groups != 1 && ga.col_groups != 2 && ga.col_groups != 4) || ntn % ga.col_groups) ga.col_groups = 8;
  const int rg = 8 / ga.col_groups;
  hipLaunchKernelGGL(gemm_fnr_kernel<BM>, dim3((ntn % ga.col_groups == 0 ? (ntm + rg - 1) / rg * rg : ntm) * ntn), dim3(512), FnrRing<BM>::bytes, s, ga);
  return hipGetLastError();
}

// Tile shape by problem size. Small batches: 64 x 128 tiles, four stages, so that every compute unit gets a tile. From
// 512 tiles of 128 x 128 on: that tile with a two-stage ring (64 KiB of LDS), two workgroups per compute unit: one's
// epilogue (side inputs from HBM, stores) and pipeline fill run under the other's products, which measured faster than
// either a deeper ring or a 256 x 128 tile with one workgroup per unit (router product, M = 4096: 43 us against 54).
// Once every compute unit gets a 256 x 256 tile (M >= 8192 at N = 2048): that tile on eight wavefronts (pipe2_body): half the operand
// bytes per flop of 128 x 128 and two wavefronts per SIMD. On random operands at M = 16384, N = K = 2048 with the mix epilogue: 146 us
// against 230 for 128 x 128. With a contraction of 64 the two shapes tie.
template <int EPI>
hipError_t launch_pipe_auto(const GemmArgs &g, hipStream_t s) {
  const int tiles128 = ((g.M + 127) / 128) * (g.N / 128);
  const int tune = fade_gemm_tune();
  if constexpr (EPI != EPI_PARTIAL) {
    const int tiles256 = ((g.M + 255) / 256) * (g.N / 256);
    if (g.N % 256 == 0 && g.M % 256 == 0 && (tune == 20 || (tune == 0 && tiles256 >= 256 && g.K >= 256))) return launch_pipe2<EPI>(g, s);
  }
  if (tune == 11 || (tune == 0 && tiles128 >= 512)) return launch_pipe<128, 128, 2, EPI>(g, s);
  if (tune == 1 || (tune == 0 && tiles128 >= 256)) return launch_pipe<128, 128, 4, EPI>(g, s);
  return launch_pipe<64, 128, 4, EPI>(g, s);
}

template <int BN, int PRO, int EPI>
hipError_t launch_f32_bn(const GemmArgs &g, hipStream_t s) {
  constexpr int BM = 256 / (BN / 8);
  const int grid = ((g.M + BM - 1) / BM) * (g.N / BN);
  hipLaunchKernelGGL((gemm_f32_kernel<BN, PRO, EPI>), dim3(grid), dim3(256), 0, s, g);
  return hipGetLastError();
}
// wide == true: N is a multiple of 128 (required by the statistics and GeGLU layouts); otherwise N in {64, 32, 16}.
template <int PRO, int EPI, bool WIDE>
hipError_t launch_f32(const GemmArgs &g, hipStream_t s) {
  if (g.K % 32 || g.M <= 0) return hipErrorInvalidValue;
  if constexpr (WIDE) {
    if (g.N % 128) return hipErrorInvalidValue;
    return launch_f32_bn<128, PRO, EPI>(g, s);
  } else {
  if (g.N % 64 == 0) return launch_f32_bn<64, PRO, EPI>(g, s);
  if (g.N % 32 == 0) return launch_f32_bn<32, PRO, EPI>(g, s);
  if (g.N % 16 == 0) return launch_f32_bn<16, PRO, EPI>(g, s);
  return hipErrorInvalidValue;
  }
}

}  // namespace

// ---------------------------------------------------------------------------------------------------
// grouped launches (bf16 path)
// ---------------------------------------------------------------------------------------------------
namespace {
size_t group_kind_lds(int kind, int stages) {  // the larger of the operand ring and the fp32 tile parked for the epilogue
  size_t ring, tile;
  switch (kind) {
    case GK_STORE_64x128: case GK_TN_64x128: ring = 8192 + 16384; tile = 64 * 132 * 4; break;
    case GK_TN_128x128: case GK_STORE_128x128: case GK_PARTIAL_128x128: ring = 16384 + 16384; tile = 128 * 132 * 4; break;
    default: ring = 8192 + 8192; tile = 64 * 68 * 4; break;  // the 64 x 64 kinds
  }
  ring *= (size_t)stages;
  return ring > tile ? ring : tile;
}
}  // namespace

// Tile shape of a weight-gradient product dW[M][N] in a grouped launch.
static bool tn_shape(int M, int N, int &kind, int &bm, int &bn) {
  if (N % 128 == 0) {
    const bool big = M % 128 == 0 && (M / 128) * (N / 128) >= 256 && fade_gemm_tune() != 8;
    kind = big ? GK_TN_128x128 : GK_TN_64x128; bm = big ? 128 : 64; bn = 128;
    return true;
  }
  if (N % 64 == 0) { kind = GK_TN_64x64; bm = 64; bn = 64; return true; }
  return false;
}
// Shape of a weight gradient that can be tiles of gemm_tn2_kernel (whether a context uses it: plan_weight_gradients).
bool fade_gemm_tn2_ok(int M, int N, int K) { return M > 0 && N > 0 && M % 256 == 0 && N % 256 == 0 && K > 0 && K % 64 == 0 && (M / 256) * (N / 256) >= 16; }
int fade_gemm_tn_tiles(int M, int N) {
  int kind, bm, bn;
  if (M <= 0 || M % 64 || !tn_shape(M, N, kind, bm, bn)) return 0;
  return (M / bm) * (N / bn);
}

// Append one product to a group; the kernel body is chosen from the operation and the shape. op is one of GEMM_X_STORE
// (C = A W, W as fragments), GEMM_PARTIAL (split-K partials [splits][M][N], fp32) and GEMM_W_TN (dW from row-major operands).
hipError_t fade_gemm_group_add(GemmGroup &gg, int op, const GemmArgs &g) {
  if (gg.count >= 4 || g.M <= 0 || g.K <= 0 || g.K % 64 || g.lda % 8) return hipErrorInvalidValue;
  int kind, bm, bn, splits = 1;
  if (op == GEMM_X_STORE) {
    bm = 64;
    const int t128 = g.N % 128 == 0 ? ((g.M + 127) / 128) * (g.N / 128) : 0;
    // 128 x 128 tiles from 256 of them on, or from 128 when the contraction is long (then the bytes per flop matter more than
    // the number of workgroups: B = 1024, K = D_h = 2048: 43 us against 48 with 64 x 128; K = 64: 12.6 against 9.0)
    // a very long contraction with few output tiles whose blocks no split divides (du = dE [W_fg W_fv]^T at D_e = 8128) is a chain of
    // hundreds of K blocks per workgroup: small tiles, many workgroups (that phase in us with 64 x 64 | without, D_h = 512: 1500 rows
    // 213-224 | 228, 4096 313 | 310, but 2100 257 | 220 and 3000 281 | 233; D_h = 2048: 700 rows 258 | 275)
    if (g.K >= 4096 && g.N % 64 == 0 && t128 < 256) { kind = GK_STORE_64x64; bn = 64; }
    else if ((t128 >= 256 || (t128 >= 128 && g.K >= 1024)) && fade_gemm_tune() != 9) { kind = GK_STORE_128x128; bm = 128; bn = 128; }
    else if (g.N % 128 == 0 && ((g.M + 63) / 64) * (g.N / 128) >= 128) { kind = GK_STORE_64x128; bn = 128; }
    else if (g.N % 64 == 0) { kind = GK_STORE_64x64; bn = 64; }
    else return hipErrorInvalidValue;
  } else if (op == GEMM_PARTIAL) {
    if (g.N % 64 || g.sum_splits) return hipErrorInvalidValue;
    if (g.N % 128 == 0) { kind = GK_PARTIAL_128x128; bm = 128; bn = 128; }
    else { kind = GK_PARTIAL_64x64; bm = 64; bn = 64; }
    splits = g.splits > 1 ? g.splits : 1;
    if (g.K % (splits * 64)) return hipErrorInvalidValue;
  } else if (op == GEMM_W_TN) {
    if (g.a_rows <= 0 || g.a_rows > g.K || g.ldb % 8 || g.M % 64) return hipErrorInvalidValue;
    splits = g.splits > 1 ? g.splits : 1;  // ranges of the batch, each leaving its own slice of C (and C3)
    if (g.K % (splits * 64)) return hipErrorInvalidValue;
    if (!tn_shape(g.M, g.N, kind, bm, bn)) return hipErrorInvalidValue;
  } else {
    return hipErrorInvalidValue;
  }
  const int p = gg.count;
  if (p == 0) gg.first_block[0] = 0;
  gg.kind[p] = kind;
  gg.tiles[p] = ((g.M + bm - 1) / bm) * (g.N / bn);
  gg.splits[p] = splits;
  gg.first_block[p + 1] = gg.first_block[p] + gg.tiles[p] * splits;
  gg.g[p] = g;
  gg.count = p + 1;
  return hipSuccess;
}
hipError_t fade_gemm_group_launch(const GemmGroup &gg, hipStream_t s) {
  if (gg.count <= 0) return hipSuccess;
  static bool attr_done = false;
  if (!attr_done) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(gemm_group_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, 4 * (16384 + 16384));
    if (e == hipSuccess)
      e = hipFuncSetAttribute(reinterpret_cast<const void *>(gemm_group2_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, 128 * 132 * 4);
    if (e != hipSuccess) return e;
    attr_done = true;
  }
  // two workgroups per compute unit pay off once the group has about two workgroups for every unit (400 of them; B = 1024: the gate / router
  // groups 52 -> 44 us, the small refiner group 18 -> 24 us if forced; B = 4096: 177 -> 139 us)
  const int tune = fade_gemm_tune();
  const int stages = (tune == 14 || (tune != 13 && gg.first_block[gg.count] >= 400)) ? 2 : 4;
  size_t lds = 0;
  for (int p = 0; p < gg.count; ++p) lds = group_kind_lds(gg.kind[p], stages) > lds ? group_kind_lds(gg.kind[p], stages) : lds;
  if (stages == 2) hipLaunchKernelGGL(gemm_group2_kernel, dim3(gg.first_block[gg.count]), dim3(256), lds, s, gg);
  else hipLaunchKernelGGL(gemm_group_kernel, dim3(gg.first_block[gg.count]), dim3(256), lds, s, gg);
  return hipGetLastError();
}

// Tuning override for experiments (FADE_GEMM_TUNE: 0 automatic, 1 force 128x128x4 stages, 2 force 64x128, 11 force 128x128x2 with two
// workgroups per compute unit, 20 force 256x256 on eight wavefronts; grouped launches: 8 weight gradients without 128x128 tiles,
// 9 activation gradients without them, 13 force the four-stage kernel, 14 force the two-stage one).
int fade_gemm_tune() {
  static int v = -1;
  if (v < 0) { const char *e = getenv("FADE_GEMM_TUNE"); v = e ? atoi(e) : 0; }
  return v;
}

// One entry per (shape class, prologue, epilogue) the model step uses.
hipError_t fade_gemm(int op, bool bf16, const GemmArgs &g, hipStream_t s) {
  if (bf16) {
    switch (op) {
      case GEMM_CONV:     return launch_bf16<4, 1, 1, 1, PRO_CONV, EPI_CONV>(g, s);       // 128 x 32 tiles
      case GEMM_GLOBAL:   return launch_pipe_auto<EPI_GLOBAL>(g, s);
      case GEMM_ROUTER:   return launch_pipe_auto<EPI_MIX>(g, s);
      case GEMM_UP:       return launch_pipe_auto<EPI_STORE>(g, s);
      case GEMM_GATE:     return launch_pipe_auto<EPI_GATE>(g, s);
      case GEMM_FNR_OUT:  return launch_pipe_auto<EPI_STORE>(g, s);
      case GEMM_FNR_IN:   // Eq. 9 in one piece (no split-K): folded LayerNorm and GeGLU in the epilogue
        if (!g.stats || !g.fold_s || !g.fold_t) return hipErrorInvalidValue;
        if (g.splits > 1)  // as the sum of ranges of K, few tiles
          return ((g.M + 31) / 32) * (g.N / 128) <= 256 ? launch_fnr<32>(g, s) : launch_fnr<64>(g, s);
        return launch_pipe_auto<EPI_GEGLU_FOLD>(g, s);
      case GEMM_PARTIAL_TALL: return launch_pipe2<EPI_PARTIAL>(g, s);
      case GEMM_PARTIAL:  // split-K products whose LayerNorm / bias / non-linearity follow in the reducing kernel
        if (g.N % 128 == 0) return launch_pipe<128, 128, 4, EPI_PARTIAL>(g, s);
        return launch_pipe<64, 64, 4, EPI_PARTIAL>(g, s);
      case GEMM_X_STORE:  // backward dX = dY W^T: W^T is kept as a second set of fragments
        if (g.N % 128) return launch_pipe<64, 64, 4, EPI_STORE>(g, s);
        return launch_pipe_auto<EPI_STORE>(g, s);
      case GEMM_CONVT:    return launch_bf16<4, 1, 1, 1, PRO_CONVT, EPI_STORE>(g, s);
      case GEMM_HEAD:     // head on H = psi(LN(V)) + lam * H_coarse formed in the operand load (Eq. 10's tail never goes to memory):
        // 32 rows x all 256 columns per workgroup (two workgroups per unit), so every row is transformed once; split-K partials as GEMM_PARTIAL leaves them
        if (!g.stats || !g.A2 || !g.gamma || !g.beta || !g.lam || g.N != 256) return hipErrorInvalidValue;
        if (g.C2) return launch_bf16<1, 4, 1, 2, PRO_FINAL, EPI_PARTIAL, true>(g, s);  // H itself kept for the update
        return launch_bf16<1, 4, 1, 2, PRO_FINAL, EPI_PARTIAL>(g, s);
      default: return hipErrorInvalidValue;
    }
  }
  switch (op) {
    case GEMM_CONV:     return launch_f32<PRO_CONV, EPI_CONV, false>(g, s);
    case GEMM_GLOBAL:   return launch_f32<PRO_PLAIN, EPI_GLOBAL, true>(g, s);
    case GEMM_ROUTER:   return launch_f32<PRO_PLAIN, EPI_MIX, true>(g, s);
    case GEMM_DOWN:     return launch_f32<PRO_LN, EPI_STORE_F32, false>(g, s);
    case GEMM_UP:       return launch_f32<PRO_PLAIN, EPI_STORE, true>(g, s);
    case GEMM_GATE:     return launch_f32<PRO_PLAIN, EPI_GATE, true>(g, s);
    case GEMM_FNR_IN:   return launch_f32<PRO_LN, EPI_GEGLU, true>(g, s);
    case GEMM_FNR_OUT:  return launch_f32<PRO_PLAIN, EPI_STORE, true>(g, s);
    case GEMM_HEAD:     return launch_f32<PRO_FINAL, EPI_STORE_F32, true>(g, s);
    case GEMM_HEAD_PLAIN: return launch_f32<PRO_PLAIN, EPI_STORE_F32, true>(g, s);
    case GEMM_X_STORE:  // W passed transposed (wt = 1)
      if (g.N % 128 == 0) return launch_f32<PRO_PLAIN, EPI_STORE, true>(g, s);
      return launch_f32<PRO_PLAIN, EPI_STORE, false>(g, s);
    case GEMM_PARTIAL:  return launch_f32<PRO_PLAIN, EPI_PARTIAL, false>(g, s);  // one "split": the full sum
    case GEMM_W:
      if (g.N % 128 == 0) return launch_f32<PRO_PLAIN, EPI_GRAD, true>(g, s);
      return launch_f32<PRO_PLAIN, EPI_GRAD, false>(g, s);
    case GEMM_CONVT:    return launch_f32<PRO_CONVT, EPI_STORE, false>(g, s);
    default: return hipErrorInvalidValue;
  }
}

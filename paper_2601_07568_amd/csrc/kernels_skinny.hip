// bfloat16 matrix-core (MFMA) kernels for gfx950: the weight-streaming GEMMs of a denoise step.
//
// Skinny GEMM (at most 64 activation rows): the step is bound by streaming each weight once from
// HBM, so a workgroup owns a few 16-row tiles of the weight matrix for the whole K extent, its
// waves split K among themselves in interleaved stages of one to four 32-element steps, every load
// of a wave is a contiguous KiB of the packed weights or of the activations straight into registers
// (one or two stages ahead), and the partial tiles are summed through LDS in a fixed order.
// The epilogue of the summed tile is the fusion point: residual add, rotary embedding + KV-cache
// write, SiLU*up, or the softmax statistics of the LM head (the logits never reach memory).
//
// The q/k/v product takes up to 128 rows.  Above 64 it reads the weights as the caller gave them (row-major) and not the packed
// copy, as every other product of such a step does: who changes a weight in place packs again for steps of few rows only.
//
#include "mfma_common.h"

namespace dllm {

enum SkEpi { SK_F32 = 1, SK_QKV = 2, SK_SWIGLU = 3, SK_LMSTATS = 4, SK_RESID = 5 };

struct SkArgs {
  const bf16_t* X;          // activations [M, K], fragment order
  const int32_t* n_lm_rows; // optional device count: the kernel does nothing if it is zero
  int M, K;
  const bf16_t* W0;         // main weight / Wq / W_gate / lm_head   (packed fragment order; QKV of more than 64 rows: row-major)
  const bf16_t* W1;         // Wk / W_up
  const bf16_t* W2;         // Wv
  int N0, N1, N2;           // rows of W0, W1, W2
  float* out_f32;           // F32: [M, N0]
  bf16_t* out_bf16;         // QKV: q [M, N0] ; SWIGLU: h [M, N0]
  // QKV
  int dh, n_q_wg, n_k_wg;   // head_dim, workgroups covering q, k
  const float* rope_cos;
  const float* rope_sin;
  const int32_t* tok_seq;
  const int32_t* tok_pos;
  bf16_t* pool_k;
  bf16_t* pool_v;
  KVView pool;
  int32_t* status;
  // Row scale of the activations (QKV, SWIGLU, LMSTATS, F32): X holds x * gain rounded to bfloat16, the row's
  // normalisation factor rsqrt(mean(x^2) + eps) is applied to the summed tile in float.  ss_in[row * ss_stride + p],
  // p < n_ss, are partial sums of squares of row `row` (added up in a fixed order); nullptr: no scale.
  const float* ss_in;
  int n_ss, ss_stride;
  float inv_d, eps;
  const float* rscale;      // more than 64 rows: the factors themselves
  // RESID (residual projection x += X W0^T): a workgroup owns 16 columns for the whole of K, adds its tile to the
  // residual stream, writes x * gain_next in fragment order as the next GEMM's input and the rows' sums of squares
  // over its 16 columns to ss_out[row * ss_stride + workgroup].
  float* x;                 // residual stream [M, N0], in/out
  const bf16_t* gain_next;  // [N0]
  bf16_t* xg_out;           // fragment order, MT tiles
  float* ss_out;
  // LMSTATS
  float* part;              // [rows, n_parts, 4]
  int n_parts;
  int32_t mask_id;
};

constexpr int SK_KB = 128;  // k-elements per block: 4 matrix instructions deep
constexpr int SK_NW = 8;    // waves of a workgroup (they split K among themselves; the LM head's have four)

// One pipeline stage: JB matrix-instruction steps (JB*32 k-elements) of NT weight tiles and MT
// activation tiles.
template <int NT, int MT, int JB>
struct SkFrag {
  u32x4 a[NT][JB];
  u32x4 b[MT][JB];
};

// Both operands are in fragment order: step u (32 k-elements) of weight tile t is the KiB at
// wt[t] + u*64 units, of activation tile m the KiB at xf + (u*MT + m)*64 units (lane offset folded
// into the pointers), so every load instruction of the wave is contiguous.  RM: row-major weights, 64 bytes of each of
// the tile's 16 rows.
template <int NT, int MT, int JB, bool TAIL, bool RM>
__device__ inline void sk_load(SkFrag<NT, MT, JB>& f, const u32x4* const (&wt)[NT], const u32x4* xf, int stage, int g,
                               int K) {
  // (all weights of the stage in front of its activations: see SkCfg)
#pragma unroll
  for (int j = 0; j < JB; ++j) {
    const int u = stage * JB + j;
    // packed weights are zero beyond K; a row-major matrix may end there
    const bool ok = !TAIL || (u * 32 + g * 8 + 8 <= K);
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      if (!RM || ok) f.a[t][j] = wt[t][u * (RM ? 4 : 64)];
      else f.a[t][j] = u32x4{0, 0, 0, 0};
    }
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int j = 0; j < JB; ++j) {
    const int u = stage * JB + j;
    // (the activation buffer holds whatever was there beyond K, and 0 * NaN is NaN)
    const bool ok = !TAIL || (u * 32 + g * 8 + 8 <= K);
#pragma unroll
    for (int t = 0; t < MT; ++t) {
      if (ok) f.b[t][j] = xf[(u * MT + t) * 64];
      else f.b[t][j] = u32x4{0, 0, 0, 0};
    }
  }
}

template <int NT, int MT, int JB>
__device__ inline void sk_mma(const SkFrag<NT, MT, JB>& f, f32x4 (&acc)[NT][MT]) {
#pragma unroll
  for (int j = 0; j < JB; ++j)
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int m = 0; m < MT; ++m) acc[t][m] = mfma16(f.a[t][j], f.b[m][j], acc[t][m]);
}

// first weight row of tile t of workgroup wg, and which matrix it belongs to
template <int NT, int EPI>
__device__ inline void sk_tile_rows(const SkArgs& a, int wg, const bf16_t* (&wbase)[NT], int (&row0)[NT],
                                    int (&nrows)[NT]) {
  if constexpr (EPI == SK_QKV) {
    // Tiles 0 and 1 are the two halves of rotary pair-tile wg (rows h*dh + j0 .. and the same + dh/2) of Wq or Wk.
    // NT == 3: tile 2 is 16-row tile wg of Wv: pair tiles and value tiles are handed out together so that the grid is
    // max(pair tiles, value tiles) equal workgroups.  NT == 2: the workgroups behind the pair tiles take two tiles of Wv.
    const int half = a.dh >> 1, per_head = half / 16;
    const int n_pairs = a.n_q_wg + a.n_k_wg;
    const int pw = wg < n_pairs ? wg : n_pairs - 1;            // clamped: the result is dropped
    const bool isq = pw < a.n_q_wg;
    const int lw = isq ? pw : pw - a.n_q_wg;
    const int h = lw / per_head, j0 = (lw - h * per_head) * 16;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      wbase[t] = isq ? a.W0 : a.W1;
      nrows[t] = isq ? a.N0 : a.N1;
      row0[t] = h * a.dh + j0 + t * half;
    }
    if constexpr (NT == 3) {
      wbase[NT - 1] = a.W2;
      nrows[NT - 1] = a.N2;
      row0[NT - 1] = wg * 16;                                  // beyond N2: clamped by the caller, dropped below
    } else if (wg >= n_pairs) {
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        wbase[t] = a.W2;
        nrows[t] = a.N2;
        row0[t] = ((wg - n_pairs) * 2 + t) * 16;
      }
    }
  } else if constexpr (EPI == SK_SWIGLU) {
    // NT = 2*P: tiles 0..P-1 are P consecutive 16-row tiles of the gate matrix, tiles P..2P-1 the same rows of up
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      wbase[t] = (t < NT / 2) ? a.W0 : a.W1;
      nrows[t] = a.N0;
      row0[t] = (wg * (NT / 2) + (t % (NT / 2))) * 16;
    }
  } else {
#pragma unroll
    for (int t = 0; t < NT; ++t) { wbase[t] = a.W0; nrows[t] = a.N0; row0[t] = wg * 16 * NT + t * 16; }
  }
}

// JB: matrix-instruction steps of a pipeline stage, D: stages that registers hold.  TPC: weight tiles whose partial sums go through LDS together.
template <int NT, int MT, int NW, int EPI, int JB, int TPC, int D, int WPS>
__global__ __launch_bounds__(NW * 64, WPS) void k_skinny(const SkArgs a) {
  constexpr bool SCALED = (EPI != SK_RESID);
  constexpr bool RM = MT > 4;                           // the weights as the caller gave them, not the packed copy
  constexpr int RPW = (MT * 16 + NW - 1) / NW;          // rows per wave when the row scales are summed
  // partial tiles go through LDS in chunks of TPC weight tiles and MC activation tiles
  constexpr int NCH = NT / TPC, MCH = NW * TPC * MT <= 144 ? 1 : 2, MC = (MT + MCH - 1) / MCH;
  static_assert(NT % TPC == 0 && (EPI != SK_LMSTATS || (TPC == 4 && MCH == 1)), "64 columns per partial of the LM head");
  constexpr int NBUF = NCH * MCH > 1 && NW * TPC * MC <= 64 ? 2 : 1;   // (of 64 KiB at most)
  __shared__ float red_buf[NBUF][NW][TPC][MC][4][64];
  __shared__ float lmst[EPI == SK_LMSTATS ? MT : 1][4][16][4];
  __shared__ float rs[MT * 16 < 64 ? 64 : MT * 16];     // row scale of the activations
  __shared__ float ssq[EPI == SK_RESID ? MT : 1][4][64];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int c = lane & 15, g = lane >> 4;
  const int wg = blockIdx.x;
  const int K = a.K;
  const int M = a.M;
  if (a.n_lm_rows && *a.n_lm_rows <= 0) return;
  if (M <= 0) return;

  constexpr int RIT = EPI == SK_RESID ? (MT * 256 + NW * 64 - 1) / (NW * 64) : 1;
  float xres[RIT], gres[RIT];                           // RESID: the thread's elements of x and of the next gain

  const bf16_t* wbase[NT];
  int row0[NT], nrows[NT];
  sk_tile_rows<NT, EPI>(a, wg, wbase, row0, nrows);
  // packed weights: the 16-row tile rt of a matrix with kpb 128-element blocks starts at unit
  // rt * kpb * 256; inside, (block, j, lane) is unit (block*4 + j)*64 + lane: one contiguous stream
  const int kpb = (K + SK_KB - 1) / SK_KB;
  const u32x4* wt[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    if constexpr (RM) {
      const int row = row0[t] + c < nrows[t] ? row0[t] + c : nrows[t] - 1;
      wt[t] = (const u32x4*)(wbase[t] + (int64_t)row * K + g * 8);
      continue;
    }
    int rt = row0[t] >> 4;
    const int rt_max = (nrows[t] + 15) / 16 - 1;
    rt = rt < rt_max ? rt : rt_max;
    wt[t] = (const u32x4*)wbase[t] + (int64_t)rt * kpb * 256 + lane;
  }
  const u32x4* xf = (const u32x4*)a.X + lane;   // rows >= M of the last tile hold stale data: their columns are dropped
  if constexpr (EPI == SK_RESID) {
    // the elements this thread will update
#pragma unroll
    for (int k = 0; k < RIT; ++k) {
      const int item = tid + k * NW * 64, m = item >> 8, iq = (item >> 6) & 3;
      const int tok = m * 16 + c, n = row0[0] + 4 * g + iq;
      const bool ok = m < MT && tok < M && n < a.N0;
      xres[k] = a.x[ok ? (int64_t)tok * a.N0 + n : 0];
      gres[k] = bf16_to_f32(a.gain_next[ok ? n : 0]);
    }
  }
  // QKV: what a thread's epilogue items need besides the sums - the rows' positions, their rotary factors - is requested
  // before the weights, the pages of their cache slots (which depend on the positions) behind the first weights: a wave
  // that waited for the positions first would start its stream a round trip late.  Addresses are clamped, not branched.
  constexpr int IPT = EPI == SK_QKV ? (MC * 256 + NW * 64 - 1) / (NW * 64) : 1;   // items of a thread and chunk
  float pcs[MCH][IPT], psn[MCH][IPT];
  int ppos[MCH][IPT], pseq[MCH][IPT], ppage[MCH][IPT];
  if constexpr (EPI == SK_QKV) {
#pragma unroll
    for (int mc = 0; mc < MCH; ++mc)
#pragma unroll
      for (int k = 0; k < IPT; ++k) {
        const int item = tid + k * NW * 64, iq = (item >> 6) & 3;
        int tok = (mc * MC + (item >> 8)) * 16 + c;
        tok = tok < M ? tok : M - 1;
        const int hj = row0[0] + 4 * g + iq, half = a.dh >> 1;
        int j = hj - (hj / a.dh) * a.dh;
        j = j < half ? j : 0;                                   // (a value row's is not used)
        ppos[mc][k] = a.tok_pos[tok];
        pseq[mc][k] = a.tok_seq[tok];
        pcs[mc][k] = a.rope_cos[(int64_t)tok * half + j];
        psn[mc][k] = a.rope_sin[(int64_t)tok * half + j];
      }
  }
  auto fetch_pages = [&]() {
    if constexpr (EPI == SK_QKV) {
#pragma unroll
      for (int mc = 0; mc < MCH; ++mc)
#pragma unroll
        for (int k = 0; k < IPT; ++k) {
          const int pos = ppos[mc][k], pi = pos >= 0 ? pos / a.pool.page_tokens : a.pool.max_pages;
          const int page = a.pool.table[(int64_t)pseq[mc][k] * a.pool.max_pages + (pi < a.pool.max_pages ? pi : a.pool.max_pages - 1)];
          ppage[mc][k] = pi < a.pool.max_pages ? page : -1;
        }
    }
  };
  // kv_locate from a position and its page
  auto locate = [&](int pos, int page, int h, int64_t& k_off, int64_t& v_off, int& v_stride) -> bool {
    const KVView& kv = a.pool;
    if (pos < 0 || page < 0 || page >= kv.n_pages) return false;
    const int slot = pos - (pos / kv.page_tokens) * kv.page_tokens;
    const int64_t ph = (int64_t)page * kv.n_kv_heads + h;
    k_off = (ph * kv.page_tokens + slot) * kv.head_dim;
    v_off = ph * kv.head_dim * kv.page_tokens + slot;
    v_stride = kv.page_tokens;
    return true;
  };

  f32x4 acc[NT][MT];
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int m = 0; m < MT; ++m) acc[t][m] = f32x4{0.f, 0.f, 0.f, 0.f};

  // Row scales: the wave adds up the partial sums of squares of rows w, w + NW, .. (one 16-byte load per lane covers
  // 256 partials of a row; lanes add their four, the wave adds its lanes in a fixed tree) and lane 0 keeps the
  // row's factor.  Called once the first weight stages are on their way: the partials come from the L2, the
  // weights from memory, so the wave waits no longer for them than it would for the weights alone.
  auto row_scales = [&]() {
    if constexpr (SCALED && MT > 4) {
      if (tid < MT * 16) rs[tid] = a.rscale[tid < M ? tid : M - 1];
    } else if constexpr (SCALED) {
      if (a.ss_in) {
        float4 ssv[RPW];
        const int idc = 4 * lane < a.ss_stride - 4 ? 4 * lane : a.ss_stride - 4;
#pragma unroll
        for (int q = 0; q < RPW; ++q) ssv[q] = *(const float4*)(a.ss_in + (int64_t)(w + q * NW) * a.ss_stride + idc);
#pragma unroll
        for (int q = 0; q < RPW; ++q) {
          const int row = w + q * NW;
          const int i0 = 4 * lane;
          float sq = (i0 < a.n_ss ? ssv[q].x : 0.f) + (i0 + 1 < a.n_ss ? ssv[q].y : 0.f) +
                     (i0 + 2 < a.n_ss ? ssv[q].z : 0.f) + (i0 + 3 < a.n_ss ? ssv[q].w : 0.f);
          for (int c0 = 256; c0 < a.n_ss; c0 += 256) {            // very wide models only
            const int i1 = c0 + 4 * lane;
            const int ic = i1 < a.ss_stride - 4 ? i1 : a.ss_stride - 4;
            const float4 v = *(const float4*)(a.ss_in + (int64_t)row * a.ss_stride + ic);
            sq += (i1 < a.n_ss ? v.x : 0.f) + (i1 + 1 < a.n_ss ? v.y : 0.f) + (i1 + 2 < a.n_ss ? v.z : 0.f) +
                  (i1 + 3 < a.n_ss ? v.w : 0.f);
          }
#pragma unroll
          for (int o = 1; o < 64; o <<= 1) sq += __shfl_xor(sq, o, 64);
          if (lane == 0 && row < 64) rs[row] = 1.0f / sqrtf(sq * a.inv_d + a.eps);
        }
      } else if (tid < 64) rs[tid] = 1.0f;
    }
  };

  // Software pipeline over this wave's stages (w, w+NW, ...): D - 1 stages are in flight while another
  // is multiplied.  No load sits inside a branch of the steady-state loop (a branch around a load
  // makes the compiler wait for every outstanding load at the join); the drain is straight-line code.
  constexpr int SKB = JB * 32;                        // k-elements per stage
  const int n_full = K / SKB;                         // stages that need no tail guard
  const int ws = __builtin_amdgcn_readfirstlane(w);   // wave index as a scalar
  const int n_w = n_full > ws ? (n_full - ws + NW - 1) / NW : 0;
#define SK_LD(F, I) sk_load<NT, MT, JB, false, RM>(F, wt, xf, ws + (I) * NW, g, K)
#define SK_MM(F) sk_mma<NT, MT, JB>(F, acc)
  if (n_w == 0) {
    fetch_pages();
    row_scales();
  } else {
    SkFrag<NT, MT, JB> f[D];
#pragma unroll
    for (int j = 0; j < D - 1; ++j) SK_LD(f[j], j < n_w ? j : n_w - 1);
    fetch_pages();
    row_scales();
    if (n_w < D - 1) {
#pragma unroll
      for (int j = 0; j < D - 2; ++j)
        if (j < n_w) SK_MM(f[j]);
    } else {
      int i = 0;
      while (i + 2 * D - 2 < n_w) {          // stages i .. i + 2D - 2 exist, the first D - 1 of them are in flight
#pragma unroll
        for (int j = 0; j < D; ++j) {
          SK_LD(f[(j + D - 1) % D], i + j + D - 1);
          SK_MM(f[j]);
        }
        i += D;
      }
      const int left = n_w - i;              // D - 1 .. 2D - 2
#pragma unroll
      for (int r = D - 1; r <= 2 * D - 2; ++r)
        if (left == r) {
#pragma unroll
          for (int j = 0; j < 2 * D - 2; ++j) {
            if (j + D - 1 < r) SK_LD(f[(j + D - 1) % D], i + j + D - 1);
            if (j < r) SK_MM(f[j % D]);
          }
        }
    }
  }
#undef SK_LD
#undef SK_MM
  if (n_full * SKB < K && ws == n_full % NW) {   // ragged last stage
    SkFrag<NT, MT, JB> ft;
    sk_load<NT, MT, JB, true, RM>(ft, wt, xf, n_full, g, K);
    sk_mma<NT, MT, JB>(ft, acc);
  }

  // Sum the waves' partial tiles in wave order, a chunk at a time (SWIGLU: gate tiles and the up tiles of the same rows).
  // Two buffers in turn: a chunk's barrier also says that every thread is done with the chunk before the last.
#pragma unroll
  for (int chunk = 0; chunk < NCH * MCH; ++chunk) {
  const int ch = chunk / MCH, mc = chunk % MCH;
  auto& red = red_buf[chunk & (NBUF - 1)];
  if (NBUF == 1 && chunk > 0) __syncthreads();
  auto tile_of = [&](int u) { return EPI == SK_SWIGLU ? (u < TPC / 2 ? ch * (TPC / 2) + u : NT / 2 + ch * (TPC / 2) + u - TPC / 2) : ch * TPC + u; };
#pragma unroll
  for (int u = 0; u < TPC; ++u)
#pragma unroll
    for (int m = 0; m < MC; ++m)
      if (mc * MC + m < MT) {
#pragma unroll
        for (int i = 0; i < 4; ++i) red[w][u][m][i][lane] = acc[tile_of(u)][mc * MC + m][i];
      }
  __syncthreads();
  const int n_items = (MT - mc * MC < MC ? MT - mc * MC : MC) * 256;

  if constexpr (EPI == SK_RESID) {
    // ---- residual projection: x += tile; next GEMM's input x * gain; sums of squares of the 16 columns per row
    static_assert(EPI != SK_RESID || NT == 1, "a residual projection's workgroup owns one 16-row weight tile");
#pragma unroll
    for (int k = 0; k < RIT; ++k) {
      const int item = tid + k * NW * 64;
      if (item >= MT * 256) break;
      const int m = item >> 8, iq = (item >> 6) & 3, ln = item & 63;
      const int tok = m * 16 + (ln & 15);
      const int n = row0[0] + 4 * (ln >> 4) + iq;
      float sum = 0.f;
#pragma unroll
      for (int ww = 0; ww < NW; ++ww) sum += red[ww][0][m][iq][ln];
      float sq = 0.f;
      if (tok < M && n < a.N0) {
        const float v = xres[k] + sum, gn = gres[k];
        a.x[(int64_t)tok * a.N0 + n] = v;
        a.xg_out[frag_offset(tok, n, MT)] = f32_to_bf16(v * gn);
        sq = v * v;
      }
      ssq[m][iq][ln] = sq;
    }
    __syncthreads();
    if (tid < MT * 16) {          // the 16 contributions of a row (4 values of iq x 4 lane groups) in a fixed order
      const int m = tid >> 4, cc = tid & 15;
      float sq = 0.f;
#pragma unroll
      for (int iq = 0; iq < 4; ++iq)
#pragma unroll
        for (int lg = 0; lg < 4; ++lg) sq += ssq[m][iq][lg * 16 + cc];
      a.ss_out[(int64_t)tid * a.ss_stride + wg] = sq;
    }
    return;
  }

#pragma unroll
  for (int k = 0; k < (MC * 256 + NW * 64 - 1) / (NW * 64); ++k) {
    const int item = tid + k * NW * 64;
    if (item >= n_items) break;
    const int m = item >> 8, i = (item >> 6) & 3, ln = item & 63;
    const int tok = (mc * MC + m) * 16 + (ln & 15);
    const int fr = 4 * (ln >> 4) + i;          // row inside the 16-row tile
    float val[TPC];
    const float rsc = SCALED ? rs[tok] : 1.0f;
#pragma unroll
    for (int t = 0; t < TPC; ++t) {
      float s = 0.f;
#pragma unroll
      for (int ww = 0; ww < NW; ++ww) s += red[ww][t][m][i][ln];
      val[t] = s * rsc;
    }
    const bool tok_ok = tok < M;
    if constexpr (EPI == SK_F32) {
#pragma unroll
      for (int t = 0; t < TPC; ++t) {
        const int n = row0[tile_of(t)] + fr;
        if (tok_ok && n < a.N0) a.out_f32[(int64_t)tok * a.N0 + n] = val[t];
      }
    } else if constexpr (EPI == SK_SWIGLU) {
#pragma unroll
      for (int t = 0; t < TPC / 2; ++t) {
        const int n = row0[tile_of(t)] + fr;
        if (tok_ok && n < a.N0) {
          const float gt = val[t];
          a.out_bf16[frag_offset(tok, n, MT)] = f32_to_bf16(gt / (1.0f + expf(-gt)) * val[t + TPC / 2]);
        }
      }
    } else if constexpr (EPI == SK_QKV) {
      if (tok_ok) {
        if (wg < a.n_q_wg + a.n_k_wg) {
          const bool isq = wg < a.n_q_wg;
          const int half = a.dh >> 1;
          const int hj = row0[0] + fr;                 // h*dh + j, j < half
          const int h = hj / a.dh, j = hj - h * a.dh;
          const float cs = pcs[mc][k], sn = psn[mc][k];
          const float v0 = val[0], v1 = val[1];
          const bf16_t r0 = f32_to_bf16(v0 * cs - v1 * sn), r1 = f32_to_bf16(v1 * cs + v0 * sn);
          if (isq) {
            a.out_bf16[(int64_t)tok * a.N0 + hj] = r0;
            a.out_bf16[(int64_t)tok * a.N0 + hj + half] = r1;
          } else {
            int64_t ko, vo;
            int vs;
            if (ppos[mc][k] < 0) {
              // a padding row: nothing of it is cached
            } else if (locate(ppos[mc][k], ppage[mc][k], h, ko, vo, vs)) {
              a.pool_k[ko + j] = r0;
              a.pool_k[ko + j + half] = r1;
            } else atomicOr(a.status, DLLM_STATUS_BAD_PAGE);
          }
        }
        if (NT == 3 || wg >= a.n_q_wg + a.n_k_wg) {
#pragma unroll
          for (int t = NT == 3 ? 2 : 0; t < NT; ++t) {
            const int n = row0[t] + fr;                // value row
            if (n >= a.N2) continue;
            const int h = n / a.dh, cn = n - h * a.dh;
            int64_t ko, vo;
            int vs;
            if (locate(ppos[mc][k], ppage[mc][k], h, ko, vo, vs)) a.pool_v[vo + (int64_t)cn * vs] = f32_to_bf16(val[t]);
          }
        }
      }
    } else if constexpr (EPI == SK_LMSTATS) {
      RowStat st;
      st.init();
#pragma unroll
      for (int t = 0; t < TPC; ++t) {
        const int n = row0[tile_of(t)] + fr;
        if (n < a.N0 && n != a.mask_id) st.merge(val[t], n, 1.0f, val[t]);
      }
      // same token: lanes ln, ln^16, ln^32, ln^48 of this wave, then the four values of i
#pragma unroll
      for (int o = 16; o < 64; o <<= 1) {
        const float m2 = __shfl_xor(st.m, o, 64), s2 = __shfl_xor(st.s, o, 64), t2 = __shfl_xor(st.t, o, 64);
        const int i2 = __shfl_xor(st.idx, o, 64);
        st.merge(m2, i2, s2, t2);
      }
      if ((ln >> 4) == 0) {
        float* p = &lmst[m][i][ln & 15][0];
        p[0] = st.m; p[1] = __int_as_float(st.idx); p[2] = st.s; p[3] = st.t;
      }
    }
  }
  if (EPI == SK_LMSTATS) {
    __syncthreads();
    if (tid < MT * 16) {
      const int m = tid >> 4, cc = tid & 15, tok = m * 16 + cc;
      if (tok < M && wg * NCH + ch < a.n_parts) {
        RowStat st;
        st.init();
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float* p = &lmst[m][i][cc][0];
          st.merge(p[0], __float_as_int(p[1]), p[2], p[3]);
        }
        float* o = a.part + ((int64_t)tok * a.n_parts + wg * NCH + ch) * 4;
        o[0] = st.m; o[1] = __int_as_float(st.idx); o[2] = st.s; o[3] = st.t;
      }
    }
  }
  }   // chunks
}

// Pipeline of a form.  What bounds a workgroup beside the memory itself is how much its CU can have outstanding: about 32 KB,
// whatever the registers could hold, and loads come back in the order in which they were issued.  So a CU reads 58 GB/s from
// memory, 149 from the L2, and 58 of both mixed: an activation load (from the L2) behind a weight load (from memory) takes as long.
// Stages are therefore as long as the registers allow with two of them in flight, and ask for all their weights first: then
// the activations behind them come at the L2's pace.  (Short stages, weights and activations in turn / these, us: residual 32 rows of
// 4096 x 12288 25.6 / 24.8, 64 rows 34.9 / 33.7, 16 rows of 2048 x 2048 8.6 / 7.0; q/k/v 12288 x 4096 64 rows 28.3 / 26.8, 96 rows
// 34.6 / 32.1; 4608 x 3584 32 rows 13.3 / 12.6; LM head 126464 x 4096 32 rows 191 / 186, 48 rows 203 / 194.  Three-tile q/k/v of
// at most 32 rows had stages of two steps before; the order alone, in turn / weights first, whole layers of 4096 channels, 32 heads
// and 12288 features at 8, 16, 24, 32, 48, 64 rows: 100.7 / 101.2, 102.0 / 102.7, 111.5 / 111.3, 112.9 / 112.7, 129.0 / 127.5, 144.6 /
// 141.2; of 3072 and 5120 channels the second is the better one at every count.)  More stages than two
// in flight bring nothing; registers beyond a wave's share cost up to twice the time.  Gate/up of 16 rows in stages of two steps / one:
// 8192 x 2048 14.1 / 12.7, 5504 x 2048 11.0 / 9.6, 12288 x 4096 37.2 / 37.3; six tiles x 32 rows two / one 37.3 / 36.4.
// SHORT (q/k/v of at most 32 rows in two tiles a workgroup): stages of one step, four of them in flight.  The long stages give the
// eight waves 1024 of K at a time, which where that leaves a rest is a round of half-idle waves, and beside a memory that nearly all CUs
// ask shows (launch_sk_qkv).
template <int NT, int MT, int NW, int EPI, bool SHORT = false>
struct SkCfg {
  static constexpr bool HEAD = EPI == SK_LMSTATS || EPI == SK_F32;
  static constexpr int JB = SHORT ? 1
                            : EPI == SK_RESID ? 4
                            : EPI == SK_QKV ? (NT == 2 ? (MT <= 4 ? 4 : 2) : MT == 8 ? 1 : 2)
                            : HEAD          ? (MT == 1 ? 4 : 2)
                                            : MT >= 3 || EPI == SK_SWIGLU ? 1 : 2;
  static constexpr int D = SHORT ? 5 : EPI == SK_RESID ? (MT <= 2 ? 3 : 2) : EPI == SK_QKV ? (NT == 3 && MT <= 2 ? 3 : 2) : HEAD ? 2 : MT == 4 ? 2 : 3;
  static constexpr int TPC = EPI == SK_SWIGLU ? 2 : NT;
  // waves per SIMD that the registers are to allow: two 8-wave workgroups per CU for the narrow gate/up form, so that one
  // workgroup's prologue and reduction overlap the other's streaming
  static constexpr int WPS = EPI == SK_SWIGLU && NT == 2 ? 4 : (NW == 4 && MT <= 2) ? 1 : 2;
};
template <int NT, int MT, int NW, int EPI, bool SHORT = false>
static hipError_t sk_go(hipStream_t s, const SkArgs& a, int grid) {
  using C = SkCfg<NT, MT, NW, EPI, SHORT>;
  k_skinny<NT, MT, NW, EPI, C::JB, C::TPC, C::D, C::WPS><<<grid, NW * 64, 0, s>>>(a);
  return hipGetLastError();
}

template <int NT, int NW, int EPI>
static hipError_t sk_launch_mt(hipStream_t s, const SkArgs& a, int grid) {
  const int mt = (a.M + 15) / 16;
  switch (mt) {
    case 1: return sk_go<NT, 1, NW, EPI>(s, a, grid);
    case 2: return sk_go<NT, 2, NW, EPI>(s, a, grid);
    case 3: return sk_go<NT, 3, NW, EPI>(s, a, grid);
    case 4: return sk_go<NT, 4, NW, EPI>(s, a, grid);
  }
  if constexpr (EPI == SK_QKV) {
    switch (mt) {
      case 5: return sk_go<NT, 5, NW, EPI>(s, a, grid);
      case 6: return sk_go<NT, 6, NW, EPI>(s, a, grid);
      case 7: return sk_go<NT, 7, NW, EPI>(s, a, grid);
      case 8: return sk_go<NT, 8, NW, EPI>(s, a, grid);
    }
  }
  return hipErrorInvalidValue;
}

// ---- weight packing ---------------------------------------------------------------------------
// [N, K] row-major -> fragment order, rows padded to 16 and K to 128 with zeros.  Unit (16 bytes)
// index ((rt * kpb + kb) * 4 + j) * 64 + g*16 + c holds row rt*16 + c, k = kb*128 + j*32 + g*8 .. +7.
__global__ void k_pack_weight(const bf16_t* __restrict__ W, u32x4* __restrict__ P, int N, int K, int64_t n_units) {
  const int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (u >= n_units) return;
  const int kpb = (K + SK_KB - 1) / SK_KB;
  const int lane = (int)(u & 63), j = (int)((u >> 6) & 3);
  const int64_t t = u >> 8;
  const int kb = (int)(t % kpb), rt = (int)(t / kpb);
  const int r = rt * 16 + (lane & 15), k = kb * SK_KB + j * 32 + (lane >> 4) * 8;
  u32x4 v = u32x4{0, 0, 0, 0};
  if (r < N && k + 8 <= K) v = *(const u32x4*)(W + (int64_t)r * K + k);
  P[u] = v;
}

size_t packed_weight_bytes(int N, int K) {
  return (size_t)((N + 15) / 16) * ((K + SK_KB - 1) / SK_KB) * 256 * 16;
}

hipError_t launch_pack_weight(hipStream_t s, const void* W, void* P, int N, int K) {
  const int64_t n_units = (int64_t)(packed_weight_bytes(N, K) / 16);
  k_pack_weight<<<(unsigned)((n_units + 255) / 256), 256, 0, s>>>((const bf16_t*)W, (u32x4*)P, N, K, n_units);
  return hipGetLastError();
}


bool mfma_supported(const dllm_ctx* c) {
  const dllm_config& f = c->cfg;
  return f.dtype == DLLM_BF16 && c->kernel_mode == 0 && c->packed != nullptr && f.d_model <= 16384 && f.d_model % 8 == 0 && f.d_ff % 8 == 0 &&
         (f.head_dim == 64 || f.head_dim == 128);
}

static SkArgs sk_base(const void* X, int M, int K) {
  SkArgs a;
  memset(&a, 0, sizeof(a));
  a.X = (const bf16_t*)X;
  a.M = M;
  a.K = K;
  return a;
}

// Residual projection x += A * W^T: one workgroup of 8 waves per 16-column tile, the waves split K.  Its epilogue
// prepares the next GEMM's input (x * gain_next in fragment order, sums of squares per row): no RMSNorm launch.
// A workgroup re-reads all of A from the L2 (twice its weight bytes); that costs less than exchanging partial
// products between workgroups would (two memory round trips at the end of every launch).
hipError_t launch_sk_resid(dllm_ctx* c, hipStream_t s, const void* A, const void* W, int M, int N, int K,
                           const void* gain_next) {
  SkArgs a = sk_base(A, M, K);
  a.W0 = (const bf16_t*)W;   // packed
  a.N0 = N;
  a.x = WSM(c, x, float);
  a.gain_next = (const bf16_t*)gain_next;
  a.xg_out = WSM(c, xn, bf16_t);
  a.ss_out = WSM(c, ss, float);
  a.ss_stride = ss_row_stride(c);
  return sk_launch_mt<1, SK_NW, SK_RESID>(s, a, (N + 15) / 16);
}

// the GEMM input comes with n_ss partial sums of squares per row
static void sk_row_scale(dllm_ctx* c, SkArgs& a, int n_ss) {
  a.ss_in = WSM(c, ss, float);
  a.n_ss = n_ss;
  a.ss_stride = ss_row_stride(c);
  a.inv_d = 1.0f / (float)c->cfg.d_model;
  a.eps = c->cfg.rms_eps;
}

// Everything a denoise step of at most 64 rows needs before its first GEMM, in one launch of one workgroup per row:
// step_row_map (lengths, token map, rotary table) and the row's embedding: x[t] = E[token[t]] in float, x * gain of the first
// norm in fragment order as the first GEMM's input (bfloat16 models; the float kernels apply the gain themselves), the row's
// sum of squares as its single partial.
template <typename T>
__global__ __launch_bounds__(256) void k_sk_prologue(const StepMap m, int n_rows, int d, int vocab, int mt, const int32_t* tokens,
                                                     const T* emb, const bf16_t* gain, float* x, bf16_t* xg, float* ss,
                                                     int ss_stride, int32_t mask_id, int cap, int32_t* rows, int32_t* cand, float* conf,
                                                     float* entropy) {
  __shared__ float red[4];
  __shared__ int s_bad;
  const int t = blockIdx.x, Q = m.Q;
  int32_t* const status = m.status;
  const int nl = step_live(m);
  step_row_map(m, t, nl, &s_bad);
  if (t == 0) {
    // the rows of the LM head (k_mask_rows for a step of at most 64 rows: one wave, row r in lane r): the masked rows
    // that are not padding, in ascending order; every other row reports its own token with confidence 1
    if (cand && threadIdx.x < 64) {
      const int r = threadIdx.x;
      bool flag = false;
      if (r < n_rows) {
        const int b2 = r / Q, j2 = r - b2 * Q;
        const bool hq = m.n_live != nullptr || m.q_valid != nullptr;
        const int qv2 = step_valid(m, b2, nl);
        const int tk = tokens[r];
        flag = !(hq && j2 >= qv2) && tk == mask_id;
        if (!flag) {
          cand[r] = tk;
          conf[r] = 1.0f;
          if (entropy) entropy[r] = 0.f;
        }
      }
      const unsigned long long bal = __ballot(flag);
      const int pre = __popcll(bal & ((1ull << r) - 1ull));
      if (flag && pre < cap) rows[pre] = r;
      if (r == 0) {
        int n = __popcll(bal);
        if (n > cap) { atomicOr(status, DLLM_STATUS_ROWS_CAP); n = cap; }
        status[1] = n;
      }
    }
  }
  // embedding: x[t] = E[token[t]] (float), x * gain in fragment order, the row's sum of squares
  int tok = tokens[t];
  if (tok < 0 || tok >= vocab) {
    if (threadIdx.x == 0) atomicOr(status, DLLM_STATUS_BAD_TOKEN);
    tok = 0;
  }
  const T* row = emb + (int64_t)tok * d;
  float sq = 0.f;
  if constexpr (sizeof(T) == 4) {
    for (int u = threadIdx.x; u < (d >> 2); u += 256) {
      const float4 v = *(const float4*)(row + 4 * u);
      *(float4*)(x + (int64_t)t * d + 4 * u) = v;
      sq = fmaf(v.x, v.x, sq); sq = fmaf(v.y, v.y, sq); sq = fmaf(v.z, v.z, sq); sq = fmaf(v.w, v.w, sq);
    }
  } else
  for (int u = threadIdx.x; u < (d >> 3); u += 256) {          // 16-byte units: 8 channels
    const uint4 ev = *(const uint4*)(row + 8 * u), gv = *(const uint4*)(gain + 8 * u);
    const uint32_t ew[4] = {ev.x, ev.y, ev.z, ev.w}, gw[4] = {gv.x, gv.y, gv.z, gv.w};
    float xv[8];
    uint32_t o[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      xv[2 * e] = __uint_as_float(ew[e] << 16);
      xv[2 * e + 1] = __uint_as_float(ew[e] & 0xffff0000u);
      o[e] = pack_bf16x2(xv[2 * e] * __uint_as_float(gw[e] << 16), xv[2 * e + 1] * __uint_as_float(gw[e] & 0xffff0000u));
      sq = fmaf(xv[2 * e], xv[2 * e], sq);
      sq = fmaf(xv[2 * e + 1], xv[2 * e + 1], sq);
    }
    float4* xr = (float4*)(x + (int64_t)t * d + 8 * u);
    xr[0] = make_float4(xv[0], xv[1], xv[2], xv[3]);
    xr[1] = make_float4(xv[4], xv[5], xv[6], xv[7]);
    *(uint4*)(xg + frag_offset(t, 8 * u, mt)) = make_uint4(o[0], o[1], o[2], o[3]);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) sq += __shfl_xor(sq, o, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = sq;
  __syncthreads();
  if (threadIdx.x == 0) ss[(int64_t)t * ss_stride] = (red[0] + red[1]) + (red[2] + red[3]);
}

hipError_t launch_sk_prologue(dllm_ctx* c, hipStream_t s, const StepGeom& g, const void* gain, int32_t* cand,
                              float* conf, float* entropy) {
  const dllm_config& f = c->cfg;
#define PROLOGUE(TYPE)                                                                                                   \
  k_sk_prologue<TYPE><<<g.T, 256, 0, s>>>(step_map(c, g, false), g.T, f.d_model, f.vocab, (g.T + 15) / 16, g.tokens,       \
                                    (const TYPE*)c->tok_emb, (const bf16_t*)gain, WSM(c, x, float), WSM(c, xn, bf16_t), \
                                    WSM(c, ss, float), ss_row_stride(c), f.mask_id, (int)c->map.r_max,                   \
                                    WSM(c, rows, int32_t), cand, conf, entropy)
  if (f.dtype == DLLM_BF16) PROLOGUE(bf16_t);
  else PROLOGUE(float);
#undef PROLOGUE
  return hipGetLastError();
}

// out[M,N] = A[M,K] * W[N,K]^T in float (debug logits)
hipError_t launch_sk_f32(dllm_ctx* c, hipStream_t s, const void* A, const void* W, float* out, int M, int N, int K,
                         int n_ss) {
  SkArgs a = sk_base(A, M, K);
  sk_row_scale(c, a, n_ss);
  a.W0 = (const bf16_t*)W;
  a.N0 = N;
  a.out_f32 = out;
  return sk_launch_mt<4, 4, SK_F32>(s, a, (N + 63) / 64);
}

// fused q/k/v projection of a denoise step: rotary embedding on q and k, q to the workspace,
// k and v into the in-flight pages of the pool
// workgroups of the q/k/v product with the value tiles apart from the rotary pairs, two to a workgroup; and of the form taken
static int sk_qkv_apart(const dllm_ctx* c) {
  const dllm_config& f = c->cfg;
  return (f.n_q_heads + f.n_kv_heads) * (f.head_dim / 32) + (f.n_kv_heads * (f.head_dim / 16) + 1) / 2;
}
int sk_qkv_grid(const dllm_ctx* c) {
  const dllm_config& f = c->cfg;
  const int apart = sk_qkv_apart(c), pairs = (f.n_q_heads + f.n_kv_heads) * (f.head_dim / 32), values = f.n_kv_heads * (f.head_dim / 16);
  return apart <= device_cus() ? apart : pairs > values ? pairs : values;
}

hipError_t launch_sk_qkv(dllm_ctx* c, hipStream_t s, const StepGeom& g, int layer, const KVView& pool, int n_ss) {
  const dllm_config& f = c->cfg;
  SkArgs a = sk_base(c->ws + c->map.xn, g.T, f.d_model);
  if (g.T > SK_MAX_ROWS) a.rscale = WSM(c, rscale, float);
  else sk_row_scale(c, a, n_ss);
  const dllm_layer_w& P = g.T > SK_MAX_ROWS ? c->layers[layer] : c->packed_layers[layer];
  a.W0 = (const bf16_t*)P.wq; a.W1 = (const bf16_t*)P.wk; a.W2 = (const bf16_t*)P.wv;
  a.N0 = f.n_q_heads * f.head_dim; a.N1 = a.N2 = f.n_kv_heads * f.head_dim;
  a.out_bf16 = WSM(c, q, bf16_t);
  a.dh = f.head_dim;
  const int per_head = f.head_dim / 2 / 16;
  a.n_q_wg = f.n_q_heads * per_head;
  a.n_k_wg = f.n_kv_heads * per_head;
  a.rope_cos = WSM(c, rope_cos, float); a.rope_sin = WSM(c, rope_sin, float);
  a.tok_seq = WSM(c, tok_seq, int32_t); a.tok_pos = WSM(c, tok_pos, int32_t);
  a.pool_k = (bf16_t*)pool.k; a.pool_v = (bf16_t*)pool.v; a.pool = pool;
  a.status = WSM(c, status, int32_t);
  // Value tiles in workgroups of their own where all then still run at once (few key heads: 128 pair tiles and 32 value
  // tiles took 128 workgroups of three tiles, most of them with one to throw away: 16.0 -> 13.1 us at 32 rows of 3584,
  // 21.4 -> 19.0 at 64, 27.8 -> 24.3 at 128).
  const int grid = sk_qkv_grid(c);
  if (sk_qkv_apart(c) <= device_cus()) {
    // Short stages on more than 13/16 of the CUs where the long ones leave a rest of K (us, long / short at 16 and 32 rows: 216
    // workgroups of K = 2304 10.0 / 8.9, 11.2 / 10.6; 240 of 2560 11.6 / 10.6, 13.4 / 12.4; 252 of 2688 12.1 / 11.2, 14.1 / 12.8 and of
    // 3584 14.0 / 13.2, 16.0 / 15.4; 224 of 3584 13.3 / 12.7, 15.1 / 15.5; but 208 of 3328 12.2 / 12.3, 14.0 / 14.8, 144 of 1536 7.2 / 8.2, 8.2
    // / 9.4, and without a rest 240 of 3072 12.1 / 11.7, 13.8 / 13.8, of 2048 10.2 / 10.1, 11.5 / 12.0).
    if (g.T <= 32 && a.K % (4 * 32 * SK_NW) != 0 && grid > device_cus() * 13 / 16)
      return g.T <= 16 ? sk_go<2, 1, SK_NW, SK_QKV, true>(s, a, grid) : sk_go<2, 2, SK_NW, SK_QKV, true>(s, a, grid);
    return sk_launch_mt<2, SK_NW, SK_QKV>(s, a, grid);
  }
  return sk_launch_mt<3, SK_NW, SK_QKV>(s, a, grid);
}

// h[M,F] = silu(xn Wg^T) * (xn Wu^T), written in fragment order for the down projection
hipError_t launch_sk_swiglu(dllm_ctx* c, hipStream_t s, int layer, int M, int n_ss) {
  const dllm_config& f = c->cfg;
  SkArgs a = sk_base(c->ws + c->map.xn, M, f.d_model);
  sk_row_scale(c, a, n_ss);
  const dllm_layer_w& P = c->packed_layers[layer];
  a.W0 = (const bf16_t*)P.w_gate; a.W1 = (const bf16_t*)P.w_up;
  a.N0 = f.d_ff;
  a.out_bf16 = WSM(c, h, bf16_t);
  // Three tile pairs per workgroup read the activations a third as often.  With one pair those reads are as many bytes as
  // the weights at 32 rows and twice as many at 64, and although the L2 serves them their time adds to the stream's (a
  // stream of 200 MB from memory with 0 / 200 / 400 / 800 MB from the L2 beside it: 32 / 37 / 46 / 64 us).  F = 12288,
  // K = 4096, us, one pair / three: 32 rows 40.0 / 38.1, 48 rows 46.4 / 40.4, 64 rows 59.2 / 42.4; F = 18944, K = 3584: 57.1 /
  // 55.1, -, 82.1 / 68.3; 16 rows 36.3 / 36.7 and 48.1 / 51.3, hence one there.  A workgroup of three fills its CU: up to 48 rows
  // they have to be one round that leaves no more than a quarter of the CUs idle (d_ff 14336 is 299 of them, 13824 288: 32 rows 50 /
  // 61 and 64 / 73, 48 rows 58 / 68 and 74 / 83; 28672 597: 177 / 183); at 64 rows the activations cost more than a last
  // round does (75 / 73, 94 / 91; 246 / 212).
  const int pairs = (f.d_ff + 15) / 16, wgs = (pairs + 2) / 3, cus = device_cus();
  if (M > 16 && wgs >= cus * 3 / 4 && (M > 48 || wgs <= cus)) return sk_launch_mt<6, SK_NW, SK_SWIGLU>(s, a, wgs);
  return sk_launch_mt<2, SK_NW, SK_SWIGLU>(s, a, pairs);
}

// The compacted rows of a forward of many tokens (ws.xn row-major x * gain; the norm has left their mean squares in
// ws.ss, from which the head's kernel takes the very factor that the norm computed) as the weight-streaming LM head reads them: fragment order in ws.h (free behind the last layer).  One workgroup per
// row; a launch of 5 us.  A refresh of 1184 tokens with the outputs of 32 rows: LM head 263 us on 128 x 128 tiles, 211 + 5
// here; one layer and the head at 300 tokens and 4 / 32 / 64 rows: 0.78 / 0.80 / 0.84 of the time on the 8B shape, 0.63 /
// 0.64 / 0.70 on the 7B shape, 0.60 / 0.66 / 0.75 at 1024 channels, 0.72 / 0.74 / 0.81 at 256 x 40000.
__global__ __launch_bounds__(256) void k_sk_head_rows(int d, int mt, const int32_t* n_rows, const bf16_t* xn, bf16_t* X) {
  const int row = blockIdx.x;
  if (row >= *n_rows) return;
  const int d_pad = (d + SK_KB - 1) / SK_KB * SK_KB;
  for (int k = threadIdx.x * 8; k < d_pad; k += 256 * 8)
    *(u32x4*)(X + frag_offset(row, k, mt)) = k < d ? *(const u32x4*)(xn + (int64_t)row * d + k) : u32x4{0, 0, 0, 0};
}
// LM heads of at most 64 rows behind a forward of many tokens: the packed weights stream faster than tiles of mostly
// padding rows read them
bool sk_head_supported(const dllm_ctx* c, int max_rows) {
  return mfma_supported(c) && max_rows <= 64 && c->cfg.d_ff >= c->cfg.d_model;
}
hipError_t launch_sk_head_rows(dllm_ctx* c, hipStream_t s, int max_rows) {
  const dllm_config& f = c->cfg;
  k_sk_head_rows<<<max_rows, 256, 0, s>>>(f.d_model, (max_rows + 15) / 16, WSM(c, status, int32_t) + 1, WSM(c, xn, bf16_t),
                                          WSM(c, h, bf16_t));
  return hipGetLastError();
}

// LM head on all rows of the step (X holds x * final gain) -> per-64-column softmax statistics of every row;
// the merge picks the masked ones.  If no row is masked (device count) nothing is computed.
hipError_t launch_sk_lmstats(dllm_ctx* c, hipStream_t s, const void* X, int T, int n_ss, int* n_parts_out) {
  const dllm_config& f = c->cfg;
  SkArgs a = sk_base(X, T, f.d_model);
  sk_row_scale(c, a, n_ss > 0 ? n_ss : 1);
  if (n_ss == 0) a.inv_d = 1.0f;
  a.n_lm_rows = WSM(c, status, int32_t) + 1;
  a.W0 = (const bf16_t*)c->packed_lm_head;
  a.N0 = f.vocab;
  a.part = WSM(c, lm_part, float);
  a.n_parts = (f.vocab + 63) / 64;
  a.mask_id = f.mask_id;
  *n_parts_out = a.n_parts;
  return sk_launch_mt<4, 4, SK_LMSTATS>(s, a, a.n_parts);
}

}  // namespace dllm

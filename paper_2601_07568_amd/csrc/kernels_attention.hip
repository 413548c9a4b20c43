// bfloat16 matrix-core (MFMA) kernels for gfx950: attention.
#include "mfma_common.h"
#include <type_traits>

namespace dllm {

// ==========================================================================================
// Block-query attention of a denoise step over the paged pool, register-direct: no LDS.
//
// One wave owns 16*QT query rows of one (sequence, kv head) -- with grouped-query attention the
// rows are (head-in-group, token) pairs -- and walks 32-key blocks.  S^T = K Q^T is computed with
// K rows as the A operand; A-row rho of tile t is given key 8*(rho/4) + rho%4 + 4t of the block,
// so that the accumulator layout (column = query, rows 4g..4g+3) leaves lane group g holding
// exactly keys 8g..8g+7 of each query: the B operand of O^T = V^T P^T without any shuffle.  V is
// stored transposed in the pool, so the A operand of that product is a 16-byte load as well.
// Softmax statistics of a query live in the lanes that hold its column.  Several units (waves)
// may split the keys of one row group; each writes an unnormalised partial (m, l, O) and
// k_attn_combine merges them.
struct AttnArgs {
  const bf16_t* q;          // [T, Hq, DH] rotated
  const int32_t* prefix_len;  // denoise step: keys = prefix_len[b] + Q (or + q_valid[b])
  const int32_t* q_valid;     // denoise step, optional: rows past q_valid[b] are padding and no keys
  const int32_t* cu;          // no-cache forward (Q == 0): sequence b is rows cu[b] .. cu[b+1], keys = its length
  bf16_t* o;                // output when n_units == 1 (row-major, or fragment order if out_mt > 0)
  int out_mt;
  KVView kv;
  int Q, Hq, Hkv, B;
  int n_units;              // key-splitting units per row group (gridDim.x * waves along keys)
  int kspl;                 // units (waves along the keys) inside a workgroup; their partials are merged in LDS
  int n_parts;              // partials per row = workgroups along the keys
  int n_rg_wg;              // row groups per workgroup
  int pt_shift;             // log2(page_tokens) if that is a power of two (0 for the packed scratch), else -1
  int pg_cap;               // k_attn_dl: page ids of a unit's blocks that its LDS copy of the block table holds
  float scale_log2;         // log2(e) / sqrt(DH)
  float* part_o;            // [T*Hq, n_units, DH]
  float* part_ml;           // [T*Hq, n_units, 2]
  int32_t* status;
};


// Online softmax of one 32-key block for QT query tiles; the lane holds raw scores of keys
// k0 + 8g + 4tt + i.  Updates the running maximum (in log2 units), the lane's share of the
// denominator and rescales the accumulators only when some maximum of the wave moved.
// Probabilities enter the second product as a bfloat16 pair hi + lo (two instructions): a
// single rounding of p would be the largest error of the whole attention and would flip the
// rounding of a good fraction of the stored outputs.
template <int DT, int QT>
__device__ __forceinline__ void attn_softmax_block(f32x4 (&s)[2][QT], int k0, int kv_len, int g, float scale_log2,
                                                   float (&m_run)[QT], float (&l_run)[QT], f32x4 (&oacc)[DT][QT],
                                                   u32x4 (&pf)[QT], u32x4 (&pl)[QT]) {
  if (k0 + 32 > kv_len) {                               // only a sequence's last block has keys to mask
#pragma unroll
    for (int tt = 0; tt < 2; ++tt)
#pragma unroll
      for (int t = 0; t < QT; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (k0 + 8 * g + 4 * tt + i >= kv_len) s[tt][t][i] = -DEV_INF;
  }
#pragma unroll
  for (int t = 0; t < QT; ++t) {
    float mx = fmaxf(fmaxf(fmaxf(s[0][t][0], s[0][t][1]), fmaxf(s[0][t][2], s[0][t][3])),
                     fmaxf(fmaxf(s[1][t][0], s[1][t][1]), fmaxf(s[1][t][2], s[1][t][3])));
    mx = rows_max(mx);
    const float m_new = fmaxf(m_run[t], mx * scale_log2);   // finite: every block has at least one valid key
    if (__builtin_amdgcn_ballot_w64(m_new > m_run[t]) != 0) {
      const float alpha = __builtin_amdgcn_exp2f(m_run[t] - m_new);   // exp2(-inf) = 0 on the first block
      l_run[t] *= alpha;
#pragma unroll
      for (int d = 0; d < DT; ++d) oacc[d][t] = oacc[d][t] * alpha;
      m_run[t] = m_new;
    }
    float p[8], ps = 0.f;
#pragma unroll
    for (int tt = 0; tt < 2; ++tt)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float e = __builtin_amdgcn_exp2f(fmaf(s[tt][t][i], scale_log2, -m_new));
        p[tt * 4 + i] = e;
        ps += e;
      }
    l_run[t] += ps;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const uint32_t h = pack_bf16x2(p[2 * e], p[2 * e + 1]);
      pf[t][e] = h;
      pl[t][e] = pack_bf16x2(p[2 * e] - __uint_as_float(h << 16), p[2 * e + 1] - __uint_as_float(h & 0xffff0000u));
    }
  }
}

// What partial results are brought to: their largest maximum, or any number if that is -inf.  Those parts have no keys (sums of 0)
// or none but scores that are NaN; their factor is 0 either way, and their NaN sums stay NaN.
__device__ __forceinline__ float attn_base(float mx) { return mx > -DEV_INF ? mx : 0.f; }

// WPS: waves per SIMD that the registers allow.  Left to itself the compiler takes 340 for heads of 128 channels and with
// them the second wave of a SIMD, whose loads fill the time that the first one's products and round trips leave (us, one /
// two waves, 32 key heads: 8 sequences of 700 keys 37.5 / 30.1 = 2.9 TB/s, 16 of 2048 126 / 117, one of 1024 14.7 / 14.6; 64
// rows, one of 1237 keys 22.2 / 18.8).  One wave where several row groups of a workgroup read the same keys through long
// units: their shared lines last longer in the L1 (a layer of 256 channels, one / two waves, 32 key heads, 64 rows: 6 sequences of
// 2500 keys 158 / 169, of 6000 249 / 287, 5 of 4000 179 / 194; 80 rows, 3 of 5000 177 / 204).
template <int DH, int QT, int WPS>
__global__ __launch_bounds__(256, WPS) void k_attn_step(const AttnArgs a) {
  constexpr int KK = DH / 32;   // k-steps of Q K^T
  constexpr int DT = DH / 16;   // 16-row tiles of O^T
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int c = lane & 15, g = lane >> 4;
  const int rg = blockIdx.y * a.n_rg_wg + (w % a.n_rg_wg);
  const int unit = blockIdx.x * a.kspl + (w / a.n_rg_wg);
  extern __shared__ __attribute__((aligned(16))) unsigned char attn_smem[];
  const int b = blockIdx.z / a.Hkv, kvh = blockIdx.z - b * a.Hkv;
  const int G = a.Hq / a.Hkv;
  const bool paged = a.Q > 0;
  const int row_base = paged ? b * a.Q : a.cu[b];               // first row of the sequence in q / o
  const int n_q = paged ? a.Q : a.cu[b + 1] - a.cu[b];          // its query rows
  const int R = n_q * G;
  if (rg * 16 * QT >= R) return;
  if (paged && a.q_valid && a.q_valid[b] < 0) return;       // the sequence is not part of this call
  const int kv_len = paged ? a.prefix_len[b] + (a.q_valid ? min(max(a.q_valid[b], 0), a.Q) : a.Q) : n_q;
  const KVView& kv = a.kv;
  const int pt = paged ? kv.page_tokens : 1;
  const bf16_t* kslab = (const bf16_t*)kv.k;
  const bf16_t* vslab = (const bf16_t*)kv.v;
  const int32_t* table = paged ? kv.table + (int64_t)b * kv.max_pages : nullptr;
  // packed scratch: K [Hkv][tpad][DH], V [Hkv][DH][tpad], the sequence starts at column cu_pad[b]
  const int64_t pcol = paged ? 0 : kv.cu_pad[b];

  // query fragments: B operand, column c = row of this wave's tile
  u32x4 qf[QT][KK];
  int64_t row_out[QT];        // (token * Hq + head) of the lane's query, -1 if beyond R
#pragma unroll
  for (int t = 0; t < QT; ++t) {
    int r = rg * 16 * QT + t * 16 + c;
    const bool ok = r < R;
    if (!ok) r = 0;
    const int hg = r / n_q, j = r - hg * n_q;
    const int64_t ro = (int64_t)(row_base + j) * a.Hq + kvh * G + hg;
    row_out[t] = ok ? ro : -1;
    const bf16_t* qp = a.q + ro * DH + g * 8;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) qf[t][kk] = *(const u32x4*)(qp + kk * 32);
  }

  f32x4 oacc[DT][QT];
#pragma unroll
  for (int d = 0; d < DT; ++d)
#pragma unroll
    for (int t = 0; t < QT; ++t) oacc[d][t] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m_run[QT], l_run[QT];
#pragma unroll
  for (int t = 0; t < QT; ++t) { m_run[t] = -DEV_INF; l_run[t] = 0.f; }
  bool bad = false;

  // A wave takes its 32-key blocks two at a time: the page ids of both, then the K and V^T
  // fragments of both are requested before the first is multiplied, so the second block's two
  // memory round trips hide behind the first block's arithmetic (at batch 1 a wave owns about
  // two blocks and the kernel is a chain of latencies).
  struct Blk {
    u32x4 kf[2][KK];   // K fragments (A operand): tile tt row c <-> key k0 + 8*(c/4) + c%4 + 4*tt
    u32x4 vf[DT];      // V^T fragments (A operand of the second product): row = channel d*16 + c, keys k0+8g..+7
    bool pbad;         // the V page is not addressable
  };
  auto key_of = [&](int kb, int which) -> int {     // which: 0, 1 = K tiles, 2 = V; clamped into the sequence
    const int k0 = kb << 5;
    if (which < 2) {
      const int key = k0 + 8 * (c >> 2) + (c & 3) + 4 * which;
      return key < kv_len ? key : kv_len - 1;       // masked at the scores; keeps the load in bounds
    }
    const int key = k0 + 8 * g;
    return key < kv_len ? key : (kv_len - 1) & ~7;  // zeroed before use
  };
  auto pages = [&](int kb, int (&pg)[3]) {
    if (paged) {
#pragma unroll
      for (int x = 0; x < 3; ++x) {
        const int pi = key_of(kb, x) / pt;
        const int v = table[pi < kv.max_pages ? pi : kv.max_pages - 1];
        pg[x] = pi < kv.max_pages ? v : -1;
      }
    }
  };
  // pages that are multiples of 32 tokens: a block lies inside one, so all lanes share the page and the slot of the block's
  // first key (a division per block instead of three per lane and block)
  auto issue_in_page = [&](int kb, int page, Blk& blk) {
    const int k0 = kb << 5, slot0 = k0 - k0 / pt * pt, left = kv_len - 1 - k0;
    const bool ok = (uint32_t)page < (uint32_t)kv.n_pages;
    bad |= !ok;
    blk.pbad = !ok;
    const int64_t ph = (int64_t)(ok ? page : 0) * kv.n_kv_heads + kvh;
    const bf16_t* kp = kslab + (ph * pt + slot0) * DH + g * 8;
#pragma unroll
    for (int tt = 0; tt < 2; ++tt) {
      const int off = 8 * (c >> 2) + (c & 3) + 4 * tt;
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) blk.kf[tt][kk] = *(const u32x4*)(kp + (off < left ? off : left) * DH + kk * 32);
    }
    const bf16_t* vp = vslab + (ph * DH + c) * pt + slot0 + (8 * g <= left ? 8 * g : left & ~7);
#pragma unroll
    for (int d = 0; d < DT; ++d) blk.vf[d] = *(const u32x4*)(vp + (int64_t)d * 16 * pt);
  };
  auto issue = [&](int kb, const int (&pg)[3], Blk& blk) {
#pragma unroll
    for (int tt = 0; tt < 2; ++tt) {
      const int key = key_of(kb, tt);
      const bf16_t* kp;
      if (paged) {
        const bool ok = (uint32_t)pg[tt] < (uint32_t)kv.n_pages;
        bad |= !ok;
        kp = kslab + (((int64_t)(ok ? pg[tt] : 0) * kv.n_kv_heads + kvh) * pt + (key - key / pt * pt)) * DH + g * 8;
      } else {
        kp = kslab + ((int64_t)kvh * kv.tpad + pcol + key) * DH + g * 8;
      }
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) blk.kf[tt][kk] = *(const u32x4*)(kp + kk * 32);
    }
    const int key = key_of(kb, 2);
    const bf16_t* vp;
    int64_t vstep;                                           // elements between channels d*16 and (d+1)*16
    blk.pbad = false;
    if (paged) {
      const bool ok = (uint32_t)pg[2] < (uint32_t)kv.n_pages;
      bad |= !ok;
      blk.pbad = !ok;
      vp = vslab + (((int64_t)(ok ? pg[2] : 0) * kv.n_kv_heads + kvh) * DH + c) * pt + (key - key / pt * pt);
      vstep = (int64_t)16 * pt;
    } else {
      vp = vslab + ((int64_t)kvh * DH + c) * kv.tpad + pcol + key;
      vstep = (int64_t)16 * kv.tpad;
    }
#pragma unroll
    for (int d = 0; d < DT; ++d) blk.vf[d] = *(const u32x4*)(vp + d * vstep);
  };
  auto compute = [&](int kb, Blk& blk) {
    const int k0 = kb << 5;
    if (__builtin_amdgcn_ballot_w64(blk.pbad) != 0 || k0 + 32 > kv_len) {
      // zero what lies beyond the sequence (or in a page that is not addressable): the slots may
      // hold anything, and 0 * NaN would poison the row
#pragma unroll
      for (int d = 0; d < DT; ++d) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          uint32_t v = blk.vf[d][e];
          const int ke = k0 + 8 * g + 2 * e;
          if (blk.pbad || ke >= kv_len) v &= 0xffff0000u;
          if (blk.pbad || ke + 1 >= kv_len) v &= 0x0000ffffu;
          blk.vf[d][e] = v;
        }
      }
    }
    // ---- S^T tiles
    f32x4 s[2][QT];
#pragma unroll
    for (int tt = 0; tt < 2; ++tt)
#pragma unroll
      for (int t = 0; t < QT; ++t) {
        f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) acc = mfma16(blk.kf[tt][kk], qf[t][kk], acc);
        s[tt][t] = acc;
      }
    // ---- online softmax per query column
    u32x4 pf[QT], pl[QT];
    attn_softmax_block<DT, QT>(s, k0, kv_len, g, a.scale_log2, m_run, l_run, oacc, pf, pl);
    // ---- O^T += V^T P^T
#pragma unroll
    for (int d = 0; d < DT; ++d)
#pragma unroll
      for (int t = 0; t < QT; ++t) {
        oacc[d][t] = mfma16(blk.vf[d], pf[t], oacc[d][t]);
        oacc[d][t] = mfma16(blk.vf[d], pl[t], oacc[d][t]);
      }
  };

  const int nkb = (kv_len + 31) >> 5;
  if (paged && pt % 32 == 0) {
    // A 32-key block lies inside one page, so its page id does not depend on where the sequence ends: the ids of a
    // wave's first two blocks are requested before the sequence length is known (the table row has max_pages
    // entries whatever the length), one memory round trip less in front of the K/V loads; later pairs' ids are
    // requested a pair ahead.
    auto block_page = [&](int kb) -> int {
      const int pi = (kb << 5) / pt;
      const int v = table[pi < kv.max_pages ? pi : kv.max_pages - 1];
      return pi < kv.max_pages ? v : -1;
    };
    int pga = block_page(unit), pgb = block_page(unit + a.n_units);
    for (int kb = unit; kb < nkb; kb += 2 * a.n_units) {
      const int kb2 = kb + a.n_units;
      const bool two = kb2 < nkb;
      Blk ba, bb;
      issue_in_page(kb, pga, ba);
      issue_in_page(two ? kb2 : kb, two ? pgb : pga, bb);   // (a repeat of the first block's loads: no branch around a load)
      pga = block_page(kb + 2 * a.n_units);
      pgb = block_page(kb2 + 2 * a.n_units);
      compute(kb, ba);
      if (two) compute(kb2, bb);
    }
  } else {
    for (int kb = unit; kb < nkb; kb += 2 * a.n_units) {
      const int kb2 = kb + a.n_units;
      const bool two = kb2 < nkb;
      const int kbb = two ? kb2 : kb;             // a repeat of the first block's loads: no branch around a load
      int pga[3], pgb[3];
      pages(kb, pga);
      pages(kbb, pgb);
      Blk ba, bb;
      issue(kb, pga, ba);
      issue(kbb, pgb, bb);
      compute(kb, ba);
      if (two) compute(kb2, bb);
    }
  }

  // ---- results: lane holds query column c, channels d*16 + 4g + i
  float l_red[QT];
#pragma unroll
  for (int t = 0; t < QT; ++t) {
    float l = l_run[t];
    l += __shfl_xor(l, 16, 64);
    l += __shfl_xor(l, 32, 64);
    l_red[t] = l;
  }
  auto store_out = [&](int d, int t, f32x4 v, float l) {       // normalised output, the row's only partial
    const float inv = l > 0.f ? 1.0f / l : 0.f;
    const int64_t ro = row_out[t];
    const int tok = (int)(ro / a.Hq), head = (int)(ro - (int64_t)tok * a.Hq);
    const int ch = d * 16 + 4 * g;
    const int64_t at = a.out_mt > 0 ? frag_offset(tok, head * DH + ch, a.out_mt) : ro * DH + ch;
    *(uint2*)(a.o + at) = make_uint2(pack_bf16x2(v[0] * inv, v[1] * inv), pack_bf16x2(v[2] * inv, v[3] * inv));
  };
  if (a.kspl > 1) {
    // The workgroup's waves hold partial results of the same rows over different keys (launched only
    // with one row group per workgroup, so every wave is here): bring them to a common maximum,
    // park them in LDS and let each wave add up a slice of the channels, in wave order.
    const int KS = a.kspl;
    float* sm_m = (float*)attn_smem;                           // [KS][QT][16]
    float* sm_l = sm_m + KS * QT * 16;                         // [KS][QT][16]
    f32x4* sm_o = (f32x4*)(attn_smem + 2 * KS * QT * 16 * sizeof(float));   // [KS][DT*QT][64]
    if (g == 0) {
#pragma unroll
      for (int t = 0; t < QT; ++t) { sm_m[(w * QT + t) * 16 + c] = m_run[t]; sm_l[(w * QT + t) * 16 + c] = l_red[t]; }
    }
    __syncthreads();
    float m_all[QT], l_all[QT];
#pragma unroll
    for (int t = 0; t < QT; ++t) {
      float mx = -DEV_INF;
      for (int ww = 0; ww < KS; ++ww) mx = fmaxf(mx, sm_m[(ww * QT + t) * 16 + c]);
      const float base = attn_base(mx);
      float ls = 0.f;
      for (int ww = 0; ww < KS; ++ww) ls = fmaf(sm_l[(ww * QT + t) * 16 + c], exp2f(sm_m[(ww * QT + t) * 16 + c] - base), ls);
      m_all[t] = mx;
      l_all[t] = ls;
      const float f = exp2f(m_run[t] - base);
#pragma unroll
      for (int d = 0; d < DT; ++d) sm_o[(w * DT * QT + d * QT + t) * 64 + lane] = oacc[d][t] * f;
    }
    __syncthreads();
    for (int u = w; u < DT * QT; u += KS) {
      const int d = u / QT, t = u - d * QT;
      f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
      for (int ww = 0; ww < KS; ++ww) acc = acc + sm_o[(ww * DT * QT + u) * 64 + lane];
      if (row_out[t] < 0) continue;
      if (a.n_parts == 1) { store_out(d, t, acc, l_all[t]); continue; }
      const int64_t slot = row_out[t] * a.n_parts + blockIdx.x;
      *(f32x4*)(a.part_o + slot * DH + d * 16 + 4 * g) = acc;
      if (d == 0 && g == 0) { a.part_ml[slot * 2] = m_all[t]; a.part_ml[slot * 2 + 1] = l_all[t]; }
    }
  } else {
#pragma unroll
    for (int t = 0; t < QT; ++t) {
      if (row_out[t] < 0) continue;
      if (a.n_parts == 1) {
#pragma unroll
        for (int d = 0; d < DT; ++d) store_out(d, t, oacc[d][t], l_red[t]);
        continue;
      }
      const int64_t slot = row_out[t] * a.n_parts + unit;
      float* po = a.part_o + slot * DH + 4 * g;
#pragma unroll
      for (int d = 0; d < DT; ++d) *(f32x4*)(po + d * 16) = oacc[d][t];
      if (g == 0) { a.part_ml[slot * 2] = m_run[t]; a.part_ml[slot * 2 + 1] = l_red[t]; }
    }
  }
  if (bad) atomicOr(a.status, DLLM_STATUS_BAD_PAGE);
}

// The merge of two partial results a row, for many rows: four channels a lane (a lane per channel, 28672 rows of 128: 7168
// workgroups of a few loads each, 13.4 us, 8.5 so).
template <int DH>
__global__ __launch_bounds__(256) void k_attn_combine2(const float* part_o, const float* part_ml, bf16_t* o, int Hq, int mt, int64_t n_rows) {
  constexpr int LR = DH / 4;                            // lanes of a row
  const int64_t row = (int64_t)blockIdx.x * (256 / LR) + threadIdx.x / LR;
  if (row >= n_rows) return;
  const int d = threadIdx.x % LR * 4;
  const float4 ml = *(const float4*)(part_ml + row * 4);               // (m0, l0, m1, l1)
  const f32x4 o0 = *(const f32x4*)(part_o + row * 2 * DH + d), o1 = *(const f32x4*)(part_o + (row * 2 + 1) * DH + d);
  const float base = attn_base(fmaxf(ml.x, ml.z));
  const float s0 = exp2f(ml.x - base), s1 = exp2f(ml.z - base), den = fmaf(ml.w, s1, ml.y * s0);
  float v[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) v[i] = den == 0.f ? 0.f : fmaf(o1[i], s1, o0[i] * s0) / den;
  const int tok = (int)(row / Hq), head = (int)(row - (int64_t)tok * Hq);
  const int64_t at = mt > 0 ? frag_offset(tok, head * DH + d, mt) : row * DH + d;
  *(uint2*)(o + at) = make_uint2((uint32_t)f32_to_bf16(v[0]) | ((uint32_t)f32_to_bf16(v[1]) << 16), (uint32_t)f32_to_bf16(v[2]) | ((uint32_t)f32_to_bf16(v[3]) << 16));
}

// merges the units' partials of one (token, head) row and stores the normalised output
// (fragment order of the [T, Hq*DH] matrix: it is the activation operand of the output projection)
template <int DH>
__global__ __launch_bounds__(512) void k_attn_combine(const float* part_o, const float* part_ml, int n_units,
                                                      bf16_t* o, int Hq, int mt, int64_t n_rows) {
  const int64_t row = (int64_t)blockIdx.x * (512 / DH) + threadIdx.x / DH;
  if (row >= n_rows) return;
  const int d = threadIdx.x % DH;
  // eight units at a time; the running (max, numerator, denominator) is rescaled between chunks.  The maxima are waited for in
  // front of the sums and outputs: a wave that asks for all of them at once keeps others' small loads waiting (us, at once / maxima
  // ahead / waited for: 16384 rows of 64 in four parts 7.5 / 7.2 / 6.6, 7168 of 128 in five 6.8 / 6.5 / 6.0, in nine 11.3 /
  // 10.9 / 9.6)
  float M = -DEV_INF, num = 0.f, den = 0.f;
  if (n_units == 2) {                                   // the common case at large batch: no padded chunk of eight
    const int64_t slot = row * 2;
    const float4 ml = *(const float4*)(part_ml + slot * 2);            // (m0, l0, m1, l1)
    const float o0 = part_o[slot * DH + d], o1 = part_o[(slot + 1) * DH + d];
    const float base = attn_base(fmaxf(ml.x, ml.z)), s0 = exp2f(ml.x - base), s1 = exp2f(ml.z - base);
    den = fmaf(ml.w, s1, ml.y * s0);
    num = fmaf(o1, s1, o0 * s0);
  } else
  for (int u0 = 0; u0 < n_units; u0 += 8) {
    float mu[8], lu[8], ou[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) mu[i] = part_ml[(row * n_units + min(u0 + i, n_units - 1)) * 2];
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(0x0F70);                 // vmcnt(0)
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int64_t slot = row * n_units + min(u0 + i, n_units - 1);
      lu[i] = part_ml[slot * 2 + 1];
      ou[i] = part_o[slot * DH + d];
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) mu[i] = u0 + i < n_units ? mu[i] : -DEV_INF;
    float Mn = M;
#pragma unroll
    for (int i = 0; i < 8; ++i) Mn = fmaxf(Mn, mu[i]);
    const float base = attn_base(Mn), r = exp2f(M - base);   // exp2(-inf) = 0 on the first chunk
    num *= r;
    den *= r;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const float sc = exp2f(mu[i] - base);             // 0 for empty units
      den = fmaf(lu[i], sc, den);
      num = fmaf(ou[i], sc, num);
    }
    M = Mn;
  }
  const int tok = (int)(row / Hq), head = (int)(row - (int64_t)tok * Hq);
  const int64_t at = mt > 0 ? frag_offset(tok, head * DH + d, mt) : row * DH + d;
  o[at] = f32_to_bf16(den == 0.f ? 0.f : num / den);     // (NaN stays NaN: a key that is not finite shows in every row that sees it)
}

// ------------------------------------------------------------------------------------------
// The same attention for many query rows per KV head (grouped-query models at large batch, and every no-cache
// forward).  The eight waves of a workgroup are row groups of 32 query rows that all need the same keys, so each 64-key
// block of K and V^T is copied from memory into LDS once per workgroup, straight (no register pass).
//
// A block is 64 K rows and DH V^T rows of 64 keys, row-major; one copy instruction of a wave fills one KiB of whole
// 128-byte lines, its 16-byte pieces xor-ed with the row so that the 16 lanes an LDS read serves at a time touch every
// bank once.  NB = 4 buffers form a ring: two blocks are in flight while the products read three (below); the only
// wait on memory is "the next block has landed", once per block, together with the barrier that frees the oldest
// buffer.  The page ids of the unit's blocks lie in LDS; keys past the sequence end are read as they lie in the page (or
// workspace), their scores are masked and their V^T columns zeroed in LDS before use, as are those of keys whose page
// id is not addressable.
//
// What bounds it: a 32-key half costs a wave 24 products of 32 x 32 x 16 (8 of scores, 16 of V^T P^T: P enters as a
// bfloat16 pair hi + lo) = 768 cycles of its SIMD's matrix pipe and about 600 cycles of vector work (16 exponentials
// of 8 cycles, the pair split).  Run one behind the other they add up, and the waves leave each barrier in the same
// phase: the kernel that did so took 2.3 times the products' time.  Here every wave runs them side by side: while it
// takes the exponentials of half u, its matrix instructions are the scores of half u+1 and V^T P^T of half u-1, one
// product and a few vector instructions in turn (sched_barrier keeps the order), LDS reads 4 .. 8 products ahead.
// (us, the kernel before it with 16 x 16 x 32 products / this one: 32 sequences of up to 8192 keys, 4 key heads of 7 x 32
// rows 219 / 191; 8 prompts of up to 2048 tokens, 4 key heads 902 / 665; 1184 tokens, 32 heads 75 / 67.  With four to six row
// groups the other waves only copy, and one workgroup of eight waves a CU still beats the two of four waves that were there:
// 32 heads, 128 rows of one sequence with 901 keys 19.6 / 16.7, 8 sequences of 128 rows 103 / 76 with 2048 keys, 37 / 35 with 300,
// 8 of 104 rows 58 / 47; 5 and 6 groups 85 / 71 and 68 / 55; 8 key heads of 4 x 32 rows, 32 sequences of 1024 keys 62 / 48; 8
// prompts of 128, 160, 256 tokens 16.2 / 14.3, 21.5 / 19.0, 27.1 / 25.8.)  (The chip's clock
// follows the products' power: 24 of them on random operands, with as many vector instructions as here between them,
// take two waves of a SIMD 0.94 us, on zeros 0.70.)
//
// 32 x 32 x 16 layouts (lane l, r = l % 32, h = l / 32): A holds row r, B column r, each the 8 k-elements 8h .. 8h+7;
// D holds column r, rows (e/4)*8 + 4h + e%4.  A row r of a score product is given key 16(r/16) + 8(r/4%2) + 4(r/8%2)
// + r%4 of the half, so that registers 8s .. 8s+7 of D are keys 16s + 8h .. +7 of the lane's query: the B operand of
// step s of V^T P^T as it stands.
//
// The running maximum (log2 units) is an integer and moves only when a score exceeds it by more than DL_SLACK: weights
// reach 2^DL_SLACK, which neither the float sums nor the bfloat16 pairs mind, and the accumulators, the sums and the
// weights that still wait for their product are then scaled by a power of two, which is exact.
#define DL_VMCNT(n) (((n) & 15) | (((n) >> 4) << 14) | 0x0F70)
constexpr float DL_SLACK = 8.0f;
// the value is computed here: neither earlier nor where it is used
template <typename T>
__device__ __forceinline__ void pin(T& x) { asm volatile("" : "+v"(x)); }
template <typename T, typename U>
__device__ __forceinline__ void pin(T& x, U& y) { asm volatile("" : "+v"(x), "+v"(y)); }
// PG: 0 packed scratch; 1 paged, a 64-key block lies inside a page; 2 paged, smaller pages (a power of two of at least 8)
template <int DH, int PG>
__device__ __forceinline__ void attn_dl_body(const AttnArgs& a) {
  constexpr int KK = DH / 16, DT = DH / 32, NM = KK + 4 * DT;   // score steps, channel tiles, products per half
  constexpr int NB = DL_NB, NW = 8;
  constexpr int NKF = DH / 8, NVF = DH / 8, NF = NKF + NVF, FPW = NF / NW;   // KiB of K, of V^T; copies of a wave
  static_assert(NKF % FPW == 0, "a wave's copies are K for all of a wave or V^T for all");
  constexpr int BLK = NF * 1024, nthr = NW * 64, KROW = DH * 2;
  extern __shared__ __attribute__((aligned(1024))) unsigned char dl_smem[];
  int32_t* s_pg = (int32_t*)(dl_smem + NB * BLK);
  const int tid = threadIdx.x;
  const int lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 31, h = lane >> 5;
  const int rg = blockIdx.y * a.n_rg_wg + w;
  const int unit = blockIdx.x;
  const int b = blockIdx.z / a.Hkv, kvh = blockIdx.z - b * a.Hkv;
  const int G = a.Hq / a.Hkv;
  const int row_base = PG ? b * a.Q : a.cu[b];
  const int n_q = PG ? a.Q : a.cu[b + 1] - a.cu[b];
  const int R = n_q * G;
  const int kv_len = PG ? a.prefix_len[b] + (a.q_valid ? min(max(a.q_valid[b], 0), a.Q) : a.Q) : n_q;
  const bool active = w < a.n_rg_wg && rg * 32 < R;   // waves beyond the rows only help loading
  if (blockIdx.y * a.n_rg_wg * 32 >= R) return;              // whole workgroup beyond this sequence's rows
  if (PG && a.q_valid && a.q_valid[b] < 0) return;           // the sequence is not part of this call
  const KVView& kv = a.kv;
  const int sh = a.pt_shift, pt = 1 << sh;
  const bf16_t* kslab = (const bf16_t*)kv.k;
  const bf16_t* vslab = (const bf16_t*)kv.v;
  const int64_t pcol = PG ? 0 : kv.cu_pad[b];
  uint32_t bad = 0;
  const int nkb = (kv_len + 63) >> 6;
  const int n_own = unit < nkb ? (nkb - 1 - unit) / a.n_units + 1 : 0;   // the unit's blocks: unit, unit + n_units, ..

  int np = 0;
  const int32_t* const table = PG ? kv.table + (int64_t)b * kv.max_pages : nullptr;
  if constexpr (PG != 0) {
    np = (kv_len + pt - 1) >> sh;
    np = np < kv.max_pages ? np : kv.max_pages;
  }
  const int ids_sh = PG == 2 ? 6 - sh : 0;                     // log2 of the page ids of a block
  const int n_ids = PG == 0 ? 0 : n_own << ids_sh < a.pg_cap ? n_own << ids_sh : a.pg_cap;

  // this lane's source offsets (bytes from the block's K or V^T base) for the wave's copies; with small pages the
  // key (from the block's first) and the offset from its page's K row or V^T column
  const bool wave_k = w * FPW < NKF;
  int foff[FPW], fkey[PG == 2 ? FPW : 1];
#pragma unroll
  for (int i = 0; i < FPW; ++i) {
    const int f = w * FPW + i;
    int key, off;
    if (f < NKF) {
      constexpr int PR = DH / 8;                              // 16-byte pieces of a K row
      key = f * (64 / PR) + lane / PR;
      const int swz = DH == 128 ? key & 15 : (key >> 1) & 7;
      off = (PG == 2 ? 0 : key * DH) + (((lane % PR) ^ swz) * 8);
    } else {
      const int ch = (f - NKF) * 8 + (lane >> 3);
      key = ((lane & 7) ^ ((ch >> 1) & 7)) * 8;
      off = ch * (PG ? pt : kv.tpad) + (PG == 2 ? 0 : key);
    }
    foff[i] = PG == 2 ? off : off * 2;                        // (small pages: elements)
    if constexpr (PG == 2) fkey[i] = key;
  }
  uint32_t badbuf = 0;                                        // PG 1: buffers with keys from a page id out of range
  // own: 0, 1, .. of the unit's blocks; past the last one it is the last one
  auto clampo = [&](int own) { return own < n_own ? own : n_own - 1; };
  auto block_of = [&](int own) { return unit + clampo(own) * a.n_units; };
  auto page_of = [&](int own) -> int {
    if constexpr (PG != 1) return 0;
    return s_pg[clampo(own)];
  };
  // The block being copied, as a descriptor that ends with it.  (The form of the copies that goes through a flat address
  // makes the compiler wait for all LDS reads wherever it waits for one; small pages, whose keys lie wherever their page
  // does, have only that.)
  const bf16_t* src = nullptr;
  __amdgpu_buffer_rsrc_t rsrc;
  auto copy_base = [&](int kb64, int buf, int page_v) {
    const int k0 = kb64 << 6;
    int64_t kb, vb;
    if constexpr (PG == 1) {
      const int page = __builtin_amdgcn_readfirstlane(page_v);
      const bool ok = (uint32_t)page < (uint32_t)kv.n_pages;
      const uint32_t miss = ok ? 0u : 1u;
      bad |= miss;
      badbuf = (badbuf & ~(1u << buf)) | (miss << buf);
      const int64_t rows = (((int64_t)(ok ? page : 0) * kv.n_kv_heads + kvh) << sh);
      kb = (rows + (k0 & (pt - 1))) * DH;
      vb = rows * DH + (k0 & (pt - 1));
    } else if constexpr (PG == 0) {
      kb = ((int64_t)kvh * kv.tpad + pcol + k0) * DH;
      vb = (int64_t)kvh * DH * kv.tpad + pcol + k0;
    } else {
      kb = vb = 0;
    }
    if constexpr (PG == 2) src = wave_k ? kslab : vslab;
    else {
      const int bytes = wave_k ? 64 * KROW : ((DH - 1) * (PG ? pt : kv.tpad) + 64) * 2;
      rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)(wave_k ? kslab + kb : vslab + vb), 0, bytes, 0x00020000);
    }
  };
  auto copy = [&](int own, int buf, int i) {
    void* const dst = dl_smem + buf * BLK + (w * FPW + i) * 1024;
    if constexpr (PG == 2) {
      const int key = (block_of(own) << 6) + fkey[i];
      const int page = s_pg[(clampo(own) << ids_sh) + (fkey[i] >> sh)];
      const bool ok = (uint32_t)page < (uint32_t)kv.n_pages;
      if (!ok && key < kv_len) bad = 1;
      const int64_t rows = (((int64_t)(ok ? page : 0) * kv.n_kv_heads + kvh) << sh);
      const bf16_t* p = src + rows * DH + (wave_k ? (key & (pt - 1)) * DH : (key & (pt - 1))) + foff[i];
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)p, (__attribute__((address_space(3))) void*)dst, 16, 0, 0);
    } else {
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (__attribute__((address_space(3))) void*)dst, 16, foff[i], 0, 0, 0);
    }
  };
  // the ring's first blocks (past the end: repeats of the last block into buffers nobody reads); their page ids come
  // straight from the table, so that the copies are on their way before anything else is waited for
  auto first_blocks = [&]() {
#pragma unroll
    for (int j = 0; j < NB - 1; ++j) {
      const int kb = block_of(j), pi = (kb << 6) >> sh;
      copy_base(kb, j, PG == 1 && pi < np ? table[pi] : -1);
#pragma unroll
      for (int i = 0; i < FPW; ++i) copy(j, j, i);
    }
  };
  if (PG != 2 && n_own > 0) first_blocks();
  if constexpr (PG != 0)
    for (int i = tid; i < n_ids; i += nthr) {
      const int pi = (((unit + (i >> ids_sh) * a.n_units) << 6) >> sh) + (i & ((1 << ids_sh) - 1));
      s_pg[i] = pi < np ? table[pi] : -1;
    }

  u32x4 qf[KK];               // B operand: column r = the lane's query
  int64_t row_out;            // its (token * Hq + head), -1 if beyond R
  {
    int rr = rg * 32 + r;
    const bool ok = active && rr < R;
    if (!ok) rr = 0;
    const int hg = rr / n_q, j = rr - hg * n_q;
    const int64_t ro = (int64_t)(row_base + j) * a.Hq + kvh * G + hg;
    row_out = ok ? ro : -1;
    const bf16_t* qp = a.q + ro * DH + h * 8;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) qf[kk] = *(const u32x4*)(qp + kk * 16);
  }
  // the buffer in front of block 0 stands for the half in front of the first: its weights are zero, its V^T as well
  {
    u32x4* vb = (u32x4*)(dl_smem + (NB - 1) * BLK + NKF * 1024);
    for (int q = tid; q < NVF * 64; q += nthr) vb[q] = u32x4{0, 0, 0, 0};
  }
  __syncthreads();                                            // page ids are in LDS

  // zeroes the V^T columns of keys past the sequence end and of keys without a page
  auto fix_tail = [&](int own, int buf) {
    const int kb64 = unit + own * a.n_units;
    bool any = (kb64 << 6) + 64 > kv_len;
    if constexpr (PG == 1) any |= (badbuf >> buf) & 1u;
    if constexpr (PG == 2) {
      for (int p = 0; p < 1 << ids_sh; ++p) any |= (uint32_t)s_pg[(own << ids_sh) + p] >= (uint32_t)kv.n_pages;
    }
    if (!any) return;
    u32x4* vb = (u32x4*)(dl_smem + buf * BLK + NKF * 1024);
    for (int q = tid; q < NVF * 64; q += nthr) {
      const int key = (kb64 << 6) + ((q & 7) ^ ((q >> 4) & 7)) * 8;
      int valid = kv_len - key;
      if constexpr (PG == 1) valid = ((badbuf >> buf) & 1u) ? 0 : valid;
      if constexpr (PG == 2) {
        if ((uint32_t)s_pg[(own << ids_sh) + ((key & 63) >> sh)] >= (uint32_t)kv.n_pages) valid = 0;
      }
      if (valid < 8) {
        u32x4 v = vb[q];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          uint32_t x = v[e];
          x = valid > 2 * e + 1 ? x : (x & 0x0000ffffu);
          x = valid > 2 * e ? x : 0u;
          v[e] = x;
        }
        vb[q] = v;
      }
    }
  };

  f32x16 oacc[DT];
#pragma unroll
  for (int d = 0; d < DT; ++d)
#pragma unroll
    for (int e = 0; e < 16; ++e) oacc[d][e] = 0.f;
  float m_run = -DEV_INF, l_run = 0.f, l_odd = 0.f;
  const float scl = a.scale_log2;

  struct Wts { u32x4 hi[2], lo[2]; };                         // weights of a half: B operands of its two steps
  f32x16 sc, sn;                                              // scores of the current half, of the next
  Wts pa, pb;
  u32x4 kf[4], v0[DT], v1[DT];
  int ka[KK], va[4];                                          // LDS addresses: K by step, V^T by 16-key step of the block
  // key of score row r, and the swizzle of its LDS row
  const int kr = 16 * (r >> 4) + 8 * ((r >> 2) & 1) + 4 * ((r >> 3) & 1) + (r & 3);
  const int k_lane = kr * KROW + ((h ^ (DH == 128 ? kr & 15 : (kr >> 1) & 7)) * 16);
  const int v_lane = NKF * 1024 + r * 128 + ((h ^ ((r >> 1) & 7)) * 16);
  // (addresses in LDS as such: with an offset to dl_smem every read adds it)
  typedef __attribute__((address_space(3))) unsigned char lds_u8;
  const int lds0 = (int)(uintptr_t)(lds_u8*)dl_smem;
  auto k_addr = [&](int buf) {
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) ka[kk] = (lds0 + buf * BLK + k_lane) ^ (kk * 32);
  };
  auto v_addr = [&](int buf) {
#pragma unroll
    for (int x = 0; x < 4; ++x) va[x] = (lds0 + buf * BLK + v_lane) ^ (x * 32);
  };
  auto rd = [&](int at) -> u32x4 { return *(const __attribute__((address_space(3))) u32x4*)(uintptr_t)(uint32_t)at; };
  auto mm = [&](u32x4 x, u32x4 y, f32x16 c) -> f32x16 {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, x), __builtin_bit_cast(bf16x8, y), c, 0, 0, 0);
  };
  const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};

  // in front of half k0's exponentials: mask, and now and then the new scale (mx: the scores' maximum, one per half wave)
  auto settle = [&](f32x16& s, float mx, int k0, Wts& open) {
    if (k0 + 32 > kv_len) {                               // only a sequence's last block has keys to mask
      mx = -DEV_INF;
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        if (k0 + 16 * (e >> 3) + 8 * h + (e & 7) >= kv_len) s[e] = -DEV_INF;
        mx = fmaxf(mx, s[e]);
      }
    }
    const uint32_t mi = __float_as_uint(mx);
    const u32x2_t sw = __builtin_amdgcn_permlane32_swap(mi, mi, false, false);
    mx = fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1])) * scl;
    if (__builtin_amdgcn_ballot_w64(mx > m_run + DL_SLACK) != 0) {
      const float m_new = fmaxf(m_run, ceilf(mx));
      const float f = __builtin_amdgcn_ldexpf(1.0f, (int)fmaxf(m_run - m_new, -200.0f));
      m_run = m_new;
      l_run *= f;
      l_odd *= f;
#pragma unroll
      for (int d = 0; d < DT; ++d)
#pragma unroll
        for (int e = 0; e < 16; ++e) oacc[d][e] *= f;
      auto scale2 = [&](uint32_t v) -> uint32_t {
        return (__float_as_uint(__uint_as_float(v << 16) * f) >> 16) | (__float_as_uint(__uint_as_float(v & 0xffff0000u) * f) & 0xffff0000u);
      };
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int e = 0; e < 4; ++e) { open.hi[x][e] = scale2(open.hi[x][e]); open.lo[x][e] = scale2(open.lo[x][e]); }
    }
  };
  // One half: the exponentials of s -> pn beside the scores of the next half (K fragments at ka + HN, four of them read)
  // -> so and V^T P^T of the one before (po; V^T steps 2*HP, 2*HP+1 of the block at va, the first one's fragments read).
  // `mid` runs behind product 2*KK - 1; behind it the fragments that the next call starts with are read: K half HN2,
  // V^T step 2*HP2.  tail(i), i < FPW: copies in the remaining places.
  auto half_step = [&](auto hn_, auto hp_, auto hn2_, auto hp2_, f32x16& s, f32x16& so, Wts& pn, const Wts& po, auto&& mid, auto&& tail) {
    constexpr int HN = decltype(hn_)::value, HP = decltype(hp_)::value, HN2 = decltype(hn2_)::value, HP2 = decltype(hp2_)::value;
    // 24 steps, three per pair of scores, about five instruction slots each.  (pin: sched_barrier does not hold plain
    // arithmetic in its place; nothing reads the weights before the next half, so all of it would move there.)
    float x0 = 0.f, x1 = 0.f, e0 = 0.f, e1 = 0.f, g0 = 0.f, g1 = 0.f;
    uint32_t hi = 0;
    auto vec = [&](int st) {
      const int i = st / 3, ph = st % 3;
      if (ph == 0) {
        pin(s);
        x0 = fmaf(s[2 * i], scl, -m_run);
        x1 = fmaf(s[2 * i + 1], scl, -m_run);
      }
      if (ph == 1) {
        pin(x0, x1);
        e0 = __builtin_amdgcn_exp2f(x0);
        e1 = __builtin_amdgcn_exp2f(x1);
      }
      if (ph == 2) {
        pin(e0, e1);
        l_run += e0;
        l_odd += e1;
        pin(l_run, l_odd);
        hi = pack_bf16x2(e0, e1);
        g0 = e0; g1 = e1;
        pn.hi[i >> 2][i & 3] = hi;
      }
      // the pair before: what its first bfloat16 numbers leave
      if ((ph == 0 && i > 0) || st == 23) {
        const int q = st == 23 ? 7 : i - 1;
        pin(hi);
        uint32_t lo = pack_bf16x2(g0 - __uint_as_float(hi << 16), g1 - __uint_as_float(hi & 0xffff0000u));
        pin(lo);
        pn.lo[q >> 2][q & 3] = lo;
      }
    };
    // the maximum of the next half's scores, in the last products' places
    float t0 = 0.f, t1 = 0.f, t2 = 0.f, t3 = 0.f;
    auto top = [&](int st) {
      auto max3 = [](float a, float b, float c) { return fmaxf(fmaxf(a, b), c); };
      if (st == 0) { pin(so); t0 = max3(so[0], so[1], so[2]); t1 = max3(so[3], so[4], so[5]); }
      if (st == 1) { pin(t1); t2 = max3(so[6], so[7], so[8]); t3 = max3(so[9], so[10], so[11]); }
      if (st == 2) { pin(t2); t0 = max3(t0, t1, t2); t3 = max3(t3, so[12], so[13]); }
      if (st == 3) { pin(t3); t3 = max3(t3, so[14], so[15]); pin(t3); }
      if (st == 4) { t0 = fmaxf(t0, t3); pin(t0); }
    };
#pragma unroll
    for (int idx = 0; idx < NM; ++idx) {
      __builtin_amdgcn_sched_barrier(0);
      if (idx < 2 * KK && (idx & 1) == 0) {
        const int kk = idx / 2;
        so = mm(kf[kk & 3], qf[kk], kk == 0 ? zero16 : so);
      } else {
        const int j = idx < 2 * KK ? idx / 2 : idx - KK, x = j / (2 * DT), lo = (j / DT) & 1, d = j % DT;
        oacc[d] = mm(x ? v1[d] : v0[d], lo ? po.lo[x] : po.hi[x], oacc[d]);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int st = 0; st < 24; ++st)
        if (st * NM / 24 == idx) vec(st);
#pragma unroll
      for (int st = 0; st < 5; ++st)
        if (2 * KK + (NM - 2 * KK) / 4 + st * (NM - 2 * KK) / 8 == idx) top(st);
      // reads: K fragments 4 .. of this half into the places just used, V^T of the second step
      if (idx < 2 * KK && (idx & 1) == 0 && idx / 2 + 4 < KK) kf[(idx / 2) & 3] = rd(ka[(idx / 2 + 4) % KK] + HN * 32 * KROW);
      if (idx >= KK && idx < KK + DT) v1[idx - KK] = rd(va[2 * HP + 1] + (idx - KK) * 4096);
      if (idx == 2 * KK - 1) mid();
      if (idx >= 2 * KK) {
        constexpr int NR = 4 + DT, SL = NM - 2 * KK;
#pragma unroll
        for (int n = 0; n < NR; ++n)
          if (2 * KK + n * SL / NR == idx) {
            const int q = n / 2;
            if (n < 2 * DT && (n & 1)) v0[q % DT] = rd(va[2 * HP2] + (q % DT) * 4096);
            else { const int k2 = n < 2 * DT ? q : n - DT; kf[k2 & 3] = rd(ka[k2 % KK] + HN2 * 32 * KROW); }
          }
#pragma unroll
        for (int i = 0; i < FPW; ++i)
          if (2 * KK + i * SL / FPW == idx) tail(i);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    return t0;
  };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;

  if (n_own > 0) {           // (a unit without keys still writes its empty partial below)
    if (PG == 2) first_blocks();
    int pg_next = page_of(NB - 1);
    // the first block has landed; with everything in front of it (PG 2), or with the q loads that were issued behind it
    if constexpr (PG == 2) __builtin_amdgcn_s_waitcnt(DL_VMCNT(2 * FPW));
    else __builtin_amdgcn_s_waitcnt(DL_VMCNT(0));
    __builtin_amdgcn_s_barrier();
    fix_tail(0, 0);           // read behind the barrier inside the loop
    int buf = 0;
    float mx = -DEV_INF;
    if (active) {
      k_addr(0);
      v_addr(NB - 1);
#pragma unroll
      for (int x = 0; x < 2; ++x) pa.hi[x] = pa.lo[x] = pb.hi[x] = pb.lo[x] = u32x4{0, 0, 0, 0};
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) sc = mm(rd(ka[kk]), qf[kk], kk == 0 ? zero16 : sc);
#pragma unroll
      for (int e = 0; e < 16; ++e) mx = fmaxf(mx, sc[e]);
#pragma unroll
      for (int x = 0; x < 4; ++x) kf[x] = rd(ka[x % KK] + 32 * KROW);
#pragma unroll
      for (int d = 0; d < DT; ++d) v0[d] = u32x4{0, 0, 0, 0};
    }
    for (int own = 0; own < n_own; ++own) {
      const int kb = unit + own * a.n_units;
      const int nbuf = buf == 0 ? NB - 1 : buf - 1;            // (buf + NB - 1) % NB: the buffer of the block before
      const int buf1 = buf + 1 == NB ? 0 : buf + 1;
      const int kn = block_of(own + NB - 1);
      if (own > 0) fix_tail(own, buf);
      // (the counts are exact only while the loop issues no other vector memory instruction: no spills to scratch,
      // which the build's resource report shows)
      auto turn = [&]() {
        __builtin_amdgcn_s_waitcnt(DL_VMCNT(FPW) & 0xF0FF);   // this wave's copies of the next block have landed, its reads are back
        __builtin_amdgcn_s_barrier();                          // everybody's; the buffer of the block before is free
        copy_base(kn, nbuf, pg_next);
      };
      if (active) {
        settle(sc, mx, kb << 6, pb);
        mx = half_step(I1{}, I1{}, I0{}, I0{}, sc, sn, pa, pb, [&]() { turn(); k_addr(buf1); v_addr(buf); }, [&](int i) { copy(own + NB - 1, nbuf, i); });
        pg_next = page_of(own + NB);
        settle(sn, mx, (kb << 6) + 32, pa);
        mx = half_step(I0{}, I0{}, I1{}, I1{}, sn, sc, pb, pa, [&]() {}, [&](int) {});
      } else {
        turn();
#pragma unroll
        for (int i = 0; i < FPW; ++i) copy(own + NB - 1, nbuf, i);
        pg_next = page_of(own + NB);
      }
      buf = buf1;
    }
    __builtin_amdgcn_s_waitcnt(DL_VMCNT(0));   // the trailing repeats must not outlive the workgroup
    if (active) {
#pragma unroll
      for (int d = 0; d < DT; ++d) v1[d] = rd(va[3] + d * 4096);
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int d = 0; d < DT; ++d) {
          oacc[d] = mm(x ? v1[d] : v0[d], pb.hi[x], oacc[d]);
          oacc[d] = mm(x ? v1[d] : v0[d], pb.lo[x], oacc[d]);
        }
    }
  }

  if (active) {
    // lane holds query column r, channels 32d + 8(e/4) + 4h + e%4
    float l = l_run + l_odd;
    l += __shfl_xor(l, 32, 64);
    if (row_out < 0) {
    } else if (a.n_units == 1) {
      const float inv = l > 0.f ? 1.0f / l : 0.f;
      const int tok = (int)(row_out / a.Hq), head = (int)(row_out - (int64_t)tok * a.Hq);
#pragma unroll
      for (int d = 0; d < DT; ++d)
#pragma unroll
        for (int e4 = 0; e4 < 4; ++e4) {
          const int ch = d * 32 + e4 * 8 + 4 * h;
          const int64_t at = a.out_mt > 0 ? frag_offset(tok, head * DH + ch, a.out_mt) : row_out * DH + ch;
          *(uint2*)(a.o + at) = make_uint2(pack_bf16x2(oacc[d][e4 * 4] * inv, oacc[d][e4 * 4 + 1] * inv),
                                           pack_bf16x2(oacc[d][e4 * 4 + 2] * inv, oacc[d][e4 * 4 + 3] * inv));
        }
    } else {
      const int64_t slot = row_out * a.n_units + unit;
      float* po = a.part_o + slot * DH + 4 * h;
#pragma unroll
      for (int d = 0; d < DT; ++d)
#pragma unroll
        for (int e4 = 0; e4 < 4; ++e4)
          *(f32x4*)(po + d * 32 + e4 * 8) = f32x4{oacc[d][e4 * 4], oacc[d][e4 * 4 + 1], oacc[d][e4 * 4 + 2], oacc[d][e4 * 4 + 3]};
      if (h == 0) { a.part_ml[slot * 2] = m_run; a.part_ml[slot * 2 + 1] = l; }
    }
  }
  if (bad) atomicOr(a.status, DLLM_STATUS_BAD_PAGE);
}

// (a kernel of its own around the body: as a kernel's own code it leaves the host without the launch stub)
template <int DH, int PG>
__global__ __launch_bounds__(512) void k_attn_dl(const AttnArgs a) { attn_dl_body<DH, PG>(a); }

bool attn_step_supported(const dllm_ctx* c, const StepGeom& g) {
  const dllm_config& f = c->cfg;
  if (!(f.dtype == DLLM_BF16 && c->kernel_mode == 0 && c->map.attn_rows > 0)) return false;
  return g.Q > 0 ? f.page_tokens % 8 == 0 : true;
}

// Attention of a denoise step (paged pool) or of a no-cache forward (packed scratch).
// merging four waves' partial results takes a little more LDS than a kernel gets by default
static bool attn_merge_ready = false;
hipError_t init_attn_kernels() {
  if (attn_merge_ready) return hipSuccess;
  hipError_t e = hipFuncSetAttribute((const void*)k_attn_step<128, 2, 2>, hipFuncAttributeMaxDynamicSharedMemorySize, 80 * 1024);
  if (e == hipSuccess) e = hipFuncSetAttribute((const void*)k_attn_step<64, 2, 2>, hipFuncAttributeMaxDynamicSharedMemorySize, 80 * 1024);
#define DL_ATTR(DHV, PG)                                                                                          \
  if (e == hipSuccess)                                                                                            \
    e = hipFuncSetAttribute((const void*)k_attn_dl<DHV, PG>, hipFuncAttributeMaxDynamicSharedMemorySize, DL_LDS_MAX)
  DL_ATTR(128, 0); DL_ATTR(128, 1); DL_ATTR(128, 2); DL_ATTR(64, 0); DL_ATTR(64, 1); DL_ATTR(64, 2);
#undef DL_ATTR
  attn_merge_ready = e == hipSuccess;
  return e;
}

hipError_t launch_attn_step(dllm_ctx* c, hipStream_t s, const StepGeom& g, const KVView& kv, bool frag_out) {
  const dllm_config& f = c->cfg;
  const AttnPlan p = attn_plan(device_cus(), f.head_dim, f.n_q_heads, f.n_kv_heads, g.B, g.Q, g.T, g.max_kv, f.page_tokens, c->map.attn_rows, attn_merge_ready);
  constexpr int QT = 2;
  AttnArgs a;
  a.q = WSM(c, q, bf16_t);
  a.prefix_len = g.prefix_len;
  a.q_valid = g.Q > 0 ? g.q_valid : nullptr;
  a.cu = g.cu_seqlens;
  a.o = WSM(c, o, bf16_t);
  a.out_mt = frag_out ? (g.T + 15) / 16 : 0;
  a.kv = kv;
  a.Q = g.Q; a.Hq = f.n_q_heads; a.Hkv = f.n_kv_heads; a.B = g.B;
  a.n_units = p.units; a.kspl = p.kspl; a.n_rg_wg = p.n_rg_wg;
  a.n_parts = p.units / p.kspl;
  a.pt_shift = p.pt_shift;
  a.pg_cap = p.pg_cap;
  a.scale_log2 = 1.4426950408889634f / sqrtf((float)f.head_dim);
  a.part_o = WSM(c, attn_part, float);
  a.part_ml = a.part_o + (size_t)c->map.attn_rows * f.head_dim;
  a.status = WSM(c, status, int32_t);
  dim3 grid((unsigned)a.n_parts, p.n_chunks, g.B * f.n_kv_heads);
  const int threads = 64 * p.n_rg_wg * p.kspl;
  if (p.staged) {
    const int pg = g.Q == 0 ? 0 : (p.pt_shift >= 6 ? 1 : 2);
#define ATTN_DL(DHV)                                                            \
  do {                                                                          \
    if (pg == 0) k_attn_dl<DHV, 0><<<grid, 512, p.lds, s>>>(a);                 \
    else if (pg == 1) k_attn_dl<DHV, 1><<<grid, 512, p.lds, s>>>(a);            \
    else k_attn_dl<DHV, 2><<<grid, 512, p.lds, s>>>(a);                         \
  } while (0)
    if (f.head_dim == 128) ATTN_DL(128);
    else ATTN_DL(64);
#undef ATTN_DL
  } else {
    if (f.head_dim == 64) k_attn_step<64, QT, 2><<<grid, threads, p.lds, s>>>(a);
    else if (p.n_rg_wg > 1 && (g.max_kv + 31) / 32 >= 16 * p.units) k_attn_step<128, QT, 1><<<grid, threads, p.lds, s>>>(a);
    else k_attn_step<128, QT, 2><<<grid, threads, p.lds, s>>>(a);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || a.n_parts == 1) return e;
  const int rows = g.T * f.n_q_heads;
  if (a.n_parts == 2 && rows >= 4096) {
    if (f.head_dim == 128) k_attn_combine2<128><<<(rows + 7) / 8, 256, 0, s>>>(a.part_o, a.part_ml, a.o, f.n_q_heads, a.out_mt, rows);
    else k_attn_combine2<64><<<(rows + 15) / 16, 256, 0, s>>>(a.part_o, a.part_ml, a.o, f.n_q_heads, a.out_mt, rows);
    return hipGetLastError();
  }
  if (f.head_dim == 128)
    k_attn_combine<128><<<(rows + 3) / 4, 512, 0, s>>>(a.part_o, a.part_ml, a.n_parts, a.o, f.n_q_heads, a.out_mt, rows);
  else
    k_attn_combine<64><<<(rows + 7) / 8, 512, 0, s>>>(a.part_o, a.part_ml, a.n_parts, a.o, f.n_q_heads, a.out_mt, rows);
  return hipGetLastError();
}

}  // namespace dllm

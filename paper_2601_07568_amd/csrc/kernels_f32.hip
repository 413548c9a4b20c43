// float kernels on the matrix cores for the denoise steps of at most 64 rows of a DLLM_F32 model.
//
// Such a step is bound by latency, not by bytes or products (the two-layer 256-wide model reads 11 MB): what counts is
// the number of launches and of dependent memory round trips in each.  So a product is cut into many small workgroups
// (16 weight rows, or a few such tiles, for the whole of K), the eight waves of a workgroup split K, every lane
// requests all its 16-byte pieces before the first product, and the epilogues carry what otherwise is a launch: row
// factor of the RMSNorm, rotary embedding and K/V write, SiLU*up, residual add with the next norm's sums of squares,
// the softmax statistics of the LM head.  The products are v_mfma_f32_16x16x4_f32: float operands, float sums.
//
// Operand layout of that instruction (lane l, c = l % 16, g = l / 16): A holds row c, k-element g; B column c, k-element
// g; D column c, rows 4g..4g+3.  A lane loads four consecutive k-elements of its row and feeds them to four
// instructions (the k-order is the same for both operands), so a step is 16 k-elements.  Weights are the A operand.
#include "mfma_common.h"

namespace dllm {

enum S32Epi { S32_STORE = 1, S32_QKV = 2, S32_SWIGLU = 3, S32_LMSTATS = 4, S32_RESID = 5 };

struct S32Args {
  const float* X;           // activations [M, K] row-major
  const float* gain;        // optional [K]: the product's input is X * gain, scaled per row by the factor from ss_in
  int M, K;
  const float *W0, *W1, *W2;   // main weight / Wq / W_gate / lm_head;  Wk / W_up;  Wv      ([out, in] row-major)
  int N0, N1, N2;
  float* out;               // STORE: [M, N0];  QKV: q [M, N0];  SWIGLU: h [M, N0]
  int dh, n_q_wg, n_k_wg;   // QKV: head_dim, 16-pair tiles covering q, k
  const float *rope_cos, *rope_sin;
  const int32_t *tok_seq, *tok_pos;
  float *pool_k, *pool_v;
  KVView pool;
  int32_t* status;
  const float* ss_in;       // partial sums of squares of the rows of X: ss_in[row * ss_stride + p], p < n_ss
  int n_ss, ss_stride;
  float inv_d, eps;
  float* x;                 // RESID: residual stream [M, N0], in/out
  float* ss_out;            // RESID: the rows' sums of squares over the workgroup's 16 columns
  float* part;              // LMSTATS: [rows, n_parts, 4]
  int n_parts;
  int32_t mask_id;
  const int32_t* n_lm_rows; // LMSTATS: optional device count, nothing is computed if it is zero
};

constexpr int S32_NW = 8;

__device__ inline f32x4 mfma4(float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

template <int NT, int MT, int EPI>
__global__ __launch_bounds__(S32_NW * 64) void k_s32(const S32Args a) {
  constexpr int NW = S32_NW;
  constexpr int UN = NT + MT <= 4 ? 4 : 2;                 // steps a wave requests together
  constexpr int RPW = MT * 16 / NW;                        // rows per wave when the row factors are summed
  __shared__ float red[NW][NT][MT][4][64];
  __shared__ float rs[MT * 16];
  __shared__ float aux[EPI == S32_LMSTATS ? MT * 4 * 16 * 4 : (EPI == S32_RESID ? MT * 4 * 64 : 1)];
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c = lane & 15, g = lane >> 4;
  const int wg = blockIdx.x, K = a.K, M = a.M, t0 = blockIdx.y * MT * 16;   // t0: the workgroup's first row
  if (EPI == S32_LMSTATS && a.n_lm_rows && *a.n_lm_rows <= 0) return;

  // the tiles' first weight rows
  const float* wb[NT];
  int row0[NT], nrows[NT];
  if constexpr (EPI == S32_QKV) {
    // tiles 0 and 1 are the two halves of rotary pair-tile wg (rows h*dh + j0 .. and the same + dh/2) of Wq or Wk,
    // tile 2 is 16-row tile wg of Wv
    const int half = a.dh >> 1, per_head = half / 16, n_pairs = a.n_q_wg + a.n_k_wg;
    const int pw = wg < n_pairs ? wg : n_pairs - 1;        // clamped: the result is dropped
    const bool isq = pw < a.n_q_wg;
    const int lw = isq ? pw : pw - a.n_q_wg, h = lw / per_head, j0 = (lw - h * per_head) * 16;
#pragma unroll
    for (int t = 0; t < 2; ++t) { wb[t] = isq ? a.W0 : a.W1; nrows[t] = isq ? a.N0 : a.N1; row0[t] = h * a.dh + j0 + t * half; }
    wb[NT - 1] = a.W2; nrows[NT - 1] = a.N2; row0[NT - 1] = wg * 16;
  } else if constexpr (EPI == S32_SWIGLU) {
#pragma unroll
    for (int t = 0; t < NT; ++t) { wb[t] = t ? a.W1 : a.W0; nrows[t] = a.N0; row0[t] = wg * 16; }
  } else {
#pragma unroll
    for (int t = 0; t < NT; ++t) { wb[t] = a.W0; nrows[t] = a.N0; row0[t] = (wg * NT + t) * 16; }
  }
  const float* wp[NT];
  const float* xp[MT];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    int r = row0[t] + c; r = r < nrows[t] ? r : nrows[t] - 1;           // rows past the matrix: dropped in the epilogue
    wp[t] = wb[t] + (int64_t)r * K + g * 4;
  }
#pragma unroll
  for (int m = 0; m < MT; ++m) {
    int r = t0 + m * 16 + c; r = r < M ? r : M - 1;
    xp[m] = a.X + (int64_t)r * K + g * 4;
  }
  const float* gp = a.gain ? a.gain + g * 4 : nullptr;

  // what the epilogue item of this thread needs besides the sums is requested now
  float xres = 0.f, pcs = 0.f, psn = 0.f;
  int ppos = -1, ppage = -1;
  {
    const int m = tid >> 8, iq = (tid >> 6) & 3, tok = t0 + m * 16 + c;
    if (EPI == S32_RESID) {
      const int n = row0[0] + 4 * g + iq;
      xres = a.x[m < MT && tok < M && n < a.N0 ? (int64_t)tok * a.N0 + n : 0];
    }
    if (EPI == S32_QKV && m < MT && tok < M) {
      ppos = a.tok_pos[tok];
      if (wg < a.n_q_wg + a.n_k_wg) {
        const int hj = row0[0] + 4 * g + iq, j = hj - (hj / a.dh) * a.dh, half = a.dh >> 1;
        pcs = a.rope_cos[(int64_t)tok * half + j];
        psn = a.rope_sin[(int64_t)tok * half + j];
      }
      const int pi = ppos >= 0 ? ppos / a.pool.page_tokens : a.pool.max_pages;
      if (pi < a.pool.max_pages) ppage = a.pool.table[(int64_t)a.tok_seq[tok] * a.pool.max_pages + pi];
    }
  }

  f32x4 acc[NT][MT];
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int m = 0; m < MT; ++m) acc[t][m] = f32x4{0.f, 0.f, 0.f, 0.f};
  // Row factors: this wave's rows.  The first 64 partials of every row are requested before anything else and added up
  // (in a fixed tree, the rows' chains side by side) while the operands are on their way.
  float ssv[RPW];
  if (a.ss_in) {
#pragma unroll
    for (int q = 0; q < RPW; ++q) {
      const int row = t0 + w * RPW + q < M ? t0 + w * RPW + q : M - 1;
      const float v = a.ss_in[(int64_t)row * a.ss_stride + (lane < a.n_ss ? lane : a.n_ss - 1)];
      ssv[q] = lane < a.n_ss ? v : 0.f;
    }
  }
  auto row_factors = [&]() {
    if (!a.ss_in) return;
    if (a.n_ss > 64) {
#pragma unroll
      for (int q = 0; q < RPW; ++q)
        for (int p = 64 + lane; p < a.n_ss; p += 64)
          ssv[q] += a.ss_in[(int64_t)(t0 + w * RPW + q < M ? t0 + w * RPW + q : M - 1) * a.ss_stride + p];
    }
#pragma unroll
    for (int o = 1; o < 64; o <<= 1)
#pragma unroll
      for (int q = 0; q < RPW; ++q) ssv[q] += __shfl_xor(ssv[q], o, 64);
    if (lane == 0) {
#pragma unroll
      for (int q = 0; q < RPW; ++q) rs[w * RPW + q] = 1.0f / sqrtf(ssv[q] * a.inv_d + a.eps);
    }
  };
  const int n_steps = (K + 15) / 16;
  bool first = true;
  for (int s0 = w; s0 < n_steps; s0 += NW * UN) {
    f32x4 fw[UN][NT], fx[UN][MT], fg[UN];
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      const int k = (s0 + u * NW) * 16;
      const bool ok = k + g * 4 + 4 <= K;                  // K % 4 == 0
      const int kk = ok ? k : 0;
      const f32x4 z = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int t = 0; t < NT; ++t) { const f32x4 v = *(const f32x4*)(wp[t] + (ok ? kk : -g * 4)); fw[u][t] = ok ? v : z; }
#pragma unroll
      for (int m = 0; m < MT; ++m) { const f32x4 v = *(const f32x4*)(xp[m] + (ok ? kk : -g * 4)); fx[u][m] = ok ? v : z; }
      fg[u] = f32x4{1.f, 1.f, 1.f, 1.f};
      if (gp) fg[u] = *(const f32x4*)(gp + (ok ? kk : -g * 4));
    }
    if (first) { first = false; row_factors(); }
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      if (s0 + u * NW >= n_steps) break;                   // (a product of zeros takes as long as another)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int m = 0; m < MT; ++m) {
          const float b = fx[u][m][e] * fg[u][e];
#pragma unroll
          for (int t = 0; t < NT; ++t) acc[t][m] = mfma4(fw[u][t][e], b, acc[t][m]);
        }
    }
  }
  if (first) row_factors();                                // a wave without a step of its own still sums its rows
  // sum the waves' partial tiles in wave order
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int i = 0; i < 4; ++i) red[w][t][m][i][lane] = acc[t][m][i];
  __syncthreads();

  for (int item = tid; item < MT * 256; item += NW * 64) {
    const int m = item >> 8, i = (item >> 6) & 3, ln = item & 63;
    const int tok = t0 + m * 16 + (ln & 15), fr = 4 * (ln >> 4) + i;     // row inside the 16-row tile
    const bool tok_ok = tok < M;
    float val[NT];
    const float rsc = a.ss_in ? rs[tok - t0] : 1.0f;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      float s = 0.f;
#pragma unroll
      for (int ww = 0; ww < NW; ++ww) s += red[ww][t][m][i][ln];
      val[t] = s * rsc;
    }
    if constexpr (EPI == S32_STORE) {
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const int n = row0[t] + fr;
        if (tok_ok && n < a.N0) a.out[(int64_t)tok * a.N0 + n] = val[t];
      }
    } else if constexpr (EPI == S32_SWIGLU) {
      const int n = row0[0] + fr;
      if (tok_ok && n < a.N0) a.out[(int64_t)tok * a.N0 + n] = val[0] / (1.0f + expf(-val[0])) * val[1];
    } else if constexpr (EPI == S32_RESID) {
      const int n = row0[0] + fr;
      float sq = 0.f;
      if (tok_ok && n < a.N0) {
        const float v = (item == tid ? xres : a.x[(int64_t)tok * a.N0 + n]) + val[0];
        a.x[(int64_t)tok * a.N0 + n] = v;
        sq = v * v;
      }
      aux[(m * 4 + i) * 64 + ln] = sq;
    } else if constexpr (EPI == S32_QKV) {
      if (!tok_ok) continue;
      const bool pre = item == tid;                        // fetched above
      const int pos = pre ? ppos : a.tok_pos[tok];
      int64_t ko = 0, vo = 0;
      int vs = 0;
      auto locate = [&](int h) -> bool {
        if (!pre) return kv_locate(a.pool, a.tok_seq[tok], pos, h, ko, vo, vs);
        if (ppage < 0 || ppage >= a.pool.n_pages) return false;
        const int slot = pos - (pos / a.pool.page_tokens) * a.pool.page_tokens;
        const int64_t ph = (int64_t)ppage * a.pool.n_kv_heads + h;
        ko = (ph * a.pool.page_tokens + slot) * a.pool.head_dim;
        vo = ph * a.pool.head_dim * a.pool.page_tokens + slot;
        vs = a.pool.page_tokens;
        return true;
      };
      if (wg < a.n_q_wg + a.n_k_wg) {
        const bool isq = wg < a.n_q_wg;
        const int half = a.dh >> 1, hj = row0[0] + fr, h = hj / a.dh, j = hj - h * a.dh;
        const float cs = pre ? pcs : a.rope_cos[(int64_t)tok * half + j], sn = pre ? psn : a.rope_sin[(int64_t)tok * half + j];
        const float r0 = val[0] * cs - val[1] * sn, r1 = val[1] * cs + val[0] * sn;
        if (isq) {
          a.out[(int64_t)tok * a.N0 + hj] = r0;
          a.out[(int64_t)tok * a.N0 + hj + half] = r1;
        } else if (pos >= 0) {                             // (a padding row: nothing of it is cached)
          if (locate(h)) { a.pool_k[ko + j] = r0; a.pool_k[ko + j + half] = r1; }
          else atomicOr(a.status, DLLM_STATUS_BAD_PAGE);
        }
      }
      const int n = row0[NT - 1] + fr;                     // value row
      if (n < a.N2 && pos >= 0) {
        const int h = n / a.dh, ch = n - h * a.dh;
        if (locate(h)) a.pool_v[vo + (int64_t)ch * vs] = val[NT - 1];
      }
    } else if constexpr (EPI == S32_LMSTATS) {
      RowStat st;
      st.init();
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const int n = row0[t] + fr;
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
        float* p = aux + ((m * 4 + i) * 16 + (ln & 15)) * 4;
        p[0] = st.m; p[1] = __int_as_float(st.idx); p[2] = st.s; p[3] = st.t;
      }
    }
  }
  if constexpr (EPI == S32_RESID) {
    __syncthreads();
    if (tid < MT * 16) {          // the 16 contributions of a row (4 values of i x 4 lane groups) in a fixed order
      const int m = tid >> 4, cc = tid & 15;
      float sq = 0.f;
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int lg = 0; lg < 4; ++lg) sq += aux[(m * 4 + i) * 64 + lg * 16 + cc];
      a.ss_out[(int64_t)(t0 + tid) * a.ss_stride + wg] = sq;
    }
  }
  if constexpr (EPI == S32_LMSTATS) {
    __syncthreads();
    if (tid < MT * 16 && t0 + tid < M) {
      const int m = tid >> 4, cc = tid & 15;
      RowStat st;
      st.init();
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float* p = aux + ((m * 4 + i) * 16 + cc) * 4;
        st.merge(p[0], __float_as_int(p[1]), p[2], p[3]);
      }
      *(f32x4*)(a.part + ((int64_t)(t0 + tid) * a.n_parts + wg) * 4) = f32x4{st.m, __int_as_float(st.idx), st.s, st.t};
    }
  }
}

// Where the weight tiles leave CUs idle every 16 rows get a workgroup of their own: a step of the 256-wide model is 64 weight
// tiles at most, and their products, sums and epilogues are as long as their rows are many (the float products of a CU's matrix
// cores run one after the other: 64 x 32 outputs of K = 256 take 1.7 us).  32 rows, together / apart, us: residual 6.3 / 4.5, gate/up
// 8.7 / 6.2, q/k/v 8.4 / 7.7, LM head 10.9 / 8.6.
template <int NT, int EPI>
static hipError_t s32_launch(hipStream_t s, const S32Args& a, int grid) {
  const int row_tiles = (a.M + 15) / 16;
  if (row_tiles > 1 && grid * row_tiles <= device_cus()) {
    k_s32<NT, 1, EPI><<<dim3(grid, row_tiles), S32_NW * 64, 0, s>>>(a);
    return hipGetLastError();
  }
  switch ((a.M + 15) / 16) {
    case 1: k_s32<NT, 1, EPI><<<grid, S32_NW * 64, 0, s>>>(a); break;
    case 2: k_s32<NT, 2, EPI><<<grid, S32_NW * 64, 0, s>>>(a); break;
    case 3: k_s32<NT, 3, EPI><<<grid, S32_NW * 64, 0, s>>>(a); break;
    case 4: k_s32<NT, 4, EPI><<<grid, S32_NW * 64, 0, s>>>(a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------
// Attention of a step over the paged pool: one workgroup of eight waves per (sequence, query head, 16 query rows); the
// waves take the 16-key tiles of the sequence in turn and merge their results in LDS, in wave order.  S^T = K Q^T
// leaves lane group g the scores of keys 4g..4g+3 of the lane's query, which is the B operand of O^T = V^T P^T; V is
// stored with the keys of a channel contiguous, so both operands are 16-byte loads (pages are multiples of 4 tokens).
// The tiles and their order depend on the sequence alone: a sequence's results do not change with the batch it is in.
template <int DH>
__global__ __launch_bounds__(512) void k_s32_attn(const float* q, float* o, const int32_t* prefix_len, const int32_t* q_valid,
                                                  KVView kv, int Q, int Hq, float scale, int32_t* status) {
  constexpr int KK = DH / 16, DT = DH / 16, NW = 8;
  __shared__ float sm_m[NW][16], sm_l[NW][16];
  __shared__ f32x4 sm_o[NW][DT][64];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, c = lane & 15, g = lane >> 4;
  const int b = blockIdx.z, h = blockIdx.y, r0 = blockIdx.x * 16;
  if (q_valid && q_valid[b] < 0) return;                   // the sequence is not part of this call
  const int kv_len = prefix_len[b] + (q_valid ? min(max(q_valid[b], 0), Q) : Q);
  const int kvh = h / (Hq / kv.n_kv_heads);
  const float* kbase = (const float*)kv.k;
  const float* vbase = (const float*)kv.v;
  const int pt = kv.page_tokens;
  const int32_t* table = kv.table + (int64_t)b * kv.max_pages;
  const int row = r0 + c < Q ? r0 + c : Q - 1;
  f32x4 qf[KK];
  const float* qp = q + ((int64_t)(b * Q + row) * Hq + h) * DH + g * 4;
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) qf[kk] = *(const f32x4*)(qp + kk * 16);
  f32x4 oacc[DT];
#pragma unroll
  for (int d = 0; d < DT; ++d) oacc[d] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m_run = -DEV_INF, l_run = 0.f;
  bool bad = false;
  const int n_tiles = (kv_len + 15) / 16;
  auto page_of = [&](int key) -> int {
    const int pi = key / pt;
    return pi < kv.max_pages ? table[pi] : -1;
  };
  for (int tile = w; tile < n_tiles; tile += NW) {
    // K: lane's key is c of the tile; V: keys 4g .. 4g+3 (inside one page)
    const int kkey = tile * 16 + c, kc = kkey < kv_len ? kkey : kv_len - 1;
    const int vkey = tile * 16 + 4 * g, vc = vkey < kv_len ? vkey : (kv_len - 1) & ~3;
    const int kpg = page_of(kc), vpg = page_of(vc);
    const bool kok = (uint32_t)kpg < (uint32_t)kv.n_pages, vok = (uint32_t)vpg < (uint32_t)kv.n_pages;
    bad |= !kok || !vok;
    const float* kp = kbase + (((int64_t)(kok ? kpg : 0) * kv.n_kv_heads + kvh) * pt + (kc - kc / pt * pt)) * DH + g * 4;
    const float* vp = vbase + (((int64_t)(vok ? vpg : 0) * kv.n_kv_heads + kvh) * DH + c) * pt + (vc - vc / pt * pt);
    f32x4 kf[KK], vf[DT];
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) kf[kk] = *(const f32x4*)(kp + kk * 16);
#pragma unroll
    for (int d = 0; d < DT; ++d) vf[d] = *(const f32x4*)(vp + (int64_t)d * 16 * pt);
    f32x4 s = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kk = 0; kk < KK; ++kk)
#pragma unroll
      for (int e = 0; e < 4; ++e) s = mfma4(kf[kk][e], qf[kk][e], s);
    // scores of keys 4g + i: -inf where the key is past the sequence or its page is not addressable
    const unsigned long long kbad = __builtin_amdgcn_ballot_w64(!kok);
    float mx = -DEV_INF;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      s[i] *= scale;
      if (tile * 16 + 4 * g + i >= kv_len || ((kbad >> (4 * g + i)) & 1)) s[i] = -DEV_INF;
      mx = fmaxf(mx, s[i]);
    }
#pragma unroll
    for (int d = 0; d < DT; ++d)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (!vok || vkey + e >= kv_len) vf[d][e] = 0.f;    // such slots may hold anything, and 0 * NaN is NaN
    mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    const float m_new = fmaxf(m_run, mx);
    const float alpha = m_run == -DEV_INF ? 0.f : expf(m_run - m_new);
    l_run *= alpha;
    float p[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      p[i] = s[i] == -DEV_INF ? 0.f : expf(s[i] - m_new);
      l_run += p[i];
    }
#pragma unroll
    for (int d = 0; d < DT; ++d) {
      oacc[d] = oacc[d] * alpha;
#pragma unroll
      for (int i = 0; i < 4; ++i) oacc[d] = mfma4(vf[d][i], p[i], oacc[d]);
    }
    m_run = m_new;
  }
  l_run += __shfl_xor(l_run, 16, 64);
  l_run += __shfl_xor(l_run, 32, 64);
  if (g == 0) { sm_m[w][c] = m_run; sm_l[w][c] = l_run; }
  __syncthreads();
  float m_all = -DEV_INF, l_all = 0.f;
#pragma unroll
  for (int ww = 0; ww < NW; ++ww) m_all = fmaxf(m_all, sm_m[ww][c]);
#pragma unroll
  for (int ww = 0; ww < NW; ++ww) l_all += sm_m[ww][c] > -DEV_INF ? sm_l[ww][c] * expf(sm_m[ww][c] - m_all) : 0.f;
  const float f = m_run > -DEV_INF ? expf(m_run - m_all) : 0.f;
#pragma unroll
  for (int d = 0; d < DT; ++d) sm_o[w][d][lane] = oacc[d] * f;
  __syncthreads();
  for (int d = w; d < DT; d += NW) {
    f32x4 v = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ww = 0; ww < NW; ++ww) v = v + sm_o[ww][d][lane];
    const float inv = l_all > 0.f ? 1.0f / l_all : 0.f;
    if (r0 + c < Q) *(f32x4*)(o + ((int64_t)(b * Q + r0 + c) * Hq + h) * DH + d * 16 + 4 * g) = v * inv;
  }
  if (bad) atomicOr(status, DLLM_STATUS_BAD_PAGE);
}

// ------------------------------------------------------------------------------------------
// float models, steps of at most 64 rows; everything the kernels load 16 bytes at a time is aligned for it.  No bound on the
// prefix or the width: against the generic kernels a step of two layers and a head takes 0.04 .. 0.19 of the time for 1 ..
// 64 rows, prefixes of 64 .. 8192 and 256 .. 4096 channels (us, 32 rows: 256 channels 801 / 95 at prefix 64, 2085 / 391 at 8192;
// 4096 channels 11647 / 837 and 24153 / 1795).
bool s32_supported(const dllm_ctx* c, const StepGeom& g) {
  const dllm_config& f = c->cfg;
  return f.dtype == DLLM_F32 && c->kernel_mode == 0 && c->f32_aligned && g.Q > 0 && g.T <= SK_MAX_ROWS && f.d_model % 4 == 0 &&
         f.d_ff % 4 == 0 && f.page_tokens % 4 == 0;
}

static S32Args s32_base(dllm_ctx* c, const float* X, int M, int K, const void* gain, int n_ss) {
  S32Args a;
  memset(&a, 0, sizeof(a));
  a.X = X; a.M = M; a.K = K;
  a.gain = (const float*)gain;
  if (gain) a.ss_in = WSM(c, ss, float);
  a.n_ss = n_ss;
  a.ss_stride = ss_row_stride(c);
  a.inv_d = 1.0f / (float)c->cfg.d_model;
  a.eps = c->cfg.rms_eps;
  return a;
}

hipError_t launch_s32_qkv(dllm_ctx* c, hipStream_t s, const StepGeom& g, int layer, const KVView& pool, int n_ss) {
  const dllm_config& f = c->cfg;
  const dllm_layer_w& L = c->layers[layer];
  S32Args a = s32_base(c, WSM(c, x, float), g.T, f.d_model, L.attn_norm, n_ss);
  a.W0 = (const float*)L.wq; a.W1 = (const float*)L.wk; a.W2 = (const float*)L.wv;
  a.N0 = f.n_q_heads * f.head_dim; a.N1 = a.N2 = f.n_kv_heads * f.head_dim;
  a.out = WSM(c, q, float);
  a.dh = f.head_dim;
  a.n_q_wg = f.n_q_heads * (f.head_dim / 32);
  a.n_k_wg = f.n_kv_heads * (f.head_dim / 32);
  a.rope_cos = WSM(c, rope_cos, float); a.rope_sin = WSM(c, rope_sin, float);
  a.tok_seq = WSM(c, tok_seq, int32_t); a.tok_pos = WSM(c, tok_pos, int32_t);
  a.pool_k = (float*)pool.k; a.pool_v = (float*)pool.v; a.pool = pool;
  a.status = WSM(c, status, int32_t);
  const int n_pairs = a.n_q_wg + a.n_k_wg, n_vt = (a.N2 + 15) / 16;
  return s32_launch<3, S32_QKV>(s, a, n_pairs > n_vt ? n_pairs : n_vt);
}

hipError_t launch_s32_attn(dllm_ctx* c, hipStream_t s, const StepGeom& g, const KVView& kv) {
  const dllm_config& f = c->cfg;
  const dim3 grid((g.Q + 15) / 16, f.n_q_heads, g.B);
  const float scale = 1.0f / sqrtf((float)f.head_dim);
  if (f.head_dim == 128)
    k_s32_attn<128><<<grid, 512, 0, s>>>(WSM(c, q, float), WSM(c, o, float), g.prefix_len, g.q_valid, kv, g.Q, f.n_q_heads, scale,
                                         WSM(c, status, int32_t));
  else
    k_s32_attn<64><<<grid, 512, 0, s>>>(WSM(c, q, float), WSM(c, o, float), g.prefix_len, g.q_valid, kv, g.Q, f.n_q_heads, scale,
                                        WSM(c, status, int32_t));
  return hipGetLastError();
}

// x += A W^T, and the rows' sums of squares for the next norm
hipError_t launch_s32_resid(dllm_ctx* c, hipStream_t s, const float* A, const void* W, int M, int K) {
  S32Args a = s32_base(c, A, M, K, nullptr, 0);
  a.W0 = (const float*)W; a.N0 = c->cfg.d_model;
  a.x = WSM(c, x, float);
  a.ss_out = WSM(c, ss, float);
  return s32_launch<1, S32_RESID>(s, a, (a.N0 + 15) / 16);
}

hipError_t launch_s32_swiglu(dllm_ctx* c, hipStream_t s, int layer, int M, int n_ss) {
  const dllm_layer_w& L = c->layers[layer];
  S32Args a = s32_base(c, WSM(c, x, float), M, c->cfg.d_model, L.mlp_norm, n_ss);
  a.W0 = (const float*)L.w_gate; a.W1 = (const float*)L.w_up; a.N0 = c->cfg.d_ff;
  a.out = WSM(c, h, float);
  return s32_launch<2, S32_SWIGLU>(s, a, (a.N0 + 15) / 16);
}

hipError_t launch_s32_logits(dllm_ctx* c, hipStream_t s, float* out, int M, int n_ss) {
  S32Args a = s32_base(c, WSM(c, x, float), M, c->cfg.d_model, c->final_norm, n_ss);
  a.W0 = (const float*)c->lm_head; a.N0 = c->cfg.vocab;
  a.out = out;
  return s32_launch<4, S32_STORE>(s, a, (a.N0 + 63) / 64);
}

// every row's softmax statistics per 64 columns; the merge picks the masked rows
hipError_t launch_s32_lmstats(dllm_ctx* c, hipStream_t s, int M, int n_ss, int* n_parts_out) {
  S32Args a = s32_base(c, WSM(c, x, float), M, c->cfg.d_model, c->final_norm, n_ss);
  a.W0 = (const float*)c->lm_head; a.N0 = c->cfg.vocab;
  a.part = WSM(c, lm_part, float);
  a.n_parts = (c->cfg.vocab + 63) / 64;
  a.mask_id = c->cfg.mask_id;
  a.n_lm_rows = WSM(c, status, int32_t) + 1;
  *n_parts_out = a.n_parts;
  return s32_launch<4, S32_LMSTATS>(s, a, a.n_parts);
}

}  // namespace dllm

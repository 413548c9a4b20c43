// Which form of a kernel a call gets, by its sizes: host code without a device, apart from the launches so that it can be
// checked (and asked) without a GPU.
#pragma once
#include <stddef.h>
#include <stdint.h>

namespace dllm {

// ---- attention
constexpr int ATTN_MAX_SPLITS = 64;
constexpr int DL_NB = 4;                        // staged kernel: buffers of its ring, 64 keys of K and of V^T each
constexpr int DL_LDS_MAX = 160 * 1024;          // ... ring plus page ids
struct AttnPlan {
  bool staged;              // k_attn_dl, else k_attn_step
  int n_rg_wg, n_chunks;    // row groups (32 query rows) of a workgroup, workgroups along them
  int units, kspl;          // along the keys; of a workgroup
  int pt_shift;             // log2(page_tokens) if that is a power of two of at least 8 (0: packed scratch), else -1
  int pg_cap;               // staged: page ids that a workgroup keeps in LDS
  size_t lds;
};
// Q: query rows of a sequence, 0: no-cache forward (max_kv: the longest sequence); T: rows of the call; part_rows: (token,
// head, unit) rows that the buffer of partial results holds; raised: the kernels may use more LDS than by default
inline AttnPlan attn_plan(int cus, int head_dim, int n_q_heads, int n_kv_heads, int B, int Q, int T, int max_kv, int page_tokens,
                          int64_t part_rows, bool raised) {
  AttnPlan p{};
  const int G = n_q_heads / n_kv_heads;
  const int max_q = Q > 0 ? Q : max_kv;                       // most query rows of a sequence
  constexpr int QT = 2;
  const int n_rg = (max_q * G + 16 * QT - 1) / (16 * QT);
  if (Q > 0) {
    p.pt_shift = -1;
    for (int sft = 3; sft < 31; ++sft) if (page_tokens == (1 << sft)) p.pt_shift = sft;
  }
  const int64_t by_space = part_rows / ((int64_t)T * n_q_heads);
  const int64_t most = by_space < 1 ? 1 : by_space > ATTN_MAX_SPLITS ? ATTN_MAX_SPLITS : by_space;   // (one unit needs no partials)
  // Many rows per KV head: K and V staged in LDS, up to 8 row groups per workgroup.  A workgroup keeps the page ids of its own
  // unit's blocks behind the ring: a sequence of more than fit is cut into that many units, if the partials' buffer allows.
  const size_t ring = (size_t)DL_NB * (head_dim / 4) * 1024;
  const int n_blk = (max_kv + 63) / 64, ids_blk = Q > 0 ? (page_tokens < 64 ? 64 / page_tokens : 1) : 0;
  const int64_t ids_fit = (int64_t)(DL_LDS_MAX - ring) / sizeof(int32_t);
  const int64_t least = ids_blk > 0 ? (n_blk + ids_fit / ids_blk - 1) / (ids_fit / ids_blk) : 1;
  p.staged = n_rg >= 4 && p.pt_shift >= 0 && raised && least <= most;
  const int nkb = (max_kv + 31) / 32;
  // Denoise steps whose row groups leave the CUs room: a workgroup per row group (they meet in the L2), and as many along the keys
  // as fill one round, each on a CU of its own, whose 32 KB of outstanding loads set the pace.  One wave alone up to eight blocks
  // each, or where the row groups fill the chip twice; else four waves, which merge their results in LDS (3 us).  One round and no
  // combine kernel where there are many sequences.  (All row groups of a key head in one workgroup, units of two blocks in up to
  // 512 workgroups / this, attention + combine, us, 32 key heads: one sequence of 512 keys 14.7 / 10.6, 1024 15.8 / 13.4, 4096 30.0 /
  // 25.5; 8 of 100 / 400 / 700 keys 18.3 / 11.8, 26.1 / 20.5, 33.7 / 25.3; 16 of 2048 118 / 96; 32 of 64 / 250 39.3 / 19.7, 44.9 / 34.9; 64
  // rows: one of 1237 23.0 / 20.6, of 5000 56.2 / 37.8, 4 of 1500 55.4 / 39.9, 8 of 1500 86.3 / 66.3.  Not where a second round would
  // hold a few workgroups of long sequences: 3 sequences of 2500 keys and 80 rows 78.9 / 90.4.)
  const int64_t groups = (int64_t)B * n_kv_heads * n_rg;
  const bool few_groups = groups <= cus || groups >= 2 * cus - cus / 4 || nkb <= 32;
  int64_t parts = cus / groups < 1 ? 1 : cus / groups;
  if (parts > (nkb + 1) / 2) parts = (nkb + 1) / 2;
  if (parts >= 8) parts = parts / 8 * 8;                       // row groups of the same keys behind the same L2
  if (parts > most) parts = most;
  // Grouped queries: the staged kernel where a wave would have more than six blocks (4 key heads of 7, 32 rows, staged / this: one
  // sequence of 600 keys 16.5 / 14.6, 2048 21.0 / 16.0, 4000 24.5 / 19.8, 8000 26.6 / 31.2; 2 of 1000 21.4 / 17.6, of 4000 27.3 / 27.9; 64
  // rows, 2048 keys 25.7 / 21.0), and always for up to four row groups (16 rows 15.9 / 15.8; 128 rows of a model with as many
  // key heads as heads 21.8 / 23.1, 39.6 / 43.4).
  if (p.staged && Q > 0 && G > 1 && n_rg > 4 && groups <= cus && nkb <= 24 * parts) p.staged = false;
  if (!p.staged && Q > 0 && raised && few_groups) {
    // Seven or eight blocks in all: four waves of one workgroup instead of one wave with all of them or two that need the combine
    // kernel, as long as the workgroups are one round (a layer of 256 channels, us, single waves / this, 190 .. 220 keys: 32 key heads, 4
    // sequences 54.4 / 53.7, 5 59.1 / 57.3, 8 62.9 / 61.2, but 10 78.0 / 78.7, 13 80.4 / 80.9; 16 key heads, 8 sequences 56.7 / 55.3, 16 60.8
    // / 59.2, but 20 64.3 / 64.9; heads of 64 channels, 32 key heads, 4 sequences 47.3 / 45.3, 8 53.0 / 51.5, 10 54.9 / 54.9).  Longer ones
    // have four waves by the rule below where a single wave would have more than eight blocks, the same launch; where there are two
    // parts of up to eight each, two single waves gain over one workgroup as often as they lose.  Pages that are no multiple of 32
    // tokens have longer chains per block: one sequence of 1000 keys in pages of 24 16.3 / 15.2.
    const bool narrow = groups < 2 * cus - cus / 4;
    const bool merge = groups <= cus && parts <= 2 && (nkb == 7 || nkb == 8);
    if (merge) parts = 1;
    const int64_t per_wave = (nkb + parts - 1) / parts;
    p.kspl = merge || (narrow && per_wave > (page_tokens % 32 == 0 ? 8 : 4)) ? 4 : 1;
    p.n_rg_wg = 1;
    p.n_chunks = n_rg;
    p.units = (int)(parts * p.kspl);
    if (p.kspl > 1) p.lds = (size_t)p.kspl * (2 * QT * 16 * sizeof(float) + (size_t)(head_dim / 16) * QT * 64 * 16);
    return p;
  }
  const int rg_cap = p.staged ? 8 : 4;                         // the register-direct kernel runs at most 4 waves
  p.n_rg_wg = n_rg < rg_cap ? n_rg : rg_cap;
  p.n_chunks = (n_rg + p.n_rg_wg - 1) / p.n_rg_wg;
  // units along the keys: short dependent chains matter more than partial traffic here (a step's
  // attention is a few MB), so give every unit about two 32-key blocks, within the partial buffer
  int64_t want = 2048 / ((int64_t)B * n_kv_heads * n_rg);
  if (want < 1) want = 1;
  int64_t by_work = p.staged ? (nkb + 7) / 8 : (nkb + 1) / 2;   // staged kernel: at least four 64-key blocks per unit ...
  if (p.staged && by_work > 1) {   // (a single unit needs no combine)
    // ... or two, or one, where that still leaves CUs without a workgroup (a layer of 256 channels, us, four / two / one: 4 key
    // heads of 7, 16 rows, 512 keys 32.7 / 31.7 / 31.6 in 12 / 20 / 36 workgroups, 1000 keys 33.9 / 31.6 / 31.9 in 16 / 32 / 64, 2048
    // keys 35.2 / 34.3 / 36.3 in 36 / 68 / 132, 4 sequences of 2048 50.5 / 57.0 / 58.2 in 144 / 272 / 528; 8 key heads of 4, 32 rows, 512 keys
    // 38.2 / 37.3 / 37.5, 1000 keys 40.0 / 39.1 / 40.6, 2048 keys 41.6 / 42.1 / 50.5; 128 rows of 32 key heads, 500 keys 60.7 / 59.0 /
    // 66.5, which keeps four for its 96 workgroups, 1000 keys 60.5 / 69.4 / 71.5)
    const int64_t per_unit = (int64_t)p.n_chunks * B * n_kv_heads;
    if ((nkb + 1) / 2 * per_unit <= 64) by_work = (nkb + 1) / 2;
    else if ((nkb + 3) / 4 * per_unit <= 128) by_work = (nkb + 3) / 4;
  }
  int64_t units = want < by_work ? want : by_work;
  if (p.staged && units < least) units = least;
  if (units > most) units = most;
  // One row group per KV head, more of them than CUs but not two rounds, and long sequences (the others have returned above): four units share a workgroup and merge their partial results in LDS, which leaves a
  // quarter of the partials to write and re-read, or none.  (A layer of 256 channels, us, units of single waves with their combine /
  // this, 32 key heads: 9 sequences of 1100 / 2000 keys 120.2 / 117.7, 147.4 / 144.4, 10 124.5 / 118.7, 154.4 / 146.7, 13 136.7 / 123.5,
  // 172.8 / 157.1; of 4000 keys 9 sequences 208.3 / 221.4, 10 221.7 / 225.5, 12 248.8 / 234.2.)
  p.kspl = 1;
  if (!p.staged && n_rg == 1 && raised && by_work >= 4) {
    p.kspl = 4;
    int64_t parts = (nkb + 2 * p.kspl - 1) / (2 * p.kspl);
    if (parts * p.kspl > want) parts = want / p.kspl;
    if (parts > by_space) parts = by_space;
    if (parts < 1) parts = 1;
    units = parts * p.kspl;
  }
  p.units = (int)units;
  if (p.staged) {
    p.pg_cap = (int)((n_blk + units - 1) / units) * ids_blk;
    p.lds = ring + (size_t)p.pg_cap * sizeof(int32_t);
  } else if (p.kspl > 1) {
    p.lds = (size_t)p.kspl * (2 * QT * 16 * sizeof(float) + (size_t)(head_dim / 16) * QT * 64 * 16);
  }
  return p;
}

// ---- products of more than 64 rows (k_gemm_tile)
// Up to this many real rows the column tiles start their sums apart, in groups of 256 columns (gate/up: of 1920 features, q/k/v
// with the rotary embedding: of 3840).
constexpr int GT_APART_ROWS = 256, GT_APART_COLS = 256, GT_APART_SWIGLU = 1920, GT_APART_ROPE = 3840;
// Column tiles of the call may start their sums apart: every tile has to lie inside one group.  Residual tiles of 224 weight rows
// (in groups of 1792, which they would fit, the other tiles take 0.2 .. 0.6 us more of 12 .. 50 at 72 .. 256 rows) and odd
// gate/up tiles that do not begin at column 0 do not.  device_rows: the rows there are come from the device, M bounds them
inline bool gt_starts_apart(int M, bool device_rows) { return M <= GT_APART_ROWS || device_rows; }

// Which tile (token rows x weight rows): the estimate counts rounds of one workgroup per CU in units of a 256 x 256 tile's time.
// A 128 x 256 tile costs 0.6 of it (half the products, three quarters of the bytes), a 128 x 128 one 0.33 (copies and products
// take equally long), a 128 x 64 one 0.22, a 256 x 160 one 0.80, a 256 x 96 one 0.54, a 128 x 160 one 0.45.  Measured against
// each other (K = 3584 .. 18944, us): 1024 x 37888: 271 / 286 / 297; 256 x 24576: 85 / 55 / 61; 128 x 24576: 85 / 50 / 39; 1024 x
// 3584 x 3584: 48 (4 K shares) / 38 (2) / 42.
// Over 200 layers of 128 .. 8192 channels and 96 .. 16384 rows, 257 .. 511 among them, what it picks takes 0.47 .. 0.98 of the
// time of the 32-deep kernels that were here before.
//
// Odd widths for gate/up: one round of one tile per CU decides there up to about 300 rows, and 128 and 256 columns
// seldom make one (256 CUs; 24576 gate and up rows: 256 tiles of 96, 37888: 237 of 160).  Measured in turn, what is taken
// without odd tiles / with them, us: 24576 x 4096: 66 rows 41.4 / 38.9 and 128 rows 48.0 / 43.3 (128 x 96), 200 rows 60.0 / 56.6
// and 256 rows 61.3 / 58.7 (256 x 96), 270 rows 87.9 / 79.0 (128 x 160); 37888 x 3584: 100 rows 65.6 / 56.3 and 128 rows 67.7 /
// 58.6 (128 x 160), 228 rows 85.2 / 73.6 and 256 rows 86.4 / 74.2 (256 x 160).  With one row tile a 128 x 256 tile costs 0.68: its
// weights are all from memory and two thirds of the CUs ask for them (residual projections of 12288 and 14336 channels, whose
// plan that decides as well, take the same time with either).  Beside their products odd tiles have 2 .. 3.5 us more (128 x 256 /
// 256 x 96 in one round: K = 1024 16.4 / 17.6, 2048 26.1 / 26.8, 4096 55.5 / 51.7; 128 x 256 / 128 x 160: K = 512 11.4 / 13.0, 1024
// 18.3 / 18.7, 2048 31.7 / 30.3; 128 x 128 / 128 x 96: 1024 14.6 / 15.4, 1536 23.9 / 22.6), and chips differ by several per cent in
// how they take a round that needs all CUs at once: 128 x 96 for 80 rows of 24576 x 4096 was 0.92, 0.92 and 1.09 of the time of
// 128 x 128 on three of them.
// Over 17 widths of 2048 .. 28672 features, five K of 1024 .. 8192 and 66 .. 16384 rows, in turn: where the odd tiles change the
// launch it takes 0.92 of the time without them on average; the residual tile of 224, over ten widths and ten K, 0.945.
enum GtTile { GT_256x256 = 0, GT_128x256 = 1, GT_128x128 = 2, GT_128x64 = 3, GT_128x96 = 4, GT_128x160 = 5, GT_256x96 = 6, GT_256x160 = 7, GT_256x224 = 8, GT_N = 9 };
constexpr unsigned GT_ODD_TILES = 0xf0u, GT_ODD_256 = 0xc0u, GT_RESID_TILES = 0xfu, GT_RESID_224 = 0x100u, GT_REST_TILES = 0x6u;
// of a mask of tiles (bit per GtTile) those that are built for this K
inline unsigned gt_built(int K, unsigned tiles) { return K % 64 == 0 ? tiles : tiles & ~0x1f2u; }
struct GtPlan { GtTile tile; int splits, k_per; double us; };
// NW: weight rows of the product; max_splits 1: no K split; width_ok: bit per tile that its widths allow
// fold_us_per_share: what each share behind the first costs (written here, read by the kernel that adds it)
inline GtPlan gt_plan(int cus, int M, int NW, int K, int max_splits, unsigned width_ok, double fold_us_per_share) {
  static const int bm[GT_N] = {256, 128, 128, 128, 128, 128, 256, 256, 256}, bn[GT_N] = {256, 256, 128, 64, 96, 160, 96, 160, 224};
  // (up to 256 rows a 128-row tile waits for its weights, which no other row tile has brought in)
  const double unit[GT_N] = {1.0, M <= 128 ? 0.68 : 0.6, M <= 256 ? 0.45 : 0.33, M <= 256 ? 0.30 : 0.22,
                             M <= 128 ? 0.39 : 0.45, M <= 128 ? 0.60 : 0.45, 0.54, 0.80, 0.90};
  static const double fill[GT_N] = {4.0, 4.0, 4.0, 4.0, 6.0, 7.5, 7.5, 7.5, 4.0};
  GtPlan best{GT_128x128, 1, K, 1e30};
  for (int c = 0; c < GT_N; ++c) {
    if (!((gt_built(K, width_ok) >> c) & 1u)) continue;
    const int tiles = ((M + bm[c] - 1) / bm[c]) * ((NW + bn[c] - 1) / bn[c]);
    for (int sp = 1; sp <= max_splits; ++sp) {
      if (sp > 1 && (K / sp < 512 || tiles * sp > cus)) break;    // shares long enough to pay for fill and drain
      const int k_per = ((K + sp - 1) / sp + 63) / 64 * 64;
      const int n_sp = (K + k_per - 1) / k_per;
      if (n_sp != sp) continue;
      const double rounds = (double)((tiles * sp + cus - 1) / cus);
      // a 256 x 256 tile takes 1.6 us per stage and about 4 us of fill and drain
      const double t = rounds * (unit[c] * 1.6 * (k_per / 64) + fill[c]) + (sp - 1) * fold_us_per_share;
      if (t < best.us) best = GtPlan{(GtTile)c, sp, k_per, t};
    }
  }
  return best;
}

// A last round of 256 x 256 tiles that fills few of the CUs takes as long as a whole one.  Returns how many column tiles
// the whole rounds hold (0: none, or not worth it) when those and then the remaining columns as a launch of smaller
// tiles, which spread over the chip, are estimated shorter than `one_us`, all columns in one launch.  The second launch
// costs its boundary and a fill of its own, 6 us.  (592 tiles of a 1024 x 37888 x 3584 product: 256 -> 225 us.  The cut in
// one launch, its remainder as a second loop of the same kernel, costs the main loop registers: 313 us.)
inline int gt_whole_rounds(int cus, int M, int NW, int K, double one_us) {
  const int tiles_m = (M + 255) / 256, tiles_n = (NW + 255) / 256, rounds = tiles_m * tiles_n / cus;
  const int n_tn = rounds * cus / tiles_m;
  if (rounds < 1 || n_tn < 1 || n_tn >= tiles_n) return 0;
  const double us = rounds * (1.6 * (K / 64) + 4.0) + gt_plan(cus, M, NW - n_tn * 256, K, 1, GT_REST_TILES, 0.0).us + 6.0;
  return us < one_us ? n_tn : 0;
}

// What a product launches: n_tn column tiles of 256 x 256 in whole rounds (0: none), the columns behind them in `tile`; without
// whole rounds the sum over K may be in several shares of k_per.
struct GtForm { GtTile tile; int splits, k_per, n_tn; };
// rest: tiles that the columns behind whole rounds may get
inline GtForm gt_form(int cus, int M, int NW, int K, const GtPlan& p, unsigned rest) {
  const int n_tn = gt_whole_rounds(cus, M, NW, K, p.us);
  if (n_tn == 0) return GtForm{p.tile, p.splits, p.k_per, 0};
  return GtForm{gt_plan(cus, M, NW - n_tn * 256, K, 1, rest, 0.0).tile, 1, K, n_tn};
}
// Residual projections: 256 x 224 at 0.90, in the place of 256 x 256 tiles alone (1024 x 3584 x 18944 in four K shares is 224 tiles
// of 256 x 256 or 256 of these, 142 / 138; 2304 x 4096 x 12288 234 / 206).  The estimate makes smaller tiles and fewer shares
// look dearer than they are: 1536 x 4096 x 4096 as 128 x 256 tiles 57, as two shares of 256 x 224 70; 1552 x 3584 x 3584 45 / 61; 6810
// x 3584 x 3584 157 / 168.
inline GtForm gt_resid_form(int cus, int M, int N, int K, int max_splits, bool starts_apart) {
  const double fold = 1.0 + 8.0 * M * (double)N / 4.0e6;
  GtPlan p = gt_plan(cus, M, N, K, max_splits, GT_RESID_TILES, fold);
  if (!starts_apart && p.tile == GT_256x256) {
    const GtPlan q = gt_plan(cus, M, N, K, p.splits, GT_RESID_224, fold);
    if (q.us < p.us) p = q;
  }
  return gt_form(cus, M, N, K, p, GT_REST_TILES);
}
// Gate/up.  Odd tiles of 128 rows are for one or two row tiles; a third that is a quarter full still pays (24576 x 4096 in 256 x
// 256 tiles takes 88 whatever the rows, in 128 x 160 79 at 270 rows, 86 at 320, 92 at 356, 97 at 384; x 5120 104 and 99 / 112
// at 270 / 320), a full one only in the place of 128 x 256 tiles (384 x 11008 x 2048 29.4 / 25.9).  Whole rounds have to pay with
// a rest of even tiles (one launch of 256 x 256 / whole rounds and 128 x 160: 1152 x 22016 x 4096 183 / 190, 1664 x 24576 x 4096
// 282 / 285; and 256 x 160: 3044 x 24576 x 4096 465 / 455, 5200 x 11008 x 2048 189 / 194); a rest that is there anyway takes any
// (1424 x 24576 x 4096 with 128 x 256 250, with 128 x 160 241; 1024 x 37888 x 3584 235 / 225).
inline GtForm gt_swiglu_form(int cus, int M, int F, int K, bool starts_apart) {
  GtPlan p = gt_plan(cus, M, 2 * F, K, 1, 0x7u | (M <= 288 ? GT_ODD_TILES : GT_ODD_256), 0.0);
  if (M <= 384 && p.tile == GT_128x256) p = gt_plan(cus, M, 2 * F, K, 1, 0x7u | GT_ODD_TILES, 0.0);
  return gt_form(cus, M, 2 * F, K, p, GT_REST_TILES | (starts_apart ? 0u : GT_ODD_TILES));
}

// q/k/v with the rotary embedding and the K/V write in its epilogue.  What a launch of a step takes, fitted over 13 widths of 1536
// .. 12288 weight rows, eight K of 1024 .. 5120 and 136 .. 2560 rows (1656 shapes, cold weights; standard deviation 4 .. 9 %).  Odd
// tiles, which are launched as one round only, with 1.5 us against them, so that what they are taken for is a gain.
inline double gt_rope_us(int cus, GtTile t, int M, int nw, int K) {
  const double s = K / 64;
  const double n = (double)((M + 127) / 128 * ((nw + 127) / 128)) / cus;       // 128 x 128 tiles a CU
  const bool few = M <= GT_APART_ROWS;
  switch (t) {
    case GT_256x256: return 1.07 * s + 19.0;
    case GT_128x96: return (few ? 0.38 : 0.41) * s + 12.5;
    case GT_128x160: return (few ? 0.53 : 0.59) * s + 16.5;
    case GT_256x96: return few ? 0.58 * s + 15.5 : 0.57 * s + 19.5;
    case GT_256x160: return few ? 0.73 * s + 23.5 : 0.72 * s + 30.5;
    default: return n <= 1.0 ? (few ? 0.47 : 0.52) * s + 10.0 : n <= 2.0 ? (0.53 + 0.22 * n) * s + 9.5 : (0.64 + 0.33 * n) * s + 15.0;
  }
}
// Odd tiles only as one round: their epilogue needs the copies' ring, so a workgroup has one tile.  `us` (a stage and beside the
// stages, from 256 x 12288 x 4096 and 1024 x 4608 x 3584: 128 x 128 tiles / these 48.3 / 42.7 and 66.9 / 52.7) is on the scale of the
// other plans; at short sums it makes odd tiles look cheaper than they are, and two even tiles a CU dearer (steps, even / odd:
// 1600 x 3072 x 1024 23.1 / 28.7, 768 x 6144 x 2048 33.6 / 36.2), so they also have to be the quicker ones by gt_rope_us.  Of those 1656
// shapes 517 take an odd tile, in 0.88 of the even one's time as steps and 0.85 as prefills on average; nine lose 2 .. 4 %.
inline GtPlan gt_rope_plan(int cus, int M, int dq, int dkv, int dh, int K) {
  const int nw = dq + 2 * dkv;
  const GtPlan even = gt_plan(cus, M, nw, K, 1, (dq % 256 == 0 && dkv % 256 == 0 && dh == 128 ? 0x1u : 0u) | 0x4u, 0.0);
  const double even_us = gt_rope_us(cus, even.tile, M, nw, K);
  static const struct { GtTile t; int bm, bn; double stage, rest; } odd[4] = {
      {GT_128x96, 128, 96, 0.53, 9.0}, {GT_128x160, 128, 160, 0.75, 10.0}, {GT_256x96, 256, 96, 0.84, 10.0}, {GT_256x160, 256, 160, 1.09, 11.0}};
  GtPlan best = even;
  for (const auto& o : odd) {
    if ((M + o.bm - 1) / o.bm * ((nw + o.bn - 1) / o.bn) > cus || gt_rope_us(cus, o.t, M, nw, K) > even_us) continue;
    const double us = o.stage * (K / 64) + o.rest;
    if (us < best.us) best = GtPlan{o.t, 1, K, us};
  }
  return best;
}

// ... taken unless the split product and the rotary kernel behind it are quicker by the estimate (the rotary kernel: about 10 us
// and its operands at 2.5 TB/s).  Measured, product + rotary kernel against the fused one (us): 15348 rows x 4608 x 3584: 464 +
// 278 / 513; 1184 x 12288 x 4096: 107 + 38 / 128; 1024 x 4608 x 3584: 42 + 21 / 53; 211 x 12288 x 4096: 43 + 13 / 41.
inline bool gt_qkv_fused(int cus, int M, int dq, int dkv, int dh, int K, int max_splits) {
  const int nw = dq + 2 * dkv;
  const GtPlan fused = gt_rope_plan(cus, M, dq, dkv, dh, K);
  const GtPlan split = gt_plan(cus, M, nw, K, max_splits, (dq % 256 == 0 && dkv % 256 == 0 ? 0x3u : 0u) | 0xcu, 0.0);
  return fused.us <= split.us + 10.0 + (4.0 * split.splits + 2.0) * M * (double)nw / 2.5e6;
}

}  // namespace dllm

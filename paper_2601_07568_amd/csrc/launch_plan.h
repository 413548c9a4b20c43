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
inline AttnPlan attn_plan(int head_dim, int n_q_heads, int n_kv_heads, int B, int Q, int T, int max_kv, int page_tokens,
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
  const int rg_cap = p.staged ? 8 : 4;                         // the register-direct kernel runs at most 4 waves
  p.n_rg_wg = n_rg < rg_cap ? n_rg : rg_cap;
  p.n_chunks = (n_rg + p.n_rg_wg - 1) / p.n_rg_wg;
  const int nkb = (max_kv + 31) / 32;
  // units along the keys: short dependent chains matter more than partial traffic here (a step's
  // attention is a few MB), so give every unit about two 32-key blocks, within the partial buffer
  int64_t want = 2048 / ((int64_t)B * n_kv_heads * n_rg);
  if (want < 1) want = 1;
  int64_t by_work = p.staged ? (nkb + 7) / 8 : (nkb + 1) / 2;   // staged kernel: at least four 64-key blocks per unit ...
  if (p.staged && by_work > 1) {   // (a single unit needs no combine)
    // ... or two, or one, where that still leaves CUs without a workgroup (kernel + combine, us, four / two / one, 4 key heads of
    // 7: 512 keys 17.3 + 4.8 / 15.5 + 4.8 / 13.7 + 4.8 in 12 / 20 / 36 workgroups, 2048 keys 19.7 + 4.8 / 16.7 + 5.3 / 15.6 + 7.2
    // in 36 / 68 / 132, 8000 keys 22.0 + 6.1 / 20.9 + 10.0 / - in 128 / 252, 4 sequences of 2048 22.6 + 6.4 / 31.5 + 9.1 / - in
    // 144 / 272)
    const int64_t per_unit = (int64_t)p.n_chunks * B * n_kv_heads;
    if ((nkb + 1) / 2 * per_unit <= 64) by_work = (nkb + 1) / 2;
    else if ((nkb + 3) / 4 * per_unit <= 128) by_work = (nkb + 3) / 4;
  }
  int64_t units = want < by_work ? want : by_work;
  if (p.staged && units < least) units = least;
  if (units > most) units = most;
  // one row group per KV head (a batch-1 block on a multi-head model): four units share a workgroup and
  // merge their partial results in LDS, which leaves a quarter of the partials to write and re-read
  p.kspl = 1;
  // (also where more than 512 such workgroups are a second round: 32 sequences of 1024 keys, 32 key heads, as two single-wave
  // units with their combine 126 + 16 us, as one workgroup of four waves 129)
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

}  // namespace dllm

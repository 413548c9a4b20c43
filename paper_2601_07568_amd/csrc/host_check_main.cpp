// Host-side exercise of the C ABI for a sanitizer build (AddressSanitizer + UndefinedBehaviorSanitizer on the host
// code only): every entry point is driven through its argument validation, the workspace map and the context
// life cycle with device pointers that are never dereferenced on the host, and the order in which the tile kernel's copies
// and products run through their work (gemm_ring.h) and the attention's launch (launch_plan.h) are checked.  No GPU is needed: nothing is launched.
// With arguments it says instead which tiles products of given sizes get.
// Exit status 0 = every call returned what it should; the sanitizers abort the process on a finding.
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <utility>
#include <vector>
#include "../../include/dllm.h"
#include "gemm_ring.h"
#include "launch_plan.h"

static int failures = 0;
#define EXPECT(call, want)                                                            \
  do {                                                                                \
    const long got_ = (long)(call);                                                   \
    if (got_ != (long)(want)) { printf("line %d: got %ld, want %ld\n", __LINE__, got_, (long)(want)); ++failures; } \
  } while (0)

static dllm_config tiny_cfg() {
  dllm_config c;
  memset(&c, 0, sizeof(c));
  c.n_layers = 2; c.d_model = 256; c.n_q_heads = 4; c.n_kv_heads = 4; c.head_dim = 64; c.d_ff = 688;
  c.vocab = 4096; c.mask_id = 4095; c.rms_eps = 1e-5f; c.rope_base = 10000.f; c.dtype = DLLM_F32;
  c.page_tokens = 16; c.max_pages_per_seq = 8; c.n_pages = 8; c.max_batch = 2; c.max_q = 32; c.max_tokens = 128;
  return c;
}

// The tile kernel's copies against what it multiplies.  Ring of `ring` buffers of one operand, `nsw` of the weights (the
// deeper ring, by which a launch is sized); item i has `stages` + i % 3 stages and starts at stage i % (their number).
// Every workgroup's copies are issued as the kernel issues them - ring - 1 stages in front of its first item, then one per
// stage, each followed by a step of the cursor that knows the item behind the one being multiplied and no other - and the
// stage a copy fetched has to be the one that is multiplied from its buffer.  Returns the number of wrong stages and of
// items that are not multiplied exactly once.  pair 1, 2: copies of two stages together, for items of `stages` +
// 2 * (i % 3) stages, as early as the kernel issues them (in the stage in front of every other one) or as late (in that one).
static int ring_errors(int ring, int nsw, int stages, int n_items, int slots, int pair = 0) {
  struct It { int id, k_first, k_begin, k_end; bool ok; };
  const int n_wg = dllm::gt_workgroups(n_items, slots, stages, nsw + (pair ? 1 : 0));
  auto item = [&](int wg, int it) {
    const int id = dllm::gt_item(wg, n_wg, it, n_items), n = stages + (id < 0 ? 0 : id) % 3 * (pair ? 2 : 1);
    return It{id, (id < 0 ? 0 : id) % n * 64, 0, n * 64, id >= 0};
  };
  int errors = 0;
  std::vector<int> seen(n_items, 0);
  for (int wg = 0; wg < n_wg; ++wg) {
    It cur = item(wg, 0);
    if (!cur.ok) continue;
    int it = 1, from = cur.id, k = cur.k_first, first = cur.k_first, begin = cur.k_begin, end = cur.k_end;
    It nxt = item(wg, it);
    std::vector<std::pair<int, int>> copied;                  // (item, k) of every copy, in order
    auto copy = [&]() {
      copied.push_back({from, k});
      GT_ADVANCE(k, first, begin, end, nxt, from = nxt.id);
    };
    for (int s = 0; s < (pair == 0 ? ring - 1 : pair == 1 ? ring : ring - 2); ++s) copy();
    for (size_t at = 0;;) {
      for (int s = 0, n = cur.k_end / 64; s < n; ++s, ++at) {
        for (int c = 0; c < (pair == 0 ? 1 : s % 2 == pair % 2 ? 2 : 0); ++c) copy();
        if (copied[at] != std::make_pair(cur.id, (cur.k_first / 64 + s) % n * 64)) ++errors;
      }
      ++seen[cur.id];
      if (!nxt.ok) break;
      cur = nxt;
      nxt = item(wg, ++it);
    }
  }
  for (int n : seen) errors += n != 1;
  return errors;
}

// The attention launch over sizes: what it asks for fits, and the staged kernel takes every call of at least four row groups
// over pages that are a power of two of at least 8 tokens (but for short ones of few sequences with grouped queries), however long its
// sequences, as long as the partials of enough units
// have room.  Returns the number of plans that break this.
static int attn_plan_errors() {
  using namespace dllm;
  int errors = 0;
  const int heads[][2] = {{28, 4}, {32, 32}, {32, 8}, {7, 1}};
  const int kvs[] = {1, 64, 97, 2048, 8192, 65536, 65537, 70032, 140032, 300032, 524288};
  for (const auto& h : heads)
    for (int dh = 64; dh <= 128; dh += 64)
      for (int B = 1; B <= 512; B *= 8)
        for (int Q = 0; Q <= 128; Q += 32)
          for (int pt = 8; pt <= 256; pt *= 2)
            for (int kv : kvs) {
              if (kv < Q || (Q == 0 && (int64_t)B * kv > 1 << 20)) continue;
              const int T = Q > 0 ? B * Q : B * kv;
              int64_t rows = (int64_t)T * h[0] * 8;           // (the workspace holds eight units, and 65536 rows at least)
              if (rows < 65536) rows = 65536;
              const AttnPlan p = attn_plan(256, dh, h[0], h[1], B, Q, T, kv, pt, rows, true);
              const int groups = ((Q > 0 ? Q : kv) * (h[0] / h[1]) + 31) / 32;
              // (steps with grouped queries and at most a workgroup per CU may take the register kernel)
              const bool few = Q > 0 && h[0] > h[1] && groups > 4 && (int64_t)B * h[1] * groups <= 256;
              const int blocks = (kv + 63) / 64, per_unit = (blocks + p.units - 1) / p.units;
              const bool ok = p.units >= 1 && p.units / p.kspl <= ATTN_MAX_SPLITS && p.units % p.kspl == 0 &&
                              (p.units == p.kspl || (int64_t)(p.units / p.kspl) * T * h[0] <= rows) &&
                              p.lds <= (size_t)DL_LDS_MAX && p.n_rg_wg * p.n_chunks >= groups && (p.staged ? groups >= 4 : groups < 4 || few) &&
                              (p.staged || (p.n_rg_wg * p.kspl <= 4 && (p.kspl == 1 || p.n_rg_wg == 1))) &&
                              (!p.staged || Q == 0 || (p.pg_cap >= per_unit * (pt < 64 ? 64 / pt : 1) &&
                                                       p.lds >= (size_t)DL_NB * dh * 256 + 4 * (size_t)p.pg_cap));
              if (!ok && errors++ < 5) printf("attention plan: heads %d/%d x %d, B %d, Q %d, %d keys, pages of %d\n", h[0], h[1], dh, B, Q, kv, pt);
            }
  return errors;
}

// "form" then (kind, rows, columns, K, starts_apart) for each product: what it launches on 256 CUs, a line each.  kind "gate-up"
// (columns: features) or "resid" (at most four K shares, one above 2048 rows): [whole rounds' column tiles +] tile [/ K shares];
// "qkv:query heads:key heads:channels" (columns: not read): the fused kernel's tile, or "split"; "attn:query heads:key
// heads:channels:page" (rows: sequences, columns: query rows of each, K: the longest prefix): "staged" or "waves" along the keys of
// a workgroup, row groups of a workgroup x parts along the keys.
static int print_forms(int n, char** v) {
  using namespace dllm;
  static const char* const name[GT_N] = {"256x256", "128x256", "128x128", "128x64", "128x96", "128x160", "256x96", "256x160", "256x224"};
  for (int i = 0; i + 4 < n; i += 5) {
    const int M = atoi(v[i + 1]), N = atoi(v[i + 2]), K = atoi(v[i + 3]);
    const bool apart = atoi(v[i + 4]) != 0;
    int hq, hkv, dh;
    if (sscanf(v[i], "qkv:%d:%d:%d", &hq, &hkv, &dh) == 3) {
      const bool fused = gt_qkv_fused(256, M, hq * dh, hkv * dh, dh, K, M <= 2048 ? 3 : 1);
      printf("%s\n", fused ? name[gt_rope_plan(256, M, hq * dh, hkv * dh, dh, K).tile] : "split");
      continue;
    }
    int page;
    if (sscanf(v[i], "attn:%d:%d:%d:%d", &hq, &hkv, &dh, &page) == 4) {
      int64_t part_rows = (int64_t)M * N * hq * 8;            // (an engine for just this call)
      if (part_rows < 65536) part_rows = 65536;
      const AttnPlan p = attn_plan(256, dh, hq, hkv, M, N, M * N, K + N, page, part_rows, true);
      if (p.staged) printf("staged:%dx%d\n", p.n_rg_wg, p.units);
      else printf("%d:%dx%d\n", p.kspl, p.n_rg_wg, p.units / p.kspl);
      continue;
    }
    const GtForm f = strcmp(v[i], "resid") == 0 ? gt_resid_form(256, M, N, K, M <= 2048 ? 4 : 1, apart) : gt_swiglu_form(256, M, N, K, apart);
    if (f.n_tn > 0) printf("%d+%s\n", f.n_tn, name[f.tile]);
    else if (f.splits > 1) printf("%s/%d\n", name[f.tile], f.splits);
    else printf("%s\n", name[f.tile]);
  }
  return 0;
}

int main(int argc, char** argv) {
  if (argc > 1 && strcmp(argv[1], "form") == 0) return print_forms(argc - 2, argv + 2);
  EXPECT(attn_plan_errors(), 0);
  const int rings[][2] = {{2, 3}, {3, 4}, {4, 5}, {4, 6}, {3, 3}, {4, 4}};
  for (const auto& r : rings)
    for (int stages = 2; stages <= 8; ++stages)
      for (int n_items = 1; n_items <= 48; ++n_items) {       // on 8 places: up to six items after each other
        EXPECT(ring_errors(r[0], r[1], stages, n_items, 8), 0);
        EXPECT(ring_errors(r[1], r[1], stages, n_items, 8), 0);
        if (r[1] >= 4)                                          // (an odd number of stages: a workgroup per item, as gt_launch has it)
          for (int pair = 1; pair <= 2; ++pair) EXPECT(ring_errors(r[1], r[1], stages, n_items, stages % 2 ? n_items + 1 : 8, pair), 0);
      }
  void* const p = (void*)0x3000;          // stands for device memory; the host never reads it
  int32_t* const ip = (int32_t*)p;
  float* const fp = (float*)p;
  for (int dtype = 0; dtype < 2; ++dtype) {
    dllm_config cfg = tiny_cfg();
    cfg.dtype = dtype;
    if (dtype == DLLM_BF16) { cfg.d_ff = 688; cfg.n_kv_heads = 2; }
    const size_t ws = dllm_workspace_bytes(&cfg), kv = dllm_kv_pool_bytes(&cfg);
    EXPECT(ws > 0 && kv > 0, 1);
    std::vector<dllm_layer_w> lw(cfg.n_layers);
    for (auto& l : lw) l = dllm_layer_w{p, p, p, p, p, p, p, p, p};
    dllm_weights w{p, p, p, lw.data()};
    dllm_ctx* ctx = nullptr;
    void* const wsp = (void*)(0x20000 * 256);
    EXPECT(dllm_create(&ctx, &cfg, &w, p, kv - 1, wsp, ws), DLLM_ENOSPACE);
    EXPECT(dllm_create(&ctx, &cfg, &w, p, kv, wsp, ws - 1), DLLM_ENOSPACE);
    EXPECT(dllm_create(&ctx, &cfg, &w, nullptr, kv, wsp, ws), DLLM_EINVAL);
    EXPECT(dllm_create(&ctx, &cfg, &w, p, kv, (char*)wsp + 8, ws), DLLM_EINVAL);
    EXPECT(dllm_create(nullptr, &cfg, &w, p, kv, wsp, ws), DLLM_EINVAL);
    { dllm_config bad = cfg; bad.head_dim = 48; EXPECT(dllm_workspace_bytes(&bad), 0); EXPECT(dllm_create(&ctx, &bad, &w, p, kv, wsp, ws), DLLM_ESHAPE); }
    { dllm_config bad = cfg; bad.mask_id = cfg.vocab; EXPECT(dllm_kv_pool_bytes(&bad), 0); }
    { dllm_config bad = cfg; bad.max_batch = 1 << 20; bad.max_q = 1 << 20; EXPECT(dllm_workspace_bytes(&bad), 0); }
    lw[1].wo = nullptr;
    EXPECT(dllm_create(&ctx, &cfg, &w, p, kv, wsp, ws), DLLM_EINVAL);
    lw[1].wo = p;
    EXPECT(dllm_create(&ctx, &cfg, &w, p, kv, wsp, ws), DLLM_OK);
    if (!ctx) { printf("no context\n"); return 2; }
    // steps
    EXPECT(dllm_denoise_step(ctx, nullptr, 0, 32, 64, ip, ip, ip, ip, fp, nullptr), DLLM_EINVAL);
    EXPECT(dllm_denoise_step(ctx, nullptr, 3, 32, 64, ip, ip, ip, ip, fp, nullptr), DLLM_ESHAPE);
    EXPECT(dllm_denoise_step(ctx, nullptr, 1, 33, 64, ip, ip, ip, ip, fp, nullptr), DLLM_ESHAPE);
    EXPECT(dllm_denoise_step(ctx, nullptr, 1, 32, 97, ip, ip, ip, ip, fp, nullptr), DLLM_ESHAPE);
    EXPECT(dllm_denoise_step(ctx, nullptr, 1, 32, -1, ip, ip, ip, ip, fp, nullptr), DLLM_EINVAL);
    EXPECT(dllm_denoise_step(ctx, nullptr, 1, 32, 64, nullptr, ip, ip, ip, fp, nullptr), DLLM_EINVAL);
    EXPECT(dllm_denoise_step(nullptr, nullptr, 1, 32, 64, ip, ip, ip, ip, fp, nullptr), DLLM_EINVAL);
    EXPECT(dllm_denoise_step_var(ctx, nullptr, 1, 32, 64, ip, ip, nullptr, ip, ip, fp, nullptr), DLLM_EINVAL);
    EXPECT(dllm_denoise_step_live(ctx, nullptr, 1, 32, 64, ip, ip, nullptr, nullptr, ip, ip, fp, nullptr), DLLM_EINVAL);
    EXPECT(dllm_denoise_step_static(ctx, nullptr, 1, 33, 64, ip, ip, ip, ip, fp, nullptr), DLLM_ESHAPE);
    EXPECT(dllm_debug_logits(ctx, nullptr, 1, 32, 64, ip, ip, ip, nullptr), DLLM_EINVAL);
    EXPECT(dllm_debug_hidden(ctx, nullptr, 1, 32, 64, ip, ip, ip, 3, fp), DLLM_EINVAL);
    // packed forwards
    EXPECT(dllm_prefill_kv(ctx, nullptr, 1, 129, 129, ip, ip, nullptr, ip), DLLM_ESHAPE);
    EXPECT(dllm_prefill_kv(ctx, nullptr, 1, 0, 0, ip, ip, nullptr, ip), DLLM_EINVAL);
    EXPECT(dllm_prefill_kv(ctx, nullptr, 1, 64, 65, ip, ip, nullptr, ip), DLLM_EINVAL);
    EXPECT(dllm_prefill_kv(ctx, nullptr, 3, 64, 64, ip, ip, nullptr, ip), DLLM_ESHAPE);
    EXPECT(dllm_refresh_cache(ctx, nullptr, 1, 64, 64, ip, ip, nullptr, ip, ip, fp, nullptr), DLLM_EINVAL);
    // selection, state machine, bookkeeping
    EXPECT(dllm_unmask(ctx, nullptr, 1, 32, 32, ip, ip, fp, 0.9f, -1, nullptr, nullptr), DLLM_EINVAL);
    EXPECT(dllm_unmask(ctx, nullptr, 1, 32, 5, ip, ip, fp, 0.9f, 1, nullptr, nullptr), DLLM_EINVAL);
    EXPECT(dllm_unmask(ctx, nullptr, 1, 4096, 2048, ip, ip, fp, 0.9f, 1, nullptr, nullptr), DLLM_ESHAPE);
    EXPECT(dllm_unmask_entropy(ctx, nullptr, 1, 32, 32, ip, ip, nullptr, 0.45f, 1, nullptr, nullptr), DLLM_EINVAL);
    EXPECT(dllm_unmask_blocks(ctx, nullptr, 1, 64, 32, ip, ip, fp, 0.45f, 1, nullptr, nullptr, nullptr), DLLM_EINVAL);
    EXPECT(dllm_unmask_traced(ctx, nullptr, 1, 32, 32, ip, ip, fp, 2.0f, 0, 1, 1, nullptr, nullptr, nullptr), DLLM_EINVAL);
    EXPECT(dllm_fsm_update(ctx, nullptr, 1, 257, 32, ip, ip, ip, 0.1, 0.95, 1, 0, nullptr, nullptr), DLLM_ESHAPE);
    EXPECT(dllm_fsm_update(ctx, nullptr, 1, 8, 32, ip, ip, ip, 0.1, 0.95, -1, 0, nullptr, nullptr), DLLM_EINVAL);
    EXPECT(dllm_fsm_plan(ctx, nullptr, 1, 8, 32, ip, ip, nullptr, -1, ip, ip, ip), DLLM_EINVAL);
    EXPECT(dllm_fsm_plan(ctx, nullptr, 1, 8, 32, ip, ip, nullptr, 4, nullptr, ip, ip), DLLM_EINVAL);
    EXPECT(dllm_fsm_window(ctx, nullptr, 1, 8, 32, 0, ip, ip, ip, 0, ip, ip, ip, ip, ip), DLLM_EINVAL);
    EXPECT(dllm_fsm_scatter(ctx, nullptr, 1, 8, 32, 2, ip, ip, nullptr, ip), DLLM_EINVAL);
    EXPECT(dllm_fsm_round_windows(ctx, nullptr, 1, 8, 32, 2, ip, ip, ip, nullptr, 0, ip, ip, ip, ip, ip, ip), DLLM_EINVAL);
    EXPECT(dllm_fsm_round_windows(ctx, nullptr, 1, 8, 32, 2, ip, ip, ip, ip, cfg.mask_id, ip, ip, ip, ip, ip, ip), DLLM_EINVAL);
    EXPECT(dllm_fsm_pack(ctx, nullptr, 1, 8, 32, 2, 0, 128, 128, ip, ip, ip, ip, ip, ip, 0, ip, ip, ip), DLLM_EINVAL);
    EXPECT(dllm_fsm_pack(ctx, nullptr, 1, 300, 32, 2, 64, 128, 128, ip, ip, ip, ip, ip, ip, 0, ip, ip, ip), DLLM_ESHAPE);
    EXPECT(dllm_fsm_unpack(ctx, nullptr, 1, 0, 128, ip, ip, ip, ip, ip, fp, nullptr, ip, fp, nullptr), DLLM_EINVAL);
    EXPECT(dllm_refresh_cache_dev(ctx, nullptr, 1, 64, 64, ip, ip, nullptr, ip, ip, fp, nullptr), DLLM_EINVAL);
    EXPECT(dllm_refresh_cache_dev(ctx, nullptr, 1, 129, 129, ip, ip, ip, ip, ip, fp, nullptr), DLLM_ESHAPE);
    EXPECT(dllm_noisy_sequence(ctx, nullptr, 1, 32, ip, ip, ip, 8, 1.5, ip), DLLM_EINVAL);
    EXPECT(dllm_eos_scan(ctx, nullptr, 1, 32, ip, 5, ip, nullptr, ip, nullptr), DLLM_EINVAL);
    EXPECT(dllm_gather_rows(ctx, nullptr, 2, 4, ip, ip, ip, ip, 0), DLLM_EINVAL);
    EXPECT(dllm_scatter_rows(ctx, nullptr, 0, 4, ip, ip, ip, ip + 64), DLLM_EINVAL);
    EXPECT(dllm_set_kernel_mode(ctx, 7), DLLM_EINVAL);
    EXPECT(dllm_set_kernel_mode(ctx, 1), DLLM_OK);
    EXPECT(dllm_read_status(ctx, nullptr, nullptr), DLLM_EINVAL);
    EXPECT(dllm_profile_read(ctx, nullptr, 0, nullptr, nullptr, nullptr), DLLM_EINVAL);
    if (dtype == DLLM_BF16) {
      EXPECT(dllm_packed_weight_bytes(&cfg) > 0, 1);
      EXPECT(dllm_pack_weights(ctx, nullptr, nullptr, 0), DLLM_EINVAL);
      EXPECT(dllm_pack_weights(ctx, nullptr, (char*)wsp + 16, dllm_packed_weight_bytes(&cfg)), DLLM_EINVAL);
      EXPECT(dllm_pack_weights(ctx, nullptr, wsp, dllm_packed_weight_bytes(&cfg) - 1), DLLM_ENOSPACE);
    } else {
      EXPECT(dllm_packed_weight_bytes(&cfg), 0);
      EXPECT(dllm_pack_weights(ctx, nullptr, wsp, 1 << 20), DLLM_ESHAPE);
    }
    EXPECT(strlen(dllm_strerror(DLLM_ESHAPE)) > 0, 1);
    EXPECT(strlen(dllm_last_hip_error(ctx)), 0);
    dllm_destroy(ctx);
  }
  dllm_destroy(nullptr);
  // a context too large for the library's own scratch array
  {
    dllm_config cfg = tiny_cfg();
    cfg.max_tokens = 16384;
    std::vector<dllm_layer_w> lw(cfg.n_layers, dllm_layer_w{p, p, p, p, p, p, p, p, p});
    dllm_weights w{p, p, p, lw.data()};
    dllm_ctx* ctx = nullptr;
    EXPECT(dllm_create(&ctx, &cfg, &w, p, dllm_kv_pool_bytes(&cfg), (void*)(0x20000 * 256), dllm_workspace_bytes(&cfg)), DLLM_OK);
    EXPECT(dllm_workspace_bytes(&cfg) > dllm_static_scratch_bytes(), 1);
    EXPECT(dllm_denoise_step_static(ctx, nullptr, 1, 32, 64, ip, ip, ip, ip, fp, nullptr), DLLM_ENOSPACE);
    dllm_destroy(ctx);
  }
  printf("host check: %d failure(s)\n", failures);
  return failures ? 1 : 0;
}

"""GPU parity of the tile kernel (products of more than 64 rows) at the edges of its tiles: row counts on both sides of
128 and 256, widths that end inside a tile, K splits with shares of unequal length, and work items that follow each
other in one workgroup.  The reference is the oracle with bfloat16 storage; the tolerance is that of the layer depth
(tests/harness.py: logit_tol), for the residual stream per row and for the LM head's statistics as everywhere."""
import numpy as np
import pytest
import torch

from oracle import dllm_oracle as O
from paper_2601_07568_amd import binding, synth
from tests import harness as H

pytestmark = pytest.mark.gpu
W = synth.as_float
ST = synth.round_bf16
# d_model 576: nine 64-deep stages, two and a quarter 256-wide tiles; d_ff 1088: 17 stages (K shares of 9 and 8),
# 2176 gate and up rows; the projections are 512 (q) and 128 (k, v) wide: no 256-wide tile fits k
EDGE = synth.ModelShape(1, 576, 8, 2, 64, 1088, 1500, 1499, dtype="bf16", lm_head_scale=8.0, name="tile-edges")
# long K over few columns: four K shares; more items than one round of a workgroup is not possible on few rows
LONG = synth.ModelShape(1, 256, 2, 2, 128, 4160, 700, 699, dtype="bf16", lm_head_scale=8.0, name="tile-long-k")


def run(ms, lens, Q, seed=5, pt=32, head=True):
    w = synth.Weights(ms, seed)
    B = len(lens)
    mp = (max(lens) + Q + pt - 1) // pt
    eng = H.make_engine(ms, w, page_tokens=pt, max_pages_per_seq=mp, n_pages=B * mp, max_batch=B, max_q=Q,
                        max_tokens=sum(lens))
    seqs = [synth.random_tokens(ms, seed + i, n) for i, n in enumerate(lens)]
    blks = [synth.masked_block(ms, seed + 10 + i, Q, max(1, Q // 2)) for i in range(B)]
    table = eng.i32(H.identity_table(eng, B))
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    eng.prefill_kv(eng.i32(np.concatenate(seqs)), eng.i32(cu), table, None, total_tokens=int(cu[-1]), max_seqlen=max(lens))
    qt, pre = eng.i32(np.stack(blks)), eng.i32(lens)
    hidden = eng.debug_hidden(qt, pre, table, ms.n_layers, max_prefix_len=max(lens)).cpu().numpy()
    cand = torch.zeros(B, Q, dtype=torch.int32, device=eng.device)
    conf = torch.zeros(B, Q, dtype=torch.float32, device=eng.device)
    ent = torch.zeros(B, Q, dtype=torch.float32, device=eng.device)
    eng.denoise_step(qt, pre, table, cand, conf, ent, max_prefix_len=max(lens))
    tol = H.logit_tol("bf16", ms.n_layers, "store")
    for b in range(B):
        ck, cv = O.prefill(w, seqs[b], widen=W, store=ST)
        logits, x = O.forward_cached(w, blks[b], ck, cv, widen=W, store=ST)
        assert H.rel_err_rows(hidden[b], x).max() <= tol, (b, H.rel_err_rows(hidden[b], x).max())
        if not head:
            continue
        r = {"logits": logits, "cand": O.confidence(logits, ms.mask_id)[0]}
        H.check_step_outputs(ms, r, blks[b] == ms.mask_id, cand.cpu().numpy()[b], conf.cpu().numpy()[b],
                             ent.cpu().numpy()[b], "bf16")
    assert eng.read_status() == 0
    eng.close()


@pytest.mark.parametrize("B,Q", [(1, 65), (1, 127), (2, 64), (3, 43), (1, 255), (4, 64), (1, 257), (3, 171), (8, 97)])
def test_row_counts_around_the_tiles(B, Q):
    """65 .. 776 rows: one to seven row tiles, the last one nearly empty, full and just full; prompts of 65 + rows are
    the no-cache forward on the same tiles."""
    run(EDGE, [70 + 3 * b for b in range(B)], Q)


@pytest.mark.parametrize("B,Q", [(1, 66), (2, 129)])
def test_k_shares_of_a_long_sum(B, Q):
    run(LONG, [9 + b for b in range(B)], Q)


def test_several_items_per_workgroup():
    """1600 rows x 2 * 8192 gate and up rows: 448 tiles of 256 x 256 on 256 places, a second one for most of them (a third
    and further: test_short_sums_with_more_than_two_tiles_per_workgroup)."""
    wide = synth.ModelShape(1, 128, 2, 1, 64, 8192, 600, 599, dtype="bf16", lm_head_scale=8.0, name="tile-items")
    run(wide, [40 + b for b in range(16)], 100)


def _short(name, d, hq, hkv, ff, vocab):
    return synth.ModelShape(1, d, hq, hkv, 64, ff, vocab, vocab - 1, dtype="bf16", lm_head_scale=8.0, name=name)


@pytest.mark.parametrize("ms,lens,Q", [
    # LM head of 256 x 128256 on 128 x 128 tiles: 1002 of them, K of four stages behind a ring of five
    (_short("short-head", 256, 2, 2, 256, 128256), [33, 40, 47], 32),
    # LM head of 128 x 131072 for 304 rows on 256 x 256 tiles: 1024 of them, two stages behind a ring of three
    (_short("short-head-256", 128, 2, 2, 128, 131072), [20 + b for b in range(19)], 32),
    # gate and up of 1600 x 32768, K of two stages: 896 tiles of 256 x 256
    (_short("short-gate-up", 128, 2, 1, 16384, 600), [40 + b for b in range(16)], 100),
    # q/k/v of 256 + 2 * 64 rows, K of three stages behind a ring of four: 128 x 64 tiles, and their ring of two a CU
    (_short("short-qkv", 192, 4, 1, 256, 600), [700 + b for b in range(32)], 8),
], ids=["head-k256", "head-k128", "gate-up-k128", "qkv-k192"])
def test_short_sums_with_more_than_two_tiles_per_workgroup(ms, lens, Q):
    """Sums shorter than the rings of copies with a third and further tile for every place on the chip (what the copies
    fetch for them is checked for all rings on the host: csrc/host_check_main.cpp)."""
    run(ms, lens, Q)


HALF = synth.ModelShape(1, 544, 8, 2, 64, 1120, 1500, 1499, dtype="bf16", lm_head_scale=8.0, name="tile-half-stage")


@pytest.mark.parametrize("ms,lens,Q", [
    (HALF, [70], 65), (HALF, [90], 127), (HALF, [33, 40, 47], 43), (HALF, [300], 257), (HALF, [20 + b for b in range(8)], 97),
    # K shares of the down projection: 65.5 stages
    (synth.ModelShape(1, 288, 2, 2, 128, 4192, 700, 699, dtype="bf16", lm_head_scale=8.0, name="half-stage-long-k"), [9, 10], 129),
    # gate and up of 1016 rows in whole rounds of 256 x 256 tiles and a rest of 128 x 128 ones
    (synth.ModelShape(1, 800, 2, 2, 64, 8544, 600, 599, dtype="bf16", lm_head_scale=8.0, name="half-stage-wide-ff"), [5 + b for b in range(8)], 127),
    # two and a half stages and more than two tiles per workgroup
    (_short("half-stage-short", 160, 2, 1, 16416, 600), [40 + b for b in range(16)], 100),
], ids=["65", "127", "129", "257", "776", "k-shares", "whole-rounds", "short"])
def test_k_of_half_a_stage_more(ms, lens, Q):
    """d_model and d_ff 32 more than a multiple of 64: the last stage of a sum is half empty."""
    assert ms.d_model % 64 == 32 and ms.d_ff % 64 == 32
    run(ms, lens, Q)


# Gate/up in tiles of 96 and 160 weight rows: (d, ff, (sequences, rows), form), sums about as short as each is taken for.  Every
# width ends inside a tile; one row tile and two, the last of them nearly empty or not.
ODD_TILES = [
    (1408, 2056, (1, 65), "128x96"), (1408, 2056, (1, 128), "128x96"),
    (1856, 16392, (1, 65), "128x160"), (1024, 5448, (3, 100), "128x160"),
    (2432, 10264, (1, 150), "256x96"), (2432, 5448, (3, 100), "256x96"),
    (768, 16392, (1, 255), "256x160"), (768, 8200, (4, 100), "256x160"),
]


@pytest.mark.parametrize("d,ff,rows,form", ODD_TILES)
def test_gate_up_in_odd_tiles(d, ff, rows, form):
    ms = synth.ModelShape(1, d, 2, 2, 64, ff, 600, 599, dtype="bf16", lm_head_scale=8.0, name=f"odd-{form}-{d}-{ff}")
    run(ms, [5 + b for b in range(rows[0])], rows[1])


# Residual projections in tiles of 224 weight rows: (d, heads, ff, (sequences, rows), form of O, form of down), all with a width
# that ends inside a tile: K of two stages and of twelve, more items than places (330 on 256); three K shares of unequal length
RESID_224 = [
    (2200, 2, 768, (83, 99), "256x224", "256x224"),
    (4680, 2, 3136, (8, 97), "128x256", "256x224/3"),
]


@pytest.mark.parametrize("d,heads,ff,rows,o,down", RESID_224)
def test_residual_projections_in_tiles_of_224(d, heads, ff, rows, o, down):
    """(The residual stream alone: with thousands of rows some sequence has a handful of near ties, whose gap lies inside twice the
    logit tolerance and binds no candidate, and one in nine of them fell the other way.)"""
    ms = synth.ModelShape(1, d, heads, 1, 64, ff, 600, 599, dtype="bf16", lm_head_scale=8.0, name=f"resid-224-{d}-{ff}")
    run(ms, [5 + b % 3 for b in range(rows[0])], rows[1], head=False)


# Whole rounds of 256 x 256 gate/up tiles and the columns behind them in smaller ones: (d, ff, (sequences, rows), form)
RESTS = [
    (512, 21776, (1, 257), "128+128x128"), (768, 23216, (1, 257), "128+128x256"), (1024, 21880, (1, 257), "128+128x160"),
    (2432, 11096, (8, 97), "64+256x96"),
]


@pytest.mark.parametrize("d,ff,rows,form", RESTS)
def test_gate_up_behind_whole_rounds(d, ff, rows, form):
    ms = synth.ModelShape(1, d, 2, 2, 64, ff, 600, 599, dtype="bf16", lm_head_scale=8.0, name=f"rest-{form}")
    run(ms, [5 + b for b in range(rows[0])], rows[1])


@pytest.mark.parametrize("ms,B,Q", [
    # gate and up of 1016 rows: 64 column tiles of 256 in one whole round, two and a half left
    (synth.ModelShape(1, 768, 2, 2, 64, 8512, 600, 599, dtype="bf16", lm_head_scale=8.0, name="wide-ff"), 8, 127),
    # down of 8217 rows: 7 of the 8 column tiles in one whole round, the last row tile of 25 rows
    (synth.ModelShape(1, 2048, 2, 1, 64, 768, 600, 599, dtype="bf16", lm_head_scale=8.0, name="wide-out"), 83, 99),
], ids=["gate-up", "down"])
def test_columns_behind_the_whole_rounds(ms, B, Q):
    """Products whose last columns are a launch of smaller tiles behind whole rounds of 256 x 256 ones."""
    run(ms, [5 + b % 3 for b in range(B)], Q)


def device_weights(ms, seed):
    """Seeded weights made on the device (wide layers): ({name: tensor}, [{name: tensor} per layer])."""
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)

    def mat(rows, cols, std=0.02):
        return torch.randn(rows, cols, generator=gen, device=dev).mul_(std).to(torch.bfloat16)

    one = torch.ones(ms.d_model, dtype=torch.bfloat16, device=dev)
    d, dq, dkv, f = ms.d_model, ms.n_q_heads * ms.head_dim, ms.n_kv_heads * ms.head_dim, ms.d_ff
    g = {"tok_emb": mat(ms.vocab, d), "lm_head": mat(ms.vocab, d, 0.02 * ms.lm_head_scale), "final_norm": one}
    layers = [{"attn_norm": one, "wq": mat(dq, d), "wk": mat(dkv, d), "wv": mat(dkv, d), "wo": mat(d, dq), "mlp_norm": one,
               "w_gate": mat(f, d), "w_up": mat(f, d), "w_down": mat(d, f)} for _ in range(ms.n_layers)]
    return g, layers


# 200 real rows behind a capacity of 1024.  The down projection of 3072 -> 4160 channels has three K shares at either size and
# sums whose starts go by 256 columns; gate/up of 37888 weight rows is whole rounds of 256 x 256 tiles and a rest that begins
# inside a group of 1920 features with a common start, and the down projection behind it has four shares again.  (One head of
# 64 channels: the q/k/v product takes the same form at either size.  Sums in another order round otherwise in about one of
# 10^4 bfloat16 numbers: of the seeds of the second case about every other one showed 64 features that were summed so.)
@pytest.mark.parametrize("d,ff,seed", [(4160, 3072, 4), (1024, 18944, 0)], ids=["down", "gate-up"])
def test_device_resident_total_sums_like_the_sized_call_whatever_its_tiles(d, ff, seed):
    """The tiles are chosen by the host's bound, where a sum starts by the rows there are: dllm_refresh_cache_dev with a
    capacity far above the total is dllm_refresh_cache of the total, bit for bit."""
    ms = synth.ModelShape(2, d, 1, 1, 64, ff, 600, 599, dtype="bf16", lm_head_scale=8.0, name=f"device-total-{d}-{ff}")
    sized, device = sized_and_device_total(ms, [120, 80], 1024, seed)
    for a, b in zip(sized, device):
        assert torch.equal(a, b)
    assert (sized[2][-16:] > 0.0).all()                     # the rows in flight are reported


def sized_and_device_total(ms, lens, cap, seed):
    """Pool, candidates, confidences and entropies of dllm_refresh_cache over prompts of these lengths, and of
    dllm_refresh_cache_dev with the same ones behind a capacity."""
    Q, pt = 16, 32
    total, B, mp = sum(lens), len(lens), 4
    w = device_weights(ms, seed)
    out = []
    for n in (total, cap):
        eng = binding.Engine(ms, None, page_tokens=pt, max_pages_per_seq=mp, n_pages=B * mp, max_batch=B, max_q=64, max_tokens=cap,
                             device_weights=w)
        toks = np.full(n, 3, dtype=np.int32)
        toks[:total] = np.concatenate([np.concatenate([synth.random_tokens(ms, 60 + b, k - Q), synth.masked_block(ms, 70 + b, Q, Q)])
                                       for b, k in enumerate(lens)])
        cu, table = eng.i32([0, lens[0], total]), eng.i32(H.identity_table(eng, B))
        ncommit = eng.i32([k - Q for k in lens])
        cand = torch.zeros(n, dtype=torch.int32, device=eng.device)
        conf, ent = (torch.zeros(n, dtype=torch.float32, device=eng.device) for _ in range(2))
        if n == total:
            eng.refresh_cache(eng.i32(toks), cu, table, ncommit, cand, conf, ent, total_tokens=n, max_seqlen=max(lens))
        else:
            eng.refresh_cache_dev(eng.i32(toks), cu, table, ncommit, cand, conf, ent, max_seqlen=max(lens))
        assert eng.read_status() == 0
        out.append([eng.kv_pool.clone(), cand[:total], conf[:total], ent[:total]])
        eng.close()
    return out


# (d, query heads, key heads, head width, prompts, capacity, tile of the sized call, tile at the capacity): q/k/v with the rotary
# embedding, K of eight to 36 stages
ROPE_PAIRS = [
    (1792, 36, 12, 64, [126, 124], 300, "128x96", "128x128"),
    (1792, 32, 16, 64, [120, 80], 263, "128x96", "128x128"),
    (512, 16, 16, 128, [100, 29], 1500, "128x128", "256x256"),
    (1792, 16, 16, 128, [100, 29], 1500, "128x96", "256x256"),
    (1536, 32, 32, 64, [100, 29], 1500, "128x128", "256x160"),
    (2304, 24, 8, 128, [120, 80], 1024, "128x96", "128x160"),
]


@pytest.mark.parametrize("d,hq,hkv,dh,lens,cap,sized,device", ROPE_PAIRS)
def test_device_resident_total_rotates_like_the_sized_call(d, hq, hkv, dh, lens, cap, sized, device):
    """As above where the q/k/v product takes another tile at the capacity: the first layer's keys and values, bit for bit, and
    everything behind them where the residual projections have the same K shares at both sizes (the first case)."""
    layers = 2 if hq == 36 else 1
    ms = synth.ModelShape(layers, d, hq, hkv, dh, 512, 600, 599, dtype="bf16", lm_head_scale=8.0, name=f"device-total-rope-{d}-{dh}")
    a, b = sized_and_device_total(ms, lens, cap, 2)
    assert torch.equal(a[0], b[0]) and int(a[0].count_nonzero()) > 0
    if layers == 2:
        assert all(torch.equal(x, y) for x, y in zip(a, b))


@pytest.mark.parametrize("ms", [EDGE, LONG], ids=["head-dim-64", "head-dim-128"])
@pytest.mark.parametrize("lens,n_cache,pt", [([129, 70, 31], [129, 64, 0], 32), ([67], [66], 24), ([300, 3, 5, 150], [299, 3, 2, 150], 64)])
def test_keys_and_values_written_by_the_projection(ms, lens, n_cache, pt):
    """The q/k/v product writes K and V itself: packed sequences that start anywhere in a tile, positions that are not
    cached, pages of 24 tokens (four tokens of a value row may end a page).  Slots past n_cache stay as they were."""
    w = synth.Weights(ms, 3)
    B = len(lens)
    mp = (max(lens) + pt - 1) // pt
    eng = H.make_engine(ms, w, page_tokens=pt, max_pages_per_seq=mp, n_pages=B * mp, max_batch=B, max_q=32,
                        max_tokens=sum(lens))
    perm = np.random.default_rng(1).permutation(B * mp)
    table = H.identity_table(eng, B, perm)
    seqs = [synth.random_tokens(ms, 20 + i, n) for i, n in enumerate(lens)]
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    eng.kv_pool.view(torch.bfloat16).fill_(7.0)
    eng.prefill_kv(eng.i32(np.concatenate(seqs)), eng.i32(cu), eng.i32(table), eng.i32(n_cache), total_tokens=int(cu[-1]),
                   max_seqlen=max(lens))
    for b in range(B):
        ck, cv = O.prefill(w, seqs[b], widen=W, store=ST)
        for which, ref in ((0, ck[0]), (1, cv[0])):
            got = H.gather_cache(eng, table[b], lens[b], 0, which)
            n = n_cache[b]
            # one bfloat16 rounding of a float sum against one of the exact sum: neighbours in bfloat16 at most (2^-7)
            assert np.abs(got[:n] - ref[:n]).max(initial=0.0) <= 2.0 ** -7 * np.abs(ref).max(), (b, which)
            assert (got[n:] == 7.0).all(), (b, which)
    assert eng.read_status() == 0
    eng.close()


# q/k/v in tiles of 96 and 160 weight rows: (d, query heads, key heads, head width, prompts, cached of each, page, form).  Tiles lie
# across the ends of q and k and end behind v; rows end inside a tile; runs of eight tokens end at a page's or a prompt's end.
ODD_ROPE = [
    (1792, 48, 8, 64, [129, 70, 31], [129, 64, 0], 24, "128x96"),
    (2240, 68, 4, 64, [500, 3, 300, 190], [499, 3, 296, 150], 32, "128x160"),
    (2560, 34, 2, 128, [257, 143, 650], [257, 100, 649], 24, "256x96"),
    (1408, 72, 3, 128, [400, 299, 201], [399, 299, 0], 64, "256x160"),
]


@pytest.mark.parametrize("d,hq,hkv,dh,lens,n_cache,pt,form", ODD_ROPE, ids=[f[-1] for f in ODD_ROPE])
def test_keys_and_values_written_from_odd_tiles(d, hq, hkv, dh, lens, n_cache, pt, form):
    ms = synth.ModelShape(1, d, hq, hkv, dh, 256, 600, 599, dtype="bf16", lm_head_scale=8.0, name=f"odd-rope-{form}")
    test_keys_and_values_written_by_the_projection(ms, lens, n_cache, pt)


@pytest.mark.parametrize("i,seqs,Q", [(0, 3, 77), (0, 2, 115), (2, 10, 105)], ids=["128x96", "128x96-one-tile-nearly-empty", "256x96"])
def test_steps_on_odd_rope_tiles(i, seqs, Q):
    """Denoise steps on the same tiles: every row of q, and the rows' keys and values through the attention."""
    d, hq, hkv, dh = ODD_ROPE[i][:4]
    ms = synth.ModelShape(1, d, hq, hkv, dh, 256, 600, 599, dtype="bf16", lm_head_scale=8.0, name=f"odd-rope-step-{i}")
    run(ms, [9 + 30 * b for b in range(seqs)], Q, head=False)


@pytest.mark.parametrize("ms,lens,Q,n_masked", [(EDGE, [80], 32, 1), (EDGE, [75, 90], 32, 17), (LONG, [70], 64, 64)],
                         ids=["one-row", "seventeen-rows-k-576", "sixty-four-rows"])
def test_few_head_rows_behind_a_forward_of_many(ms, lens, Q, n_masked):
    """Outputs of a refresh with at most 64 rows of the LM head (which then reads the packed weights): every sequence's
    last Q tokens, n_masked of them masked, against the forward without cache."""
    w = synth.Weights(ms, 7)
    B, pt = len(lens), 32
    mp = (max(lens) + pt - 1) // pt
    eng = H.make_engine(ms, w, page_tokens=pt, max_pages_per_seq=mp, n_pages=B * mp, max_batch=B, max_q=Q, max_tokens=sum(lens))
    seqs = [np.concatenate([synth.random_tokens(ms, 40 + i, n - Q), synth.masked_block(ms, 50 + i, Q, n_masked)])
            for i, n in enumerate(lens)]
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    cand = torch.zeros(sum(lens), dtype=torch.int32, device=eng.device)
    conf, ent = (torch.zeros(sum(lens), dtype=torch.float32, device=eng.device) for _ in range(2))
    eng.refresh_cache(eng.i32(np.concatenate(seqs)), eng.i32(cu), eng.i32(H.identity_table(eng, B)), eng.i32([n - Q for n in lens]),
                      cand, conf, ent, total_tokens=int(cu[-1]), max_seqlen=max(lens))
    for b, n in enumerate(lens):
        full, _, _, _ = O.forward_full(w, seqs[b], widen=W, store=ST)
        rows = slice(int(cu[b]) + n - Q, int(cu[b]) + n)
        r = {"logits": full[n - Q:], "cand": O.confidence(full[n - Q:], ms.mask_id)[0]}
        H.check_step_outputs(ms, r, seqs[b][n - Q:] == ms.mask_id, cand.cpu().numpy()[rows], conf.cpu().numpy()[rows],
                             ent.cpu().numpy()[rows], "bf16")
    assert eng.read_status() == 0
    eng.close()


def test_few_head_rows_scale_by_the_norms_own_factor():
    """The LM head's outputs behind a forward of many tokens and behind a denoise step run through the same kernel; with no
    layers, 256 channels and embeddings of small whole numbers (every sum of squares and every product exact) the row
    factor is all that could differ, and must not by a bit."""
    ms = synth.ModelShape(0, 256, 2, 2, 64, 256, 512, 511, dtype="bf16", lm_head_scale=8.0, name="head-only")
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(11)
    g = {"tok_emb": torch.randint(-9, 10, (512, 256), generator=gen, device=dev).to(torch.bfloat16),
         "lm_head": torch.randn(512, 256, generator=gen, device=dev).mul_(0.2).to(torch.bfloat16),
         "final_norm": torch.ones(256, device=dev, dtype=torch.bfloat16)}
    from paper_2601_07568_amd.binding import Engine
    eng = Engine(ms, None, page_tokens=16, max_pages_per_seq=2, n_pages=2, max_batch=1, max_q=8, max_tokens=24, device_weights=(g, []))
    table, zero = eng.i32([[0, 1]]), eng.i32([0])
    q = torch.full((1, 8), ms.mask_id, dtype=torch.int32, device=dev)
    for _ in range(64):
        g["tok_emb"][ms.mask_id] = torch.randint(-9, 10, (256,), generator=gen, device=dev).to(torch.bfloat16)
        out = []
        for many in (False, True):
            cand = torch.zeros(24, dtype=torch.int32, device=dev)
            conf, ent = (torch.zeros(24, dtype=torch.float32, device=dev) for _ in range(2))
            if many:
                toks = torch.cat([torch.arange(16, dtype=torch.int32, device=dev), q[0]])
                eng.refresh_cache(toks, eng.i32([0, 24]), table, eng.i32([16]), cand, conf, ent, total_tokens=24, max_seqlen=24)
                out.append((cand[16:], conf[16:], ent[16:]))
            else:
                c1, f1, e1 = cand[:8].view(1, 8), conf[:8].view(1, 8), ent[:8].view(1, 8)
                eng.denoise_step(q, zero, table, c1, f1, e1, max_prefix_len=0)
                out.append((c1[0], f1[0], e1[0]))
        for a, b in zip(*out):
            assert torch.equal(a, b), (a, b)
        assert 0.0 < float(out[0][1][0]) < 1.0
    assert eng.read_status() == 0
    eng.close()


@pytest.mark.parametrize("ms,Q", [(EDGE, 16), (EDGE, 32), (EDGE, 43), (EDGE, 120), (HALF, 43), (synth.TINY, 16)],
                         ids=["48-rows", "96-rows", "129-rows", "360-rows", "half-stage", "float-48-rows"])
def test_rows_that_are_not_finite_stay_to_themselves(ms, Q):
    """Infinities in one sequence (an embedding only it uses) and in the LM head's column of the mask token, which takes no
    part in the distribution, leave the other sequences' outputs as they are, bit for bit: also where the end of a row is
    copied next to the beginning of another.  The sequence itself, all NaN, reports confidences that no threshold accepts
    and candidates that are token ids."""
    w = synth.Weights(ms, 6)
    B, pt = 3, 16
    mp = (Q + pt - 1) // pt
    eng = H.make_engine(ms, w, page_tokens=pt, max_pages_per_seq=mp, n_pages=B * mp, max_batch=B, max_q=Q)
    table, zero = eng.i32(H.identity_table(eng, B)), eng.i32([0] * B)
    odd = 17
    q = np.stack([synth.masked_block(ms, 20 + b, Q, Q // 2) for b in range(B)])
    q[q == odd] = odd + 1
    q[1, 0] = q[1, -1] = odd
    out = []
    for poison in (False, True):
        if poison:
            eng.g["tok_emb"][odd] = float("inf")
            eng.g["lm_head"][ms.mask_id] = float("inf")
            if ms.dtype == "bf16":
                off = (-eng.packed.data_ptr()) % 256
                eng._check(binding.lib().dllm_pack_weights(eng.ctx, eng._stream(), eng.packed.data_ptr() + off, eng.packed.numel() - 256))
        cand = torch.zeros(B, Q, dtype=torch.int32, device=eng.device)
        conf, ent = (torch.zeros(B, Q, dtype=torch.float32, device=eng.device) for _ in range(2))
        eng.denoise_step(eng.i32(q), zero, table, cand, conf, ent, max_prefix_len=0)
        hidden = eng.debug_hidden(eng.i32(q), zero, table, ms.n_layers, max_prefix_len=0)
        out.append((cand, conf, ent, hidden))
    for a, b in zip(*out):
        assert torch.equal(a[0], b[0]) and torch.equal(a[2], b[2])
    cand, conf, _, hidden = out[1]
    masked = torch.from_numpy(q[1] == ms.mask_id).to(eng.device)
    assert torch.isfinite(hidden[::2]).all() and not torch.isfinite(hidden[1]).any()
    assert torch.isnan(conf[1][masked]).all() and torch.isfinite(out[0][1]).all()
    assert ((cand[1] >= 0) & (cand[1] < ms.vocab)).all() and (cand[1][masked] != ms.mask_id).all()
    eng.close()


# Products that took a tile they are slower in (us, the form below / that one): odd 128-row tiles at nearly three row tiles
# (89 / 97), 256 x 96 and 128 x 160 at a short K (17 / 19, 11 / 13), whole rounds for the sake of an odd rest (183 / 190), and residual projections
# in K shares of 256 x 224 where one launch of smaller tiles does (57 / 70, 45 / 61, 158 / 168, 56 / 75).
KEPT = [
    ("gate-up", 384, 12288, 4096, "256x256"), ("gate-up", 1000, 2752, 1024, "128x256"), ("gate-up", 256, 9216, 512, "128x256"),
    ("gate-up", 1152, 11008, 4096, "256x256"),
    ("resid", 1536, 4096, 4096, "128x256"), ("resid", 1552, 3584, 3584, "128x256"), ("resid", 6810, 3584, 3584, "128x256"),
    ("resid", 1424, 2048, 8192, "128x128"),
]

# (kind, rows, columns, K, form) of the products that the tests above are written for: tests/test_abi_host.py holds them against
# the library's own rules
FORMS = ([("gate-up", b * q, ff, d, form) for d, ff, (b, q), form in ODD_TILES + RESTS] +
         [("resid", b * q, d, heads * 64, o) for d, heads, ff, (b, q), o, down in RESID_224] +
         [("resid", b * q, d, ff, down) for d, heads, ff, (b, q), o, down in RESID_224] +
         [("gate-up", 8 * 127, 8512, 768, "64+128x128"), ("resid", 83 * 99, 2048, 768, "7+128x128"),
          ("gate-up", 8 * 127, 8544, 800, "64+128x128")] + KEPT +
         [(f"qkv:{hq}:{hkv}:{dh}", sum(lens), 0, d, form) for d, hq, hkv, dh, lens, n_cache, pt, form in ODD_ROPE] +
         [("qkv:48:8:64", 231, 0, 1792, "128x96"), ("qkv:48:8:64", 230, 0, 1792, "128x96"), ("qkv:34:2:128", 1050, 0, 2560, "256x96")] +
         [(f"qkv:{hq}:{hkv}:{dh}", n, 0, d, form) for d, hq, hkv, dh, lens, cap, *forms in ROPE_PAIRS for n, form in zip((sum(lens), cap), forms)] +
         [("resid", n, 1792, k, form) for n in (250, 300) for k, form in ((2304, "128x64/3"), (512, "128x64"))])

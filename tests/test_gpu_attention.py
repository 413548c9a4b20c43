"""GPU parity of the bfloat16 attention kernels at the edges of their key blocks, over caches that stress the running
softmax: keys whose scores grow along the sequence by far more than the kernels let the running maximum lag behind, and
pool slots past every sequence's end that hold NaN.  The reference is the oracle with bfloat16 storage on the same
cache; the tolerance is that of a one-layer model (tests/harness.py: logit_tol)."""
import numpy as np
import pytest
import torch

from oracle import dllm_oracle as O
from paper_2601_07568_amd import binding, synth
from tests import harness as H

pytestmark = pytest.mark.gpu
W = synth.as_float
ST = synth.round_bf16


def shape(hq, hkv, dh):
    return synth.ModelShape(1, 256, hq, hkv, dh, 512, 700, 699, dtype="bf16", lm_head_scale=8.0, name=f"attn-{hq}-{hkv}-{dh}")


# 7 and 4 heads a key head: seven and four groups of 32 query rows at 32 rows a sequence, one per wave; 1: the few-row
# kernels
SHAPES = {"g7-128": shape(7, 1, 128), "g4-128": shape(8, 2, 128), "g7-64": shape(7, 1, 64), "g8-64": shape(8, 1, 64),
          "g1-128": shape(2, 2, 128), "g1-64": shape(3, 3, 64)}
# prefixes: keys (prefix + rows) on both sides of 32 and 64, inside and past a page, several blocks per workgroup
LENS = {32: [0, 1, 31, 33, 95, 97, 480, 1500], 40: [0, 23, 24, 25, 88, 300], 64: [0, 63, 65, 700], 100: [28, 29, 155, 400]}


@pytest.mark.parametrize("name,Q,pt", [("g7-128", 32, 64), ("g7-128", 32, 8), ("g7-128", 40, 32), ("g4-128", 32, 128), ("g4-128", 64, 16),
                                       ("g7-64", 32, 64), ("g8-64", 40, 8), ("g8-64", 64, 256), ("g1-128", 32, 64), ("g1-128", 40, 24),
                                       ("g1-128", 64, 32), ("g1-128", 100, 64), ("g1-64", 100, 16)])
@pytest.mark.parametrize("ramp", [1.0, 60.0])
def test_key_block_edges_growing_scores_and_nan_slots(name, Q, pt, ramp):
    ms, lens = SHAPES[name], LENS[Q]
    B = len(lens)
    w = synth.Weights(ms, 3)
    mp = (max(lens) + Q + pt - 1) // pt + 1
    eng = H.make_engine(ms, w, page_tokens=pt, max_pages_per_seq=mp, n_pages=B * mp, max_batch=B, max_q=Q, max_tokens=0)
    rng = np.random.default_rng(17)
    table = H.identity_table(eng, B, perm=rng.permutation(B * mp))
    eng.kv_pool.view(torch.bfloat16).fill_(float("nan"))
    ks, vs = eng.kv_slab(0, 0), eng.kv_slab(0, 1)
    cache = []
    for b, n in enumerate(lens):
        size = np.geomspace(1.0, ramp, max(n, 1))[:n, None, None]
        k = ST(rng.standard_normal((n, ms.n_kv_heads, ms.head_dim)) * size)
        v = ST(rng.standard_normal((n, ms.n_kv_heads, ms.head_dim)))
        for p0 in range(0, n, pt):
            m = min(pt, n - p0)
            page = int(table[b, p0 // pt])
            ks[page, :, :m] = torch.as_tensor(np.asarray(k[p0:p0 + m]).transpose(1, 0, 2).copy()).to(eng.device, torch.bfloat16)
            vs[page, :, :m] = torch.as_tensor(np.asarray(v[p0:p0 + m]).transpose(1, 0, 2).copy()).to(eng.device, torch.bfloat16)
        cache.append(([k], [v]))
    blks = [synth.masked_block(ms, 30 + b, Q, Q // 2) for b in range(B)]
    hidden = eng.debug_hidden(eng.i32(np.stack(blks)), eng.i32(lens), eng.i32(table), 1, max_prefix_len=max(lens)).cpu().numpy()
    tol = H.logit_tol("bf16", 1, "store")
    for b in range(B):
        _, x = O.forward_cached(w, blks[b], *cache[b], widen=W, store=ST, want_logits=False)
        err = H.rel_err_rows(hidden[b], x).max()
        assert err <= tol, (lens[b], err)
    assert eng.read_status() == 0
    eng.close()


@pytest.mark.parametrize("B", [1, 293])
def test_more_page_ids_than_a_workgroup_keeps(B):
    """One sequence of 66000 keys in pages of 8 (8250 page ids, of which LDS holds 8192 beside the ring), alone and first of
    many short ones, where it would be a single unit along the keys.  The pages repeat: a pool of 64 stands for all of them."""
    ms, Q, pt, n = SHAPES["g7-128"], 32, 8, 66000
    w = synth.Weights(ms, 4)
    lens = [n] + [40] * (B - 1)
    mp, pool, own = (n + Q) // pt, 64, Q // pt
    rng = np.random.default_rng(23)
    eng = H.make_engine(ms, w, page_tokens=pt, max_pages_per_seq=mp, n_pages=pool + B * own, max_batch=B, max_q=Q, max_tokens=0)
    table = rng.integers(0, pool, (B, mp)).astype(np.int32)
    for b, k in enumerate(lens):
        table[b, k // pt:k // pt + own] = pool + b * own + np.arange(own)
    eng.kv_pool.view(torch.bfloat16).fill_(float("nan"))
    k, v = (ST(rng.standard_normal((pool, ms.n_kv_heads, pt, ms.head_dim))) for _ in range(2))
    for which, x in ((0, k), (1, v)):
        eng.kv_slab(0, which)[:pool] = torch.as_tensor(np.asarray(x)).to(eng.device, torch.bfloat16)
    blks = [synth.masked_block(ms, 30 + b, Q, Q // 2) for b in range(B)]
    hidden = eng.debug_hidden(eng.i32(np.stack(blks)), eng.i32(lens), eng.i32(table), 1, max_prefix_len=n).cpu().numpy()
    for b in {0, B // 2, B - 1}:
        cache = [[np.asarray(x)[table[b, :lens[b] // pt]].transpose(0, 2, 1, 3).reshape(lens[b], ms.n_kv_heads, ms.head_dim)] for x in (k, v)]
        _, x = O.forward_cached(w, blks[b], *cache, widen=W, store=ST, want_logits=False)
        err = H.rel_err_rows(hidden[b], x).max()
        assert err <= H.logit_tol("bf16", 1, "store"), (b, err)
    assert eng.read_status() == 0
    eng.close()


def _many(lens, n):
    return [lens[b % len(lens)] for b in range(n)]


# (shape, rows, page, prefixes): a workgroup per row group, keys in parts of single waves and of four that merge, with one part and
# several, and a part that a short sequence leaves empty; grouped queries with room for a workgroup per row group; and, with more
# row groups than CUs, the staged kernel for seven to ten of them; between one and two rounds of row groups long sequences in one
# workgroup each.  Last: the form as host_check prints it
FORMS = {
    "one-wave-64-parts": ("g1-128", 32, 64, [5000], "1:1x64"),
    "four-waves-8-parts": ("g1-64", 32, 64, [3000, 64, 700, 33, 2000, 0, 1500, 31], "4:1x8"),
    "four-waves-8-parts-page-24": ("g1-64", 32, 24, [3000, 64, 700, 33, 2000, 0, 1500, 31], "4:1x8"),
    "four-waves-1-part": ("g1-128", 32, 32, _many([200, 224, 0, 150, 31], 72), "4:1x1"),
    "one-wave-1-part": ("g1-128", 32, 32, _many([300, 31, 100], 230), "1:1x1"),
    "one-wave-1-part-second-round": ("g1-128", 32, 32, _many([200, 224, 0, 150, 31], 129), "1:1x1"),
    "four-waves-1-part-long": ("g1-128", 32, 32, _many([1100, 3, 40, 0, 64], 150), "4:1x1"),
    "two-row-groups-long": ("g1-128", 64, 64, _many([3300, 5, 64, 700], 75), "1:2x6"),
    "two-row-groups": ("g1-128", 64, 64, [1237, 5, 64], "1:1x16"),
    "two-row-groups-48": ("g1-128", 48, 96, [4000, 77], "1:1x32"),
    "three-row-groups": ("g1-64", 72, 128, [2500, 600, 9], "4:1x8"),
    "grouped-one-sequence": ("g7-128", 32, 64, [2048], "1:1x32"),
    "grouped-7500-keys": ("g7-64", 32, 64, [24000], "4:1x32"),
    "staged-7": ("g7-128", 32, 8, _many([480, 31, 33, 1500, 0], 40), "staged:7x6"),
    "staged-7-64": ("g7-64", 32, 64, _many([480, 31, 33, 1500, 0], 40), "staged:7x6"),
    "staged-8": ("g4-128", 64, 16, _many([63, 65, 700, 0], 17), "staged:8x3"),
    "staged-10": ("g8-64", 40, 8, _many([23, 24, 88, 300], 30), "staged:8x2"),
    # two parts of at least 4096 (token, head) rows
    "two-parts-4096-rows": ("g1-128", 32, 32, _many([60, 31, 0, 33], 64), "1:1x2"),
    "two-parts-4096-rows-64": ("g8-64", 32, 32, _many([60, 31, 0, 33], 16), "1:1x2"),
    "staged-two-parts": ("g7-128", 32, 32, _many([400, 31, 255, 0], 37), "staged:7x2"),
}


@pytest.mark.parametrize("form", FORMS)
def test_forms_of_the_launch(form, monkeypatch):
    name, Q, pt, lens, _ = FORMS[form]
    monkeypatch.setitem(LENS, Q, lens)
    test_key_block_edges_growing_scores_and_nan_slots(name, Q, pt, 20.0)


@pytest.mark.parametrize("n", [70, 130, 500, 3000, 9000])
@pytest.mark.parametrize("where", ["first", "last"])
def test_a_key_that_is_not_a_number_shows_in_every_row_of_its_sequence(n, where):
    """One NaN among the cached keys of the second of two sequences, in two, three, eight and more parts along the keys: all of that
    sequence's rows become NaN, the other's stay as they are, bit for bit."""
    ms, Q, pt = SHAPES["g1-128"], 32, 32
    w = synth.Weights(ms, 5)
    mp = (n + Q + pt - 1) // pt
    out = []
    for poison in (False, True):
        eng = H.make_engine(ms, w, page_tokens=pt, max_pages_per_seq=mp, n_pages=2 * mp, max_batch=2, max_q=Q, max_tokens=0)
        gen = torch.Generator(device=eng.device)
        gen.manual_seed(3)
        eng.kv_pool.view(torch.bfloat16)[:].normal_(generator=gen)
        if poison:
            at = 0 if where == "first" else n - 1
            eng.kv_slab(0, 0)[mp + at // pt, 0, at % pt, 5] = float("nan")
            eng.kv_slab(0, 0)[mp + at // pt, 1, at % pt, 5] = float("nan")
        q = np.stack([synth.masked_block(ms, 40 + b, Q, Q // 2) for b in range(2)])
        out.append(eng.debug_hidden(eng.i32(q), eng.i32([n, n]), eng.i32(H.identity_table(eng, 2)), 1, max_prefix_len=n).clone())
        assert eng.read_status() == 0
        eng.close()
    assert torch.equal(out[0][0], out[1][0]) and torch.isfinite(out[0]).all()
    assert torch.isnan(out[1][1]).all()


def test_a_key_that_is_not_a_number_among_many_rows_of_two_parts():
    """As above for 64 sequences of 60 keys, two parts each (4096 rows to merge)."""
    ms, Q, pt, n, B = SHAPES["g1-128"], 32, 32, 60, 64
    w = synth.Weights(ms, 5)
    eng = H.make_engine(ms, w, page_tokens=pt, max_pages_per_seq=3, n_pages=3 * B, max_batch=B, max_q=Q, max_tokens=0)
    gen = torch.Generator(device=eng.device)
    gen.manual_seed(3)
    eng.kv_pool.view(torch.bfloat16)[:].normal_(generator=gen)
    q = eng.i32(np.stack([synth.masked_block(ms, 40 + b, Q, Q // 2) for b in range(B)]))
    table, pre = eng.i32(H.identity_table(eng, B)), eng.i32([n] * B)
    good = eng.debug_hidden(q, pre, table, 1, max_prefix_len=n).clone()
    assert torch.isfinite(good).all()
    for b, at in ((5, 0), (50, n - 1)):
        for head in range(ms.n_kv_heads):
            eng.kv_slab(0, 0)[3 * b + at // pt, head, at % pt, 7] = float("nan")
    bad = eng.debug_hidden(q, pre, table, 1, max_prefix_len=n)
    others = [b for b in range(B) if b not in (5, 50)]
    assert torch.isnan(bad[[5, 50]]).all() and torch.equal(bad[others], good[others])
    assert eng.read_status() == 0
    eng.close()


# Launches in which every score of a row is NaN, or every score but those of the block's own keys: single waves and four that merge,
# one, two, up to eight and more parts along the keys, and the staged kernel: (shape, rows, page, prefixes, form as host_check prints it)
ALL_NAN = {
    "one-wave-1-part": ("g1-128", 32, 32, [30], "1:1x1"),
    "one-wave-2-parts": ("g1-128", 32, 32, [70, 90], "1:1x2"),
    "one-wave-8-parts": ("g1-128", 32, 64, [500], "1:1x8"),
    "one-wave-32-parts": ("g1-128", 32, 64, [2000], "1:1x32"),
    "four-waves-1-part": ("g1-128", 32, 32, _many([200, 150, 224], 72), "4:1x1"),
    "four-waves-2-parts": ("g1-128", 32, 32, _many([600, 550], 50), "4:1x2"),
    "four-waves-8-parts": ("g1-64", 32, 64, _many([3000, 2500], 8), "4:1x8"),
    "four-waves-16-parts": ("g1-128", 32, 64, _many([5000, 4200], 8), "4:1x16"),
    "two-parts-4096-rows": ("g1-128", 32, 32, _many([60, 40], 64), "1:1x2"),
    "staged-1-unit": ("g7-128", 32, 8, _many([60, 50], 300), "staged:7x1"),
    "staged-2-units": ("g7-128", 32, 32, _many([400, 300], 37), "staged:7x2"),
    "staged-24-units": ("g4-128", 32, 16, [1500], "staged:4x24"),
}


@pytest.mark.parametrize("poison", ["query", "keys"])
@pytest.mark.parametrize("form", ALL_NAN)
def test_rows_without_a_score_that_is_a_number_are_nan(form, poison):
    """A channel of the query projection that is NaN, or all cached keys: the rows come out NaN from every form of the launch, not
    zero from those that take an attention part without a finite maximum for an empty one."""
    name, Q, pt, lens, _ = ALL_NAN[form]
    ms, B = SHAPES[name], len(lens)
    w = synth.Weights(ms, 5)
    mp = (max(lens) + Q + pt - 1) // pt
    eng = H.make_engine(ms, w, page_tokens=pt, max_pages_per_seq=mp, n_pages=B * mp, max_batch=B, max_q=Q, max_tokens=0)
    gen = torch.Generator(device=eng.device)
    gen.manual_seed(3)
    eng.kv_pool.view(torch.bfloat16)[:].normal_(generator=gen)
    if poison == "keys":
        eng.kv_slab(0, 0).fill_(float("nan"))
    else:
        eng.layers[0]["wq"][5::ms.head_dim] = float("nan")
        off = (-eng.packed.data_ptr()) % 256
        eng._check(binding.lib().dllm_pack_weights(eng.ctx, eng._stream(), eng.packed.data_ptr() + off, eng.packed.numel() - 256))
    q = eng.i32(np.stack([synth.masked_block(ms, 40 + b, Q, Q // 2) for b in range(B)]))
    hidden = eng.debug_hidden(q, eng.i32(lens), eng.i32(H.identity_table(eng, B)), 1, max_prefix_len=max(lens))
    assert torch.isnan(hidden).all(), int(torch.isfinite(hidden).sum())
    assert eng.read_status() == 0
    eng.close()


# (kind, sequences, rows of each, longest prefix, form): tests/test_abi_host.py holds them against the library's own rules
def _planned(shape_name, Q, pt, lens, form):
    ms = SHAPES[shape_name]
    return f"attn:{ms.n_q_heads}:{ms.n_kv_heads}:{ms.head_dim}:{pt}", len(lens), Q, max(lens), form


PLANS = [_planned(*f) for f in (*FORMS.values(), *ALL_NAN.values())]

"""GPU parity of the weight-streaming kernels' forms that the small models of the other tests do not reach: gate/up with
three tile pairs per workgroup (d_ff of at least 9216), the q/k/v product with the value tiles beside the rotary pairs
(many heads) and in workgroups of their own (few key heads), the latter also at 65 .. 128 rows behind a norm that writes in
fragment order, at row counts on both sides of every 16-row tile and at sums with no, one and several stages per wave and a
ragged end.  Reference and tolerance as in test_gpu_gemm_tiles.py."""
import numpy as np
import pytest
import torch

from paper_2601_07568_amd import synth
from tests import harness as H
from tests.test_gpu_gemm_tiles import run

pytestmark = pytest.mark.gpu


def shape(d, hq, hkv, dh, ff, vocab=600):
    return synth.ModelShape(1, d, hq, hkv, dh, ff, vocab, vocab - 1, dtype="bf16", lm_head_scale=8.0, name=f"forms-{d}-{hq}-{hkv}-{ff}")


# 577 tile pairs: the last workgroup has one of three; d_model 104: no whole 128, a ragged last stage
WIDE = shape(104, 2, 2, 64, 9232)
# 33 stages of 32: one to five a wave; 580 pairs
DEEP = shape(1056, 4, 1, 64, 9280)
# 192 pair tiles and 192 value tiles (three tiles per workgroup)
HEADS = shape(136, 24, 24, 128, 320)
# 72 pair tiles, 8 value tiles in four workgroups
GROUPED = shape(264, 17, 1, 128, 320)


@pytest.mark.parametrize("B,Q", [(1, 7), (1, 17), (1, 32), (3, 11), (1, 48), (7, 7), (2, 32)])
@pytest.mark.parametrize("ms", [WIDE, DEEP, HEADS, GROUPED], ids=["wide", "deep", "heads", "grouped"])
def test_rows_of_a_step(ms, B, Q):
    run(ms, [40 + 9 * b for b in range(B)], Q)


# 240 workgroups of the q/k/v product, value tiles apart, K that leaves a rest of 1024: short stages up to 32 rows; K without one
@pytest.mark.parametrize("B,Q", [(1, 1), (1, 16), (1, 17), (4, 8), (3, 11)])
@pytest.mark.parametrize("d,hq,hkv,dh", [(264, 40, 40, 64), (1096, 72, 24, 64), (2088, 20, 20, 128), (1024, 40, 40, 64)])
def test_qkv_of_few_rows_on_nearly_all_compute_units(B, Q, d, hq, hkv, dh):
    run(shape(d, hq, hkv, dh, 256), [40 + 9 * b for b in range(B)], Q)


@pytest.mark.parametrize("B,Q", [(1, 65), (1, 80), (3, 27), (1, 96), (1, 111), (4, 32), (1, 129)])
@pytest.mark.parametrize("ms", [DEEP, HEADS, GROUPED], ids=["deep", "heads", "grouped"])
def test_qkv_of_65_to_128_rows(ms, B, Q):
    run(ms, [40 + 9 * b for b in range(B)], Q)


# wide gate/up products of short sums over row counts on both sides of 128 and 256 (the odd tiles: test_gpu_gemm_tiles.py)
@pytest.mark.parametrize("rows", [(1, 65), (1, 128), (3, 43), (1, 160), (2, 128), (3, 100)])
@pytest.mark.parametrize("d,ff", [(192, 12352), (512, 12352), (192, 18944)])
def test_wide_gate_up(d, ff, rows):
    run(shape(d, 2, 2, 64, ff), [5 + b for b in range(rows[0])], rows[1])


@pytest.mark.parametrize("B,Q", [(1, 65), (3, 32), (1, 128), (1, 129)])
@pytest.mark.parametrize("ms", [DEEP, HEADS, GROUPED], ids=["deep", "heads", "grouped"])
def test_steps_of_more_than_64_rows_read_the_weights_as_given(ms, B, Q):
    """Layer weights changed in place behind dllm_pack_weights: a step of more than 64 rows is that of an engine which has had
    the new weights from the start, packed or not, bit for bit (the packed copy is for steps of at most 64 rows)."""
    def engine(w, **kw):
        return H.make_engine(ms, w, page_tokens=32, max_pages_per_seq=5, n_pages=5 * B, max_batch=B, max_q=Q, **kw)

    def step(eng):
        rng = np.random.default_rng(2)
        q = np.stack([synth.masked_block(ms, 7 + b, Q, Q // 2) for b in range(B)])
        table = eng.i32(H.identity_table(eng, B, rng.permutation(5 * B)))
        eng.kv_pool.zero_()
        hidden = eng.debug_hidden(eng.i32(q), eng.i32([0] * B), table, 1, max_prefix_len=0)
        assert eng.read_status() == 0
        return hidden, eng.kv_pool.clone()

    new = engine(synth.Weights(ms, 9))
    want = step(new)
    plain = engine(synth.Weights(ms, 9), pack=False)
    changed = engine(synth.Weights(ms, 3))
    before = step(changed)
    changed.g["tok_emb"].copy_(new.g["tok_emb"])
    for name, t in changed.layers[0].items():
        t.copy_(new.layers[0][name])
    for eng in (changed, plain):
        for a, b in zip(step(eng), want):
            assert torch.equal(a, b)
    assert not torch.equal(before[0], want[0])
    for eng in (new, plain, changed):
        eng.close()

"""GPU parity of the float kernels for steps of at most 64 rows at the edges of their tiles: 1 .. 64 rows, widths that are no
multiple of 16 (model, MLP, vocabulary), both head sizes, grouped heads, pages of 4 tokens, prefixes around the 16-key
tiles and the eight waves that share them, padding rows.  Reference: the float64 oracle; tolerance: float (1e-4 per row of
logits, tests/harness.py)."""
import numpy as np
import pytest
import torch

from oracle import dllm_oracle as O
from paper_2601_07568_amd import synth
from tests import harness as H

pytestmark = pytest.mark.gpu
ODD = synth.ModelShape(2, 196, 4, 2, 64, 300, 1003, 1002, dtype="f32", lm_head_scale=8.0, name="odd-f32")
WIDE = synth.ModelShape(1, 1040, 3, 1, 128, 2052, 515, 514, dtype="f32", lm_head_scale=8.0, name="wide-f32")
# 130 workgroups of 16 residual or gate/up columns, 144 of rotary pairs, 129 of 64 vocabulary columns: with more than one row tile
# more than the 256 compute units hold at a time, so a workgroup keeps all rows (narrower models have one for every 16 rows)
BIG = synth.ModelShape(1, 2068, 32, 4, 128, 2068, 8250, 8249, dtype="f32", lm_head_scale=8.0, name="big-f32")
BIG_64 = synth.ModelShape(1, 2080, 66, 33, 64, 4100, 8200, 8199, dtype="f32", lm_head_scale=8.0, name="big-f32-64")


@pytest.mark.parametrize("ms,lens,Q,pt", [(BIG, [17], 17, 8), (BIG, [40], 32, 16), (BIG, [5, 0, 33], 16, 16), (BIG, [20, 64], 32, 32),
                                          (BIG_64, [3], 32, 4), (BIG_64, [9], 33, 16), (BIG_64, [16, 2, 7], 17, 8),
                                          (ODD, [1], 1, 4), (ODD, [15, 16, 17], 7, 4), (ODD, [130], 64, 16), (ODD, [31], 33, 8),
                                          (WIDE, [127, 1], 16, 16), (WIDE, [300], 48, 12), (WIDE, [0, 5], 32, 32)])
def test_float_step_around_the_tiles(ms, lens, Q, pt):
    w = synth.Weights(ms, 4)
    B = len(lens)
    mp = (max(lens) + Q + pt - 1) // pt
    eng = H.make_engine(ms, w, page_tokens=pt, max_pages_per_seq=mp, n_pages=B * mp, max_batch=B, max_q=Q,
                        max_tokens=max(1, sum(lens)))
    perm = np.random.default_rng(2).permutation(B * mp)
    table = H.identity_table(eng, B, perm)
    dt = eng.i32(table)
    seqs = [synth.random_tokens(ms, 3 + i, n) if n else np.zeros(0, np.int32) for i, n in enumerate(lens)]
    blks = [synth.masked_block(ms, 13 + i, Q, (Q + 1) // 2) for i in range(B)]
    if sum(lens):
        cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
        eng.prefill_kv(eng.i32(np.concatenate(seqs).astype(np.int32)), eng.i32(cu), dt, None, total_tokens=int(cu[-1]), max_seqlen=max(lens))
    qt, pre = eng.i32(np.stack(blks)), eng.i32(lens)
    logits = eng.debug_logits(qt, pre, dt, max_prefix_len=max(lens)).cpu().numpy()
    cand = torch.zeros(B, Q, dtype=torch.int32, device=eng.device)
    conf = torch.zeros(B, Q, dtype=torch.float32, device=eng.device)
    ent = torch.zeros(B, Q, dtype=torch.float32, device=eng.device)
    eng.denoise_step(qt, pre, dt, cand, conf, ent, max_prefix_len=max(lens))
    for b in range(B):
        if lens[b]:
            ck, cv = O.prefill(w, seqs[b])
        else:
            shape = (0, ms.n_kv_heads, ms.head_dim)
            ck = cv = [np.zeros(shape) for _ in range(ms.n_layers)]
        z, x = O.forward_cached(w, blks[b], ck, cv)
        assert H.rel_err_rows(logits[b], z).max() <= 1e-4
        r = {"logits": z, "cand": O.confidence(z, ms.mask_id)[0]}
        H.check_step_outputs(ms, r, blks[b] == ms.mask_id, cand.cpu().numpy()[b], conf.cpu().numpy()[b], ent.cpu().numpy()[b],
                             "f32", gpu_logits=logits[b])
    assert eng.read_status() == 0
    # padding rows: the valid rows' outputs are those of a call without the others, bit for bit
    if Q > 2:
        valid = eng.i32([max(1, Q - 2 - b) for b in range(B)])
        c2, f2 = torch.zeros_like(cand), torch.zeros_like(conf)
        eng.denoise_step_var(qt, pre, valid, dt, c2, f2, None, max_prefix_len=max(lens))
        n0 = max(1, Q - 2)
        c3 = torch.zeros(1, n0, dtype=torch.int32, device=eng.device)
        f3 = torch.zeros(1, n0, dtype=torch.float32, device=eng.device)
        eng.denoise_step(qt[:1, :n0].contiguous(), pre[:1], dt[:1], c3, f3, None, max_prefix_len=lens[0])
        assert torch.equal(c2[0, :n0], c3[0]) and torch.equal(f2[0, :n0], f3[0])
    eng.close()


def test_profile_of_a_float_step_records_what_the_generic_kernels_record():
    """dllm_profile_read after a step on the few-row kernels: launches and work of every class as on the generic ones."""
    ms = synth.TINY
    eng = H.make_engine(ms, synth.Weights(ms, 1), page_tokens=16, max_pages_per_seq=4, n_pages=4, max_batch=1, max_q=32)
    table, zero = eng.i32(H.identity_table(eng, 1)), eng.i32([0])
    q = eng.i32([synth.masked_block(ms, 3, 32, 16)])
    cand = torch.zeros(1, 32, dtype=torch.int32, device=eng.device)
    conf = torch.zeros(1, 32, dtype=torch.float32, device=eng.device)
    got = []
    for mode in (1, 0):
        eng.set_kernel_mode(mode)
        eng.profile_enable(True)
        eng.denoise_step(q, zero, table, cand, conf, None, max_prefix_len=0)
        got.append([eng.profile_read(cls)[::2] for cls in range(6)])
        eng.profile_enable(False)
    assert got[0] == got[1] and got[1][0][0] == got[1][5][0] == ms.n_layers, got
    eng.close()

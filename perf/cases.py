"""What is measured when this library's speed is judged: the forwards a decoding program makes, through the binding.

A case is a dict of plain values:
  model   "tiny" (float32, 2 layers), "llada8b" or "dream7b" (bfloat16, the shapes of paper_2601_07568_amd.synth)
  call    "step"     dllm_denoise_step of the model cut to `layers` layers, LM head included (the tiny model: with the
                     unmask selection behind it, as its decode loop does)
          "layers"   the same forward without the LM head (dllm_debug_hidden): the layers of a denoise step alone
          "refresh"  dllm_refresh_cache with the step outputs of the in-flight rows
          "prefill"  dllm_prefill_kv
  layers  depth.  The full models have 32 and 28 layers of these shapes; a cut keeps inputs quick to make and the
          outputs within what bfloat16 storage lets two correct implementations agree on.
  batch   sequences;  rows: query rows per sequence ("step", "layers") or in-flight rows ("refresh")
  length  the longest prefix ("step", "layers") or sequence ("refresh", "prefill"); the others are up to a quarter shorter
  masked  share of the query rows that hold the mask token;  page: tokens per cache page

Weights are N(0, 0.02) with gains around one, tokens uniform, cached keys and values N(0, 1), pages of the pool in random
order: what the repository's benchmark and tests use.  The candidate tokens of bfloat16 steps are not among the outputs:
with random weights the gap between the two largest of 126 thousand logits is often below what a change of summation
order moves, so they would say nothing; their probabilities, the entropies and the keys and values written are.
"""
import math

import torch

from paper_2601_07568_amd import synth
from paper_2601_07568_amd.binding import Engine

MODELS = {"tiny": synth.TINY, "llada8b": synth.LLADA_8B, "dream7b": synth.DREAM_7B}


def _case(name, model, call, layers, batch, rows, length, masked=0.75, page=64):
    c = {"model": model, "call": call, "layers": layers, "batch": batch, "rows": rows, "length": length, "masked": masked,
         "page": page}
    return dict(c, name=name) if name else c


def listed():
    return [
        # the float32 model of the tests, one step of its decode: the smallest call, all latency and launches
        _case("tiny_step", "tiny", "step", 2, 1, 32, 64, 0.75, 32),
        # the headline workload: one block of one sequence against a 1024-token prompt
        _case("8b_step", "llada8b", "step", 8, 1, 32, 1024, 1.0),
        # one layer and the LM head at prefix 512: the head of a batch-1 step
        _case("8b_layer_and_head", "llada8b", "step", 1, 1, 32, 512),
        # multi-block decoding at batch 1: two and four blocks in flight, a prefix that ends inside a page
        _case("8b_two_blocks", "llada8b", "layers", 4, 1, 64, 1237),
        _case("8b_four_blocks", "llada8b", "layers", 4, 1, 128, 901),
        # a small serving batch on the multi-head model, ragged prefixes, the binding's default page size
        _case("8b_batch8", "llada8b", "layers", 4, 8, 32, 700, 0.75, 32),
        # the grouped-query model at batch 1
        _case("dream_step_b1", "dream7b", "layers", 4, 1, 32, 2048),
        # 16 sequences with two blocks in flight each
        _case("dream_two_blocks_b16", "dream7b", "layers", 4, 16, 64, 2048, 0.5),
        # the long-context batch: 32 sequences, 8192 cached tokens each, LM head on half of the 1024 rows
        _case("dream_long_step", "dream7b", "step", 4, 32, 32, 8192, 0.5),
        # the cache refresh at a block boundary of the headline workload, with the outputs of the block in flight
        _case("8b_refresh", "llada8b", "refresh", 4, 1, 32, 1184, 1.0),
        # a short prompt
        _case("8b_prefill_short", "llada8b", "prefill", 8, 1, 0, 211),
        # a batch of long prompts: the largest call
        _case("dream_prefill", "dream7b", "prefill", 8, 8, 0, 2048),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["tiny", "batch1", "batch1", "blocks", "batch", "batch", "packed", "packed"])
    page = rng.choice([32, 64, 64, 128])
    masked = rng.choice([0.25, 0.5, 0.75, 1.0])
    if kind == "tiny":
        return _case(None, "tiny", "step", 2, 1, rng.choice([16, 32, 64]), _log_int(rng, 8, 480), masked, rng.choice([16, 32]))
    model = rng.choice(["llada8b", "dream7b"])
    call = rng.choice(["step", "layers"])
    layers = rng.randint(2, 4)
    if kind == "batch1":
        return _case(None, model, call, layers, 1, rng.choice([8, 16, 24, 32, 32, 32, 48, 64]), _log_int(rng, 64, 8192), masked, page)
    if kind == "blocks":
        return _case(None, model, call, layers, rng.randint(1, 3), rng.choice([32, 64, 72]) + 8 * rng.randint(0, 4), _log_int(rng, 64, 4096), masked,
                     page)
    if kind == "batch":
        batch, rows = _log_int(rng, 4, 32), rng.choice([32, 32, 64])
        batch = min(batch, 1024 // rows)
        most = 262144 if model == "dream7b" else 32768          # cached tokens of the call
        return _case(None, model, call, layers, batch, rows, _log_int(rng, 64, max(128, min(8192, most // batch))), masked, page)
    if rng.random() < 0.5:
        return _case(None, model, "refresh", layers, rng.randint(1, 2), rng.choice([32, 64]), _log_int(rng, 128, 1600), 1.0, page)
    batch = _log_int(rng, 1, 8)
    return _case(None, model, "prefill", layers, batch, 0, _log_int(rng, 33, 2048), 1.0, page)


# --------------------------------------------------------------------------------------------------- inputs

def _shape(case):
    return MODELS[case["model"]].with_layers(case["layers"])


def _lengths(case):
    """Prefix (or sequence) lengths: the first is the longest, the others up to a quarter shorter."""
    n = case["length"]
    return [n - (37 * b) % (1 + n // 4) for b in range(case["batch"])]


def _masked_rows(case):
    return max(1, int(round(case["masked"] * case["rows"]))) if case["rows"] else 0


def _weights(ms, gen, dev):
    dt = torch.bfloat16 if ms.dtype == "bf16" else torch.float32

    def mat(rows, cols, std=0.02):
        return torch.randn(rows, cols, generator=gen, device=dev, dtype=torch.float32).mul_(std).to(dt)

    def gain():
        return (1 + 0.1 * torch.randn(ms.d_model, generator=gen, device=dev, dtype=torch.float32)).to(dt)

    d, dq, dkv, f = ms.d_model, ms.n_q_heads * ms.head_dim, ms.n_kv_heads * ms.head_dim, ms.d_ff
    g = {"tok_emb": mat(ms.vocab, d), "lm_head": mat(ms.vocab, d, 0.02 * ms.lm_head_scale), "final_norm": gain()}
    layers = [{"attn_norm": gain(), "wq": mat(dq, d), "wk": mat(dkv, d), "wv": mat(dkv, d), "wo": mat(d, dq),
               "mlp_norm": gain(), "w_gate": mat(f, d), "w_up": mat(f, d), "w_down": mat(d, f)} for _ in range(ms.n_layers)]
    return g, layers


def _pool_pages(case):
    """(pages per sequence, per-sequence count of pages whose positions all precede the prefix end, pages in the pool)"""
    pt, q = case["page"], case["rows"] if case["call"] in ("step", "layers") else 0
    lens = _lengths(case)
    per_seq = [(n + q + pt - 1) // pt for n in lens]
    full = [n // pt for n in lens] if q else [0] * len(lens)
    return per_seq, full, sum(per_seq)


def _inputs(case, seed, dev):
    """Everything the call reads, drawn from the seed: weights, pool contents, tokens, block table, lengths."""
    ms = _shape(case)
    gen = torch.Generator(device=dev)
    gen.manual_seed(int(seed))
    cpu = torch.Generator()
    cpu.manual_seed(int(seed))
    g, layers = _weights(ms, gen, dev)
    per_seq, full, n_pages = _pool_pages(case)
    lens, mp = _lengths(case), max(per_seq)
    # physical pages in random order; the pages of the rows in flight come last, so that the keys and values a step
    # writes are one slice of the pool
    n_full = sum(full)
    old, new = torch.randperm(n_full, generator=cpu), n_full + torch.randperm(n_pages - n_full, generator=cpu)
    table = torch.zeros(case["batch"], mp, dtype=torch.int32)
    io = iw = 0
    for b, (n, k) in enumerate(zip(per_seq, full)):
        table[b, :k] = old[io:io + k]
        table[b, k:n] = new[iw:iw + n - k]
        io, iw = io + k, iw + n - k
    slab = n_pages * ms.n_kv_heads * case["page"] * ms.head_dim
    pool = torch.empty(max(1, 2 * ms.n_layers * slab), dtype=torch.bfloat16 if ms.dtype == "bf16" else torch.float32, device=dev)
    pool.normal_(generator=gen)
    if case["call"] in ("step", "layers"):
        tokens = torch.randint(0, ms.vocab - 1, (case["batch"], case["rows"]), generator=cpu, dtype=torch.int32)
        for b in range(case["batch"]):
            tokens[b, torch.randperm(case["rows"], generator=cpu)[:_masked_rows(case)]] = ms.mask_id
    else:
        tokens = torch.randint(0, ms.vocab - 1, (sum(lens),), generator=cpu, dtype=torch.int32)
        end = 0
        for n in lens:
            end += n
            q = min(case["rows"], n)
            tokens[end - q + torch.randperm(q, generator=cpu)[:_masked_rows(case)]] = ms.mask_id
    return {"ms": ms, "g": g, "layers": layers, "pool": pool, "table": table.to(dev), "lens": lens, "tokens": tokens.to(dev),
            "n_full": n_full, "n_pages": n_pages, "max_pages": mp}


def prepare(case, seed):
    dev = torch.device("cuda:0")
    s = _inputs(case, seed, dev)
    ms, lens, B = s["ms"], s["lens"], case["batch"]
    step = case["call"] in ("step", "layers")
    eng = Engine(ms, None, page_tokens=case["page"], max_pages_per_seq=s["max_pages"], n_pages=s["n_pages"], max_batch=B,
                 max_q=max(32, case["rows"]), max_tokens=0 if step else sum(lens), device_weights=(s["g"], s["layers"]))
    pool = eng.kv_pool.view(s["pool"].dtype)[:s["pool"].numel()]
    pool.copy_(s["pool"])
    s.update(eng=eng, case=case, pool=None, kv=pool.view(ms.n_layers, 2, s["n_pages"], -1)[:, :, s["n_full"]:], longest=max(lens))
    i32 = dict(dtype=torch.int32, device=dev)
    n_out = (B, case["rows"]) if step else (sum(lens),)
    s["cand"] = torch.zeros(n_out, **i32)
    s["conf"] = torch.zeros(n_out, dtype=torch.float32, device=dev)
    s["ent"] = torch.zeros(n_out, dtype=torch.float32, device=dev)
    s["work_tokens"] = s["tokens"].clone()
    if step:
        s["prefix"] = torch.tensor(lens, **i32)
    else:
        cu = [0]
        for n in lens:
            cu.append(cu[-1] + n)
        s["cu"], s["total"] = torch.tensor(cu, **i32), cu[-1]
        s["n_commit"] = torch.tensor([max(0, n - case["rows"]) for n in lens], **i32)
    return s


def run(s):
    eng, call = s["eng"], s["case"]["call"]
    if call == "step":
        q = s["tokens"]
        if s["case"]["model"] == "tiny":
            q = s["work_tokens"]
            q.copy_(s["tokens"])
        eng.denoise_step(q, s["prefix"], s["table"], s["cand"], s["conf"], s["ent"], max_prefix_len=s["longest"])
        out = {"conf": s["conf"], "entropy": s["ent"], "kv": s["kv"]}
        if s["case"]["model"] == "tiny":
            eng.unmask(q, s["cand"], s["conf"], 0.9, 1)
            out["cand"], out["tokens"] = s["cand"], q
        return out
    if call == "layers":
        hidden = eng.debug_hidden(s["tokens"], s["prefix"], s["table"], s["ms"].n_layers, max_prefix_len=s["longest"])
        return {"hidden": hidden, "kv": s["kv"]}
    if call == "refresh":
        eng.refresh_cache(s["tokens"], s["cu"], s["table"], s["n_commit"], s["cand"], s["conf"], s["ent"],
                          total_tokens=s["total"], max_seqlen=s["longest"])
        return {"conf": s["conf"], "entropy": s["ent"], "kv": s["kv"]}
    eng.prefill_kv(s["tokens"], s["cu"], s["table"], None, total_tokens=s["total"], max_seqlen=s["longest"])
    return {"kv": s["kv"]}


# --------------------------------------------------------------------------------------------------- what it costs

def work(case):
    """Weights, cached keys and values and outputs once each; the products of the rows that the outputs depend on."""
    ms, lens = _shape(case), _lengths(case)
    es = 2 if ms.dtype == "bf16" else 4
    d, dq, dkv, f = ms.d_model, ms.n_q_heads * ms.head_dim, ms.n_kv_heads * ms.head_dim, ms.d_ff
    step = case["call"] in ("step", "layers")
    rows = case["batch"] * case["rows"] if step else sum(lens)
    w_kv, w_rest = 2 * dkv * d, 2 * dq * d + 3 * f * d
    pairs = sum((n + case["rows"]) * case["rows"] for n in lens) if step else sum(n * n for n in lens)
    full = ms.n_layers - (1 if case["call"] == "prefill" else 0)    # a prefill needs no more than K and V of its last layer
    flops = 2.0 * rows * (ms.n_layers * w_kv + full * w_rest) + 4.0 * dq * pairs * full
    bytes_ = es * (ms.n_layers * w_kv + full * w_rest + rows * d)
    cached = sum(lens) if step else 0
    bytes_ += es * 2.0 * dkv * ms.n_layers * (cached + rows)
    if case["call"] == "layers":
        bytes_ += 4.0 * rows * d
    elif case["call"] != "prefill":
        n_lm = case["batch"] * _masked_rows(case)
        bytes_ += es * ms.vocab * d + 12.0 * rows
        flops += 2.0 * n_lm * ms.vocab * d
    return {"bytes": bytes_, "flops": flops}


def tolerance(case):
    if case["model"] == "tiny":
        return {"rel": 1e-5, "max": 1e-3, "differ": 0.0}
    # bfloat16 storage, float sums: a rounding that falls the other way travels through the layers behind it.  Measured
    # with the sums in another order (scalar kernels against matrix cores, three seeds): up to 0.0064 (largest single
    # difference 0.04) over 4 layers, 0.0069 (0.055) on keys and values and 0.014 on confidences over 8
    return {"rel": 0.025, "max": 0.2} if case["layers"] <= 4 else {"rel": 0.03, "max": 0.25}


# --------------------------------------------------------------------------------------------------- in 64 bits

def _norm(x, gain, eps):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + eps) * gain.double()


def _rope(x, pos, base):
    half = x.shape[-1] // 2
    ang = pos.double()[:, None] * base ** (-torch.arange(half, device=x.device, dtype=torch.float64) / half)
    c, s = torch.cos(ang)[:, None, :], torch.sin(ang)[:, None, :]
    a, b = x[..., :half], x[..., half:]
    return torch.cat([a * c - b * s, b * c + a * s], -1)


def _attend(q, k, v):
    """q [n, Hq, dh], k and v [m, Hkv, dh]: softmax attention without a mask, query heads in groups per key head."""
    n, hq, dh = q.shape
    hkv = k.shape[1]
    qg = q.reshape(n, hkv, hq // hkv, dh).permute(1, 2, 0, 3).reshape(hkv, -1, dh).contiguous()
    o = torch.empty_like(qg)
    kt, vv = k.permute(1, 2, 0).contiguous(), v.permute(1, 0, 2).contiguous()
    for h in range(hkv):
        o[h] = torch.softmax(qg[h] @ kt[h] / math.sqrt(dh), -1) @ vv[h]
    return o.reshape(hkv, hq // hkv, n, dh).permute(2, 0, 1, 3).reshape(n, hq * dh)


def exact(case, seed):
    dev = torch.device("cuda:0")
    s = _inputs(case, seed, dev)
    ms, lens, pt, call = s["ms"], s["lens"], case["page"], case["call"]
    hq, hkv, dh = ms.n_q_heads, ms.n_kv_heads, ms.head_dim
    step = call in ("step", "layers")
    n_rows = [case["rows"]] * case["batch"] if step else lens
    start = lens if step else [0] * len(lens)                     # position of a sequence's first row
    keep = [n + case["rows"] for n in lens] if step else [n - min(n, case["rows"]) for n in lens]   # positions cached after the call
    pos = torch.cat([torch.arange(a, a + n, device=dev) for a, n in zip(start, n_rows)])
    pool = s["pool"].view(ms.n_layers, 2, s["n_pages"], -1)
    out_kv = pool[:, :, s["n_full"]:].double()
    x = s["g"]["tok_emb"][s["tokens"].reshape(-1).long()].double()
    for l, w in enumerate(s["layers"]):
        h = _norm(x, w["attn_norm"], ms.rms_eps)
        q = _rope((h @ w["wq"].double().T).view(-1, hq, dh), pos, ms.rope_base)
        k = _rope((h @ w["wk"].double().T).view(-1, hkv, dh), pos, ms.rope_base)
        v = (h @ w["wv"].double().T).view(-1, hkv, dh)
        ks, vs = pool[l, 0].view(-1, hkv, pt, dh), pool[l, 1].view(-1, hkv, dh, pt)
        ok, ov = out_kv[l, 0].view(-1, hkv, pt, dh), out_kv[l, 1].view(-1, hkv, dh, pt)
        parts, at = [], 0
        for b, n in enumerate(n_rows):
            kb, vb, qb = k[at:at + n], v[at:at + n], q[at:at + n]
            pages = s["table"][b].long()
            if step:
                idx = pages[:(lens[b] + pt - 1) // pt]
                kp = ks[idx].permute(0, 2, 1, 3).reshape(-1, hkv, dh)[:lens[b]].double()
                vp = vs[idx].permute(0, 3, 1, 2).reshape(-1, hkv, dh)[:lens[b]].double()
                kb, vb = torch.cat([kp, kb]), torch.cat([vp, vb])
            p = torch.arange(start[b], keep[b], device=dev)
            pg = pages[p // pt] - s["n_full"]
            ok[pg, :, p % pt] = kb[p - (0 if step else start[b])]
            ov[pg, :, :, p % pt] = vb[p - (0 if step else start[b])]
            parts.append(_attend(qb, kb, vb))
            at += n
        x = x + torch.cat(parts) @ w["wo"].double().T
        h = _norm(x, w["mlp_norm"], ms.rms_eps)
        gate = h @ w["w_gate"].double().T
        x = x + (gate * torch.sigmoid(gate) * (h @ w["w_up"].double().T)) @ w["w_down"].double().T
        del gate
    if call == "layers":
        return {"hidden": x.view(case["batch"], case["rows"], -1), "kv": out_kv}
    if call == "prefill":
        return {"kv": out_kv}
    flat = s["tokens"].reshape(-1)
    shown = torch.ones_like(flat, dtype=torch.bool) if step else torch.cat(
        [torch.arange(n, device=dev) >= n - min(n, case["rows"]) for n in lens])
    conf = shown.double()
    ent = torch.zeros_like(conf)
    rows = torch.nonzero(shown & (flat == ms.mask_id))[:, 0]
    z = _norm(x[rows], s["g"]["final_norm"], ms.rms_eps) @ s["g"]["lm_head"].double().T
    z[:, ms.mask_id] = -math.inf
    logp = torch.log_softmax(z, -1)
    del z
    conf[rows] = logp.max(-1).values.exp()
    logp[:, ms.mask_id] = 0.0
    p = logp.exp()
    p[:, ms.mask_id] = 0.0
    ent[rows] = -(p * logp).sum(-1)
    out = {"conf": conf.view(s["tokens"].shape), "entropy": ent.view(s["tokens"].shape), "kv": out_kv}
    if case["model"] == "tiny":
        out["cand"] = out["tokens"] = None
    elif rows.numel() < 256:
        # a few dozen values whose bfloat16 errors share their causes: the size of that error is a draw, no measure
        out["conf"] = out["entropy"] = None
    return out

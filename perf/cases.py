"""The work this library is measured on: decode-attention steps through the public entry points, over the range of shapes
a serving or long-generation program gives them.

A case is one decoding step (or the end of a prefill) of `layers` attention layers that share one context, each with its
own K / V cache, queries and index sets, called layer after layer on one stream as a model's forward pass does:

  op "fast"    sfi_fast_step per layer (sparse attention over sink ++ selected ++ recent rows)
  op "slow"    sfi_slow_step per layer (dense attention, then the Selector's refreshed index set)
  op "dense"   sfi_dense_attn per layer (full attention, nothing selected)
  op "mixed"   a ragged batch in which `n_slow` sequences take a slow step and the others a fast one: sfi_mixed_step_desc
               (packed descriptor) per layer, or with `compact` sfi_mixed_step_compact (two-segment layout)
  op "window"  the end of a prefill: sfi_evidence_add_causal per window query (evidence only), then sfi_evidence_select

Contexts run from `ctx_lo` to `ctx_hi` rows in even steps over the batch (the seed decides which sequence has which), so
a case's work does not depend on the seed.  K, V and q are N(0, 1) in bf16 with `support` of the K rows scaled by 4, the
stand-in for the few stable positions that attention concentrates on.
"""
import math

import torch

import paper_2603_12038_amd as sfi
from paper_2603_12038_amd.binding import SfiContext

D = 128
N_SINK = 4
# hyper-parameters of the full Selector (mode 1)
FULL_SELECTOR = dict(gamma=0.5, beta=1.0, p=2.0, eta=0.5, lambda_clip=0.02, alpha_soft=0.5, alpha_cross=0.35, temp=1.0,
                     eps=1e-8, nms_radius=2)


def _case(op, batch, hq, hkv, ctx_lo, ctx_hi, budget, recent, layers=1, **more):
    c = dict(op=op, batch=batch, hq=hq, hkv=hkv, ctx_lo=ctx_lo, ctx_hi=ctx_hi, budget=budget, recent=recent, layers=layers,
             support=0.01, n_slow=0, window=0, selector=0, alpha=1.0, page=0, compact=False, out_bf16=False)
    assert set(more) <= set(c) | {"name"}
    c.update(more)
    return c


def listed():
    return [
        # one short chat stream on a small model, one layer: what a call costs when there is hardly any work
        _case("fast", 1, 8, 2, 4096, 4096, 256, 64, name="fast tiny"),
        _case("slow", 1, 8, 2, 4096, 4096, 256, 64, name="slow tiny"),
        # a few users of an 8B-class model at 32K: the ordinary fast step, and the slow step that refreshes it
        _case("fast", 4, 32, 8, 32768, 32768, 2048, 128, layers=8, name="fast llama8b"),
        _case("slow", 4, 32, 8, 32768, 32768, 2048, 128, layers=2, name="slow llama8b"),
        # one user with a very long document: few sequences to spread over the chip
        _case("fast", 1, 32, 8, 131072, 131072, 4096, 256, layers=8, support=0.016, name="fast long"),
        # ... and its slow step with the full Selector (prior, fusion, Soft-NMS, cross-head exclusivity)
        _case("slow", 1, 32, 8, 131071, 131071, 4096, 256, selector=1, support=0.016, name="slow long full selector"),
        # long chain-of-thought generation on a paged cache, outputs in the model's bf16, sequences of odd lengths
        _case("slow", 8, 40, 8, 20011, 24571, 1024, 128, page=16, support=0.0, out_bf16=True, name="slow cot paged"),
        _case("fast", 8, 40, 8, 20011, 24571, 1024, 128, layers=4, page=16, support=0.0, out_bf16=True, name="fast cot paged"),
        # high-batch serving: every sequence at its own length, two of them due for a refresh in this step
        _case("mixed", 32, 64, 8, 16384, 65536, 2048, 128, support=0.005, n_slow=2, name="mixed serving"),
        # the same kind of step over the two-segment layout, a smaller batch
        _case("mixed", 12, 32, 8, 5003, 30011, 1024, 128, layers=2, n_slow=1, compact=True, name="mixed compact"),
        # full attention for a batch at 16K (before the method is switched on, or with it off)
        _case("dense", 16, 32, 8, 16384, 16384, 0, 128, name="dense batch 16"),
        # the first index set of a request: evidence of the last 16 prompt tokens (power mean 1/2)
        _case("window", 2, 32, 8, 12000, 16384, 2048, 256, window=16, selector=1, alpha=0.5, name="window prefill"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges: batches of 1 to 32, contexts of 512 to 131072 rows, budgets of 64 to 4096."""
    while True:
        op = rng.choice(["fast", "fast", "fast", "slow", "slow", "slow", "mixed", "mixed", "dense", "window"])
        hkv = rng.choice([2, 4, 8, 8])
        hq = hkv * rng.choice([1, 2, 4, 4, 5, 7, 8, 16])
        batch = _log_int(rng, 1, 32)
        ctx_hi = _log_int(rng, 512, 131072)
        ctx_lo = int(ctx_hi * rng.choice([1.0, rng.uniform(0.25, 1.0)]))
        budget = min(_log_int(rng, 64, 4096), max(16, ctx_lo // 4))
        recent = rng.choice([64, 128, 128, 256, rng.randint(50, 300)])
        more = dict(layers=_log_int(rng, 1, 8), support=rng.choice([0.0, 0.005, 0.01]), page=rng.choice([0, 0, 16, 64]),
                    out_bf16=rng.random() < 0.3)
        if op == "slow":
            more.update(selector=rng.choice([0, 0, 1]), alpha=rng.choice([1.0, 1.0, 0.5]))
        elif op == "mixed":
            batch = max(batch, 2)
            more.update(n_slow=rng.randint(0, max(1, batch // 8)), compact=rng.random() < 0.3)
        elif op == "window":
            more.update(window=rng.randint(4, 16), selector=rng.choice([0, 1]), alpha=rng.choice([1.0, 0.5]), layers=1,
                        out_bf16=False)
        elif op == "dense":
            budget = 0
        c = _case(op, batch, hq, hkv, ctx_lo, ctx_hi, budget, recent, **more)
        cache = 4 * c["layers"] * batch * hkv * ctx_hi * D
        # no more work than the listed cases have, caches of at most 9 GB
        if cache <= 9e9 and work(c)["bytes"] <= 9e8:
            return c


def _lengths(c):
    """Context length of the sequence of each rank, shortest first."""
    n, lo, hi = c["batch"], c["ctx_lo"], c["ctx_hi"]
    return [hi if n == 1 else lo + (hi - lo) * i // (n - 1) for i in range(n)]


def _slow_ranks(c):
    """Which ranks take the slow step of a mixed case: spread over the lengths."""
    n, k = c["batch"], c["n_slow"]
    return {(2 * i + 1) * n // (2 * k) for i in range(k)} if k else set()


def _shape_cache(c, gen, lens):
    """One K and one V for every layer: [B, Hkv, L, d], or block pools [blocks, Hkv, page, d] with a block table."""
    b, hkv, n, layers = c["batch"], c["hkv"], c["ctx_hi"], c["layers"]
    page = c["page"]
    if page:
        per = (n + page - 1) // page
        shape = (layers, b * per, hkv, page, D)
        table = torch.randperm(b * per, generator=gen, device="cuda").to(torch.int32).view(b, per)
    else:
        shape, table = (layers, b, hkv, n, D), None
    K = torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    V = torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    if c["support"]:
        x4 = torch.rand(shape[:-1], generator=gen, device="cuda") < c["support"]
        K.mul_((1 + 3 * x4).to(torch.bfloat16).unsqueeze(-1))
    return K, V, table


def _index_sets(c, gen, lens):
    """The index sets an earlier slow step left: per layer and KV head `budget` positions of the candidate range, ascending."""
    b, hkv, k, layers = c["batch"], c["hkv"], c["budget"], c["layers"]
    sel = torch.full((layers, b, hkv, k), -1, dtype=torch.int32, device="cuda")
    n_sel = torch.zeros((layers, b, hkv), dtype=torch.int32, device="cuda")
    for i, n in enumerate(lens):
        n_j = n - c["recent"] - N_SINK
        m = max(0, min(k, n_j))
        if m:
            pick = torch.rand((layers, hkv, n_j), generator=gen, device="cuda").topk(m, dim=-1).indices
            sel[:, i, :, :m] = (pick.sort(dim=-1).values + N_SINK).to(torch.int32)
            n_sel[:, i] = m
    return sel, n_sel


def prepare(case, seed):
    c = case
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    b, hq, hkv, layers = c["batch"], c["hq"], c["hkv"], c["layers"]
    order = torch.randperm(b, generator=gen, device="cuda").tolist()
    ranked = _lengths(c)
    lens = [ranked[r] for r in order]
    slow = [int(r in _slow_ranks(c)) for r in order]
    K, V, table = _shape_cache(c, gen, lens)
    s = {"case": c, "K": K, "V": V, "table": table, "max_len": c["ctx_hi"], "budget": c["budget"]}
    s["ctx"] = SfiContext(b, hq, hkv, c["ctx_hi"], max(c["budget"], 1), N_SINK, c["recent"], K[0], V[0],
                          selector=FULL_SELECTOR if c["selector"] else None, alpha=c["alpha"], page_size=c["page"],
                          page_layout="htd", out_bf16=c["out_bf16"])
    s["h"] = s["ctx"].handle
    if table is not None:
        sfi.sfi_set_block_table(s["h"], table, table.numel())
    s["ctx_len"] = torch.tensor(lens, dtype=torch.int32, device="cuda")
    s["recent_start"] = (s["ctx_len"] - c["recent"]).clamp(min=N_SINK)
    n_q = c["window"] if c["op"] == "window" else layers
    s["q"] = torch.empty((n_q, b, hq, D), dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    s["out"] = torch.zeros((layers, b, hq, D), dtype=torch.bfloat16 if c["out_bf16"] else torch.float32, device="cuda")
    s["sel"], s["n_sel"] = _index_sets(c, gen, lens)
    if c["op"] == "mixed":
        desc = torch.zeros((b, 4), dtype=torch.int32)
        desc[:, 0], desc[:, 1] = s["ctx_len"].cpu(), s["recent_start"].cpu()
        desc[:, 2] = torch.tensor(slow, dtype=torch.int32)
        s["desc"] = desc.cuda()
        s["is_slow"] = torch.tensor(slow, dtype=torch.uint8, device="cuda")
    if c["compact"]:
        rows = N_SINK + c["budget"]
        s["Kc"] = torch.zeros((layers, b, hkv, rows, D), dtype=torch.bfloat16, device="cuda")
        s["Vc"] = torch.zeros_like(s["Kc"])
        for i in range(layers):
            sfi.sfi_reorg(s["h"], K[i], V[i], s["sel"][i], s["n_sel"][i], c["budget"], s["ctx_len"], None, s["Kc"][i], s["Vc"][i])
    if c["op"] == "window":  # query tau of the window sits at row L - W + tau and sees the rows up to its own
        s["q_len"] = [s["ctx_len"] - (c["window"] - 1 - t) for t in range(c["window"])]
    # what a model holds per layer: its own tensors
    names = [n for n in ("K", "V", "out", "sel", "n_sel", "Kc", "Vc") if n in s]
    s["layers"] = [{n: s[n][i] for n in names} for i in range(layers)]
    for i, l in enumerate(s["layers"]):
        l["q"] = s["q"][i]
    return s


def run(s):
    op, h, ctx_len, max_len, budget = s["case"]["op"], s["h"], s["ctx_len"], s["max_len"], s["budget"]
    if op == "fast":
        rs = s["recent_start"]
        for l in s["layers"]:
            sfi.sfi_fast_step(h, l["q"], l["K"], l["V"], l["sel"], l["n_sel"], budget, rs, ctx_len, l["out"])
        return s["out"]
    if op == "slow":
        for l in s["layers"]:
            sfi.sfi_slow_step(h, l["q"], l["K"], l["V"], ctx_len, max_len, budget, l["out"], l["sel"], l["n_sel"])
        return s["out"], s["sel"], s["n_sel"]
    if op == "dense":
        for l in s["layers"]:
            sfi.sfi_dense_attn(h, l["q"], l["K"], l["V"], ctx_len, max_len, l["out"])
        return s["out"]
    if op == "mixed":
        if s["case"]["compact"]:
            for l in s["layers"]:
                sfi.sfi_mixed_step_compact(h, l["q"], l["K"], l["V"], s["is_slow"], ctx_len, s["recent_start"], max_len, budget,
                                           l["out"], l["sel"], l["n_sel"], l["Kc"], l["Vc"])
        else:
            for l in s["layers"]:
                sfi.sfi_mixed_step_desc(h, l["q"], l["K"], l["V"], s["desc"], max_len, budget, l["out"], l["sel"], l["n_sel"])
        return s["out"], s["sel"], s["n_sel"]
    l = s["layers"][0]  # window
    for t, q_len in enumerate(s["q_len"]):
        sfi.sfi_evidence_add_causal(h, s["q"][t], l["K"], None, ctx_len, q_len, max_len, None, t == 0)
    sfi.sfi_evidence_select(h, len(s["q_len"]), ctx_len, max_len, budget, l["sel"], l["n_sel"])
    return s["sel"], s["n_sel"]


def work(case):
    """Rows of K and V the step has to read (256 bytes each), once per layer, and its results; 4 * G * 128 operations per row
    pair.  The queries of a window share their K rows, which are counted once; an index set is written by slow sequences
    and read by fast ones."""
    c = case
    g = c["hq"] // c["hkv"]
    slow = _slow_ranks(c)
    rows = ids = 0
    for r, n in enumerate(_lengths(c)):
        n_sel = max(0, min(c["budget"], n - c["recent"] - N_SINK))
        fast_rows = min(n, N_SINK) + n_sel + min(c["recent"], max(0, n - N_SINK))
        dense = c["op"] in ("slow", "dense", "window") or (c["op"] == "mixed" and r in slow)
        rows += n if dense else fast_rows
        ids += n_sel if c["op"] != "dense" else 0
    rows, ids = rows * c["hkv"], ids * c["hkv"]
    io = c["batch"] * c["hq"] * D * (2 + (2 if c["out_bf16"] else 4))
    if c["op"] == "window":
        w = c["window"]
        return {"bytes": rows * 2 * D + w * c["batch"] * c["hq"] * D * 2 + 4 * ids, "flops": w * rows * 2 * g * D}
    return {"bytes": c["layers"] * (rows * 4 * D + 4 * ids + io), "flops": c["layers"] * rows * 4 * g * D}


def tolerance(case):
    """fp32 results of fp32 sums whose softmax weights carry 16 bits into the matrix cores; bf16 results are the same values
    rounded.  Index sets are whole numbers; two positions whose scores agree to fp32 rounding may trade places."""
    if case["op"] == "window":
        return {"rel": 0.0, "differ": 0.01}
    t = {"rel": 4e-3, "max": 8e-3} if case["out_bf16"] else {"rel": 3e-5, "max": 3e-4}
    if case["op"] in ("slow", "mixed"):
        t["differ"] = 0.01
    return t

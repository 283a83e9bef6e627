"""GPU parity at the sizes where the launches change: the Selector's forms (one workgroup per pair that scores as well, one
that reads keys, segments with histograms of their own), the dense launch planned on the device (equal and unequal
lengths, more sequences than lanes, empty contexts, the most records one sequence can have) and the fast step's merge by
one to four waves.  The bars are the library's own: outputs within 2e-3 row-relative of the fp64 oracle (bf16 inputs,
probabilities kept as two bf16 terms), index sets identical outside the 1e-5 band of tied scores."""
import dataclasses

import numpy as np
import pytest

import sfi_synth as syn
from helpers import Runner, check_out, check_selection
from oracle.sfi_oracle import SelectorParams

pytestmark = pytest.mark.gpu

N_SINK, RECENT = 4, 64


def _workload(B, Hkv, G, lens, budget, seed):
    w = syn.make_tiny(L0=max(int(max(lens)), RECENT + 16), steps=3, budget=budget, recent=RECENT, n_support=4, B=B, Hq=G * Hkv,
                      Hkv=Hkv, seed=seed)
    w.n_sink = N_SINK
    w.L0 = np.array(lens, np.int32)
    return w


def _check_slow(oracle, w, r, sp=None):
    q, c = w.q(0), w.ctx_len(0)
    out, sel, nsel = r.slow(q, c, w.budget, max_len=int(c.max()))
    check_out(out, oracle.dense(q, w.K, w.V, c))
    kw = {} if sp is None else dict(sp=sp)
    sel_ref, nsel_ref, z = oracle.selector(q, w.K, c, w.budget, w.n_sink, w.recent, **kw)
    check_selection(sel, nsel, sel_ref, nsel_ref, z, c, w.n_sink, w.recent, w.budget)
    return sel, nsel


# |J| on either side of 4096, 8192 and 16384 positions, and of 24576 logits per pair; head groups around the built sizes
@pytest.mark.parametrize("n_j,G", [(0, 4), (1, 4), (4096, 5), (4097, 5), (4097, 8), (3072, 8), (3073, 8), (1536, 16), (1537, 16),
                                   (4915, 5), (4916, 5), (6144, 4), (6145, 4), (8192, 3), (8193, 1), (16384, 2), (16385, 2),
                                   (18433, 7)])
@pytest.mark.parametrize("mode", [0, 1])
def test_selector_where_its_form_changes(oracle, n_j, G, mode):
    print(f"[gpu-edges] selector mode {mode}: |J| = {n_j}, G = {G}", flush=True)
    w = _workload(1, 2, G, [n_j + N_SINK + RECENT], 129, seed=4000 + n_j + G)
    sp, d = None, None
    if mode == 1:
        sp = dataclasses.replace(SelectorParams(mode=1), alpha=1.0)
        d = {k: getattr(sp, k) for k in ("gamma", "beta", "p", "eta", "lambda_clip", "alpha_soft", "alpha_cross", "temp", "eps",
                                          "nms_radius")}
    r = Runner(w, selector=d, alpha=1.0 if d else 0.0)
    try:
        _check_slow(oracle, w, r, sp)
    finally:
        r.close()


PLANNED = {
    "equal": (8, 8, 4, [4100] * 8),
    "one long, the others short": (8, 8, 4, [4133] + [33, 64, 65, 1, 100, 97, 31]),
    "empty contexts among them": (8, 8, 2, [0, 4097, 0, 2000, 3000, 0, 1, 4096]),
    "unequal": (8, 8, 5, [1024, 4096, 2500, 3333, 1111, 2048, 4095, 3900]),
    "more sequences than lanes": (65, 4, 2, [1100 - 13 * (i % 40) for i in range(64)] + [1]),
    "more sequences than lanes, equal": (65, 4, 2, [1060] * 65),
    "most records per sequence": (2, 2, 2, [65536, 33]),
    "heads that do not divide the units": (9, 6, 3, [5000 - 431 * i for i in range(9)]),
}


@pytest.mark.parametrize("page", [0, 16])
@pytest.mark.parametrize("name", list(PLANNED))
def test_planned_dense_launch(oracle, name, page):
    B, Hkv, G, lens = PLANNED[name]
    print(f"[gpu-edges] planned dense launch: {name}, page {page}", flush=True)
    w = _workload(B, Hkv, G, lens, 65, seed=77 + len(name))
    r = Runner(w, page_size=page)
    try:
        q, c = w.q(0), w.ctx_len(0)
        check_out(r.dense(q, c, max_len=int(c.max())), oracle.dense(q, w.K, w.V, c))
        _check_slow(oracle, w, r)
        assert r.sfi.sfi_device_status(r.ctx.handle) == 0
    finally:
        r.close()


@pytest.mark.parametrize("G", [1, 2, 3, 4, 5, 8, 9, 16])
@pytest.mark.parametrize("tiles_per_wave", [1, 33])
def test_fast_step_merge(oracle, G, tiles_per_wave):
    """One workgroup per pair (33 tiles per wave) and as many as the list has tiles for (1), twice on one context: the
    arrival counters have to be back at zero after the first."""
    print(f"[gpu-edges] fast step: G = {G}, {tiles_per_wave} tiles per wave", flush=True)
    w = _workload(2, 2, G, [2500, 1999], 777, seed=900 + G)
    r = Runner(w)
    try:
        sel, nsel = _check_slow(oracle, w, r)
        r.sfi.sfi_set_tuning(r.ctx.handle, -1, tiles_per_wave, 1)
        for t in (1, 2):
            q, c, rs = w.q(t), w.ctx_len(t), w.recent_start(t)
            check_out(r.fast(q, sel, nsel, rs, c), oracle.sparse(q, w.K, w.V, sel, nsel, rs, c, w.n_sink))
    finally:
        r.close()


# evidence alone (no output): several workgroups per compute unit, shares that fill the LDS stash more than once
@pytest.mark.parametrize("B,Hkv,G,lens", [(2, 8, 4, [4200, 700]), (2, 8, 16, [9000, 8990]), (2, 8, 15, [4097, 33]), (1, 8, 4, [2000]),
                                          (9, 8, 5, [1500] * 8 + [70]), (1, 8, 1, [131])])
@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("page", [0, 16])
def test_evidence_of_a_window(oracle, B, Hkv, G, lens, mode, page):
    import torch
    from helpers import i32_dev, to_dev
    print(f"[gpu-edges] evidence: B={B} Hkv={Hkv} G={G} {lens} mode={mode} page={page}", flush=True)
    W = 3
    w = _workload(B, Hkv, G, lens, 65, seed=300 + G + mode)
    sp = dataclasses.replace(SelectorParams(mode=mode), alpha=1.0)
    d = {k: getattr(sp, k) for k in ("gamma", "beta", "p", "eta", "lambda_clip", "alpha_soft", "alpha_cross", "temp", "eps",
                                      "nms_radius")} if mode else None
    r = Runner(w, selector=d, alpha=1.0, page_size=page)
    try:
        ctx = w.ctx_len(0)
        ctx_d = i32_dev(ctx)
        sel = torch.full((B, Hkv, w.budget), -7, dtype=torch.int32, device="cuda")
        nsel = torch.full((B, Hkv), -7, dtype=torch.int32, device="cuda")
        vis = np.zeros((B, Hkv * W * G), np.int32)
        q_cat = np.empty((B, Hkv * W * G, w.d), np.uint16)
        for t in range(W):
            q, q_len = w.q(t), (ctx - W + t + 1).astype(np.int32)
            r.sfi.sfi_evidence_add_causal(r.ctx.handle, to_dev(q), r.K, None, ctx_d, i32_dev(q_len), int(ctx.max()), None, t == 0)
            for h in range(Hkv):
                q_cat[:, h * W * G + t * G:h * W * G + (t + 1) * G] = q[:, h * G:(h + 1) * G]
                vis[:, h * W * G + t * G:h * W * G + (t + 1) * G] = q_len[:, None]
        r.sfi.sfi_evidence_select(r.ctx.handle, W, ctx_d, int(ctx.max()), w.budget, sel, nsel)
        torch.cuda.synchronize()
        sel_ref, nsel_ref, z = oracle.selector(q_cat, w.K, ctx, w.budget, w.n_sink, w.recent, sp=sp, vis=vis)
        check_selection(sel.cpu().numpy(), nsel.cpu().numpy(), sel_ref, nsel_ref, z, ctx, w.n_sink, w.recent, w.budget)
        assert r.sfi.sfi_device_status(r.ctx.handle) == 0
    finally:
        r.close()


# the evidence launch: a wave has two tiles of 32 rows in flight; |J| around one tile, one and two tiles of a workgroup's four
# waves, and a sink that leaves no J (the last one is as large as an int: first rows are requested before the length is known)
@pytest.mark.parametrize("n_j", [0, 1, 31, 32, 33, 127, 128, 129, 255, 256, 257, 511, 513, 1025, -1])
@pytest.mark.parametrize("mode,G,page", [(0, 2, 0), (1, 4, 0), (1, 16, 0), (0, 16, 16), (1, 3, 16)])
def test_evidence_at_the_edges_of_its_tiles(oracle, n_j, mode, G, page):
    import torch
    from helpers import i32_dev, to_dev
    print(f"[gpu-edges] evidence: |J| = {n_j}, G = {G} mode={mode} page={page}", flush=True)
    w = _workload(2, 2, G, [n_j + N_SINK + RECENT, max(n_j - 40, 3) + N_SINK + RECENT], 65, seed=800 + n_j)
    if n_j < 0:
        w.n_sink = 2 ** 31 - 1
    sp = dataclasses.replace(SelectorParams(mode=mode), alpha=0.5)
    d = {k: getattr(sp, k) for k in ("gamma", "beta", "p", "eta", "lambda_clip", "alpha_soft", "alpha_cross", "temp", "eps",
                                      "nms_radius")} if mode else None
    r = Runner(w, selector=d, alpha=0.5, page_size=page)
    try:
        c = w.ctx_len(0)
        sel = torch.full((2, 2, w.budget), -7, dtype=torch.int32, device="cuda")
        nsel = torch.full((2, 2), -7, dtype=torch.int32, device="cuda")
        qs = [w.q(t) for t in range(2)]
        for t, q in enumerate(qs):
            r.sfi.sfi_evidence_add(r.ctx.handle, to_dev(q), r.K, None, i32_dev(c), int(c.max()), None, t == 0)
        r.sfi.sfi_evidence_select(r.ctx.handle, 2, i32_dev(c), int(c.max()), w.budget, sel, nsel)
        torch.cuda.synchronize()
        if n_j < 0:
            assert (nsel == 0).all() and (sel == -1).all()
        else:
            q_all = np.stack([q.reshape(2, 2, G, w.d) for q in qs], axis=2).reshape(2, 4 * G, w.d)
            sel_ref, nsel_ref, z = oracle.selector(q_all, w.K, c, w.budget, w.n_sink, w.recent, sp=sp)
            check_selection(sel.cpu().numpy(), nsel.cpu().numpy(), sel_ref, nsel_ref, z, c, w.n_sink, w.recent, w.budget)
        assert r.sfi.sfi_device_status(r.ctx.handle) == 0
    finally:
        r.close()


# the evidence launch whose K may be larger than the caches (288 MB): whole-line requests, through the caches where the lengths say
# that K fits after all (|J| around its tiles) and streamed where it does not; two heads share 294912 rows of two sequences
@pytest.mark.parametrize("lens", [[69, 101], [196, 197], [581, 580], [1093, 8000], [295500, 295463]], ids=str)
@pytest.mark.parametrize("mode,G,page", [(0, 1, 0), (1, 4, 0), (0, 16, 16), (1, 3, 64)])
def test_evidence_of_a_k_beyond_the_caches(oracle, lens, mode, G, page):
    import torch
    import paper_2603_12038_amd as sfi
    from helpers import i32_dev
    print(f"[gpu-edges] evidence by whole lines: lens={lens} mode={mode} G={G} page={page}", flush=True)
    B, Hkv, d, budget, max_ctx = 2, 2, 128, 65, 295552  # a multiple of 64 rows; K is 303 MB
    gen = torch.Generator(device="cuda").manual_seed(sum(lens) + G)
    L = -(-max(lens) // 64) * 64
    K = torch.empty((B, Hkv, L, d), dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    K.mul_((1 + 3 * (torch.rand(K.shape[:-1], generator=gen, device="cuda") < 0.01)).to(torch.bfloat16).unsqueeze(-1))
    qs = torch.empty((2, B, Hkv * G, d), dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    if page:
        pages = max_ctx // page
        table = torch.zeros((B, pages), dtype=torch.int32, device="cuda")  # (entries beyond the rows in use: any block)
        n = L // page
        table[:, :n] = torch.randperm(B * n, generator=gen, device="cuda").to(torch.int32).view(B, n)
        pool = torch.empty((B * n, Hkv, page, d), dtype=torch.bfloat16, device="cuda")
        pool[table[:, :n].long()] = K.view(B, Hkv, n, page, d).transpose(1, 2)
    else:
        pool = torch.zeros((B, Hkv, max_ctx, d), dtype=torch.bfloat16, device="cuda")
        pool[:, :, :L] = K
    sp = dataclasses.replace(SelectorParams(mode=mode), alpha=0.5)
    sel_cfg = {k: getattr(sp, k) for k in ("gamma", "beta", "p", "eta", "lambda_clip", "alpha_soft", "alpha_cross", "temp", "eps",
                                           "nms_radius")} if mode else None
    ctx = sfi.SfiContext(B, Hkv * G, Hkv, max_ctx, budget, N_SINK, RECENT, pool, pool, selector=sel_cfg, alpha=0.5, page_size=page,
                         page_layout="htd")
    try:
        if page:
            sfi.sfi_set_block_table(ctx.handle, table, pool.shape[0])
        c = i32_dev(lens)
        bits = lambda t: t.contiguous().view(torch.int16).cpu().numpy().view(np.uint16)
        q_all = np.stack([bits(q).reshape(B, Hkv, G, d) for q in qs], axis=2).reshape(B, 2 * Hkv * G, d)
        sel_ref, nsel_ref, z = oracle.selector(q_all, bits(K), np.array(lens, np.int32), budget, N_SINK, RECENT, sp=sp)
        for max_len in ((max_ctx,) if max(lens) > 10000 else (max_ctx, max(lens))):  # by whole lines, by the plain requests
            sel = torch.full((B, Hkv, budget), -7, dtype=torch.int32, device="cuda")
            nsel = torch.full((B, Hkv), -7, dtype=torch.int32, device="cuda")
            for t in range(2):
                sfi.sfi_evidence_add(ctx.handle, qs[t], pool, None, c, max_len, None, t == 0)
            sfi.sfi_evidence_select(ctx.handle, 2, c, max(lens), budget, sel, nsel)
            torch.cuda.synchronize()
            check_selection(sel.cpu().numpy(), nsel.cpu().numpy(), sel_ref, nsel_ref, z, np.array(lens), N_SINK, RECENT, budget)
        assert sfi.sfi_device_status(ctx.handle) == 0
    finally:
        ctx.close()


# the hand-over of a split fast step: device scope (0), the L2 of one XCD (1), and workgroups dealt to different XCDs, whose last
# wave does the list again (2); pairs in rows of eight and of a sequence, a row that is not full, heads that keep
# device scope (3, and 3 pairs with more than four workgroups; with 16, mode 2 does as well), more records than the merge reads at a time, bf16 outputs.
# Two queries in turn, so that a record of the launch before is a wrong one; the counters have to be back at zero each time.
# Bits tell which way was taken: records merged are the same sums at either scope, a list done again is another order.
@pytest.mark.parametrize("B,Hkv,G,L0,budget", [(1, 8, 4, 1500, 333), (4, 2, 4, 1500, 333), (2, 4, 8, 1500, 333), (8, 1, 5, 1500, 333),
                                               (1, 2, 3, 1500, 333), (3, 1, 16, 1500, 333), (1, 16, 9, 1500, 333), (2, 3, 4, 1500, 333),
                                               (3, 1, 4, 1500, 555), (1, 8, 4, 4200, 2600), (2, 4, 16, 4200, 2300)])
@pytest.mark.parametrize("page", [0, 16])
@pytest.mark.parametrize("bf16", [False, True])
def test_fast_step_hand_over(oracle, B, Hkv, G, L0, budget, page, bf16):
    from helpers import check_out_bf16
    print(f"[gpu-edges] hand-over: B={B} Hkv={Hkv} G={G} budget={budget} page={page} bf16={bf16}", flush=True)
    w = _workload(B, Hkv, G, [L0 - 13 * i for i in range(B)], budget, seed=600 + G)
    r = Runner(w, page_size=page, out_bf16=bf16)
    check = check_out_bf16 if bf16 else check_out
    try:
        q0, c0 = w.q(0), w.ctx_len(0)
        _, sel, nsel = r.slow(q0, c0, w.budget)
        r.reorg(sel, nsel, c0)
        qs, c, rs = [w.q(1), w.q(2)], w.ctx_len(1), w.recent_start(1)
        want = [oracle.sparse(q, w.K, w.V, sel, nsel, rs, c, w.n_sink) for q in qs]
        for tiles_per_wave in (-1, 1):
            r.sfi.sfi_set_tuning(r.ctx.handle, -1, tiles_per_wave, 1)
            got = {}
            for i, mode in enumerate((0, 2, 1, 1, 2, 0)):
                r.sfi.sfi_set_handover(r.ctx.handle, mode)
                q = qs[i % 2]
                fast = r.fast(q, sel, nsel, rs, c)
                compact = r.fast_compact(q, nsel, sel.shape[2], rs, c)
                check(fast, want[i % 2])
                check(compact, want[i % 2])
                got.setdefault(mode, {})[i % 2] = (fast, compact)
            splits = r.sfi.sfi_query_splits(r.ctx.handle)[1]
            assert splits > (16 if budget > 2000 and tiles_per_wave == 1 else 1)
            through_l2 = Hkv == 8 or (Hkv in (1, 2, 4) and (B * Hkv % 8 == 0 or (B * Hkv < 8 and splits <= 4)))
            for t in range(2):
                for path in range(2):
                    at = [got[m][t][path] for m in (0, 1, 2)]
                    assert np.array_equal(at[0], at[1]), "records merged, nothing done again"
                    if not through_l2:
                        assert np.array_equal(at[0], at[2])
                    elif not bf16:
                        assert not np.array_equal(at[0], at[2]), "the list done again by one wave"
        with pytest.raises(RuntimeError):
            r.sfi.sfi_set_handover(r.ctx.handle, 3)
    finally:
        r.close()


ATTN, ATTN2 = 0, 6  # stages whose launches are counted


# the ragged step's attention in one launch (up to one fast cell per unit) and in two (more, or records at device scope): none,
# some and all sequences slow, both fast paths, every hand-over, rows of cells that are not full
@pytest.mark.parametrize("B,Hkv,G,budget,one", [(32, 8, 2, 40, (0, 1, 2)), (33, 8, 1, 40, ()), (4, 2, 9, 300, (1, 2)), (3, 1, 4, 500, ()),
                                                (3, 1, 4, 300, (1, 2)), (2, 2, 4, 300, (1, 2)), (2, 8, 16, 300, (1, 2)), (5, 4, 5, 200, ())])
@pytest.mark.parametrize("page", [0, 16])
def test_ragged_step_in_one_launch(oracle, B, Hkv, G, budget, one, page):
    """one: the hand-overs with which the step is one launch."""
    import torch
    from helpers import i32_dev, to_dev
    print(f"[gpu-edges] ragged step: B={B} Hkv={Hkv} G={G} budget={budget} page={page}", flush=True)
    w = _workload(B, Hkv, G, [1400 - 37 * (i % 30) for i in range(B)], budget, seed=1000 + B)
    r = Runner(w, page_size=page)
    try:
        q0, c0 = w.q(0), w.ctx_len(0)
        _, sel0, nsel0 = r.slow(q0, c0, budget, max_len=int(c0.max()))
        c, rs = w.ctx_len(1), w.recent_start(1)
        steps = []  # two queries in turn: a record of the step before is a wrong one
        for q in (w.q(1), w.q(2)):
            steps.append((q, oracle.dense(q, w.K, w.V, c), oracle.sparse(q, w.K, w.V, sel0, nsel0, rs, c, w.n_sink),
                          oracle.selector(q, w.K, c, budget, w.n_sink, w.recent)))
        for slow in ([], [1], [0, B - 1], list(range(B))):
            flags = np.zeros(B, np.uint8)
            flags[slow] = 1
            for compact in (False, True):
                for i, mode in enumerate((1, 2, 0)):
                    q, dense, sparse, (sel_ref, nsel_ref, z) = steps[i % 2]
                    r.sfi.sfi_set_handover(r.ctx.handle, mode)
                    r.reorg(sel0, nsel0, c0)
                    sel, nsel = i32_dev(sel0), i32_dev(nsel0)
                    r.out.fill_(float("nan"))
                    args = (r.ctx.handle, to_dev(q), r.K, r.V, torch.from_numpy(flags).cuda(), i32_dev(c), i32_dev(rs), int(c.max()), budget, r.out, sel, nsel)
                    r.sfi.sfi_set_profiling(r.ctx.handle, 1)
                    if compact:
                        r.sfi.sfi_mixed_step_compact(*args, r.Kc, r.Vc)
                    else:
                        r.sfi.sfi_mixed_step(*args)
                    count = r.sfi.sfi_stage_times(r.ctx.handle)[1]
                    r.sfi.sfi_set_profiling(r.ctx.handle, 0)
                    assert (count[ATTN], count[ATTN2]) == (1, 0 if mode in one else 1)
                    torch.cuda.synchronize()
                    check_out(r.out.cpu().numpy(), np.where(flags[:, None, None] != 0, dense, sparse))
                    got, ngot = sel.cpu().numpy(), nsel.cpu().numpy()
                    keep = flags == 0
                    assert (got[keep] == sel0[keep]).all() and (ngot[keep] == nsel0[keep]).all()
                    for b in slow:
                        check_selection(got[b:b + 1], ngot[b:b + 1], sel_ref[b:b + 1], nsel_ref[b:b + 1], z[b:b + 1], c[b:b + 1], w.n_sink, w.recent, budget)
        assert r.sfi.sfi_device_status(r.ctx.handle) == 0
    finally:
        r.close()


# Cells of more than 24 tiles (768 rows with the sink and the recent window): the dense shares are cut by what a workgroup has had
# already.  None, one, a quarter, half, all but one and all sequences slow: equal shares, one size of shares (the cells are more
# work than the list has for their workgroups) and two sizes, with lists that cross sequences on either side.  Several
# cells a pair by force (tiles per wave), in rows that are full and not; more sequences than lanes.
@pytest.mark.parametrize("B,Hkv,G,lo,hi,budget,tiles_per_wave", [(32, 8, 2, 1100, 1400, 800, -1), (16, 8, 4, 900, 3000, 850, 9), (4, 2, 9, 2000, 5000, 1800, 8),
                                                                 (3, 1, 4, 3000, 6000, 2600, 8), (5, 3, 1, 1500, 3500, 900, 9), (100, 2, 5, 850, 1200, 800, 9)])
@pytest.mark.parametrize("page", [0, 16])
def test_ragged_step_of_long_cells(oracle, B, Hkv, G, lo, hi, budget, tiles_per_wave, page):
    import torch
    from helpers import i32_dev, to_dev
    print(f"[gpu-edges] ragged step, long cells: B={B} Hkv={Hkv} G={G} rows {lo}..{hi} budget={budget} page={page}", flush=True)
    w = _workload(B, Hkv, G, [lo + (hi - lo) * (7 * i % B) // B for i in range(B)], budget, seed=2000 + B)
    r = Runner(w, page_size=page)
    try:
        q0, c0 = w.q(0), w.ctx_len(0)
        _, sel0, nsel0 = r.slow(q0, c0, budget, max_len=int(c0.max()))
        q, c, rs = w.q(1), w.ctx_len(1), w.recent_start(1)
        dense, sparse = oracle.dense(q, w.K, w.V, c), oracle.sparse(q, w.K, w.V, sel0, nsel0, rs, c, w.n_sink)
        sel_ref, nsel_ref, z = oracle.selector(q, w.K, c, budget, w.n_sink, w.recent)
        r.sfi.sfi_set_tuning(r.ctx.handle, -1, tiles_per_wave, 1)
        every = list(range(B))
        for slow in ([], [1], every[::4], every[1::2], every[1:], every):
            flags = np.zeros(B, np.uint8)
            flags[slow] = 1
            for compact in (False, True):
                r.reorg(sel0, nsel0, c0)
                sel, nsel = i32_dev(sel0), i32_dev(nsel0)
                r.out.fill_(float("nan"))
                args = (r.ctx.handle, to_dev(q), r.K, r.V, torch.from_numpy(flags).cuda(), i32_dev(c), i32_dev(rs), int(c.max()), budget, r.out, sel, nsel)
                r.sfi.sfi_set_profiling(r.ctx.handle, 1)
                if compact:
                    r.sfi.sfi_mixed_step_compact(*args, r.Kc, r.Vc)
                else:
                    r.sfi.sfi_mixed_step(*args)
                count = r.sfi.sfi_stage_times(r.ctx.handle)[1]
                r.sfi.sfi_set_profiling(r.ctx.handle, 0)
                splits = r.sfi.sfi_query_splits(r.ctx.handle)[1]
                assert (count[ATTN], count[ATTN2]) == (1, 0) and N_SINK + budget + RECENT > 24 * 32 * splits
                torch.cuda.synchronize()
                check_out(r.out.cpu().numpy(), np.where(flags[:, None, None] != 0, dense, sparse))
                got, ngot = sel.cpu().numpy(), nsel.cpu().numpy()
                keep = flags == 0
                assert (got[keep] == sel0[keep]).all() and (ngot[keep] == nsel0[keep]).all()
                on = flags != 0
                if on.any():
                    check_selection(got[on], ngot[on], sel_ref[on], nsel_ref[on], z[on], c[on], w.n_sink, w.recent, budget)
        assert r.sfi.sfi_device_status(r.ctx.handle) == 0
    finally:
        r.close()

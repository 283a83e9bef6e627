"""GPU parity of the Selector at the limits of its inputs: logits whose exponentials overflow, head groups between the built
ones, tie classes and threshold bins of the long form, and windows over more rows than a unit's first shares hold, as evidence
alone and with the queries' outputs (the dense launch planned on the device).
Against the fp64 oracle with the library's own bars, as in the other parity tests."""
import dataclasses

import numpy as np
import pytest

import sfi_synth as syn
from helpers import Runner, check_out, check_selection, i32_dev, to_dev
from oracle.sfi_oracle import SelectorParams
from test_gpu_dispatch_edges import N_SINK, RECENT, _workload

pytestmark = pytest.mark.gpu


def _selector(mode):
    """Oracle parameters and the context's selector argument (None in mode 0)."""
    sp = dataclasses.replace(SelectorParams(mode=mode), alpha=1.0)
    keys = ("gamma", "beta", "p", "eta", "lambda_clip", "alpha_soft", "alpha_cross", "temp", "eps", "nms_radius")
    return sp, {k: getattr(sp, k) for k in keys} if mode else None


def _check_slow(oracle, w, r, sp, q, **bars):
    c = w.ctx_len(0)
    out, sel, nsel = r.slow(q, c, w.budget, max_len=int(c.max()))
    check_out(out, oracle.dense(q, w.K, w.V, c))
    sel_ref, nsel_ref, z = oracle.selector(q, w.K, c, w.budget, w.n_sink, w.recent, **({} if sp is None else dict(sp=sp)))
    check_selection(sel, nsel, sel_ref, nsel_ref, z, c, w.n_sink, w.recent, w.budget, **bars)
    return sel, nsel


def _check_window(oracle, w, r, sp, queries, with_out=False, **bars):
    """Evidence of the queries of the last rows (causal), and their outputs if asked for, then the index set."""
    import torch
    B, Hkv, G, W = w.B, w.Hkv, w.Hq // w.Hkv, len(queries)
    c = w.ctx_len(0)
    c_d, max_len = i32_dev(c), int(c.max())
    sel = torch.full((B, Hkv, w.budget), -7, dtype=torch.int32, device="cuda")
    nsel = torch.full((B, Hkv), -7, dtype=torch.int32, device="cuda")
    vis = np.empty((B, Hkv, W, G), np.int32)
    for t, q in enumerate(queries):
        q_len = np.maximum(c - W + t + 1, 0).astype(np.int32)
        r.out.fill_(float("nan"))
        r.sfi.sfi_evidence_add_causal(r.ctx.handle, to_dev(q), r.K, r.V if with_out else None, c_d, i32_dev(q_len), max_len,
                                      r.out if with_out else None, t == 0)
        vis[:, :, t] = q_len[:, None, None]
        if with_out:
            torch.cuda.synchronize()
            check_out(r.out.cpu().numpy(), oracle.dense(q, w.K, w.V, q_len))
    r.sfi.sfi_evidence_select(r.ctx.handle, W, c_d, max_len, w.budget, sel, nsel)
    torch.cuda.synchronize()
    q_all = np.stack([q.reshape(B, Hkv, G, w.d) for q in queries], axis=2).reshape(B, Hkv * W * G, w.d)
    sel_ref, nsel_ref, z = oracle.selector(q_all, w.K, c, w.budget, w.n_sink, w.recent, sp=sp, vis=vis.reshape(B, -1))
    check_selection(sel.cpu().numpy(), nsel.cpu().numpy(), sel_ref, nsel_ref, z, c, w.n_sink, w.recent, w.budget, **bars)
    assert r.sfi.sfi_device_status(r.ctx.handle) == 0


def _raise_logits(w, steps):
    """Element 0 of every row is 12 and of every query 128: every logit grows by 12 * 128 / sqrt(128) = 136, far beyond
    ln(2^128) = 88.7.  The softmax is what it was, but an exponential taken without its maximum overflows."""
    k0, q0 = syn.f32_to_bf16_bits(np.array([12.0, 128.0], np.float32))
    w.K[..., 0] = k0
    queries = [w.q(t).copy() for t in range(steps)]
    for q in queries:
        q[..., 0] = q0
    return queries


# |J| of each form: one workgroup that also scores, scoring launch and one workgroup, segments.  G between the built head counts,
# whose kernels carry columns beyond the last head.  Band: the fp32 sums behind a logit reach 1536, where half an ulp is
# 6.1e-5; the largest of eight roundings one way, over sqrt(128), 4.3e-5, for a score and the one it is compared with twice
# that, times the full Selector's 1 + alpha_soft + alpha_cross = 1.85.
BAND = {0: 8.7e-5, 1: 1.6e-4}


@pytest.mark.parametrize("n_j", [1500, 9000, 17000])
@pytest.mark.parametrize("G", [3, 6, 7, 9])
@pytest.mark.parametrize("mode", [0, 1])
def test_columns_beyond_the_last_head_count_for_nothing(oracle, n_j, G, mode):
    print(f"[gpu-limits] large logits: |J| = {n_j}, G = {G}, mode {mode}", flush=True)
    w = _workload(1, 2, G, [n_j + N_SINK + RECENT], 129, seed=500 + G)
    queries = _raise_logits(w, 2)
    sp, d = _selector(mode)
    r = Runner(w, selector=d, alpha=1.0)
    try:
        _check_slow(oracle, w, r, sp, queries[0], band=BAND[mode])
        _check_window(oracle, w, r, sp, queries, band=BAND[mode])
    finally:
        r.close()


# |J| = 20000 and 16900: ten and nine segments of 2048 positions.  The tie class spans three of them and is larger than any.
@pytest.mark.parametrize("case", ["random", "ties", "all_equal"])
def test_long_form_takes_ties_by_index_across_segments(oracle, case):
    w = _workload(2, 2, 4, [20000 + N_SINK + RECENT, 16900 + N_SINK + RECENT], 700, seed=91)
    if case == "ties":
        w.K[:, :, 3000:7200] = w.K[:, :, 3000:3001]
    if case == "all_equal":
        w.K[:] = 0
    r = Runner(w, max_budget=20100)
    try:
        q, c = w.q(0), w.ctx_len(0)
        for budget in (700, 1, 64, 2500, 16900, 20100):
            print(f"[gpu-limits] long form, {case}, budget {budget}", flush=True)
            sel_ref, nsel_ref, z = oracle.selector(q, w.K, c, budget, w.n_sink, w.recent)
            _, sel, nsel = r.slow(q, c, budget, max_len=int(c.max()))
            check_selection(sel, nsel, sel_ref, nsel_ref, z, c, w.n_sink, w.recent, budget)
            if case == "all_equal":
                for b in range(w.B):
                    k = int(nsel[b, 0])
                    assert (sel[b, :, :k] == N_SINK + np.arange(k)).all()
        assert r.sfi.sfi_device_status(r.ctx.handle) == 0
    finally:
        r.close()


# Logits of standard deviation 19 (scale 1.6): the 1200th best of 20000 positions has a weight of 2^-67 and less, below the
# histogram's range, whose lowest bin holds keys of any magnitude.  The oracle ranks by log(f + eps) with eps far below
# every weight.  Band: |y| stays below 256, where half an ulp is 7.6e-6; eight roundings of the logit, its scaling and the
# subtraction of the maximum, in log2, for a score and the one it is compared with: 2 * 10 * 7.6e-6 * ln 2.
@pytest.mark.parametrize("budget", [300, 1200, 4000])
def test_long_form_threshold_below_the_histograms_range(oracle, budget):
    print(f"[gpu-limits] threshold below the histogram's range, budget {budget}", flush=True)
    w = _workload(1, 2, 1, [20000 + N_SINK + RECENT], budget, seed=17)
    w.K[:, :, :] = syn.normal_bf16(np.random.default_rng(5), w.K.shape)
    sp = dataclasses.replace(SelectorParams(mode=0), eps=1e-300)
    r = Runner(w, scale=1.6)
    try:
        q, c = w.q(0), w.ctx_len(0)
        sel_ref, nsel_ref, z = oracle.selector(q, w.K, c, budget, w.n_sink, w.recent, sp=sp, scale=1.6)
        kth = [np.sort(z[0, h, N_SINK:N_SINK + 20000])[-budget] / np.log(2.0) for h in range(w.Hkv)]
        assert all(-126 < t for t in kth) and (budget < 1200 or all(t < -63 for t in kth)), kth
        _, sel, nsel = r.slow(q, c, budget, max_len=int(c.max()))
        check_selection(sel, nsel, sel_ref, nsel_ref, z, c, w.n_sink, w.recent, budget, band=1.1e-4)
    finally:
        r.close()


# 8 sequences of 8 KV heads and 8200 rows at most.  Without an output: 16 workgroups per pair, four tiles a wave.  With one: 16
# tiles per wave of every unit, twice what the dense launch planned on the device asks for; it guesses equal lengths, which
# then has to hold for the rows that the query sees as well.
@pytest.mark.parametrize("lens", [[8200, 6000, 7777, 5001, 8199, 4100, 7001, 8000], [8200] * 8], ids=["unequal", "equal"])
@pytest.mark.parametrize("page", [0, 16])
@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("with_out", [False, True], ids=["evidence", "out"])
def test_window_of_many_tiles(oracle, with_out, mode, page, lens):
    print(f"[gpu-limits] window of many tiles: with_out {with_out}, mode {mode}, page {page}, {lens}", flush=True)
    w = _workload(8, 8, 2, lens, 129, seed=300)
    sp, d = _selector(mode)
    r = Runner(w, selector=d, alpha=1.0, page_size=page)
    try:
        _check_window(oracle, w, r, sp, [w.q(t) for t in range(3)], with_out)
    finally:
        r.close()


# 280000 positions: 137 segments, three groups of 64 whose histograms are added up first (from 129 segments on); the other
# sequence has one group.  The tie class spans the border of the first two groups (segment 64 begins at position 131072).
@pytest.mark.parametrize("case", ["random", "ties"])
def test_very_long_form_adds_histograms_by_groups(oracle, case):
    import torch
    w = _workload(2, 1, 2, [280000 + N_SINK + RECENT, 100000 + N_SINK + RECENT], 30000, seed=61)
    if case == "ties":
        w.K[:, :, 125000:140000] = w.K[:, :, 125000:125001]
    r = Runner(w)
    try:
        q, c = w.q(0), w.ctx_len(0)
        for budget in (700, 30000):
            print(f"[gpu-limits] histograms by groups, {case}, budget {budget}", flush=True)
            sel_ref, nsel_ref, z = oracle.selector(q, w.K, c, budget, w.n_sink, w.recent)
            _, sel, nsel = r.slow(q, c, budget, max_len=int(c.max()))
            check_selection(sel, nsel, sel_ref, nsel_ref, z, c, w.n_sink, w.recent, budget)
            # the ragged step, whose launches take the slow sequences from a list: same evidence, same sets
            sel_d = torch.full((2, 1, budget), -7, dtype=torch.int32, device="cuda")
            nsel_d = torch.zeros((2, 1), dtype=torch.int32, device="cuda")
            r.sfi.sfi_mixed_step(r.ctx.handle, to_dev(q), r.K, r.V, torch.ones(2, dtype=torch.uint8, device="cuda"), i32_dev(c),
                                 i32_dev(w.recent_start(0)), int(c.max()), budget, r.out, sel_d, nsel_d)
            torch.cuda.synchronize()
            check_selection(sel_d.cpu().numpy(), nsel_d.cpu().numpy(), sel_ref, nsel_ref, z, c, w.n_sink, w.recent, budget)
        assert r.sfi.sfi_device_status(r.ctx.handle) == 0
    finally:
        r.close()


# 300 slow sequences: more than the Selector's launches have workgroups along the list, so each walks several entries.
# (A group of nine heads: as many pairs are scored in a launch of their own.)
@pytest.mark.parametrize("G, mode", [(4, 0), (4, 1), (9, 0)])
def test_more_slow_sequences_than_workgroups(oracle, G, mode):
    import torch
    print(f"[gpu-limits] 300 slow sequences, G = {G}, mode {mode}", flush=True)
    lens = [60 + (37 * i) % 500 for i in range(300)]
    w = _workload(300, 8, G, lens, 33, seed=12)
    sp, d = _selector(mode)
    r = Runner(w, selector=d, alpha=1.0)
    try:
        q, c = w.q(0), w.ctx_len(0)
        flags = np.ones(300, np.uint8)
        flags[[0, 7, 299]] = 0
        sel = torch.full((300, 8, 33), -7, dtype=torch.int32, device="cuda")
        nsel = torch.zeros((300, 8), dtype=torch.int32, device="cuda")
        r.sfi.sfi_mixed_step(r.ctx.handle, to_dev(q), r.K, r.V, torch.from_numpy(flags).cuda(), i32_dev(c), i32_dev(w.recent_start(0)),
                             int(c.max()), 33, r.out, sel, nsel)
        torch.cuda.synchronize()
        sel_ref, nsel_ref, z = oracle.selector(q, w.K, c, 33, w.n_sink, w.recent, sp=sp)
        on = flags != 0
        check_out(r.out.cpu().numpy()[on], oracle.dense(q, w.K, w.V, c)[on])
        check_selection(sel.cpu().numpy()[on], nsel.cpu().numpy()[on], sel_ref[on], nsel_ref[on], z[on], c[on], w.n_sink, w.recent, 33)
        assert (sel.cpu().numpy()[~on] == -7).all()
        assert r.sfi.sfi_device_status(r.ctx.handle) == 0
    finally:
        r.close()


# A ragged step of one sequence is launched as a slow step: same outputs and index sets, bit for bit, and nothing when it is fast
@pytest.mark.parametrize("page", [0, 16])
@pytest.mark.parametrize("n", [1, 60, 1000, 5003, 17000])
@pytest.mark.parametrize("mode", [0, 1])
def test_ragged_step_of_one_sequence(oracle, mode, n, page):
    import torch
    print(f"[gpu-limits] ragged step of one sequence: {n} rows, mode {mode}, page {page}", flush=True)
    w = _workload(1, 2, 5, [n], 65, seed=700 + n)
    sp, d = _selector(mode)
    r = Runner(w, selector=d, alpha=1.0, page_size=page)
    try:
        q, c, rs = w.q(0), w.ctx_len(0), w.recent_start(0)
        out, sel, nsel = r.slow(q, c, 65, max_len=n)
        check_out(out, oracle.dense(q, w.K, w.V, c))
        for slow in (1, 0):
            sel_d, nsel_d = i32_dev(sel), i32_dev(nsel)
            if slow:
                sel_d.fill_(-7)
                nsel_d.fill_(-7)
            r.out.fill_(float("nan"))
            r.sfi.sfi_mixed_step(r.ctx.handle, to_dev(q), r.K, r.V, torch.full((1,), slow, dtype=torch.uint8, device="cuda"), i32_dev(c),
                                 i32_dev(rs), n, 65, r.out, sel_d, nsel_d)
            torch.cuda.synchronize()
            got = r.out.cpu().numpy()
            assert (sel_d.cpu().numpy() == sel).all() and (nsel_d.cpu().numpy() == nsel).all()
            if slow:
                assert (got == out).all()
            else:
                check_out(got, oracle.sparse(q, w.K, w.V, sel, nsel, rs, c, w.n_sink))
        assert r.sfi.sfi_device_status(r.ctx.handle) == 0
    finally:
        r.close()


# Paged dense launch with one workgroup per unit (few workgroups, or long shares) and with two (many short shares)
@pytest.mark.parametrize("B, lens", [(1, [17000]), (1, [1]), (3, [700, 33, 512]), (48, [100 + 9 * i for i in range(48)]),
                                     (48, [15 + 4 * i for i in range(48)])],
                         ids=["one long", "one row", "few", "long shares", "short shares"])
def test_paged_dense_launch_by_workgroups_per_unit(oracle, B, lens):
    print(f"[gpu-limits] paged dense launch: {B} sequences of up to {max(lens)} rows", flush=True)
    w = _workload(B, 8, 3, lens, 33, seed=40 + B)
    r = Runner(w, page_size=16)
    try:
        q, c = w.q(0), w.ctx_len(0)
        check_out(r.dense(q, c, max_len=int(c.max())), oracle.dense(q, w.K, w.V, c))
        assert r.sfi.sfi_device_status(r.ctx.handle) == 0
    finally:
        r.close()


# Dense attention with one to four heads per merging wave, few and many records, in the kernel and in a launch of its own
@pytest.mark.parametrize("page", [0, 16])
@pytest.mark.parametrize("G", [1, 8, 9, 12, 13, 16])
def test_dense_attention_merges_groups_of_any_size(oracle, G, page):
    w = _workload(2, 4, G, [9001, 4100], 33, seed=900 + G)
    r = Runner(w, page_size=page)
    try:
        for lens in ([9001, 4100], [2100, 2099], [300, 77], [1, 0]):  # up to 63 records per head, 16, 3, none to merge
            print(f"[gpu-limits] dense attention, G = {G}, page {page}, {lens}", flush=True)
            c = np.array(lens, np.int32)
            check_out(r.dense(w.q(0), c, max_len=int(c.max())), oracle.dense(w.q(0), w.K, w.V, c))
        assert r.sfi.sfi_device_status(r.ctx.handle) == 0
    finally:
        r.close()


# A recent window longer than a workgroup's 1024 positions, with J shorter and longer than it: a masked query sees no more of
# J than the whole window has, which is what the accumulating launch covers
@pytest.mark.parametrize("mode", [0, 1])
def test_window_behind_a_long_recent_window(oracle, mode):
    print(f"[gpu-limits] window behind a recent window of 1500 rows, mode {mode}", flush=True)
    w = _workload(4, 2, 2, [3999, 1700, 1505, 2600], 129, seed=73)
    w.recent = 1500
    sp, d = _selector(mode)
    r = Runner(w, selector=d, alpha=1.0)
    try:
        _check_window(oracle, w, r, sp, [w.q(t) for t in range(3)])
    finally:
        r.close()


# A stage counts launches: where one workgroup does all (short J) or reads the window's evidence, the scoring stage has none
@pytest.mark.parametrize("n_j, mode, want", [(1500, 0, dict(score=0, cand=0, write=1)), (9000, 0, dict(score=1, cand=0, write=1)),
                                             (17000, 0, dict(score=1, cand=1, write=1)), (1500, 1, dict(score=1, cand=0, write=1))])
def test_stages_count_what_was_launched(n_j, mode, want):
    import torch
    from paper_2603_12038_amd.binding import STAGE_NAMES
    print(f"[gpu-limits] stage counts: |J| = {n_j}, mode {mode}", flush=True)
    w = _workload(1, 2, 4, [n_j + N_SINK + RECENT], 65, seed=8)
    sp, d = _selector(mode)
    r = Runner(w, selector=d, alpha=1.0)
    try:
        q, c, h = w.q(0), w.ctx_len(0), r.ctx.handle
        r.slow(q, c, 65, max_len=int(c.max()))
        r.sfi.sfi_set_profiling(h, 1)
        r.slow(q, c, 65, max_len=int(c.max()))
        ms, cnt = r.sfi.sfi_stage_times(h)
        got = dict(zip(STAGE_NAMES, cnt))
        assert {k: got[k] for k in want} == want, got
        assert ms[STAGE_NAMES.index("score")] > 0 or want["score"] == 0
        if mode == 0 and n_j <= 16384:
            sel = torch.empty((1, 2, 65), dtype=torch.int32, device="cuda")
            nsel = torch.empty((1, 2), dtype=torch.int32, device="cuda")
            r.sfi.sfi_evidence_add(h, to_dev(q), r.K, None, i32_dev(c), int(c.max()), None, True)
            r.sfi.sfi_set_profiling(h, 1)
            r.sfi.sfi_evidence_select(h, 1, i32_dev(c), int(c.max()), 65, sel, nsel)
            got = dict(zip(STAGE_NAMES, r.sfi.sfi_stage_times(h)[1]))
            assert (got["score"], got["write"]) == (0, 1), got
    finally:
        r.close()


# Groups of more than eight heads score in the selecting workgroup up to 64 pairs, in a launch before it with more
@pytest.mark.parametrize("B", [8, 9])
@pytest.mark.parametrize("G", [8, 9, 16])
def test_large_groups_score_by_the_number_of_pairs(oracle, G, B):
    print(f"[gpu-limits] scoring of {8 * B} pairs, G = {G}", flush=True)
    w = _workload(B, 8, G, [1100 - 97 * i for i in range(B)], 65, seed=30 + G + B)
    r = Runner(w)
    try:
        _check_slow(oracle, w, r, None, w.q(0))
    finally:
        r.close()


# A J of more segments than a grid's second index takes: the segments move to the first one.  One block of 65536 rows stands behind every entry of
# the block table, so that each of its rows comes 2049 times: the index set is the first copies of the row with the largest logit.
def test_more_segments_than_the_second_grid_index_takes():
    import torch
    import paper_2603_12038_amd as sfi
    page, n_page, budget, recent = 65536, 2049, 100, 64
    L = page * n_page - 77
    print(f"[gpu-limits] one sequence of {L} rows, paged onto one block", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(11)
    K = torch.empty((1, 1, page, 128), dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    V = torch.empty((1, 1, page, 128), dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    q = torch.empty((1, 1, 128), dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    y = (K[0, 0].float() * q[0, 0].float()).sum(-1)
    best = int(y.argmax())
    assert float(y.max() - y[torch.arange(page, device="cuda") != best].max()) > 1e-3
    want = [p for p in range(best, L - recent, page) if p >= N_SINK][:budget]
    ctx = sfi.SfiContext(1, 1, 1, page * n_page, budget, N_SINK, recent, K, V, page_size=page, page_layout="htd")
    try:
        sfi.sfi_set_block_table(ctx.handle, torch.zeros((1, n_page), dtype=torch.int32, device="cuda"), 1)
        out = torch.zeros((1, 1, 128), device="cuda")
        sel = torch.full((1, 1, budget), -7, dtype=torch.int32, device="cuda")
        nsel = torch.full((1, 1), -7, dtype=torch.int32, device="cuda")
        sfi.sfi_slow_step(ctx.handle, q, K, V, i32_dev([L]), L, budget, out, sel, nsel)
        torch.cuda.synchronize()
        assert int(nsel) == budget and sel.flatten().tolist() == want
        p = torch.softmax(y.double() / 128 ** 0.5, 0)  # (the 77 rows that are missing from the last copy do not show)
        ref = p @ V[0, 0].double()
        assert float((out[0, 0].double() - ref).abs().max() / ref.abs().max()) < 2e-3
    finally:
        ctx.close()

"""GPU parity of the Selector at the limits of its inputs: logits whose exponentials overflow, head groups between the built
ones, tie classes and threshold bins of the long form, and windows large enough for the launch planned on the device.
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
    sel_ref, nsel_ref, z = oracle.selector(q, w.K, c, w.budget, w.n_sink, w.recent, sp=sp)
    check_selection(sel, nsel, sel_ref, nsel_ref, z, c, w.n_sink, w.recent, w.budget, **bars)
    return sel, nsel


def _check_window(oracle, w, r, sp, queries, **bars):
    """Evidence of the queries of the last rows (causal, no output), then the index set."""
    import torch
    B, Hkv, G, W = w.B, w.Hkv, w.Hq // w.Hkv, len(queries)
    c = w.ctx_len(0)
    c_d, max_len = i32_dev(c), int(c.max())
    sel = torch.full((B, Hkv, w.budget), -7, dtype=torch.int32, device="cuda")
    nsel = torch.full((B, Hkv), -7, dtype=torch.int32, device="cuda")
    vis = np.empty((B, Hkv, W, G), np.int32)
    for t, q in enumerate(queries):
        q_len = np.maximum(c - W + t + 1, 0).astype(np.int32)
        r.sfi.sfi_evidence_add_causal(r.ctx.handle, to_dev(q), r.K, None, c_d, i32_dev(q_len), max_len, None, t == 0)
        vis[:, :, t] = q_len[:, None, None]
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

"""The C-ABI boundary on the host (no GPU): the library loads, exports what include/sfi.h declares,
and rejects bad arguments with error codes before anything is launched."""
import ctypes as C
import os
import re

import pytest

import paper_2603_12038_amd as sfi
from paper_2603_12038_amd.binding import SfiConfig

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
OK, EINVAL, EUNSUPPORTED, EWORKSPACE, EALIGN = 0, -1, -2, -3, -4


def good_cfg(**over):
    c = SfiConfig()
    c.batch, c.n_q_heads, c.n_kv_heads, c.head_dim = 2, 8, 2, 128
    c.max_ctx, c.max_budget, c.n_sink, c.recent = 4096, 256, 4, 64
    c.scale, c.selector_mode = 0.0, 0
    c.k_stride_t, c.k_stride_h, c.k_stride_b = 128, 128 * 4096, 2 * 128 * 4096
    c.v_stride_t, c.v_stride_h, c.v_stride_b = 128, 128 * 4096, 2 * 128 * 4096
    for k, v in over.items():
        setattr(c, k, v)
    return c


def test_library_exports_every_declared_symbol():
    lib = sfi.load_library()
    header = open(os.path.join(ROOT, "include", "sfi.h")).read()
    header = re.sub(r"/\*.*?\*/", "", header, flags=re.S)
    declared = set(re.findall(r"\b(sfi_[a-z_]+)\s*\(", header))
    assert {"sfi_slow_step", "sfi_fast_step", "sfi_mixed_step", "sfi_create", "sfi_workspace_bytes"} <= declared
    for name in sorted(declared):
        assert hasattr(lib, name), f"{name} declared in sfi.h but not exported"
    assert declared == set(sfi.binding.EXPORTS), "binding and header disagree on the entry points"


def test_workspace_bytes_and_config_validation():
    assert sfi.sfi_workspace_bytes(good_cfg()) > 0
    assert sfi.sfi_workspace_bytes(good_cfg()) % 256 == 0
    bigger = sfi.sfi_workspace_bytes(good_cfg(max_ctx=8192))
    assert bigger > sfi.sfi_workspace_bytes(good_cfg())
    for bad in (dict(batch=0), dict(n_kv_heads=0), dict(n_q_heads=7), dict(head_dim=64), dict(max_ctx=0),
                dict(max_budget=-1), dict(n_sink=-1), dict(recent=-1), dict(k_stride_t=100), dict(v_stride_h=12),
                dict(selector_mode=2), dict(n_q_heads=64, n_kv_heads=2), dict(scale=-1.0), dict(alpha=1.5),
                dict(alpha=-0.1), dict(max_ctx=1 << 24, k_stride_t=128 * 8)):
        assert sfi.sfi_workspace_bytes(good_cfg(**bad)) == 0, bad
    assert sfi.sfi_workspace_bytes(good_cfg(alpha=0.5)) == sfi.sfi_workspace_bytes(good_cfg())


def test_workspace_has_no_hand_over_for_steps_that_cannot_score():
    """What the dense launch hands over where it scores, 512 bytes per query head and sequence (and 132 KB per pair), only for contexts whose
    dense launch can: another 32 query heads are otherwise their records, logits and statistics."""
    def heads(**shape):
        cfg = dict(k_stride_b=0, v_stride_b=0, n_kv_heads=8, **shape)
        return sfi.sfi_workspace_bytes(good_cfg(n_q_heads=64, **cfg)) - sfi.sfi_workspace_bytes(good_cfg(n_q_heads=32, **cfg))

    for batch, ctx, scores in ((32, 32768, True), (33, 32768, False), (64, 32768, False), (1024, 32768, False), (32, 16384, False), (32, 16384 + 68, False)):
        ld = (ctx + 2047) // 2048 * 2048
        assert heads(batch=batch, max_ctx=ctx) == batch * 32 * (64 * 528 + 4 * ld + 8 + (512 if scores else 0)), (batch, ctx)


FULL = dict(selector_mode=1, gamma=0.5, beta=1.0, p=2.0, eta=0.5, lambda_clip=0.02, alpha_soft=0.5, alpha_cross=0.35,
            temp=1.0, eps=1e-8, nms_radius=2)


def test_full_selector_config_validation():
    """Mode 1 needs its hyper-parameters in range; its workspace is larger (prior, Soft-NMS scores, key norms)."""
    assert sfi.sfi_workspace_bytes(good_cfg(**FULL)) > sfi.sfi_workspace_bytes(good_cfg())
    for bad in (dict(temp=0.0), dict(gamma=-1.0), dict(p=0.5), dict(eta=-0.1), dict(lambda_clip=1.5), dict(lambda_clip=-0.1),
                dict(alpha_soft=-1.0), dict(alpha_cross=-1.0), dict(nms_radius=-1), dict(nms_radius=65), dict(eps=-1e-8),
                dict(eps=2.0), dict(alpha_soft=3.0, alpha_cross=1.0)):
        assert sfi.sfi_workspace_bytes(good_cfg(**{**FULL, **bad})) == 0, bad
    assert sfi.sfi_workspace_bytes(good_cfg(**{**FULL, "eps": 0.0})) > 0  # 0 selects 1e-8


def test_create_rejects_bad_arguments_without_touching_a_device():
    lib = sfi.load_library()
    need = sfi.sfi_workspace_bytes(good_cfg())
    h = C.c_void_p()
    fake = 0x10000  # never dereferenced: creation only records the address
    assert lib.sfi_create(None, fake, need, C.byref(h)) == EINVAL
    assert lib.sfi_create(C.byref(good_cfg()), None, need, C.byref(h)) == EINVAL
    assert lib.sfi_create(C.byref(good_cfg()), fake, need, None) == EINVAL
    assert lib.sfi_create(C.byref(good_cfg()), fake + 8, need, C.byref(h)) == EWORKSPACE
    assert lib.sfi_create(C.byref(good_cfg()), fake, need - 1, C.byref(h)) == EWORKSPACE
    assert lib.sfi_create(C.byref(good_cfg(head_dim=96)), fake, need, C.byref(h)) == EUNSUPPORTED
    assert lib.sfi_create(C.byref(good_cfg(k_stride_t=132)), fake, need, C.byref(h)) == EALIGN
    assert h.value is None


def test_status_texts():
    for code in (0, -1, -2, -3, -4, -5, -6):
        assert sfi.sfi_strerror(code) and sfi.sfi_strerror(code) != "unknown status"
    assert sfi.sfi_strerror(-99) == "unknown status"
    assert sfi.sfi_destroy is not None
    with pytest.raises(sfi.SfiError):
        sfi.sfi_destroy(None)


def test_bench_refuses_more_than_one_gpu():
    import subprocess
    import sys
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True, text=True)
    assert r.returncode != 0 and "one GPU" in r.stderr


def test_hot_calls_reject_bad_arguments_before_any_launch():
    """A context over a never-dereferenced workspace address: every call below returns an error code
    from the host-side checks, so nothing is launched (this runs without a GPU)."""
    lib = sfi.load_library()
    cfg = good_cfg()
    need = sfi.sfi_workspace_bytes(cfg)
    h = C.c_void_p()
    assert lib.sfi_create(C.byref(cfg), 0x10000, need, C.byref(h)) == OK and h.value
    p = 0x20000  # stands for any 16-byte aligned device pointer; never used by a failing call
    try:
        assert lib.sfi_slow_step(h, None, p, p, p, 0, 64, p, p, p, None) == EINVAL
        assert lib.sfi_slow_step(h, p, p, p, p, 0, 64, p, None, p, None) == EINVAL
        assert lib.sfi_slow_step(h, p, p, p, p, 0, cfg.max_budget + 1, p, p, p, None) == EINVAL
        assert lib.sfi_slow_step(h, p, p, p, p, 0, -1, p, p, p, None) == EINVAL
        assert lib.sfi_slow_step(h, p, p, p, p, cfg.max_ctx + 1, 64, p, p, p, None) == EINVAL
        assert lib.sfi_slow_step(h, p + 2, p, p, p, 0, 64, p, p, p, None) == EALIGN
        assert lib.sfi_slow_step(h, p, p, p, p, 0, 64, p + 4, p, p, None) == EALIGN
        assert lib.sfi_dense_attn(h, p, p, None, p, 0, p, None) == EINVAL
        assert lib.sfi_fast_step(h, p, p, p, None, p, 64, p, p, p, None) == EINVAL
        assert lib.sfi_fast_step(h, p, p, p, p, p, cfg.max_budget + 1, p, p, p, None) == EINVAL
        assert lib.sfi_fast_step(h, p, p, p, p, p, 64, p + 1, p, p, None) == EALIGN
        assert lib.sfi_mixed_step(h, p, p, p, None, p, p, 0, 64, p, p, p, None) == EINVAL
        assert lib.sfi_slow_attn(h, p, p, p, None, 0, p, None) == EINVAL
        assert lib.sfi_slow_attn(h, p, p, p, p, -1, p, None) == EINVAL
        assert lib.sfi_slow_select(h, p, 0, 64, None, p, None) == EINVAL
        assert lib.sfi_slow_select(h, p, 0, cfg.max_budget + 1, p, p, None) == EINVAL
        assert lib.sfi_slow_select(h, p + 2, 0, 64, p, p, None) == EALIGN
        assert lib.sfi_evidence_add(h, p, p, None, p, 0, p, 1, None) == EINVAL   # an output needs V
        assert lib.sfi_evidence_add(h, p, None, None, p, 0, None, 1, None) == EINVAL
        assert lib.sfi_evidence_add(h, p, p + 2, None, p, 0, None, 1, None) == EALIGN
        assert lib.sfi_evidence_add(h, p, p, p, p, cfg.max_ctx + 1, p, 1, None) == EINVAL
        assert lib.sfi_device_status(h, None, 1, None) == EINVAL
        assert lib.sfi_device_status(None, C.byref(C.c_int32()), 1, None) == EINVAL
        assert lib.sfi_evidence_select(h, 0, p, 0, 64, p, p, None) == EINVAL
        assert lib.sfi_evidence_select(h, 4, p, 0, 64, None, p, None) == EINVAL
        assert lib.sfi_evidence_select(h, 4, p, 0, cfg.max_budget + 1, p, p, None) == EINVAL
        # compact buffers: c_rows >= n_sink + sel_stride, strides cover the rows, 16-byte aligned bases
        rows = cfg.n_sink + 64
        sb, sh = 2 * rows * 128, rows * 128
        i64 = C.c_int64
        assert lib.sfi_reorg(h, p, p, p, p, 64, p, None, None, p, i64(sb), i64(sh), rows, None) == EINVAL
        assert lib.sfi_reorg(h, p, p, p, p, 64, p, None, p, p, i64(sb), i64(sh), rows - 1, None) == EINVAL
        assert lib.sfi_reorg(h, p, p, p, p, 64, p, None, p, p, i64(sb), i64(sh - 8), rows, None) == EINVAL
        assert lib.sfi_reorg(h, p, p, p, p, 64, p, None, p, p, i64(sh), i64(sh), rows, None) == EINVAL
        assert lib.sfi_reorg(h, p, p, p, p, cfg.max_budget + 1, p, None, p, p, i64(8 * sb), i64(4 * sh), 4 * rows, None) == EINVAL
        assert lib.sfi_reorg(h, p, p, p, p, 64, p, None, p + 8, p, i64(sb), i64(sh), rows, None) == EALIGN
        assert lib.sfi_reorg(h, p, p, None, p, 64, p, None, p, p, i64(sb), i64(sh), rows, None) == EINVAL
        assert lib.sfi_fast_step_compact(h, p, p, p, i64(sb), i64(sh), rows - 1, p, 64, p, p, p, p, p, None) == EINVAL
        assert lib.sfi_fast_step_compact(h, p, None, p, i64(sb), i64(sh), rows, p, 64, p, p, p, p, p, None) == EINVAL
        assert lib.sfi_fast_step_compact(h, p, p, p, i64(sb), i64(sh), rows, None, 64, p, p, p, p, p, None) == EINVAL
        assert lib.sfi_fast_step_compact(h, p, p, p, i64(4 * sb), i64(sh + 4), rows, p, 64, p, p, p, p, p, None) == EALIGN
        assert lib.sfi_trigger(h, None, p, 100, 8, p, p, None) == EINVAL
        assert lib.sfi_trigger(h, p, p, 0, 8, p, p, None) == EINVAL
        assert lib.sfi_trigger(h, p, p, 100, -1, p, p, None) == EINVAL
        assert lib.sfi_trigger(h, p, p + 2, 100, 8, p, p, None) == EALIGN
        assert lib.sfi_advance(h, None, p, None) == EINVAL
        assert lib.sfi_stage_times(h, None, None) == EINVAL
        assert lib.sfi_set_profiling(h, -1) == EINVAL
        assert lib.sfi_set_tuning(None, 1, 1, 0) == EINVAL
        assert lib.sfi_set_tuning(h, 0, 0, 3) == EINVAL
        assert lib.sfi_set_tuning(h, 0, 0, 2) == OK
        assert lib.sfi_plan_splits(None, 0, 64, None, None) == EINVAL
        assert lib.sfi_plan_splits(h, cfg.max_ctx + 1, 64, None, None) == EINVAL
        assert lib.sfi_plan_splits(h, 0, cfg.max_budget + 1, None, None) == EINVAL
        d, f = C.c_int32(-1), C.c_int32(-1)
        assert lib.sfi_query_splits(h, C.byref(d), C.byref(f)) == OK and d.value == 0 and f.value == 0
    finally:
        assert lib.sfi_destroy(h) == OK


def paged_cfg(**over):
    """[blocks][Hkv][page][128] pools of 64-row blocks."""
    c = good_cfg(page_size=64, k_stride_b=0, v_stride_b=0, k_stride_t=128, v_stride_t=128, k_stride_h=64 * 128,
                 v_stride_h=64 * 128, k_stride_page=2 * 64 * 128, v_stride_page=2 * 64 * 128)
    for k, v in over.items():
        setattr(c, k, v)
    return c


def test_paged_config_and_block_table_validation():
    assert sfi.sfi_workspace_bytes(paged_cfg()) == sfi.sfi_workspace_bytes(good_cfg())
    assert sfi.sfi_workspace_bytes(paged_cfg(k_stride_page=0, v_stride_page=0, k_stride_t=256, v_stride_t=256,
                                             k_stride_h=128, v_stride_h=128)) > 0  # [blocks][page][Hkv][128]
    for bad in (dict(page_size=8), dict(page_size=48), dict(page_size=1 << 17), dict(k_stride_b=4096),
                dict(k_stride_page=64 * 128 + 8), dict(v_stride_page=0), dict(v_stride_page=4 * 64 * 128),
                dict(k_stride_page=32 * 128, v_stride_page=32 * 128), dict(k_stride_page=-128)):
        assert sfi.sfi_workspace_bytes(paged_cfg(**bad)) == 0, bad
    lib = sfi.load_library()
    p = 0x20000
    for cfg, cases in ((good_cfg(), [((p, 64, 10), EINVAL)]),          # a flat context takes no table
                       (paged_cfg(), [((p, 63, 10), EINVAL),           # 4096 rows need 64 entries per sequence
                                      ((p, 64, 0), EINVAL), ((p + 2, 64, 10), EALIGN),
                                      ((p, 64, 1 << 25), EUNSUPPORTED),  # more rows than a 32-bit row number addresses
                                      ((p, 64, 1000), OK), ((None, 0, 0), OK)])):
        h = C.c_void_p()
        assert lib.sfi_create(C.byref(cfg), 0x10000, sfi.sfi_workspace_bytes(cfg), C.byref(h)) == OK
        try:
            for (tbl, stride, n_blocks), want in cases:
                assert lib.sfi_set_block_table(h, tbl, stride, n_blocks) == want, (tbl, stride, n_blocks)
            if cfg.page_size:  # detached: hot calls refuse to run
                assert lib.sfi_dense_attn(h, p, p, p, p, 0, p, None) == EINVAL
                assert lib.sfi_reorg(h, p, p, p, p, 64, p, None, p, p, C.c_int64(2 * 68 * 128), C.c_int64(68 * 128), 68, None) == EINVAL
        finally:
            assert lib.sfi_destroy(h) == OK


def _plan(B, Hkv, ctx, budget, recent=128, tuning=None):
    """Launch plan (dense splits, fast splits) of a context of this shape; the library assumes 256
    compute units where there is no device."""
    lib = sfi.load_library()
    c = good_cfg(batch=B, n_q_heads=4 * Hkv, n_kv_heads=Hkv, max_ctx=ctx, max_budget=budget, recent=recent,
                 k_stride_h=128 * ctx, k_stride_b=Hkv * 128 * ctx, v_stride_h=128 * ctx, v_stride_b=Hkv * 128 * ctx)
    h = C.c_void_p()
    assert lib.sfi_create(C.byref(c), 0x10000, sfi.sfi_workspace_bytes(c), C.byref(h)) == OK
    try:
        if tuning:
            assert lib.sfi_set_tuning(h, *tuning) == OK
        d, f = C.c_int32(-1), C.c_int32(-1)
        assert lib.sfi_plan_splits(h, 0, budget, C.byref(d), C.byref(f)) == OK
        return d.value, f.value
    finally:
        assert lib.sfi_destroy(h) == OK


def test_launch_plan_loads_the_compute_units_evenly():
    """Host logic of the launch policy (256 compute units).  Where the (sequence, KV head) pairs divide the
    compute units the plan is one workgroup per unit; where they do not, it must not leave a second round
    that is almost empty (264 pairs: one workgroup per pair would take two shares of time for 1.03 of work)."""
    import torch
    if torch.cuda.is_available():
        pytest.skip("the plan depends on the device's compute-unit count; this test pins the 256-unit default")
    # the benchmark's shape: 256 dense workgroups; the fast step's 69 tiles make three trips per wave with 6,
    # 7 or 8 workgroups per pair alike, so it takes the fewest
    assert _plan(4, 8, 32768 + 64, 2048) == (8, 6)
    # one long stream: two trips per wave need 18 workgroups per pair; more only add records to merge
    assert _plan(1, 8, 131072 + 64, 4096, recent=256) == (32, 18)
    assert _plan(32, 8, 32768, 2048) == (1, 1)                # one pair per unit: no split, no merge
    assert _plan(64, 8, 32768, 2048) == (1, 1)                # two full rounds
    for B in (12, 24, 33, 40, 48):
        pairs = 8 * B
        d, f = _plan(B, 8, 32768, 2048)
        for s, tiles in ((d, 1024 + 5), (f, (4 + 2048 + 128 + 31) // 32)):
            r = pairs * s / 256
            assert 1 <= s <= 63 and 4 * s <= tiles + 3
            assert r / -(-r // 1) >= 0.68, f"B={B}: {s} workgroups per pair load the units {r:.2f} rounds"
    assert _plan(33, 8, 32768, 2048)[0] in (8, 9)              # 8.25 or 9.28 rounds of workgroups, not 1.03
    # a tiny problem spreads over as many workgroups as it has tiles for
    assert _plan(1, 2, 777, 50, recent=32) == (7, 1 + (4 + 50 + 32) // 128)
    # knobs: a total for the dense launch, tiles per wave for the gather launch; negative restores the default
    assert _plan(4, 8, 32768, 2048, tuning=(512, 1, 0)) == (16, 18)
    assert _plan(4, 8, 32768, 2048, tuning=(-1, -1, 0)) == (8, 6)


def test_header_is_plain_c_and_the_binding_mirrors_its_config_layout(tmp_path):
    """include/sfi.h compiles as strict C99 on its own, and every field of the ctypes mirror of
    sfi_config sits at the offset and has the size the C compiler gives it (a field added to one side
    only would shift everything behind it without any error)."""
    import subprocess

    lines = ['#include <stddef.h>', '#include <stdio.h>', '#include "sfi.h"', 'int main(void) {',
             '  printf("sizeof %zu\\n", sizeof(sfi_config));']
    for name, _ in SfiConfig._fields_:
        lines.append(f'  printf("{name} %zu %zu\\n", offsetof(sfi_config, {name}), sizeof(((sfi_config*)0)->{name}));')
    lines += ['  return 0;', '}']
    src = tmp_path / "layout.c"
    src.write_text("\n".join(lines) + "\n")
    exe = tmp_path / "layout"
    subprocess.run(["gcc", "-std=c99", "-pedantic", "-Wall", "-Wextra", "-Werror", "-I", os.path.join(ROOT, "include"),
                    str(src), "-o", str(exe)], check=True)
    got = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split("\n")
    assert got[0] == f"sizeof {C.sizeof(SfiConfig)}"
    seen = {}
    for ln in got[1:]:
        if ln:
            name, off, size = ln.split()
            seen[name] = (int(off), int(size))
    for name, ctype in SfiConfig._fields_:
        assert seen[name] == (getattr(SfiConfig, name).offset, C.sizeof(ctype)), name
    # and the header has no field the mirror lacks: its struct body names exactly these identifiers
    text = open(os.path.join(ROOT, "include", "sfi.h")).read()
    body = text[text.index("typedef struct sfi_config"):]
    body = body[:body.index("} sfi_config;")]
    body = re.sub(r"/\*.*?\*/", "", body, flags=re.S)
    decl = re.findall(r"\b(?:int32_t|int64_t|float)\s+([^;]+);", body)
    names = [n.strip() for d in decl for n in d.split(",")]
    assert names == [n for n, _ in SfiConfig._fields_]

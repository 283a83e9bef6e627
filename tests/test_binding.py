"""The Python side of the boundary (no GPU): which library the hot calls run, and how arguments become C values."""
import ctypes as C
import os
import shutil
import subprocess
import sys

import numpy as np
import pytest

import paper_2603_12038_amd as sfi

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PACKAGE = os.path.basename(os.path.dirname(sfi.__file__))

COPY_PROBE = """
import os, {package} as sfi
assert os.path.dirname(os.path.realpath(sfi.__file__)) == {want!r}, sfi.__file__
sfi.load_library()
try:
    sfi.sfi_fast_step(0, 0, 0, 0, 0, 0, 1, 0, 0, 0, 0)  # no context: refused before anything is launched
except sfi.SfiError as e:
    assert e.code == -1, e.code
else:
    raise SystemExit("a call without a context was accepted")
maps = {{ln.split()[-1] for ln in open("/proc/self/maps") if "sfi" in os.path.basename(ln.split()[-1])}}
print(sorted(os.path.realpath(m) for m in maps))
"""


def test_a_copied_package_runs_its_own_library(tmp_path):
    """A built tree may be moved: context calls (ctypes) and hot calls (CPython module) both run the copy's libsfi.so."""
    here = os.path.join(os.path.realpath(tmp_path), PACKAGE)
    shutil.copytree(os.path.dirname(sfi.__file__), here, ignore=shutil.ignore_patterns("__pycache__", "csrc"))
    env = {**os.environ, "PYTHONPATH": str(tmp_path)}
    r = subprocess.run([sys.executable, "-c", COPY_PROBE.format(package=PACKAGE, want=here)], cwd=tmp_path, env=env,
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    assert r.stdout.strip() == str([os.path.join(here, "_sfi.so"), os.path.join(here, "libsfi.so")])


FAST_STEP = dict(ctx=0, q=0, K=0, V=0, sel_idx=0, n_sel=0, sel_stride=1, recent_start=0, ctx_len=0, out=0, stream=0)


class _Unusable:
    """No tensor, address or ctypes pointer; counts how often it is asked for anything."""
    asked = 0

    def __getattr__(self, name):
        type(self).asked += 1
        raise AttributeError(f"no {name} here")


@pytest.mark.parametrize("name, value, error, text", [
    ("sel_stride", 1.5, TypeError, "'float' object cannot be interpreted as an integer"),
    ("sel_stride", "1", TypeError, "'str' object cannot be interpreted as an integer"),
    ("sel_stride", None, TypeError, "'NoneType' object cannot be interpreted as an integer"),
    ("K", 1.5, AttributeError, "'float' object has no attribute 'data_ptr'"),
    ("ctx", [], AttributeError, "'list' object has no attribute 'data_ptr'"),
    ("stream", 1.5, AttributeError, "'float' object has no attribute 'cuda_stream'"),
])
def test_an_argument_of_the_wrong_type_raises_its_own_error(name, value, error, text):
    """The first bad argument's error comes out, whatever follows it (a ctypes pointer's conversion looks for data_ptr first)."""
    args = {**FAST_STEP, "out": C.c_void_p(0), name: value}
    with pytest.raises(error, match=text):
        sfi.sfi_fast_step(*args.values())


def test_no_argument_is_looked_at_behind_a_bad_one():
    _Unusable.asked = 0
    with pytest.raises(TypeError):
        sfi.sfi_fast_step(*{**FAST_STEP, "sel_stride": 1.5, "out": _Unusable()}.values())
    assert _Unusable.asked == 0


def test_accepted_forms_reach_the_library():
    """None, addresses, ctypes pointers and integer-like objects: the call gets as far as the library's own refusal."""
    for over in (dict(q=None), dict(ctx=C.c_void_p(None)), dict(out=C.c_void_p(64)), dict(sel_stride=np.int32(1))):
        with pytest.raises(sfi.SfiError) as e:
            sfi.sfi_fast_step(*{**FAST_STEP, **over}.values())
        assert e.value.code == -1

"""The Python side of the boundary (no GPU): which library the hot calls run, and how arguments become C values."""
import os
import shutil
import subprocess
import sys

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

"""What the library asks the HIP runtime for, counted by a preloaded shim (no GPU: the launches fail,
after the host side of the calls has run)."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SHIM = r"""
static int asked;
extern "C" int shim_asked() { return asked; }
extern "C" int hipGetDevice(int *dev) { *dev = 0; return 0; }
extern "C" int hipDeviceGetAttribute(int *v, int attr, int dev) { (void)attr; (void)dev; ++asked; *v = 163840; return 0; }
"""

CALLS = r"""
import ctypes as C, sys
import paper_2504_14966_amd.sloanneal as sl
L, shim = sl.load_library(), C.CDLL(sys.argv[1])
q = sl._Queue(24, 256, 256, 256, 256)
static, cont = (sl._Model(8, p, 2000, 40, 8000, 300, 2, 0, 1 << 31) for p in (0, 1))
fit = sl.FitModel(8, 0, **sl.TABLE2_10NS)
calls = (lambda: L.sched_eval(C.byref(q), C.byref(static), 256, 4, 256, None, None),
         lambda: L.sched_eval(C.byref(q), C.byref(cont), 256, 4, 256, None, None),
         lambda: L.sched_eval_batches(C.byref(q), C.byref(static), 256, 256, 4, 256, None, None),
         lambda: L.sched_eval_fit(C.byref(q), C.byref(fit), None, 256, None, 4, 256, None, None))
for c in calls * 3:
    print(c(), shim.shim_asked())
"""


def test_evaluation_calls_ask_for_the_device_limits_once(tmp_path):
    """A small evaluation call is bound by the host's launch: the limits of a device, which never
    change, are asked for by the first call only."""
    import torch
    if torch.cuda.is_available():
        pytest.skip("counts host calls where no kernel can start")
    (tmp_path / "shim.cpp").write_text(SHIM)
    so = str(tmp_path / "shim.so")
    subprocess.run(["g++", "-shared", "-fPIC", "-O1", str(tmp_path / "shim.cpp"), "-o", so], check=True)
    env = dict(os.environ, PYTHONPATH=ROOT)
    env["LD_PRELOAD"] = ":".join([so] + ([env["LD_PRELOAD"]] if env.get("LD_PRELOAD") else []))
    out = subprocess.run([sys.executable, "-c", CALLS, so], env=env, cwd=ROOT, capture_output=True, text=True, timeout=300)
    assert out.returncode == 0, out.stderr[-2000:]
    got = [tuple(int(x) for x in line.split()) for line in out.stdout.strip().splitlines()]
    assert len(got) == 12 and all(rc == -4 for rc, _ in got), got  # SCHED_EHIP: no device to launch on
    assert [asked for _, asked in got] == [2] * 12, got

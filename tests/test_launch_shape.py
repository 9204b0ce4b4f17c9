"""Workgroup shapes of the kernels with a block of LDS per chain (host arithmetic, compiled with g++)."""
import ctypes as C
import os
import subprocess
import sys

import numpy as np
import pytest

sys.path.insert(0, os.path.dirname(__file__))
from gpu_helpers import lane_shape  # noqa: E402

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2504_14966_amd", "csrc")
LIM, CUS = 160 * 1024, 256

SHIM = r"""
#include "launch_shape.h"
extern "C" void shapes(long k, const int *chains, const long *shared, const long *per, int lim, int cus, int *out) {
  for (long i = 0; i < k; ++i) {
    const sa::LdsShape s = sa::lds_shape(chains[i], (size_t)shared[i], (size_t)per[i], lim, cus);
    out[3 * i] = s.fit;
    out[3 * i + 1] = s.waves;
    out[3 * i + 2] = sa::lds_suffices(s, chains[i], cus);
    out[3 * i + 2] |= sa::lds_shape_small(chains[i], (size_t)shared[i], (size_t)per[i], lim, cus).waves << 8;
  }
}
"""


@pytest.fixture(scope="module")
def shapes(tmp_path_factory):
    d = tmp_path_factory.mktemp("shape")
    (d / "shim.cpp").write_text(SHIM)
    so = str(d / "shim.so")
    subprocess.run(["g++", "-std=c++17", "-O2", "-shared", "-fPIC", "-I", CSRC, str(d / "shim.cpp"), "-o", so], check=True)
    lib = C.CDLL(so)

    def call(chains, shared, per, small=False):
        chains, shared, per = np.broadcast_arrays(chains, shared, per)
        c, s, p = (np.ascontiguousarray(a, t) for a, t in ((chains, np.int32), (shared, np.int64), (per, np.int64)))
        out = np.zeros((c.size, 3), np.int32)
        lib.shapes(C.c_long(c.size), c.ctypes, s.ctypes, p.ctypes, LIM, CUS, out.ctypes)
        fit, waves, rest = out.reshape(c.shape + (3,)).transpose(-1, *range(c.ndim))
        return (fit, waves, rest & 255) + ((rest >> 8,) if small else ())
    return call


def _static_chain_bytes(n, B):
    """LDS of one chain of the kernel with several batches per row: the order (u16), the finish
    offsets (u32, a spare one) and two 48-byte records per batch."""
    return (2 * n + 15) // 16 * 16 + (4 * (n + 1) + 15) // 16 * 16 + 2 * 48 * -(-n // B)


def test_delta_kernels_keep_what_power_of_two_workgroups_gave_them(shapes):
    """Workgroups of 1, 2, 4, 8 or 16 chains were accepted when they held four chains or when one
    pass held every chain. Every such call keeps the delta kernel, whatever count spreads its chains:
    1500 chains where five fit go as workgroups of three."""
    per = np.arange(1000, 60000, 331)[:, None, None]
    shared = np.array([1056, 4816, 9616, 14416, 16400])[None, :, None]
    chains = np.concatenate([np.arange(1, 2400, 7), np.arange(2400, 9000, 97)])[None, None, :]
    full = np.broadcast_arrays(chains, shared, per)
    waves = np.ones(full[0].shape, np.int64)
    for _ in range(4):
        waves = np.where((waves < 16) & (waves * CUS < full[0]), waves * 2, waves)
    for _ in range(4):
        waves = np.where((waves > 1) & (full[1] + full[2] * waves > LIM), waves // 2, waves)
    was = (full[1] + full[2] * waves <= LIM) & ((waves >= 4) | (waves * CUS >= full[0]))
    fit, spread, now = shapes(chains, shared, per)
    assert was.any() and (~was).any()
    assert not (was & (now == 0)).any()
    # never more chains in a workgroup than fit, and enough workgroups in the passes for all
    assert ((spread >= 1) == (fit >= 1)).all() and (spread <= fit).all() and (fit <= 16).all()
    held = fit > 0
    passes = np.where(held, -(-full[0] // np.maximum(fit * CUS, 1)), 1)
    assert (spread * passes * CUS >= full[0])[held].all()


@pytest.mark.parametrize("n,B,chains", [(900, 4, 1500), (300, 1, 1500), (600, 2, 1200), (1024, 4, 2200), (700, 3, 1300)])
def test_delta_kernel_sizes_where_the_spread_is_three(shapes, n, B, chains):
    fit, waves, now = shapes(chains, 16 * (n + 1), _static_chain_bytes(n, B))
    assert fit in (4, 5) and waves == 3 and now == 1


EVAL_SHIM = r"""
#include "launch_shape.h"
extern "C" int any_pays(int n, int B, int chains, int cus) { return sa::reg_any_pays(n, B, chains, cus); }
extern "C" int rows_pay(int n, int B) { return sa::rows_pay(n, B); }
extern "C" int reg(int chains, int cus) { return sa::reg_shape(chains, cus); }
extern "C" int grid(long rows, int waves, long lds, int per_simd, double beyond, int lim, int cus) {
  return sa::eval_grid(rows, waves, (size_t)lds, sa::EvalShape{per_simd, beyond}, lim, cus);
}
"""


@pytest.fixture(scope="module")
def eval_grid(tmp_path_factory):
    d = tmp_path_factory.mktemp("grid")
    (d / "shim.cpp").write_text(EVAL_SHIM)
    so = str(d / "shim.so")
    subprocess.run(["g++", "-std=c++17", "-O2", "-shared", "-fPIC", "-I", CSRC, str(d / "shim.cpp"), "-o", so], check=True)
    lib = C.CDLL(so)
    lib.grid.argtypes = [C.c_long, C.c_int, C.c_long, C.c_int, C.c_double, C.c_int, C.c_int]
    def call(rows, waves, lds, per_simd, beyond):
        return lib.grid(rows, waves, lds, per_simd, beyond, LIM, CUS)
    call.reg, call.any_pays, call.rows_pay = lib.reg, lib.any_pays, lib.rows_pay
    return call


# (per SIMD, beyond, waves, LDS of a workgroup, held at once): the static, fitted, layout and any-width
# kernels at short and long queues
@pytest.mark.parametrize("per_simd,beyond,waves,lds,held", [(8, 1.5, 4, 2304, 2048), (8, 1.5, 4, 32384, 1280),
                                                            (7, 1.5, 4, 6144, 1792), (7, 2.5, 4, 14000, 1792),
                                                            (5, 2.5, 4, 6000, 1280), (5, 2.5, 4, 91000, 256),
                                                            (5, 2.5, 2, 122000, 256), (5, 2.5, 2, 40000, 1024)])
def test_eval_workgroups_leave_no_thin_last_pass(eval_grid, per_simd, beyond, waves, lds, held):
    """Rows in workgroups held at once, or enough workgroups beyond them: a count a little above what
    the GPU holds (registers and LDS) waits for a last pass that is nearly empty."""
    for rows in sorted({1, 3, 4, 5, 255 * waves, held * waves, held * waves + 1, *range(700, 400000, 911), 1 << 20, 1 << 24}):
        g, want = eval_grid(rows, waves, lds, per_simd, beyond), -(-rows // waves)
        assert 1 <= g <= want and g <= max(8192, held), rows
        assert g == want if want <= held else (g == held or g >= beyond * held), (rows, g)


def test_eval_workgroups_of_measured_calls(eval_grid):
    assert eval_grid(4500, 4, 91136, 5, 2.5) == 256    # continuous, 700 requests: 281 took 1.6 times as long
    assert eval_grid(32768, 4, 14144, 7, 2.5) == 1792  # layouts, 400 requests: 2048 took 1.4 times as long
    assert eval_grid(32768, 4, 1500, 8, 1.5) == 2048   # 10 requests: 8192 took twice as long
    assert eval_grid(1 << 20, 4, 8000, 8, 1.5) == 8192


def test_fitted_chains_beyond_one_workgroup_per_cu(shapes):
    """Blocks of 28 bytes per request and a fixed part: beyond 16 chains per CU the workgroups are of
    four, one chain per SIMD, while the LDS holds five of them; up to there the spread of the others."""
    n = np.arange(65, 1025, 13)[:, None]
    chains = np.concatenate([np.arange(1, 4097, 61), [4096], np.arange(4097, 20000, 307)])[None, :]
    per = (2 * n + 15) // 16 * 16 + (n + 15) // 16 * 16 + 1440
    fit, waves, _, small = shapes(chains, 16 * n, per, small=True)
    nn, cc, pp = np.broadcast_arrays(n, chains, per)
    packed = (cc > 16 * CUS) & (5 * (16 * nn + 4 * pp) <= LIM)
    assert (fit == 16).all() and packed.any() and (packed != (cc > 16 * CUS)).any()
    assert (small[packed] == 4).all() and (small[~packed] == waves[~packed]).all()
    assert shapes(5000, 16 * 256, 2208, small=True)[3] == 4


@pytest.mark.parametrize("kind,B,longest", [("static", 1, 47), ("static", 4, 144), ("static", 16, 306), ("static", 64, 431),
                                            ("layout", 4, 52), ("layout", 8, 88), ("layout", 16, 144), ("layout", 32, 200),
                                            ("layout", 64, 256)])
def test_longest_queues_of_the_lane_kernels(kind, B, longest):
    """Four waves per workgroup or none: where the LDS ends. (300 requests by layout go to the
    one-order-per-wave kernel at any row count.)"""
    rows = 1 << 20
    taken = [n for n in range(2, 1025) if lane_shape(kind, n, B, rows)[0]]
    assert taken[-1] == longest and taken == list(range(2, longest + 1))
    assert lane_shape("layout", 300, 64, rows)[0] == 0
    waves, lds, cap = lane_shape(kind, longest, B, rows)
    assert waves == 4 and lds <= LIM - 1024 and cap >= -(-longest // B)


def test_continuous_lane_kernel_steps_its_waves_down():
    rows = 1 << 20
    got = {(n, B): lane_shape("continuous", n, B, rows) for n in (2, 24, 256, 1024) for B in (1, 9, 32, 64)}
    assert all(w > 0 and lds <= LIM - 1024 for w, lds, _ in got.values())
    assert got[(1024, 64)][0] < got[(256, 32)][0] == 4
    assert [got[(1024, B)][2] for B in (1, 9, 32, 64)] == [8, 16, 32, 64]
    assert lane_shape("continuous", 256, 32, 32767)[0] == 0 and lane_shape("continuous", 1024, 32, 8192)[0] > 0


def test_register_kernels_put_one_chain_on_a_simd(eval_grid):
    """From three chains per CU on, one workgroup per CU holds what it must: no two of them share SIMDs
    while others idle. Up to two per CU one chain each."""
    for chains in range(1, 6000):
        w = eval_grid.reg(chains, CUS)
        assert w == 1 if chains <= 2 * CUS else w in (3, 4), chains
        assert chains <= 2 * CUS or w * CUS >= min(chains, 4 * CUS), chains
        assert chains < 4 * CUS or w == 4, chains


def test_kernel_of_two_batches(eval_grid):
    """Two batches of 17 to 32: the register kernel, but the delta kernel between 8 and 16 chains per CU,
    and never limit rows; one batch: the delta kernel; three and more keep theirs at any chain count."""
    for B in range(17, 33):
        for chains in (1, 64, 2048, 2049, 3000, 4096, 4097, 20000):
            for n in range(2, 65):
                want = n > B and (n > 2 * B or not 8 * CUS < chains <= 16 * CUS)
                assert eval_grid.any_pays(n, B, chains, CUS) == want, (n, B, chains)
        assert [n for n in range(2, 1025) if eval_grid.rows_pay(n, B)] == list(range(2 * B + 1, 32 * B + 1))[:1024 - 2 * B]
    for B in (3, 5, 12, 15):
        assert all(eval_grid.any_pays(n, B, 3000, CUS) for n in range(B + 1, 65)) and not eval_grid.rows_pay(400, B)
    assert all(eval_grid.rows_pay(n, B) for n in (2, 50, 64, 1024) for B in (33, 48, 64))
    assert not eval_grid.any_pays(64, 33, 1, CUS)

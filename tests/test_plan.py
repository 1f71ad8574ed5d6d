"""Launch plans (host only): what the planner's rules promise about filling the
chip, for grids on both sides of their lines."""
import ctypes

import pytest

import paper_1812_04135_amd as R
import workloads as W

CUS = 256


def _plan(n, bc="periodic"):
    return R.rsst_plan(R.make_config(W.base_cfg(len(n), n, xi=2.0, bc_lo=[bc] * len(n))))


def test_plan_refuses_what_init_refuses():
    L = R.lib()
    a = (ctypes.c_int * 5)()
    bad = R.make_config(W.base_cfg(2, [64, 64], xi=2.0))
    bad.xi = 0.5
    assert L.rsst_plan(ctypes.byref(bad), a) == -1
    assert L.rsst_plan(ctypes.byref(R.make_config(W.base_cfg(2, [1025, 8], xi=2.0))), a) == -4
    assert L.rsst_plan(None, a) == -1
    assert L.rsst_plan(ctypes.byref(R.make_config(W.base_cfg(1, [64], xi=2.0))), None) == -1


@pytest.mark.parametrize("nx,ns,waves,per_cu", [(8, 4, 2, 4), (64, 4, 2, 4), (64, 6, 3, 2), (8, 8, 4, 2), (128, 4, 4, 2),
                                                (100, 5, 4, 2), (8, 10, 5, 1), (128, 6, 6, 1), (64, 16, 8, 1),
                                                (200, 4, 8, 1), (512, 4, 8, 1)])
@pytest.mark.parametrize("nz", [300, 500, 1000, 2000, 4000])
def test_3d_tiles_fill_the_cus(nx, ns, waves, per_cu, nz):
    """Eight waves to a CU: a grid with fewer rows than a tile runs several
    workgroups on each, in one round where a chunk of 128 planes allows it,
    and that round at least 0.8 full where the chunk is of four or more."""
    p = _plan([nx, ns, nz])
    assert p["waves"] == waves
    tiles = p["blocks"] // -(-nz // p["chunk"])
    assert p["blocks"] <= CUS * per_cu * max(1, -(-tiles * -(-nz // 128) // (CUS * per_cu)))
    if p["chunk"] >= 4:
        assert p["blocks"] >= 0.8 * CUS * per_cu

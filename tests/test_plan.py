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


# whole rows or strips: (grid, walls in x, rows)
@pytest.mark.parametrize("n,bc,rows", [
    ([64, 100], "periodic", 0), ([64, 100], "reflect", 1), ([60, 100], "reflect", 0), ([64, 4096], "reflect", 1), ([64, 4100], "reflect", 0), ([64, 65536], "reflect", 1),
    ([64, 10 ** 6], "reflect", 1), ([128, 2048], "periodic", 1), ([128, 30000], "periodic", 1), ([120, 30000], "periodic", 0),
    ([256, 1024], "periodic", 1), ([256, 1100], "periodic", 0), ([256, 16384], "periodic", 1), ([240, 16384], "periodic", 0),
    ([192, 1365], "periodic", 1), ([192, 5000], "periodic", 0), ([192, 20000], "periodic", 1), ([320, 204], "periodic", 1), ([320, 400], "periodic", 0),
    ([448, 256], "periodic", 1), ([448, 585], "periodic", 0), ([512, 512], "periodic", 1), ([512, 513], "periodic", 0),
    ([512, 2000], "periodic", 0), ([512, 16384], "periodic", 0), ([1024, 16], "periodic", 0), ([1024, 3000], "periodic", 0),
    ([1024, 32768], "periodic", 0), ([1000, 30000], "periodic", 0), ([700, 40000], "periodic", 0)])
def test_2d_whole_rows_where_their_waves_are_full_and_even(n, bc, rows):
    p = _plan(n, bc)
    assert p["rows"] == rows
    assert p["waves"] == (-(-n[0] // 64) if rows else 4)


@pytest.mark.parametrize("nx", [64, 128, 192, 256, 512])
@pytest.mark.parametrize("nm", [64, 1000, 4096, 20000, 65536, 262144, 10 ** 6])
def test_2d_whole_row_chunks(nx, nm):
    """At most about one round of all the workgroups that fit (each reads the
    maxima of all), or 35 rows, and no chunk of a power of two of 8 rows or
    more."""
    if nx * nm * 32 >= 1 << 31:
        pytest.skip("a 2D state of 2 GiB")
    p = _plan([nx, nm], "reflect")
    if not p["rows"]:
        return
    full = CUS * (16 // (nx // 64))
    assert p["blocks"] == -(-nm // p["chunk"])
    assert p["chunk"] <= max(35, -(-nm // full) + 1)
    assert p["chunk"] < 8 or p["chunk"] % 2 == 1

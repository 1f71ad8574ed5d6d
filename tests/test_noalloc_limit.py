"""Which states fit the fixed scratch of rsst_step_noalloc: the state's size
alone decides (its copy and 512 B within 64 MiB), not the launch plan, whose
count of maxima differs from shape to shape and from planner to planner."""
import ctypes

import numpy as np
import pytest

import paper_1812_04135_amd as R
import workloads as W

torch = pytest.importorskip("torch")

LIMIT = 64 << 20
# rows of 4, 60, 64, 256, 1000 cells and the widest 3D tiles, each grid the
# largest along its last axis; and many tiles of few planes
SHAPES = [[4, None], [5, None], [60, None], [64, None], [120, None], [256, None], [500, None], [1000, None],
          [4, 4, None], [8, 6, None], [8, 5, None], [64, 64, None], [200, None, 4], [4, None, 4], [512, None, 4]]


def _grid(shape, size):
    """shape with its open axis as long as fits, and one longer."""
    nv = len(shape) + 2
    per = nv * size
    for v in shape:
        per *= v or 1
    m = (LIMIT - 512) // per
    return [v or m for v in shape], [v or m + 1 for v in shape]


def _code(n, prec, bc):
    c = R.make_config(W.base_cfg(len(n), n, xi=2.0, bc_lo=[bc] * len(n)), prec=prec)
    if prec != "fp64":
        c.bg = ctypes.c_void_p(8)  # never touched
    return R.lib().rsst_step_noalloc(ctypes.byref(c), ctypes.c_void_p(0x1000), ctypes.c_double(0.0), None, None)


@pytest.mark.skipif(torch.cuda.is_available(), reason="the state pointer is not a state: no device may run it")
@pytest.mark.parametrize("bc", ["periodic", "reflect"])
@pytest.mark.parametrize("prec,size", [("fp64", 8), ("fp32_pert", 4)])
def test_limit_is_the_states_size(prec, size, bc):
    for shape in SHAPES:
        fits, over = _grid(shape, size)
        assert _code(fits, prec, bc) != R.RSST_E_SCRATCH, fits
        assert _code(over, prec, bc) == R.RSST_E_SCRATCH, over


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [[4, None], [256, None], [8, 6, None]])
def test_largest_states_step_like_a_handle(shape):
    n, _ = _grid(shape, 8)
    cfg = W.base_cfg(len(n), n, xi=4.0)
    gen = torch.Generator(device="cuda").manual_seed(17)
    sh = list(reversed(n))
    noise = [0.01 * torch.rand(sh, dtype=torch.float64, device="cuda", generator=gen) for _ in range(len(n) + 2)]
    U0 = torch.stack([1.0 + noise[0]] + noise[1:-1] + [1.5 + noise[-1]]).contiguous()
    print(f"[noalloc limit] n={n}", flush=True)
    U, V = U0.clone(), U0.clone()
    f = torch.full((1,), 7, dtype=torch.int32, device="cuda")
    R.rsst_step_noalloc(R.make_config(cfg), U, 0.0, f)
    s = R.Solver(cfg)
    s.step(V)
    torch.cuda.synchronize()
    assert int(f.item()) == 0 and s.poll() == 0
    s.close()
    assert torch.equal(U, V) and not np.array_equal(U[:, ..., :1].cpu().numpy(), U0[:, ..., :1].cpu().numpy())

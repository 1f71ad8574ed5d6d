"""rsst_steps on 1D rows around the widths at which the waves of the one-launch
run change (56 cells each, 16 waves at most, the seam form beyond): bitwise
the separate rsst_step calls, with walls and a force (whose ghost lanes are
mirror images), both storage types, and an end time inside the run."""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

R = None


def setup_module(module):
    global R
    import paper_1812_04135_amd as lib
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    lib.lib()
    R = lib


def _run(cfg, U0, how, nsteps, **kw):
    U = torch.from_numpy(np.ascontiguousarray(U0)).cuda()
    s = R.Solver(cfg, **kw)
    if how == "steps":
        s.steps(U, nsteps)
    else:
        for _ in range(nsteps):
            s.step(U)
    out = (U.cpu().numpy(), *s.time(), s.poll())
    s.close()
    return out


@pytest.mark.parametrize("bc,g", [("periodic", 0.0), ("reflect", -0.6)])
@pytest.mark.parametrize("n", [4, 5, 8, 55, 56, 57, 112, 113, 169, 256, 895, 896, 897])
def test_widths(n, bc, g):
    cfg, U0 = W.random_state(1, [n], seed_k=1700 + n, xi=3.0, form="pvs", bc_lo=[bc], g=[g])
    print(f"[steps1d halo] n={n} {bc}", flush=True)
    a, b = _run(cfg, U0, "steps", 9), _run(cfg, U0, "step", 9)
    assert np.array_equal(a[0], b[0]) and a[1:] == b[1:]


@pytest.mark.parametrize("axis", [-1, 0])
@pytest.mark.parametrize("bc", ["periodic", "reflect"])
def test_fp32_perturbation(bc, axis):
    n = 117
    cfg, U0 = W.random_state(1, [n], seed_k=1790, xi=3.0, form="dvs", bc_lo=[bc], g=[-0.4 if bc == "reflect" else 0.0])
    bg = U0.mean(axis=1, keepdims=True) if axis == -1 else 0.9 * U0
    kw = dict(prec="fp32_pert", bg=torch.from_numpy(np.ascontiguousarray(bg)).cuda(), bg_axis=axis)
    P0 = (U0 - bg).astype(np.float32)
    a, b = _run(cfg, P0, "steps", 9, **kw), _run(cfg, P0, "step", 9, **kw)
    assert np.array_equal(a[0], b[0]) and a[1:] == b[1:]


def test_end_time_inside_the_run():
    cfg, U0 = W.random_state(1, [130], seed_k=1795, xi=3.0)
    t5 = _run(cfg, U0, "step", 5)[1]
    a, b = _run(cfg, U0, "steps", 12, t_end=t5), _run(cfg, U0, "step", 12, t_end=t5)
    assert np.array_equal(a[0], b[0]) and a[1] == b[1] == t5 and a[3] == b[3] == 0

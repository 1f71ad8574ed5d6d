"""The 3D adjoint passes on both sides of the size up to which every axis of a
cell has a thread of its own (131072 cells), at ragged and smallest sizes:
the dot-product identity with the oracle's forward-mode tangents, with walls
and wraps on every axis, at 1e-10 of the sum of absolute products."""
import numpy as np
import pytest

import oracle
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


CASES = [
    ([64, 32, 64], "pvs", ["periodic", "periodic", "reflect"], [0.0, 0.0, -0.5]),   # 131072: split
    ([65, 32, 64], "pvs", ["reflect", "periodic", "periodic"], [0.3, 0.0, 0.0]),    # above: one thread per cell
    ([4, 4, 4], "dms", ["reflect", "reflect", "reflect"], [0.1, -0.2, -0.4]),
    ([5, 4, 7], "pms", ["periodic", "reflect", "periodic"], [0.0, -0.2, 0.0]),
    ([33, 5, 13], "dvs", ["periodic", "periodic", "periodic"], [0.0, 0.0, 0.0]),
    ([4, 130, 257], "pd", ["periodic", "reflect", "reflect"], [0.0, 0.1, -0.4]),    # above, narrow rows
]


@pytest.mark.parametrize("n,form,bc,g", CASES, ids=[f"{'x'.join(map(str, c[0]))}-{c[1]}" for c in CASES])
def test_dot_product(n, form, bc, g):
    cfg, U0 = W.random_state(3, n, seed_k=1500 + sum(n), xi=4.0, form=form, bc_lo=bc, g=g)
    dt = 0.5 * oracle.cfl_dt(cfg, U0)
    rng = np.random.default_rng(W.seed(91))
    lamN = rng.standard_normal(U0.shape)
    print(f"[adjoint3d] n={n} form={form} bc={bc}", flush=True)
    s = R.Solver(cfg, adjoint=True)
    U = torch.from_numpy(U0).cuda()
    lam = torch.from_numpy(lamN.copy()).cuda()
    dxi = torch.zeros(1, dtype=torch.float64, device="cuda")
    s.adjoint_step(U, lam, dt, dxi)
    torch.cuda.synchronize()
    lam0, dJdxi = lam.cpu().numpy(), float(dxi.item())
    s.close()
    K = 3
    d = rng.standard_normal((K, U0.size)) * 1e-2
    d[1] = 0.0
    c = np.array([0.0, 1.0, 0.7])
    _, T = oracle.run_tangent(cfg, U0, d, c, 1, dt)
    for k in range(K):
        lhs = float(np.dot(lamN.ravel(), T[k]))
        rhs = float(np.dot(lam0.ravel(), d[k])) + dJdxi * c[k]
        scale = float(np.abs(lamN.ravel() * T[k]).sum()) + 1e-300
        assert abs(lhs - rhs) <= 1e-10 * scale, (k, lhs, rhs)

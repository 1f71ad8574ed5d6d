"""Single 2D stages by whole-row workgroups and by strips, over the chunk
lengths the planner takes and forced ones: separate rsst_step calls on grids
whose rows take 1, 2, 4 and 8 waves, with even and odd heights, ragged last
chunks and chunks longer than the grid, in both storage types.  Every path gives
the same bits (the runs of steps in one launch are the reference where a grid
has them, else another chunk length), and the oracle bounds them."""
import numpy as np
import pytest

import oracle
import paper_1812_04135_amd as R
import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# (grid, walls in x, whole rows or strips); the last of each width lies beyond
# the 4096 wave-rows up to which whole rows are always taken
CASES = [([61, 40], True, 1), ([64, 4101], True, 0), ([63, 5002], True, 1),
         ([128, 33], False, 1), ([125, 1024], True, 1), ([122, 2203], False, 1),
         ([256, 97], False, 1), ([245, 512], True, 1), ([241, 3001], False, 1),
         ([512, 34], True, 1), ([490, 129], False, 1), ([384, 256], False, 1), ([190, 10923], False, 1),
         ([1000, 1030], False, 0), ([384, 257], True, 0), ([256, 1100], False, 0), ([512, 520], False, 0), ([70, 61], True, 0)]


def _case(n, walls, seed=0):
    return W.random_state(2, n, seed_k=2100 + sum(n) + seed, xi=4.0, bc_lo=["reflect" if walls else "periodic", "reflect"],
                          g=[0.0, -0.5])


def _run(cfg, U0, nsteps, how="step", **kw):
    U = torch.from_numpy(np.ascontiguousarray(U0)).cuda()
    s = R.Solver(cfg, **kw)
    if how == "step":
        for _ in range(nsteps):
            s.step(U)
    else:
        s.steps(U, nsteps)
    out = (U.cpu().numpy(), *s.time(), s.poll())
    s.close()
    return out


def _same(a, b):
    return np.array_equal(a[0], b[0]) and a[1:] == b[1:]


def _pert(U0, axis):
    bg = U0.mean(axis=2 if axis == 1 else (1, 2)).reshape(4, -1)
    P0 = (U0 - bg.reshape((4, -1, 1) if axis == 1 else (4, 1, 1))).astype(np.float32)
    return P0, dict(prec="fp32_pert", bg=torch.from_numpy(np.ascontiguousarray(bg)).cuda(), bg_axis=axis)


@pytest.mark.parametrize("n,walls,rows", CASES, ids=[f"{c[0][0]}x{c[0][1]}" for c in CASES])
def test_steps_agree_over_chunks_and_match_oracle(n, walls, rows, monkeypatch):
    cfg, U0 = _case(n, walls)
    p = R.rsst_plan(R.make_config(cfg))
    print(f"[rows2d] n={n} {p}", flush=True)
    assert p["rows"] == rows
    for U, kw in ((U0, {}), _pert(U0, 1), _pert(U0, -1)):
        ref = _run(cfg, U, 3, **kw)
        assert ref[3] == 0
        if p["step"]:
            assert _same(_run(cfg, U, 3, "steps", **kw), ref)
        for km in ("1", "2", "7", str(p["chunk"] + 1), "4096"):
            monkeypatch.setenv("RSST_KM", km)
            assert _same(_run(cfg, U, 3, **kw), ref), km
            if km != "4096":  # a pair of one-launch steps, where the grid has them, and a single one
                assert _same(_run(cfg, U, 3, "steps", **kw), ref), km
        monkeypatch.delenv("RSST_KM")
        if not kw and n[0] * n[1] <= 1 << 20:
            Uo, to, _ = oracle.run(cfg, U0, 3)
            a = float(np.sqrt(W.GAMMA * 2.0 / 0.4))  # bound of the sound speed of these states
            scale = [np.abs(Uo[0]).max(), np.abs(Uo[0]).max() * a, np.abs(Uo[0]).max() * a, np.abs(Uo[3]).max()]
            assert abs(ref[1] - to) <= 1e-13 * to
            for v in range(4):
                assert np.abs(ref[0][v] - Uo[v]).max() <= 1e-12 * scale[v], v

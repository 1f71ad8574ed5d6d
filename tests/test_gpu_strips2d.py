"""2D grids: the strips of a row (a whole periodic row of at most 64 cells, or
strips of at most 60 or 56 cells with halo lanes), the whole-row workgroups,
and both stages of a step in one launch.  Every path forms the same face
states with the same code, so all give the same bits: a run of steps
(rsst_steps: pairs of one-launch steps), separate rsst_step calls, kept
trajectories (rsst_steps_out) and forced chunk lengths; and the oracle bounds
each of them."""
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


PER, WALL = ["periodic", "periodic"], ["reflect", "reflect"]
# row lengths around the strip widths (56, 60, 64 and their multiples) and
# heights around the tiles (4 rows) and the smallest grid
CASES = [
    ([4, 4], PER, None, "pvs", {}), ([4, 5], WALL, None, "pms", {}), ([33, 7], PER, [0.3, -0.4], "dvs", {}),
    ([56, 9], WALL, [0.3, -0.4], "pvs", {}), ([57, 8], WALL, [0.3, -0.4], "dms", {}), ([60, 6], WALL, None, "pd", {}),
    ([61, 13], PER, None, "pvs", {}), ([61, 13], WALL, [0.2, 0.0], "pvs", {}), ([63, 4], PER, None, "euler", {}),
    ([64, 21], PER, [0.0, -0.5], "pms", {}), ([65, 12], PER, None, "pvs", {}), ([112, 16], PER, None, "dvs", {}),
    ([113, 17], ["periodic", "reflect"], [0.0, -0.5], "pvs", {}), ([121, 10], ["reflect", "periodic"], None, "pvs", {}),
    ([256, 30], PER, None, "pvs", {}), ([128, 66], ["periodic", "reflect"], [0.0, -0.5], "pvs", {"cmax": 0.5}),
    ([70, 45], ["periodic", "hydro"], [0.0, -0.5], "pms", {}), ([58, 20], ["reflect", "hydro"], [0.0, -0.5], "pvs", {}),
    ([67, 22], PER, None, "dms", {"gas": W.VDW}), ([1024, 7], PER, None, "pvs", {}), ([389, 41], WALL, None, "pvs", {}),
]


def _case(n, bc, g, form, opts):
    o = dict(opts)
    cfg, U0 = W.random_state(2, n, seed_k=1300 + sum(n), xi=1.0 if form == "euler" else 4.0, form=form, bc_lo=bc, g=g,
                             gas=o.pop("gas", None))
    cfg.update(o)
    return cfg, U0


def _run(cfg, U0, how, nsteps, dt=0.0, t_end=0.0, **kw):
    U = torch.from_numpy(np.ascontiguousarray(U0)).cuda()
    s = R.Solver(cfg, t_end=t_end, **kw)
    if how == "steps":
        s.steps(U, nsteps, dt)
    elif how == "step":
        for _ in range(nsteps):
            s.step(U, dt)
    else:  # a kept trajectory
        traj = [U] + [torch.empty_like(U) for _ in range(nsteps)]
        stage = [torch.empty_like(U) for _ in range(nsteps)]
        s.steps_out(traj, stage, dt)
        U = traj[-1]
    t, dt_next = s.time()
    flags = s.poll()
    out = U.cpu().numpy()
    s.close()
    return out, t, dt_next, flags


@pytest.mark.parametrize("n,bc,g,form,opts", CASES, ids=[f"{c[0][0]}x{c[0][1]}-{c[3]}-{c[1][0][0]}{c[1][1][0]}" for c in CASES])
def test_paths_agree_and_match_oracle(n, bc, g, form, opts):
    cfg, U0 = _case(n, bc, g, form, opts)
    print(f"[strips2d] n={n} bc={bc} form={form} {opts}", flush=True)
    ref = _run(cfg, U0, "step", 5)
    assert ref[3] == 0
    for how in ("steps", "out"):
        got = _run(cfg, U0, how, 5)
        assert np.array_equal(got[0], ref[0]) and got[1:] == ref[1:], how
    Uo, to, _ = oracle.run(cfg, U0, 5)
    assert abs(ref[1] - to) <= 1e-13 * to
    a = float(np.sqrt(W.GAMMA * 2.0 / 0.4))  # bound of the sound speed of these states
    scale = [np.abs(Uo[0]).max(), np.abs(Uo[0]).max() * a, np.abs(Uo[0]).max() * a, np.abs(Uo[3]).max()]
    for v in range(4):
        assert np.abs(ref[0][v] - Uo[v]).max() <= 1e-12 * scale[v], v


@pytest.mark.parametrize("r", ["1", "2", "3", "7", "15"])
def test_tile_heights_change_no_bit(r, monkeypatch):
    cfg, U0 = _case([150, 131], ["periodic", "reflect"], [0.0, -0.5], "pvs", {})
    ref = _run(cfg, U0, "step", 4)
    monkeypatch.setenv("RSST_KM", r)
    got = _run(cfg, U0, "steps", 4)
    assert np.array_equal(got[0], ref[0]) and got[1:] == ref[1:]


@pytest.mark.parametrize("axis", [-1, 0, 1])
@pytest.mark.parametrize("n", [[50, 19], [131, 24]])
def test_fp32_perturbation_paths_agree(n, axis):
    cfg, U0 = _case(n, PER, None, "pvs", {})
    m = {-1: (1, 2), 0: (1,), 1: (2,)}[axis]
    bg = U0.mean(axis=m).reshape(4, -1)
    sh = {-1: (4, 1, 1), 0: (4, 1, n[0]), 1: (4, n[1], 1)}[axis]
    P0 = (U0 - bg.reshape(sh)).astype(np.float32)
    kw = dict(prec="fp32_pert", bg=torch.from_numpy(np.ascontiguousarray(bg)).cuda(), bg_axis=axis)
    ref = _run(cfg, P0, "step", 4, **kw)
    for how in ("steps", "out"):
        got = _run(cfg, P0, how, 4, **kw)
        assert np.array_equal(got[0], ref[0]) and got[1:] == ref[1:], how


@pytest.mark.parametrize("nsteps", [1, 2, 3, 6])
def test_fixed_steps_and_end_time(nsteps):
    cfg, U0 = _case([90, 33], PER, None, "pvs", {})
    _, t1, dt1, _ = _run(cfg, U0, "step", 1)
    for kw in (dict(dt=0.4 * dt1), dict(t_end=t1 + 0.3 * dt1)):
        ref = _run(cfg, U0, "step", nsteps, **kw)
        for how in ("steps", "out"):
            got = _run(cfg, U0, how, nsteps, **kw)
            assert np.array_equal(got[0], ref[0]) and got[1:] == ref[1:], (how, kw)


def test_odd_captured_run_replays():
    """Three steps per replay: a pair of one-launch steps and a split one."""
    cfg, U0 = _case([80, 40], PER, None, "pvs", {})
    ref, _, _, _ = _run(cfg, U0, "step", 12)
    U = torch.from_numpy(U0).cuda()
    s = R.Solver(cfg)
    s.prime(U)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        s.steps(U, 3)
    for _ in range(4):
        g.replay()
        torch.cuda.synchronize()
    assert np.array_equal(U.cpu().numpy(), ref)
    s.close()


@pytest.mark.parametrize("sizes,prec", [([40, 61, 64, 100, 128, 200, 256, 33, 90, 150, 250, 70], "fp64"),
                                        ([256, 64, 31], "fp64"),  # too uneven for a queue per XCD
                                        ([64] * 24, "fp32_pert"), ([5, 9, 17, 64, 65] * 4, "fp32_pert")])
def test_batch_boxes_equal_single_runs(sizes, prec):
    rng = np.random.default_rng(W.seed(77))
    boxes = [W.strat2d_box(n, 10.0, 5.0, rng) for n in sizes]
    b = R.Batch([c for c, _, _ in boxes], prec=prec, bgs=[m["bg"] for _, _, m in boxes], max_steps=8)
    pert = [U - m["bg"][:, :, None] for _, U, m in boxes] if prec == "fp32_pert" else [U for _, U, _ in boxes]
    U = b.pack(pert)
    for _ in range(2):
        b.run(U, 6)
    assert b.poll() == 0
    t = b.times()
    got = b.unpack(U)
    b.close()
    for q in range(0, len(sizes), max(1, len(sizes) // 8)):
        cfg, _, m = boxes[q]
        kw = dict(prec=prec, bg=torch.from_numpy(m["bg"]).cuda(), bg_axis=1) if prec == "fp32_pert" else {}
        P0 = pert[q].astype(np.float32) if prec == "fp32_pert" else pert[q]
        ref, tr, _, _ = _run(cfg, P0, "step", 12, **kw)
        assert np.array_equal(got[q], ref) and t[q] == tr, (q, sizes[q])


def test_reused_workspace_starts_clean():
    """A solver made after another was closed may take its workspace: its
    results are those of a first solver, also from a larger or a smaller
    block, with an adjoint workspace or not, and with two alive at once."""
    cases = [_case(n, PER, None, "pvs", {}) for n in ([64, 40], [60, 40], [80, 41], [64, 40])]
    refs = []
    for cfg, U0 in cases:
        refs.append(_run(cfg, U0, "steps", 5))
    for rep in range(3):
        for (cfg, U0), ref in zip(cases, refs):
            other = R.Solver(cases[rep][0], adjoint=rep == 1)
            got = _run(cfg, U0, "steps", 5)
            other.close()
            assert np.array_equal(got[0], ref[0]) and got[1:] == ref[1:]

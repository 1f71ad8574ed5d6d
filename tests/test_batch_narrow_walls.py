"""Boxes whose rows of 61 to 64 cells lie between walls in x (one wave wide, two
strips): the row blocks a small batch and a large one make of them (host
only), and their results against single runs."""
import numpy as np
import pytest

import paper_1812_04135_amd as R
import workloads as W


def _cfg(nx, ny, xbc):
    return W.base_cfg(2, [nx, ny], xi=4.0, bc_lo=[xbc, "reflect"], g=[0.0, -0.5])


def _rows(boxes, strip=(16, 16, 16, 16)):
    """Rows per full block of the first box."""
    tab = R.rsst_batch_plan([_cfg(*b) for b in boxes], strip)
    first = tab[tab[:, 0] == 0]
    # blocks cover the box, and each waits for the blocks within two rows of its own
    assert first[0, 2] == 0 and first[-1, 3] == boxes[0][1] and np.all(first[1:, 2] == first[:-1, 3])
    for p, r in enumerate(first):
        near = [q for q, s in enumerate(first) if s[2] - 2 < r[3] and r[2] < s[3] + 2]
        assert list(r[5:5 + r[4]]) == near, p
    return int(first[0, 3] - first[0, 2])


@pytest.mark.parametrize("nx", [61, 62, 64])
def test_blocks_are_halved_in_small_batches(nx):
    assert _rows([(nx, 200, "reflect")]) == 32
    assert _rows([(nx, 200, "periodic")]) == 64
    assert _rows([(60, 200, "reflect")]) == 64
    assert _rows([(65, 200, "reflect")]) == 32  # two waves
    # 4 blocks of 64 rows each: 1020 and 1024
    assert _rows([(nx, 200, "reflect")] * 255) == 32
    assert _rows([(nx, 200, "reflect")] * 256) == 64
    assert _rows([(nx, 9, "reflect")], (8, 8, 8, 8)) == 9
    assert _rows([(nx, 256, "reflect")], (8, 8, 8, 8)) == 16
    assert _rows([(nx, 256, "reflect")] * 128, (8, 8, 8, 8)) == 32


@pytest.mark.gpu
@pytest.mark.parametrize("nbox", [1, 5, 260])
@pytest.mark.parametrize("prec", ["fp64", "fp32_pert"])
def test_equal_single_runs(nbox, prec):
    torch = pytest.importorskip("torch")
    shapes = [(64, 200), (61, 33), (62, 130), (63, 8), (64, 64)]
    rng = np.random.default_rng(W.seed(2300))
    cfgs, states, bgs = [], [], []
    for b in range(nbox):
        cfg, U = W.random_state(2, list(shapes[b % 5] if nbox < 260 else (61 + b % 4, 200)), seed_k=2300 + b % 7,
                                xi=4.0, bc_lo=["reflect", "reflect"], g=[0.0, -0.5])
        cfgs.append(cfg)
        bgs.append(U.mean(axis=2) * (1.0 + 0.01 * rng.random()))
        states.append(U if prec == "fp64" else (U - bgs[-1][:, :, None]).astype(np.float32))
    print(f"[narrow walls] {nbox} boxes {prec}", flush=True)
    b = R.Batch(cfgs, prec=prec, bgs=bgs if prec == "fp32_pert" else None, max_steps=8)
    U = b.pack(states)
    for _ in range(2):
        b.run(U, 3)
    assert b.poll() == 0
    got, t = b.unpack(U), b.times()
    b.close()
    for q in range(0, nbox, max(1, nbox // 12)):
        V = torch.from_numpy(np.ascontiguousarray(states[q])).cuda()
        kw = dict(prec=prec, bg=torch.from_numpy(bgs[q]).cuda(), bg_axis=1) if prec == "fp32_pert" else {}
        s = R.Solver(cfgs[q], **kw)
        s.steps(V, 6)
        assert np.array_equal(got[q], V.cpu().numpy()) and t[q] == s.time()[0], q
        s.close()

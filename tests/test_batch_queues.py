"""The two ways a batch hands out its items: one queue per XCD (waits between
CUs that share an L2, no write-backs) and one queue for the chip.  Which one a
list of boxes takes (host only), and on both, with wide boxes of several strips
and several row blocks, walls and periodic y, each box bitwise its own run by
rsst_step, over two runs, also after every wait was given up."""
import numpy as np
import pytest

import paper_1812_04135_amd as R
import workloads as W


def _cfg(nx, ny, ybc="reflect"):
    return W.base_cfg(2, [nx, ny], xi=4.0, bc_lo=["periodic", ybc], g=[0.0, -0.5 if ybc == "reflect" else 0.0])


@pytest.mark.parametrize("sizes,queues", [
    ([256], 1), ([64] * 6, 1), ([64] * 7, 8), ([64] * 8, 8), ([64] * 9, 1), ([64] * 12, 1), ([64] * 13, 8), ([64] * 16, 8), ([64] * 17, 1),
    ([64] * 20, 8), ([64] * 25, 1), ([64] * 26, 8), ([256, 64, 31], 1), ([256] + [40] * 40, 1), ([256] * 8 + [40] * 3, 8),
    ([40, 61, 64, 100, 128, 200, 256, 33, 90, 150, 250, 70], 1)])
def test_even_lists_take_a_queue_per_xcd(sizes, queues):
    """Largest queue at most 1.25 of the mean, boxes dealt largest first."""
    assert R.rsst_batch_queues([_cfg(n, n) for n in sizes]) == queues


def test_queues_refuse_what_the_batch_refuses():
    with pytest.raises(R.RsstError) as e:
        R.rsst_batch_queues([dict(_cfg(16, 12), eos="vdw", eos_a=0.2, eos_b=0.1)])
    assert e.value.code == -4


SIZES = [(40, 90), (130, 70), (200, 66), (256, 100), (64, 140)]
# (how often each size comes, queues)
LISTS = [(16, 8), (8, 8), (1, 1)]


def _batch(times, prec):
    cfgs, states, bgs = [], [], []
    for q in range(times):
        for s, (nx, ny) in enumerate(SIZES):
            ybc = "periodic" if (q + s) % 2 else "reflect"
            cfg, U = W.random_state(2, [nx, ny], seed_k=2500 + s + 5 * (q % 3), xi=2.0 + s, bc_lo=["periodic", ybc],
                                    g=[0.0, -0.5 if ybc == "reflect" else 0.0])
            bg = U.mean(axis=2)
            cfgs.append(cfg)
            bgs.append(bg)
            states.append(U if prec == "fp64" else (U - bg[:, :, None]).astype(np.float32))
    return cfgs, states, bgs


def _singles(torch, cfgs, states, bgs, prec, nsteps):
    """Each distinct box by separate steps."""
    out = {}
    for cfg, P, bg in zip(cfgs, states, bgs):
        key = (P.tobytes(), cfg["n"][1], cfg["xi"], cfg["bc_lo"][1])
        if key not in out:
            U = torch.from_numpy(np.ascontiguousarray(P)).cuda()
            kw = dict(prec=prec, bg=torch.from_numpy(bg).cuda(), bg_axis=1) if prec == "fp32_pert" else {}
            s = R.Solver(cfg, **kw)
            for _ in range(nsteps):
                s.step(U)
            out[key] = (U.cpu().numpy(), s.time()[0])
            s.close()
        yield out[key]


@pytest.mark.gpu
@pytest.mark.parametrize("prec", ["fp64", "fp32_pert"])
@pytest.mark.parametrize("times,queues", LISTS)
def test_every_box_equals_its_own_run(times, queues, prec):
    torch = pytest.importorskip("torch")
    cfgs, states, bgs = _batch(times, prec)
    assert R.rsst_batch_queues(cfgs) == queues
    print(f"[queues] {len(cfgs)} boxes {prec} {queues} queues", flush=True)
    b = R.Batch(cfgs, prec=prec, bgs=bgs if prec == "fp32_pert" else None, max_steps=8)
    for strip in (16, 8):
        b.set_tiles([strip] * 4)
        U = b.pack(states)
        b.set_times(np.zeros(len(cfgs)))
        for _ in range(2):
            b.run(U, 4)
        assert b.poll() == 0
        got, t = b.unpack(U), b.times()
        for q, (ref, tr) in enumerate(_singles(torch, cfgs, states, bgs, prec, 8)):
            assert np.array_equal(got[q], ref) and t[q] == tr, (strip, q, cfgs[q]["n"])
    b.close()


@pytest.mark.gpu
@pytest.mark.parametrize("prec", ["fp64", "fp32_pert"])
def test_given_up_waits_drain_a_queue_per_xcd(prec):
    """A wait limit of 0: every wait that is not satisfied at once is given up
    (nothing stored, but signalled), the kernel ends, the run is flagged; with
    the limit restored the next run is exact."""
    torch = pytest.importorskip("torch")
    cfgs, states, bgs = _batch(8, prec)
    assert R.rsst_batch_queues(cfgs) == 8
    b = R.Batch(cfgs, prec=prec, bgs=bgs if prec == "fp32_pert" else None, max_steps=8)
    b.set_tiles([8] * 4)
    U = b.pack(states)
    b.set_wait_limit(0.0)
    b.run(U, 6)
    torch.cuda.synchronize()
    with pytest.raises(R.RsstError) as e:
        b.poll()
    assert e.value.code == R.RSST_E_DEVICE and (e.value.flags & 8), (e.value.code, e.value.flags)
    assert b.poll() == 0  # cleared
    b.set_wait_limit(10.0)
    U = b.pack(states)
    b.set_times(np.zeros(len(cfgs)))
    b.run(U, 6)
    assert b.poll() == 0
    got, t = b.unpack(U), b.times()
    for q, (ref, tr) in enumerate(_singles(torch, cfgs, states, bgs, prec, 6)):
        assert np.array_equal(got[q], ref) and t[q] == tr, q
    b.close()

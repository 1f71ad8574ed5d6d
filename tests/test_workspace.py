"""Where a solver's workspace lies and what becomes of it: the library's own is
freed with the solver, a caller's stays the caller's, and the rollout's is
torch's."""
import ctypes
import time

import pytest

import paper_1812_04135_amd as R
import workloads as W

torch = pytest.importorskip("torch")


def _cfg(n, **kw):
    return R.make_config(W.base_cfg(len(n), n, xi=3.0), **kw)


def test_size_and_arguments_on_host():
    """rsst_workspace_bytes and the checks of rsst_init_in, before any device
    call (the work pointers are never touched)."""
    L = R.lib()
    n = ctypes.c_size_t()
    h = ctypes.c_void_p()
    for shape, adjoint in (([64], False), ([64, 64], False), ([64, 64], True), ([24, 20, 16], True), ([512, 512, 512], False)):
        c = _cfg(shape, adjoint=adjoint)
        assert L.rsst_workspace_bytes(ctypes.byref(c), ctypes.byref(n)) == 0
        state = 8 * (len(shape) + 2)
        for v in shape:
            state *= v
        assert n.value % 256 == 0 and n.value >= state * (2 if adjoint else 1), shape

        def init_in(work, size):
            return L.rsst_init_in(ctypes.byref(c), ctypes.c_void_p(work), ctypes.c_size_t(size), None, ctypes.byref(h))

        assert init_in(0x10000, n.value - 1) == -1
        assert init_in(0x10000 + 128, n.value) == -1
        assert init_in(0, n.value) == -1
        assert not h.value
    bad = _cfg([64])
    bad.gamma = 1.0
    assert L.rsst_workspace_bytes(ctypes.byref(bad), ctypes.byref(n)) == -1
    assert L.rsst_workspace_bytes(ctypes.byref(_cfg([1025])), ctypes.byref(n)) == -4
    assert L.rsst_workspace_bytes(None, ctypes.byref(n)) == -1
    assert L.rsst_workspace_bytes(ctypes.byref(_cfg([64])), None) == -1
    assert L.rsst_init_in(ctypes.byref(_cfg([64])), ctypes.c_void_p(0x10000), ctypes.c_size_t(1 << 30), None, None) == -1
    assert R.rsst_workspace_bytes(_cfg([64, 64])) >= 8 * 4 * 64 * 64


def _outside():
    """Device memory in use but for what torch has reserved, whose cache grows and
    shrinks with the tensors of other tests."""
    torch.cuda.synchronize()
    free, total = torch.cuda.mem_get_info()
    return total - free - torch.cuda.memory_reserved()


def _held(most=0):
    """Bytes of live tensors, once they are at most `most` or five seconds have
    passed: autograd's worker thread drops its references to a gradient a moment
    after the caller has it, for which it has to wait for the interpreter lock."""
    end = time.monotonic() + 5.0
    while torch.cuda.memory_allocated() > most and time.monotonic() < end:
        time.sleep(0.01)
    return torch.cuda.memory_allocated()


@pytest.mark.gpu
def test_closing_a_solver_returns_its_memory():
    R.Solver(W.base_cfg(2, [64, 64], xi=3.0)).close()  # the library and its kernels are loaded
    before = _outside()
    s = R.Solver(W.base_cfg(2, [1024, 1000], xi=3.0))  # 33 MB
    assert _outside() >= before + 32_000_000
    s.close()
    assert _outside() <= before + 4_000_000


@pytest.mark.gpu
@pytest.mark.parametrize("n,adjoint", [([70], False), ([70, 33], True), ([20, 9, 8], True)])
def test_solver_in_a_used_block_equals_its_own(n, adjoint):
    """A caller's block holds what its last user left there."""
    cfg, U0 = W.random_state(len(n), n, seed_k=1900 + sum(n), xi=4.0)
    out = []
    for limit in (0, 1 << 30):
        if limit:
            dirt = torch.full((R.rsst_workspace_bytes(R.make_config(cfg, adjoint=adjoint)),), 255, dtype=torch.uint8,
                              device="cuda")
            del dirt
        U = torch.from_numpy(U0).cuda()
        s = R.Solver(cfg, adjoint=adjoint, torch_workspace=limit)
        assert (s._work is not None) == bool(limit)
        s.steps(U, 5)
        res = [U, torch.tensor(s.time()), torch.from_numpy(s.diag(U))]
        if adjoint:
            lam = torch.ones_like(U)
            dxi = torch.zeros(1, dtype=torch.float64, device="cuda")
            s.adjoint_run([U, U], None, lam, 1e-4, dxi)
            res += [lam, dxi]
        assert s.poll() == 0
        s.close()
        out.append(res)
    assert all(torch.equal(a, b) for a, b in zip(*out))


@pytest.mark.gpu
@pytest.mark.parametrize("every,graph", [(1, True), (3, False), (3, True)])
def test_rollout_keeps_nothing_from_torch(every, graph):
    from paper_1812_04135_amd.rollout import rollout

    cfg, U0 = W.random_state(2, [256, 200], seed_k=1950, xi=4.0)

    def gradient():
        U = torch.from_numpy(U0).cuda().requires_grad_(True)
        xi = torch.tensor(4.0, dtype=torch.float64, device="cuda", requires_grad=True)
        out = rollout(U, xi, cfg, 12, 1e-4, every, graph)
        return torch.autograd.grad(out, (U, xi), torch.ones_like(out))

    first = [g.cpu() for g in gradient()]
    held, before = _held(), _outside()
    for _ in range(3):
        assert all(torch.equal(a, b.cpu()) for a, b in zip(first, gradient()))
    assert _held(held) <= held
    assert _outside() <= before + 4_000_000

"""Batched Rayleigh-Ritz where its side streams are shared or stay idle, bit by bit against one
call per problem: two threads on one context (one of them finds the side streams taken), kernel
timing on, a workspace that does not hold the dense parts of all problems, and a context that
autotunes (the first batch times its products one by one, the second uses those choices)."""
import threading

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1603_04339_amd import sparc as sp
from paper_1603_04339_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = sp.Context(0)
    yield c
    c.close()


def _problem(ctx, i, n, ns, dt):
    cplx = dt in (sp.C128, sp.C64)
    cell, rng = wl.draw_cell(93, i, n, tuple(0.5 * v for v in n), 2, (0,), 2.0, ns)
    ham = sp.Hamiltonian(ctx, cell, dt, kpt=(0.1, 0.2, -0.1) if cplx else (0.0, 0.0, 0.0))
    X = rng.standard_normal((cell.n_d, ns)) + (1j * rng.standard_normal((cell.n_d, ns)) if cplx else 0.0)
    X = np.linalg.qr(X)[0]
    return ham, torch.from_numpy(np.ascontiguousarray(X.T)).to(sp.TORCH_DTYPE[dt]).cuda()


def _single(hams, Xs):
    out = []
    for h, X in zip(hams, Xs):
        Y, r = X.clone(), torch.zeros(X.shape[0], dtype=torch.float64, device="cuda")
        sp.rayleigh_ritz(h, Y, r, sp.workspace(h, X.shape[0], sp.OP_RR))
        out.append((Y, r))
    return out


def _batched(ctx, hams, Xs):
    Ys = [X.clone() for X in Xs]
    rs = [torch.zeros(X.shape[0], dtype=torch.float64, device="cuda") for X in Xs]
    sp.rayleigh_ritz_batched(ctx, hams, Ys, rs, sp.GEMM_NATIVE, work=sp.rr_batched_workspace(ctx, hams, Xs))
    torch.cuda.synchronize()
    return list(zip(Ys, rs))


def _same(a, b):
    return all(torch.equal(x, y) for p, q in zip(a, b) for x, y in zip(p, q))


def _set(ctx, first):
    return list(zip(*[_problem(ctx, first + i, n, ns, dt) for i, (n, ns, dt) in enumerate(
        [((24, 22, 26), 40, sp.R64), ((20, 24, 24), 30, sp.C128), ((24, 24, 24), 64, sp.R64), ((26, 20, 24), 17, sp.R32)])]))


def test_two_threads_on_one_context(ctx):
    sets = [_set(ctx, 0), _set(ctx, 10)]
    want = [_single(*s) for s in sets]
    torch.cuda.synchronize()
    got, start = [[], []], threading.Barrier(2)

    def work(i):
        start.wait()
        for _ in range(4):
            got[i].append(_batched(ctx, *sets[i]))

    threads = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for i in range(2):
        assert len(got[i]) == 4 and all(_same(want[i], g) for g in got[i])


def test_timing_on(ctx):
    hams, Xs = _set(ctx, 20)
    want = _single(hams, Xs)
    ctx.set_timing(True)
    assert _same(want, _batched(ctx, hams, Xs))
    assert ctx.kernel_time("gram")[1] >= 2 * len(hams)
    ctx.set_timing(False)


def test_dense_parts_past_the_workspace(ctx):
    hams, Xs = zip(*[_problem(ctx, 30 + i, (12, 10, 8), 480, sp.R64) for i in range(4)])
    assert _same(_single(hams, Xs), _batched(ctx, hams, Xs))


def test_autotune(ctx):
    hams, Xs = _set(ctx, 40)
    sp.set_autotune(ctx, True)
    try:
        first = _batched(ctx, hams, Xs)
        want = _single(hams, Xs)
        assert _same(want, first) and _same(want, _batched(ctx, hams, Xs))
    finally:
        sp.set_autotune(ctx, False)

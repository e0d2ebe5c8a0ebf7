"""Batched Rayleigh-Ritz with the problems' dense parts on side streams against one call per
problem.  The kernels and their operands are the same in both, so the results are compared bit
by bit, over: all four types in one batch, sizes from 1 state to several tiles, leading
dimensions above N_d, blocks that need two passes first, last and in between (they go one by
one), two problems on overlapping blocks and a split-product mode (one by one throughout), a
context on a stream of its own, and a second batch on the same streams."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1603_04339_amd import sparc as sp
from paper_1603_04339_amd import workloads as wl

pytestmark = pytest.mark.gpu

CODES = {"r64": sp.R64, "r32": sp.R32, "c128": sp.C128, "c64": sp.C64}


@pytest.fixture(params=["default", "own"])
def ctx(request):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    stream = None if request.param == "default" else torch.cuda.Stream()
    with torch.cuda.stream(stream):
        c = sp.Context(0)
        yield c
        torch.cuda.synchronize()
        c.close()


def _problem(ctx, i, n, ns, dt, hard, pad=0):
    cplx = dt.startswith("c")
    cell, rng = wl.draw_cell(97, i, n, tuple(0.5 * v for v in n), 3, (0, 1), 2.0, ns)
    ham = sp.Hamiltonian(ctx, cell, CODES[dt], kpt=(0.1, 0.2, -0.1) if cplx else (0.0, 0.0, 0.0))
    X = rng.standard_normal((cell.n_d, ns)) + (1j * rng.standard_normal((cell.n_d, ns)) if cplx else 0.0)
    X = np.linalg.qr(X)[0]
    if hard and ns > 1:      # condition number of the Gram matrix ~ 1e4
        X[:, 1:] = X[:, :1] + 0.02 * X[:, 1:]
    t = torch.zeros(ns, cell.n_d + pad, dtype=sp.TORCH_DTYPE[CODES[dt]], device="cuda")
    t[:, :cell.n_d] = torch.from_numpy(np.ascontiguousarray(X.T)).to(t.dtype)
    return ham, t


def _check(ctx, hams, Xs, mode=sp.GEMM_NATIVE):
    alone = [X.clone() for X in Xs]
    want = [torch.zeros(X.shape[0], dtype=torch.float64, device="cuda") for X in Xs]
    got = [torch.zeros_like(r) for r in want]
    for h, X, r in zip(hams, alone, want):
        sp.rayleigh_ritz(h, X, r, sp.workspace(h, X.shape[0], sp.OP_RR), mode)
    sp.rayleigh_ritz_batched(ctx, hams, Xs, got, mode, work=sp.rr_batched_workspace(ctx, hams, Xs))
    torch.cuda.synchronize()
    for a, b, X, Y in zip(want, got, alone, Xs):
        assert torch.equal(a, b)
        assert torch.equal(X, Y)


G = [(18, 17, 16), (16, 16, 16), (20, 16, 24), (24, 24, 24)]


@pytest.mark.parametrize("hard", [(), (0,), (2, 3), (5,), (0, 1, 2, 3, 4, 5)])
def test_batch_equals_single_calls(ctx, hard):
    spec = [(64, "r64", 0), (30, "c128", 3), (70, "r32", 0), (1, "r64", 1), (96, "c64", 0), (130, "r64", 0)]
    probs = [_problem(ctx, i, G[i % 4], ns, dt, i in hard, pad) for i, (ns, dt, pad) in enumerate(spec)]
    for _ in range(2):      # the second batch: rotated blocks, one pass each
        _check(ctx, [p[0] for p in probs], [p[1] for p in probs])


@pytest.mark.parametrize("count", [1, 2, 9])
def test_batch_sizes(ctx, count):
    probs = [_problem(ctx, i, G[i % 4], 20 + 11 * i, "c128" if i % 2 else "r64", False) for i in range(count)]
    _check(ctx, [p[0] for p in probs], [p[1] for p in probs])


def test_split_products(ctx):
    probs = [_problem(ctx, i, G[i], 32, "r32", False) for i in range(3)]
    _check(ctx, [p[0] for p in probs], [p[1] for p in probs], sp.GEMM_BF16X3)


def test_overlapping_blocks(ctx):
    """The same block twice: rotated by the first problem, then again by the second."""
    ham, X = _problem(ctx, 0, G[0], 40, "r64", False)
    Y = X.clone()
    want = [torch.zeros(40, dtype=torch.float64, device="cuda") for _ in range(2)]
    got = [torch.zeros_like(r) for r in want]
    work = sp.workspace(ham, 40, sp.OP_RR)
    for r in want:
        sp.rayleigh_ritz(ham, Y, r, work)
    sp.rayleigh_ritz_batched(ctx, [ham, ham], [X, X], got, work=work)
    torch.cuda.synchronize()
    assert torch.equal(X, Y) and all(torch.equal(a, b) for a, b in zip(want, got))

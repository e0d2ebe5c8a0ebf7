"""The one-launch conjugate-gradient iteration against the same iteration in two launches: nodes
are dealt to blocks alike and every sum is taken in one order, so residual, search direction, A r,
A p, solution and step scalars are compared bit by bit over several iterations, from the first on,
at the edges of the form: blocks that divide the grid or not, blocks that end inside a row, more
blocks than work-groups, directions shorter than the stencil's reach, the longest row it takes.
And the potential of a cell with rows past that, which takes two launches, through the SCF: its
residual may exceed the tolerance of the first solve (1e-4) by rounding only: the recurrence's
residual drifts from the true one by about eps times the operator's condition number (2e6) an
iteration, so by less than 1e-6 in a few thousand."""
import ctypes as C

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle.fd import Grid
from oracle.scf import laplacian_symbol
from paper_1603_04339_amd import sparc as sp
from paper_1603_04339_amd import workloads as wl

pytestmark = pytest.mark.gpu

BLOCKS = 1024


class CgIter(C.Structure):
    _fields_ = ([(k, C.c_void_p) for k in ("r", "w", "s", "p", "x", "sc", "part")] +
                [("nparts", C.c_int), ("it", C.c_int)] + [(k, C.c_void_p) for k in ("rn", "wn", "sn", "partn")])


def _fn(name, *args):
    f = getattr(sp.load(), name)
    f.restype, f.argtypes = C.c_int, list(args)
    return f


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = sp.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("n,n_o", [((16, 16, 16), 6), ((17, 25, 21), 6), ((13, 14, 15), 6), ((40, 40, 40), 6),
                                   ((9, 10, 7), 2), ((5, 33, 6), 1), ((18, 17, 19), 8), ((300, 9, 8), 4),
                                   ((2048, 9, 8), 4), ((66, 68, 70), 6), ((80, 80, 80), 5)])
@pytest.mark.parametrize("shift", [0.0, 0.7])
def test_one_launch_equals_two(ctx, n, n_o, shift):
    apply_ = _fn("_ZN5sparc8cg_applyEP9sparc_hamddRKNS_6CgIterE", C.c_void_p, C.c_double, C.c_double, C.c_void_p)
    forms = [_fn(f"_ZN5sparc{len(s)}{s}EP9sparc_hamddRNS_6CgIterE", C.c_void_p, C.c_double, C.c_double, C.c_void_p)
             for s in ("cg_iterate", "cg_iterate_two")]
    blocks = _fn("_ZN5sparc9cg_blocksEPK9sparc_ham", C.c_void_p)
    cell, rng = wl.draw_cell(96, sum(n), n, tuple(0.5 * v for v in n), 1, (0,), 1.2, 1)
    ham = sp.Hamiltonian(ctx, cell, sp.R64, n_o=n_o)
    r0 = torch.from_numpy(rng.standard_normal(cell.n_d)).cuda()
    r0 -= r0.mean()
    got = []
    for form in forms:
        buf = {k: torch.zeros(cell.n_d, dtype=torch.float64, device="cuda") for k in ("r", "w", "s", "p", "x", "rn", "wn", "sn")}
        buf.update({k: torch.zeros(2 * BLOCKS, dtype=torch.float64, device="cuda") for k in ("part", "partn")})
        buf["sc"] = torch.zeros(12, dtype=torch.float64, device="cuda")
        buf["r"].copy_(r0)
        it = CgIter(nparts=blocks(ham.handle), it=0, **{k: v.data_ptr() for k, v in buf.items()})
        where = {v.data_ptr(): v for v in buf.values()}
        assert apply_(ham.handle, 2.0, shift, C.byref(it)) == sp.OK
        steps = []
        for _ in range(5):
            assert form(ham.handle, 2.0, shift, C.byref(it)) == sp.OK
            torch.cuda.synchronize()
            steps.append([where[getattr(it, k)].clone() for k in ("r", "w", "s", "p", "x")] +
                         [buf["sc"][:3].clone(), buf["sc"][4:7].clone(),
                          where[it.part].view(2, BLOCKS)[:, :it.nparts].clone()])
        got.append(steps)
    for a, b in zip(*got):
        for u, v in zip(a, b):
            assert torch.equal(u, v)
    assert all(bool(torch.isfinite(t).all()) for t in got[0][-1])


def test_long_rows(ctx):
    n, n_o, ns = (2304, 9, 8), 4, 4
    cell, rng = wl.draw_cell(98, 1, n, tuple(0.5 * v for v in n), 2, (0,), 1.5, ns)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    zeros = lambda m: torch.zeros(m, dtype=torch.float64, device="cuda")  # noqa: E731
    prm = dict(n_s=ns, degree=4, n_first_passes=1, max_iter=2, lanczos_steps=8, mix_history=2, kT=0.01, mix=0.2,
               tol=1e6, n_elec=cell.n_elec, poisson_tol=1e-10, filt=sp.R64, rr=sp.GEMM_NATIVE, final_fp64_pass=0,
               x0_dev=dev(rng.standard_normal((ns, cell.n_d))), lanczos_v0_dev=dev(rng.standard_normal(cell.n_d)))
    rho, phi = zeros(cell.n_d), zeros(cell.n_d)
    out = sp.sparc_scf_run(ctx, cell, prm, rho, zeros(ns), phi_out=phi, n_o=n_o)
    assert out["converged"] and out["iterations"] <= 1
    sig = laplacian_symbol(Grid(n=n, L=cell.L, n_o=n_o))
    as3 = lambda t: t.cpu().numpy().reshape(n[2], n[1], n[0])  # noqa: E731
    rhs = 4.0 * np.pi * (as3(rho) - as3(rho).mean())
    res = rhs - np.fft.ifftn(sig * np.fft.fftn(as3(phi))).real
    assert np.linalg.norm(res) <= 1.01e-4 * np.linalg.norm(rhs)

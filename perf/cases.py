"""Performance cases of the framework: what a user's program has it do, over the sizes,
element types and directions that the configurations, tests and the benchmark use.

A case is a dict of plain values.  listed() gives the fixed ones, draw(rng) another of
the same ranges, prepare() what a program holds before the call, run() one pass through
the public entry points, work() the bytes and operations a pass cannot do without, and
exact() the same outputs from plain torch in 64 bits.

Kinds:
  apply    Y = H X of a block of orbitals (each residual, each Lanczos step).
  filter   the Chebyshev filter on a copy of a kept start block (the next k-point or the
           next geometry starts from the same block).
  pass     one CheFSI pass of one cell: filter, Rayleigh-Ritz, Fermi level, density; the
           next pass's cut is the largest Ritz value.  Orbitals are defined up to sign
           and rotation of degenerate levels, so a pass returns the Ritz values, the
           occupations and the density they give.
  kpoints  the same pass for all k-points of a complex Bloch cell in one filter plan.
  cells    the same pass for a batch of independent uneven cells in one filter plan.
  forces   local and non-local atomic forces of a converged state.
  scf      a whole self-consistent run from the atomic superposition, a fixed number of
           iterations.
  net      the density network: forward (the SCF start), or a training step.
"""
import math
import os

import numpy as np
import torch

from paper_1603_04339_amd import sparc as sp
from paper_1603_04339_amd import workloads as wl

DT = {"r64": (sp.R64, torch.float64), "r32": (sp.R32, torch.float32),
      "c128": (sp.C128, torch.complex128), "c64": (sp.C64, torch.complex64)}
N_O = 6           # 12th-order stencil
KT = 0.01         # Ha
NET_CH, NET_DIL = (2, 16, 32, 32, 1), (1, 2, 4, 8)


def listed():
    return [
        # one application on the smallest cell: launch latency
        dict(name="apply_24_r64", kind="apply", n1=24, n2=24, n3=24, h=0.5, atoms=8, p=False, n_s=32, dtype="r64"),
        # a ragged complex cell in single precision with a ragged number of states
        dict(name="filter_odd_c64", kind="filter", n1=45, n2=38, n3=51, h=0.5, atoms=11, p=True, n_s=37, degree=18,
             dtype="c64"),
        # the filter of the largest cell, in both precisions of the Gamma-point path
        dict(name="filter_96_r64", kind="filter", n1=96, n2=96, n3=96, h=0.4, atoms=64, p=True, n_s=512, degree=24,
             dtype="r64"),
        dict(name="filter_96_r32", kind="filter", n1=96, n2=96, n3=96, h=0.4, atoms=64, p=True, n_s=512, degree=24,
             dtype="r32"),
        # one pass of an SCF cell, and of the largest cell
        dict(name="pass_40_r64", kind="pass", n1=40, n2=40, n3=40, h=0.5, atoms=31, p=False, n_s=56, degree=20,
             dtype="r64"),
        dict(name="pass_96_r64", kind="pass", n1=96, n2=96, n3=96, h=0.4, atoms=64, p=True, n_s=512, degree=24,
             dtype="r64"),
        # eight Monkhorst-Pack points of a Bloch cell
        dict(name="kpoints_48_c128", kind="kpoints", n1=48, n2=48, n3=48, h=0.5, atoms=16, p=False, n_s=128,
             degree=20, n_k=8, dtype="c128"),
        # independent cells of uneven sizes (grid:atoms:states:degree)
        dict(name="cells_r64", kind="cells", h=0.5, dtype="r64",
             cells="64:32:128:20,32:8:32:16,80:48:256:24,48:16:64:18,32:8:32:16,48:16:64:18,64:32:128:20,48:16:64:18"),
        # forces after convergence: every geometry step has one
        dict(name="forces_64_r64", kind="forces", n1=64, n2=64, n3=64, h=0.5, atoms=32, p=True, n_s=128, dtype="r64"),
        # a whole SCF call
        dict(name="scf_40", kind="scf", n1=40, n2=40, n3=40, h=0.5, atoms=31, p=False, n_s=56, degree=20, iters=10,
             dtype="r64"),
        # training step of the density network (mini-batch of eight), and its use as SCF start
        dict(name="net_train_40", kind="net", n1=40, n2=40, n3=40, h=0.5, atoms=20, batch=8, train=True),
        dict(name="net_forward_40", kind="net", n1=40, n2=40, n3=40, h=0.5, atoms=20, batch=1, train=False),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["apply", "filter", "filter", "pass", "pass", "kpoints", "cells", "forces", "net"])
    if kind == "net":
        n = [rng.randint(17, 40) for _ in range(3)]
        return dict(kind="net", n1=n[0], n2=n[1], n3=n[2], h=0.5, atoms=rng.randint(4, 32), batch=rng.randint(1, 8),
                    train=rng.random() < 0.5)
    if kind == "cells":
        cells = []
        for _ in range(rng.randint(2, 8)):
            n = rng.randint(30, 72)
            cells.append("%d:%d:%d:%d" % (n, rng.randint(6, 32), 24 + _log_int(rng, 8, 128), rng.randint(16, 24)))
        return dict(kind="cells", h=0.5, dtype="r64", cells=",".join(cells))
    top = {"apply": 96, "filter": 96, "pass": 80, "kpoints": 48, "forces": 72}[kind]
    m = _log_int(rng, 24, top)
    n = [max(20, min(top, m + rng.randint(-6, 6))) for _ in range(3)]
    c = dict(kind=kind, n1=n[0], n2=n[1], n3=n[2], h=rng.choice([0.4, 0.5]), p=rng.random() < 0.5)
    vol = n[0] * n[1] * n[2] * c["h"] ** 3
    c["atoms"] = max(4, min(64, int(round(vol / rng.uniform(250.0, 900.0)))))
    c["n_s"] = _log_int(rng, 24, 320) if kind in ("apply", "filter") else c["atoms"] + 8 + _log_int(rng, 16, 160)
    if kind == "kpoints":
        c["n_s"] = min(c["n_s"], 128)
        c["n_k"] = rng.choice([2, 4, 8])
    if kind in ("filter", "pass", "kpoints"):
        c["degree"] = rng.randint(16, 24)
    c["dtype"] = {"apply": rng.choice(list(DT)), "filter": rng.choice(list(DT)), "pass": "r64", "kpoints": "c128",
                  "forces": rng.choice(["r64", "c128"])}[kind]
    return c


# ------------------------------------------------------------------------------- inputs
def _cell(case, seed):
    n = (case["n1"], case["n2"], case["n3"])
    rng = np.random.default_rng([17, seed])
    cell, _ = wl.draw_cell(0, 0, n, tuple(case["h"] * v for v in n), case["atoms"],
                           (0, 1) if case.get("p") else (0,), 3.5 if case.get("p") else 3.0, case.get("n_s", 0),
                           case.get("degree", 20), 1, rng=rng)
    return cell


def _kpt(case, cell):
    return tuple(2 * math.pi / cell.L[s] * f for s, f in enumerate((0.25, -0.25, 0.25))) \
        if case["dtype"].startswith("c") else (0.0, 0.0, 0.0)


def _block(seed, which, n_s, n_d, dtype):
    g = torch.Generator(device="cuda").manual_seed(1000003 * seed + which)
    return torch.randn(n_s, n_d, dtype=DT[dtype][1], device="cuda", generator=g)


def _kinetic_max(cell):
    """Largest eigenvalue of -1/2 the FD Laplacian (the alternating mode)."""
    t = 0.0
    for s in range(3):
        w0, w = _lap_weights(cell.L[s] / cell.n[s])
        t -= 0.5 * (2 * w0 + 2 * sum(w[q - 1] * (-1) ** q for q in range(1, N_O + 1)))
    return t


def _bounds(cell):
    """Filter interval of a block that has seen a few passes: everything above a tenth of
    the spectrum is damped."""
    lmax = _kinetic_max(cell) + 2.0
    return 0.1 * lmax, lmax


def _gaussians(cell, amp):
    """sum_J sum_images amp_J exp(-|x - R_J - L|^2 / (2 w_J^2)) on the grid (separable)."""
    f = []
    for s in range(3):
        x = torch.arange(cell.n[s], dtype=torch.float64, device="cuda") * (cell.L[s] / cell.n[s])
        R = torch.from_numpy(np.ascontiguousarray(cell.positions[:, s])).cuda()
        w = torch.from_numpy(cell.width).cuda()
        m = int(math.ceil(10.0 * float(cell.width.max()) / cell.L[s])) + 1
        d = x[None, None, :] - R[:, None, None] - cell.L[s] * torch.arange(-m, m + 1, device="cuda").double()[None, :, None]
        f.append(torch.exp(-d * d / (2 * w * w)[:, None, None]).sum(1))
    a = torch.as_tensor(amp, dtype=torch.float64, device="cuda")
    out = torch.zeros(cell.n[2], cell.n[1], cell.n[0], dtype=torch.float64, device="cuda")
    for J in range(len(a)):
        out += a[J] * f[2][J][:, None, None] * f[1][J][None, :, None] * f[0][J][None, None, :]
    return out.reshape(-1)


def _sad(cell):
    rho = _gaussians(cell, cell.Z / (2 * math.pi * cell.width ** 2) ** 1.5)
    dV = math.prod(cell.L[s] / cell.n[s] for s in range(3))
    return rho * (cell.n_elec / (rho.sum() * dV))


def _vloc(cell):
    return _gaussians(cell, -cell.depth)


def _occ(n_s, n_occ):
    """Occupations of a converged state: full levels, a thermal edge, empty levels."""
    i = torch.arange(n_s, dtype=torch.float64, device="cuda")
    g = 0.5 * (1 - torch.tanh((i - n_occ) / 2.0))
    return torch.where(g < 1e-12, torch.zeros_like(g), g)


def _net_inputs(case, seed):
    xs, ys = [], []
    for b in range(case["batch"]):
        cell = _cell(case, seed * 131 + b)
        rho, v = _sad(cell), _vloc(cell)
        y = _gaussians(cell, cell.depth)
        xs.append(torch.stack([rho / rho.mean(), -v], dim=1).float().reshape(-1))
        ys.append((y / y.mean()).float())
    rng = np.random.default_rng([18, seed])
    th = []
    for ci, co in zip(NET_CH[:-1], NET_CH[1:]):
        std = math.sqrt(2.0 / (27 * ci)) * (0.1 if co == 1 else 1.0)
        th += [rng.standard_normal(27 * ci * co) * std, rng.standard_normal(co) * 0.01]
    return torch.cat(xs), torch.cat(ys), np.concatenate(th).astype(np.float32)


def _pass_state(ctx, cells, hams, Xs, dtype):
    """A CheFSI loop's state: bounds by Lanczos, as the SCF has them."""
    lcut, lmax = [], []
    for i, h in enumerate(hams):
        lo, hi = sp.lanczos_bounds(h, Xs[i][0].contiguous(), 20, sp.workspace(h, 20, sp.OP_LANCZOS))
        lcut.append(0.5 * (lo + hi))
        lmax.append(hi)
    ns = [x.shape[0] for x in Xs]
    return dict(ctx=ctx, cells=cells, hams=hams, Xs=Xs, lcut=lcut, lmax=lmax, dt=DT[dtype][0],
                ritz=[torch.zeros(n, dtype=torch.float64, device="cuda") for n in ns],
                occ=[torch.zeros(1, n, dtype=torch.float64, device="cuda") for n in ns],
                rho=[torch.zeros(c.n_d, dtype=torch.float64, device="cuda") for c in cells])


_context = []


def _ctx():
    """One context per process, kept as a program keeps it."""
    if not _context:
        _context.append(sp.Context(0))
    return _context[0]


def prepare(case, seed):
    kind, ctx = case["kind"], _ctx()
    st = dict(case=case, ctx=ctx)
    if kind == "net":
        x, y, th = _net_inputs(case, seed)
        net = sp.DensityNet(ctx, (case["n1"], case["n2"], case["n3"]), max_batch=case["batch"])
        net.set_params(th)
        return dict(st, net=net, x=x, y=y, d=torch.empty_like(y))
    if kind == "cells":
        cells, hams, Xs = [], [], []
        for i, t in enumerate(case["cells"].split(",")):
            n, na, ns, deg = (int(v) for v in t.split(":"))
            cells.append(_cell(dict(case, n1=n, n2=n, n3=n, atoms=na, n_s=ns, degree=deg), seed * 131 + i))
            hams.append(sp.Hamiltonian(ctx, cells[-1], DT[case["dtype"]][0]))
            Xs.append(_block(seed, i, ns, cells[-1].n_d, case["dtype"]))
        st.update(_pass_state(ctx, cells, hams, Xs, case["dtype"]))
        st["plan"] = sp.FilterPlan(ctx, hams, Xs, [c.degree for c in cells])
        st["work"] = sp.rr_batched_workspace(ctx, hams, Xs)
        return st
    cell = _cell(case, seed)
    if kind == "kpoints":
        ks, wk = wl.mp2_kpoints(cell.L)
        ks, nk = ks[:case["n_k"]], case["n_k"]
        hams = [sp.Hamiltonian(ctx, cell, DT[case["dtype"]][0], kpt=k) for k in ks]
        Xs = [_block(seed, b, case["n_s"], cell.n_d, case["dtype"]) for b in range(nk)]
        st.update(_pass_state(ctx, [cell], hams, Xs, case["dtype"]))
        st["plan"] = sp.FilterPlan(ctx, hams, Xs, [cell.degree] * nk)
        st["work"] = sp.rr_batched_workspace(ctx, hams, Xs)
        lam = torch.zeros(nk, case["n_s"], dtype=torch.float64, device="cuda")
        st.update(lam=lam, ritz=list(lam), occ=torch.zeros_like(lam), wk=[1.0 / nk] * nk)
        return st
    if kind == "scf":
        X0 = _block(seed, 0, case["n_s"], cell.n_d, "r64")
        v0 = _block(seed, 1, 1, cell.n_d, "r64")[0].contiguous()
        prm = dict(n_s=case["n_s"], degree=case["degree"], n_first_passes=4, max_iter=case["iters"], lanczos_steps=20,
                   mix_history=8, kT=KT, mix=0.15, tol=1e-12, n_elec=cell.n_elec, poisson_tol=1e-10, filt=sp.R64,
                   rr=sp.GEMM_NATIVE, final_fp64_pass=0, x0_dev=X0, lanczos_v0_dev=v0)
        z = lambda n: torch.zeros(n, dtype=torch.float64, device="cuda")  # noqa: E731
        return dict(st, cell=cell, prm=prm, rho=z(cell.n_d), ritz=z(case["n_s"]), phi=z(cell.n_d))
    ham = sp.Hamiltonian(ctx, cell, DT[case["dtype"]][0], kpt=_kpt(case, cell))
    X0 = _block(seed, 0, case["n_s"], cell.n_d, case["dtype"])
    st.update(cell=cell, ham=ham, X0=X0)
    if kind == "apply":
        st.update(Y=torch.empty_like(X0), work=sp.workspace(ham, case["n_s"], sp.OP_APPLY))
    elif kind == "filter":
        st.update(X=torch.empty_like(X0), work=sp.workspace(ham, case["n_s"], sp.OP_FILTER), bounds=_bounds(cell))
    elif kind == "pass":
        st.update(_pass_state(ctx, [cell], [ham], [X0], case["dtype"]))
        st["work"] = (sp.workspace(ham, case["n_s"], sp.OP_FILTER), sp.workspace(ham, case["n_s"], sp.OP_RR))
    elif kind == "forces":
        X0 /= torch.linalg.vector_norm(X0, dim=1, keepdim=True)
        st.update(rho=_sad(cell), occ=_occ(case["n_s"], cell.n_elec / 2), work=sp.workspace(ham, case["n_s"], sp.OP_FORCES))
        st["F"] = [torch.zeros(case["atoms"], 3, dtype=torch.float64, device="cuda") for _ in range(2)]
    return st


# --------------------------------------------------------------------------------- run
def run(st):
    case, kind = st["case"], st["case"]["kind"]
    if kind == "apply":
        return sp.fd_hamiltonian_apply(st["ham"], st["X0"], st["Y"], st["work"])
    if kind == "filter":
        st["X"].copy_(st["X0"])
        return sp.chebyshev_filter(st["ham"], st["X"], case["degree"], *st["bounds"], st["work"])
    if kind == "pass":
        ham, X, ritz, occ, rho = st["hams"][0], st["Xs"][0], st["ritz"][0], st["occ"][0], st["rho"][0]
        sp.chebyshev_filter(ham, X, case["degree"], st["lcut"][0], st["lmax"][0], st["work"][0])
        sp.rayleigh_ritz(ham, X, ritz, st["work"][1])
        sp.sparc_fermi(st["ctx"], ritz.view(1, -1), [1.0], st["cell"].n_elec, KT, occ)
        sp.density_from_orbitals(st["ctx"], [X], occ, ham.dV, rho, st["dt"])
        st["lcut"][0] = float(ritz[-1])
        return {"ritz": ritz, "occ": occ, "rho": rho}
    if kind == "kpoints":
        st["plan"].run(st["lcut"], st["lmax"])
        sp.rayleigh_ritz_batched(st["ctx"], st["hams"], st["Xs"], st["ritz"], work=st["work"])
        sp.sparc_fermi(st["ctx"], st["lam"], st["wk"], st["cells"][0].n_elec, KT, st["occ"])
        sp.density_from_orbitals(st["ctx"], st["Xs"], st["occ"], st["hams"][0].dV, st["rho"][0], st["dt"])
        st["lcut"] = st["lam"][:, -1].tolist()
        return {"ritz": st["lam"], "occ": st["occ"], "rho": st["rho"][0]}
    if kind == "cells":
        st["plan"].run(st["lcut"], st["lmax"])
        sp.rayleigh_ritz_batched(st["ctx"], st["hams"], st["Xs"], st["ritz"], work=st["work"])
        for i, c in enumerate(st["cells"]):
            sp.sparc_fermi(st["ctx"], st["ritz"][i].view(1, -1), [1.0], c.n_elec, KT, st["occ"][i])
            sp.density_from_orbitals(st["ctx"], [st["Xs"][i]], st["occ"][i], st["hams"][i].dV, st["rho"][i], st["dt"])
        st["lcut"] = torch.stack([r[-1] for r in st["ritz"]]).tolist()
        return {"ritz": st["ritz"], "occ": st["occ"], "rho": st["rho"]}
    if kind == "forces":
        for F in st["F"]:
            F.zero_()
        sp.forces_local(st["ham"], st["rho"], st["F"][0])
        sp.forces_nonlocal(st["ham"], st["X0"], st["occ"], st["F"][1], st["work"])
        return st["F"]
    if kind == "scf":
        out = sp.sparc_scf_run(st["ctx"], st["cell"], st["prm"], st["rho"], st["ritz"], phi_out=st["phi"])
        return {"energy": out["energy"], "mu": out["mu"], "iterations": out["iterations"], "rho": st["rho"],
                "ritz": st["ritz"], "phi": st["phi"]}
    if case["train"]:
        loss, grad = st["net"].loss_grad(st["x"], st["y"])
        st["net"].adam_step(1e-3)
        return {"loss": loss, "grad": grad}
    return st["net"].forward(st["x"], st["d"])


# -------------------------------------------------------------------------------- work
def _entries(case):
    """(node, projector) entries of a cell: the nodes of each cutoff sphere."""
    rc, per = (3.5, 4) if case.get("p") else (3.0, 1)
    return case["atoms"] * per * 4.0 / 3.0 * math.pi * (rc / case["h"]) ** 3


def _step_flops(case, n_d, n_s):
    """Operations of one H X: per direction and tap one sum and one fused product, the
    centre, the potential and the recurrence operand, and both projector products."""
    real = n_d * n_s * (9.0 * N_O + 6.0) + 4.0 * _entries(case) * n_s
    return real * (2.0 if case["dtype"].startswith("c") else 1.0)


def _pass_work(case, n_d, n_s, n_k=1):
    z = 4.0 if case["dtype"].startswith("c") else 1.0
    eb = DT[case["dtype"]][1].itemsize
    b = 2.0 * n_d * n_s * eb + 16.0 * n_d
    # filter and H X; two Hermitian products and the rotation; the dense eigenproblem
    f = (case["degree"] + 1) * _step_flops(case, n_d, n_s) + z * (4.0 * n_d * n_s ** 2 + 9.0 * n_s ** 3)
    return n_k * b, n_k * f


def work(case):
    kind = case["kind"]
    if kind == "cells":
        b = f = 0.0
        for t in case["cells"].split(","):
            n, na, ns, deg = (int(v) for v in t.split(":"))
            w = _pass_work(dict(case, atoms=na, degree=deg), n ** 3, ns)
            b, f = b + w[0], f + w[1]
        return {"bytes": b, "flops": f}
    n_d = case["n1"] * case["n2"] * case["n3"]
    if kind == "net":
        par = sum(ci * co for ci, co in zip(NET_CH[:-1], NET_CH[1:]))
        v = n_d * case["batch"]
        if case["train"]:   # forward, weight gradients, input gradients of all but the first layer
            return {"bytes": 12.0 * v, "flops": 54.0 * v * (3 * par - NET_CH[0] * NET_CH[1])}
        return {"bytes": 12.0 * v, "flops": 54.0 * v * par}
    n_s, eb = case["n_s"], DT[case["dtype"]][1].itemsize
    if kind in ("apply", "filter"):
        steps = case.get("degree", 1)
        return {"bytes": 2.0 * n_d * n_s * eb + 8.0 * n_d, "flops": steps * _step_flops(case, n_d, n_s)}
    if kind == "forces":
        w = 2.0 if case["dtype"].startswith("c") else 1.0
        n_occ = min(n_s, case["atoms"] + 28)    # states with weight
        ent = _entries(case)
        nodes = ent / (4 if case["p"] else 1)
        gauss = case["atoms"] * 4.0 / 3.0 * math.pi * (10 * 1.15 / case["h"]) ** 3
        return {"bytes": nodes * n_occ * eb + 8.0 * n_d,
                "flops": w * n_occ * (nodes * 3 * 3 * N_O + 4.0 * 4 * ent) + 20.0 * gauss}
    b, f = _pass_work(case, n_d, n_s, case.get("n_k", 1))
    if kind == "scf":
        passes = case["iters"] + 3
        return {"bytes": b, "flops": passes * f + case["iters"] * 80 * n_d * (9.0 * N_O + 12.0)}
    return {"bytes": b, "flops": f}


# ------------------------------------------------------------------------------- exact
def _lap_weights(h):
    w0 = -sum(1.0 / (q * q) for q in range(1, N_O + 1)) / (h * h)
    f = math.factorial(N_O)
    return w0, [2.0 * (-1) ** (q + 1) * f * f / (h * h * q * q * math.factorial(N_O - q) * math.factorial(N_O + q))
                for q in range(1, N_O + 1)]


def _shift(X, p, dim, kL):
    """X at index + p along a grid direction, with the Bloch factor of each wrap."""
    n = X.shape[dim]
    i = torch.arange(n, device=X.device) + p
    w = torch.div(i, n, rounding_mode="floor")
    Y = X.index_select(dim, i - w * n)
    if X.is_complex():
        s = [1] * X.dim()
        s[dim] = n
        Y = Y * torch.exp(1j * kL * w.double()).reshape(s)
    return Y


def _projectors(cell, kpt):
    """(atom, gamma, nodes, values) of every projector function."""
    h = [cell.L[s] / cell.n[s] for s in range(3)]
    dV, out = math.prod(h), []
    for c in range(len(cell.chan_atom)):
        J, rc = int(cell.chan_atom[c]), float(cell.chan_rc[c])
        R, sig = cell.positions[J], float(cell.chan_rc[c]) / 4.0
        ax = [np.arange(math.ceil((R[s] - rc) / h[s]), math.floor((R[s] + rc) / h[s]) + 1) for s in range(3)]
        k, j, i = (a.reshape(-1) for a in np.meshgrid(ax[2], ax[1], ax[0], indexing="ij"))
        d = [i * h[0] - R[0], j * h[1] - R[1], k * h[2] - R[2]]
        r2 = d[0] ** 2 + d[1] ** 2 + d[2] ** 2
        keep = r2 <= rc * rc
        i, j, k, r2 = i[keep], j[keep], k[keep], r2[keep]
        w = [i // cell.n[0], j // cell.n[1], k // cell.n[2]]
        g = (i - w[0] * cell.n[0]) + cell.n[0] * ((j - w[1] * cell.n[1]) + cell.n[1] * (k - w[2] * cell.n[2]))
        ph = np.exp(-1j * sum(kpt[s] * cell.L[s] * w[s] for s in range(3)))
        rad = np.exp(-r2 / (2 * sig * sig))
        for f in ([rad] if cell.chan_l[c] == 0 else [rad * v[keep] / sig for v in d]):
            v = ph * f / math.sqrt(dV * float((f * f).sum()))
            val = torch.from_numpy(v if any(kpt) else v.real.copy()).cuda()
            out.append((J, float(cell.chan_gamma[c]), torch.from_numpy(g).cuda(), val))
    return out


class _H:
    """The Hamiltonian in plain torch, 64 bits, on rows of orbitals."""

    def __init__(self, cell, kpt):
        self.cell, self.V, self.P = cell, _vloc(cell), _projectors(cell, kpt)
        self.kL = [kpt[s] * cell.L[s] for s in range(3)]
        self.dV = math.prod(cell.L[s] / cell.n[s] for s in range(3))

    def apply(self, X):
        c = self.cell
        G = X.reshape(-1, c.n[2], c.n[1], c.n[0])
        Y = (self.V * X).reshape(G.shape)
        for s in range(3):
            w0, w = _lap_weights(c.L[s] / c.n[s])
            Y -= w0 * G
            for q in range(1, N_O + 1):
                Y -= 0.5 * w[q - 1] * (_shift(G, q, 3 - s, self.kL[s]) + _shift(G, -q, 3 - s, self.kL[s]))
        Y = Y.reshape(X.shape)
        for _, gam, g, v in self.P:
            a = self.dV * (X[:, g] * v.conj()).sum(1)
            Y.index_add_(1, g, gam * a[:, None] * v)
        return Y

    def filter(self, X, degree, lcut, lmax):
        c, e = 0.5 * (lmax + lcut), 0.5 * (lmax - lcut)
        prev, cur = X, (self.apply(X) - c * X) / e
        for _ in range(1, degree):
            prev, cur = cur, (2 / e) * (self.apply(cur) - c * cur) - prev
        return cur


def _by_rows(X, fn):
    """fn over groups of orbitals, so that the temporaries stay small."""
    rows = max(1, int(2 ** 27 // X.shape[1]))
    return torch.cat([fn(X[a:a + rows]) for a in range(0, X.shape[0], rows)])


def _wide(X):
    return X.to(torch.complex128 if X.is_complex() else torch.float64)


def _exact_pass(H, X, cell, degree):
    """One pass from the first cut, for blocks small enough for a dense eigensolve."""
    v, vs, al, be = X[0] / torch.linalg.vector_norm(X[0]), [], [], []
    for _ in range(20):   # the Lanczos interval
        vs.append(v)
        w = H.apply(v[None])[0]
        al.append(float(torch.vdot(v, w).real))
        for _ in range(2):
            for u in vs:
                w = w - torch.vdot(u, w) * u
        be.append(float(torch.linalg.vector_norm(w)))
        v = w / be[-1]
    th, S = np.linalg.eigh(np.diag(al) + np.diag(be[:-1], 1) + np.diag(be[:-1], -1))
    lmax = th[-1] + abs(be[-1] * S[-1, -1])
    lmax += 0.01 * abs(lmax)
    Y = H.filter(X, degree, 0.5 * (th[0] + lmax), lmax)
    Q = torch.linalg.qr((Y / torch.linalg.vector_norm(Y, dim=1, keepdim=True)).T)[0]
    A = Q.conj().T @ H.apply(Q.T.contiguous()).T
    lam, Z = torch.linalg.eigh(0.5 * (A + A.conj().T))
    U = (Q @ Z).T
    lo, hi = float(lam[0]) - 2, float(lam[-1]) + 2
    for _ in range(200):
        mu = 0.5 * (lo + hi)
        g = 0.5 * (1 - torch.tanh((lam - mu) / (2 * KT)))
        lo, hi = (mu, hi) if float(2 * g.sum()) < cell.n_elec else (lo, mu)
    return {"ritz": lam, "occ": g[None], "rho": (2 / H.dV) * (g[:, None] * U.abs() ** 2).sum(0)}


def _exact_forces(case, cell, H, X):
    rho, occ = _sad(cell), _occ(case["n_s"], cell.n_elec / 2)
    h = [cell.L[s] / cell.n[s] for s in range(3)]
    Fl = torch.zeros(case["atoms"], 3, dtype=torch.float64, device="cuda")
    r3 = rho.reshape(cell.n[2], cell.n[1], cell.n[0])
    for J in range(case["atoms"]):    # separable: per direction the sums of e and of d e over the images
        w, e, de = float(cell.width[J]), [], []
        for s in range(3):
            m = int(math.ceil(10 * w / cell.L[s])) + 1
            d = torch.arange(cell.n[s], device="cuda").double()[None, :] * h[s] - cell.positions[J][s] \
                - cell.L[s] * torch.arange(-m, m + 1, device="cuda").double()[:, None]
            x = torch.exp(-d * d / (2 * w * w))
            e.append(x.sum(0))
            de.append((d * x).sum(0))
        for s in range(3):
            f = [de[q] if q == s else e[q] for q in range(3)]
            Fl[J, s] = H.dV * float(cell.depth[J]) / w ** 2 * torch.einsum("kji,k,j,i->", r3, f[2], f[1], f[0])
    on = torch.nonzero(occ)[:, 0]
    X, occ = X[on], occ[on]
    G = X.reshape(-1, cell.n[2], cell.n[1], cell.n[0])
    f, grads = math.factorial(N_O), []
    for s in range(3):
        D = torch.zeros_like(G)
        for q in range(1, N_O + 1):
            wt = (-1) ** (q + 1) * f * f / (h[s] * q * math.factorial(N_O - q) * math.factorial(N_O + q))
            D += wt * (_shift(G, q, 3 - s, H.kL[s]) - _shift(G, -q, 3 - s, H.kL[s]))
        grads.append(D.reshape(X.shape))
    Fn = torch.zeros_like(Fl)
    for J, gam, g, v in H.P:
        a = H.dV * (X[:, g] * v.conj()).sum(1)
        for s in range(3):
            b = H.dV * (grads[s][:, g] * v.conj()).sum(1)
            Fn[J, s] += -4 * gam / H.dV * (occ * (a.conj() * b).real).sum()
    return [Fl, Fn]


def _exact_net(case, seed):
    x, y, th = _net_inputs(case, seed)
    B, n = case["batch"], (case["n3"], case["n2"], case["n1"])
    x = x.double().reshape(B, *n, 2)
    th = torch.from_numpy(th).cuda().double().requires_grad_(True)
    a, o = x, 0
    for l, (ci, co) in enumerate(zip(NET_CH[:-1], NET_CH[1:])):
        W = th[o:o + 27 * ci * co].reshape(co, ci, 27)
        o += 27 * ci * co
        z = th[o:o + co] + torch.zeros(B, *n, co, dtype=torch.float64, device="cuda")
        o += co
        for t in range(27):
            s = tuple(NET_DIL[l] * (1 - v) for v in (t // 9, t // 3 % 3, t % 3))
            z = z + torch.roll(a, s, (1, 2, 3)) @ W[:, :, t].T
        a = torch.relu(z) if l < 3 else z
    d = a.reshape(B, -1)
    if not case["train"]:
        return d.detach().reshape(-1)
    s = x[..., 0].reshape(B, -1) + d - d.mean(1, keepdim=True)
    loss = ((s - y.double().reshape(B, -1)) ** 2).mean()
    loss.backward()
    return {"loss": float(loss), "grad": th.grad}


def exact(case, seed):
    kind = case["kind"]
    if kind == "net":
        return _exact_net(case, seed)
    if kind in ("cells", "kpoints", "scf"):
        return None
    n_d = case["n1"] * case["n2"] * case["n3"]
    if kind == "pass" and n_d * case["n_s"] > 4e7:
        return None
    cell = _cell(case, seed)
    H = _H(cell, _kpt(case, cell))
    X = _block(seed, 0, case["n_s"], cell.n_d, case["dtype"])
    if kind == "apply":
        return _by_rows(X, lambda x: H.apply(_wide(x)))
    if kind == "filter":
        return _by_rows(X, lambda x: H.filter(_wide(x), case["degree"], *_bounds(cell)))
    if kind == "pass":
        return _exact_pass(H, X, cell, case["degree"])
    X /= torch.linalg.vector_norm(X, dim=1, keepdim=True)
    return _exact_forces(case, cell, H, X)

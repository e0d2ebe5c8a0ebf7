"""Matrix-core kernels of the density network at the edges of their tiles: the smallest
grid, voxel counts that no tile divides, batches whose voxel shares end inside a cell, and
a cell large enough for two voxel tiles per wave, against the oracle in FP64.

Tolerances.  Forward: four layers of up to 864 FP32 products per sum, 4 sqrt(864) 2^-24 =
7e-6 of the output's norm, taken as 2e-5.  Gradient: the sums alone give the same, but a
pre-activation within its own rounding error (1e-6 of its scale) of zero may take the other
side of the ReLU; that fraction of uncorrelated terms moves a gradient by sqrt(1e-6) = 1e-3
of its norm."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import density_net as dn
from paper_1603_04339_amd import sparc as sp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,B", [((9, 9, 9), 1), ((9, 10, 11), 3), ((17, 16, 23), 2), ((33, 18, 20), 5),
                                 ((51, 52, 50), 1)])
def test_forward_and_gradient(n, B):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(sum(n) + B)
    f32 = lambda a: a.astype(np.float32).astype(np.float64)
    th = f32(dn.init_params(rng) + 0.02 * rng.standard_normal(dn.num_params()))
    shape = (n[2], n[1], n[0])
    xs = [f32(1.5 * np.abs(rng.standard_normal(shape))) for _ in range(B)]
    us = [f32(2.0 * np.abs(rng.standard_normal(shape))) for _ in range(B)]
    ys = [f32(np.maximum(x + 0.3 * rng.standard_normal(shape), 0.0)) for x in xs]
    net = sp.DensityNet(sp.Context(0), n, max_batch=B)
    net.set_params(th)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda().reshape(-1)
    x = dev(np.stack([np.stack([a, b], axis=-1) for a, b in zip(xs, us)]))
    d = torch.full((B * xs[0].size,), 7.0, dtype=torch.float32, device="cuda:0")
    net.forward(x, d)
    ref = np.stack([dn.forward(th, a, b)[1][1][-1][0] for a, b in zip(xs, us)]).reshape(-1)
    assert np.linalg.norm(d.cpu().numpy() - ref) < 2e-5 * np.linalg.norm(ref)
    loss, g = net.loss_grad(x, dev(np.stack(ys)))
    lref, gref = dn.loss_and_grad(th, xs, us, ys)
    assert abs(loss - lref) < 2e-5 * lref
    assert np.linalg.norm(g - gref) < 1e-3 * np.linalg.norm(gref)
    # and layer by layer, weights and biases apart; the last bias has no part of its own, its
    # gradient is zero (the loss removes the mean of d)
    o, shapes = 0, dn.layer_shapes()
    for l, (ws, bs) in enumerate(shapes):
        for size in (int(np.prod(ws)), bs[0] if l + 1 < len(shapes) else 0):
            part = slice(o, o + size)
            assert np.linalg.norm(g[part] - gref[part]) <= 1e-3 * np.linalg.norm(gref[part])
            o += size

"""The fused network kernels at the edges of their tiles, against the FP64
reference network: widths around the 16-feature tiles and the 256 and 512
limits, layer widths that are not multiples of 4 (unaligned weight rows),
batches around the 16- and 64-sample blocks and on both sides of 2048, 8192 and
16384 (one launch per layer, whole-network kernel, its wide tiles), one layer
and nine, and the learned guess against the host features and the network.

Tolerances from FP32 rounding, u = 6e-8: a layer sums K products with a random
walk of sqrt(K) u, at most 23 u = 1.4e-6 for K = 512, and layers add up: 1e-5
for outputs and loss (nine layers: below 1.3e-5 in the worst direction, whose
signs do not line up).  A gradient sums n samples of such values: 1e-4, as the
tests of the learned guess hold it.
"""
import numpy as np
import pytest

import workloads as w

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from oracle import mlp as ref  # noqa: E402
from paper_2407_21724_amd import mlfma  # noqa: E402

CASES = [((1, 1), 1), ((3, 17, 2), 15), ((43, 256, 120), 17), ((16, 64, 33, 6), 65), ((43, 257, 30), 48),
         ((7, 512, 40), 33), ((7, 513, 8), 20), ((5,) + (24,) * 8 + (4,), 19), ((11, 37, 256, 9), 2049),
         ((7, 300, 12), 2050), ((9, 40), 2051), ((6, 18, 513, 5), 2052), ((12, 40, 40, 10), 16385),
         ((30, 300, 8), 16390), ((1, 2, 1), 8193)]


def _net(sizes, seed):
    net = mlfma.Mlp(sizes, seed=seed)
    p = net.get_params()
    p += (0.05 * np.random.default_rng(seed).standard_normal(p.size)).astype(np.float32)
    net.set_params(p)
    return net, p, [(W.astype(np.float64), b.astype(np.float64)) for W, b in net.layers(p)]


@pytest.mark.parametrize("sizes,n", CASES)
def test_network_at_tile_edges(sizes, n):
    print(f"network {sizes} batch {n}", flush=True)
    net, p, layers = _net(sizes, 5)
    rng = np.random.default_rng(6)
    X = rng.standard_normal((n, sizes[0])).astype(np.float32)
    T = rng.standard_normal((n, sizes[-1])).astype(np.float32)
    Xd, Td = torch.as_tensor(X, device="cuda"), torch.as_tensor(T, device="cuda")
    y_ref = ref.forward(layers, X.astype(np.float64))[0]
    y = net.forward(Xd).cpu().numpy()
    assert np.linalg.norm(y - y_ref) < 1e-5 * np.linalg.norm(y_ref)
    loss, g = net.loss_grad(Xd, Td)
    assert abs(loss / ref.loss(layers, X.astype(np.float64), T.astype(np.float64)) - 1) < 1e-5
    assert np.array_equal(net.get_params(), p)
    g_ref = np.concatenate([a.ravel() for W, b in ref.gradients(layers, X.astype(np.float64), T.astype(np.float64))
                            for a in (W, b)])
    assert np.linalg.norm(g - g_ref) < 1e-4 * np.linalg.norm(g_ref)
    # Adam's first step from these gradients (large ones: the others are rounding over eps)
    assert abs(net.train_step(Xd, Td, 1e-3) / loss - 1) < 1e-6
    big = np.abs(g) > 1e-3 * np.abs(g).max()
    step = p - net.get_params()
    assert np.abs(step[big] - 1e-3 * np.sign(g[big])).max() < 1e-6


@pytest.mark.parametrize("nx,ny,R,precision,width", [(5, 4, 1, 0, 40), (7, 3, 5, 1, 40), (4, 4, 2, 0, 600),
                                                       (26, 10, 9, 0, 40), (26, 10, 8, 1, 270), (45, 46, 4, 0, 40)])
def test_guess_is_the_network_on_the_host_features(nx, ny, R, precision, width):
    v, t = w.icosphere(0.15, 1)
    e = w.edge_table(t)
    M, _ = mlfma.static_modes(v, t, e, 3, 3)
    rng = np.random.default_rng(nx)
    sites = np.sort(rng.permutation(nx * ny)[:nx * ny - 2])            # two sites empty
    sites[0], sites[-1] = 0, nx * ny - 1
    cen = w.lattice(nx, ny, 0.5)[sites]
    cls = (np.arange(len(cen)) % 2).astype(np.int32)
    ctx = mlfma.Context(cen, cls, 2, mlfma.default_params(precision=precision))
    for c in (0, 1):
        ctx.set_static_modes(c, v, t, e, 3, 3, M, 4.0)
    net = _net((13, width, 24), 9)[0]
    th = rng.uniform(0, 0.4, R)
    khat = np.stack([np.sin(th), 0.1 * th, np.sqrt(1 - np.sin(th) ** 2 - 0.01 * th ** 2)], -1)
    dia = np.array([0.13, 0.31])
    X = ctx.guess_features(dia, 0.4, khat)
    y = net.forward(torch.as_tensor(X.reshape(-1, 13), device="cuda")).cpu().numpy().astype(np.float64)
    want = (y[:, 0::2] + 1j * y[:, 1::2]).reshape(R, len(cen), 12) * np.exp(-2j * np.pi * (khat @ cen.T))[:, :, None]
    got = ctx.learned_guess(net, dia, 0.4, khat).cpu().numpy()
    # the same network outputs times one rotation: two roundings of the result
    assert np.linalg.norm(got - want) < (3e-7 if precision == 0 else 1e-14) * np.linalg.norm(want)

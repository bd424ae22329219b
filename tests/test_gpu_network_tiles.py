"""Layers in launches of their own at the edges of their large tiles (128 features
x 64 samples, 64 x 128): networks that the fused kernel does not take, wider than
512 or deeper than eight layers, with feature counts inside and at the end of a
tile, rows that 16-byte loads do and do not reach, batches that end inside a tile
and inside 16 samples, the tiles as first, inner and last layer and backward.
Against the FP64 reference network.

Tolerances from FP32 rounding, u = 6e-8: a layer sums K products with a random
walk of sqrt(K) u, at most 32 u = 2e-6 for K = 1030: 1e-5 for outputs and loss of
up to four layers, 1e-4 for gradients, which sum the samples as well."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from oracle import mlp as ref  # noqa: E402
from paper_2407_21724_amd import mlfma  # noqa: E402

CASES = [((43, 600, 120), 3331), ((8, 520, 64), 32770), ((7, 515, 190, 3), 10901), ((12, 1024, 600, 16), 8200),
         ((12, 576, 40), 7301), ((16, 40, 2048), 1030), ((9, 33, 1030), 1823), ((5, 1024, 1030, 2), 4097)]


@pytest.mark.parametrize("sizes,n", CASES)
def test_layers_in_large_tiles(sizes, n):
    print(f"network {sizes} batch {n}", flush=True)
    rng = np.random.default_rng(n)
    net = mlfma.Mlp(sizes, seed=2)
    p = net.get_params() + (0.05 * rng.standard_normal(net.num_params)).astype(np.float32)
    net.set_params(p)
    layers = [(W.astype(np.float64), b.astype(np.float64)) for W, b in net.layers(p)]
    X = rng.standard_normal((n, sizes[0])).astype(np.float32)
    T = rng.standard_normal((n, sizes[-1])).astype(np.float32)
    Xd, Td = torch.as_tensor(X, device="cuda"), torch.as_tensor(T, device="cuda")
    X, T = X.astype(np.float64), T.astype(np.float64)
    y_ref = ref.forward(layers, X)[0]
    y = net.forward(Xd).cpu().numpy()
    assert np.linalg.norm(y - y_ref) < 1e-5 * np.linalg.norm(y_ref)
    loss, g = net.loss_grad(Xd, Td)
    assert abs(loss / ref.loss(layers, X, T) - 1) < 1e-5
    g_ref = np.concatenate([a.ravel() for W, b in ref.gradients(layers, X, T) for a in (W, b)])
    assert np.linalg.norm(g - g_ref) < 1e-4 * np.linalg.norm(g_ref)

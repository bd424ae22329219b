"""A training step is synchronous: when it returns, nothing of it is left on its
stream, and the parameters read then are the step's result.  On a stream of its
own, which the copies that read and write parameters do not wait for, with the
layers in launches of their own (256 and 1024 samples), fused (4096) and fused
in wide blocks (20,000)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2407_21724_amd import mlfma  # noqa: E402


@pytest.mark.parametrize("n", [256, 1024, 4096, 20000])
def test_training_step_is_done_when_it_returns(n):
    print(f"batch {n}", flush=True)
    rng = np.random.default_rng(n)
    X = torch.as_tensor(rng.standard_normal((n, 43)).astype(np.float32), device="cuda")
    T = torch.as_tensor(rng.standard_normal((n, 120)).astype(np.float32), device="cuda")
    net = mlfma.Mlp((43, 256, 256, 256, 120), seed=3)
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    for _ in range(5):
        net.train_step(X, T, 1e-3, stream=s)
        idle = s.query()
        p = net.get_params()
        torch.cuda.synchronize()
        assert idle
        assert np.array_equal(p, net.get_params())

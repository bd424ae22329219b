"""The near partials of a class-pair array are in the product whichever kernel
takes its receive: leaf spheres of 8 to 50 samples (a receive whose k fit one
chunk of the grouped kernel, and one with more), batches below and above its
128 column tiles, an array with one far level and one with three, into outputs
that held other values.  Against the FP64 context, every right-hand side.

FP32 rounding (u = 6e-8): a row sums at most 9 x 16 near and 400 far products,
random-walk error below 24 u = 1.4e-6 of the terms' size; 5e-6 holds it."""
import numpy as np
import pytest

import workloads as w

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2407_21724_amd import mlfma  # noqa: E402


@pytest.mark.parametrize("nx,R,params", [
    (4, 128, {"L_leaf": 2}), (4, 128, {"L_leaf": 3}), (4, 127, {"L_leaf": 4}), (4, 128, {"L_leaf": 4}),
    (4, 131, {"L_leaf": 4}), (4, 128, {"L_leaf": 5}), (12, 16, {"L_leaf": 4, "L_rule": 1, "interp_order": 4})])
def test_near_part_is_in_the_product(nx, R, params):
    print(f"{nx} x {nx}, R {R}, {params}", flush=True)
    cen = np.zeros((nx * nx, 3))
    cen[:, 0], cen[:, 1] = 0.5 * (np.arange(nx * nx) % nx), 0.5 * (np.arange(nx * nx) // nx)
    cls = (np.arange(nx * nx) % nx % 2).astype(np.int32)
    ctx = []
    for prec in (mlfma.C64, mlfma.C128):
        c = mlfma.Context(cen, cls, 2, mlfma.default_params(precision=prec, **params))
        for k in range(2):
            v, t = w.icosphere(0.12 + 0.02 * k, 1)
            m = (v, t, w.edge_table(t))
            c.set_static_modes(k, *m, 2, 2, mlfma.static_modes(*m, 2, 2)[0], 4.0)
        ctx.append(c)
    x = torch.as_tensor(w.random_complex((R, nx * nx, 8), 5)).cuda().to(torch.complex64)
    want = ctx[1].matvec(x.to(torch.complex128))
    y = torch.full_like(x, 7.0)
    for _ in range(2):
        ctx[0].matvec(x, out=y)
        err = ((y - want).flatten(1).norm(dim=1) / want.flatten(1).norm(dim=1)).max()
        assert float(err) < 5e-6

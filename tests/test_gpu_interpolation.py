"""Disaggregation is the transpose of aggregation: with it, and the symmetry of
the directions, the far part obeys reciprocity, x_j^T D Z D x_i = x_i^T Z x_j with
D = diag(I, -I) over the two currents (the translation to r at khat is the one to
-r at -khat, and the receiving patterns are the radiating ones conjugated).  The
arrays make the strips, windows and chunks of both kernels partial: odd and
narrow grids (children missing from parents), stencils of 4 and 6 points, finest
levels of 8 to 12, doubling levels (the widest windows), and chunks of 1 row up.
(Finest levels of 16, or doubling from 11, are no test of this: there the
Hankel functions of the translation amplify its own rounding to 3e-5.)

The two sides differ by rounding alone, of the products' size: 6e-7 of the
vectors' norms in FP32 as measured against 64 bits at the start of the parity
tests' range, 4e-14 in FP64; 5e-6 and 1e-12 hold them.
"""
import numpy as np
import pytest

import workloads as w

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2407_21724_amd import mlfma  # noqa: E402


@pytest.fixture(scope="module")
def modes():
    v, t = w.icosphere(0.15, 1)
    e = w.edge_table(t)
    return v, t, e, mlfma.static_modes(v, t, e, 3, 3)[0]


def _context(modes, nx, ny, **params):
    v, t, e, M = modes
    ctx = mlfma.Context(w.lattice(nx, ny, 0.5), np.zeros(nx * ny, np.int32), 1, mlfma.default_params(**params))
    ctx.set_static_modes(0, v, t, e, 3, 3, M, 4.0)
    return ctx


@pytest.mark.parametrize("nx,ny,R,params", [
    (5, 3, 1, {}), (7, 6, 2, {}), (13, 9, 3, {}), (25, 2, 1, {}), (1, 26, 5, {}), (33, 21, 1, {}),
    (12, 12, 2, {"interp_order": 4}), (26, 19, 1, {"interp_order": 4, "L_leaf": 10}), (14, 11, 1, {"L_leaf": 8}),
    (14, 11, 2, {"L_leaf": 12}), (14, 11, 1, {"L_rule": 1, "L_leaf": 8}), (27, 13, 1, {"L_rule": 1, "L_leaf": 9, "interp_order": 4})])
@pytest.mark.parametrize("precision", [0, 1])
def test_far_part_is_reciprocal(modes, nx, ny, R, params, precision):
    print(f"reciprocity {nx}x{ny} R {R} {params} precision {precision}", flush=True)
    ctx = _context(modes, nx, ny, precision=precision, **params)
    x = w.random_complex((R + 1, nx * ny, 12), 4)
    dev = lambda a: torch.as_tensor(np.ascontiguousarray(a)).to("cuda", ctx.dtype)  # noqa: E731
    D = np.r_[np.ones(6), -np.ones(6)]
    Zx = ctx.matvec_parts(dev(x[1:]), mlfma.PART_FAR).cpu().numpy().astype(complex)
    ZDx = ctx.matvec_parts(dev(x[:1] * D), mlfma.PART_FAR).cpu().numpy().astype(complex)[0]
    for r in range(R):
        a, b = np.sum(x[0] * Zx[r]), np.sum(x[1 + r] * D * ZDx)
        size = np.linalg.norm(x[0]) * np.linalg.norm(Zx[r])
        assert abs(a - b) < (1e-12 if precision else 5e-6) * size


@pytest.mark.parametrize("precision", [0, 1])
def test_rows_per_chunk_change_nothing(modes, precision):
    ctx = _context(modes, 21, 14, precision=precision)
    x = torch.as_tensor(w.random_complex((3, 294, 12), 8)).to("cuda", ctx.dtype)
    want = ctx.matvec(x).clone()
    n = ctx.info()["n_levels"]
    for rows in (1, 2, 3, 5, 7, 1000):
        ctx.set_tuning([rows] * n, [rows] * n)
        assert torch.equal(ctx.matvec(x), want), rows

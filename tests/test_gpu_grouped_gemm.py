"""The grouped GEMM and k_gemm_stream at the edges of their tiles: every
product, its near part and the preconditioner against the FP64 context's, for
particle counts around the 16-column tiles and the blocks of a group (128
columns over the batch), batches that split a particle's right-hand sides over
blocks (more than 128), classes of one particle, empty sites, mode counts whose
rows end inside a tile, and mode counts above the grouped kernel's LDS chunks.

FP32 rounding (u = 6e-8): a row sums at most 2 x 968 products with random-walk
error below 44 u = 2.7e-6 of the terms' size; the parity tests measure 6e-7.
5e-6 holds the products; the preconditioner's sums have 160 products at most but
its matrices are inverses (condition below 10): 5e-6 as well."""
import numpy as np
import pytest

import workloads as w

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2407_21724_amd import mlfma  # noqa: E402

_modes = {}


def _mesh(c):
    v, t = w.icosphere(0.12 + 0.02 * c, 1)
    return v, t, w.edge_table(t)


def _ctx(sites, cls, n_modes, precision):
    n_cls = int(max(cls)) + 1
    cen = np.zeros((len(sites), 3))
    cen[:, :2] = 0.5 * np.asarray(sites)
    ctx = mlfma.Context(cen, np.asarray(cls, np.int32), n_cls, mlfma.default_params(precision=precision))
    for c in range(n_cls):
        m = _mesh(c)
        if (c, n_modes) not in _modes:
            _modes[c, n_modes] = mlfma.static_modes(*m, n_modes, n_modes)[0]
        ctx.set_static_modes(c, *m, n_modes, n_modes, _modes[c, n_modes], 4.0)
    return ctx


def _grid(nx, ny, holes=()):
    return [(i, j) for j in range(ny) for i in range(nx) if (i, j) not in holes]


# sites, classes, modes per kind, right-hand sides
CASES = [
    (_grid(3, 1), [0] * 3, 1, 1), (_grid(17, 1), [0] * 17, 3, 16), (_grid(16, 8), [0] * 128, 2, 32),
    (_grid(16, 8), [0] * 128, 2, 33), (_grid(43, 6), [0] * 258, 2, 16), (_grid(4, 3), [0] * 12, 2, 400),
    (_grid(6, 5), [0] * 30, 8, 140), (_grid(5, 5), [0] * 25, 17, 3), (_grid(4, 4), [0] * 16, 20, 6),
    (_grid(3, 3), [0, 1, 2, 3, 0, 1, 2, 3, 4], 2, 1), (_grid(9, 7), [i % 5 for i in range(63)], 3, 5),
    (_grid(9, 7), [i % 5 for i in range(63)], 3, 129), (_grid(8, 8, {(3, 3), (0, 5)}), [i * i % 4 for i in range(62)], 5, 16),
    (_grid(30, 30), [i * 7 % 3 for i in range(900)], 2, 4), (_grid(6, 6), [i % 2 for i in range(36)], 18, 2),
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_products_and_preconditioner_against_fp64(case):
    sites, cls, nm, R = CASES[case]
    print(f"case {case}: {len(sites)} particles, {max(cls) + 1} classes, {4 * nm} unknowns, R {R}", flush=True)
    a, b = _ctx(sites, cls, nm, mlfma.C64), _ctx(sites, cls, nm, mlfma.C128)
    x = torch.as_tensor(w.random_complex((R, len(sites), 4 * nm), 3)).cuda()
    x32 = x.to(torch.complex64)
    x64 = x32.to(torch.complex128)
    for f in (lambda c, v: c.matvec(v), lambda c, v: c.matvec_parts(v, mlfma.PART_NEAR),
              lambda c, v: c.matvec_parts(v, mlfma.PART_FAR), lambda c, v: c.precondition(v)):
        y, want = f(a, x32).to(torch.complex128), f(b, x64)
        assert bool(torch.isfinite(torch.view_as_real(y)).all())
        if float(want.norm()) == 0:
            assert float(y.norm()) == 0
            continue
        err = ((y - want).flatten(1).norm(dim=1) / want.flatten(1).norm(dim=1)).max()
        assert float(err) < 5e-6

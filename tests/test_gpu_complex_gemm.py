"""The complex GEMM of the FP64 product (and of FP32 contexts told to leave the
matrix cores) at the edges of its tiles: every product, its near part and the
preconditioner against the FP32 matrix-core context's, and each row of a batch
against the row alone, for particle counts around the 16 columns of a block,
classes of one particle, empty sites, mode counts whose rows and k-steps end
inside a tile, and batches that split one particle's right-hand sides.

FP32 rounding decides the difference between the two contexts: 5e-6, as for the
FP32 kernels' own test.  A wrong tile or lane is an error of order one.  FP64
alone: rows sum at most 720 products, 4 partial sums, so a row in a batch and the
row alone (same blocks, other columns) differ by rounding, 720 x 2^-53 = 8e-14 at
most; 1e-12 for the whole product holds the other stages as well."""
import numpy as np
import pytest

from test_gpu_grouped_gemm import _ctx, _grid
import workloads as w

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2407_21724_amd import mlfma  # noqa: E402

# sites, classes, modes per kind, right-hand sides
CASES = [
    (_grid(3, 1), [0] * 3, 1, 1), (_grid(17, 1), [0] * 17, 3, 1), (_grid(4, 4), [0] * 16, 4, 7),
    (_grid(5, 5), [0] * 25, 17, 3), (_grid(6, 5), [0] * 30, 8, 33), (_grid(3, 3), [0, 1, 2, 3, 0, 1, 2, 3, 4], 2, 2),
    (_grid(8, 8, {(3, 3), (0, 5)}), [i * i % 4 for i in range(62)], 5, 16), (_grid(2, 2), [0] * 4, 20, 40),
]


def _diff(y, want):
    y, want = y.to(torch.complex128), want.to(torch.complex128)
    assert bool(torch.isfinite(torch.view_as_real(y)).all())
    if float(want.norm()) == 0:
        return float(y.norm())
    return float(((y - want).flatten(1).norm(dim=1) / want.flatten(1).norm(dim=1)).max())


OPS = [lambda c, v: c.matvec(v), lambda c, v: c.matvec_parts(v, mlfma.PART_NEAR),
       lambda c, v: c.matvec_parts(v, mlfma.PART_FAR), lambda c, v: c.precondition(v)]


@pytest.mark.parametrize("case", range(len(CASES)))
@pytest.mark.parametrize("precision", ["c128", "c64"])
def test_complex_gemm(case, precision, monkeypatch):
    sites, cls, nm, R = CASES[case]
    print(f"case {case}: {len(sites)} particles, {max(cls) + 1} classes, {4 * nm} unknowns, R {R}", flush=True)
    ref = _ctx(sites, cls, nm, mlfma.C64)
    x = torch.as_tensor(w.random_complex((R, len(sites), 4 * nm), 4)).cuda().to(torch.complex64)
    want = [f(ref, x) for f in OPS]
    if precision == "c64":
        monkeypatch.setenv("MLFMA_NO_MFMA", "1")
        ctx = _ctx(sites, cls, nm, mlfma.C64)
    else:
        x = x.to(torch.complex128)
        ctx = _ctx(sites, cls, nm, mlfma.C128)
    for f, g in zip(OPS, want):
        y = f(ctx, x)
        assert _diff(y, g) < 5e-6
        if precision == "c128":
            for r in {0, R // 2, R - 1}:
                assert _diff(f(ctx, x[r:r + 1].contiguous()), y[r:r + 1]) < 1e-12

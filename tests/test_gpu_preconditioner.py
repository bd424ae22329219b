"""The FP32 preconditioner on every route its batch can take (blocks of one column
tile streamed, and from 256 tiles on grouped blocks of 1, 2, 4 and 8 tiles cut at
whole columns or inside one), and products whose few blocks take 1, 2 or 4 column
tiles: one class and several, empty sites, batches that are and are not multiples
of 2 and 4, more modes than the grouped kernel holds, and contexts with BF16-split
products, whose preconditioner is FP32.  Against the FP64 context, every
right-hand side.

FP32 rounding (u = 6e-8): the inverse blocks' sums have 160 products at most, a
product's row 1936, random-walk error below 44 u = 2.7e-6 of the terms' size:
5e-6."""
import numpy as np
import pytest

from test_gpu_grouped_gemm import _ctx, _grid
import workloads as w

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2407_21724_amd import mlfma  # noqa: E402

ONE, SOME = [0] * 128, [i * 5 % 3 for i in range(126)]
GRID, HOLES = _grid(16, 8), _grid(16, 8, {(2, 2), (15, 3)})
# sites, classes, modes per kind, right-hand sides, whole product too
CASES = [(GRID, ONE, 2, 1, False), (GRID, ONE, 2, 4, False), (GRID, ONE, 2, 31, False), (GRID, ONE, 2, 32, False),
         (GRID, ONE, 2, 68, False), (GRID, ONE, 8, 141, False), (GRID, ONE, 2, 300, False), (HOLES, SOME, 3, 36, False),
         (HOLES, SOME, 3, 130, False), (HOLES, SOME, 1, 517, False), (_grid(4, 4), [0] * 16, 20, 8, True),
         (GRID, ONE, 20, 6, True), (GRID, ONE, 20, 33, True), (GRID, ONE, 20, 64, True), (HOLES, SOME, 18, 12, True)]


@pytest.mark.parametrize("case", range(len(CASES)))
@pytest.mark.parametrize("precision", ["c64", "bf16"])
def test_preconditioner_routes(case, precision):
    sites, cls, nm, R, product = CASES[case]
    print(f"case {case}: {len(sites)} particles, {max(cls) + 1} classes, {4 * nm} unknowns, R {R}", flush=True)
    a = _ctx(sites, cls, nm, mlfma.C64 if precision == "c64" else mlfma.C64_BF16)
    b = _ctx(sites, cls, nm, mlfma.C128)
    x = torch.as_tensor(w.random_complex((R, len(sites), 4 * nm), 12)).cuda().to(torch.complex64)
    ops = [lambda c, v: c.precondition(v)]
    if product and precision == "c64":
        ops.append(lambda c, v: c.matvec(v))
    for f in ops:
        y, want = f(a, x).to(torch.complex128), f(b, x.to(torch.complex128))
        assert bool(torch.isfinite(torch.view_as_real(y)).all())
        err = ((y - want).flatten(1).norm(dim=1) / want.flatten(1).norm(dim=1)).max()
        assert float(err) < 5e-6

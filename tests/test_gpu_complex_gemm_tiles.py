"""The complex GEMM where each wave takes a column tile of its own (launches from
1536 tiles on in FP64, 4096 in FP32 on the vector unit): the near part and the
preconditioner of every right-hand side bit for bit those of the right-hand side
alone, whose few tiles split k over a block's waves (both sum the same quarters of
k in the same order), and the whole product to rounding.  One class and three,
classes that end inside a block of 64 columns, empty sites, rows and k-steps that
end inside a tile.

Whole product: a row sums at most 1100 products of each stage, whose order a batch
may change; 1e-12 in FP64 and 5e-6 in FP32 as in the kernels' other tests."""
import numpy as np
import pytest

from test_gpu_grouped_gemm import _ctx, _grid
import workloads as w

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2407_21724_amd import mlfma  # noqa: E402

# sites, classes, modes per kind, right-hand sides in FP64, in FP32
CASES = [(_grid(16, 8), [0] * 128, 2, 200, 530), (_grid(9, 7), [i % 3 for i in range(63)], 1, 401, 1100),
         (_grid(8, 8, {(3, 3), (0, 5)}), [0] * 62, 5, 140, 370), (_grid(5, 5), [0] * 25, 17, 230, 570)]


@pytest.mark.parametrize("case", range(len(CASES)))
@pytest.mark.parametrize("precision", ["c128", "c64"])
def test_whole_tiles_equal_split_ones(case, precision, monkeypatch):
    sites, cls, nm, r64, r32 = CASES[case]
    R = r64 if precision == "c128" else r32
    print(f"case {case}: {len(sites)} particles, {max(cls) + 1} classes, {4 * nm} unknowns, R {R}", flush=True)
    if precision == "c64":
        monkeypatch.setenv("MLFMA_NO_MFMA", "1")
    ctx = _ctx(sites, cls, nm, mlfma.C64 if precision == "c64" else mlfma.C128)
    x = torch.as_tensor(w.random_complex((R, len(sites), 4 * nm), 8)).cuda().to(ctx.dtype)
    near = lambda v: ctx.matvec_parts(v, mlfma.PART_NEAR)  # noqa: E731
    yn, yp, y = near(x), ctx.precondition(x), ctx.matvec(x)
    for r in (0, 1, R // 2, R - 1):
        xr = x[r:r + 1].contiguous()
        assert torch.equal(near(xr), yn[r:r + 1])
        assert torch.equal(ctx.precondition(xr), yp[r:r + 1])
        want = ctx.matvec(xr)
        assert float((y[r:r + 1] - want).norm() / want.norm()) < (1e-12 if precision == "c128" else 5e-6)

"""The register-tiled translation against the gathered interaction lists, which
add the same terms in the same order, where a block takes one, two and four
components (batches up to 2048 tiles, odd and even, and above 32768), on grids whose
tiles all touch the edge, end inside a tile, or are narrower than the window.

A sum has 27 terms of 4 rounded products at most: 108 u = 6.5e-6 of its terms'
size in the worst case, 10 u by chance; the two kernels may contract differently.
1e-6 of the product's norm."""
import pytest

from test_gpu_grouped_gemm import _ctx, _grid
import workloads as w

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2407_21724_amd import mlfma  # noqa: E402


@pytest.mark.parametrize("nx, ny, R", [(4, 4, 1), (3, 9, 2), (11, 1, 3), (13, 10, 7), (23, 17, 5), (40, 40, 1),
                                       (40, 40, 3), (40, 40, 50), (33, 38, 61)])
def test_blocks_of_components(nx, ny, R, monkeypatch):
    print(f"{nx} x {ny}, R {R}", flush=True)
    x = torch.as_tensor(w.random_complex((R, nx * ny, 4), 6)).cuda().to(torch.complex64)
    y = _ctx(_grid(nx, ny), [0] * (nx * ny), 1, mlfma.C64).matvec_parts(x, mlfma.PART_FAR)
    monkeypatch.setenv("MLFMA_TRANSLATE", "0")
    want = _ctx(_grid(nx, ny), [0] * (nx * ny), 1, mlfma.C64).matvec_parts(x, mlfma.PART_FAR)
    assert bool(torch.isfinite(torch.view_as_real(y)).all())
    d, n = (y - want).flatten(1).norm(dim=1), want.flatten(1).norm(dim=1)
    assert bool((d <= 1e-6 * n).all())

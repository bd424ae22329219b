"""One GMRES cycle of m steps leaves the smallest residual over the m-dimensional
Krylov space.  Here that is found by least squares in FP64 from the context's own
product and preconditioner, for vectors shorter than a block and just around its
256 and 1024 elements, several right-hand sides (one of them zero), one step,
bases at and past the vectors that a step loads, one pass or two, and both basis
precisions.

FP64 context and basis: products agree to 1e-14, the least squares over the
orthogonalised space loses at most the ratio of first to last residual (1e4):
1e-8 relative holds with room.  An FP32 basis perturbs each direction by 6e-8, so
the residual by about 6e-8 |b| per step (m <= 9): 1e-6 |b|.  An FP32 product is off
by 6.5e-7: 1e-5 |b|."""
import numpy as np
import pytest

from test_gpu_grouped_gemm import _ctx, _grid
import workloads as w

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2407_21724_amd import mlfma  # noqa: E402

# sites, modes per kind, right-hand sides, steps
CASES = [(_grid(3, 1), 1, 1, 1), (_grid(3, 1), 2, 3, 4), (_grid(4, 4), 4, 2, 5), (_grid(5, 4), 4, 1, 8),
         (_grid(5, 13), 4, 3, 9), (_grid(16, 4), 4, 2, 3)]


def _smallest_residuals(ctx, b, m):
    out = []
    for r in range(b.shape[0]):
        br = b[r:r + 1]
        if float(br.norm()) == 0:
            out.append(0.0)
            continue
        V, AV = [br / br.norm()], []
        for _ in range(m):
            a = ctx.matvec(ctx.precondition(V[-1]))
            AV.append(a.flatten())
            for _ in range(2):
                for v in V:
                    a = a - torch.sum(v.conj() * a) * v
            V.append(a / a.norm())
        A = torch.stack(AV, 1).cpu().numpy()
        y = np.linalg.lstsq(A, br.flatten().cpu().numpy(), rcond=None)[0]
        out.append(float(np.linalg.norm(br.flatten().cpu().numpy() - A @ y) / float(br.norm())))
    return np.array(out)


@pytest.mark.parametrize("case", range(len(CASES)))
@pytest.mark.parametrize("always", [False, True])
def test_one_cycle_leaves_the_smallest_residual(case, always):
    sites, nm, R, m = CASES[case]
    print(f"case {case}: {len(sites)} particles, {4 * nm} unknowns, R {R}, {m} steps", flush=True)
    b = torch.as_tensor(w.random_complex((R, len(sites), 4 * nm), 5)).cuda()
    if R > 2:
        b[1] = 0
    c64, c128 = (_ctx(sites, [0] * len(sites), nm, p) for p in (mlfma.C64, mlfma.C128))
    want = _smallest_residuals(c128, b, m)
    for ctx, fp32_basis, tol in ((c128, False, 0.0), (c128, True, 1e-6), (c64, False, 1e-5), (c64, True, 1e-5)):
        v = b.to(torch.complex64 if ctx is c64 else torch.complex128)
        x, st, _ = ctx.gmres_solve(v, rtol=1e-30, max_iter=m, restart=m, always_reorth=always, fp32_basis=fp32_basis)
        assert bool(torch.isfinite(torch.view_as_real(x)).all())
        got = np.array([s["true_rel_res"] for s in st])
        assert np.all(np.abs(got - want) <= 1e-8 * want + 1e-12 + tol), (got, want)
        for r, s in enumerate(st):
            if float(b[r].norm()) == 0:
                assert float(x[r].norm()) == 0
            else:
                assert s["iterations"] == m and (not always or s["reorth"] == m)

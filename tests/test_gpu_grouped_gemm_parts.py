"""The grouped GEMM with 8, 4, 2 and 1 waves to a column tile (the more tiles a
launch has, the fewer), held to the streamed kernel and to FP64, with batches that
are and are not multiples of 4, blocks cut at whole columns and inside a column's
right-hand sides, classes whose columns end inside a block, and the near sum in the
receive's store.  The kernels that ran are read back from the library, so that a
comparison of a kernel with itself fails.

FP32 rounding (u = 6e-8): a row sums at most 1936 products, random-walk error below
44 u = 2.7e-6 of the terms' size: 5e-6 against FP64.  Two FP32 kernels: 5e-6 as
well."""
import numpy as np
import pytest

from test_gpu_grouped_gemm import _ctx, _grid
import workloads as w

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2407_21724_amd import mlfma  # noqa: E402

SQ, ONE, THREE = _grid(40, 40), [0] * 1600, [i * 7 % 3 for i in range(1600)]
RAGGED = _grid(16, 9, {(4, 4), (15, 8)})
# sites, classes, modes per kind, right-hand sides, receive's kernel (template arguments: modes, waves per tile, near sum)
CASES = [
    (SQ, ONE, 1, 8, "k_gemm_group<2, 8, false"), (SQ, ONE, 1, 23, "k_gemm_group<2, 4, false"),
    (SQ, ONE, 1, 41, "k_gemm_group<2, 2, false"), (SQ, ONE, 1, 84, "k_gemm_group<2, 1, false"),
    (SQ, ONE, 1, 83, "k_gemm_group<2, 2, false"),
    (SQ, THREE, 1, 3, "k_gemm_group<2, 8, true"), (SQ, THREE, 1, 21, "k_gemm_group<2, 4, true"),
    (SQ, THREE, 1, 41, "k_gemm_group<2, 2, true"), (SQ, THREE, 1, 84, "k_gemm_group<2, 1, true"),
    (SQ, THREE, 1, 85, "k_gemm_group<2, 2, true"),
    (RAGGED, [i * i % 5 for i in range(142)], 2, 240, "k_gemm_group<2, 4, true"),
    (RAGGED, [i * i % 5 for i in range(142)], 3, 470, "k_gemm_group<2, 2, true"),
    (RAGGED, [0] * 142, 8, 64, "k_gemm_group<2, 8, false"),
]


def _receive(ctx, x):
    ctx.profile(True)
    y = ctx.matvec(x)
    kernels = {s["name"]: s["kernel"] for s in ctx.profile_read()}
    ctx.profile(False)
    return y, kernels["receive"]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_waves_per_tile(case, monkeypatch):
    sites, cls, nm, R, want = CASES[case]
    print(f"case {case}: {len(sites)} particles, {max(cls) + 1} classes, {4 * nm} unknowns, R {R}", flush=True)
    a, b = _ctx(sites, cls, nm, mlfma.C64), _ctx(sites, cls, nm, mlfma.C128)
    a.prepare()  # (the switch below is read when the engine is created)
    monkeypatch.setenv("MLFMA_GEMM", "stream")
    c = _ctx(sites, cls, nm, mlfma.C64)
    c.prepare()
    x = torch.as_tensor(w.random_complex((R, len(sites), 4 * nm), 6)).cuda().to(torch.complex64)
    y, kernel = _receive(a, x)
    ys, stream = _receive(c, x)
    assert kernel.startswith(want) and stream.startswith("k_gemm_stream")
    ref = b.matvec(x.to(torch.complex128))
    n = ref.flatten(1).norm(dim=1)
    assert float(((y - ref).flatten(1).norm(dim=1) / n).max()) < 5e-6
    assert float(((ys - ref).flatten(1).norm(dim=1) / n).max()) < 5e-6
    assert float(((y.to(torch.complex128) - ys).flatten(1).norm(dim=1) / n).max()) < 5e-6


@pytest.mark.parametrize("name,nx,R", [("c2", 6, 128), ("c2", 6, 130), ("c4", 8, 32), ("c4", 8, 33)])
def test_grouped_and_streamed_workloads(name, nx, R, monkeypatch):
    """The same of the cylinder and lens workloads at batches that do take the
    grouped kernel; the near blocks of the lens, which one wave sums in the same
    order in both, bit for bit."""
    wl = w.workload(name, nx, nx)
    Ms = {}
    for c in sorted(set(wl.class_id.tolist())):
        v, t, e = wl.meshes[c]
        Ms[c], _ = mlfma.static_modes(v, t, e, wl.n_perp, wl.n_par)
    ctx = []
    for env in (None, "stream"):
        if env:
            monkeypatch.setenv("MLFMA_GEMM", env)
        k = mlfma.Context(wl.centers, wl.class_id, len(wl.meshes), mlfma.default_params(precision=mlfma.C64))
        for c, M in Ms.items():
            k.set_static_modes(c, *wl.meshes[c], wl.n_perp, wl.n_par, M, wl.eps_r)
        k.prepare()
        ctx.append(k)
    x = torch.as_tensor(w.random_complex((R, wl.n_particles, 60), R)).cuda().to(torch.complex64)
    out = []
    for k in ctx:
        k.profile(True)
        y = k.matvec(x)
        out.append((y, {s["name"]: s["kernel"] for s in k.profile_read()}))
        k.profile(False)
    (y, ka), (ys, kb) = out
    assert ka["near+project"].startswith("k_gemm_group") and kb["near+project"].startswith("k_gemm_stream")
    assert kb["receive"].startswith("k_gemm_stream")
    if name == "c4":
        assert ka["receive"].startswith("k_gemm_group")
        near = [k.matvec_parts(x, mlfma.PART_NEAR) for k in ctx]
        assert torch.equal(*near)
    d = ((y - ys).flatten(1).norm(dim=1) / ys.flatten(1).norm(dim=1)).max()
    assert float(d) < 5e-6

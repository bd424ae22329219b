"""Fields of more (right-hand side, point) pairs than one launch has threads for
along one axis (2^32, 16 of them to a value of the chunk sum): 64 right-hand sides
at 1.42 million points of three spheres, 2.7e8 values.  Each point's sums do not
depend on the others, so runs of points at both ends and in the middle are bit for
bit those of the points alone.  And the right-hand sides that go through the
expansions in groups (1.42 million points; a leaf sphere whose pattern buffer is
smaller than the batch's expansions): bit for bit those of each alone."""
import numpy as np
import pytest

import workloads as w

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2407_21724_amd import mlfma  # noqa: E402


def test_fields_of_many_points():
    R, n = 64, 1_420_000
    v, t = w.icosphere(0.15, 1)
    m = (v, t, w.edge_table(t))
    ctx = mlfma.Context(w.lattice(3, 1, 0.5), np.zeros(3, np.int32), 1, mlfma.default_params())
    ctx.set_static_modes(0, *m, 2, 2, mlfma.static_modes(*m, 2, 2)[0], 4.0)
    x = torch.as_tensor(w.random_complex((R, 3, 8), 1)).cuda().to(torch.complex64)
    rng = np.random.default_rng(2)
    pts = np.c_[rng.uniform(-3, 4, (n, 2)), rng.uniform(1, 5, n)]
    E = ctx.fields(x, pts)
    for a in (0, n // 2, n - 1000):
        assert torch.equal(E[:, a:a + 1000], ctx.fields(x, pts[a:a + 1000]))
    assert torch.equal(E[5:6], ctx.fields(x[5:6].contiguous(), pts))
    assert torch.equal(E[R - 1:], ctx.fields(x[R - 1:].contiguous(), pts))


@pytest.mark.parametrize("L,R,n", [(10, 7, 70), (10, 16, 300), (6, 9, 5), (8, 21, 130)])
def test_fields_of_groups_of_right_hand_sides(L, R, n):
    print(f"L {L}, R {R}, {n} points", flush=True)
    v, t = w.icosphere(0.15, 1)
    m = (v, t, w.edge_table(t))
    ctx = mlfma.Context(w.lattice(5, 4, 0.5), np.zeros(20, np.int32), 1, mlfma.default_params(L_leaf=L, L_rule=1))
    ctx.set_static_modes(0, *m, 2, 2, mlfma.static_modes(*m, 2, 2)[0], 4.0)
    x = torch.as_tensor(w.random_complex((R, 20, 8), 3)).cuda().to(torch.complex64)
    rng = np.random.default_rng(4)
    pts = np.c_[rng.uniform(-3, 4, (n, 2)), rng.uniform(1, 5, n)]
    E = ctx.fields(x, pts)
    for r in range(R):
        assert torch.equal(E[r:r + 1], ctx.fields(x[r:r + 1].contiguous(), pts))

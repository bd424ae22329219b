"""The field sum's harmonic expansion against the Legendre series it stands
for, summed term by term in FP64 from the library's host leaf patterns
(mlfma_debug_leaf_pattern): E(r) = -jk sum_p sum_s w_s T_L(khat_s, r - c_p) U_p(s).
Point counts straddle the kernel's 64-point sets (1, 64, 65, 129, 193), the
15 particles its staged groups of 8 and 4, R its groups of right-hand sides.

Tolerance, from FP32 rounding (2^-24 = 6e-8): the projection sums 40 products,
the expansion 484 and the field sum 144 a particle, each with a random-walk
error of about sqrt(terms) roundings of a term no larger than a few times the
sum, and the harmonics carry one rounding per degree: below 80 roundings, 5e-6.
"""
import numpy as np
import pytest

import workloads as w

K0 = 2 * np.pi


@pytest.mark.gpu
@pytest.mark.parametrize("R,npts,L", [(1, 1, 11), (2, 64, 11), (3, 65, 11), (4, 129, 10), (5, 193, 9), (1, 300, 11)])
def test_field_sum_is_the_legendre_series(R, npts, L):
    import torch

    from paper_2407_21724_amd import mlfma
    v, t = w.icosphere(0.15, 1)
    e = w.edge_table(t)
    M, _ = mlfma.static_modes(v, t, e, 10, 10)
    cen = w.lattice(5, 3, 0.5)
    ctx = mlfma.Context(cen, np.zeros(15, np.int32), 1, mlfma.default_params(L_leaf=L))
    ctx.set_static_modes(0, v, t, e, 10, 10, M, 4.0)
    print(f"fields R {R} points {npts} L {L}", flush=True)
    x = w.random_complex((R, 15, 40), 11)
    rng = np.random.default_rng(3)
    pts = np.stack([rng.uniform(-3, 5, npts), rng.uniform(-3, 4, npts), rng.uniform(0.6, 9, npts)], -1)
    E = ctx.fields(torch.as_tensor(x).to("cuda", torch.complex64), pts).cpu().numpy()
    kh, ws = ctx.debug_level_grid(0)
    th = np.stack([kh[:, 2] * kh[:, 0], kh[:, 2] * kh[:, 1], kh[:, 2] ** 2 - 1], -1)
    th /= np.linalg.norm(th, axis=1)[:, None]
    ph = np.cross(kh, th)
    pat = ctx.debug_leaf_pattern(0).conj()                    # [K][theta, phi][N]
    xe, xm = x[..., :20].astype(np.complex64), x[..., 20:].astype(np.complex64)
    U = [np.einsum("rpn,kn->rpk", xe, pat[:, 0]) + np.einsum("rpn,kn->rpk", xm, pat[:, 1]),
         np.einsum("rpn,kn->rpk", xe, pat[:, 1]) - np.einsum("rpn,kn->rpk", xm, pat[:, 0])]
    ref = np.zeros((R, npts, 3), complex)
    for p in range(15):
        d = pts - cen[p]
        D = np.linalg.norm(d, axis=1)
        mu, z = (d / D[:, None]) @ kh.T, K0 * D
        h = [1j * np.exp(-1j * z) / z, np.exp(-1j * z) * (1j / z ** 2 - 1 / z)]
        leg = [np.ones_like(mu), mu]
        for l in range(1, L):
            h.append((2 * l + 1) / z * h[l] - h[l - 1])
            leg.append(((2 * l + 1) * mu * leg[l] - l * leg[l - 1]) / (l + 1))
        T = sum((-1j) ** l * (2 * l + 1) * h[l][:, None] * leg[l] for l in range(L + 1)) * (-1j * K0 / (4 * np.pi) ** 2)
        for r in range(R):
            ref[r] += -1j * K0 * ((T * ws) @ (U[0][r, p][:, None] * th + U[1][r, p][:, None] * ph))
    assert np.linalg.norm(E - ref) / np.linalg.norm(ref) < 5e-6

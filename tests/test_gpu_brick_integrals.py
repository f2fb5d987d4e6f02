"""Brick integrals where the lanes that share a brick, the build and the integrals alone can
differ: elements ill-conditioned at one end only, sides near the ends of FP32's range,
long elements in FP32."""
import numpy as np
import pytest
import torch

import paper_1501_04784_amd as kb

pytestmark = pytest.mark.gpu

SIGNS = np.array([(-1, -1, -1), (1, -1, -1), (1, 1, -1), (-1, 1, -1), (-1, -1, 1), (1, -1, 1), (1, 1, 1), (-1, 1, 1)])


def alone(x):
    """Bricks [n, 8, 3] that share no node, on the GPU: (conn, coords, coef of ones)."""
    n = x.shape[0]
    return (torch.arange(8 * n, dtype=torch.int32, device="cuda").reshape(n, 8),
            torch.from_numpy(np.ascontiguousarray(x.reshape(-1, 3))).cuda(),
            torch.ones(n, dtype=torch.float64, device="cuda"))


def condition(x):
    """Largest infinity-norm condition number of the Jacobian at the four points of r = -g and of
    r = +g, [n, 2]."""
    g = 1 / np.sqrt(3.0)
    out = []
    for p in [(r, s, t) for r in (-g, g) for s in (-g, g) for t in (-g, g)]:
        f = 1 + SIGNS * p
        dn = np.stack([SIGNS[:, 0] * f[:, 1] * f[:, 2], f[:, 0] * SIGNS[:, 1] * f[:, 2],
                       f[:, 0] * f[:, 1] * SIGNS[:, 2]])
        out.append(np.linalg.cond(np.einsum("ia,naj->nij", dn / 8, x), np.inf))
    return np.stack(out, 1).reshape(-1, 2, 4).max(2)


def test_fallback_counts_elements():
    """An element is ill-conditioned at the points of r = +g only, of r = -g only, at all or
    at none: it is counted once in the first three, whichever kernel integrates it."""
    rng = np.random.default_rng(0)
    n = 700  # of each kind
    x = (SIGNS * 0.5 + 0.5)[None] + rng.uniform(-0.02, 0.02, (4, n, 8, 3))
    thin = 0.03
    for kind, side in ((0, 1), (1, -1)):  # squeezed in z at one end of r
        x[kind][:, SIGNS[:, 0] == side, 2] *= thin
    x[2][..., 2] *= thin
    x = x.reshape(4 * n, 8, 3)[rng.permutation(4 * n)]
    tau = 5.0
    cond = condition(x)
    assert not np.any((cond > tau / 1.15) & (cond < tau * 1.15))  # no half near the threshold
    lo, hi = (cond > tau).T
    assert (hi & ~lo).sum() == (lo & ~hi).sum() == (lo & hi).sum() == n
    mesh, tuning = alone(x), kb.Tuning(fb_tau=tau)
    print("[fallback count]", flush=True)
    _, status = kb.integrate_lower(*mesh, 8, prec="fp32fb64", tuning=tuning)
    assert int(status[1]) == 3 * n
    assert kb.build_lower_csr(*mesh, 8, prec="fp32fb64", tuning=tuning).n_fallback == 3 * n


@pytest.mark.parametrize("prec", ["fp32", "fp32fb64"])
@pytest.mark.parametrize("side", [1e-12, 1e12, 5e12])
def test_sides_near_the_ends_of_fp32(side, prec):
    """The determinant of a brick goes with the cube of its side, which FP32 holds for sides
    from about 5e-13 to 8e12: there the integrals are those of the unit brick times the side."""
    x = np.random.default_rng(1).uniform(-0.1, 0.1, (1000, 8, 3)) + (SIGNS * 0.5 + 0.5)
    conn, unit, coef = alone(x)
    ref, _ = kb.integrate_lower(conn, unit, coef, 8, prec="fp64")
    print(f"[fp32 range] {side:g} {prec}", flush=True)
    got, _ = kb.integrate_lower(conn, unit * side, coef, 8, prec=prec)
    k = kb.build_lower_csr(conn, unit * side, coef, 8, prec=prec)
    for vals in (got, k.vals.reshape(-1, 36)):  # (a row's columns ascend: the packed order)
        err = (vals.double() / side - ref).abs().max().item() / ref.max().item()
        assert err < 2e-6  # some dozen roundings to 24 bits


@pytest.mark.parametrize("prec", ["fp32", "fp32fb64"])
def test_integrals_alone_as_accurate_as_the_build(prec):
    """Long distorted bricks in FP32: both form what the Jacobian is made of in FP64 from
    the coordinates, so the integrals alone are no further off than the matrix."""
    c = (SIGNS * 0.5 + 0.5) * (1, 1, 10)
    x = c + np.random.default_rng(2).uniform(-0.25, 0.25, (20000, 8, 3))
    mesh = alone(x)
    ref, _ = kb.integrate_lower(*mesh, 8, prec="fp64")
    print(f"[fp32 integrals] {prec}", flush=True)
    tuning = kb.Tuning(fb_tau=1e6)  # (FP32 geometry throughout)
    got, _ = kb.integrate_lower(*mesh, 8, prec=prec, tuning=tuning)
    k = kb.build_lower_csr(*mesh, 8, prec=prec, tuning=tuning)
    rms = [(((v.double() - ref).norm(dim=1) / ref.norm(dim=1)) ** 2).mean().sqrt().item()
           for v in (got, k.vals.reshape(-1, 36))]
    assert rms[0] < 1.05 * rms[1], rms  # (20,000 elements: the rms is good to about 1%)

"""The rotation of the inner kernels on the Gram matrix (rotation_h) against the
formulas (4.3)-(4.6) in extended precision, through the kernels' own device function.

With eps = 2^-53, d = h_qq - t h_pp and b = 2 h_pq: tan within 4 eps of the smaller
root of (4.4) (for a hyperbolic pair times the root's condition number, |d| /
sqrt(d^2 - b^2)); cos belongs to the computed tan and is rounded once: cos^2 (1 + t
tan^2) - 1 is within 1.5 eps where cos < 1, whose half unit is eps / 2, and within 2
eps for hyperbolic pairs, whose cos is in [1, 2), where it is eps; zero on average
(0.1 eps is allowed for).  Extended precision adds 2^-64 = eps / 2048 per operation:
eps / 256 for the residual.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

EPS = np.longdouble(2.0) ** -53
X = np.longdouble


def _run(hpp, hqq, hpq, hyp):
    import torch
    from paper_1401_2720_amd import _binding as B
    tn, cs = B.diag_rotation(*(torch.from_numpy(x).cuda() for x in (hpp, hqq, hpq)), hyp)
    return tn.cpu().numpy(), cs.cpu().numpy()


def _pairs(g, count, spread):
    """h_pp, h_qq apart by up to 2^spread, and the sign and relative size of h_pq."""
    e = g.integers(-450 + spread, 449 - spread, count)
    hpp = np.ldexp(g.uniform(1.0, 2.0, count), e)
    hqq = np.ldexp(g.uniform(1.0, 2.0, count), e + g.integers(-spread, spread + 1, count))
    near = g.random(count) < 0.2  # nearly equal, and equal, diagonal entries
    hqq = np.where(near, hpp * (1.0 + g.integers(-64, 65, count) * 2.0 ** -52), hqq)
    r = g.choice([-1.0, 1.0], count) * np.exp(g.uniform(np.log(1e-15), 0.0, count))
    return hpp, hqq, r


@pytest.mark.parametrize("spread", [0, 4, 60, 400])
def test_trigonometric(spread):
    hpp, hqq, r = _pairs(np.random.default_rng(spread), 200000, spread)
    hpq = r * np.sqrt(hpp) * np.sqrt(hqq)
    tn, cs = _run(hpp, hqq, hpq, False)
    d, b = X(hqq) - X(hpp), 2 * X(hpq)
    ref = np.abs(b) / (np.abs(d) + np.sqrt(d * d + b * b))
    ref = np.where((d > 0) == (b > 0), ref, -ref)
    assert np.max(np.abs(X(tn) - ref) / np.abs(ref)) <= 4 * EPS
    res = X(cs) * X(cs) * (1 + X(tn) * X(tn)) - 1
    assert np.max(np.abs(res)) <= 1.5 * EPS
    assert abs(np.mean(res)) <= 0.1 * EPS
    assert np.all((cs > 0) & (cs <= 1.0))


@pytest.mark.parametrize("spread", [0, 4, 60, 400])
def test_hyperbolic(spread):
    hpp, hqq, r = _pairs(np.random.default_rng(100 + spread), 200000, spread)
    hpq = 0.8 * r * 0.5 * (hpp + hqq)  # |coth 2phi| >= 5/4
    tn, cs = _run(hpp, hqq, hpq, True)
    d, b = X(hqq) + X(hpp), 2 * X(hpq)
    root = np.sqrt((d - np.abs(b)) * (d + np.abs(b)))
    ref = -b / (d + root)
    assert np.max(np.abs(X(tn) - ref) / (np.abs(ref) * (d / root))) <= 4 * EPS
    res = X(cs) * X(cs) * (1 - X(tn) * X(tn)) - 1
    assert np.max(np.abs(res)) <= (2 + X(1) / 256) * EPS
    assert abs(np.mean(res)) <= 0.1 * EPS


def test_clamped():
    """|coth 2phi| <= 1 is replaced by 5/4 (Section 4.3.1): |tan| = 1/2."""
    hpp, hqq, r = _pairs(np.random.default_rng(7), 1000, 4)
    hpq = np.sign(r) * (1.0 + np.abs(r)) * 0.5 * (hpp + hqq)
    tn, cs = _run(hpp, hqq, hpq, True)
    assert np.array_equal(tn, -0.5 * np.sign(hpq))
    assert np.max(np.abs(X(cs) * X(cs) * X(0.75) - 1)) <= (2 + X(1) / 256) * EPS

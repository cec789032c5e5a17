"""V's updates of two p-steps at once (w = 32, n >= 2560): orders whose steps
all go two by two but the last (96 here has two single ones in the sweep too),
partly filled and empty last blocks, row counts off the 16-row slices, every
ordering (round robin has no such steps), hyperbolic pairs, and the last V
updates after a sweep limit.

U and V are orthogonal and U S V^T = A within 1e-13 n, as for the other sizes
(V^T J V = J' and G V = U S within 1e-13 n ||V||^2 for the hyperbolic SVD); after
a limited number of sweeps V is orthogonal and A V = U S within the same.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _torch():
    import torch
    import paper_1401_2720_amd as jsvd
    return torch, jsvd


def _ortho(torch, V):
    n = V.shape[1]
    return (V.t() @ V - torch.eye(n, dtype=V.dtype, device=V.device)).abs().max().item()


@pytest.mark.parametrize("m,n,strategy", [(2560, 2560, "rrev"), (2600, 2561, "rrev"),
                                          (2700, 2700, "c"), (2817, 2817, "rrev"),
                                          (3001, 3000, "r"), (2600, 2590, "rr")])
def test_two_steps_at_once(m, n, strategy):
    torch, jsvd = _torch()
    A = torch.randn(m, n, dtype=torch.float64, device="cuda",
                    generator=torch.Generator("cuda").manual_seed(n))
    U, S, V, info = jsvd.gesvd(A, block_w=32, strategy=strategy, qr="off")
    assert info["status"] == 0
    assert _ortho(torch, V) <= 1e-13 * n
    assert (A - (U * S) @ V.t()).norm().item() <= 1e-13 * n * A.norm().item()
    assert _ortho(torch, U) <= 1e-13 * n


@pytest.mark.parametrize("sweeps", [1, 2])
def test_sweep_limit(sweeps):
    torch, jsvd = _torch()
    n = 2600
    A = torch.randn(n, n, dtype=torch.float64, device="cuda",
                    generator=torch.Generator("cuda").manual_seed(5))
    U, S, V, info = jsvd.gesvd(A, block_w=32, max_sweeps=sweeps, qr="off")
    assert info["sweeps"] == sweeps
    assert _ortho(torch, V) <= 1e-13 * n
    assert (A @ V - U * S).norm().item() <= 1e-13 * n * A.norm().item()


def test_hyperbolic():
    torch, jsvd = _torch()
    n = 2600
    G = torch.randn(n + 50, n, dtype=torch.float64, device="cuda",
                    generator=torch.Generator("cuda").manual_seed(6))
    G += 3 * n ** 0.5 * torch.eye(n + 50, n, dtype=torch.float64, device="cuda")
    J = np.ones(n, np.int8)
    J[1500:] = -1
    U, S, V, Jo, info = jsvd.hsvd(G, J, block_w=32)
    assert info["status"] == 0
    Jd = torch.tensor(J, dtype=torch.float64, device="cuda")
    Jt = torch.tensor(np.asarray(Jo), dtype=torch.float64, device="cuda")
    k = V.norm(2).item() ** 2
    assert (V.t() @ (Jd[:, None] * V) - torch.diag(Jt)).abs().max().item() <= 1e-13 * n * k
    assert (G @ V - U * S).norm().item() <= 1e-13 * n * k * G.norm().item()


def test_workspace_holds_the_slots_in_use():
    """Four slots of V' where two p-steps' V updates are done at once, else two."""
    from paper_1401_2720_amd import _binding as B

    def size(n, **opts):
        return B.workspace_size(n, n, block_w=32, qr="off", **opts)

    slot = B.strategy_order((3000 + 31) // 32) // 2 * 64 * 64 * 8
    assert size(3000) - size(3000, want_v=False) >= 2 * slot
    for n, opts in ((2048, {}), (2559, {}), (3000, {"factorize": "qr"})):
        assert size(n, **opts) == size(n, want_v=False, **opts)

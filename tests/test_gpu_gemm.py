"""The general FP64 product through the SVD adjoint (op(A) and op(B) plain and
transposed, beta, the added diagonal) at the edges of its 32 x 32 and 64 x 64
tiles and of its K steps of 32, against the oracle's adjoint.

Given factors: Haar U and V, s_i = 2 - i / n, so F is at most n.  A product
over K terms is off by K eps of its factors' norms, J - J^T is multiplied by
F <= n, and a chain has two more products: within 8 (m + 2 n) n eps of the
result's norm (3e-9 at 1025 x 700, 6e-12 at n <= 32).
"""
import numpy as np
import pytest

from oracle import adjoint

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("b,m,n", [
    (1, 1, 1), (2, 33, 31), (3, 65, 32), (1, 97, 33), (2, 64, 64), (1, 129, 65),
    (260, 40, 31), (130, 65, 33), (70, 129, 64), (1, 1025, 700)])
def test_adjoint_at_tile_edges(b, m, n):
    import torch
    import paper_1401_2720_amd as jsvd
    rng = np.random.default_rng(1000 * m + n)
    U = np.linalg.qr(rng.standard_normal((b, m, n)))[0]
    V = np.linalg.qr(rng.standard_normal((b, n, n)))[0]
    S = np.broadcast_to(2.0 - np.arange(n) / n, (b, n)).copy()
    dU, dS, dV = (rng.standard_normal(x.shape) for x in (U, S, V))
    t = lambda x: torch.from_numpy(x).cuda()
    got = jsvd.svd_backward(t(U), t(S), t(V), t(dU), t(dS), t(dV)).cpu().numpy()
    tol = max(1e-13, 8 * (m + 2 * n) * n * np.finfo(float).eps)
    for i in range(b):
        want = adjoint.svd_adjoint(U[i], S[i], V[i], dU[i], dS[i], dV[i])
        assert np.linalg.norm(got[i] - want) <= tol * np.linalg.norm(want), i

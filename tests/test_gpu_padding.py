"""Padding columns of the last blocks, unit vectors in the pivot Gram matrices, beside
columns of smaller norm: they must not change places with them when the columns of a
pair are ordered by norm.  Every width, with the padding in one block, over a whole
block, and over more than one; columns of one scale, of several, and zero.

Tolerances: sigma within 1e-12 sigma + 1e-13 sigma_1, orthogonality and the
reconstruction within 1e-13 n, as for the other parity tests.
"""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def _columns(kind, m, n):
    g = np.random.default_rng(1000 * m + n)
    A = g.standard_normal((m, n)) * 1e-3
    if kind == "scales":
        A *= 10.0 ** -np.linspace(0.0, 6.0, n)[g.permutation(n)]
    elif kind == "zeros":
        A[:, g.random(n) < 0.3] = 0.0
    return A


@pytest.mark.parametrize("w", [16, 32, 64])
@pytest.mark.parametrize("m,n", [(20, 3), (21, 17), (70, 65), (130, 100), (200, 129), (200, 193),
                                 (340, 330)])
@pytest.mark.parametrize("kind", ["one scale", "scales", "zeros"])
def test_padding_keeps_its_place(kind, m, n, w):
    import torch
    import paper_1401_2720_amd as jsvd
    A = _columns(kind, m, n)
    U, S, V, info = jsvd.gesvd(torch.from_numpy(A).cuda(), block_w=w, qr="off")
    assert info["status"] == 0 and info["block_w"] == w
    U, S, V = (x.cpu().numpy() for x in (U, S, V))
    ref = oracle.gesvj(A)["S"]
    assert np.all(np.abs(S - ref) <= 1e-12 * ref + 1e-13 * ref[0])
    assert np.max(np.abs(V.T @ V - np.eye(n))) <= 1e-13 * n
    assert np.linalg.norm(A - (U * S) @ V.T) <= 1e-13 * n * np.linalg.norm(A)


@pytest.mark.parametrize("n", [33, 40, 65, 129, 250])
def test_batched_padding_keeps_its_place(n):
    import torch
    import paper_1401_2720_amd as jsvd
    mats = [_columns(kind, n + 5, n) for kind in ("one scale", "scales", "zeros")]
    b = jsvd.Batch(mats)
    jsvd.gesvd_batched(b)
    torch.cuda.synchronize()
    assert b.status.tolist() == [0, 0, 0]
    for i, A in enumerate(mats):
        U, S, V = b.results(i)
        ref = oracle.gesvj(A)["S"]
        assert np.all(np.abs(S - ref) <= 1e-12 * ref + 1e-13 * ref[0])
        assert np.max(np.abs(V.T @ V - np.eye(n))) <= 1e-13 * n
        assert np.linalg.norm(A - (U * S) @ V.T) <= 1e-13 * n * np.linalg.norm(A)

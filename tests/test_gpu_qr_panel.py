"""The QR panel kernel's two workgroup sizes, with one workgroup and with
several: row counts at the edges (512, 1024 and 8192 rows per change of size or
count), a partly filled last panel and one column, and the output order of many
columns, against numpy.

Tolerances: sigma within 1e-12 sigma + 1e-13 sigma_1, orthogonality and the
reconstruction within 1e-13 n, as for the other parity tests.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n", [(40, 1), (512, 33), (513, 40), (1024, 64), (1025, 70), (1060, 96),
                                 (8192, 31), (8193, 40), (8230, 70), (20000, 37)])
def test_qr_row_edges(m, n):
    import torch
    import paper_1401_2720_amd as jsvd
    A = np.random.default_rng(m + n).standard_normal((m, n)) * np.geomspace(1, 1e-2, n)
    U, S, V, info = jsvd.gesvd(torch.from_numpy(A).cuda(), qr="on")
    assert info["status"] == 0
    U, S, V = (x.cpu().numpy() for x in (U, S, V))
    ref = np.linalg.svd(A, compute_uv=False)
    assert np.all(np.abs(S - ref) <= 1e-12 * ref + 1e-13 * ref[0])
    assert np.max(np.abs(V.T @ V - np.eye(n))) <= 1e-13 * n
    assert np.max(np.abs(U.T @ U - np.eye(n))) <= 1e-13 * n
    assert np.linalg.norm(A - (U * S) @ V.T) <= 1e-13 * n * np.linalg.norm(A)


@pytest.mark.parametrize("n,n_plus", [(33, 33), (300, 300), (257, 100)])
def test_output_order(n, n_plus):
    """Diagonal input with ties: nothing rotates, the order is the kernel's."""
    import torch
    import paper_1401_2720_amd as jsvd
    d = np.random.default_rng(n).integers(1, 40, n).astype(float)
    D = torch.from_numpy(np.diag(d)).cuda()
    J = np.ones(n, np.int8)
    J[n_plus:] = -1
    if n_plus == n:
        _, S, V, _ = jsvd.gesvd(D, qr="off", max_sweeps=1)
        want = np.argsort(-d, kind="stable")
    else:
        _, S, V, _, _ = jsvd.hsvd(D, J, max_sweeps=1)
        want = np.r_[np.argsort(-d[:n_plus], kind="stable"),
                     n_plus + np.argsort(d[n_plus:], kind="stable")]
    assert np.array_equal(S.cpu().numpy(), d[want])
    assert np.array_equal(np.abs(V.cpu().numpy()), np.eye(n)[:, want])

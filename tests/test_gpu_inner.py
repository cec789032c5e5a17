"""The inner kernel that rotates the pivot Gram matrix (unscaled Cholesky
path): sizes at the edges of its block pairs, every ordering, both widths,
more than one inner sweep, hyperbolic pairs, and inputs whose Gram matrices
are only semidefinite, against the oracle.

Tolerances: sigma within 1e-12 sigma + 1e-13 sigma_1, orthogonality and the
reconstruction within 1e-13 n, as for the other parity tests.
"""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def _jsvd():
    import torch
    import paper_1401_2720_amd as jsvd
    return torch, jsvd


def _check(A, U, S, V, ref):
    n = A.shape[1]
    assert np.all(np.abs(S - ref) <= 1e-12 * ref + 1e-13 * ref[0])
    assert np.max(np.abs(V.T @ V - np.eye(n))) <= 1e-13 * n
    assert np.linalg.norm(A - (U * S) @ V.T) <= 1e-13 * n * np.linalg.norm(A)


# one column; one block pair with padding in either block; a padding block; a
# full pair; one column more
@pytest.mark.parametrize("m,n,w", [(5, 1, 16), (33, 15, 16), (40, 17, 16), (40, 32, 16),
                                   (90, 33, 16), (70, 31, 32), (70, 33, 32), (64, 64, 32),
                                   (150, 65, 32)])
@pytest.mark.parametrize("strategy", ["rrev", "c", "rr"])
def test_edges(m, n, w, strategy):
    torch, jsvd = _jsvd()
    A = np.random.default_rng(100 * n + w).standard_normal((m, n))
    U, S, V, info = jsvd.gesvd(torch.from_numpy(A).cuda(), block_w=w, strategy=strategy, qr="off")
    assert info["status"] == 0
    _check(A, U.cpu().numpy(), S.cpu().numpy(), V.cpu().numpy(), oracle.gesvj(A)["S"])


@pytest.mark.parametrize("w", [16, 32])
def test_more_inner_sweeps(w):
    torch, jsvd = _jsvd()
    A = np.random.default_rng(w).standard_normal((120, 100))
    U, S, V, info = jsvd.gesvd(torch.from_numpy(A).cuda(), block_w=w, max_inner_sweeps=4,
                               qr="off")
    assert info["status"] == 0 and info["inner_sweeps"] > info["pair_updates"]
    _check(A, U.cpu().numpy(), S.cpu().numpy(), V.cpu().numpy(), oracle.gesvj(A)["S"])


@pytest.mark.parametrize("w", [16, 32])
@pytest.mark.parametrize("n_plus", [1, 40, 69])
def test_hyperbolic(w, n_plus):
    torch, jsvd = _jsvd()
    n = 70
    G = np.random.default_rng(7).standard_normal((90, n))
    J = np.r_[np.ones(n_plus), -np.ones(n - n_plus)].astype(np.int8)
    U, S, V, Jo, info = jsvd.hsvd(torch.from_numpy(G).cuda(), J, block_w=w)
    assert info["status"] == 0
    U, S, V = U.cpu().numpy(), S.cpu().numpy(), V.cpu().numpy()
    lam = np.linalg.eigvalsh((G * J) @ G.T)
    lam = np.sort(lam[np.argsort(-np.abs(lam))[:n]])[::-1]
    assert np.max(np.abs(Jo * S * S - lam)) <= 1e-12 * np.max(np.abs(lam))
    vmax = max(1.0, np.max(np.abs(V)) ** 2)
    assert np.max(np.abs(V.T @ (J[:, None] * V) - np.diag(Jo))) <= 1e-13 * n * vmax
    assert np.linalg.norm(G @ V - U * S) <= 1e-13 * n * np.linalg.norm(G) * np.linalg.norm(V, 2)


# zero columns, repeated columns, columns of one direction: pivots of the
# Gram matrices that are zero or negative by rounding
@pytest.mark.parametrize("kind", ["zero", "repeated", "rank1", "rank20"])
@pytest.mark.parametrize("w", [16, 32])
def test_semidefinite(kind, w):
    torch, jsvd = _jsvd()
    g = np.random.default_rng(11)
    A = g.standard_normal((80, 50))
    if kind == "zero":
        A[:, ::3] = 0.0
    elif kind == "repeated":
        A[:, 25:] = A[:, :25]
    elif kind == "rank1":
        A = np.outer(g.standard_normal(80), g.standard_normal(50))
    else:
        A = g.standard_normal((80, 20)) @ g.standard_normal((20, 50))
    U, S, V, info = jsvd.gesvd(torch.from_numpy(A).cuda(), block_w=w, qr="off")
    assert info["status"] == 0
    _check(A, U.cpu().numpy(), S.cpu().numpy(), V.cpu().numpy(),
           np.linalg.svd(A, compute_uv=False))


@pytest.mark.parametrize("value", [np.nan, np.inf])
def test_nonfinite(value):
    torch, jsvd = _jsvd()
    A = np.random.default_rng(3).standard_normal((60, 40))
    A[7, 5] = value
    with pytest.raises(jsvd.JsvdError) as e:
        jsvd.gesvd(torch.from_numpy(A).cuda(), qr="off", scaled="off")
    assert e.value.code == 3


# the batched path's blocked method: one block pair and its padding, odd and
# even block counts, the largest n; columns that repeat; a NaN in one problem
@pytest.mark.parametrize("n", [33, 47, 48, 49, 64, 65, 96, 97, 130, 256])
def test_batched_blocked_edges(n):
    torch, jsvd = _jsvd()
    g = np.random.default_rng(n)
    mats = [g.standard_normal((n + k, n)) for k in (0, 1, 17)]
    mats[1][:, n // 2:2 * (n // 2)] = mats[1][:, :n // 2]
    bad = g.standard_normal((n, n))
    bad[3, 2] = np.nan
    b = jsvd.Batch(mats + [bad])
    jsvd.gesvd_batched(b)
    torch.cuda.synchronize()
    assert b.status.tolist() == [0, 0, 0, 3]
    for i, A in enumerate(mats):
        U, S, V = b.results(i)
        _check(A, U, S, V, np.linalg.svd(A, compute_uv=False))


# the batched path's one-wave problems: every lane-group width (n up to 4, 8,
# 16, 32), rows in registers or not, and the first sizes that do not fit a wave
@pytest.mark.parametrize("want_v", [True, False])
def test_batched_wave_edges(want_v):
    torch, jsvd = _jsvd()
    g = np.random.default_rng(5)
    sizes = [(1, 1), (7, 1), (3, 2), (70, 2), (4, 4), (33, 5), (8, 8), (9, 9), (17, 12), (16, 16),
             (65, 16), (17, 17), (33, 25), (32, 32), (64, 32), (65, 32), (90, 24), (300, 7),
             (300, 20), (40, 33)]
    mats = [g.standard_normal(s) for s in sizes]
    mats.append(g.standard_normal((30, 18)) * 10.0 ** -np.linspace(0, 12, 18))
    mats.append(np.zeros((12, 6)))
    mats.append(np.repeat(g.standard_normal((20, 1)), 5, axis=1))
    b = jsvd.Batch(mats, want_v=want_v)
    jsvd.gesvd_batched(b)
    torch.cuda.synchronize()
    assert int(b.status.abs().sum()) == 0
    for i, A in enumerate(mats):
        U, S, V = b.results(i)
        ref = oracle.gesvj(A)["S"]
        if want_v:
            _check(A, U, S, V, ref)
        assert np.all(np.abs(S - ref) <= 1e-12 * ref + 1e-13 * ref[0])
        U = U[:, S > 1e-10 * S[0]]
        assert np.max(np.abs(U.T @ U - np.eye(U.shape[1])), initial=0.0) <= 1e-13 * 40

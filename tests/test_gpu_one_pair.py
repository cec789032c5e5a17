"""The whole solve of one pivot pair (n <= 32, w = 16) in one launch, against
the oracle: one column, padding in either block, a full pair, rows at the edges
of the 16-row slices and of the eight waves' 128, and the largest m (768; 769
takes the block path); every ordering, no V, no sort, more inner sweeps, sweep
limits, hyperbolic pairs, and inputs that it leaves to the block path or that
have nothing to do.

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


def _host(*x):
    return [t.cpu().numpy() for t in x]


@pytest.mark.parametrize("m,n", [(1, 1), (17, 1), (15, 15), (16, 16), (17, 17), (24, 17), (31, 31),
                                 (32, 32), (127, 20), (129, 32), (768, 32), (769, 32)])
@pytest.mark.parametrize("strategy", ["rrev", "c", "rr"])
def test_sizes(m, n, strategy):
    torch, jsvd = _jsvd()
    A = np.random.default_rng(100 * m + n).standard_normal((m, n))
    U, S, V, info = jsvd.gesvd(torch.from_numpy(A).cuda(), block_w=16, strategy=strategy, qr="off")
    assert info["status"] == 0 and info["converged"] == 1 and info["n_blocks"] == 2
    assert info["pair_updates"] <= info["sweeps"] <= 12
    _check(A, *_host(U, S, V), oracle.gesvj(A)["S"])


def test_options():
    torch, jsvd = _jsvd()
    A = np.random.default_rng(3).standard_normal((60, 29))
    T = torch.from_numpy(A).cuda()
    ref = oracle.gesvj(A)["S"]
    U, S, V, info = jsvd.gesvd(T, block_w=16, max_inner_sweeps=4, qr="off")
    assert info["inner_sweeps"] > info["pair_updates"]
    _check(A, *_host(U, S, V), ref)
    _, S, V, info = jsvd.gesvd(T, block_w=16, want_v=False, qr="off")
    assert V is None and np.all(np.abs(S.cpu().numpy() - ref) <= 1e-12 * ref)
    U, S, V, info = jsvd.gesvd(T, block_w=16, sort=False, qr="off")
    U, S, V = _host(U, S, V)
    p = np.argsort(-S)
    _check(A, U[:, p], S[p], V[:, p], ref)
    U, S, V, info = jsvd.gesvd(T, block_w=16, max_sweeps=2, qr="off")
    assert info["sweeps"] == 2 and info["status"] == 1 and info["converged"] == 0
    U, S, V = _host(U, S, V)
    assert np.max(np.abs(V.T @ V - np.eye(29))) <= 1e-13 * 29
    assert np.linalg.norm(A - (U * S) @ V.T) <= 1e-13 * 29 * np.linalg.norm(A)


@pytest.mark.parametrize("n_plus", [1, 13, 22])
def test_hyperbolic(n_plus):
    torch, jsvd = _jsvd()
    n = 23
    rng = np.random.default_rng(8)
    G = rng.standard_normal((70, n))
    J = np.ones(n, np.int8)
    J[rng.permutation(n)[n_plus:]] = -1
    U, S, V, Jo, info = jsvd.hsvd(torch.from_numpy(G).cuda(), J, block_w=16)
    assert info["status"] == 0
    U, S, V = _host(U, S, V)
    k = np.linalg.norm(V, 2) ** 2
    assert np.max(np.abs(V.T @ (J[:, None] * V) - np.diag(Jo))) <= 1e-13 * n * k
    assert np.linalg.norm(G @ V - U * S) <= 1e-13 * n * k * np.linalg.norm(G)


@pytest.mark.parametrize("scale", [2.0 ** 390, 2.0 ** -390, 2.0 ** 700, 2.0 ** -700])
def test_scales(scale):
    torch, jsvd = _jsvd()
    A = np.random.default_rng(9).standard_normal((40, 21))
    U, S, V, info = jsvd.gesvd(torch.from_numpy(A * scale).cuda(), block_w=16, qr="off")
    assert info["status"] == 0 and info["scaled"] == (abs(np.log2(scale)) > 480)
    U, S, V = _host(U, S, V)
    _check(A, U, S / scale, V, oracle.gesvj(A)["S"])


def test_nothing_to_do_and_nonfinite():
    torch, jsvd = _jsvd()
    Z = torch.zeros(30, 12, dtype=torch.float64, device="cuda")
    U, S, V, info = jsvd.gesvd(Z, block_w=16, qr="off")
    assert info["status"] == 0 and info["rotations"] == 0 and not S.any() and not U.any()
    D = torch.diag(torch.arange(1.0, 21.0, dtype=torch.float64, device="cuda"))
    U, S, V, info = jsvd.gesvd(D, block_w=16, qr="off")
    assert info["sweeps"] == 1 and info["rotations"] == 0
    assert torch.equal(S.cpu(), torch.arange(20.0, 0.0, -1.0, dtype=torch.float64))
    _, S, _, _ = jsvd.gesvd(D, block_w=16, qr="off", sort=False)  # no rotation orders them
    assert torch.equal(S.cpu(), torch.arange(1.0, 21.0, dtype=torch.float64))
    Z[3, 4] = float("nan")
    _, _, _, info = jsvd.gesvd(Z, block_w=16, qr="off", allow=(1, 2, 3, 4, 5))
    assert info["status"] not in (0, 1)

"""The batched path's one-wave kernel: every lane-group width (n up to 4, 8, 16,
32), rows at the edges of what a lane keeps in registers and beyond, with V and
without, zero, repeated and graded columns; and the three kernels of a large
mixed batch side by side.  The library says which kernels take a batch; every
problem occurs many times, so that the batch is large, all copies have to come
out with the same bits, and the first is compared with the oracle.

Tolerances: sigma within 1e-12 sigma + 1e-13 sigma_1, orthogonality and the
reconstruction within 1e-13 n, as for the other parity tests.
"""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

# largest n of the batch (a lane-group width), its (m, n)
WIDTHS = {
    4: [(1, 1), (31, 1), (700, 1), (2, 2), (33, 2), (3, 3), (63, 3), (4, 4), (64, 4), (65, 4),
        (257, 4), (764, 4)],
    8: [(5, 5), (32, 5), (33, 6), (7, 7), (64, 7), (8, 8), (65, 8), (128, 8), (129, 8), (300, 8),
        (376, 8)],
    16: [(9, 9), (32, 9), (33, 10), (13, 13), (16, 16), (64, 16), (65, 15), (65, 16), (130, 12),
         (176, 16)],
    32: [(17, 17), (32, 17), (33, 18), (20, 20), (25, 25), (31, 31), (32, 32), (33, 32), (64, 31),
         (64, 32)],
}
NO_V = {32: [(65, 17), (65, 32), (79, 24), (96, 32)], 16: [(192, 16), (129, 11)],
        8: [(384, 8)], 4: [(768, 4)]}
COPIES = 250


def _jsvd():
    import torch
    import paper_1401_2720_amd as jsvd
    return torch, jsvd


def _special(n):
    """Zero, repeated, parallel and graded columns."""
    g = np.random.default_rng(n)
    m = n + 7
    z = g.standard_normal((m, n))
    z[:, ::2] = 0.0
    graded = g.standard_normal((m, n)) * 10.0 ** -np.linspace(0, 12, n)
    return [np.zeros((m, n)), z, np.repeat(g.standard_normal((m, 1)), n, axis=1),
            np.outer(g.standard_normal(m), g.standard_normal(n)), graded]


def _run(mats, want_v, kernels):
    torch, jsvd = _jsvd()
    from paper_1401_2720_amd import _binding as B
    b = jsvd.Batch(mats * COPIES, want_v=want_v)
    assert B.batched_kernels(b) == kernels
    print(f"{b.count} problems, max_m {b.max_m}, max_n {b.max_n}", flush=True)
    jsvd.gesvd_batched(b)
    torch.cuda.synchronize()
    assert int(b.status.abs().sum()) == 0
    for x in (b.A, b.S, b.V) if want_v else (b.A, b.S):
        x = x.view(COPIES, -1)
        assert torch.equal(x, x[:1].expand_as(x))
    for i, A in enumerate(mats):
        n = A.shape[1]
        U, S, V = b.results(i)
        ref = oracle.gesvj(A)["S"]
        assert np.all(np.abs(S - ref) <= 1e-12 * ref + 1e-13 * ref[0]), A.shape
        U1 = U[:, S > 1e-10 * S[0]] if S[0] > 0 else U[:, :0]
        assert np.max(np.abs(U1.T @ U1 - np.eye(U1.shape[1])), initial=0.0) <= 1e-13 * 40, A.shape
        if want_v:
            assert np.max(np.abs(V.T @ V - np.eye(n))) <= 1e-13 * n, A.shape
            assert np.linalg.norm(A - (U * S) @ V.T) <= 1e-13 * n * np.linalg.norm(A), A.shape


@pytest.mark.parametrize("want_v", [True, False])
@pytest.mark.parametrize("width", list(WIDTHS))
def test_every_lane_group_width(width, want_v):
    g = np.random.default_rng(width)
    sizes = WIDTHS[width] + ([] if want_v else NO_V[width])
    mats = [g.standard_normal(s) for s in sizes] + _special(width)
    _run(mats, want_v, {"wave"})


@pytest.mark.parametrize("want_v", [True, False])
def test_beside_the_other_kernels(want_v):
    """Problems that fit a wave, that do not although n <= 32, and larger ones."""
    g = np.random.default_rng(5)
    sizes = [(1, 1), (70, 2), (33, 5), (8, 8), (17, 12), (65, 16), (33, 25), (32, 32), (64, 32),
             (90, 24), (90, 25), (300, 7), (300, 20), (400, 31), (97, 32), (40, 33), (64, 48),
             (120, 64)]
    mats = [g.standard_normal(s) for s in sizes] + _special(6) + _special(21) + _special(33)
    _run(mats, want_v, {"blocked", "wave", "pointwise"})


def _uniform(A, count, want_v, kernels):
    torch, jsvd = _jsvd()
    from paper_1401_2720_amd import _binding as B
    b = jsvd.Batch.from_uniform(torch.from_numpy(A).cuda().expand(count, *A.shape), want_v=want_v)
    assert B.batched_kernels(b) == kernels, count
    assert B.batched_kernels(b, scaled="on") == {"pointwise"}
    jsvd.gesvd_batched(b)
    torch.cuda.synchronize()
    assert int(b.status.abs().sum()) == 0
    A, S = b.A.view(count, -1), b.S.view(count, -1)
    assert torch.equal(S, S[:1].expand_as(S)) and torch.equal(A, A[:1].expand_as(A))
    return A[0].cpu().numpy(), S[0].cpu().numpy()


@pytest.mark.parametrize("m,n,want_v,turns", [
    (64, 24, False, 0), (65, 24, False, 2), (96, 32, False, 2), (65, 9, True, 2), (64, 16, True, 0),
    (97, 8, True, 1), (96, 8, True, 0), (513, 4, True, 1), (512, 4, True, 0), (52, 32, True, 0),
    (53, 32, True, 1), (64, 20, True, 0), (64, 21, True, 1)])
def test_few_problems_of_many_rows_stay_in_a_workgroup(m, n, want_v, turns):
    """Up to `turns` problems per CU the pointwise kernel takes a batch of so many rows,
    from there on the one-wave kernel does.  (For the longer columns the sort decides
    up to six times as many problems: one more of equal size is enough.)"""
    torch, _ = _jsvd()
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    A = np.random.default_rng(m + n).standard_normal((m, n))
    ref = oracle.gesvj(A)["S"]
    many = _uniform(A, 12 * cus + 1, want_v, {"wave"})
    sort = turns and (m > 64 or n <= 8)
    more = _uniform(A, turns * cus + 1, want_v, {"wave", "pointwise"} if sort else {"wave"})
    assert np.array_equal(more[0], many[0]) and np.array_equal(more[1], many[1])
    for _, S in [many] + ([_uniform(A, turns * cus, want_v, {"pointwise"})] if turns else []):
        assert np.all(np.abs(S - ref) <= 1e-12 * ref + 1e-13 * ref[0])


@pytest.mark.parametrize("m,n,turns", [(100, 24, 2), (300, 8, 1)])
def test_the_sort_decides_by_all_sizes(m, n, turns):
    """One long problem among small ones: pointwise until the sum of n exceeds
    `turns` problems of that one's n per CU.  Which kernel had it shows in U's bits."""
    torch, jsvd = _jsvd()
    from paper_1401_2720_amd import _binding as B
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    A = np.random.default_rng(m * n).standard_normal((m, n))
    by_wave = _uniform(A, 12 * cus + 1, True, {"wave"})[0]
    by_workgroup = _uniform(A, cus, True, {"pointwise"})[0]
    assert not np.array_equal(by_wave, by_workgroup)
    room = turns * cus * n - n  # for the other problems' n, k of each but the last few
    k = n // 4
    for extra, want in ((0, by_workgroup), (1, by_wave)):
        small = np.random.default_rng(1).standard_normal((k + 3, k))
        ones = room % k + extra
        b = jsvd.Batch([A] + [small] * (room // k) + [small[:, :1]] * ones)
        assert turns * cus < b.count <= 6 * turns * cus
        assert B.batched_kernels(b) == {"wave", "pointwise"}
        jsvd.gesvd_batched(b)
        torch.cuda.synchronize()
        assert int(b.status.abs().sum()) == 0
        assert np.array_equal(b.results(0)[0].ravel(order="F"), want), extra


def test_the_sort_leaves_short_problems_to_waves():
    """Bounds of more than 64 rows, but only a problem for the blocked kernel has them.
    Which kernel had the first one shows in U's bits."""
    torch, jsvd = _jsvd()
    from paper_1401_2720_amd import _binding as B
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    g = np.random.default_rng(2)
    A, big = g.standard_normal((60, 30)), g.standard_normal((90, 40))
    by_wave = _uniform(A, 12 * cus + 1, False, {"wave"})[0]
    for others in (1, 2 * cus):
        b = jsvd.Batch([A, big] + [g.standard_normal((2, 1))] * others, want_v=False)
        assert B.batched_kernels(b) == {"blocked", "wave", "pointwise"}
        jsvd.gesvd_batched(b)
        torch.cuda.synchronize()
        assert int(b.status.abs().sum()) == 0
        assert np.array_equal(b.results(0)[0].ravel(order="F"), by_wave)
        ref = oracle.gesvj(big)["S"]
        assert np.all(np.abs(b.results(1)[1] - ref) <= 1e-12 * ref + 1e-13 * ref[0])


def test_the_sort_decides_anew_at_every_replay():
    """The sizes of a captured batch may change between replays (within its bounds):
    the sort gives the problems to waves or to workgroups each time, and the bits are
    those of an eager call."""
    torch, jsvd = _jsvd()
    from paper_1401_2720_amd import _binding as B
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    count, m, n = 2 * cus + 40, 100, 24
    g = np.random.default_rng(3)
    b = jsvd.Batch([g.standard_normal((m, n)) for _ in range(count)])
    assert B.batched_kernels(b) == {"wave", "pointwise"}
    small = torch.full_like(b.n, 5)
    small[0] = n
    sizes = {"all": torch.full_like(b.n, n), "one": small}
    eager = {}
    for name, ns in sizes.items():
        b.n.copy_(ns)
        jsvd.gesvd_batched(b)
        torch.cuda.synchronize()
        eager[name] = [x.clone() for x in (b.A, b.S, b.V)]
    graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph, stream=side):
            jsvd.gesvd_batched(b, restore=False)
    torch.cuda.current_stream().wait_stream(side)
    for name in ("one", "all", "one", "all", "all"):
        b.n.copy_(sizes[name])
        b.A.copy_(b.A0)
        b.S.copy_(eager[name][1]).mul_(0.0 if name == "all" else 1.0)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        used = [slice(None)] * 3
        if name == "one":  # the others' buffers beyond 5 columns keep what was there
            used = [slice(0, m * n), slice(0, n), slice(0, n * n)]
        for x, y, u in zip((b.A, b.S, b.V), eager[name], used):
            assert torch.equal(x[u], y[u]), name
        assert int(b.status.abs().sum()) == 0

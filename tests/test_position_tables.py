"""The host tables by which the inner kernels move the entries of the Gram matrix and
the columns of V', and by which V's updates of two p-steps go together, against the
strategy table and by playing the moves (no GPU needed)."""
import numpy as np
import pytest

import paper_1401_2720_amd as jsvd
from paper_1401_2720_amd import _binding as B

KINDS = ["rrev", "r", "crev", "c", "rr"]


@pytest.mark.parametrize("order", [32, 64])
@pytest.mark.parametrize("kind", KINDS)
def test_positions_follow_the_strategy(order, kind):
    ref = jsvd.strategy_table(order, kind) - 1
    t, pos0 = B.position_table(order, kind)
    t = t.astype(int)
    ns, np_ = order - 1, order // 2
    pos = np.full((ns, order), -1)
    for s in range(ns):
        x, y = t[s, :, 4], t[s, :, 5]
        assert sorted(map(tuple, np.sort(np.c_[x, y], axis=1))) == sorted(map(tuple, ref[s]))
        pos[s, x], pos[s, y] = np.arange(np_), np_ + np.arange(np_)
    assert np.array_equal(pos[0], pos0)
    for s in range(ns):
        x, y = t[s, :, 4], t[s, :, 5]
        before, after = pos[s - 1], pos[(s + 1) % ns]
        assert np.array_equal(t[s, :, :4], np.c_[before[x], before[y], after[x], after[y]])
        # two columns of one pair meet in no other one: the entry that is annihilated next
        # lies in the block of two different pairs
        assert np.all(before[x] % np_ != before[y] % np_)
        # the columns written by a wave go to different rows (columns) of positions
        assert len(set(after[x] % np_)) == len(set(after[y] % np_)) == np_
        assert np.array_equal(t[s, :, 6] & 1, (x > y).astype(int))


@pytest.mark.parametrize("order", [32, 64])
@pytest.mark.parametrize("kind", KINDS)
def test_slots_keep_and_send_the_right_columns(order, kind):
    """The V waves' moves: a slot keeps one column, sends the other, and has the next
    pair when the one sent to it has come."""
    t, _ = B.position_table(order, kind)
    t = t.astype(int)
    ns, np_ = order - 1, order // 2
    kept = [t[0, k, 5] if t[0, k, 6] & 2 else t[0, k, 4] for k in range(np_)]
    other = [t[0, k, 4] if t[0, k, 6] & 2 else t[0, k, 5] for k in range(np_)]
    for s in range(ns):
        for k in range(np_):
            x, y, flags = t[s, k, 4:7]
            assert (kept[k], other[k]) == ((y, x) if flags & 2 else (x, y)), (s, k)
        if s + 1 == ns:
            assert np.all(t[s, :, 6] & 4)
            break
        stay = [kept[k] if t[s, k, 6] & 4 else other[k] for k in range(np_)]
        sent = [other[k] if t[s, k, 6] & 4 else kept[k] for k in range(np_)]
        assert sorted(t[s, :, 7]) == list(range(np_))
        kept, other = stay, [None] * np_
        for k in range(np_):
            other[t[s, k, 7]] = sent[k]


def test_position_table_refuses_bad_arguments():
    L, buf = jsvd.lib(), np.zeros(1 << 16, np.uint8)
    assert L.jsvd_position_table(16, 0, buf.ctypes.data) == -1
    assert L.jsvd_position_table(128, 0, buf.ctypes.data) == -1
    assert L.jsvd_position_table(32, 9, buf.ctypes.data) == -2
    assert L.jsvd_position_table(32, 0, None) == -3


@pytest.mark.parametrize("order", [2, 4, 6, 8, 12, 24, 32, 40, 64, 80, 88, 96, 128, 160])
@pytest.mark.parametrize("kind", KINDS)
def test_steps_two_by_two(order, kind):
    t = jsvd.strategy_table(order, kind) - 1
    at, quads = B.step_groups(order, kind)
    np_ = order // 2

    def together(s):  # do steps s and s + 1 exchange blocks inside groups of two pairs?
        where = {b: i for i, pr in enumerate(t[s]) for b in pr}
        feeds = {}
        for j, (p, q) in enumerate(t[s + 1]):
            if where[p] == where[q]:
                return False
            feeds.setdefault(frozenset((where[p], where[q])), []).append(j)
        return all(len(v) == 2 for v in feeds.values())

    s, used = 0, 0
    while s < order - 1:
        if s + 2 < order and order > 2 and together(s):
            assert at[s] == at[s + 1] == used
            old, new = set(), set()
            for ia, ib, jx, jy, a0, b0, z0, z1 in quads[used:used + np_ // 2]:
                assert z0 == z1 == 0
                pa, pb = set(t[s][ia]), set(t[s][ib])
                assert a0 in pa and b0 in pb
                (a1,), (b1,) = pa - {a0}, pb - {b0}
                assert set(t[s + 1][jx]) == {a0, b0} and set(t[s + 1][jy]) == {a1, b1}
                old |= {ia, ib}
                new |= {jx, jy}
            assert old == new == set(range(np_))
            used += np_ // 2
            s += 2
        else:
            assert at[s] == -1
            s += 1
    assert used == len(quads)
    if kind == "rr" and order >= 8:
        assert used == 0
    if kind != "rr" and order in (32, 64, 128):
        assert np.count_nonzero(at < 0) == 1


def test_step_groups_refuse_bad_arguments():
    L, buf = jsvd.lib(), np.zeros(1 << 12, np.int32)
    p = buf.ctypes.data
    assert L.jsvd_step_groups(26, 0, p, p) == -1
    assert L.jsvd_step_groups(7, 0, p, p) == -1
    assert L.jsvd_step_groups(8, 9, p, p) == -2
    assert L.jsvd_step_groups(8, 0, None, p) == -3
    assert L.jsvd_step_groups(8, 0, p, None) == -3

"""The orders in which the BCSR tile kernels deal block-rows (host code, no GPU): every block-row once, even lists."""
import numpy as np
import pytest

from test_wcsr_lists import lists_of  # noqa: F401  (the program that prints them)


@pytest.mark.parametrize("lengths", [
    [3], [0, 0, 5, 0], list(range(40)),
    list(np.random.default_rng(1).binomial(28, 0.1, 148)),          # 18944 x 3584 in 128-row blocks at 90 %
    list(np.random.default_rng(2).binomial(148, 0.1, 28)),          # 3584 x 18944
    list(np.random.default_rng(3).geometric(0.05, 300)),
    list(np.random.default_rng(4).geometric(0.05, 4096 + 37)),      # long lists
])
def test_every_block_row_once_in_even_lists(lists_of, lengths):  # noqa: F811
    lengths = [int(n) for n in lengths]
    got = lists_of("order", *lengths)
    first = np.concatenate([[0], np.cumsum(lengths)])
    filled = sum(n > 0 for n in lengths)
    for lists in (16, 32, 64):
        rows = got[str(lists)]
        assert sorted(r[0] for r in rows) == list(range(len(lengths)))
        assert all(r[1] == first[r[0]] and r[2] == lengths[r[0]] for r in rows)
        assert all(r[2] > 0 for r in rows[:filled]) and not any(r[2] for r in rows[filled:])
        assert [v[0] for v in got["prefix%d" % lists]] == [0] + list(np.cumsum([r[2] + 1 for r in rows]))
        sums = [sum(r[2] + 1 for r in rows[:filled][j::lists]) for j in range(lists)]
        if filled >= 4 * lists:   # a few entries in every list: within one median block-row and a tenth of the mean
            assert max(sums) <= 1.1 * np.mean(sums) + np.median(lengths) + 1


@pytest.mark.parametrize("lengths", [
    [3], [0, 0, 5, 0], [0, 0],
    list(np.random.default_rng(1).binomial(28, 0.1, 148)),
    list(np.random.default_rng(2).binomial(148, 0.1, 28)),
    list(np.random.default_rng(3).geometric(0.05, 300)),
    list(np.random.default_rng(4).geometric(0.05, 512)), [1] * 513,  # the most block-rows that get shares, and one more
])
def test_shares_hold_every_block_row_once_per_tile(lists_of, lengths):  # noqa: F811
    lengths = [int(n) for n in lengths]
    got = lists_of("shares", *lengths)
    filled = [r for r, n in enumerate(lengths) if n > 0]
    if not 0 < len(filled) <= 512:
        assert set(got) == {"passes"} and got["passes"][0] == [0, 0]
        return
    at = np.concatenate([[0], np.cumsum(lengths)])
    whole = got["whole"]   # the order for whole tiles, with the empty block-rows (whose rows of C are cleared) at its end
    assert whole == lists_of("order", *lengths)["32"]
    once = [sum(r[2] + 2 for r in whole[:len(filled)][j::32]) for j in range(32)]
    back = [sum(r[2] + 2 for r in whole[:len(filled)][::-1][j::32]) for j in range(32)]
    assert got["passes"][0] == [max(once), max(x + y for x, y in zip(once, back))]
    for t in range(1, 25):
        rows, first = got["t%d" % t], [v[0] for v in got["first%d" % t]]
        assert sorted(r[0] for r in rows) == filled
        assert all(r[1] == at[r[0]] and r[2] == lengths[r[0]] for r in rows)
        per_tile = 256 // t
        assert first[0] == 0 and first == sorted(first) and set(first[per_tile:]) == {len(filled)}
        sums = [sum(r[2] + 2 for r in rows[first[j]:first[j + 1]]) for j in range(per_tile)]
        assert got["longest%d" % t][0] == [max(sums)]
        # no worse than a longest-first deal: below the mean plus the heaviest block-row
        assert max(sums) <= sum(sums) / per_tile + max(lengths) + 2


def _partly_empty(rows, empty, seed):
    rng = np.random.default_rng(seed)
    return np.where(rng.random(rows) < empty, 0, rng.binomial(64, 0.3, rows))


# (column tiles, block-row lengths): few tiles, many, half and more of the block-rows empty (whose runs of equal weight are short
# of work to launch or too long), one filled block-row
@pytest.mark.parametrize("n_tiles,lengths", [
    (2, _partly_empty(400, 0, 1)), (16, _partly_empty(400, 0, 2)), (16, np.random.default_rng(3).geometric(0.05, 300)),
    (3, _partly_empty(2048, 0.5, 4)), (3, _partly_empty(2048, 0.6, 5)), (6, _partly_empty(2048, 0.75, 6)),
    (16, _partly_empty(2048, 0.75, 7)), (1, np.r_[6250, np.zeros(1199, int)]), (64, np.zeros(40, int)),
])
def test_register_staged_runs_weigh_the_same(lists_of, n_tiles, lengths):  # noqa: F811
    got = lists_of("staged", n_tiles, 256, *lengths)
    start, rows = [v[0] for v in got["start"]], len(lengths)
    assert start[0] == 0 and start[8] == rows * n_tiles and start == sorted(start)
    by_length = got["sorted"][0][0]
    order = [v[0] for v in got["order"]] if by_length else range(rows)
    assert sorted(order) == list(range(rows))
    assert max(np.diff(start)) <= 4 * -(-rows * n_tiles // 8)
    tile = 3 if 2 * np.count_nonzero(lengths) <= rows else 1   # a tile's own cost, in blocks
    weight = np.tile(lengths[np.array(order)] + tile, n_tiles)
    runs = [int(weight[a:b].sum()) for a, b in zip(start, start[1:])]
    # in the order of length runs of equal weight, to one tile; in the stored order an eighth of the tiles, wherever the long ones are
    eighth = -(-rows * n_tiles // 8)
    even = [int(c.sum()) for c in np.split(np.tile(lengths + tile, n_tiles), range(eighth, rows * n_tiles, eighth))]
    assert max(runs) <= (weight.sum() / 8 + max(lengths) + tile if by_length else max(even))

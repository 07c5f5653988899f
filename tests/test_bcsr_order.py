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

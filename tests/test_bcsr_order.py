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

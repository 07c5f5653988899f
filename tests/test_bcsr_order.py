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
        assert got == {"infos": [[0]]}
        return
    at = np.concatenate([[0], np.cumsum(lengths)])
    whole = got["whole"]   # the order for whole tiles, with the empty block-rows (whose rows of C are cleared) at its end
    assert whole == lists_of("order", *lengths)["32"]
    for t in (t for t in range(1, 24) if t % 8):
        rows, first = got["t%d" % t], [v[0] for v in got["first%d" % t]]
        assert sorted(r[0] for r in rows) == filled
        assert all(r[1] == at[r[0]] and r[2] == lengths[r[0]] for r in rows)
        per_tile = 256 // t
        assert first[0] == 0 and first == sorted(first) and set(first[per_tile:]) == {len(filled)}
        sums = [sum(r[2] + 2 for r in rows[first[j]:first[j + 1]]) for j in range(per_tile)]
        assert [v[0] for v in got["load%d" % t]] == sums + [0] * (256 - per_tile)
        # no worse than a longest-first deal: below the mean plus the heaviest block-row
        assert max(sums) <= sum(sums) / per_tile + max(lengths) + 2


def _walked(n_tiles, t, orders, shares, start):
    """Blocks + 2 a tile of every workgroup of a launch of 128x512 tiles, tile by tile as the kernel takes them: workgroup w of an
    XCD the tiles w, w + 32, ... of the XCD's run, then a list of one of the t shared N-tiles."""
    load = np.zeros((8, 32), int)
    whole = n_tiles - t
    for x in range(8):
        if t:
            rows = [r for r in shares["whole"] if r[2] > 0]
            first, last, group = whole // 8 * x * len(rows), whole // 8 * (x + 1) * len(rows), 1
        else:
            rows = [r for r in orders["16"] if r[2] > 0]
            first, last, group = start[x], start[x + 1], 2
        for w in range(32):
            for tile in range(first + w, last, 32):
                g, rest = divmod(tile, group * len(rows))
                place = rest // min(group, n_tiles - g * group)
                load[x, w] += rows[len(rows) - 1 - place if g % 2 else place][2] + 2
            if t and (x * 32 + w) // (256 // t) < t:
                l = (x * 32 + w) % (256 // t)
                f = [v[0] for v in shares["first%d" % t]]
                load[x, w] += sum(r[2] + 2 for r in shares["t%d" % t][f[l]:f[l + 1]])
    return load


# (N-tiles, K, block-row lengths)
_UNEVEN = [(n, k, lengths) for k, lengths in [
    (18944, np.random.default_rng(2).binomial(148, 0.1, 28)), (18944, np.random.default_rng(5).binomial(148, 0.1, 16)),
    (18944, np.minimum(148, np.random.default_rng(6).geometric(0.07, 40))), (3584, np.random.default_rng(1).binomial(28, 0.1, 148)),
    (8192, np.random.default_rng(7).binomial(64, 0.1, 64)), (2048, np.r_[np.zeros(9, int), np.arange(60) % 16]),
] for n in (3, 9, 13, 17, 26, 36)]


@pytest.mark.parametrize("n_tiles,k,lengths", _UNEVEN, ids=lambda v: len(v) if np.ndim(v) else v)
def test_shared_tiles_by_what_is_walked(lists_of, n_tiles, k, lengths):  # noqa: F811
    orders, shares = lists_of("order", *lengths), lists_of("shares", *lengths)
    for xt in (0, 1):
        got = lists_of("wide", n_tiles, k, xt, 256, *lengths)
        start = [v[0] for v in got["start"]]
        heaviest = dict(got["heaviest"])
        assert sorted(heaviest) == [0] + [t for t in range(1, 24) if t <= n_tiles and (n_tiles - t) % 8 == 0]
        for t, most in heaviest.items():
            load = _walked(n_tiles, t, orders, shares, start)
            assert load.sum() == n_tiles * sum(n + 2 for n in lengths if n) and load.max() == most
        # whatever is taken for the sake of L2, no workgroup walks much more than with pairs of N-tiles
        assert heaviest[got["shared"][0][0]] <= 1.3 * heaviest[0]
    assert lists_of("wide", n_tiles, k, 0, 128, *lengths)["shared"] == [[0]]   # the lists are for 256 workgroups


# (column tiles, K, block, width, workgroups to a compute unit, block-row lengths): an XCD's runs that end inside the lists
@pytest.mark.parametrize("n_tiles,k,b,width,per_cu,lengths", [
    (5, 2560, 64, 256, 2, np.random.default_rng(1).binomial(40, 0.1, 160)), (12, 1536, 64, 128, 2, np.random.default_rng(2).binomial(24, 0.1, 44)),
    (37, 18944, 64, 64, 4, np.random.default_rng(3).binomial(296, 0.1, 56)), (9, 2688, 128, 128, 2, np.random.default_rng(4).binomial(21, 0.1, 54)),
    (3, 600, 32, 256, 2, np.r_[np.zeros(7, int), np.random.default_rng(5).geometric(0.1, 90)]), (1, 64, 128, 64, 2, [1]), (2, 64, 32, 64, 4, [0, 0, 3]),
], ids=lambda v: len(v) if np.ndim(v) else v)
def test_ring_walks_even_workgroups(lists_of, n_tiles, k, b, width, per_cu, lengths):  # noqa: F811
    orders = lists_of("order", *lengths)
    resident = 32 * per_cu                   # workgroups of an XCD
    for xt in (0, 1):
        got = lists_of("ring", n_tiles, k, b, width, xt, per_cu, *lengths)
        most = {}
        for group, lists, heaviest, *start in got["walk"]:
            assert start[0] == 0 and start[8] == n_tiles * len(lengths)
            rows = orders[str(lists)]
            wgs = min(resident, max(max(np.diff(start)), 1, n_tiles * len(lengths) // 8))
            load = np.zeros((8, wgs), int)
            for x in range(8):
                for tile in range(start[x], start[x + 1]):
                    g, rest = divmod(tile, group * len(rows))
                    place = rest // min(group, n_tiles - g * group)
                    load[x, (tile - start[x]) % wgs] += rows[len(rows) - 1 - place if g % 2 else place][2] + 1
            assert load.sum() == n_tiles * (sum(lengths) + len(lengths)) and load.max() == heaviest
            most[group, lists] = heaviest
        taken = tuple(got["taken"][0])
        assert most[taken] <= 1.35 * min(most.values())   # (the price of slabs and of A may ask for a little)
        assert b < 128 or taken[1] < 64                   # these handles have no such order


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


@pytest.mark.parametrize("block,brows,units,longest,tokens,row_tiles", [
    (128, 28, 414, 22, 256, 2), (128, 28, 414, 22, 1024, 4),     # 3584 x 18944 at 90 %
    (128, 28, 414, 22, 32, 0), (32, 500, 9000, 30, 500, 0),      # no more than 32 tokens; 32-row blocks
    (128, 52, 104, 8, 71, 0), (128, 48, 72, 6, 80, 0),           # 6656 x 2816, 6144 x 1024: little work, most of it start and end
    (64, 178, 552, 9, 82, 0), (64, 178, 552, 9, 300, 2),         # 11392 x 1920
    (128, 28, 281, 14, 263, 0), (128, 28, 281, 40, 263, 2),      # 3520 x 6208: 280 strips of about a length; of very different ones
])
def test_products_that_take_staged_strips(lists_of, block, brows, units, longest, tokens, row_tiles):  # noqa: F811
    assert lists_of("xt", block, brows, units, longest, tokens)["staged"] == [[row_tiles]]


@pytest.mark.parametrize("block,brows,widths", [
    (32, 6250, {1: 64, 64: 64, 65: 128, 70: 128, 127: 128, 130: 256, 257: 128, 300: 128, 385: 256, 513: 128, 641: 256, 2050: 256}),
    (64, 3125, {33: 64, 70: 128, 129: 256, 201: 256, 257: 128, 390: 256, 600: 128, 770: 256}),
    (128, 1563, {70: 128, 130: 256, 300: 128, 390: 256, 1290: 256}),
    (128, 391, {70: 64, 127: 64, 257: 128, 450: 128, 513: 128, 641: 128, 1290: 256}),      # few tiles: narrower ones
    (64, 20, {70: 64, 4000: 64, 8001: 128, 30000: 256}),
])
def test_unaligned_rows_take_tiles_that_they_fill(lists_of, block, brows, widths):  # noqa: F811
    assert lists_of("unaligned", block, brows, *widths)["bn"] == [[bn] for bn in widths.values()]


@pytest.mark.parametrize("block,brows,units,longest,widths", [
    (128, 148, 207, 6, {2048: 0, 3072: 1, 4096: 1}), (128, 100, 200, 10, {4096: 1, 3712: 0, 3840: 1}),    # short block-rows
    (128, 100, 200, 11, {3840: 0, 4864: 0, 5120: 1}),
    (64, 296, 1658, 14, {2048: 0, 3328: 0, 3456: 1, 8192: 1}), (64, 206, 3300, 26, {8192: 0}),            # unequal; long and alike
    (32, 592, 6600, 22, {2048: 1, 8192: 1}), (32, 592, 30000, 80, {2048: 0, 4096: 1}), (32, 592, 6600, 60, {2048: 0, 4096: 1}),
])
def test_fp32_tiles_by_one_wave(lists_of, block, brows, units, longest, widths):  # noqa: F811
    assert lists_of("f32", block, brows, units, longest, *widths)["one"] == [[one] for one in widths.values()]

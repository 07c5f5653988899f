"""The work lists of WCSR handles (host code, no GPU) at sizes that no matrix of a test reaches: a small C++ program calls the
list builder itself."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2604_17834_amd")
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"


@pytest.fixture(scope="module")
def lists_of(tmp_path_factory):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not found")
    exe = str(tmp_path_factory.mktemp("lists") / "lists")
    subprocess.check_call([HIPCC, "-x", "hip", "--offload-arch=gfx950", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "include"),
                           "-I", os.path.join(PKG, "csrc"), os.path.join(ROOT, "tests", "wcsr_lists_main.cpp"),
                           "-L", PKG, "-lasyncsparse", "-Wl,-rpath," + PKG, "-o", exe])

    def run(*args):
        out = subprocess.check_output([exe] + [str(a) for a in args], text=True)
        lists = {}
        for line in out.splitlines():
            name, *v = line.split()
            lists.setdefault(name, []).append([int(x) for x in v])
        return lists
    return run


def test_scratch_rows_that_pass_int32_stay_with_the_tiles(lists_of):
    for first in (0, 2**27 - 80):                 # scratch rows 16 * slot: the last one is 2^31 - 1
        got = lists_of("slots", first)
        assert len(got["split"]) == 32 and "tile" not in got
        rows = sorted(c[1] for c in got["chunk"] if c[2] < c[3])
        assert rows == sorted(set(rows)) and rows[0] == 16 * first and rows[-1] < 2**31
        assert all(s[1] >= 0 and s[1] + s[2] <= 16 * (first + 80) for s in got["split"])
    got = lists_of("slots", 2**27 - 60)             # the second window's scratch rows would pass 2^31 - 1
    assert len(got["split"]) == 16 and all(s[0] < 16 and s[1] >= 0 for s in got["split"])
    assert got["tile_split"] == [[1]] and all(t[0] == 1 for t in got["tile"])
    got = lists_of("slots", 2**27 - 1)
    assert "split" not in got and "chunk" not in got and got["tile_split"] == [[0], [1]]


@pytest.mark.parametrize("esize", [4, 2])
@pytest.mark.parametrize("m,k,task_cols,lengths", [
    (2000, 60000, 512, [0, 1, 63, 64, 65, 300, 511, 512, 513, 2000]),          # either side of the shortest grouped row and of a task
    (9000, 40000, 48, [900, 64, 70, 5] * 4 + [49, 63, 20, 3] * 4),             # rows longer than a task that are no members
    (20000, 30000, 512, [520, 70, 3]),                                         # more rows than 256 groups hold
    (400, 100000, 512, [40000] + [2000] * 99),                                 # rows dealt to several groups
])
def test_rows_in_groups_are_the_rows(lists_of, esize, m, k, task_cols, lengths):
    got = lists_of("groups", m, k, 0, task_cols, esize, *lengths)
    assert got["groups"][0][0] >= 256 and got["largest"][0][0] > 0
    assert got["scratch"][0][1] <= got["scratch"][0][0]
    tiles = got.get("tile", [])
    assert len(got["row"]) + len(tiles) == m and len(got["row"]) > m // 2
    assert all(diff == 0 and times == 1 for _, diff, times in got["row"]) and not any(times for _, times in tiles)


@pytest.mark.parametrize("m,k,lengths", [
    (100, 20000, [2000]),                 # few rows
    (4000, 1000000, [300, 600]),          # that share no columns
    (400, 20000, [100, 300, 600]),        # less than 64 entries a task
    (4000, 3000, [63, 20]),               # no row long enough
])
def test_no_groups_where_they_do_not_pay(lists_of, m, k, lengths):
    assert lists_of("groups", m, k, 0, 512, 4, *lengths)["groups"] == [[0]]


@pytest.mark.parametrize("esize", [4, 2])
@pytest.mark.parametrize("m,k,width,task_cols,lengths", [
    (20000, 100000, 0, 512, [70, 64, 300, 6, 5, 900, 7, 3]),                    # all columns
    (20000, 100000, 5000, 512, [70, 64, 300, 6, 5, 900, 7, 3]),                 # communities smaller than a range of columns
    (20000, 100000, 20000, 512, [70, 64, 300, 6, 5, 900, 7, 3]),                # larger than one
    (20000, 100000, 5000, 64, [70, 64, 300, 6, 5, 900, 7, 3]),                  # short tasks: sums no longer than those
    (4000, 100000, 100000, 512, [20000, 70, 70, 70, 70, 70, 70, 70]),
    (80000, 20000, 0, 512, [70, 66, 64]),                                       # eight or nine entries of every row in a range
])
def test_sums_are_short_and_tasks_even_whatever_the_columns(lists_of, esize, m, k, width, task_cols, lengths):
    got = lists_of("groups", m, k, width, task_cols, esize, *lengths)
    (largest, entries), (groups,) = got["largest"][0], got["groups"][0]
    assert groups >= 256 and got["terms"][0][0] <= min(160, task_cols)
    assert largest * 8 * groups <= 1.25 * entries + 16 * 8 * groups
    assert got["scratch"][0][1] <= got["scratch"][0][0]
    assert all(diff == 0 and times == 1 for _, diff, times in got["row"])


@pytest.mark.parametrize("m,k,width,near", [
    (40000, 20000, 0, True),         # 131 072 consecutive ones of 5.1 million entries meet in 20 000 columns
    (40000, 1000000, 0, False),
    (40000, 1000000, 5000, False),   # communities, but neighbours are in different ones
    (35000, 20000, 0, False),        # not as many entries
])
def test_columns_that_near_rows_meet_in(lists_of, m, k, width, near):
    got = lists_of("groups", m, k, width, 512, 4, 300, 64, 20)
    assert got["groups"][0][0] >= 256
    assert 10000 < got["near"][0][0] <= k if near else got["near"] == [[0]]


@pytest.mark.parametrize("task_cols,hubs,many", [
    (512, [90000, 20000, 400], 1),   # a row of more than 512 pieces among short ones
    (512, [8000, 7000, 400], 0),
    (64, [60000, 20000, 40000], 2),
])
def test_rows_of_many_pieces_come_first(lists_of, task_cols, hubs, many):
    lengths = [n for hub in hubs for n in [hub] + [300] * 999]
    got = lists_of("groups", 3000, 100000, 0, task_cols, 4, *lengths)
    n, fewest, most = got["many"][0]
    assert got["groups"][0][0] >= 256 and n == many and fewest > 512 >= most
    assert all(diff == 0 and times == 1 for _, diff, times in got["row"])


@pytest.mark.parametrize("length,many", [(3300, False), (6000, True)])   # 32 and 48 pieces of a row; 7 and 12 chunks without groups
def test_sums_count_the_pieces_that_they_add(lists_of, length, many):
    got = lists_of("groups", 400, 100000, 0, 512, 4, length)
    assert got["groups"][0][0] >= 256 and got["sums"] == [[400 if many else 0, 400]]


def test_no_groups_of_short_pieces(lists_of):
    for task_cols, groups in ((32, False), (40, False), (48, True)):
        got = lists_of("groups", 9000, 40000, 0, task_cols, 4, 900, 64, 70, 5)
        assert (got["groups"][0][0] > 0) == groups


@pytest.mark.parametrize("m,k,height,task_cols,lengths", [
    (6000, 250000, 16, 40, [200]),                             # 94 times 64 rows, 0.05 entries of each 64 in a column
    (6000, 100000, 16, 40, [200]),
    (6400, 200000, 64, 32, [100, 400]),
    (44 * 16, 100000, 16, 512, [10000] + [2] * 15),            # 4.4 entries a column
    (64 * 16, 100000, 16, 512, [6000] + [2] * 15),
])
def test_no_dense_rows_where_64_of_them_do_not_meet(lists_of, m, k, height, task_cols, lengths):
    assert lists_of("dense", m, k, height, task_cols, *lengths)["dense"][0][0] == 0


@pytest.mark.parametrize("n,per_pass", [(46, 46), (64, 64), (65, 0), (89, 0), (92, 46), (127, 64), (130, 0), (141, 47), (150, 50)])
def test_dense_rows_are_taken_in_equal_passes(lists_of, n, per_pass):
    got = lists_of("dense", 16 * n, 100000, 16, 512, 10000, 300, *[2] * 14)
    if not per_pass:                                     # passes of 33 to 45 rows: 3.3 to 4.5 entries a column
        assert got["dense"][0][0] == 0
        return
    ranges, blocks, rows, table, taken = got["dense"][0]
    assert rows == n and taken == per_pass and 64 <= ranges <= min(256, blocks) and blocks == 391
    assert 10 * got["fewest"][0][0] >= 45 * 99900 and 36 * 4 * table <= 8 * 10000 * rows
    assert len(got["row"]) == 16 * n and all(diff == 0 and times == 1 for _, diff, times in got["row"])


@pytest.mark.parametrize("k,rows,shared,tenths,widths", [
    (300_000, 50, 9000, 60, {63: 0, 64: 0, 65: 0, 111: 0, 112: 1, 128: 1, 129: 0, 160: 0, 192: 0, 256: 0, 320: 1}),
    (600_000, 50, 9000, 60, {64: 0, 65: 1, 128: 1, 130: 0, 159: 0, 160: 1, 192: 1, 200: 0, 214: 1, 256: 1, 257: 0, 1000: 1}),
    (600_000, 50, 0, 60, {64: 0, 65: 1, 128: 1, 130: 1, 200: 1, 257: 1}),
    (600_000, 50, 0, 47, {65: 1, 128: 1, 130: 0, 160: 0, 192: 1, 200: 0, 257: 0}),
    (2_000_000, 50, 0, 60, {32: 0, 63: 0, 64: 1, 72: 1, 130: 1, 159: 1, 192: 1}),
    (300_000, 100, 0, 60, {112: 0, 128: 0, 130: 0, 192: 1}), (600_000, 100, 0, 60, {64: 0, 72: 1, 128: 1, 130: 0, 160: 0, 200: 0, 256: 1}),
])
def test_products_that_take_dense_rows_through_lds(lists_of, k, rows, shared, tenths, widths):
    assert lists_of("apply", k, rows, shared, tenths, *widths)["apply"] == [[taken] for taken in widths.values()]


@pytest.mark.parametrize("waves", [0, 5, 2**26 - 33, 2**26 - 32, 2**26 - 31, 2**26, 3 * 2**26])
@pytest.mark.parametrize("teams", [0, 8, 4096, 131072])
def test_a_launch_of_the_walk_by_rows_takes_fewer_than_2_to_the_32_threads(lists_of, waves, teams):
    got = lists_of("launches", waves, teams).get("launch", [])
    assert all(workgroups * 256 < 2**32 for _, _, workgroups in got)
    assert [first for first, _, _ in got] == [0, *(end for _, end, _ in got[:-1])][:len(got)]
    assert not got or got[-1][1] == waves
    assert len(got) == (1 if waves + teams else 0) if waves <= 2**26 - 32 - 4 * teams else len(got) >= 2
    assert sum(workgroups for _, _, workgroups in got) == teams + -(-waves // 4)


@pytest.mark.parametrize("height,tasks,columns", [
    (64, 469, {16: 1, 32: 1, 33: 2, 64: 2, 65: 2, 100: 2, 128: 2, 129: 4, 160: 4, 256: 4}),
    (64, 512, {80: 2}), (64, 513, {80: 4, 128: 4}), (64, 1024, {128: 4, 160: 2, 193: 4}), (64, 1025, {128: 2}), (64, 1365, {72: 2, 128: 2}), (64, 1366, {128: 4}),
    (64, 2389, {128: 2}), (64, 2390, {128: 4}), (64, 3200, {80: 4}),
    (64, 1875, {72: 4, 128: 4}), (64, 9375, {64: 2, 66: 4, 80: 4, 128: 4, 160: 2}),     # two waves for one: more rounds of them
    (32, 469, {32: 1, 64: 2, 80: 4, 128: 4}), (32, 20000, {80: 4, 160: 2, 200: 4}), (16, 20000, {16: 4, 160: 4}),
])
def test_columns_of_a_lane(lists_of, height, tasks, columns):
    assert lists_of("columns", height, tasks, *columns)["columns"] == [[c] for c in columns.values()]


@pytest.mark.parametrize("m,k,height,task_cols,lengths,dense", [
    (48 * 16, 100000, 16, 512, [10000, 300, 64, 65] + [2] * 12, True),      # nearly dense rows, and whole rows around the shortest
    (30 * 16, 100000, 16, 512, [10000, 1500] + [2] * 14, True),             # long rows that are not, beside them
    (20 * 16, 100000, 16, 512, [20000] + [2] * 15 + [9000] + [2] * 15, True),   # chunks of more and of less than 100 entries
    (700, 300000, 16, 512, [2000, 513, 512, 65, 64, 63, 1, 0], False),
    (700, 300000, 64, 100, [2000, 101, 100, 66, 65, 64, 1, 0], False),      # short tasks
    (64, 50000, 16, 512, [40, 3], False),                                   # nothing to share
])
def test_rows_and_chunks_that_workgroups_share(lists_of, m, k, height, task_cols, lengths, dense):
    got = lists_of("teams", m, k, height, task_cols, *lengths)
    (teams, wide, count, length), (least, of_dense, as_long) = got["teams"][0], got["least"][0]
    assert teams % 8 == 0 and wide % 8 == 0 and (count > 0) == dense and 0 <= count <= wide <= 2 * count and (length > 100) == dense
    assert (least >= 65 or teams == 0) and of_dense == 0 and as_long == 0 and got["moved"] == [[0]]
    assert len(got["row"]) == m and all(row[1:] == [0, 1, 0, 1] for row in got["row"])


@pytest.mark.parametrize("bf16,N,chunks,length,shared", [
    (0, 64, 100, 512, 0), (0, 65, 100, 128, 1), (0, 128, 0, 0, 0), (0, 128, 2500, 128, 1), (0, 128, 2501, 128, 0), (0, 128, 5000, 192, 1),
    (0, 128, 5001, 192, 0), (0, 129, 60000, 128, 1), (1, 128, 100, 512, 0), (1, 129, 100, 128, 1), (1, 160, 4500, 128, 0),
    (1, 160, 60000, 192, 1), (1, 161, 4500, 128, 1),
])
def test_chunks_of_nearly_dense_rows_that_workgroups_share(lists_of, bf16, N, chunks, length, shared):
    assert lists_of("share", bf16, N, chunks, length)["share"] == [[shared]]

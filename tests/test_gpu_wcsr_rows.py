"""WCSR products whose windows are walked entry by entry (rows that share few columns), and the tile kernels at widths and
alignments that do not allow 16-byte rows: edges of the lanes' column ranges, batches of 8 entries, chunks of long rows.

Tolerances as everywhere: fp32 1e-5 * S, bf16 1e-2 * S + 1e-5, S = |A| x |B| from the oracle."""
import numpy as np
import pytest

from paper_2604_17834_amd import binding as asp
from paper_2604_17834_amd import synth
from test_gpu_parity import check_against_oracle, gpu_spmm

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _rows_of_lengths(lengths, k, dtype, seed):
    """One row per length, distinct random columns; U(-1, 1) values."""
    rng = np.random.default_rng(seed)
    cols = [np.sort(rng.choice(k, n, replace=False)) for n in lengths]
    rp = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    v = rng.uniform(-1, 1, rp[-1]).astype(np.float32)
    v = synth.f32_to_bf16_bits(v) if dtype == "bf16" else v
    return synth.Csr(len(lengths), k, rp, np.concatenate(cols).astype(np.int32), v, dtype)


# around the batch of 8 entries, empty rows in front, between and behind, rows of 1 .. 5 chunks at task_cols = 32
LENGTHS = [0, 0, 1, 7, 8, 9, 0, 15, 16, 17, 31, 32, 33, 64, 65, 160, 0, 2, 3, 1, 1, 0, 24, 23] + [1] * 70 + [0] * 70 + [5, 0]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("N", [1, 2, 3, 4, 7, 8, 63, 64, 65, 100, 127, 129, 255, 257, 511, 513])
def test_rows_walked_entry_by_entry(dtype, N):
    a = _rows_of_lengths(LENGTHS, 5000, dtype, seed=N)
    B = synth.dense_normal(a.k, N, dtype, seed=1000 + N)
    C = gpu_spmm(a, "wcsr", 16, 8, B, task_cols=32, misalign=N % 2 == 1)
    check_against_oracle(a, B, C)
    assert not C[np.diff(a.row_ptr) == 0].any()


@pytest.mark.parametrize("N", [3, 64, 130, 257])
def test_chunks_of_long_rows_without_scratch_are_added_with_atomics(N):
    a = _rows_of_lengths(LENGTHS, 5000, "f32", seed=3)
    B = synth.dense_normal(a.k, N, "f32", seed=4)
    check_against_oracle(a, B, gpu_spmm(a, "wcsr", 16, 8, B, task_cols=32, reserve=False))


@pytest.mark.parametrize("dtype,b_row", [("f32", 16), ("f32", 64), ("bf16", 16), ("bf16", 32)])
@pytest.mark.parametrize("N", [64, 9])
def test_band_and_long_rows_in_one_matrix(dtype, b_row, N):
    # band windows go tile by tile, the long rows' windows entry by entry; enough tasks that they are dealt to the XCDs
    a = synth.banded_plus_dense_rows(9000, seed=5, n_dense_rows=24, dense_row_nnz=3000, dtype=dtype)
    B = synth.dense_normal(a.k, N, dtype, seed=6)
    h = asp.asp_create_from_csr("wcsr", dtype, b_row, 8, a.m, a.k, a.row_ptr, a.col_idx, a.values, task_cols=64)
    try:
        C = gpu_spmm(a, "wcsr", b_row, 8, B, handle=h)
        assert np.array_equal(C.view(np.uint8), gpu_spmm(a, "wcsr", b_row, 8, B, handle=h).view(np.uint8))
        check_against_oracle(a, B, C)
    finally:
        asp.asp_destroy(h)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("b_row", [16, 32, 64])
@pytest.mark.parametrize("N,misalign,reserve", [(5, False, True), (9, True, True), (61, False, True), (129, True, True),
                                                (67, True, False), (259, False, False), (64, True, False)])
def test_dense_windows_at_any_width_and_alignment(dtype, b_row, N, misalign, reserve):
    a = synth.random_csr(200, 300, 0.5, seed=N, dtype=dtype)
    B = synth.dense_normal(a.k, N, dtype, seed=7 + N)
    check_against_oracle(a, B, gpu_spmm(a, "wcsr", b_row, 8, B, task_cols=128, misalign=misalign, reserve=reserve))


@pytest.mark.parametrize("dtype,reserve", [("f32", True), ("bf16", True), ("f32", False)])
@pytest.mark.parametrize("N", [16, 32, 64, 100, 128, 256, 512])
def test_only_rows_that_store_a_column_see_its_values(dtype, reserve, N):
    # Inf and NaN in some rows of B; tasks that begin with empty rows and at entries that are no multiple of 8, chunks of
    # every length: a row is Inf or NaN exactly where the sum of its own products is
    rng = np.random.default_rng(N)
    lengths = rng.choice([0, 0, 0, 1, 1, 2, 3, 5], 6000)
    lengths[rng.integers(0, 6000, 60)] = rng.integers(33, 400, 60)
    a = _rows_of_lengths(list(lengths), 5000, dtype, seed=N)
    a.values[:] = a.values & 0x7FFF if dtype == "bf16" else np.abs(a.values)
    B = synth.dense_normal(a.k, N, dtype, seed=8)
    bad = rng.random(a.k)
    B[bad < 0.05] = 0x7F80 if dtype == "bf16" else np.inf
    B[bad > 0.99] = 0x7FC1 if dtype == "bf16" else np.nan
    C = synth.to_f64(gpu_spmm(a, "wcsr", 16, 8, B, task_cols=32, reserve=reserve), dtype)
    inf, nan = (bad < 0.05)[a.col_idx], (bad > 0.99)[a.col_idx]
    row = np.repeat(np.arange(a.m), np.diff(a.row_ptr))
    has_inf, has_nan = np.bincount(row[inf], minlength=a.m) > 0, np.bincount(row[nan], minlength=a.m) > 0
    assert (has_inf & ~has_nan).sum() > 100 and has_nan.sum() > 50
    assert np.isnan(C[has_nan]).all()
    assert np.isposinf(C[has_inf & ~has_nan]).all()
    assert np.isfinite(C[~has_inf & ~has_nan]).all()
    assert not C[np.diff(a.row_ptr) == 0].any()


@pytest.mark.parametrize("dtype,b_row,N", [
    ("f32", 16, 320), ("f32", 16, 384), ("f32", 16, 512),       # 64-, 128- and 256-wide tiles, several of each
    ("f32", 16, 456), ("f32", 16, 905), ("f32", 16, 1024),      # 256 wide, rows that end inside a cache line; B and C past 512 MB
    ("f32", 32, 300), ("f32", 64, 129), ("bf16", 16, 200), ("bf16", 32, 385), ("bf16", 64, 129), ("bf16", 16, 64),
])
@pytest.mark.parametrize("windows", [1500, 5003])
def test_several_column_tiles_of_a_task(dtype, b_row, N, windows):
    # lists that are dealt to the XCDs (up to 4096 tasks) and lists that are not; a ragged last window
    a = synth.banded_plus_dense_rows(windows * b_row - 5, seed=7, n_dense_rows=0, dense_row_nnz=0, half_band=4, dtype=dtype)
    rng = np.random.default_rng(N)
    cols = np.unique(np.r_[0:8, N - 8:N, rng.integers(0, N, 16)])
    g = torch.Generator(device="cuda").manual_seed(N)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    Bd = torch.randn((a.k, N), dtype=tdt, device="cuda", generator=g)
    Cd = torch.full((a.m, N), float("nan"), dtype=tdt, device="cuda")
    h = asp.asp_create_from_csr("wcsr", dtype, b_row, 8, a.m, a.k, a.row_ptr, a.col_idx, a.values)
    try:
        asp.asp_spmm(h, Bd.data_ptr(), Cd.data_ptr(), N, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
    finally:
        asp.asp_destroy(h)
    assert not bool(torch.isnan(Cd).any())       # every output written
    ct = torch.from_numpy(cols).cuda()
    bits = (lambda t: t.contiguous().view(torch.int16).cpu().numpy().view(np.uint16)) if dtype == "bf16" else \
        (lambda t: t.contiguous().cpu().numpy())
    check_against_oracle(a, bits(Bd[:, ct]), bits(Cd[:, ct]))


@pytest.mark.parametrize("dtype,N", [("f32", n) for n in (33, 63, 64, 65, 127, 129, 257)] + [("bf16", n) for n in (65, 127, 128, 129, 257)])
def test_long_rows_in_groups(dtype, N):
    # rows from one to 4000 entries, members of groups from 64 on, some of them dealt to several groups; Inf and NaN in some
    # rows of B reach the rows that store those columns only; the handle without scratch walks the same rows one by one
    rng = np.random.default_rng(N)
    lengths = np.concatenate([rng.integers(64, 4000, 300), rng.integers(0, 70, 3001)])
    rng.shuffle(lengths)
    a = _rows_of_lengths(list(lengths), 60000, dtype, seed=N)
    B = synth.dense_normal(a.k, N, dtype, seed=8)
    h = asp.asp_create_from_csr("wcsr", dtype, 16, 8, a.m, a.k, a.row_ptr, a.col_idx, a.values, task_cols=64)
    try:
        if dtype == "f32":
            check_against_oracle(a, B, gpu_spmm(a, "wcsr", 16, 8, B, handle=h, reserve=False))
        C = gpu_spmm(a, "wcsr", 16, 8, B, handle=h)
        check_against_oracle(a, B, C)
        assert np.array_equal(C.view(np.uint8), gpu_spmm(a, "wcsr", 16, 8, B, handle=h).view(np.uint8))
        assert not C[np.diff(a.row_ptr) == 0].any()
        bad = rng.integers(0, a.k, 3)
        B[bad[:2]] = 0x7F80 if dtype == "bf16" else np.inf
        B[bad[2]] = 0x7FC1 if dtype == "bf16" else np.nan
        C = synth.to_f64(gpu_spmm(a, "wcsr", 16, 8, B, handle=h), dtype)
    finally:
        asp.asp_destroy(h)
    row = np.repeat(np.arange(a.m), np.diff(a.row_ptr))
    touched = np.bincount(row[np.isin(a.col_idx, bad)], minlength=a.m) > 0
    assert touched.sum() > 20 and not np.isfinite(C[touched]).any() and np.isfinite(C[~touched]).all()


@pytest.mark.parametrize("dtype,b_row,N", [("f32", 16, 64), ("f32", 32, 100), ("f32", 64, 129), ("bf16", 32, 100), ("bf16", 64, 129)])
def test_long_rows_of_communities_in_groups(dtype, b_row, N):
    # every row's columns in one of 20 blocks: it leaves pieces in one or two of the eight ranges of columns only
    rng = np.random.default_rng(N)
    lengths = np.concatenate([rng.integers(64, 1500, 300), rng.integers(0, 70, 3001)])
    rng.shuffle(lengths)
    home = rng.integers(0, 20, len(lengths)) * 6000
    cols = [h + np.sort(rng.choice(6000, n, replace=False)) for h, n in zip(home, lengths)]
    rp = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    v = rng.uniform(-1, 1, rp[-1]).astype(np.float32)
    a = synth.Csr(len(lengths), 120000, rp, np.concatenate(cols).astype(np.int32), synth.f32_to_bf16_bits(v) if dtype == "bf16" else v, dtype)
    B = synth.dense_normal(a.k, N, dtype, seed=8)
    C = gpu_spmm(a, "wcsr", b_row, 8, B, task_cols=64)
    check_against_oracle(a, B, C)
    assert not C[np.diff(a.row_ptr) == 0].any()


@pytest.mark.parametrize("dtype,N", [("f32", 40), ("f32", 65), ("bf16", 100)])
def test_a_row_of_many_pieces_among_short_ones(dtype, N):
    lengths = np.full(1500, 200)
    lengths[[77, 901]] = 79000, 30000
    a = _rows_of_lengths(list(lengths), 80000, dtype, seed=N)
    B = synth.dense_normal(a.k, N, dtype, seed=9)
    check_against_oracle(a, B, gpu_spmm(a, "wcsr", 16, 8, B, task_cols=64))


@pytest.mark.parametrize("dtype,b_row", [("f32", 16), ("f32", 32), ("f32", 64), ("bf16", 16), ("bf16", 32), ("bf16", 64)])
def test_groups_under_capture_and_with_static_scratch(dtype, b_row):
    # a B beyond 4 MB and rows enough for groups: both entry points give the same bits, eagerly and replayed with eager work
    # between the replays
    rng = np.random.default_rng(b_row)
    lengths = np.concatenate([rng.integers(64, 900, 600), rng.integers(0, 20, 2000)])
    rng.shuffle(lengths)
    a = _rows_of_lengths(list(lengths), 24000, dtype, seed=b_row)
    N = 96
    tdt = torch.int16 if dtype == "bf16" else torch.float32
    Bs = [synth.dense_normal(a.k, N, dtype, seed=20 + r) for r in range(3)]
    dev = [torch.from_numpy(B.view(np.int16) if dtype == "bf16" else B).cuda() for B in Bs]
    Bd, Cd = dev[0].clone(), torch.empty((a.m, N), dtype=tdt, device="cuda")
    h = asp.asp_create_from_csr("wcsr", dtype, b_row, 8, a.m, a.k, a.row_ptr, a.col_idx, a.values, task_cols=256)
    try:
        asp.asp_reserve(h, N)
        calls = [lambda f=f: f(h, Bd.data_ptr(), Cd.data_ptr(), N, torch.cuda.current_stream().cuda_stream)
                 for f in (asp.asp_spmm, asp.asp_spmm_static_scratch)]

        def result(go):
            Cd.fill_(0x7FC1 if dtype == "bf16" else float("nan"))
            go()
            torch.cuda.synchronize()
            return Cd.cpu().numpy().view(np.uint16 if dtype == "bf16" else np.float32).copy()

        graphs = []
        for call in calls:
            call()
            torch.cuda.synchronize()
            graphs.append(torch.cuda.CUDAGraph())
            with torch.cuda.graph(graphs[-1]):
                call()
        for r in (1, 2, 0):
            Bd.copy_(dev[r])
            want = result(calls[0])
            check_against_oracle(a, Bs[r], want)
            for go in (graphs[0].replay, calls[1], graphs[1].replay, graphs[0].replay):
                assert np.array_equal(result(go).view(np.uint8), want.view(np.uint8))
    finally:
        torch.cuda.synchronize()
        asp.asp_destroy(h)

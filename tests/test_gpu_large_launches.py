"""Launches with 2^32 threads and more: HIP takes fewer along a dimension, so they are cut up or given larger tiles."""
import numpy as np
import pytest

from paper_2604_17834_amd import binding as asp
from paper_2604_17834_amd import synth
from test_gpu_large_offsets import _bits, _check, _device_normal, _poisoned

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _written(C, rows=1 << 16):
    """No poison is left in any row."""
    for r in range(0, C.shape[0], rows):
        part = C[r:r + rows]
        bad = part.view(torch.int16) == 0x7FC1 if C.dtype == torch.bfloat16 else torch.isnan(part)
        if bool(bad.any()):
            return False
    return True


def test_xt_strips_of_four_million_tokens():
    # 129 block-rows x 131070 token tiles x 256 threads
    m, k, N = 4100, 33, asp.ASP_MAX_N
    a = synth.block_sparse_bernoulli(m, k, 32, 32, 0.3, seed=910, dtype="bf16")
    print("case xt m", m, "k", k, "tokens", N, flush=True)
    X = _device_normal(N, k, "bf16", seed=911)
    Y = _poisoned(N, m, "bf16")
    h = asp.asp_create_from_csr("bcsr", "bf16", 32, 32, a.m, a.k, a.row_ptr, a.col_idx, a.values)
    try:
        asp.asp_spmm_xt(h, X.data_ptr(), Y.data_ptr(), N, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
    finally:
        asp.asp_destroy(h)
    step = (2**32 - 1) // (129 * 256) * 32             # tokens of the first launch
    tok = torch.from_numpy(np.r_[0:16, 1234567:1234583, step - 16:step + 16, N - 16:N]).cuda()
    _check(a, np.ascontiguousarray(_bits(X[tok]).T), np.ascontiguousarray(_bits(Y[tok]).T))
    assert _written(Y)


def _few_block_rows(m, k, b, N, dtype):
    """m rows of which 12 block-rows (at both ends and in the middle) are not empty, against the oracle."""
    part = synth.block_sparse_bernoulli(4 * b, k, b, b, 0.3, seed=912, dtype=dtype)
    first = [0, (m // 2) // b * b, m - (m % b) - 3 * b]
    lens = np.diff(part.row_ptr)
    row_ptr = np.zeros(m + 1, np.int32)
    rows = np.concatenate([np.arange(f, min(m, f + 4 * b)) for f in first])
    keep = np.concatenate([lens[:min(m, f + 4 * b) - f] for f in first])
    row_ptr[rows + 1] = keep
    np.cumsum(row_ptr, out=row_ptr, dtype=np.int32)
    take = np.concatenate([np.arange(part.row_ptr[min(m, f + 4 * b) - f]) for f in first])
    a = synth.Csr(m, k, row_ptr, part.col_idx[take], part.values[take], dtype)
    print("case rows", m, dtype, "b", b, "N", N, flush=True)
    B = _device_normal(k, N, dtype, seed=913)
    C = _poisoned(m, N, dtype)
    h = asp.asp_create_from_csr("bcsr", dtype, b, b, a.m, a.k, a.row_ptr, a.col_idx, a.values)
    try:
        asp.asp_spmm(h, B.data_ptr(), C.data_ptr(), N, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
    finally:
        asp.asp_destroy(h)
    assert _written(C, 1 << 26)
    sub = synth.Csr(len(rows), k, np.concatenate([[0], np.cumsum(keep)]).astype(np.int32), a.col_idx, a.values, dtype)
    _check(sub, _bits(B), _bits(C[torch.from_numpy(rows).cuda()]))
    assert sum(int((C[r:r + (1 << 26)] != 0).any(dim=1).sum()) for r in range(0, m, 1 << 26)) == int((keep > 0).sum())


@pytest.mark.parametrize("b,N", [(128, 1), (32, 9)])
def test_fp32_blocks_of_268_million_rows(b, N):
    _few_block_rows((1 << 28) + 5, 300, b, N, "f32")       # 32 x 32 tiles of eight waves: 2^32 threads from 2^28 rows on


def test_strips_of_537_million_rows():
    _few_block_rows((1 << 29) + 5, 300, 32, 1, "bf16")     # strips of 32 rows, four waves each: 2^32 threads from 2^29 rows on


def test_wcsr_seventeen_million_split_rows():
    # every row is longer than task_cols: one sum per row, 256 threads each
    m, per_row, k, N = (1 << 24) + 24, 9, 16 * 9 * 7, 1
    r = np.arange(m, dtype=np.int32)
    # row r of a window takes columns first(window) + r + 16 j: ascending, no two rows of a window share one
    col_idx = ((r // 16 % 7) * 144 + r % 16)[:, None] + 16 * np.arange(per_row, dtype=np.int32)[None, :]
    row_ptr = np.arange(m + 1, dtype=np.int32) * per_row
    values = np.random.default_rng(914).uniform(-1.0, 1.0, m * per_row).astype(np.float32)
    a = synth.Csr(m, k, row_ptr, col_idx.ravel(), values, "f32")
    print("case wcsr split rows", m, "nnz", m * per_row, flush=True)
    h = asp.asp_create_from_csr("wcsr", "f32", 16, 8, a.m, a.k, a.row_ptr, a.col_idx, a.values, task_cols=8)
    try:
        B = _device_normal(k, N, "f32", seed=915)
        C = _poisoned(m, N, "f32")
        asp.asp_reserve(h, N)
        asp.asp_spmm(h, B.data_ptr(), C.data_ptr(), N, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
    finally:
        asp.asp_destroy(h)
    _check(a, _bits(B), _bits(C))


def test_wcsr_seventeen_million_empty_windows_without_scratch():
    # 2^24 windows to clear before the atomics of the one that is split
    m, k, N = (1 << 28) + 5, 4000, 2
    row_ptr = np.zeros(m + 1, np.int32)
    row_ptr[m // 2 + 1:] = 2000
    row_ptr[m:] = 2003
    col_idx = np.r_[np.arange(0, 4000, 2), 5, 17, 3999].astype(np.int32)
    values = np.random.default_rng(916).uniform(-1.0, 1.0, 2003).astype(np.float32)
    a = synth.Csr(m, k, row_ptr, col_idx, values, "f32")
    print("case wcsr empty windows, rows", m, flush=True)
    B = _device_normal(k, N, "f32", seed=917)
    C = _poisoned(m, N, "f32")
    h = asp.asp_create_from_csr("wcsr", "f32", 16, 8, a.m, a.k, a.row_ptr, a.col_idx, a.values)
    try:
        asp.asp_spmm(h, B.data_ptr(), C.data_ptr(), N, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
    finally:
        asp.asp_destroy(h)
    assert _written(C, 1 << 26)
    sub = synth.Csr(2, k, np.array([0, 2000, 2003], np.int32), col_idx, values, "f32")
    _check(sub, _bits(B), _bits(C[[m // 2, m - 1]]))
    assert int((C != 0).any(dim=1).sum()) == 2

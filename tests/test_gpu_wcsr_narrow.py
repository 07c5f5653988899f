"""fp32 WCSR tiles at heights 32 and 64: the widths at which a wave takes 32, 64 or 128 columns, with split windows (scratch, and
atomics without it) and windows of one task, and columns that no row stores.

1e-5 * S, S = |A| x |B| from the oracle, as everywhere in fp32.  A slice of B's columns gives a slice of C, bit for bit."""
import numpy as np
import pytest
import torch

import oracle
from paper_2604_17834_amd import binding as asp
from paper_2604_17834_amd import synth

pytestmark = pytest.mark.gpu


def product(h, B, m):
    N = B.shape[1]
    Bd = torch.from_numpy(np.ascontiguousarray(B)).cuda()
    out = torch.full((m * N + 64,), float("nan"), device="cuda")
    asp.asp_spmm(h, Bd.data_ptr(), out.data_ptr(), N, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    assert np.isnan(got[m * N:]).all()
    return got[:m * N].reshape(m, N)


@pytest.mark.parametrize("height", [32, 64])
@pytest.mark.parametrize("m,half,task_cols,reserve", [(1000, 13, 0, True), (1000, 60, 24, True), (1000, 60, 24, False), (58_000, 3, 0, True)])
def test_widths(height, m, half, task_cols, reserve):
    a = synth.banded_plus_dense_rows(m, seed=half, half_band=half, n_dense_rows=0)
    widths = [1, 2, 3, 16, 31, 32, 33, 63, 64, 65, 100, 128, 129, 160, 192, 193] if m < 10000 else [33, 160]
    B = synth.dense_normal(a.k, max(widths), "f32", seed=m)
    stored = np.zeros(a.k, bool)
    stored[a.col_idx] = True
    B[~stored] = np.inf
    h = asp.asp_create_from_csr("wcsr", "f32", height, 8, a.m, a.k, a.row_ptr, a.col_idx, a.values, task_cols=task_cols)
    if reserve:
        asp.asp_reserve(h, max(widths))
    clean = np.where(np.isfinite(B), B, 0).astype(np.float32)
    whole = None
    for N in reversed(widths):
        got = product(h, B[:, :N], a.m)
        ref, S = oracle.spmm(a.m, a.k, a.row_ptr, a.col_idx, a.values, "f32", np.ascontiguousarray(clean[:, :N]))
        assert np.isfinite(got).all() and (np.abs(got - ref) <= 1e-5 * S).all(), N
        whole = got if whole is None else whole
        if reserve:
            assert np.array_equal(got.view(np.uint32), np.ascontiguousarray(whole[:, :N]).view(np.uint32)), N
    asp.asp_destroy(h)

"""WCSR tiles: the widths at which a wave takes 16 to 128 columns, with split windows (scratch, and in fp32 atomics without it) and
windows of one task.

fp32: 1e-5 * S, bf16: 1e-2 * S + 1e-5, S = |A| x |B| from the oracle, as everywhere.  In fp32 a slice of B's columns gives a slice of C, bit for bit."""
import numpy as np
import pytest
import torch

import oracle
from paper_2604_17834_amd import binding as asp
from paper_2604_17834_amd import synth

pytestmark = pytest.mark.gpu


def product(h, B, m, dtype):
    N = B.shape[1]
    Bd = torch.from_numpy(np.ascontiguousarray(B).view(np.int16 if dtype == "bf16" else np.float32)).cuda()
    out = (torch.full((m * N + 64,), float("nan"), device="cuda") if dtype == "f32" else
           torch.full((m * N + 64,), 0x7FC1, dtype=torch.int16, device="cuda"))
    asp.asp_spmm(h, Bd.data_ptr(), out.data_ptr(), N, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    got = got if dtype == "f32" else got.view(np.uint16)
    assert np.isnan(synth.to_f64(got[m * N:], dtype)).all()
    return got[:m * N].reshape(m, N)


@pytest.mark.parametrize("dtype,m,half,task_cols,reserve", [
    (dtype, *shape) for dtype in ("f32", "bf16") for shape in ((1000, 13, 0, True), (1000, 60, 24, True), (1000, 60, 24, False), (58_000, 3, 0, True))
    if dtype == "f32" or shape[-1]])                                        # (bf16 needs scratch for split windows)
@pytest.mark.parametrize("height", [16, 32, 64])
def test_widths(dtype, height, m, half, task_cols, reserve):
    a = synth.banded_plus_dense_rows(m, seed=half, half_band=half, n_dense_rows=0)
    values = a.values if dtype == "f32" else synth.f32_to_bf16_bits(a.values)
    widths = [1, 2, 3, 8, 15, 16, 17, 31, 32, 33, 63, 64, 65, 100, 128, 129, 160, 192, 193] if m < 10000 else [33, 160]
    B = synth.dense_normal(a.k, max(widths), dtype, seed=m)
    h = asp.asp_create_from_csr("wcsr", dtype, height, 8, a.m, a.k, a.row_ptr, a.col_idx, values, task_cols=task_cols)
    if reserve:
        asp.asp_reserve(h, max(widths))
    whole = None
    for N in reversed(widths):
        got = product(h, B[:, :N], a.m, dtype)
        ref, S = oracle.spmm(a.m, a.k, a.row_ptr, a.col_idx, values, dtype, np.ascontiguousarray(B[:, :N]))
        bound = 1e-5 * S if dtype == "f32" else 1e-2 * S + 1e-5
        value = synth.to_f64(got, dtype)
        assert np.isfinite(value).all() and (np.abs(value - ref) <= bound).all(), N
        whole = got if whole is None else whole
        if reserve and dtype == "f32":
            assert np.array_equal(got.view(np.uint32), np.ascontiguousarray(whole[:, :N]).view(np.uint32)), N
    asp.asp_destroy(h)

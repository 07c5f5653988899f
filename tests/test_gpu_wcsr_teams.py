"""WCSR rows and chunks that a workgroup's four waves share: lengths around the shortest such row, the quarters' batches and
task_cols, in every width class, with scratch and (fp32) without.

fp32: 1e-5 * S, bf16: 1e-2 * S + 1e-5, S = |A| x |B| from the oracle, as everywhere.  Columns that a row does not store hold Inf."""
import numpy as np
import pytest
import torch

import oracle
from paper_2604_17834_amd import binding as asp
from paper_2604_17834_amd import synth

pytestmark = pytest.mark.gpu

LENGTHS = [64, 65, 66, 0, 1, 80, 127, 128, 129, 191, 255, 257, 0, 400, 511, 512, 513, 514, 700, 1024, 1025, 2000, 3, 96]


def matrix(dtype):
    rng = np.random.default_rng(5)
    k, stored = 60000, 59900                     # the last columns are stored by no row
    cols = [np.sort(rng.choice(stored, n, replace=False)) for n in LENGTHS for _ in range(2)]
    row_ptr = np.r_[0, np.cumsum([len(c) for c in cols])].astype(np.int32)
    values = rng.uniform(-1, 1, row_ptr[-1]).astype(np.float32)
    return len(cols), k, row_ptr, np.concatenate(cols).astype(np.int32), synth.f32_to_bf16_bits(values) if dtype == "bf16" else values


@pytest.mark.parametrize("dtype,reserve", [("f32", True), ("f32", False), ("bf16", True)])   # (bf16 needs scratch for split windows)
@pytest.mark.parametrize("height", [16, 64])
@pytest.mark.parametrize("N", [1, 7, 16, 17, 33, 64, 65, 100, 128, 130, 260])
def test_team_rows(dtype, reserve, height, N):
    m, k, row_ptr, col_idx, values = matrix(dtype)
    B = synth.dense_normal(k, N, dtype, seed=N)
    Bx = B.copy()
    Bx[59900:] = 0x7F80 if dtype == "bf16" else np.inf
    Bd = torch.from_numpy(Bx.view(np.int16) if dtype == "bf16" else Bx).cuda()
    Cd = torch.full((m * N + 64,), 0x7FC1 if dtype == "bf16" else float("nan"), dtype=torch.int16 if dtype == "bf16" else torch.float32, device="cuda")
    h = asp.asp_create_from_csr("wcsr", dtype, height, 8, m, k, row_ptr, col_idx, values)
    if reserve:
        asp.asp_reserve(h, N)
    asp.asp_spmm(h, Bd.data_ptr(), Cd.data_ptr(), N, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    asp.asp_destroy(h)
    got = Cd.cpu().numpy()
    got = synth.to_f64(got.view(np.uint16), "bf16") if dtype == "bf16" else got.astype(np.float64)
    assert np.isnan(got[m * N:]).all()
    got = got[:m * N].reshape(m, N)
    ref, S = oracle.spmm(m, k, row_ptr, col_idx, values, dtype, B)
    bound = 1e-2 * S + 1e-5 if dtype == "bf16" else 1e-5 * S
    assert np.isfinite(got).all() and (np.abs(got - ref) <= bound).all()
    assert not got[np.diff(row_ptr) == 0].any()

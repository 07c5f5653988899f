"""Nearly dense rows of a WCSR matrix in fp32 that are walked over columns of B in LDS: more than the 64 rows of one workgroup (a
few, which stay with their chunks, and enough for a second one), an odd width, columns that no row stores, rows that are empty in whole blocks of columns or full in some, beside shorter rows.

1e-5 * S, S = |A| x |B| from the oracle, as everywhere in fp32; and, from the 64-bit result, no further than by chunks."""
import numpy as np
import pytest
import torch

import oracle
from paper_2604_17834_amd import binding as asp
from paper_2604_17834_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_dense,k,N,height", [(64, 530_001, 64, 16), (70, 300_007, 131, 16), (112, 300_007, 131, 16), (48, 530_001, 65, 64)])
def test_dense_rows(n_dense, k, N, height):
    rng = np.random.default_rng(n_dense + N)
    m, stored = 16 * (n_dense + 4), k - 100
    cols = []
    for r in range(m):
        if r % 16 == 3 and r // 16 < n_dense:
            c = rng.choice(stored, stored // 9, replace=False)
            if r < 64:                                            # nothing in some blocks of 256 columns, all of others
                c = np.r_[c[(c < 2560) | (c >= 5120)], np.arange(7680, 8448), np.arange(10240, 10300)]
            cols.append(np.unique(c))
        else:
            cols.append(np.unique(rng.integers(0, stored, [3, 0, 40, 700][r % 4] if r % 37 == 0 else 2)))
    row_ptr = np.r_[0, np.cumsum([len(c) for c in cols])].astype(np.int32)
    col_idx = np.concatenate(cols).astype(np.int32)
    values = rng.uniform(-1, 1, row_ptr[-1]).astype(np.float32)
    B = synth.dense_normal(k, N, "f32", seed=N)
    Bx = B.copy()
    Bx[stored:] = np.inf
    Bd = torch.from_numpy(Bx).cuda()
    out = torch.full((m * N + 64,), float("nan"), device="cuda")
    h = asp.asp_create_from_csr("wcsr", "f32", height, 8, m, k, row_ptr, col_idx, values)
    asp.asp_reserve(h, N)
    results = []
    for _ in range(2):
        out[:m * N] = float("nan")
        asp.asp_spmm(h, Bd.data_ptr(), out.data_ptr(), N, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        results.append(out.cpu().numpy())
    asp.asp_destroy(h)
    assert np.array_equal(results[0].view(np.uint32), results[1].view(np.uint32))
    assert np.isnan(results[0][m * N:]).all()
    got = results[0][:m * N].reshape(m, N).astype(np.float64)
    ref, S = oracle.spmm(m, k, row_ptr, col_idx, values, "f32", B)
    assert np.isfinite(got).all() and (np.abs(got - ref) <= 1e-5 * S).all()
    dense = np.diff(row_ptr) > 10000
    assert np.linalg.norm((got - ref)[dense]) <= 3e-7 * np.linalg.norm(ref[dense])

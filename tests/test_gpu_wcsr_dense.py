"""Nearly dense rows of a WCSR matrix in fp32, walked over columns of B in LDS or, where that is not faster, in chunks: the rows of one
workgroup and of two, odd widths, columns that no row stores, rows that are empty in whole blocks of columns or full in some, beside
shorter rows.

1e-5 * S, S = |A| x |B| from the oracle, as everywhere in fp32; and, from the 64-bit result, no further than by chunks."""
import numpy as np
import pytest
import torch

import oracle
from paper_2604_17834_amd import binding as asp
from paper_2604_17834_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_dense,k,N,height", [(64, 530_001, 64, 16), (70, 300_007, 131, 16), (64, 920_001, 64, 16),
                                                  (112, 331_001, 127, 16), (48, 500_001, 191, 16), (48, 530_001, 65, 64)])
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


def test_whole_rows_do_not_depend_on_the_width():
    """Whole rows beside dense ones, either side of the length from which a workgroup shares a row (172 entries: all entries / 16384): a
    slice of B's columns gives a slice of C, bit for bit, at widths that walk the dense rows in chunks and at those that do not (65, 128)."""
    rng = np.random.default_rng(3)
    n_dense, k = 48, 530_001
    whole = [64, 65, 66, 80, 100, 128, 150, 170, 171, 172, 173, 174, 200, 300, 400, 511, 512]
    lengths = np.full(16 * n_dense, 2)
    lengths[3::16] = k // 9
    lengths[5::16] = (whole * 3)[:n_dense]
    cols = [np.unique(rng.choice(k, n, replace=False)) for n in lengths]
    row_ptr = np.r_[0, np.cumsum(lengths)].astype(np.int32)
    values = rng.uniform(-1, 1, row_ptr[-1]).astype(np.float32)
    m = len(lengths)
    h = asp.asp_create_from_csr("wcsr", "f32", 16, 8, m, k, row_ptr, np.concatenate(cols).astype(np.int32), values)
    asp.asp_reserve(h, 130)
    B = torch.from_numpy(synth.dense_normal(k, 130, "f32", seed=4)).cuda()
    got = {}
    for N in (17, 63, 65, 128, 130):
        C = torch.full((m, N), float("nan"), device="cuda")
        Bn = B[:, :N].contiguous()
        asp.asp_spmm(h, Bn.data_ptr(), C.data_ptr(), N, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        got[N] = C.cpu().numpy()[lengths <= 512]
    asp.asp_destroy(h)
    assert np.isfinite(got[130]).all()
    for N in (17, 63, 65, 128):
        assert np.array_equal(got[N].view(np.uint32), np.ascontiguousarray(got[130][:, :N]).view(np.uint32)), N

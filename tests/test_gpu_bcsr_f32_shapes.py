"""fp32 BCSR products at the edges of the wave tiles (32, 64 and 128 columns, with and without a split K loop), at any width and
alignment.  Tolerance as everywhere in fp32: 1e-5 * S, S = |A| x |B| from the oracle."""
import numpy as np
import pytest

from paper_2604_17834_amd import synth
from test_gpu_parity import check_against_oracle, gpu_spmm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("b", [32, 64, 128])
@pytest.mark.parametrize("m,k,misalign", [(520, 390, False), (515, 1111, True), (3, 5, True), (128, 20000, False)])
@pytest.mark.parametrize("N", [1, 2, 3, 4, 31, 33, 65, 130])
def test_narrow(b, m, k, misalign, N):
    a = synth.block_sparse_bernoulli(m, k, b, b, 0.5 if m > 3 else 0.0, seed=b + m + N, dtype="f32", std=1.0)
    B = synth.dense_normal(k, N, "f32", seed=N)
    check_against_oracle(a, B, gpu_spmm(a, "bcsr", b, b, B, misalign=misalign))


@pytest.mark.parametrize("b", [32, 64, 128])
@pytest.mark.parametrize("m,k,N,misalign", [
    (3000, 700, 513, False), (3000, 700, 1151, True),     # 32 x 64 tiles of four waves
    (5003, 331, 1279, False), (5003, 331, 1280, True),    # 64 x 128 of four waves
    (9003, 270, 3967, False), (9003, 270, 3968, True),    # 64 x 128 of two waves (32-row blocks: of one); empty block-rows
    (9003, 270, 7935, False), (9003, 270, 7936, True),    # 64 x 128, one wave each
    (520, 256, 161, True), (3000, 640, 513, False), (5003, 384, 1280, True), (9003, 256, 3967, False), (9003, 256, 7936, True),   # K % b == 0
])
def test_wide(b, m, k, N, misalign):
    a = synth.block_sparse_bernoulli(m, k, b, b, 0.7, seed=b + N, dtype="f32", std=1.0)
    B = synth.dense_normal(k, N, "f32", seed=N)
    C = gpu_spmm(a, "bcsr", b, b, B, misalign=misalign)
    assert not C[np.diff(a.row_ptr) == 0].any() and np.isfinite(C).all()   # (the poison is a NaN)
    check_against_oracle(a, B, C, np.r_[0:20, 120:136, N - 20:N])


def test_rows_past_k_do_not_meet_the_padding():
    a = synth.block_sparse_bernoulli(512, 1001, 64, 64, 0.5, seed=1, dtype="f32", std=1.0)
    B = synth.dense_normal(a.k, 40, "f32", seed=2)
    B[-1] = np.inf                       # only rows of A that store the last column see it
    C = gpu_spmm(a, "bcsr", 64, 64, B)
    has_last = np.array([a.row_ptr[i + 1] > a.row_ptr[i] and a.col_idx[a.row_ptr[i + 1] - 1] == a.k - 1 for i in range(a.m)])
    assert not np.isfinite(C[has_last]).any() and np.isfinite(C[~has_last]).all()

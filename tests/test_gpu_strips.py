"""asp_spmm on launches that run as strips of block-rows (K loop split over waves), at the edges of their tiles, any width and
alignment; and the register-staged kernel's last columns.

Tolerance as everywhere in bf16: 1e-2 * S + 1e-5, S = |A| x |B| from the oracle."""
import numpy as np
import pytest

from paper_2604_17834_amd import synth
from test_gpu_parity import check_against_oracle, gpu_spmm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("b", [32, 64, 128])
@pytest.mark.parametrize("m,k,misalign", [(1024, 2048, False), (1001, 1999, False), (515, 1111, True), (3, 5, True)])
@pytest.mark.parametrize("N", [1, 5, 7, 8, 31, 37, 64, 101, 128, 200, 333])
def test_strips(b, m, k, misalign, N):
    a = synth.block_sparse_bernoulli(m, k, b, b, 0.5 if m > 3 else 0.0, seed=b + m + N, dtype="bf16")
    B = synth.dense_normal(k, N, "bf16", seed=N)
    C = gpu_spmm(a, "bcsr", b, b, B, misalign=misalign)
    check_against_oracle(a, B, C)


@pytest.mark.parametrize("b", [32, 64, 128])
@pytest.mark.parametrize("m,k,N,sparsity", [
    (512, 20000, 320, 0.9), (128, 20000, 40, 0.2),  # few long block-rows, more blocks than one look-up of columns holds
    (6000, 1000, 520, 0.9), (6000, 1003, 523, 0.9),  # many short ones, empty ones among them
    (2000, 3000, 2050, 0.9), (2000, 3001, 9003, 0.9),
])
def test_strips_of_long_and_of_many_rows(b, m, k, N, sparsity):
    a = synth.block_sparse_bernoulli(m, k, b, b, sparsity, seed=b + m, dtype="bf16")
    B = synth.dense_normal(k, N, "bf16", seed=N)
    C = gpu_spmm(a, "bcsr", b, b, B)
    assert not C[np.diff(a.row_ptr) == 0].any()
    check_against_oracle(a, B, C, np.r_[0:24, N - 24:N])


@pytest.mark.parametrize("N", [40, 45])
def test_rows_past_k_do_not_meet_the_padding(N):
    # K is no multiple of the block: whatever lies behind the last row of B must not reach the product
    a = synth.block_sparse_bernoulli(512, 1000, 64, 64, 0.5, seed=N, dtype="bf16")
    B = synth.dense_normal(a.k, N, "bf16", seed=N)
    B[-1] = 0x7FC1                       # NaN in the last row: only rows of A that store its column see it
    C = gpu_spmm(a, "bcsr", 64, 64, B)
    has_last = np.zeros(a.m, bool)
    for i in range(a.m):
        cols = a.col_idx[a.row_ptr[i]:a.row_ptr[i + 1]]
        has_last[i] = len(cols) and cols[-1] == a.k - 1
    nan = (C & 0x7FFF) > 0x7F80
    assert nan[has_last].all() and not nan[~has_last].any()

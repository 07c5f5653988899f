"""asp_spmm_xt below the size of the 128 x 512 tiles: the strip kernel (K loop split over waves) at the edges of its token
tiles, any K, M and alignment, and the ring kernel on K-contiguous operands, also where the last K slice crosses K.

Tolerance as everywhere in bf16: 1e-2 * S + 1e-5, S = |A| x |B| from the oracle."""
import numpy as np
import pytest

from paper_2604_17834_amd import synth
from test_gpu_parity import check_against_oracle, gpu_spmm_xt

pytestmark = pytest.mark.gpu


def _check(a, X, Y, tokens=None):
    tok = np.arange(len(X)) if tokens is None else tokens
    assert not ((Y & 0x7F80) == 0x7F80).any()   # no element left unwritten (the poison is a NaN)
    check_against_oracle(a, np.ascontiguousarray(X[tok].T), np.ascontiguousarray(Y[tok].T))


@pytest.mark.parametrize("b", [32, 64, 128])
@pytest.mark.parametrize("m,k,misalign", [(1024, 2048, False), (1000, 1992, False), (1001, 999, False), (515, 1111, True),
                                          (3, 5, True)])
@pytest.mark.parametrize("N", [1, 31, 32, 33, 65, 200])
def test_strips(b, m, k, misalign, N):
    a = synth.block_sparse_bernoulli(m, k, b, b, 0.5 if m > 3 else 0.0, seed=b + m + N, dtype="bf16")
    X = synth.dense_normal(N, k, "bf16", seed=N)
    _check(a, X, gpu_spmm_xt(a, b, X, misalign=misalign))


@pytest.mark.parametrize("b", [32, 64, 128])
@pytest.mark.parametrize("m,k,N,sparsity", [
    (512, 20000, 300, 0.9),     # few long block-rows, more blocks than one look-up of columns holds
    (128, 20000, 40, 0.2),
    (6000, 1000, 700, 0.9),     # many short ones
])
def test_strips_of_long_and_of_many_rows(b, m, k, N, sparsity):
    a = synth.block_sparse_bernoulli(m, k, b, b, sparsity, seed=b + m, dtype="bf16")
    X = synth.dense_normal(N, k, "bf16", seed=N)
    _check(a, X, gpu_spmm_xt(a, b, X), np.r_[0:24, N - 24:N])


@pytest.mark.parametrize("b", [32, 64, 128])
@pytest.mark.parametrize("m,k,N,sparsity", [(4104, 1000, 1501, 0.9), (4104, 1000, 3000, 0.5), (4096, 1024, 5000, 0.9),
                                            (2048, 4096, 2048, 0.9), (8192, 520, 900, 0.5)])
def test_ring_kernel_on_k_contiguous_operands(b, m, k, N, sparsity):
    a = synth.block_sparse_bernoulli(m, k, b, b, sparsity, seed=b + N, dtype="bf16")
    X = synth.dense_normal(N, k, "bf16", seed=N)
    _check(a, X, gpu_spmm_xt(a, b, X), np.r_[0:24, 250:262, N - 24:N])


@pytest.mark.parametrize("b", [32, 64, 128])
@pytest.mark.parametrize("k,N", [(1000, 64), (1001, 64), (1000, 3000)])
def test_tokens_do_not_reach_each_other(b, k, N):
    # every other token is all NaN: the zero padding of the last block column must not meet its values
    a = synth.block_sparse_bernoulli(4096, k, b, b, 0.5, seed=b + N, dtype="bf16")
    X = synth.dense_normal(N, k, "bf16", seed=N)
    Xn = X.copy()
    Xn[1::2] = 0x7FC1
    assert np.array_equal(gpu_spmm_xt(a, b, Xn)[::2], gpu_spmm_xt(a, b, X)[::2])


@pytest.mark.parametrize("b", [64, 128])
@pytest.mark.parametrize("m,k,N,sparsity", [
    (12808, 1032, 33, 0.5), (12808, 1032, 64, 0.5), (8200, 1992, 65, 0.5),   # edges of a token tile; a last unit of 8 k
    (8200, 1992, 700, 0.5), (8200, 200, 500, 0.0), (8200, 384, 300, 0.0),    # 128-row strips; few units, the last of 8 k; whole ones
    (12808, 2056, 33, 0.5), (12808, 2056, 64, 0.5), (8200, 1992, 129, 0.5),  # edges of a token tile again, with work for these strips
])
def test_staged_strips(b, m, k, N, sparsity):
    a = synth.block_sparse_bernoulli(m, k, b, b, sparsity, seed=b + m + N, dtype="bf16")
    X = synth.dense_normal(N, k, "bf16", seed=N)
    Y = gpu_spmm_xt(a, b, X)
    _check(a, X, Y, np.r_[0:24, N - 24:N])
    X[1::2] = 0x7FC1   # NaN in every other token stays there, also where a block passes the last k
    assert np.array_equal(gpu_spmm_xt(a, b, X)[::2], Y[::2])

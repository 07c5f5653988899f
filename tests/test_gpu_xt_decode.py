"""asp_spmm_xt of up to 32 tokens: strips of 16 rows, around their tokens, rows that end inside a strip and block columns that end
past K, in 4 and 8 waves, and the launches beside them that keep the other strips.

Tolerance as everywhere in bf16: 1e-2 * S + 1e-5, S = |A| x |X| from the oracle.  Tokens behind Y stay as they are."""
import numpy as np
import pytest
import torch

from paper_2604_17834_amd import binding as asp
from paper_2604_17834_amd import synth
from test_gpu_parity import check_against_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("b", [32, 64, 128])
@pytest.mark.parametrize("m,k,sparsity", [(8, 8, 0.0), (1000, 3336, 0.7), (4096, 1032, 0.9), (6024, 520, 0.3), (600, 16384, 0.8),
                                          (5200, 6400, 0.5)])
@pytest.mark.parametrize("N", [1, 2, 15, 16, 17, 31, 32, 33])
def test_few_tokens(b, m, k, sparsity, N):
    a = synth.block_sparse_bernoulli(m, k, b, b, sparsity, seed=b + m + N, dtype="bf16")
    X = synth.dense_normal(N, k, "bf16", seed=N)
    Xd = torch.from_numpy(X.view(np.int16)).cuda()
    out = torch.full(((N + 2) * m,), 0x7FC1, dtype=torch.int16, device="cuda")
    h = asp.asp_create_from_csr("bcsr", "bf16", b, b, m, k, a.row_ptr, a.col_idx, a.values)
    asp.asp_spmm_xt(h, Xd.data_ptr(), out.data_ptr(), N, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    asp.asp_destroy(h)
    got = out.cpu().numpy().view(np.uint16).reshape(N + 2, m)
    assert (got[N:] == 0x7FC1).all()
    check_against_oracle(a, np.ascontiguousarray(X.T), np.ascontiguousarray(got[:N].T))


@pytest.mark.parametrize("b", [32, 64, 128])
def test_columns_past_k_do_not_meet_the_padding(b):
    # K ends inside a block: what lies behind a token's last element (here the next token) must not reach the product
    m, k, N = 256, 1000, 9
    a = synth.block_sparse_bernoulli(m, k, b, b, 0.3, seed=b, dtype="bf16")
    X = synth.dense_normal(N, k, "bf16", seed=N)
    X[1::2] = 0x7F80
    Xd = torch.from_numpy(X.view(np.int16)).cuda()
    Y = torch.full((N, m), 0x7FC1, dtype=torch.int16, device="cuda")
    h = asp.asp_create_from_csr("bcsr", "bf16", b, b, m, k, a.row_ptr, a.col_idx, a.values)
    asp.asp_spmm_xt(h, Xd.data_ptr(), Y.data_ptr(), N, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    asp.asp_destroy(h)
    got = Y.cpu().numpy().view(np.uint16)[::2]
    check_against_oracle(a, np.ascontiguousarray(X[::2].T), np.ascontiguousarray(got.T))

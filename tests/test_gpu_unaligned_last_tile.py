"""bf16 products whose rows are not 16-byte aligned: the last column tile of the strips moves left, and the last 8 columns of the
register-staged kernel, so that columns are shared with a neighbour, for widths around the tiles' and a last block column that
reaches past K.

Tolerance as everywhere in bf16: 1e-2 * S + 1e-5, S = |A| x |B| from the oracle.  The columns behind C stay as they are."""
import numpy as np
import pytest
import torch

from paper_2604_17834_amd import binding as asp
from paper_2604_17834_amd import synth
from test_gpu_parity import check_against_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("b", [32, 64, 128])
@pytest.mark.parametrize("m,k", [(300, 1000), (9000, 131)])   # strips; the register-staged kernel from some hundred columns on
@pytest.mark.parametrize("N", [1, 7, 9, 15, 17, 31, 33, 63, 65, 127, 129, 1021, 2049])
def test_last_tile(b, m, k, N):
    product(b, m, k, N)


@pytest.mark.parametrize("b", [32, 64, 128])
@pytest.mark.parametrize("N", [1, 7, 9, 15, 63, 65, 71, 127, 129, 191, 255, 257, 385])
def test_tall(b, N):
    product(b, 150_001, 131, N)   # register-staged: tiles of 64, 128 and 256 columns, some of them mostly past N


def product(b, m, k, N):
    a = synth.block_sparse_bernoulli(m, k, b, b, 0.4, seed=b + m + N, dtype="bf16")
    B = synth.dense_normal(k, N, "bf16", seed=N)
    Bd = torch.from_numpy(B.view(np.int16)).cuda()
    out = torch.full((m * N + 64,), 0x7FC1, dtype=torch.int16, device="cuda")
    h = asp.asp_create_from_csr("bcsr", "bf16", b, b, m, k, a.row_ptr, a.col_idx, a.values)
    asp.asp_spmm(h, Bd.data_ptr(), out.data_ptr(), N, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    asp.asp_destroy(h)
    got = out.cpu().numpy().view(np.uint16)
    assert (got[m * N:] == 0x7FC1).all()
    C = got[:m * N].reshape(m, N)
    assert not ((C & 0x7F80) == 0x7F80).any()
    check_against_oracle(a, B, C, np.unique(np.r_[0:min(N, 8), max(0, N - 72):N]))

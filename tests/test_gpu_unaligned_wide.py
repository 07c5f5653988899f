"""bf16 BCSR products whose rows are not 16-byte aligned, wide enough for the register-staged kernel (128- and 256-wide tiles):
tiles' edges and the last columns.  Tolerance as everywhere in bf16: 1e-2 * S + 1e-5, S = |A| x |B| from the oracle."""
import numpy as np
import pytest

from paper_2604_17834_amd import synth
from test_gpu_parity import check_against_oracle, gpu_spmm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("b", [32, 64, 128])
@pytest.mark.parametrize("m,k,N,misalign", [(5003, 331, 8001, False), (5003, 331, 8007, False), (9001, 270, 9000, True),
                                            (700, 1999, 8065, False)])
def test_unaligned_rows(b, m, k, N, misalign):
    a = synth.block_sparse_bernoulli(m, k, b, b, 0.5, seed=b + N, dtype="bf16")
    B = synth.dense_normal(k, N, "bf16", seed=N)
    C = gpu_spmm(a, "bcsr", b, b, B, misalign=misalign)
    assert not ((C & 0x7F80) == 0x7F80).any()   # no element left unwritten (the poison is a NaN)
    check_against_oracle(a, B, C, np.r_[0:16, 120:136, N - 16:N])

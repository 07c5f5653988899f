"""Launches with 2^32 threads and more: HIP takes fewer along a dimension, so they are cut up or given larger tiles."""
import numpy as np
import pytest

from paper_2604_17834_amd import binding as asp
from paper_2604_17834_amd import synth
from test_gpu_large_offsets import _bits, _check, _device_normal, _poisoned

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _written(C, rows=1 << 16):
    """No poison is left in any row."""
    for r in range(0, C.shape[0], rows):
        part = C[r:r + rows]
        bad = part.view(torch.int16) == 0x7FC1 if C.dtype == torch.bfloat16 else torch.isnan(part)
        if bool(bad.any()):
            return False
    return True


def test_xt_strips_of_four_million_tokens():
    # 129 block-rows x 131070 token tiles x 256 threads
    m, k, N = 4100, 33, asp.ASP_MAX_N
    a = synth.block_sparse_bernoulli(m, k, 32, 32, 0.3, seed=910, dtype="bf16")
    print("case xt m", m, "k", k, "tokens", N, flush=True)
    X = _device_normal(N, k, "bf16", seed=911)
    Y = _poisoned(N, m, "bf16")
    h = asp.asp_create_from_csr("bcsr", "bf16", 32, 32, a.m, a.k, a.row_ptr, a.col_idx, a.values)
    try:
        asp.asp_spmm_xt(h, X.data_ptr(), Y.data_ptr(), N, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
    finally:
        asp.asp_destroy(h)
    step = (2**32 - 1) // (129 * 256) * 32             # tokens of the first launch
    tok = torch.from_numpy(np.r_[0:16, 1234567:1234583, step - 16:step + 16, N - 16:N]).cuda()
    _check(a, np.ascontiguousarray(_bits(X[tok]).T), np.ascontiguousarray(_bits(Y[tok]).T))
    assert _written(Y)

"""bf16 BCSR products that reach the kernel shapes which the dispatch rules choose beyond those of test_gpu_strips.py and
test_gpu_xt_short.py (on 256 compute units): strips of every wave tile and K split, with and without 16-byte rows, and
the row-major ring kernel at every tile size, with K a multiple of the block and not.

Tolerance as everywhere in bf16: 1e-2 * S + 1e-5, S = |A| x |B| from the oracle."""
import dataclasses
import functools

import numpy as np
import pytest

from paper_2604_17834_amd import synth
from test_gpu_parity import check_against_oracle, gpu_spmm, gpu_spmm_xt

pytestmark = pytest.mark.gpu


def _edges(N):
    return np.arange(N) if N <= 96 else np.r_[0:40, N // 2 - 8:N // 2 + 8, N - 40:N]


# (rows x columns of a wave tile in units of 32) x waves that split the K loop
@pytest.mark.parametrize("b,m,k,N,sparsity", [
    (32, 512, 500, 64, 0.8), (32, 513, 501, 129, 0.95),        # 1 x 1, 4 waves
    (64, 512, 1000, 64, 0.95), (128, 512, 500, 16, 0.8),
    (32, 512, 500, 2000, 0.8), (32, 513, 501, 1501, 0.9),      # 1 x 2, 4
    (32, 1000, 500, 1496, 0.8),                                # 1 x 4, 2
    (64, 512, 1000, 2000, 0.5), (64, 513, 1001, 1001, 0.5),    # 2 x 2, 8
    (128, 512, 1000, 2000, 0.5), (128, 1001, 9001, 1001, 0.95),
    (64, 2048, 500, 296, 0.9), (128, 2048, 500, 200, 0.9),     # 2 x 2, 4
])
def test_row_major_strips(b, m, k, N, sparsity):
    a = synth.block_sparse_bernoulli(m, k, b, b, sparsity, seed=1, dtype="bf16")
    B = synth.dense_normal(k, N, "bf16", seed=N)
    C = gpu_spmm(a, "bcsr", b, b, B)
    assert not ((C & 0x7F80) == 0x7F80).any()   # no element left unwritten (the poison is a NaN)
    check_against_oracle(a, B, C, _edges(N))


@pytest.mark.parametrize("b,m,k,N,sparsity", [
    (32, 512, 2000, 1496, 0.9), (32, 513, 501, 1001, 0.95),       # 1 x 1, 4 waves
    (64, 512, 1000, 696, 0.8), (64, 1000, 500, 256, 0.95),        # 2 x 1, 8
    (128, 512, 2000, 512, 0.95), (128, 513, 501, 401, 0.95),
    (64, 1000, 1000, 696, 0.8), (64, 1000, 500, 696, 0.95),       # 2 x 1, 4
    (128, 512, 1000, 1496, 0.8), (128, 513, 501, 1001, 0.95),
    (64, 2048, 1000, 2000, 0.8), (64, 2048, 500, 1496, 0.95),     # 2 x 2, 4
    (128, 1536, 1000, 2000, 0.8), (128, 1536, 500, 2000, 0.95),
    (128, 1536, 2000, 3000, 0.5), (128, 513, 2001, 3001, 0.5),    # 4 x 2, 4
    (128, 8000, 2000, 3000, 0.5),                                 # the ring kernel's 128 x 256 tiles
])
def test_k_contiguous(b, m, k, N, sparsity):
    a = synth.block_sparse_bernoulli(m, k, b, b, sparsity, seed=1, dtype="bf16")
    X = synth.dense_normal(N, k, "bf16", seed=N)
    Y = gpu_spmm_xt(a, b, X)
    assert not ((Y & 0x7F80) == 0x7F80).any()
    tok = _edges(N)
    check_against_oracle(a, np.ascontiguousarray(X[tok].T), np.ascontiguousarray(Y[tok].T))


# more than 64 MB of B: no strips; the number of block-rows sets the tile width
@pytest.mark.parametrize("mask", ["bernoulli", "geometric"])
@pytest.mark.parametrize("k", [4096, 4104])
@pytest.mark.parametrize("rows,bn", [(10, 256), (5, 128), (3, 64)])
@pytest.mark.parametrize("b", [32, 64, 128])
def test_row_major_ring(b, rows, bn, k, mask):
    gen = synth.block_sparse_bernoulli if mask == "bernoulli" else synth.block_sparse_geometric
    N = 8200
    a = gen(rows * b - 8, k, b, b, 0.5 if mask == "bernoulli" else 0.8, seed=rows + b, dtype="bf16")
    B = synth.dense_normal(k, N, "bf16", seed=rows)
    C = gpu_spmm(a, "bcsr", b, b, B)
    assert not C[np.diff(a.row_ptr) == 0].any() and not ((C & 0x7F80) == 0x7F80).any()
    check_against_oracle(a, B, C, np.r_[0:24, 4000:4136, N - 72:N])


@functools.lru_cache(maxsize=1)
def _many_rows(b, rows, sparsity, k):
    return synth.block_sparse_geometric(rows * b - 8, k, b, b, sparsity, seed=rows + b, dtype="bf16")


# one column tile and more block-rows than resident workgroups: requests run on into the next tiles, empty ones among them
@pytest.mark.parametrize("b,rows,sparsity", [(32, 6000, 0.7), (64, 3000, 0.75), (128, 1500, 0.75)])
@pytest.mark.parametrize("k", [1000, 1024])
@pytest.mark.parametrize("N", [64, 128, 256, 248])
def test_row_major_ring_over_many_tiles(b, rows, sparsity, k, N):
    a = _many_rows(b, rows, sparsity, k)
    B = synth.dense_normal(k, N, "bf16", seed=N)
    C = gpu_spmm(a, "bcsr", b, b, B)
    assert not C[np.diff(a.row_ptr) == 0].any() and not ((C & 0x7F80) == 0x7F80).any()
    check_against_oracle(a, B, C, np.r_[0:8, N // 2:N // 2 + 8, N - 8:N])


# groups of one, two and four N-tiles, in 16, 32 and 64 lists: (block, m, k, N) with more tiles than the chip holds and fewer
@pytest.mark.parametrize("b,m,k,N", [
    (32, 2048, 5000, 2504), (32, 2100, 600, 2056),     # one; four, whose slab fits L2
    (64, 2048, 3000, 2504), (64, 8192, 500, 2056),
    (128, 2048, 3000, 4104), (128, 10240, 500, 2056),  # one round of tiles, and more
    (64, 16500, 512, 4616), (128, 16512, 256, 8704), (128, 16400, 256, 16384),   # 128x512 tiles, more than 128 rows of them
])
@pytest.mark.parametrize("xt", [False, True])
def test_groups_of_column_tiles(b, m, k, N, xt):
    m -= m % 8 if xt else 0
    a = synth.block_sparse_bernoulli(m, k, b, b, 0.75, seed=3, dtype="bf16")
    e = _edges(N)
    if xt:
        X = synth.dense_normal(N, k, "bf16", seed=N)
        Y = gpu_spmm_xt(a, b, X)
        assert not ((Y & 0x7F80) == 0x7F80).any()
        check_against_oracle(a, np.ascontiguousarray(X[e].T), np.ascontiguousarray(Y[e].T))
    else:
        B = synth.dense_normal(k, N, "bf16", seed=N)
        C = gpu_spmm(a, "bcsr", b, b, B)
        assert not ((C & 0x7F80) == 0x7F80).any()
        check_against_oracle(a, B, C, e)


# 128x512 tiles whose number does not divide among the XCDs, with empty block-rows: (block, m, k, N); 4, 10, 13, 21, 9, 15 and 26
# N-tiles, shared whole, after one or two rounds of whole tiles, in two or three to an XCD
@pytest.mark.parametrize("b,m,k,N", [
    (128, 17000, 512, 1544), (64, 8200, 512, 4616), (32, 4160, 256, 6168), (128, 3200, 640, 10248), (128, 5004, 1000, 4104),
    (64, 3400, 300, 7680), (32, 2048, 96, 13000),
])
@pytest.mark.parametrize("xt", [False, True])
def test_shared_column_tiles(b, m, k, N, xt):
    test_groups_of_column_tiles(b, m, k, N, xt)


# register-staged tiles (operands without 16-byte rows, block-rows short for the work: no strips): as many tiles as the chip holds, as
# stored; more, longest block-rows first; empty block-rows at the end, as stored where one XCD would get half of all tiles,
# longest first where that is less
@pytest.mark.parametrize("b,m,k,N,sparsity,empty", [
    (32, 4000, 1000, 1021, 0.5, 0), (64, 3900, 320, 1021, 0.1, 0), (64, 3000, 333, 2001, 0.75, 0), (128, 5000, 400, 4097, 0.75, 0),
    (32, 40000, 512, 127, 0.5, 0), (32, 30720, 1280, 127, 0.0, 46080), (32, 32000, 512, 255, 0.5, 96000),
])
def test_register_staged_tile_order(b, m, k, N, sparsity, empty):
    a = synth.block_sparse_bernoulli(m, k, b, b, sparsity, seed=9, dtype="bf16")
    a = dataclasses.replace(a, m=m + empty, row_ptr=np.r_[a.row_ptr, np.full(empty, a.row_ptr[-1], a.row_ptr.dtype)])
    B = synth.dense_normal(k, N, "bf16", seed=N)
    C = gpu_spmm(a, "bcsr", b, b, B)
    assert not C[np.diff(a.row_ptr) == 0].any() and not ((C & 0x7F80) == 0x7F80).any()
    check_against_oracle(a, B, C, _edges(N))

"""SparseLinear without a stream argument: the product goes to torch's current stream, also while that one is captured."""
import numpy as np
import pytest
import torch

from paper_2604_17834_amd import synth
from paper_2604_17834_amd.binding import AspError
from paper_2604_17834_amd.linear import SparseLinear

pytestmark = pytest.mark.gpu


def test_current_stream_is_captured():
    w = synth.block_sparse_bernoulli(256, 384, 64, 64, 0.5, seed=1, dtype="bf16")
    layer = SparseLinear(256, 384, w.row_ptr, w.col_idx, w.values, block=64)
    draw = lambda seed: torch.from_numpy(synth.dense_normal(7, 384, "bf16", seed=seed).view(np.int16)).cuda()
    x, y = draw(2), torch.zeros((7, 256), dtype=torch.int16, device="cuda")
    layer(x, y)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        layer(x, y)
    for seed in (3, 4, 5):
        x.copy_(draw(seed))
        y.fill_(-1)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, layer(x, torch.zeros_like(y)))
    layer.close()
    with pytest.raises(AspError):
        layer(x, y)


@pytest.mark.parametrize("x,y", [((7, 383), (7, 256)), ((7, 384), (8, 256)), ((7, 384), (7, 255))])
def test_shapes_are_refused(x, y):
    w = synth.block_sparse_bernoulli(256, 384, 64, 64, 0.5, seed=1, dtype="bf16")
    layer = SparseLinear(256, 384, w.row_ptr, w.col_idx, w.values, block=64)
    dev = lambda shape, dtype=torch.int16: torch.zeros(shape, dtype=dtype, device="cuda")
    with pytest.raises(ValueError):
        layer(dev(x), dev(y))
    with pytest.raises(ValueError):
        layer(dev((7, 384), torch.int32), dev((7, 256)))
    with pytest.raises(ValueError):
        layer(dev((384, 7)).t(), dev((7, 256)))
    with pytest.raises(ValueError):
        layer(dev((7, 384)).cpu(), dev((7, 256)))

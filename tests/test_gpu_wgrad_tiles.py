"""The weight-gradient kernel at the edges of its tiles (32 x 4 x 2 sites,
runs of tiles along z that end inside a column or pass on to the next one),
through the per-layer entry point: lattices smaller than a tile, one site past
and short of a tile in every direction, odd depths, and one whose blocks take
several tiles each.  Same operands and the same bar as the layer checks of
the surrogate kernels: exact bfloat16 products accumulated in FP32 per block
and in FP64 over blocks against the FP64 oracle, 1e-5 of the largest value."""
import numpy as np
import pytest
import torch

from oracle import cnn
from paper_0901_3293_amd import inputs
from tests.hlbtest import rel, say
from tests.test_gpu_nn import CI, CO, COP, channels_last, to_bf16_bits

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(4, 4, 4), (31, 5, 7), (33, 9, 5), (64, 4, 6), (40, 36, 69)])
@pytest.mark.parametrize("layer", [0, 2, 3])
def test_wgrad_tile_edges(shape, layer):
    from paper_0901_3293_amd import hlb

    say("case: wgrad tile edges", shape, layer)
    rng = np.random.default_rng(50 + layer)
    net = hlb.Net(shape)
    p = inputs.cnn_params(seed=6)
    net.set_params(p)
    W, _ = cnn.unflatten(p)[layer]
    x = rng.normal(size=(CI[layer],) + shape[::-1])
    dz = rng.normal(size=(CO[layer],) + shape[::-1])
    xb = to_bf16_bits(channels_last(x, 32))
    dzb = to_bf16_bits(channels_last(dz, COP[layer]))
    _, g = net.layer_backward(layer, xb, dzb)
    _, g2 = net.layer_backward(layer, xb, dzb)
    dW, db, _ = cnn.layer_backward(cnn.bf16(torch.tensor(x)), cnn.bf16(torch.tensor(dz)), cnn.bf16(W))
    e_w = rel(g[:-CO[layer]], dW.reshape(-1).numpy())
    e_b = rel(g[-CO[layer]:], db.numpy())
    say("rel err dW, db", e_w, e_b)
    assert e_w <= 1e-5 and e_b <= 1e-5
    assert np.array_equal(g, g2)

"""The convolution kernel at the edges of its tiles (16 x 8 x 4 sites, two
LDS bricks in turn), through the per-layer entry points: lattices smaller than
a tile, one site past and short of a tile in every direction, and one whose
blocks take several tiles each.  Same operands and the same bar as the layer
checks of the surrogate kernels: at most 864 exact bfloat16 products
accumulated in FP32 against the FP64 oracle, 1e-5 of the largest value."""
import numpy as np
import pytest
import torch

from oracle import cnn
from paper_0901_3293_amd import inputs
from tests.hlbtest import rel, say
from tests.test_gpu_nn import CI, CO, COP, channels_last, from_channels_last, to_bf16_bits

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(4, 4, 4), (15, 7, 5), (17, 9, 4), (32, 8, 9), (80, 72, 44)])
@pytest.mark.parametrize("layer", [1, 3])
def test_conv_tile_edges(shape, layer):
    from paper_0901_3293_amd import hlb

    say("case: conv tile edges", shape, layer)
    rng = np.random.default_rng(40 + layer)
    net = hlb.Net(shape)
    p = (inputs.cnn_params(seed=6) + rng.normal(0, 0.02, size=cnn.param_count())).astype(np.float32)
    net.set_params(p)
    W, b = cnn.unflatten(p)[layer]
    x = rng.normal(size=(CI[layer],) + shape[::-1])
    z = net.layer_forward(layer, to_bf16_bits(channels_last(x, 32)))
    ref = cnn.conv(cnn.bf16(torch.tensor(x)), cnn.bf16(W), b).numpy()
    e_f = rel(from_channels_last(z, CO[layer], shape), ref)
    dz = rng.normal(size=(CO[layer],) + shape[::-1])
    dx, _ = net.layer_backward(layer, to_bf16_bits(channels_last(x, 32)), to_bf16_bits(channels_last(dz, COP[layer])))
    _, _, dxr = cnn.layer_backward(cnn.bf16(torch.tensor(x)), cnn.bf16(torch.tensor(dz)), cnn.bf16(W))
    e_b = rel(from_channels_last(dx, CI[layer], shape), dxr.numpy())
    say("rel err forward, backward-data", e_f, e_b)
    assert e_f <= 1e-5 and e_b <= 1e-5

"""The fused jump at the tile lengths it chooses: the bits of the
layer-by-layer forward pass combined as u + (64 r s) out in FP32.  Small
batches take short tiles, large ones up to 864 points; lengths at which a
tile ends inside a block of rows, at a block's edge, and one point short."""
import numpy as np
import pytest

from test_gpu_nn import dev, fp32_params, make_net, rods

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("width,batch", [
    (128, 1),       # two tiles of 64
    (4096, 1),      # 128 tiles of 32
    (512, 64),      # one block's worth more than the halo
    (896, 300),     # two tiles of 448
    (768, 300),     # one tile a rod
    (4096, 260),    # five tiles of 828: whole blocks in layer 5
    (1664, 512),    # two tiles of 832
])
def test_jump_tiles_give_the_layered_bits(width, batch):
    assert torch.cuda.is_available()
    params = fp32_params(5)
    r, u, _ = rods(17, batch, width, levels=0)
    net = make_net(width, batch, params)
    out, scale = net.forward(dev(u), dev(r))
    o = out.cpu().numpy().reshape(batch, width)
    amp = (np.float32(64.0) * r) * scale.cpu().numpy()
    un = net.jump(dev(u), dev(r)).cpu().numpy().reshape(batch, width)
    np.testing.assert_array_equal(un, u + amp[:, None] * o)

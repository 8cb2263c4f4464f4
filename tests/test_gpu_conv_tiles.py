"""One-layer networks at the edges of the convolution's 32 x 4 x 4 (3D) and
32 x 16 (2D) tiles: forward, weight and input gradients against the FP64
reference on BF16-rounded operands, so only the FP32 accumulation order
differs (27 taps x 16 channels: sqrt(432) * 6e-8 = 1.2e-6 per output, and
sqrt(points) * 6e-8 <= 1e-5 for a weight gradient)."""
import numpy as np
import pytest

from oracle import cnn_ref
from test_gpu_cnn import bf16

pytestmark = pytest.mark.gpu

SHAPES = {2: [(1, 16, 32), (2, 17, 33), (3, 1, 1), (1, 15, 70)],
          3: [(1, 4, 4, 32), (2, 5, 5, 33), (1, 1, 1, 1), (1, 3, 9, 31), (1, 8, 8, 64)]}


@pytest.mark.parametrize("channels", [(4, 8), (3, 2), (8, 5), (16, 16)])
@pytest.mark.parametrize("dim,shape", [(d, s) for d in SHAPES for s in SHAPES[d]])
def test_one_layer_at_tile_edges(dim, shape, channels):
    import torch
    import paper_2001_10424_amd as gk
    print("[case] conv tiles", dim, shape, channels, flush=True)
    rng = np.random.default_rng(2)
    net = gk.CNN(dim, channels, seed=5)
    net.params = net.params + 0.1 * rng.standard_normal(net.n_params).astype(np.float32)
    params = net.params.astype(np.float64)
    x = rng.standard_normal(shape + (channels[0],)).astype(np.float32)
    dy = bf16(rng.standard_normal(shape + (channels[1],))).astype(np.float32)

    def dev(a, shift):  # shift: a buffer that is not 16-byte aligned
        buf = torch.empty(a.size + 1, device="cuda")
        out = buf[shift:shift + a.size].view(a.shape)
        out.copy_(torch.from_numpy(a))
        return out
    W, b = cnn_ref.unflatten(params, dim, channels)[0]
    ref = cnn_ref.conv(bf16(x), bf16(W), b, dim)
    gr, dxr = cnn_ref.backward(bf16(x), bf16(params), dim, channels, dy)
    for shift in (0, 1):
        y = net.forward(dev(x, shift)).cpu().numpy()
        assert np.abs(y - ref).max() <= 1e-5 * np.abs(ref).max()
        g, dx = net.backward(dev(x, shift), dev(dy, shift))
        assert np.linalg.norm(g - gr) <= 1e-5 * np.linalg.norm(gr)
        assert np.linalg.norm(dx.cpu().numpy() - dxr) <= 1e-5 * np.linalg.norm(dxr)

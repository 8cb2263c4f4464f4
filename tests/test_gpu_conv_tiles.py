"""One-layer networks at the edges of the convolution's 32 x 4 x 4 (3D) and
32 x 16 (2D) tiles: forward, weight and input gradients against the FP64
reference on BF16-rounded operands, so only the FP32 accumulation order
differs (27 taps x 16 channels: sqrt(432) * 6e-8 = 1.2e-6 per output, and
sqrt(points) * 6e-8 <= 1e-5 for a weight gradient)."""
import numpy as np
import pytest

from oracle import cnn_ref
from test_gpu_cnn import _ref_backward_bf16, bf16

pytestmark = pytest.mark.gpu

SHAPES = {2: [(1, 16, 32), (2, 17, 33), (3, 1, 1), (1, 15, 70)],
          3: [(1, 4, 4, 32), (2, 5, 5, 33), (1, 1, 1, 1), (1, 3, 9, 31), (1, 8, 8, 64)]}


@pytest.mark.parametrize("channels", [(4, 8), (3, 2), (8, 5), (16, 16), (12, 7)])
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


@pytest.mark.parametrize("channels", [(4, 8), (8, 3), (16, 5), (8, 16)])
@pytest.mark.parametrize("dim", [2, 3])
def test_non_finite_inputs_stay_local(dim, channels):
    """An infinity or NaN reaches the points whose taps see it and no other:
    these are the same bits as without it (the two points of a pair share
    their taps inside the kernel)."""
    import itertools

    import torch
    import paper_2001_10424_amd as gk
    print("[case] conv non-finite", dim, channels, flush=True)
    shape = (1, 18, 66) if dim == 2 else (1, 6, 9, 66)
    net = gk.CNN(dim, channels, seed=5)
    gen = torch.Generator(device="cuda").manual_seed(1)
    x = torch.randn(shape + (channels[0],), generator=gen, device="cuda")
    n = shape[1:]
    spots = [tuple([n[a] // 2 for a in range(dim - 1)] + [i]) for i in (0, 7, 20, 31, 32, 45, n[-1] - 1)]
    bad, near = x.clone(), np.zeros(n, bool)
    for q, p in enumerate(spots):
        bad[(0,) + p + (q % channels[0],)] = (float("inf"), float("-inf"), float("nan"))[q % 3]
        x[(0,) + p + (q % channels[0],)] = 0.0
        for d in itertools.product((-1, 0, 1), repeat=dim):
            at = tuple(a + b for a, b in zip(p, d))
            if all(0 <= a < b for a, b in zip(at, n)):
                near[at] = True
    y, z = net.forward(x)[0].cpu().numpy(), net.forward(bad)[0].cpu().numpy()
    assert np.array_equal(y[~near], z[~near])
    assert not np.isfinite(z[near]).any()


def _integer_network(dim, channels, rng):
    """Flat parameters: every output channel takes one tap of one input
    channel with weight 1 or -1, biases 0 to 2."""
    parts = []
    taps = 3 ** dim
    for cin, cout in zip(channels[:-1], channels[1:]):
        W = np.zeros((taps, cin, cout))
        for co in range(cout):
            W[rng.integers(taps), co % cin, co] = 1.0
        parts += [W.ravel(), rng.integers(0, 3, cout).astype(float)]
    return np.concatenate(parts)


@pytest.mark.parametrize("channels", [(4, 8, 16, 3, 8, 12, 5, 9, 2), (16, 4, 1), (1, 16, 8)])
@pytest.mark.parametrize("dim", [2, 3])
def test_layers_reduced_together(dim, channels):
    """The weight gradients of all layers are added up in one launch: every
    layer's block of the gradient, up to the eight layers a network can have
    and with channel groups of 4, 8 and 16 side by side.  All stored values
    are integers below 256 (exact in BF16) and all sums below 2^24 (exact in
    FP32), so the gradients have to be equal."""
    import torch
    import paper_2001_10424_amd as gk
    print("[case] conv layers", dim, channels, flush=True)
    rng = np.random.default_rng(4)
    shape = SHAPES[dim][1]
    params = _integer_network(dim, channels, rng)
    x = rng.integers(-2, 3, shape + (channels[0],)).astype(np.float32)
    dy = rng.integers(-1, 2, shape + (channels[-1],)).astype(np.float32)
    want, dxw = _ref_backward_bf16(x, params, dim, channels, dy)
    assert np.abs(want).max() < 2 ** 24
    assert all(W.any() and b.any() for W, b in cnn_ref.unflatten(want, dim, channels))
    net = gk.CNN(dim, channels, seed=6)
    net.params = params.astype(np.float32)
    for _ in range(2):
        got, dx = net.backward(torch.from_numpy(x).cuda(), torch.from_numpy(dy).cuda())
        assert np.array_equal(np.asarray(got, np.float64), want)
        assert np.array_equal(dx.cpu().numpy().astype(np.float64), dxw)


@pytest.mark.parametrize("dim", [2, 3])
def test_one_layer_on_its_own_buffers(dim):
    """A single layer whose output lies on its input (y on x; dx on dy, and on
    x): the same bits as in buffers of their own."""
    import ctypes as C

    import torch
    import paper_2001_10424_amd as gk
    print("[case] conv in place", dim, flush=True)
    shape = (2, 90, 70) if dim == 2 else (2, 17, 22, 35)
    net = gk.CNN(dim, (8, 8), seed=3)
    gen = torch.Generator(device="cuda").manual_seed(2)
    x, dy = (torch.randn(shape + (8,), generator=gen, device="cuda") for _ in range(2))
    y = net.forward(x)
    grad, dx = net.backward(x, dy)
    L, geom = gk.library(), net._geom(x, dim)
    ptr = lambda t: C.c_void_p(t.data_ptr())  # noqa: E731
    a = x.clone()
    assert L.gkb_cnn_forward(net._h, *geom, ptr(a), ptr(a)) == 0
    assert torch.equal(a, y)
    for on_x in (False, True):
        a, b, g = x.clone(), dy.clone(), np.empty_like(grad)
        out = a if on_x else b
        assert L.gkb_cnn_backward(net._h, *geom, ptr(a), ptr(b), ptr(out),
                                  g.ctypes.data_as(C.c_void_p)) == 0
        assert torch.equal(out, dx) and np.array_equal(g, grad)


@pytest.mark.parametrize("channels", [(4, 8), (8, 3), (16, 5), (12, 16)])
@pytest.mark.parametrize("dim,shape", [(2, (1, 18, 40)), (2, (2, 5, 31)), (3, (1, 5, 6, 33)),
                                       (3, (2, 4, 4, 32)), (3, (1, 3, 9, 65))])
def test_non_finite_weight_gradients_stay_local(dim, shape, channels):
    """An infinite activation in the last column, row or plane makes the
    gradients of the taps non-finite that combine it with a point of the grid,
    and no other: these are the same bits as without it (a tile's points past
    the grid take no part)."""
    import itertools

    import torch
    import paper_2001_10424_amd as gk
    print("[case] conv weight gradient non-finite", dim, shape, channels, flush=True)
    net = gk.CNN(dim, channels, seed=5)
    gen = torch.Generator(device="cuda").manual_seed(1)
    x = torch.randn(shape + (channels[0],), generator=gen, device="cuda")
    dy = torch.rand(shape + (channels[1],), generator=gen, device="cuda") + 0.5
    for axis in range(dim):
        # the last entry along the axis, in the middle of the others
        at = [n // 2 for n in shape[1:]]
        at[axis] = shape[1 + axis] - 1
        spot = (0, *at, axis)
        bad = x.clone()
        x[spot], bad[spot] = 0.0, float("inf")
        g0, _ = net.backward(x, dy, want_dx=False)
        g1, _ = net.backward(bad, dy, want_dx=False)
        w0, w1 = (cnn_ref.unflatten(g, dim, channels)[0] for g in (g0, g1))
        assert np.array_equal(w0[1], w1[1])  # the bias gradient sees dy alone
        for tap, d in enumerate(itertools.product((-1, 0, 1), repeat=dim)):
            seen = all(0 <= a - b < n for a, b, n in zip(at, d, shape[1:]))
            for ci in range(channels[0]):
                row0, row1 = w0[0][tap, ci], w1[0][tap, ci]
                if seen and ci == axis:
                    assert not np.isfinite(row1).any(), (axis, tap, ci)
                else:
                    assert np.array_equal(row0, row1), (axis, tap, ci)


def test_more_tiles_than_a_launch_takes():
    """A batch of more small grids than one launch has blocks for (2^32
    threads): every part of it the same bits as by itself."""
    import torch
    import paper_2001_10424_amd as gk
    print("[case] conv batch", flush=True)
    n, m = (1 << 24) + 11, 4096
    net = gk.CNN(2, (1, 12), seed=3)
    part = torch.randn((m, 1, 1, 1), generator=torch.Generator(device="cuda").manual_seed(5),
                       device="cuda")
    want = net.forward(part)
    x = part.repeat(n // m + 1, 1, 1, 1)[:n].contiguous()
    y = net.forward(x)
    full = n // m * m
    assert bool((y[:full].view(-1, m, 12) == want.view(1, m, 12)).all())
    assert torch.equal(y[full:], want[:n - full])

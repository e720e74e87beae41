"""All four loops in one launch (fused_small.hip): edges of its items (16 filters x 16 tiles), of its steps (8 or 16 channels)
and of images, against the oracle; the calls are small enough for WINO_FLAG_AUTO to take it."""
import numpy as np
import pytest

from oracle import direct
from gpu_util import check_close, rel_err, require_gpu, to_gpu

pytestmark = pytest.mark.gpu

TOL = {2: 1e-5, 4: 1e-4, 6: 1e-4}
SHAPES = [
    # N, C, H, W, K, pad
    (1, 1, 8, 8, 1, 1),          # one channel, one filter
    (1, 8, 9, 8, 16, 1),         # whole steps and items (m = 4, 6)
    (3, 16, 12, 12, 17, 1),      # one filter more than an item
    (2, 17, 15, 9, 20, 1),       # the last step is one channel; the last tile of a row reaches past the image
    (5, 5, 5, 10, 9, 0),         # several images per item
    (2, 9, 11, 13, 33, 0),
    (1, 24, 8, 31, 16, 1),
    (1, 10, 30, 14, 40, 0),
    (7, 3, 7, 11, 12, 1),
]


def data(N, C, H, W, K, seed):
    rng = np.random.default_rng(seed)
    return (rng.standard_normal((N, C, H, W)).astype(np.float32),
            (rng.standard_normal((K, C, 3, 3)) * np.sqrt(2.0 / (9 * C))).astype(np.float32))


def inside(torch, x):
    """`x` on the GPU with NaNs right in front of it and right behind."""
    room = torch.full((x.size + 8,), float("nan"), device="cuda")
    t = room[4:4 + x.size].view(x.shape)
    t.copy_(to_gpu(x))
    return t


@pytest.mark.parametrize("m", [2, 4, 6])
@pytest.mark.parametrize("N,C,H,W,K,pad", SHAPES)
def test_small_layers(N, C, H, W, K, pad, m):
    torch, w = require_gpu()
    D, G = data(N, C, H, W, K, N + C + H + W + K)
    ref = direct.conv2d_fwd(D, G, pad=pad)
    d, g = inside(torch, D), inside(torch, G)
    ws = w.alloc_workspace(N, C, H, W, K, pad, m, w.WINO_F32)
    for kw in ({"G": g}, {"U": w.wino_filter_transform(g, m), "K": K}):
        ws.fill_(0xff)                                         # NaNs: nothing in it is read
        Y = torch.full(ref.shape, float("nan"), device="cuda")
        w.wino_conv2d_fwd_ex(d, pad=pad, m=m, Y=Y, workspace=ws, **kw)
        check_close(Y.cpu().numpy(), ref, TOL[m], "m=%d %s %s" % (m, (N, C, H, W, K, pad), list(kw)), m=m)
        assert bool((ws == 0xff).all()) == w.wino_small_layer(N, C, H, W, K, pad, m, filters=w.FILTERS_G if "G" in kw else w.FILTERS_U)


@pytest.mark.parametrize("m", [2, 4, 6])
@pytest.mark.parametrize("N,C,H,W,K", [(2, 20, 13, 10, 12), (1, 16, 12, 17, 35), (3, 1, 9, 9, 8)])
def test_small_input_gradients(N, C, H, W, K, m):
    torch, w = require_gpu()
    rng = np.random.default_rng(N + C + K)
    _, G = data(N, C, H, W, K, 1)
    E = rng.standard_normal((N, K, H, W)).astype(np.float32)
    got = w.wino_conv2d_bwd_data(inside(torch, E), G=inside(torch, G), pad=1, m=m).cpu().numpy()
    check_close(got, direct.conv2d_bwd_data(E, G, H, W, pad=1), TOL[m], "m=%d" % m, m=m)


@pytest.mark.parametrize("m", [2, 4, 6])
def test_small_layers_are_at_least_as_precise(m):
    """Sums in 64 bits: the distance to float64 is that of the transforms, and below the four stages'."""
    torch, w = require_gpu()
    N, C, H, W, K = 1, 32, 24, 24, 32
    D, G = data(N, C, H, W, K, 5)
    ref = direct.conv2d_fwd(D, G, pad=1)
    d, g = to_gpu(D), to_gpu(G)
    one = rel_err(w.wino_conv2d_fwd_ex(d, G=g, pad=1, m=m).cpu().numpy(), ref)
    four = rel_err(w.wino_conv2d_fwd_ex(d, G=g, pad=1, m=m, flags=w.FLAG_UNFUSED).cpu().numpy(), ref)
    print("m=%d: one launch %.2e, four stages %.2e" % (m, one, four))
    assert one <= four


def test_bench_times_the_launch_that_the_layer_makes():
    torch, w = require_gpu()
    import bench
    L = bench.make_layers(1, np.float32, "2", 1, shapes=[("layer", 32, 56, 32)])[0]
    ws = torch.empty(L.ws_bytes, dtype=torch.uint8, device="cuda").fill_(0xff)
    plans, nbytes, kernel, _ = bench.stage_plan(torch, w, L, ws, 1)
    assert w.wino_small_layer(1, 32, 56, 56, 32, 1, 2) and kernel.startswith("fused_small_kernel<2")
    assert [name for name, _ in plans[0]] == list(nbytes) == ["fused"]
    plans[0][0][1]()
    assert bool((ws == 0xff).all())
    assert rel_err(L.Y.cpu().numpy(), direct.conv2d_fwd(L.D_host, L.G_host, pad=1)) <= TOL[2]

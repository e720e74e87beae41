"""All four loops in one launch (fused_small.hip): edges of its items (16 filters x 16 tiles), of its steps (8 or 16 channels)
and of images, against the oracle.  That a call took it is seen by a workspace full of NaNs that it leaves as it was."""
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


def forward(torch, w, d, kw, shape, m):
    """A layer into NaNs with a workspace of NaNs, and whether the workspace was left alone."""
    N, C, H, W, K, pad = shape
    ws = w.alloc_workspace(N, C, H, W, K, pad, m, w.WINO_F32).fill_(0xff)
    Y = torch.full((N, K, H + 2 * pad - 2, W + 2 * pad - 2), float("nan"), device="cuda")
    w.wino_conv2d_fwd_ex(d, pad=pad, m=m, Y=Y, workspace=ws, **kw)
    return Y.cpu().numpy(), bool((ws == 0xff).all())


@pytest.mark.parametrize("m,shape", [
    (6, (1, 16, 226, 226, 32, 1)),       # two steps
    (6, (4, 21, 151, 146, 13, 0)),       # three, the last of five channels
    (6, (4, 39, 150, 147, 16, 1)),       # five
    (6, (42, 1, 48, 48, 34, 1)),         # 504 items: two rounds of workgroups
    (6, (31, 3, 172, 172, 9, 1)),        # 1630 items
    (4, (6, 32, 84, 86, 16, 1)),         # four steps
    (4, (10, 20, 120, 123, 40, 1)),      # 1746 items, three steps
    (4, (9, 13, 100, 99, 50, 0)),        # 1408 items, two steps
    (2, (3, 97, 57, 58, 20, 1)),         # seven steps, the last of one channel
    (2, (2, 20, 100, 101, 40, 1)),       # 957 items
    (2, (9, 13, 50, 51, 30, 1)),         # 732 items, one step
])
def test_several_steps_and_rounds(m, shape):
    """The longest loops over channels and the most items that the rule sends here."""
    torch, w = require_gpu()
    N, C, H, W, K, pad = shape
    D, G = data(N, C, H, W, K, sum(shape))
    ref = direct.conv2d_fwd(D, G, pad=pad)
    d, g = inside(torch, D), inside(torch, G)
    assert w.wino_small_layer(*shape, m)
    for kw, filters in (({"G": g}, w.FILTERS_G), ({"U": w.wino_filter_transform(g, m), "K": K}, w.FILTERS_U)):
        Y, alone = forward(torch, w, d, kw, shape, m)
        check_close(Y, ref, TOL[m], "m=%d %s %s" % (m, shape, list(kw)), m=m)
        assert alone == w.wino_small_layer(*shape, m, filters=filters)
    if pad == 1:                                               # the gradient whose exchanged layer has these extents
        ws = w.alloc_workspace(N, C, H, W, K, 1, m, w.WINO_F32).fill_(0xff)
        Gb = np.ascontiguousarray(G.transpose(1, 0, 2, 3))     # [C errors][K inputs]
        dD = w.wino_conv2d_bwd_data(d, G=inside(torch, Gb), pad=1, m=m, workspace=ws).cpu().numpy()
        check_close(dD, direct.conv2d_bwd_data(D, Gb, H, W, pad=1), TOL[m], "m=%d %s, gradient" % (m, shape), m=m)
        assert bool((ws == 0xff).all()) and w.wino_small_layer(*shape, m, filters=w.FILTERS_G_BWD)


@pytest.mark.parametrize("m", [2, 4, 6])
@pytest.mark.parametrize("N,C,H,W,K", [(2, 20, 13, 10, 12), (1, 16, 12, 17, 35), (3, 1, 9, 9, 8)])
def test_small_input_gradients(N, C, H, W, K, m):
    torch, w = require_gpu()
    rng = np.random.default_rng(N + C + K)
    _, G = data(N, C, H, W, K, 1)
    E = rng.standard_normal((N, K, H, W)).astype(np.float32)
    ws = w.alloc_workspace(N, K, H, W, C, 1, m, w.WINO_F32).fill_(0xff)
    got = w.wino_conv2d_bwd_data(inside(torch, E), G=inside(torch, G), pad=1, m=m, workspace=ws).cpu().numpy()
    check_close(got, direct.conv2d_bwd_data(E, G, H, W, pad=1), TOL[m], "m=%d" % m, m=m)
    small = w.wino_small_layer(N, K, H, W, C, 1, m, filters=w.FILTERS_G_BWD)
    assert bool((ws == 0xff).all()) == small
    assert small or K > {2: 64, 4: 24, 6: 16}[m]               # (few tiles: channels up to which the rule sends them here)


@pytest.mark.parametrize("m,shape", [(2, (1, 32, 24, 24, 32, 1)), (4, (1, 24, 24, 24, 32, 1)), (6, (4, 39, 150, 147, 16, 1))])
def test_small_layers_are_at_least_as_precise(m, shape):
    """Sums in 64 bits: the distance to float64 is that of the transforms, and below the four stages'."""
    torch, w = require_gpu()
    D, G = data(*shape[:5], 5)
    ref = direct.conv2d_fwd(D, G, pad=1)
    d, g = to_gpu(D), to_gpu(G)
    Y, alone = forward(torch, w, d, {"G": g}, shape, m)
    assert alone
    one = rel_err(Y, ref)
    four = rel_err(w.wino_conv2d_fwd_ex(d, G=g, pad=1, m=m, flags=w.FLAG_UNFUSED).cpu().numpy(), ref)
    print("m=%d: one launch %.2e, four stages %.2e" % (m, one, four))
    assert one <= four


@pytest.mark.parametrize("m", [2, 4, 6])
@pytest.mark.parametrize("value", [np.inf, np.nan])
def test_values_that_are_not_finite_stay_in_their_tiles(m, value):
    """At the corners of images, where tiles reach outside, and in the last channel: neighbours in an item keep their bits."""
    torch, w = require_gpu()
    shape = N, C, H, W, K, pad = 3, 7, 2 * m + 1, 3 * m + 1, 18, 1
    D, G = data(*shape[:5], 9)
    g = to_gpu(G)
    plain, alone = forward(torch, w, to_gpu(D), {"G": g}, shape, m)
    assert alone
    for n, c, x, y in ((0, 0, 0, 0), (1, 6, H - 1, W - 1), (2, 3, m, m - 1)):
        X = D.copy()
        X[n, c, x, y] = value
        Y, _ = forward(torch, w, to_gpu(X), {"G": g}, shape, m)
        near = np.zeros(Y.shape, dtype=bool)                   # outputs of the tiles that have (x, y) among their inputs
        for tx in range(-(-H // m)):
            for ty in range(-(-W // m)):
                if m * tx - 1 <= x <= m * tx + m and m * ty - 1 <= y <= m * ty + m:
                    near[n, :, m * tx:m * tx + m, m * ty:m * ty + m] = True
        assert (Y[~near] == plain[~near]).all()
        reach = np.zeros(Y.shape, dtype=bool)                  # the definition's outputs of (x, y)
        reach[n, :, max(x - 1, 0):x + 2, max(y - 1, 0):y + 2] = True
        assert not np.isfinite(Y[reach]).any()


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

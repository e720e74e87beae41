"""The one-kernel fp32 layer on the bf16 matrix units (64 filters x 32 tiles per item, 64 for F(2x2,3x3); 128 items and
more), at the edges of its items, channel steps, XCD groups and shared last rounds."""
import numpy as np
import pytest

from oracle import direct
from paper_1509_09308_amd import synth
from gpu_util import TOL, check_close, rel_err, require_gpu, to_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,shape", [
    (4, (20, 17, 28, 60, 70)),       # 132 items, two channel steps (the second one channel deep), 38 padded filters read twice
    (4, (33, 16, 28, 20, 256)),      # one step; items over several images, last tile block ragged
    (4, (5, 40, 66, 128, 96)),       # last tile row half outside; 96 filters: the second block half empty
    (4, (17, 128, 28, 44, 513)),     # 369 items: a full round, then 15 items per XCD in two shares; nine filter blocks
    (4, (4, 144, 48, 96, 500)),      # 288 items of nine steps, which no number of shares divides
    (4, (4, 256, 48, 96, 520)),      # 324 items: XCDs with 9 items and one with 5 in their last round
    (2, (13, 17, 30, 46, 70)),
    (2, (3, 130, 65, 64, 200)),      # odd height
    (2, (6, 256, 48, 60, 400)),
])
@pytest.mark.parametrize("given", ["G", "U"])
def test_split_layer(m, shape, given):
    torch, w = require_gpu()
    N, C, H, W, K = shape
    items = -(-w.wino_num_tiles(N, H, W, 1, m) // (32 if m == 4 else 64)) * -(-K // 64)
    assert items >= 128 and sum(p[0] for p in w.wino_one_kernel_plan(N, C, H, W, K, 1, m)[1]) == items       # this kernel's
    D, G = synth.make_layer(N, C, H, W, K, seed=sum(shape) + m)
    d, g = to_gpu(D), to_gpu(G)
    ws = w.alloc_workspace(N, C, H, W, K, 1, m)
    ws.view(torch.float32).fill_(float("nan"))
    kw = dict(G=g) if given == "G" else dict(U=w.wino_filter_transform(g, m), K=K)
    Y = torch.full((N, K, H, W), float("nan"), device="cuda")
    w.wino_conv2d_fwd_ex(d, pad=1, m=m, flags=w.FLAG_FUSED, workspace=ws, Y=Y, **kw)
    Y2 = w.wino_conv2d_fwd_ex(d, pad=1, m=m, flags=w.FLAG_FUSED, workspace=ws, **kw)
    pts = synth.sample_points((N, K, H, W), 3000, seed=1, edge=m)
    got = Y.cpu().numpy()
    assert np.isfinite(got).all()
    assert torch.equal(Y, Y2)
    ref = direct.conv2d_points(D, G, pts, pad=1)
    e, worst = check_close(got[tuple(pts.T)], ref, TOL[("f32", m)], "%s %s" % (shape, given), m)
    print("F(%d) %s %s: rel err %.2e, max %.2e" % (m, shape, given, e, worst))


def test_split_layer_input_gradient():
    torch, w = require_gpu()
    N, C, H, W, K = 20, 72, 28, 60, 40          # 132 items, F(2x2,3x3) 264
    _, G = synth.make_layer(1, C, 4, 4, K, seed=3)
    E = np.random.default_rng(4).standard_normal((N, K, H, W)).astype(np.float32)
    for m in (2, 4):
        dD = w.wino_conv2d_bwd_data(to_gpu(E), G=to_gpu(G), pad=1, m=m, flags=w.FLAG_FUSED).cpu().numpy()
        check_close(dD, direct.conv2d_bwd_data(E, G, H, W, pad=1), TOL[("f32", m)], "input gradient F(%d)" % m, m)


@pytest.mark.parametrize("shape", [(20, 17, 28, 60, 70), (33, 16, 28, 20, 256), (5, 40, 66, 128, 96), (17, 128, 28, 44, 513),
                                   (4, 256, 48, 96, 520)])
@pytest.mark.parametrize("given", ["G", "U"])
@pytest.mark.parametrize("y", ["f32", "f16"])
def test_split_layer_f16(shape, given, y):
    torch, w = require_gpu()
    N, C, H, W, K = shape
    D, G = synth.make_layer(N, C, H, W, K, seed=sum(shape), dtype=np.float16)
    d, g = to_gpu(D), to_gpu(G)
    ws = torch.full((w.wino_workspace_bytes(N, C, H, W, K, 1, 4, w.WINO_F16) // 4 + 1,), float("nan"), device="cuda").view(torch.uint8)
    kw = dict(G=g) if given == "G" else dict(U=w.wino_filter_transform(g, 4), K=K)
    Y = torch.full((N, K, H, W), float("nan"), device="cuda", dtype=torch.float32 if y == "f32" else torch.float16)
    w.wino_conv2d_fwd_ex(d, pad=1, m=4, flags=w.FLAG_FUSED, workspace=ws, Y=Y, **kw)
    Y2 = w.wino_conv2d_fwd_ex(d, pad=1, m=4, flags=w.FLAG_FUSED, workspace=ws, y_dtype=Y.dtype, **kw)
    assert torch.equal(Y, Y2)
    pts = synth.sample_points((N, K, H, W), 3000, seed=2, edge=4)
    got = Y.float().cpu().numpy()
    assert np.isfinite(got).all()
    ref = direct.conv2d_points(D.astype(np.float32), G.astype(np.float32), pts, pad=1)
    check_close(got[tuple(pts.T)], ref, TOL[("f16", 4)], "%s %s" % (shape, given), 4)


@pytest.mark.parametrize("C", [3072, 4096])
@pytest.mark.parametrize("m", [2, 4])
@pytest.mark.parametrize("data", ["positive", "near one"])
def test_long_channel_sums(m, C, data):
    """One-signed data: one component of a tile holds one large sum, in which small products could get lost (those of
    operands between 1 and 1 + 2^-7 all have one sign)."""
    torch, w = require_gpu()
    N, H, K = 24, 28, 256
    gen = torch.Generator(device="cuda")
    gen.manual_seed(C + m)
    def make(*shape):
        x = torch.rand(shape, generator=gen, device="cuda")
        return x if data == "positive" else 1.0 + x * 2.0 ** -7
    D, G = make(N, C, H, H), make(K, C, 3, 3)
    Y = w.wino_conv2d_fwd_ex(D, G=G, pad=1, m=m, flags=w.FLAG_FUSED)[-1, ::37].cpu().numpy()
    d, g = D[-1:].cpu().numpy(), G[::37].cpu().numpy()
    ref = direct.conv2d_fwd(d, g, pad=1)[0]
    chain = np.zeros((len(g), H - 2, H - 2), dtype=np.float32)    # the centre taps alone, fp32 multiply-adds (rounded twice)
    centre = np.zeros((len(g), H - 2, H - 2))
    for c in range(C):
        x, y = d[0, c, 1:-1, 1:-1], g[:, c, 1, 1]
        chain += x * y[:, None, None]
        centre += x.astype(np.float64) * y[:, None, None]
    e, ec = rel_err(Y, ref), rel_err(chain, centre)
    print("F(%d) C=%d %s: rel err %.2e, fp32 chain %.2e" % (m, C, data, e, ec))
    assert e <= 1.3 * ec            # (the transforms round a few times more)

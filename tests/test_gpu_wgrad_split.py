"""Filter gradient in one kernel on the bf16 matrix units, at the edges of its steps (8 blocks), rows of blocks, 64 x 64
blocks of M and shares; and its rounding over many shares."""
import numpy as np
import pytest

from oracle import direct
from oracle import winograd as wg
from paper_1509_09308_amd import synth
from gpu_util import check_close, rel_err, require_gpu, to_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,C,H,W,K", [
    (1, 5, 2, 4, 7),             # two blocks in all
    (1, 64, 3, 8, 64),           # odd height: the last error row has no partner
    (3, 33, 6, 12, 65),          # rows of six blocks: pairs of one step in two rows and two images
    (2, 64, 16, 16, 64),         # whole steps
    (5, 70, 9, 20, 130),         # 225 blocks: the last step and share ragged
    (2, 300, 12, 16, 40),        # more than 256 channels
    (3, 320, 28, 28, 288),
])
def test_wgrad_in_one_kernel(N, C, H, W, K):
    torch, w = require_gpu()
    rng = np.random.default_rng(N + C + H + W + K)
    D = rng.standard_normal((N, C, H, W)).astype(np.float32)
    E = rng.standard_normal((N, K, H, W)).astype(np.float32)
    need = w.wino_bwd_filter_workspace_bytes(N, C, H, W, K)
    ws = torch.full((need // 4 + 1,), float("nan"), device="cuda").view(torch.uint8)[:need]
    dG = w.wino_conv2d_bwd_filter(to_gpu(D), to_gpu(E), pad=1, workspace=ws).cpu().numpy()
    check_close(dG, direct.conv2d_bwd_filter(D, E, pad=1), 1e-5, "%s" % ((N, C, H, W, K),))


def inside(torch, x):
    """`x` with NaNs right in front of it and right behind."""
    room = torch.full((x.numel() + 8,), float("nan"), device="cuda")
    t = room[4:4 + x.numel()].view(x.shape)
    t.copy_(x)
    return t


def gradient(torch, w, D, E):
    """The gradient with a workspace of NaNs, and whether one kernel formed it: the separate stages write all of the workspace
    but what alignment leaves between their tensors."""
    (N, C, H, W), K = D.shape, E.shape[1]
    need = w.wino_bwd_filter_workspace_bytes(N, C, H, W, K)
    ws = torch.full((need // 4,), float("nan"), device="cuda")
    dG = w.wino_conv2d_bwd_filter(D, E, pad=1, workspace=ws.view(torch.uint8))
    return dG, int(torch.isnan(ws).sum()) > 1024


@pytest.mark.parametrize("N,C,H,W,K", [(30, 64, 30, 30, 64), (47, 112, 11, 11, 390)])
def test_small_layers_of_any_width_in_stages(N, C, H, W, K):
    torch, w = require_gpu()
    gen = torch.Generator(device="cuda")
    gen.manual_seed(N + C + H + W + K)
    D, E = (inside(torch, torch.randn((N, x, H, W), generator=gen, device="cuda")) for x in (C, K))
    dG, one = gradient(torch, w, D, E)
    assert not one
    ks, cs = [0, K // 2, K - 1], [0, C // 2, C - 1]
    ref = direct.conv2d_bwd_filter(D[:, cs].cpu().numpy(), E[:, ks].cpu().numpy(), pad=1)
    check_close(dG[ks][:, cs].cpu().numpy(), ref, 2e-6, "%s" % ((N, C, H, W, K),))


@pytest.mark.parametrize("N,C,H,W,K", [
    (600, 33, 7, 5, 70),         # rows of three blocks: the last pair has one, of one column
    (700, 64, 8, 6, 64),         # of two columns
    (260, 40, 9, 7, 130),        # rows of four blocks, the last of one column
    (120, 70, 9, 13, 130),
    (6, 16, 75, 101, 65),        # pairs of one step in two rows, the last step of a share ragged
    (30, 256, 94, 94, 256),      # shares of more than 2048 blocks
])
def test_wgrad_in_one_kernel_any_width(N, C, H, W, K):
    """Widths that 4 does not divide, from 64 MB of transformed operands on (smaller layers take the separate stages).
    What lies before and behind D and E must not matter: rows end where the next one, the next image or nothing begins.
    Bound: as for the small layers on the separate stages, twice the largest that is measured (9.8e-7)."""
    torch, w = require_gpu()
    gen = torch.Generator(device="cuda")
    gen.manual_seed(N + C + H + W + K)
    D, E = (inside(torch, torch.randn((N, x, H, W), generator=gen, device="cuda")) for x in (C, K))
    dG, one = gradient(torch, w, D, E)
    assert one
    assert bool(torch.isfinite(dG).all())
    ks, cs = sorted({0, K // 2, K - 1}), sorted({0, C // 2, C - 1})
    ref = direct.conv2d_bwd_filter(D[:, cs].cpu().numpy(), E[:, ks].cpu().numpy(), pad=1)
    check_close(dG[ks][:, cs].cpu().numpy(), ref, 2e-6, "%s" % ((N, C, H, W, K),))


@pytest.mark.parametrize("H,W", [(112, 112), (111, 113), (112, 110), (112, 111)])
def test_rounding_does_not_add_up_over_shares(H, W):
    """Positive data: every product of the first component grows the sums, the case in which a rounding that always goes
    one way shows most.  fp32 sums of n terms rounded to nearest stay within sqrt(n) 2^-24 of a share's sum."""
    torch, w = require_gpu()
    N, C, K = 4, 64, 64
    rng = np.random.default_rng(1)
    D = rng.uniform(0.0, 1.0, (N, C, H, W)).astype(np.float32)
    E = rng.uniform(0.0, 1.0, (N, K, H, W)).astype(np.float32)
    dG = w.wino_conv2d_bwd_filter(to_gpu(D), to_gpu(E), pad=1).cpu().numpy()
    pts = np.array([[k, c, u, v] for k in (0, 31, 63) for c in (0, 40, 63) for u in range(3) for v in range(3)], dtype=np.int32)
    ref = direct.conv2d_bwd_filter_points(D, E, pts, pad=1)
    e = np.linalg.norm(dG[tuple(pts.T)] - ref) / np.linalg.norm(ref)
    print("rel err %.2e" % e)
    assert e <= 1e-6


@pytest.mark.parametrize("data", ["positive", "near one", "normal"])
@pytest.mark.parametrize("N,C,H,K", [(64, 512, 14, 512),        # widths that 4 does not divide: eight shares of 448 blocks
                                     (30, 256, 93, 250),        # ... 32 shares of 2128, set aside on the way
                                     (30, 256, 94, 250),
                                     (32, 256, 91, 250),
                                     (10, 1030, 28, 1030),      # one share of 1960 blocks
                                     (32, 1030, 28, 1030),      # 6272 blocks in four shares
                                     (32, 640, 28, 640),        # five shares of 1264
                                     (66, 256, 112, 256)])      # 32 shares of 6480 blocks, set aside on the way
def test_long_shares_are_as_precise_as_fp32(N, C, H, K, data):
    """Few, long shares: nothing may add up along them.  Operands between 1 and 1 + 2^-7 have products of low parts that
    are all of one sign; the sums of such and of positive data hold one large component, in which those could get lost."""
    torch, w = require_gpu()
    gen = torch.Generator(device="cuda")
    gen.manual_seed(N + C)
    def make(*shape):
        if data == "normal":
            return torch.randn(shape, generator=gen, device="cuda")
        x = torch.rand(shape, generator=gen, device="cuda")
        return x if data == "positive" else 1.0 + x * 2.0 ** -7
    D, E = make(N, C, H, H), make(N, K, H, H)
    dG = w.wino_conv2d_bwd_filter(D, E, pad=1)
    ks, cs = [0, 70, K - 1], [0, 65, C - 2]
    d, e = D[:, cs].cpu().numpy(), E[:, ks].cpu().numpy()
    ref = direct.conv2d_bwd_filter(d, e, pad=1)
    got = dG[ks][:, cs].cpu().numpy()
    # the same blocks, one after the other, in fp32: every component is a chain of multiply-adds (rounded twice)
    Wt, V = (x.astype(np.float32) for x in (wg.wgrad_error_transform(e), wg.wgrad_data_transform(d)))
    assert Wt.shape[3] == N * ((H + 1) // 2) ** 2
    M = np.zeros((4, 4, len(ks), len(cs)), dtype=np.float32)
    for b in range(Wt.shape[3]):
        M += Wt[..., b][:, :, :, None] * V[..., b][:, :, None, :]
    chain = wg.wgrad_inverse_transform(M)
    err, ec = rel_err(got, ref), rel_err(chain, ref)
    print("%s %s: rel err %.2e, fp32 chain %.2e" % ((N, C, K), data, err, ec))
    assert err <= 1.2 * ec


def no_less_precise(w, D, E, ks, cs):
    """Every filter by itself over the channels `cs` (data and error on the GPU): its error against that of a chain of fp32
    multiply-adds over the blocks.  (Some tens of sums, over which the two vary by a third; where a sum has few blocks that count, the
    2^-24 of a product that six bf16 products leave out is as much again as the chain's half unit: 2.)"""
    torch = require_gpu()[0]
    dG, one = gradient(torch, w, D, E)
    assert one or D.shape[3] % 4 == 0
    got = dG[ks][:, cs].cpu().numpy()
    d, e = D[:, cs].cpu().numpy(), E[:, ks].cpu().numpy()
    ref = direct.conv2d_bwd_filter(d, e, pad=1)
    Wt, V = (x.astype(np.float32) for x in (wg.wgrad_error_transform(e), wg.wgrad_data_transform(d)))
    M = np.zeros((4, 4, len(ks), len(cs)), dtype=np.float32)
    for b in range(Wt.shape[3]):
        M += Wt[..., b][:, :, :, None] * V[..., b][:, :, None, :]
    chain = wg.wgrad_inverse_transform(M)
    for i, k in enumerate(ks):
        err, ec = rel_err(got[i], ref[i]), rel_err(chain[i], ref[i])
        assert err <= 2.0 * ec, "filter %d: %.2e, fp32 chain %.2e" % (k, err, ec)


# two steps per row of blocks; rows of any width in one kernel (W % 4 = 1, 2, 3); shares of more than 2048 blocks
APART = [(8, 40, 30, 32, 130), (3, 300, 20, 32, 70), (220, 40, 13, 13, 70), (220, 40, 13, 14, 70), (220, 40, 13, 15, 70),
         (30, 256, 94, 96, 250)]


@pytest.mark.parametrize("shape,bits", [(s, b) for s in APART for b in ([0, 12, 16, 20, 24, 36, 60] if s[0] != 30 else [16, 36])])
@pytest.mark.parametrize("which", ["data", "error"])
@pytest.mark.parametrize("kind", ["dark half", "zeros", "dark rows"])
def test_filter_gradient_far_apart(shape, bits, which, kind):
    """Rows whose magnitudes change from step to step, and others that see the small blocks alone.  dark half: every second step
    2^-bits; zeros: a first image 2^bits above the rest, then every second step zero; dark rows: blocks by the row of the image."""
    torch, w = require_gpu()
    N, C, H, W, K = shape
    gen = torch.Generator(device="cuda")
    gen.manual_seed(sum(shape))
    D, E = (torch.randn((N, x, H, W), generator=gen, device="cuda") for x in (C, K))
    X, Z = (D, E) if which == "data" else (E, D)                 # X has the magnitudes, every other row of Z sees the small ones alone
    half, rows = W // 2, torch.arange(H, device="cuda") // 2 % 3 == 1
    if kind == "dark half":
        X[..., half:] *= 2.0 ** -bits
        Z[:, ::2, :, :half + 2] = 0
    elif kind == "zeros":
        X[0] *= 2.0 ** bits
        X[1:, ..., :half] = 0
        Z[0, ::2] = 0
        Z[1:, ::2, :, :half + 2] = 0
    else:
        X[:, :, rows] *= 2.0 ** -bits
        X[:, :, ~rows] *= (torch.arange(X.shape[1], device="cuda") % 4 != 3)[None, :, None, None]
        Z[:, ::2] *= rows[None, None, :, None]
    ks, cs = [0, 1, 8, K // 2, K - 2], [0, 1, 3, 4, 7, C // 2, C - 1]
    no_less_precise(w, D, E, ks, cs)


@pytest.mark.parametrize("N,C,H,W,K", [(1, 16, 4096, 4096, 16), (2, 256, 1280, 1280, 16), (1, 40, 2500, 2502, 24), (1, 24, 2501, 2503, 40),
                                       (1, 20, 2502, 2501, 70)])
def test_images_of_gigabytes(N, C, H, W, K):
    """Images whose 64 planes, or that by themselves, are more than a share's buffer reaches."""
    torch, w = require_gpu()
    gen = torch.Generator(device="cuda")
    gen.manual_seed(N + C + H + W + K)
    D, E = (inside(torch, torch.randn((N, x, H, W), generator=gen, device="cuda")) for x in (C, K))
    dG, one = gradient(torch, w, D, E)
    assert one or W % 4 == 0
    ks, cs = [0, K // 2, K - 1], [0, C // 2, C - 1]
    e = E[:, ks].double().transpose(0, 1).reshape(len(ks), -1)
    ref = torch.zeros((len(ks), len(cs), 3, 3), dtype=torch.float64)
    for j, c in enumerate(cs):
        d = torch.nn.functional.pad(D[:, c].double(), (1, 1, 1, 1))
        for u in range(3):
            for v in range(3):
                ref[:, j, u, v] = (e @ d[:, u:u + H, v:v + W].reshape(-1)).cpu()
    check_close(dG[ks][:, cs].cpu().numpy(), ref.numpy(), 2e-6, "%s" % ((N, C, H, W, K),))

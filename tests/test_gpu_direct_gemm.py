"""Direct layers as a product on the matrix units, at the edges of its steps (16 taps), quads, blocks and groups."""
import numpy as np
import pytest

from oracle import direct
from gpu_util import check_close, rel_err, require_gpu, to_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "f16"])
@pytest.mark.parametrize("N,C,H,W,K,R,S,pad,stride", [
    (3, 5, 9, 11, 33, 1, 1, 0, 1),          # fewer taps than a step, blocks over several images
    (2, 16, 13, 10, 32, 1, 1, 0, 2),        # one whole step, 32 filters
    (1, 7, 12, 9, 65, 3, 3, 1, 2),          # 63 taps
    (2, 3, 17, 20, 40, 5, 3, 2, 3),         # 45 taps (odd), filters higher than wide
    (1, 6, 8, 31, 17, 2, 7, 3, 1),          # rows of taps longer than a quad, padding wider than the filter is high
    (70, 9, 3, 3, 70, 3, 3, 1, 1),          # whole images of nine pixels
    (1, 40, 14, 14, 64, 3, 3, 1, 1),        # few blocks: four groups
    (4, 24, 56, 52, 96, 3, 3, 0, 2),        # two groups
    (6, 12, 112, 100, 72, 3, 3, 1, 1),      # wide blocks
    (1, 1, 40, 520, 16, 1, 512, 4, 1),      # the longest row of taps
    (1, 150, 14, 14, 64, 3, 3, 1, 1),       # the table of taps starts again every 16 channels, groups in the middle of it
    (4, 70, 56, 52, 96, 3, 3, 0, 2),        # ... two groups
    (6, 35, 112, 100, 72, 3, 3, 1, 1),      # ... one group
    (1, 17, 30, 26, 16, 19, 17, 5, 2),      # two groups, because the table would be too large beside four
    (1, 17, 22, 40, 16, 16, 20, 5, 1),      # the largest table beside four groups
    (1, 18, 8, 518, 40, 1, 512, 2, 1),      # the largest table of all
    (2, 20, 8, 9, 40, 1, 1, 2, 1),          # windows without any part inside the image
])
def test_direct_product(N, C, H, W, K, R, S, pad, stride, dtype):
    torch, w = require_gpu()
    rng = np.random.default_rng(N + C + H + W + K + R + S)
    D = rng.standard_normal((N, C, H, W)).astype(np.float32)
    G = (rng.standard_normal((K, C, R, S)) * np.sqrt(2.0 / (C * R * S))).astype(np.float32)
    if dtype == "f16":
        D, G = D.astype(np.float16), G.astype(np.float16)
    # the tensors end where NaNs begin, and begin where NaNs end: nothing outside them may be used
    def guarded(a):
        buf = torch.full((a.size + 4096,), float("nan"), dtype=torch.from_numpy(a).dtype, device="cuda")
        buf[2048:2048 + a.size] = to_gpu(a).reshape(-1)
        return buf[2048:2048 + a.size].view(a.shape)
    Y = w.direct_conv2d_fwd(guarded(D), guarded(G), pad=pad, stride=stride).cpu().numpy()
    ref = direct.conv2d_fwd(D.astype(np.float32), G.astype(np.float32), pad=pad, stride=stride)
    # fp32: a rounding per tap at most (2^-24 each, random: under 1e-6 in norm); fp16: one rounding of Y, 2^-11 at most
    check_close(Y, ref, 1e-6 if dtype == "f32" else 4.9e-4, "direct %s" % dtype)


@pytest.mark.parametrize("data", ["positive", "near one"])
@pytest.mark.parametrize("C,H,K,R,stride,N", [
    (2100, 20, 72, 1, 1, 2),         # four groups of steps, 525 taps each
    (13000, 9, 40, 1, 1, 2),         # the same, set aside
    (13000, 9, 24, 1, 1, 2),         # 32 filters
    (677, 47, 72, 3, 1, 7),          # two groups of 3046 taps
    (700, 47, 72, 3, 1, 7),          # two groups, set aside
    (530, 47, 72, 3, 1, 10),         # one group, 4770 taps
    (240, 48, 136, 3, 1, 13),        # wide blocks, 2160 taps
    (240, 48, 20, 3, 1, 32),
])
def test_long_sums_are_as_precise_as_fp32(C, H, K, R, stride, N, data):
    """Small products must not be lost against a large sum; operands between 1 and 1 + 2^-7 have those of one sign."""
    torch, w = require_gpu()
    rng = np.random.default_rng(C + H + K + R)
    make = (lambda *s: (1.0 + rng.random(s) * 2.0 ** -7).astype(np.float32)) if data == "near one" else \
           (lambda *s: rng.random(s).astype(np.float32))
    D, G = make(N, C, H, H), make(K, C, R, R)
    Y = w.direct_conv2d_fwd(to_gpu(D), to_gpu(G), pad=0, stride=stride).cpu().numpy()
    pts = np.array([[n, k, x, y] for n in (0, N - 1) for k in range(0, K, 5) for x in (0, H // 2 - R) for y in (1, H // 2 - R)], dtype=np.int32)
    ref = direct.conv2d_points(D, G, pts, pad=0, stride=stride)
    chain = np.zeros(len(pts), dtype=np.float32)                # fp32 multiply-adds in tap order (rounded twice)
    for c in range(C):
        for u in range(R):
            for v in range(R):
                chain += D[pts[:, 0], c, pts[:, 2] * stride + u, pts[:, 3] * stride + v] * G[pts[:, 1], c, u, v]
    e, ec = rel_err(Y[tuple(pts.T)], ref), rel_err(chain, ref)
    print("%s %s: rel err %.2e, fp32 chain %.2e" % ((C, H, K, R, N), data, e, ec))
    assert e <= ec


@pytest.mark.parametrize("N,C,H,W,K,R,pad,stride,bound", [
    (1, 16, 28, 28, 64, 3, 1, 2, 9.2e-8),        # nine steps: groups of 2, 2, 2, 3 are 8.8e-8 off, of 3, 3, 3, 0 9.8e-8
    (10, 3, 79, 31, 34, 7, 0, 2, 9.6e-8),        # ten: 9.2e-8, of 3, 3, 3, 1 1.01e-7
    (1, 23, 40, 40, 30, 3, 1, 2, 1.1e-7),        # thirteen: 1.06e-7, of 4, 4, 4, 1 1.15e-7
])
def test_groups_share_the_steps_evenly(N, C, H, W, K, R, pad, stride, bound):
    """The error grows with the longest sums of the four groups (N(0,1) data; measured on other seeds, which differ by 1 %)."""
    torch, w = require_gpu()
    err = []
    for seed in range(3):
        rng = np.random.default_rng(seed)
        D, G = rng.standard_normal((N, C, H, W)).astype(np.float32), rng.standard_normal((K, C, R, R)).astype(np.float32)
        Y = w.direct_conv2d_fwd(to_gpu(D), to_gpu(G), pad=pad, stride=stride).cpu().numpy()
        err.append(rel_err(Y, direct.conv2d_fwd(D, G, pad=pad, stride=stride)))
    print("rel err %s" % err)
    assert np.sqrt(np.mean(np.square(err))) <= bound

"""Filter gradient in one kernel on the bf16 matrix units, at the edges of its steps (8 blocks), rows of blocks, 64 x 64
blocks of M and shares; and its rounding over many shares."""
import numpy as np
import pytest

from oracle import direct
from paper_1509_09308_amd import synth
from gpu_util import check_close, require_gpu, to_gpu

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


def test_rounding_does_not_add_up_over_shares():
    """Positive data: every product of the first component grows the sums, the case in which a rounding that always goes
    one way shows most.  fp32 sums of n terms rounded to nearest stay within sqrt(n) 2^-24 of a share's sum."""
    torch, w = require_gpu()
    N, C, H, W, K = 4, 64, 112, 112, 64
    rng = np.random.default_rng(1)
    D = rng.uniform(0.0, 1.0, (N, C, H, W)).astype(np.float32)
    E = rng.uniform(0.0, 1.0, (N, K, H, W)).astype(np.float32)
    dG = w.wino_conv2d_bwd_filter(to_gpu(D), to_gpu(E), pad=1).cpu().numpy()
    pts = np.array([[k, c, u, v] for k in (0, 31, 63) for c in (0, 40, 63) for u in range(3) for v in range(3)], dtype=np.int32)
    ref = direct.conv2d_bwd_filter_points(D, E, pts, pad=1)
    e = np.linalg.norm(dG[tuple(pts.T)] - ref) / np.linalg.norm(ref)
    print("rel err %.2e" % e)
    assert e <= 1e-6

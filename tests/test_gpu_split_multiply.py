"""fp32 products on the bf16 matrix units (every value the exact sum of three bf16 values, six of the nine products):
no less precise than a chain of fp32 multiply-adds, at the edges of the multiply's slabs, blocks and shares."""
import numpy as np
import pytest

from oracle import winograd as wg
from gpu_util import require_gpu, rel_err

pytestmark = pytest.mark.gpu


# (K, C, P): 128 x 128 blocks of 16-channel slabs (odd and even number of slabs, ragged edges), the narrow blocks with
# 32-channel slabs whose last one is half empty
@pytest.mark.parametrize("K,C,P", [(256, 16, 3600), (256, 48, 3600), (200, 64, 3300), (128, 48, 130), (70, 80, 300),
                                   (40, 112, 100)])
@pytest.mark.parametrize("spread", [0, 6, "low parts"])
def test_multiply_is_as_precise_as_fp32(K, C, P, spread):
    torch, w = require_gpu()
    m, a = 2, 4
    worst = spread == "low parts"
    spread = 0 if worst else spread
    rng = np.random.default_rng(K + C + P + spread)
    # `spread`: magnitudes over 2^+-spread, so that the parts of the values meet in every combination of orders
    u = (rng.standard_normal((a, a, K, C)) * 2.0 ** rng.integers(-spread, spread + 1, (a, a, K, C))).astype(np.float32)
    v = (rng.standard_normal((a, a, C, P)) * 2.0 ** rng.integers(-spread, spread + 1, (a, a, C, P))).astype(np.float32)
    if worst:       # operands whose products of parts that are left out are as large as they can be, 2^-24 of the product
        u, v = np.sign(u) * np.float32(1 + 2.0 ** -8 - 2.0 ** -17), np.sign(v) * np.float32(1 + 2.0 ** -8 - 2.0 ** -17)
    M = w.unpack_m(w.wino_batched_gemm(w.pack_u(u, m), w.pack_v(v, m), K, C, P, m), K, P, m)
    ref = wg.multiply(u.astype(np.float64), v.astype(np.float64))
    # every term may be off by the products left out (2^-24 of it), every sum by six accumulations per 16 channels, each
    # off by a unit in the last place of what it holds (2^-23) at most
    bound = (1 + 12 * -(-C // 16)) * 2.0 ** -24 * wg.multiply(np.abs(u).astype(np.float64), np.abs(v).astype(np.float64))
    assert (np.abs(M - ref) <= bound).all()
    if worst:
        return
    chain = np.zeros((a, a, K, P), dtype=np.float32)            # fp32 multiply-adds in channel order (rounded twice)
    for c in range(C):
        chain += u[:, :, :, c, None] * v[:, :, None, c, :]
    e, ec = rel_err(M, ref), rel_err(chain, ref)
    print("K=%d C=%d P=%d spread %d: rel err %.2e, fp32 chain %.2e" % (K, C, P, spread, e, ec))
    assert e <= 1.2 * ec


def test_multiply_shares_of_sixteen_channels():
    """A channel sum split between workgroups whose shares end inside a 32-channel slab: the layer adds them up."""
    torch, w = require_gpu()
    from oracle import direct
    from paper_1509_09308_amd import synth
    from gpu_util import TOL, check_close, to_gpu
    N, C, HW, K = 1, 96, 10, 64
    assert w.wino_gemm_launch_shape(K, C, 25, 2)[2] > 1
    D, G = synth.make_layer(N, C, HW, HW, K, seed=96)
    Y = w.wino_conv2d_fwd_ex(to_gpu(D), G=to_gpu(G), pad=1, m=2, flags=w.FLAG_UNFUSED).cpu().numpy()
    check_close(Y, direct.conv2d_fwd(D, G, pad=1), TOL[("f32", 2)], "three slabs in two shares", 2)


@pytest.mark.parametrize("C", [16, 48])
def test_multiply_of_many_tiles(C):
    """Components of V up to 4 GiB are taken: a pipeline's requests past the last slab must not count."""
    torch, w = require_gpu()
    K, P, m = 32, 14000000, 2               # one component of V is 0.9 GB (C = 16) or 2.7 GB, all of them 14 or 43 GB
    Kp, Cp, Pp = w.wino_padded_dims(K, C, P, m)
    assert Cp * Pp * 4 < 2 ** 32 <= (Cp + 64) * Pp * 4
    U = torch.randint(-3, 4, (16, Cp, Kp), device="cuda").float()
    V = torch.empty((16, Cp, Pp), device="cuda")
    b = torch.arange(Pp, device="cuda")
    for c in range(Cp):
        row = ((b * (2 * c + 1) + c * c) % 7 - 3).float()
        for e in range(16):
            V[e, c] = row if e % 2 else -row
    M = w.wino_batched_gemm(U.reshape(-1), V.reshape(-1), K, C, P, m).view(16, Kp, Pp)
    for e in range(16):
        for p in range(0, P, 3000000):      # whole numbers below 2^24: exact in any order
            assert torch.equal(M[e, :, p:min(p + 3000000, P)], U[e].t().contiguous() @ V[e, :, p:min(p + 3000000, P)])


def near_one(rng, *shape):
    """Values between 1 and 1 + 2^-7: the products of their low parts have one sign."""
    return (1.0 + rng.random(shape) * 2.0 ** -7).astype(np.float32)


@pytest.mark.parametrize("data", ["positive", "near one"])
@pytest.mark.parametrize("K,C,P", [(40, 2048, 40), (40, 2100, 40), (130, 3100, 1000), (40, 20000, 40)])
def test_long_sums_are_as_precise_as_fp32(K, C, P, data):
    """Small products must not be lost against a large sum."""
    torch, w = require_gpu()
    m, a = 2, 4
    rng = np.random.default_rng(K + C + P)
    make = near_one if data == "near one" else (lambda r, *shape: r.random(shape).astype(np.float32))
    u, v = make(rng, 1, 1, K, C), make(rng, 1, 1, C, P)
    full = lambda x: np.broadcast_to(x, (a, a) + x.shape[2:])
    M = w.unpack_m(w.wino_batched_gemm(w.pack_u(full(u), m), w.pack_v(full(v), m), K, C, P, m), K, P, m)
    assert (M == M[:1, :1]).all()
    ref = u[0, 0].astype(np.float64) @ v[0, 0].astype(np.float64)
    chain = np.zeros((K, P), dtype=np.float32)                  # fp32 multiply-adds in channel order (rounded twice)
    for c in range(C):
        chain += u[0, 0, :, c, None] * v[0, 0, None, c, :]
    e, ec = rel_err(M[0, 0], ref), rel_err(chain, ref)
    print("K=%d C=%d P=%d %s: rel err %.2e, fp32 chain %.2e" % (K, C, P, data, e, ec))
    assert e <= ec


@pytest.mark.parametrize("K,P", [(40, 100), (200, 3300)])
@pytest.mark.parametrize("C", [1, 2, 3])
def test_few_channels(K, P, C):
    torch, w = require_gpu()
    rng = np.random.default_rng(K + C)
    u, v = rng.standard_normal((4, 4, K, C)).astype(np.float32), rng.standard_normal((4, 4, C, P)).astype(np.float32)
    M = w.unpack_m(w.wino_batched_gemm(w.pack_u(u, 2), w.pack_v(v, 2), K, C, P, 2), K, P, 2)
    if C == 1:
        assert np.array_equal(M, u * v)          # a single product, rounded to nearest
    ref = wg.multiply(u.astype(np.float64), v.astype(np.float64))
    chain = u[..., :1] * v[:, :, :1]                            # fp32 multiply-adds, every sum rounded once
    for c in range(1, C):
        chain = (chain.astype(np.float64) + u[..., c, None].astype(np.float64) * v[:, :, None, c]).astype(np.float32)
    e, ec = rel_err(M, ref), rel_err(chain, ref)
    print("C=%d: rel err %.2e, fp32 chain %.2e" % (C, e, ec))
    assert e <= 1.01 * ec

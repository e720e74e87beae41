"""fp32 entry points over the whole range of fp32 values: tiny, huge and infinite ones give what chains of fp32
multiply-adds give, and the sums that such a value does not enter keep their bits."""
import numpy as np
import pytest

from oracle import direct
from oracle import winograd as wg
from paper_1509_09308_amd import synth
from gpu_util import TOL, rel_err, require_gpu, to_gpu

pytestmark = pytest.mark.gpu

FLT_MAX = np.finfo(np.float32).max
# (scale of the first operand, of the second): the low bits of a tiny operand lie below what a bf16 part of it can hold;
# products of the huge ones, and sums of those, stay within fp32
SCALES = {"tiny data": (2.0 ** -118, 2.0 ** 20), "tiny filters": (2.0 ** 20, 2.0 ** -118), "subnormal data": (2.0 ** -132, 2.0 ** 40),
          "huge data": (2.0 ** 112, 2.0 ** -30), "huge filters": (2.0 ** -30, 2.0 ** 112)}


def scaled(a, s):
    return (a.astype(np.float64) * s).astype(np.float32)


def check(got, ref, tol, what):
    """The same infinities and NaNs, everything else within `tol` in norm."""
    got, ref = np.asarray(got, dtype=np.float64), np.asarray(ref, dtype=np.float64)
    assert (np.isnan(got) == np.isnan(ref)).all(), "%s: %d NaNs, expected %d" % (what, np.isnan(got).sum(), np.isnan(ref).sum())
    inf = np.isinf(ref)
    assert (np.isinf(got) == inf).all() and (got[inf] == ref[inf]).all(), what
    ok = np.isfinite(ref)
    e = rel_err(got[ok], ref[ok])
    print("%s: rel err %.2e" % (what, e))
    assert e <= tol, "%s: %.3e > %.1e" % (what, e, tol)


def terms(mat, x, axis):
    """mat x along `axis` as the kernels form it: coefficients of zero stand for no term at all."""
    x = np.moveaxis(x, axis, 0)
    out = []
    for row in np.asarray(mat, dtype=np.float64):
        out.append(sum(float(c) * x[j] for j, c in enumerate(row) if c != 0))
    return np.moveaxis(np.stack(out), 0, axis)


# ---- direct layers ------------------------------------------------------------------------------

DIRECT = [(2, 16, 13, 10, 32, 1, 1, 0, 2), (1, 40, 14, 14, 64, 3, 3, 1, 1), (4, 24, 56, 52, 96, 3, 3, 0, 2),
          (6, 12, 112, 100, 72, 3, 3, 1, 1)]     # one step; four groups of steps, two, one with wide blocks


def direct_layer(shape):
    N, C, H, W, K, R, S, pad, stride = shape
    rng = np.random.default_rng(sum(shape))
    return (rng.standard_normal((N, C, H, W)).astype(np.float32),
            (rng.standard_normal((K, C, R, S)) * np.sqrt(2.0 / (C * R * S))).astype(np.float32), dict(pad=pad, stride=stride))


@pytest.mark.parametrize("shape", DIRECT)
@pytest.mark.parametrize("scale", list(SCALES))
def test_direct_scaled(shape, scale):
    torch, w = require_gpu()
    D, G, kw = direct_layer(shape)
    D, G = scaled(D, SCALES[scale][0]), scaled(G, SCALES[scale][1])
    Y = w.direct_conv2d_fwd(to_gpu(D), to_gpu(G), **kw).cpu().numpy()
    check(Y, direct.conv2d_fwd(D, G, **kw), 1e-6, "direct %s %s" % (shape, scale))


@pytest.mark.parametrize("shape", DIRECT)
@pytest.mark.parametrize("value", [np.inf, -np.inf, FLT_MAX, -FLT_MAX, np.nan])
def test_direct_single_values(shape, value):
    torch, w = require_gpu()
    D, G, kw = direct_layer(shape)
    G *= 2.0 ** -6
    g = to_gpu(G)
    plain = w.direct_conv2d_fwd(to_gpu(D), g, **kw).cpu().numpy()
    for at in ((0, 0, 0, 0), (-1, -1, 6, 4), (-1, shape[1] // 2, 3, -1)):
        X = D.copy()
        X[at] = value
        Y = w.direct_conv2d_fwd(to_gpu(X), g, **kw).cpu().numpy()
        ref = direct.conv2d_fwd(X, G, **kw)
        check(Y, ref, 1e-6, "direct %s, %g at %s" % (shape, value, at))
        X[at] = np.nan
        out = ~np.isnan(direct.conv2d_fwd(X, G, **kw))
        assert (Y[out] == plain[out]).all()


# ---- the multiply -------------------------------------------------------------------------------

GEMM = [(40, 16, 100), (200, 16, 3300), (70, 80, 300), (256, 48, 3600)]     # one slab, several; 64- and 128-wide blocks


def gemm_operands(K, C, P):
    rng = np.random.default_rng(K + C + P)
    return rng.standard_normal((4, 4, K, C)).astype(np.float32), rng.standard_normal((4, 4, C, P)).astype(np.float32)


def gemm(w, u, v):
    K, C, P = u.shape[2], u.shape[3], v.shape[3]
    return w.unpack_m(w.wino_batched_gemm(w.pack_u(u, 2), w.pack_v(v, 2), K, C, P, 2), K, P, 2)


@pytest.mark.parametrize("K,C,P", GEMM)
@pytest.mark.parametrize("scale", list(SCALES))
def test_multiply_scaled(K, C, P, scale):
    torch, w = require_gpu()
    u, v = gemm_operands(K, C, P)
    u, v = scaled(u, SCALES[scale][1]), scaled(v, SCALES[scale][0])
    check(gemm(w, u, v), wg.multiply(u.astype(np.float64), v.astype(np.float64)), 1e-6, "multiply %s %s" % ((K, C, P), scale))


@pytest.mark.parametrize("K,C,P", GEMM)
@pytest.mark.parametrize("value", [np.inf, FLT_MAX, -FLT_MAX, np.nan])
def test_multiply_single_values(K, C, P, value):
    torch, w = require_gpu()
    u, v = gemm_operands(K, C, P)
    u *= 2.0 ** -6
    plain = gemm(w, u, v)
    x = v.copy()
    x[1, 2, C - 1, P - 3] = value
    x[3, 0, 0, 5] = value
    got = gemm(w, u, x)
    check(got, wg.multiply(u.astype(np.float64), x.astype(np.float64)), 1e-6, "multiply %s, %g" % ((K, C, P), value))
    rest = np.ones_like(got, dtype=bool)
    rest[1, 2, :, P - 3] = rest[3, 0, :, 5] = False
    assert (got[rest] == plain[rest]).all()


# ---- one-kernel layers --------------------------------------------------------------------------

# 132 items; a full round and 15 items per XCD in two shares; F(2x2,3x3): whole items; a shared last round
LAYERS = [(4, (20, 17, 28, 60, 70)), (4, (17, 128, 28, 44, 513)), (2, (13, 17, 30, 46, 70)), (2, (6, 256, 48, 60, 400))]


def points_check(w, torch, D, G, Y, m, tol, what):
    pts = synth.sample_points(Y.shape, 2000, seed=5, edge=m)
    check(Y[tuple(pts.T)], direct.conv2d_points(D, G, pts, pad=1), tol, what)


@pytest.mark.parametrize("m,shape", LAYERS)
@pytest.mark.parametrize("given", ["G", "U"])
@pytest.mark.parametrize("scale", ["tiny data", "tiny filters", "huge data", "huge filters"])
def test_layer_scaled(m, shape, given, scale):
    torch, w = require_gpu()
    N, C, H, W, K = shape
    D, G = synth.make_layer(N, C, H, W, K, seed=sum(shape) + m)
    D, G = scaled(D, SCALES[scale][0]), scaled(G, SCALES[scale][1])
    g = to_gpu(G)
    kw = dict(G=g) if given == "G" else dict(U=w.wino_filter_transform(g, m), K=K)
    Y = w.wino_conv2d_fwd_ex(to_gpu(D), pad=1, m=m, flags=w.FLAG_FUSED, **kw)
    Y2 = w.wino_conv2d_fwd_ex(to_gpu(D), pad=1, m=m, flags=w.FLAG_FUSED, **kw)
    assert torch.equal(Y, Y2)
    points_check(w, torch, D, G, Y.cpu().numpy(), m, TOL[("f32", m)], "F(%d) %s %s %s" % (m, shape, given, scale))


def wino_layer(D, G, m, image):
    """One image by the definition of the algorithm, on terms as the kernels form them."""
    Bt, Gm, At = (np.array(x, dtype=np.float64) for x in wg.matrices(m))
    C, H, W = D.shape[1:]
    Th, Tw = -(-H // m), -(-W // m)
    d = np.zeros((C, Th * m + 2, Tw * m + 2))
    d[:, 1:H + 1, 1:W + 1] = D[image]
    tiles = np.stack([np.stack([d[:, m * x:m * x + m + 2, m * y:m * y + m + 2] for y in range(Tw)]) for x in range(Th)])
    v = terms(Bt, terms(Bt, tiles, 3), 4)                         # [Th][Tw][C][a][a]
    u = terms(Gm, terms(Gm, G.astype(np.float64), 2), 3)          # [K][C][a][a]
    M = np.zeros((G.shape[0], Th, Tw, m + 2, m + 2))
    for c in range(C):
        M += u[:, c, None, None] * v[None, :, :, c]
    y = terms(At, terms(At, M, 3), 4)                             # [K][Th][Tw][m][m]
    return y.transpose(0, 1, 3, 2, 4).reshape(G.shape[0], Th * m, Tw * m)[:, :H, :W]


@pytest.mark.parametrize("m,shape", [(4, (20, 17, 28, 60, 70)), (2, (13, 17, 30, 46, 70))])
@pytest.mark.parametrize("value", [np.inf, -np.inf, FLT_MAX, np.nan])
def test_layer_single_values(m, shape, value):
    torch, w = require_gpu()
    N, C, H, W, K = shape
    if m == 4 and value == FLT_MAX:
        value = np.float32(2.0 ** 120)                            # (16 times FLT_MAX, which the transform forms, is infinite)
    D, G = synth.make_layer(N, C, H, W, K, seed=sum(shape) + m)
    G *= np.float32(2.0 ** -6)
    g = to_gpu(G)
    plain = w.wino_conv2d_fwd_ex(to_gpu(D), G=g, pad=1, m=m, flags=w.FLAG_FUSED).cpu().numpy()
    for at in ((0, 0, 0, 0), (N - 1, C - 1, H - 1, W - 1), (4, 3, 13, 31)):
        X = D.copy()
        X[at] = value
        Y = w.wino_conv2d_fwd_ex(to_gpu(X), G=g, pad=1, m=m, flags=w.FLAG_FUSED).cpu().numpy()
        with np.errstate(invalid="ignore"):
            check(Y[at[0]], wino_layer(X, G, m, at[0]), TOL[("f32", m)], "F(%d) %s, %g at %s" % (m, shape, value, at))
        X[at] = np.nan
        out = np.ones(Y.shape, dtype=bool)
        out[at[0]] = ~np.isnan(wino_layer(X, G, m, at[0]))
        assert (Y[out] == plain[out]).all()


def test_layer_single_value_in_a_shared_item():
    """The last round's items of this layer are summed from shares of their channels: an infinite value in the last tile."""
    torch, w = require_gpu()
    m, (N, C, H, W, K) = 2, (6, 256, 48, 60, 400)
    D, G = synth.make_layer(N, C, H, W, K, seed=11)
    g = to_gpu(G)
    plain = w.wino_conv2d_fwd_ex(to_gpu(D), G=g, pad=1, m=m, flags=w.FLAG_FUSED).cpu().numpy()
    D[N - 1, 200, H - 1, W - 1] = np.inf
    Y = w.wino_conv2d_fwd_ex(to_gpu(D), G=g, pad=1, m=m, flags=w.FLAG_FUSED).cpu().numpy()
    near = np.zeros(Y.shape, dtype=bool)
    near[N - 1, :, H - 2:, W - 2:] = True
    assert (Y[~near] == plain[~near]).all()
    with np.errstate(invalid="ignore"):
        ref = wino_layer(D[:, :, H - 8:, W - 8:], G, m, N - 1)[:, -2:, -2:]
    check(Y[N - 1, :, -2:, -2:], ref, TOL[("f32", m)], "shared item")


# ---- filter gradient ----------------------------------------------------------------------------

WGRAD = [(5, 70, 9, 20, 130), (3, 320, 28, 28, 288),
         (220, 40, 13, 13, 70), (220, 40, 13, 14, 70), (220, 40, 13, 15, 70)]      # W % 4 = 1, 2, 3: 110 MB and more transformed


@pytest.mark.parametrize("N,C,H,W,K", WGRAD)
@pytest.mark.parametrize("scale", list(SCALES))
def test_filter_gradient_scaled(N, C, H, W, K, scale):
    torch, w = require_gpu()
    rng = np.random.default_rng(N + C + H + W + K)
    D = scaled(rng.standard_normal((N, C, H, W)), SCALES[scale][0])
    E = scaled(rng.standard_normal((N, K, H, W)), SCALES[scale][1])
    dG = w.wino_conv2d_bwd_filter(to_gpu(D), to_gpu(E), pad=1).cpu().numpy()
    check(dG, direct.conv2d_bwd_filter(D, E, pad=1), 1e-5, "filter gradient %s %s" % ((N, C, H, W, K), scale))


@pytest.mark.parametrize("value", [np.inf, FLT_MAX, np.nan])
@pytest.mark.parametrize("which", ["data", "error"])
@pytest.mark.parametrize("shape,at", [((5, 70, 9, 20, 130), (4, 7)),
                                      # W % 4 = 1, 2, 3 in one kernel (110 MB and more transformed): the last column of a row, the
                                      # first of the next
                                      ((220, 40, 13, 13, 70), (4, 12)), ((220, 40, 13, 13, 70), (5, 0)),
                                      ((220, 40, 13, 14, 70), (4, 13)), ((220, 40, 13, 14, 70), (5, 0)),
                                      ((220, 40, 13, 15, 70), (4, 14)), ((220, 40, 13, 15, 70), (12, 14))])
def test_filter_gradient_single_values(value, which, shape, at):
    torch, w = require_gpu()
    N, C, H, W, K = shape
    rng = np.random.default_rng(7)
    D = rng.standard_normal((N, C, H, W)).astype(np.float32)
    E = (rng.standard_normal((N, K, H, W)) * 2.0 ** -6).astype(np.float32)
    if which == "error":
        D, E = (D * 2.0 ** -6).astype(np.float32), (E * 2.0 ** 6).astype(np.float32)
    plain = w.wino_conv2d_bwd_filter(to_gpu(D), to_gpu(E), pad=1).cpu().numpy()
    line = min(66, C - 4) if which == "data" else 66
    (D if which == "data" else E)[(3, line) + at] = value
    dG = w.wino_conv2d_bwd_filter(to_gpu(D), to_gpu(E), pad=1).cpu().numpy()
    rest = np.ones(dG.shape, dtype=bool)
    if which == "data":
        rest[:, line] = False
    else:
        rest[line] = False
    assert (dG[rest] == plain[rest]).all()
    Bt, Gm, At = (np.array(x, dtype=np.float64) for x in wg.matrices(3, 2))
    d = np.zeros((N, C, H + 3, W + 3))
    d[:, :, 1:H + 1, 1:W + 1] = D
    e = np.zeros((N, K, H + 1, W + 1))
    e[:, :, :H, :W] = E
    if which == "data":
        d = d[:, line:line + 1]
    else:
        e = e[:, line:line + 1]
    bx, by = (H + 1) // 2, (W + 1) // 2
    tiles = np.stack([d[:, :, 2 * x:2 * x + 4, 2 * y:2 * y + 4] for x in range(bx) for y in range(by)])
    blocks = np.stack([e[:, :, 2 * x:2 * x + 2, 2 * y:2 * y + 2] for x in range(bx) for y in range(by)])
    with np.errstate(invalid="ignore"):
        v, u = terms(Bt, terms(Bt, tiles, 3), 4), terms(Gm, terms(Gm, blocks, 3), 4)     # [b][n][c or k][4][4]
        M = np.zeros((u.shape[2], v.shape[2], 4, 4))
        for b in range(bx * by):
            for n in range(N):
                M += u[b, n][:, None] * v[b, n][None]
        ref = terms(At, terms(At, M, 2), 3)
    got = dG[:, line:line + 1] if which == "data" else dG[line:line + 1]
    check(got, ref, 1e-5, "filter gradient, %g in the %s" % (value, which))

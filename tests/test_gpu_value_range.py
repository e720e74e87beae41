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


# ---- filter gradient ----------------------------------------------------------------------------

WGRAD = [(5, 70, 9, 20, 130), (3, 320, 28, 28, 288)]


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
def test_filter_gradient_single_values(value, which):
    torch, w = require_gpu()
    N, C, H, W, K = 5, 70, 9, 20, 130
    rng = np.random.default_rng(7)
    D = rng.standard_normal((N, C, H, W)).astype(np.float32)
    E = (rng.standard_normal((N, K, H, W)) * 2.0 ** -6).astype(np.float32)
    if which == "error":
        D, E = (D * 2.0 ** -6).astype(np.float32), (E * 2.0 ** 6).astype(np.float32)
    plain = w.wino_conv2d_bwd_filter(to_gpu(D), to_gpu(E), pad=1).cpu().numpy()
    line = 66
    (D if which == "data" else E)[3, line, 4, 7] = value
    dG = w.wino_conv2d_bwd_filter(to_gpu(D), to_gpu(E), pad=1).cpu().numpy()
    rest = np.ones(dG.shape, dtype=bool)
    if which == "data":
        rest[:, line] = False
    else:
        rest[line] = False
    assert (dG[rest] == plain[rest]).all()
    Bt, Gm, At = (np.array(x, dtype=np.float64) for x in wg.matrices(3, 2))
    d = np.zeros((N, C, H + 3, W + 2))
    d[:, :, 1:H + 1, 1:W + 1] = D
    e = np.zeros((N, K, H + 1, W))
    e[:, :, :H] = E
    if which == "data":
        d = d[:, line:line + 1]
    else:
        e = e[:, line:line + 1]
    bx, by = (H + 1) // 2, W // 2
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

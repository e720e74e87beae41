"""The work that performance is measured on: calls of the public entry points as a user's program makes them.

Sizes are those of the repository's own workloads (the 3x3 layers of VGG-16 at batch 1, 32 and 64, the 512 -> 512 layer
at 28 x 28 and batch 8, the 32 -> 32 layer at 56 x 56) and generic ones of the same ranges, odd extents among them.
Data is N(0,1), filters are He-scaled, as everywhere in this repository.

Kinds of case:
  layer       one forward layer from untransformed filters, caller-owned workspace and output
  layer_fx    the same with filters transformed once ahead of the calls (weights that do not change)
  short       one forward layer through the entry point that owns its workspace and allocates its output
  bwd_data    gradient with respect to the input
  bwd_filter  gradient with respect to the filters
  direct      a layer that the fast algorithm does not cover
  stack       the 13 layers of the stack forward, each on its own data
  train       the 13 layers forward and both their gradients
"""
import math

import torch

import paper_1509_09308_amd as w
from paper_1509_09308_amd import synth

DTYPES = {"f32": (torch.float32, w.WINO_F32), "f16": (torch.float16, w.WINO_F16)}


def _layer(name, kind, N, C, H, W, K, m, pad=1, dtype="f32", y="f32"):
    return {"name": name, "kind": kind, "N": N, "C": C, "H": H, "W": W, "K": K, "m": m, "pad": pad, "dtype": dtype, "y": y}


def _direct(name, N, C, H, W, K, R, S, pad, stride, dtype="f32"):
    return {"name": name, "kind": "direct", "N": N, "C": C, "H": H, "W": W, "K": K, "R": R, "S": S, "pad": pad,
            "stride": stride, "dtype": dtype}


def listed():
    return [
        # the smallest layer of the workloads, one image: a call whose latency is all that counts
        _layer("small_n1", "short", 1, 32, 56, 56, 32, 2),
        # one image through the whole stack: interactive inference
        {"name": "stack_n1", "kind": "stack", "N": 1, "dtype": "f32", "policy": "n1"},
        # an ordinary layer at a small batch, both algorithms
        _layer("layer_n8_f4", "layer", 8, 512, 28, 28, 512, 4),
        _layer("layer_n8_f2", "layer", 8, 512, 28, 28, 512, 2),
        # inference with fixed weights at an ordinary batch
        _layer("fixed_weights_n16", "layer_fx", 16, 256, 56, 56, 256, 4),
        # extents that divide nothing, no padding: crops, pyramids, other people's networks
        _layer("ragged_n6", "layer", 6, 100, 45, 37, 150, 4, pad=0),
        # the headline: the stack at batch 64 in fp32
        {"name": "stack_n64", "kind": "stack", "N": 64, "dtype": "f32", "policy": "auto"},
        # the stack at batch 32 with fp16 storage
        {"name": "stack_n32_f16", "kind": "stack", "N": 32, "dtype": "f16", "policy": "4"},
        # half-precision layer of an odd width, fp16 in and out
        _layer("ragged_n5_f16", "layer", 5, 96, 30, 30, 160, 4, dtype="f16", y="f16"),
        # a training step of the stack: forward, input gradient, filter gradient
        {"name": "train_n16", "kind": "train", "N": 16, "dtype": "f32", "policy": "auto"},
        # the filter gradient of a wide layer at the batch where training is measured
        _layer("filter_grad_n64", "bwd_filter", 64, 256, 56, 56, 256, 2),
        # a downsampling layer: stride 2 is outside the fast algorithm
        _direct("direct_stride2_n16", 16, 64, 56, 56, 128, 3, 3, 1, 2),
    ]


# ---- drawn cases --------------------------------------------------------------------------------

MAX_LAYER_FLOPS = 2.5e11          # direct-convolution flops; the largest listed case has 1.96e12
MAX_DIRECT_FLOPS = 4.0e10
MAX_ELEMENTS = 2.2e8              # of the larger of input and output


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _extent(rng, lo, hi, q):
    """An extent spread over [lo, hi] on a log scale; two times in three a multiple of q, as networks have them."""
    x = _log_int(rng, lo, hi)
    if rng.random() < 0.67:
        x = max(q, (x + q // 2) // q * q)
    return x


def draw(rng):
    kind = rng.choice(["layer", "layer", "layer", "layer_fx", "short", "bwd_data", "bwd_filter", "direct", "stack"])
    if kind == "stack":
        dtype = rng.choice(["f32", "f16"])
        return {"kind": "stack", "N": _log_int(rng, 1, 48), "dtype": dtype,
                "policy": rng.choice(["auto", "n1", "2", "4"] if dtype == "f32" else ["4", "2"])}
    while True:
        N = _log_int(rng, 1, 64)
        C, K = _extent(rng, 8, 640, 16), _extent(rng, 16, 640, 16)
        H = _extent(rng, 7, 226, 4)
        W = H if rng.random() < 0.6 else _extent(rng, 7, 226, 4)
        if kind == "direct":
            if rng.random() < 0.4:
                C = rng.choice([1, 3, 4])
            R = rng.choice([1, 3, 3, 5, 7])
            stride = rng.choice([1, 2]) if R != 3 or C > 4 else rng.choice([1, 1, 2])
            pad = rng.choice([0, R // 2])
            Ho, Wo = (H + 2 * pad - R) // stride + 1, (W + 2 * pad - R) // stride + 1
            flops, limit = 2.0 * N * K * C * R * R * Ho * Wo, MAX_DIRECT_FLOPS
        else:
            Ho, Wo = H, W
            flops, limit = 18.0 * N * K * C * H * W, MAX_LAYER_FLOPS
        # a call of some microseconds at least, no larger than the listed ones
        if flops < 2e7 or flops > limit or N * max(C * H * W, K * Ho * Wo) > MAX_ELEMENTS:
            continue
        if kind == "direct":
            c = _direct("", N, C, H, W, K, R, R, pad, stride, rng.choice(["f32", "f32", "f16"]))
        else:
            m = rng.choice([2, 4, 4, 4, 6])
            dtype = y = "f32"
            if kind in ("layer", "layer_fx", "bwd_data") and m != 6 and rng.random() < 0.35:
                dtype, y = "f16", rng.choice(["f32", "f16"])
            if kind == "bwd_filter":
                m = 2
            pad = 0 if kind in ("layer", "layer_fx", "short") and rng.random() < 0.2 else 1
            c = _layer("", kind, N, C, H, W, K, m, pad, dtype, y)
        del c["name"]
        return c


# ---- one case -----------------------------------------------------------------------------------

def _stack_m(HW, policy):
    """The algorithms the workloads name: F(4x4) where 4 divides the image, else F(2x2); for one image F(2x2) from
    28 x 28 down; or one for all layers."""
    if policy == "auto":
        return 4 if HW % 4 == 0 else 2
    if policy == "n1":
        return 4 if HW % 4 == 0 and HW > 28 else 2
    return int(policy)


def _stack(case):
    for i, (name, C, HW, K) in enumerate(synth.VGG16_LAYERS):
        yield i, C, HW, K, _stack_m(HW, case["policy"])


class _Random:
    def __init__(self, seed):
        self.gen = torch.Generator(device="cuda")
        self.gen.manual_seed(seed)

    def normal(self, shape, dtype, scale=1.0):
        x = torch.randn(shape, generator=self.gen, device="cuda", dtype=torch.float32)
        return (x * scale).to(dtype) if scale != 1.0 or dtype != torch.float32 else x

    def filters(self, K, C, R, S, dtype):
        return self.normal((K, C, R, S), dtype, math.sqrt(2.0 / (R * S * C)))


def prepare(case, seed):
    rnd = _Random(seed)
    tdt, dt = DTYPES[case["dtype"]]
    N = case["N"]
    if case["kind"] in ("stack", "train"):
        layers, need = [], 0
        for i, C, HW, K, m in _stack(case):
            L = {"m": m, "direct": C < 16, "D": rnd.normal((N, C, HW, HW), tdt), "G": rnd.filters(K, C, 3, 3, tdt)}
            L["Y"] = torch.empty((N, K, HW, HW), dtype=tdt if L["direct"] else torch.float32, device="cuda")
            if not L["direct"]:
                need = max(need, w.wino_workspace_bytes(N, C, HW, HW, K, 1, m, dt))
            if case["kind"] == "train":
                L["E"] = rnd.normal((N, K, HW, HW), tdt)
                L["dG"] = torch.empty_like(L["G"])
                need = max(need, w.wino_bwd_filter_workspace_bytes(N, C, HW, HW, K))
                if not L["direct"]:
                    L["dD"] = torch.empty_like(L["D"])
                    need = max(need, w.wino_workspace_bytes(N, K, HW, HW, C, 1, m, dt))
            layers.append(L)
        return {"case": case, "layers": layers, "ws": torch.empty(need, dtype=torch.uint8, device="cuda")}

    C, H, W, K = case["C"], case["H"], case["W"], case["K"]
    if case["kind"] == "direct":
        R, S, pad, st = case["R"], case["S"], case["pad"], case["stride"]
        D, G = rnd.normal((N, C, H, W), tdt), rnd.filters(K, C, R, S, tdt)
        Y = torch.empty((N, K, (H + 2 * pad - R) // st + 1, (W + 2 * pad - S) // st + 1), dtype=tdt, device="cuda")
        return {"case": case, "D": D, "G": G, "Y": Y}
    m, pad = case["m"], case["pad"]
    ydt = DTYPES[case["y"]][0]
    s = {"case": case}
    G = rnd.filters(K, C, 3, 3, tdt)
    if case["kind"] in ("layer", "layer_fx", "short"):
        s["D"] = rnd.normal((N, C, H, W), tdt)
        if case["kind"] == "layer_fx":
            s["U"] = w.wino_filter_transform(G, m)
        else:
            s["G"] = G
        if case["kind"] != "short":
            s["Y"] = torch.empty((N, K, H + 2 * pad - 2, W + 2 * pad - 2), dtype=ydt, device="cuda")
            s["ws"] = w.alloc_workspace(N, C, H, W, K, pad, m, dt)
    elif case["kind"] == "bwd_data":
        s["G"], s["E"] = G, rnd.normal((N, K, H, W), tdt)
        s["dD"] = torch.empty((N, C, H, W), dtype=ydt, device="cuda")
        s["ws"] = w.alloc_workspace(N, K, H, W, C, pad, m, dt)
    else:
        s["D"], s["E"] = rnd.normal((N, C, H, W), tdt), rnd.normal((N, K, H, W), tdt)
        s["dG"] = torch.empty((K, C, 3, 3), dtype=torch.float32, device="cuda")
        s["ws"] = torch.empty(w.wino_bwd_filter_workspace_bytes(N, C, H, W, K), dtype=torch.uint8, device="cuda")
    return s


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind in ("stack", "train"):
        ws, out = state["ws"], []
        for L in state["layers"]:
            if L["direct"]:
                out.append(w.direct_conv2d_fwd(L["D"], L["G"], pad=1, Y=L["Y"]))
            else:
                out.append(w.wino_conv2d_fwd_ex(L["D"], G=L["G"], pad=1, m=L["m"], Y=L["Y"], workspace=ws))
        if kind == "train":
            for L in reversed(state["layers"]):
                out.append(w.wino_conv2d_bwd_filter(L["D"], L["E"], pad=1, dG=L["dG"], workspace=ws))
                if not L["direct"]:             # nobody needs the gradient of the images
                    out.append(w.wino_conv2d_bwd_data(L["E"], G=L["G"], pad=1, m=L["m"], dD=L["dD"], workspace=ws))
        return out
    if kind == "direct":
        return w.direct_conv2d_fwd(state["D"], state["G"], pad=case["pad"], stride=case["stride"], Y=state["Y"])
    if kind == "short":
        return w.wino_conv2d_fwd(state["D"], state["G"], pad=case["pad"], m=case["m"])
    if kind == "layer":
        return w.wino_conv2d_fwd_ex(state["D"], G=state["G"], pad=case["pad"], m=case["m"], Y=state["Y"],
                                    workspace=state["ws"])
    if kind == "layer_fx":
        return w.wino_conv2d_fwd_ex(state["D"], U=state["U"], K=case["K"], pad=case["pad"], m=case["m"], Y=state["Y"],
                                    workspace=state["ws"])
    if kind == "bwd_data":
        return w.wino_conv2d_bwd_data(state["E"], G=state["G"], pad=1, m=case["m"], dD=state["dD"],
                                      workspace=state["ws"])
    return w.wino_conv2d_bwd_filter(state["D"], state["E"], pad=1, dG=state["dG"], workspace=state["ws"])


# ---- what a pass cannot do without, and how far correct results may lie apart --------------------------

def _wino_work(N, C, Ho, Wo, H, W, K, m, s_in, s_out, filter_bytes):
    """The multiplications of F(m x m, 3 x 3) on whole tiles; input, filters and output once."""
    tiles = N * ((Ho + m - 1) // m) * ((Wo + m - 1) // m)
    return (N * C * H * W * s_in + filter_bytes + N * K * Ho * Wo * s_out, 2 * (m + 2) ** 2 * K * C * tiles)


def _direct_work(N, C, H, W, K, R, S, Ho, Wo, s):
    return (N * C * H * W + K * C * R * S + N * K * Ho * Wo) * s, 2 * N * K * C * R * S * Ho * Wo


def _filter_grad_work(N, C, H, W, K):
    """F(3 x 3, 2 x 2): 16 multiplications per 2 x 2 block of the error; both tensors read, the gradient written."""
    blocks = N * ((H + 1) // 2) * ((W + 1) // 2)
    return (N * (C + K) * H * W + 9 * K * C) * 4, 32 * K * C * blocks


def work(case):
    s_in = 4 if case["dtype"] == "f32" else 2
    N, parts = case["N"], []
    if case["kind"] in ("stack", "train"):
        for i, C, HW, K, m in _stack(case):
            if C < 16:
                parts.append(_direct_work(N, C, HW, HW, K, 3, 3, HW, HW, s_in))
            else:
                parts.append(_wino_work(N, C, HW, HW, HW, HW, K, m, s_in, 4, 9 * K * C * s_in))
            if case["kind"] == "train":
                # (with 3 channels 16 products per block are more than the 36 of the definition divided by 2.25)
                parts.append(_filter_grad_work(N, C, HW, HW, K))
                if C >= 16:
                    parts.append(_wino_work(N, K, HW, HW, HW, HW, C, m, s_in, 4, 9 * K * C * s_in))
    elif case["kind"] == "direct":
        R, S, pad, st = case["R"], case["S"], case["pad"], case["stride"]
        Ho, Wo = (case["H"] + 2 * pad - R) // st + 1, (case["W"] + 2 * pad - S) // st + 1
        parts.append(_direct_work(N, case["C"], case["H"], case["W"], case["K"], R, S, Ho, Wo, s_in))
    else:
        C, H, W, K, m, pad = case["C"], case["H"], case["W"], case["K"], case["m"], case["pad"]
        s_out = 4 if case["y"] == "f32" else 2
        Ho, Wo = H + 2 * pad - 2, W + 2 * pad - 2
        if case["kind"] == "bwd_filter":
            parts.append(_filter_grad_work(N, C, H, W, K))
        elif case["kind"] == "bwd_data":
            parts.append(_wino_work(N, K, H, W, H, W, C, m, s_in, s_out, 9 * K * C * s_in))
        else:
            fb = ((m + 2) ** 2 if case["kind"] == "layer_fx" else 9) * K * C * s_in
            parts.append(_wino_work(N, C, Ho, Wo, H, W, K, m, s_in, s_out, fb))
    return {"bytes": int(sum(p[0] for p in parts)), "flops": int(sum(p[1] for p in parts))}


def tolerance(case):
    """About four times the distance between a pass and the same layer evaluated in float64 (2-norm; the largest
    element grows with the largest row of the inverse transform)."""
    kind = case["kind"]
    if kind in ("stack", "train"):
        ms = {m for _, C, _, _, m in _stack(case) if C >= 16}
        m = max(ms)
    elif kind == "direct":
        return {"rel": 2e-6, "max": 2e-5} if case["dtype"] == "f32" else {"rel": 1e-3, "max": 4e-3}
    elif kind == "bwd_filter":
        m = 2
    else:
        m = case["m"]
    if case["dtype"] == "f16":
        return {"rel": 2e-3, "max": 2e-2} if m == 2 else {"rel": 1.2e-2, "max": 0.25}
    if kind == "bwd_filter":
        return {"rel": 4e-6, "max": 4e-5}
    return {2: {"rel": 3e-6, "max": 3e-5}, 4: {"rel": 2e-5, "max": 4e-4}, 6: {"rel": 4e-5, "max": 1e-3}}[m]

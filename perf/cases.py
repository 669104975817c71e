"""Performance cases of the sparse convolution: the layers a user of the library runs, and random ones like them.

A case is a dict of plain values:
    op          "forward" (sconv_forward), "pool" (sconv_pool_forward), "encode" (sconv_encode) or "chain" (layers fed
                by the previous layer's output)
    N C H W K R S stride pad groups, pool_h pool_w pool_stride (0: none)
    zeros       zero ratio of the feature map; zeros_spread: half width of the uniform range every channel's own
                ratio is drawn from; clustered: dead planes and patches of zeros instead of independent zeros
    call        "plain" (x and w only), "ws" (a workspace passed with the call) or "prepared" (prepared filters and a
                workspace)
    hint        the zero ratio travels with the call, as a program that probed it once does
    bias        the layer's bias is passed (plain and prepared calls)
    fmt         "ecr" or "pecr" (encode only)

Shapes and zero ratios are those of the repository's benchmark layers (VGG-19, ResNet-50, DenseNet-121,
RegNetX-16GF and the single layers on small maps).
"""
import math

import torch

import paper_1909_09927_amd as sconv


def _conv(name, op, N, C, HW, K, RS, stride=1, pad=None, groups=1, pool=(0, 0, 0), zeros=0.7, spread=0.0,
          clustered=False, call="ws", hint=False, bias=False, fmt="ecr"):
    return {"name": name, "op": op, "N": N, "C": C, "H": HW, "W": HW, "K": K, "R": RS, "S": RS, "stride": stride,
            "pad": RS // 2 if pad is None else pad, "groups": groups, "pool_h": pool[0], "pool_w": pool[1],
            "pool_stride": pool[2], "zeros": zeros, "zeros_spread": spread, "clustered": clustered, "call": call,
            "hint": hint, "bias": bias, "fmt": fmt}


# The 28x28 and 14x14 stages of a VGG-19-shaped network: (C, map, K, pooled).  The ratios are what ReLU and pooling
# leave of a first input with 60 % zeros when the filters' mean is -0.03 standard deviations.
_CHAIN = [(256, 28, 512, False), (512, 28, 512, False), (512, 28, 512, False), (512, 28, 512, True),
          (512, 14, 512, False), (512, 14, 512, False), (512, 14, 512, True)]
_CHAIN_ZEROS = [0.60, 0.76, 0.77, 0.78, 0.41, 0.88, 0.68]


def listed():
    return [
        # the smallest call: a thumbnail-sized layer without any set-up; latency of one launch
        _conv("tiny-3x3-plain", "forward", 1, 16, 28, 32, 3, zeros=0.7, call="plain"),
        # batch-1 inference of a deep ResNet layer: few positions, 9.4 MB of filters
        _conv("resnet-3x3-512x7-n1", "forward", 1, 512, 7, 512, 3, zeros=0.65, spread=0.15),
        # a 5x5 inception branch: a small layer of the general kernel, with its bias
        _conv("googlenet-5x5-48to128x7-n32", "forward", 32, 48, 7, 128, 5, zeros=0.95, call="plain", bias=True),
        # bottleneck entry: 1x1, bound by the map's trip through memory
        _conv("resnet-1x1-256to64x56-n32", "forward", 32, 256, 56, 64, 1, zeros=0.65, spread=0.15),
        # transition layer: 1x1 fused with 2x2 pooling
        _conv("densenet-T-1x1-pool-n16", "pool", 16, 512, 28, 256, 1, pool=(2, 2, 2), zeros=0.7),
        # strided downsampling layer
        _conv("resnet-3x3-128x56-s2-n32", "forward", 32, 128, 56, 128, 3, stride=2, zeros=0.65, spread=0.15),
        # grouped layer as the simplest program calls it: no workspace, no hint; zeros in clusters as ReLU leaves them
        _conv("regnetx-896x14-g7-n32", "forward", 32, 896, 14, 896, 3, groups=7, zeros=0.7, clustered=True, call="plain"),
        # the benchmark's slowest layer, zero ratio probed
        _conv("vgg-256x56-n8", "forward", 8, 256, 56, 256, 3, zeros=0.60, hint=True),
        # a deep layer in the serving set-up: filters prepared, zero ratio probed
        _conv("vgg-512x28-n8-prepared", "forward", 8, 512, 28, 512, 3, zeros=0.75, call="prepared", hint=True),
        # convolution + ReLU + pooling in one pass, serving set-up
        _conv("vgg-512x14-pool-n8-prepared", "pool", 8, 512, 14, 512, 3, pool=(2, 2, 2), zeros=0.85, call="prepared",
              hint=True),
        # conversion alone: the format materialised for inspection or another consumer
        _conv("encode-ecr-256x56", "encode", 1, 256, 56, 256, 3, zeros=0.60),
        # several layers in sequence, each on what the previous one left: serving a network's tail
        _conv("vgg-tail-7-layers-n8", "chain", 8, 256, 28, 512, 3, zeros=0.60, call="prepared", hint=True, bias=True),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _channels(rng, lo, hi):
    """A channel count: usually a multiple of 16 as networks have them, sometimes any number."""
    n = _log_int(rng, lo, hi)
    return n if rng.random() < 0.25 else max(lo, n // 16 * 16 if n >= 16 else n)


def draw(rng):
    while True:
        op = rng.choice(["forward", "forward", "forward", "pool", "encode"])
        rs = rng.choice([3, 3, 3, 3, 1, 1, 5, 7])
        stride = rng.choice([1, 1, 1, 1, 2, 3]) if rs > 1 else rng.choice([1, 1, 1, 1, 2])
        pool = (0, 0, 0)
        fmt = rng.choice(["ecr", "pecr"]) if op == "encode" else "ecr"
        if op == "pool" or fmt == "pecr":
            pool = rng.choice([(2, 2, 2), (2, 2, 2), (2, 2, 2), (3, 3, 2)])
        groups = rng.choice([1, 1, 1, 1, 2, 4])
        C = groups * _channels(rng, 3 if rs > 3 else 8, max(16, (128 if rs > 3 else 768) // groups))
        K = groups * _channels(rng, 16, max(32, 768 // groups))
        H, W = _log_int(rng, 6, 64), 0
        W = H if rng.random() < 0.7 else _log_int(rng, 6, 64)
        N = _log_int(rng, 1, 32)
        pad = rng.choice([rs // 2, rs // 2, rs // 2, 0])
        OH, OW = (H + 2 * pad - rs) // stride + 1, (W + 2 * pad - rs) // stride + 1
        if min(OH, OW) < max(pool[0], pool[1], 1):
            continue
        case = {"op": op, "N": N, "C": C, "H": H, "W": W, "K": K, "R": rs, "S": rs, "stride": stride, "pad": pad,
                "groups": groups, "pool_h": pool[0], "pool_w": pool[1], "pool_stride": pool[2],
                "zeros": round(rng.uniform(0.4, 0.95), 2), "zeros_spread": 0.0, "clustered": rng.random() < 0.4,
                "call": rng.choice(["plain", "ws", "prepared"]), "hint": rng.random() < 0.5, "fmt": fmt}
        if op == "encode":
            case.update(call="plain", hint=False)
        case["bias"] = op != "encode" and case["call"] != "ws" and rng.random() < 0.4
        dense = 2.0 * N * K * OH * OW * (C // groups) * rs * rs
        if op == "encode":
            rows, slots = sconv.sconv_encode_sizes(_desc(case), _fmt(case))
            if not 1e5 <= rows * slots * 8 <= 2e8:
                continue
        elif not 1e7 <= dense <= 2.5e10:
            continue
        return case


def _pool(case):
    return (case["pool_h"], case["pool_w"], case["pool_stride"]) if case["pool_h"] else None


def _fmt(case):
    return sconv.FMT_PECR if case["fmt"] == "pecr" else sconv.FMT_ECR


def _desc(case):
    return sconv.make_desc(case["N"], case["C"], case["H"], case["W"], case["K"], case["R"], case["S"], case["stride"],
                           case["pad"], case["groups"], _pool(case), True)


def _feature_map(case, gen):
    """fp32 NCHW map on the GPU: |N(0,1)| where kept, exact zeros elsewhere."""
    N, C, H, W, z = case["N"], case["C"], case["H"], case["W"], case["zeros"]
    shape = (N, C, H, W)
    x = torch.randn(shape, generator=gen, device="cuda").abs_().clamp_min_(1e-6)
    if case["clustered"]:
        # a share 0.3*z of the planes is dead, the other zeros form patches on a 4x4 coarser grid
        dead = 0.3 * z
        alive_z = (z - dead) / (1.0 - dead)
        field = torch.randn((N, C, (H + 3) // 4, (W + 3) // 4), generator=gen, device="cuda")
        field = field.repeat_interleave(4, 2).repeat_interleave(4, 3)[:, :, :H, :W].contiguous()
        field += 0.5 * torch.randn(shape, generator=gen, device="cuda")
        rank = max(1, min(H * W, round(alive_z * H * W)))
        cut = field.view(N, C, -1).sort(dim=2).values[:, :, rank - 1]
        keep = (field > cut[:, :, None, None]) & (torch.rand((N, C, 1, 1), generator=gen, device="cuda") >= dead)
    else:
        ratio = z + case["zeros_spread"] * (2.0 * torch.rand((1, C, 1, 1), generator=gen, device="cuda") - 1.0)
        keep = torch.rand(shape, generator=gen, device="cuda") >= ratio
    return torch.where(keep, x, torch.zeros((), device="cuda")).contiguous()


def _filters(K, Cg, rs, gen, shift=0.0):
    std = math.sqrt(2.0 / (Cg * rs * rs))
    return (torch.randn((K, Cg, rs, rs), generator=gen, device="cuda") + shift) * std


def _workspace(desc, pooled):
    n = sconv.sconv_workspace_size(desc, pooled)
    return torch.empty(n, dtype=torch.uint8, device="cuda") if n else None


def _prepare_chain(case, gen):
    x = _feature_map(case, gen)
    layers, ws_bytes, cur = [], 0, x
    for C, hw, K, pooled in _CHAIN:
        w = _filters(K, C, 3, gen, shift=-0.03)
        desc = sconv.make_desc(case["N"], C, hw, hw, K, 3, 3, 1, 1, 1, (2, 2, 2) if pooled else None, True)
        ws_bytes = max(ws_bytes, sconv.sconv_workspace_size(desc, pooled))
        bias = 0.01 * torch.randn(K, generator=gen, device="cuda") if case["bias"] else None
        layers.append({"w": w, "wprep": sconv.sconv_filter_prep(w), "bias": bias, "pooled": pooled, "zeros": None})
    ws = torch.empty(ws_bytes, dtype=torch.uint8, device="cuda")
    state = {"op": "chain", "x": x, "layers": layers, "ws": ws}
    if case["hint"]:   # set-up of a serving program: one pass with the density probe on every layer's input
        for layer in layers:
            layer["zeros"] = sconv.zero_ratio_of(sconv.sconv_density(cur))
            cur = _chain_layer(cur, layer, ws)
    return state


def _chain_layer(x, layer, ws):
    if layer["pooled"]:
        return sconv.sconv_pool_forward(x, layer["w"], (2, 2, 2), 1, 1, bias=layer["bias"], ws=ws,
                                        zero_ratio=layer["zeros"], wprep=layer["wprep"])
    return sconv.sconv_forward(x, layer["w"], 1, 1, relu=True, bias=layer["bias"], ws=ws, zero_ratio=layer["zeros"],
                               wprep=layer["wprep"])


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    if case["op"] == "chain":
        return _prepare_chain(case, gen)
    x = _feature_map(case, gen)
    state = {"op": case["op"], "x": x}
    conv = {"stride": case["stride"], "pad": case["pad"], "groups": case["groups"]}
    Cg = case["C"] // case["groups"]
    if case["op"] == "encode":
        return dict(state, args=((case["K"], Cg, case["R"], case["S"]), _fmt(case)), kw=dict(conv, pool=_pool(case)))
    w = _filters(case["K"], Cg, case["R"], gen)
    pooled = case["op"] == "pool"
    kw = dict(conv)
    if not pooled:
        kw["relu"] = True
    if case["hint"]:
        kw["zero_ratio"] = sconv.zero_ratio_of(sconv.sconv_density(x))
    if case["bias"]:
        kw["bias"] = 0.01 * torch.randn(case["K"], generator=gen, device="cuda")
    if case["call"] == "prepared":
        # None where no kernel reads the prepared layout: such a program makes the plain call
        kw["wprep"] = sconv.sconv_filter_prep(w, case["groups"], case["stride"], case["pad"])
    if case["call"] != "plain" and not (case["bias"] and kw.get("wprep") is None):
        kw["ws"] = _workspace(_desc(case), pooled)
    return dict(state, args=(w, _pool(case)) if pooled else (w,), kw=kw)


def run(state):
    op = state["op"]
    if op == "chain":
        outs, cur = [], state["x"]
        for layer in state["layers"]:
            cur = _chain_layer(cur, layer, state["ws"])
            outs.append(cur)
        return outs
    call = {"forward": sconv.sconv_forward, "pool": sconv.sconv_pool_forward, "encode": sconv.sconv_encode}[op]
    return call(state["x"], *state["args"], **state["kw"])


def work(case):
    """Bytes: input, filters and outputs once each.  Flops: one multiply-add per nonzero and filter."""
    if case["op"] == "chain":
        nbytes, flops, N = 0.0, 0.0, case["N"]
        for (C, hw, K, pooled), z in zip(_CHAIN, _CHAIN_ZEROS):
            out = N * K * (hw // 2 if pooled else hw) ** 2
            nbytes += 4.0 * (N * C * hw * hw + K * C * 9 + out)
            flops += 2.0 * N * K * hw * hw * C * 9 * (1.0 - z)
        return {"bytes": nbytes, "flops": flops}
    N, C, K, Cg = case["N"], case["C"], case["K"], case["C"] // case["groups"]
    desc = _desc(case)
    OH, OW, PH, PW = sconv.sconv_output_dims(desc)
    x_elems = N * C * case["H"] * case["W"]
    if case["op"] == "encode":
        rows, slots = sconv.sconv_encode_sizes(desc, _fmt(case))
        return {"bytes": 4.0 * x_elems + 8.0 * rows * slots + 4.0 * rows, "flops": 0.0}
    out = N * K * (PH * PW if case["op"] == "pool" else OH * OW)
    taps = Cg * case["R"] * case["S"]
    return {"bytes": 4.0 * (x_elems + K * taps + out),
            "flops": 2.0 * N * K * OH * OW * taps * (1.0 - case["zeros"])}


def tolerance(case):
    """Measured against the same sums in 64 bits: 0.6e-7 to 2.7e-7 (relative) for one layer of 81 to 4896 terms; the
    chain's seven layers pass the error on."""
    if case["op"] == "encode":
        return "exact"
    return {"rel": 4e-6 if case["op"] == "chain" else 1.2e-6}

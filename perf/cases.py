"""The calls whose speed counts: single depthwise and group convolution layers and one whole depthwise stack, through the
public entry points, over the range of sizes, layouts, storage types and directions that a training program meets.

A case is one layer (or the stack) with everything that its descriptor takes.  `passes` says what the program runs:
"fwd" (inference), "train" (forward, filter gradient, input gradient as three calls) or "fused" (forward, then the whole
backward pass in one call; depthwise only).
"""
import math

import torch

import paper_1803_09926_amd as dw
from paper_1803_09926_amd import workloads as wl

LAYOUTS = {"NCHW": dw.NCHW, "NHWC": dw.NHWC}
DTYPES = {"f32": dw.F32, "bf16": dw.BF16}
TORCH = {"f32": torch.float32, "bf16": torch.bfloat16}


def _layer(name, N, C, H, W=None, K=3, stride=1, mult=1, groups=0, layout="NCHW", dtype="f32", passes="train"):
    """groups 0: a depthwise layer of C * mult outputs; otherwise a group convolution with C inputs and C outputs."""
    return {"name": name, "kind": "layer", "N": N, "C": C, "H": H, "W": W or H, "K": K, "stride": stride, "pad": K // 2,
            "mult": mult, "groups": groups, "layout": layout, "dtype": dtype, "passes": passes}


def listed():
    return [
        # one image through one late layer: the latency of a single small call
        _layer("one_image", 1, 512, 14, layout="NHWC", passes="fwd"),
        # the single-layer configuration (batch 8, 32 channels, 112 x 112): a small training step, three short calls
        _layer("single_layer", 8, 32, 112),
        # the benchmark's stack of thirteen depthwise layers at its batch of 128: ordinary training, most of the time here
        {"name": "stack", "kind": "stack", "N": 128, "layout": "NHWC", "dtype": "f32", "passes": "train"},
        # Xception-style shapes as an NCHW program has them: rows that are no whole number of 16-byte vectors
        _layer("rows_of_74", 32, 256, 74, dtype="bf16"),
        _layer("rows_of_19", 32, 728, 19, passes="fused"),
        # the 5x5 variant of a stride-1 layer, at the batch of the bf16 configuration
        _layer("five_by_five", 256, 256, 28, K=5, layout="NHWC", dtype="bf16"),
        # 5x5 where the map is halved, as networks with 5x5 depthwise filters do
        _layer("five_by_five_s2", 64, 128, 56, K=5, stride=2, layout="NHWC"),
        # large filters: 7x7 depthwise at a middle resolution
        _layer("seven_by_seven", 64, 256, 28, K=7),
        # channel multiplier 2: the Xception-style layer, channels first
        _layer("multiplier", 32, 256, 56, mult=2),
        # group convolutions: four channels a group on a large map, eight where the map is halved, sixteen on a small map
        _layer("group4", 128, 128, 56, groups=32),
        _layer("group8_s2", 16, 256, 56, stride=2, groups=32, dtype="bf16"),
        _layer("group16", 32, 512, 14, groups=32, layout="NHWC", dtype="bf16"),
    ]


def draw(rng):
    """One layer of the listed ones' ranges: batch 1 to 256, planes of 4 to 150, filters 3, 5 and 7, stride 1 and 2,
    multiplier 1 and 2, 2 to 32 channels a group, both layouts and types, at a size that one call of the listed layers has."""
    pick = rng.choice
    K, stride = pick([3, 3, 3, 5, 7]), pick([1, 1, 1, 2])
    group = pick([0, 0, 0, 2, 4, 8, 16, 32])
    H = int(round(math.exp(rng.uniform(math.log(4), math.log(150)))))
    W = H if rng.random() < 0.7 else max(4, min(150, int(round(H * rng.uniform(0.6, 1.6)))))
    if group:
        K = pick([3, 3, 3, 5])
        C = group * int(round(math.exp(rng.uniform(math.log(2), math.log(max(2, 512 // group))))))
        most = (1 << 24) * 9 // (K * K) // group
    else:
        C = int(round(math.exp(rng.uniform(math.log(8), math.log(1024)))))
        if rng.random() < 0.8:
            C = max(8, C // 8 * 8)
        most = (1 << 24) * 9 // (K * K)
    N = int(round(math.exp(rng.uniform(0, math.log(256)))))
    N = max(1, min(N, most // (C * H * W)))
    while C * H * W > most and H > 4:
        H, W = max(4, H // 2), max(4, W // 2)
    mult = pick([1, 1, 1, 2]) if not group else 1
    passes = pick(["fwd", "train", "train", "train"] + ([] if group else ["fused"]))
    case = _layer("", N, C, H, W, K, stride, mult, C // group if group else 0, pick(sorted(LAYOUTS)), pick(sorted(DTYPES)), passes)
    del case["name"]
    return case


def _one(case):
    return wl.Layer("layer", case["C"], case["H"], case["W"], case["K"], case["stride"], case["pad"], case["mult"],
                    case["C"] // case["groups"] if case["groups"] else 1)


def _layers(case):
    return list(wl.MOBILENET_V1) if case["kind"] == "stack" else [_one(case)]


def prepare(case, seed):
    """For each layer the descriptor, inputs, output buffers and workspace that a training program holds."""
    layout, dtype = LAYOUTS[case["layout"]], DTYPES[case["dtype"]]
    state = []
    for i, l in enumerate(_layers(case)):
        x, w, dy = wl.make_inputs_device(l, case["N"], layout, dtype, 1000 * seed + i)
        group = case.get("groups", 0) > 0
        if group:
            d = dw.group_desc(case["N"], l.C, l.H, l.W, l.K, l.stride, l.pad, case["groups"], l.C, layout, dtype)
            need = dw.gconv_bwd_filter_workspace_bytes(d)
        else:
            d = dw.desc(case["N"], l.C, l.H, l.W, l.K, l.stride, l.pad, l.mult, layout, dtype)
            need = max(dw.bwd_filter_workspace_bytes(d), dw.bwd_workspace_bytes(d))
        s = {"d": d, "group": group, "passes": case["passes"], "x": x, "w": w, "dy": dy, "y": torch.empty_like(dy)}
        if case["passes"] != "fwd":
            s["dx"], s["dw"] = torch.empty_like(x), torch.empty(w.shape, device="cuda", dtype=torch.float32)
            s["ws"] = torch.empty(max(need, 16), device="cuda", dtype=torch.uint8)
        state.append(s)
    return state


def run(state):
    out = []
    for s in state:
        d, x, w, dy, y = s["d"], s["x"], s["w"], s["dy"], s["y"]
        if s["group"]:
            dw.gconv_fwd(d, x, w, y)
        else:
            dw.fwd(d, x, w, y)
        if s["passes"] == "fwd":
            out.append({"y": y})
            continue
        dx, g, ws = s["dx"], s["dw"], s["ws"]
        if s["passes"] == "fused":
            dw.bwd(d, x, dy, w, dx, g, ws)
        elif s["group"]:
            dw.gconv_bwd_filter(d, x, dy, g, ws)
            dw.gconv_bwd_data(d, dy, w, dx)
        else:
            dw.bwd_filter(d, x, dy, g, ws)
            dw.bwd_data(d, dy, w, dx)
        out.append({"y": y, "dx": dx, "dw": g})
    return out


def work(case):
    """Each pass reads its input tensor(s) and the filter once and writes its output once."""
    size = 4 if case["dtype"] == "f32" else 2
    nbytes = flops = 0
    for l in _layers(case):
        x, y, w = l.x_elems(case["N"]), l.y_elems(case["N"]), l.O * l.cg * l.K * l.K
        if case["passes"] == "fwd":
            nbytes += (x + y + w) * size
        elif case["passes"] == "fused":
            nbytes += (3 * x + 2 * y + 2 * w) * size + 4 * w
        else:
            nbytes += (3 * x + 3 * y + 2 * w) * size + 4 * w
        flops += l.pass_flops(case["N"]) * (1 if case["passes"] == "fwd" else 3)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """Four times what the calls differ from the 64-bit result by: fp32 up to 7e-7 (a filter gradient that adds 50 000
    products one after the other; the other passes stay below 4e-7), bf16 1.7e-3 (one rounding of each output)."""
    return {"rel": 3e-6} if case["dtype"] == "f32" else {"rel": 7e-3}


def _exact_layer(s, layout, l, groups):
    """The three passes in 64 bits as K * K shifted products, image chunk by image chunk."""
    nhwc, cg, og = layout == "NHWC", l.C // groups, l.O // groups
    K, st, p, Ho, Wo = l.K, l.stride, l.pad, l.Ho, l.Wo
    x, dy, w = s["x"], s["dy"], s["w"].double()
    if nhwc:
        w = w.permute(2, 0, 1) if w.dim() == 3 else w.permute(3, 2, 0, 1)
    w = w.reshape(groups, og, cg, K, K)
    back = s["passes"] != "fwd"
    first = (lambda t: t.permute(0, 3, 1, 2)) if nhwc else (lambda t: t)
    last = (lambda t: t.permute(0, 2, 3, 1).contiguous()) if nhwc else (lambda t: t)
    N = x.shape[0]
    step = max(1, (1 << 25) // max(l.C * l.H * l.W, l.O * Ho * Wo))
    ys, dxs = [], []
    gw = torch.zeros_like(w)
    for n in range(0, N, step):
        xs = torch.nn.functional.pad(first(x[n:n + step]).double(), (p, p, p, p))
        b = xs.shape[0]
        g = first(dy[n:n + step]).double().reshape(b, groups, og, Ho * Wo) if back else None
        y = torch.zeros(b, groups, og, Ho * Wo, dtype=torch.float64, device=x.device)
        dxp = torch.zeros_like(xs) if back else None
        for kh in range(K):
            for kw in range(K):
                rows, cols = slice(kh, kh + st * (Ho - 1) + 1, st), slice(kw, kw + st * (Wo - 1) + 1, st)
                t = xs[:, :, rows, cols].reshape(b, groups, cg, Ho * Wo)
                m = w[:, :, :, kh, kw]
                for o in range(og):
                    if cg == 1:
                        y[:, :, o] += m[:, o] * t[:, :, 0]
                    else:
                        y[:, :, o] += (m[:, o, :, None] * t).sum(2)
                if back:
                    back_t = torch.zeros_like(t)
                    for o in range(og):
                        gw[:, o, :, kh, kw] += (g[:, :, o:o + 1] * t).sum(3).sum(0)
                        back_t += m[:, o, :, None] * g[:, :, o:o + 1]
                    dxp[:, :, rows, cols] += back_t.reshape(b, l.C, Ho, Wo)
        ys.append(last(y.reshape(b, l.O, Ho, Wo)))
        if back:
            dxs.append(last(dxp[:, :, p:p + l.H, p:p + l.W]))
    out = {"y": torch.cat(ys)}
    if back:
        gw = gw.reshape(l.O, cg, K, K)
        if s["group"]:
            gw = gw.permute(2, 3, 1, 0).contiguous() if nhwc else gw
        else:
            gw = gw[:, 0].permute(1, 2, 0).contiguous() if nhwc else gw[:, 0].contiguous()
        out["dx"], out["dw"] = torch.cat(dxs), gw
    return out


def exact(case, seed):
    return [_exact_layer(s, case["layout"], l, case["groups"] if case.get("groups") else l.C)
            for s, l in zip(prepare(case, seed), _layers(case))]

"""The convolution calls whose speed this repository answers for.

Each case is a call (or a whole network's calls) that a program doing batch-1
inference makes, through the package's public entry points:

  kind "layer"  one convolution: sizes (c_in, h, w, c_out, k, stride, pad),
                bias or none, epilogue ("none", "relu", "relu_pool": ReLU and
                a 2x2 max-pool), weights "oihw" as they are or "packed" once
                for the plan, and how it is called: "call" (the plain function,
                which allocates its output) or "launcher" (arguments marshalled
                once, output kept, as a program that runs the same layer again
                and again holds it);
  kind "stack"  the VGG-16-shaped stack of 13 convolutions on packed weights,
                each with its fused epilogue, one launcher per layer.

Activations are post-ReLU-like (uniform in [0, 1]), weights He-normal, biases
normal(0, 0.01): the values that trained layers of these networks see.
"""
import math

import torch
import torch.nn.functional as F

import paper_1909_02765_amd as ilpm
import workloads

EPILOGUES = {"none": 0, "relu": ilpm.EPI_RELU, "relu_pool": ilpm.EPI_RELU | ilpm.EPI_MAXPOOL2}


def _layer(name, c_in, h, w, c_out, k, stride, pad, bias=True, epilogue="none", weights="oihw", how="launcher"):
    case = {"kind": "layer", "c_in": c_in, "h": h, "w": w, "c_out": c_out, "k": k, "stride": stride, "pad": pad,
            "bias": bias, "epilogue": epilogue, "weights": weights, "how": how}
    if name:
        case["name"] = name
    return case


def listed():
    return [
        # The smallest call: a thumbnail's first layer, where the call itself is the cost.
        _layer("tiny_3to16_32", 3, 32, 32, 16, 3, 1, 1, how="call"),
        # A classifier's first layer on a full image, 7x7 with stride 2, called as it stands.
        _layer("stem7x7_3to64_224", 3, 224, 224, 64, 7, 2, 3, epilogue="relu", how="call"),
        # The early VGG layer, the framework's headline shape.
        _layer("early_64to64_224", 64, 224, 224, 64, 3, 1, 1),
        # The end of a VGG stage: packed weights, ReLU and pooling fused.
        _layer("stage_end_128to128_112", 128, 112, 112, 128, 3, 1, 1, epilogue="relu_pool", weights="packed"),
        # A bottleneck's pointwise layer at an ordinary size.
        _layer("pointwise_256to128_56", 256, 56, 56, 128, 1, 1, 0, bias=False, epilogue="relu"),
        # The middle of a residual network, and its strided layer.
        _layer("mid_256to256_14", 256, 14, 14, 256, 3, 1, 1, bias=False),
        _layer("strided_128to256_28", 128, 28, 28, 256, 3, 2, 1, bias=False),
        # Deep layers on a 7x7 map: pointwise and 5x5.
        _layer("deep1x1_512_7", 512, 7, 7, 512, 1, 1, 0, bias=False, weights="packed"),
        _layer("deep5x5_512_7", 512, 7, 7, 512, 5, 1, 2, bias=False),
        # Sizes that no tile divides: a pruned network's layer on a cropped frame.
        _layer("ragged_75to150_61x45", 75, 61, 45, 150, 3, 1, 1, epilogue="relu", how="call"),
        # A camera frame through an early layer: the largest single call.
        _layer("frame_64to96_301x403", 64, 301, 403, 96, 3, 1, 1, epilogue="relu"),
        # A whole batch-1 inference.
        {"name": "vgg16_stack", "kind": "stack", "hw": workloads.VGG16_HW},
    ]


def _flops(case):
    ho = ilpm.out_size(case["h"], case["k"], case["stride"], case["pad"])
    wo = ilpm.out_size(case["w"], case["k"], case["stride"], case["pad"])
    return 2.0 * case["c_out"] * case["c_in"] * case["k"] ** 2 * ho * wo


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


# A drawn layer is no more work than the largest listed layer.
_MOST_FLOPS = 2.0 * 96 * 64 * 9 * 301 * 403


def draw(rng):
    while True:
        h = _log_int(rng, 7, 320)
        w = h if rng.random() < 0.5 else min(320, max(7, int(round(h * rng.uniform(0.6, 1.7)))))
        if rng.random() < 0.2:  # a first layer
            c_in, c_out = rng.choice([1, 3, 3, 4]), _log_int(rng, 8, 96)
            k = rng.choice([3, 3, 5, 7])
        else:
            c_in, c_out = _log_int(rng, 16, 640), _log_int(rng, 16, 640)
            if rng.random() < 0.6:  # most networks keep to multiples of 16
                c_in, c_out = (c_in + 15) // 16 * 16, (c_out + 15) // 16 * 16
            k = rng.choice([1, 1, 3, 3, 3, 3, 5])
        stride = rng.choice([1, 1, 1, 2])
        pad = k // 2
        epilogue = rng.choice(["none", "relu", "relu", "relu_pool"])
        case = _layer(None, c_in, h, w, c_out, k, stride, pad, rng.random() < 0.6, epilogue,
                      rng.choice(["oihw", "oihw", "packed"]), rng.choice(["call", "launcher"]))
        if _flops(case) <= _MOST_FLOPS:
            return case


def _device():
    return "cuda" if torch.cuda.is_available() else "cpu"


def _layer_inputs(case, seed):
    dev = _device()
    g = torch.Generator(device=dev)
    g.manual_seed(seed)
    x = torch.rand((1, case["c_in"], case["h"], case["w"]), generator=g, device=dev)
    w = torch.randn((case["c_out"], case["c_in"], case["k"], case["k"]), generator=g, device=dev)
    w *= workloads.he_std(case["c_in"], case["k"])
    b = 0.01 * torch.randn((case["c_out"],), generator=g, device=dev) if case["bias"] else None
    return x, w, b


def _stack_inputs(case, seed):
    dev = _device()
    g = torch.Generator(device=dev)
    g.manual_seed(seed)
    x = torch.rand((1, 3, case["hw"], case["hw"]), generator=g, device=dev)
    layers = []
    for _, ci, co, hw, pool, _ in workloads.vgg16_layers():
        w = workloads.he_std(ci, 3) * torch.randn((co, ci, 3, 3), generator=g, device=dev)
        b = 0.01 * torch.randn((co,), generator=g, device=dev)
        layers.append((w, b, hw * case["hw"] // workloads.VGG16_HW, pool))
    return x, layers


def prepare(case, seed):
    if case["kind"] == "stack":
        x, layers = _stack_inputs(case, seed)
        launchers, t = [], x
        for w, b, hw, pool in layers:
            co, ci = w.shape[:2]
            epi = EPILOGUES["relu_pool" if pool else "relu"]
            plan = ilpm.plan_for(ci, hw, hw, co, 3, 1, 1, epi, prepacked=True)
            out = torch.empty(ilpm.epilogue_out_shape(co, hw, hw, 3, 1, 1, epi), device=x.device)
            launchers.append(ilpm.conv2d_prepacked_epilogue_launcher(t, ilpm.prepack_weights(w, plan), co, 3, b, 1, 1,
                                                                     epi, out, plan))
            t = out
        return {"launchers": launchers, "out": t}
    x, w, b = _layer_inputs(case, seed)
    c_in, h, wd, c_out, k, s, p = (case[n] for n in ("c_in", "h", "w", "c_out", "k", "stride", "pad"))
    epi = EPILOGUES[case["epilogue"]]
    state = {"x": x, "w": w, "b": b, "k": k, "stride": s, "pad": p, "epi": epi, "c_out": c_out}
    if case["weights"] == "packed":
        state["plan"] = ilpm.plan_for(c_in, h, wd, c_out, k, s, p, epi, prepacked=True)
        state["packed"] = ilpm.prepack_weights(w, state["plan"])
    if case["how"] == "launcher":
        out = torch.empty(ilpm.epilogue_out_shape(c_out, h, wd, k, s, p, epi), device=x.device)
        if case["weights"] == "packed":
            one = ilpm.conv2d_prepacked_epilogue_launcher(x, state["packed"], c_out, k, b, s, p, epi, out,
                                                          state["plan"])
        elif epi:
            one = ilpm.conv2d_epilogue_launcher(x, w, b, s, p, epi, out)
        else:
            one = ilpm.conv2d_launcher(x, w, b, s, p, out)
        state["launchers"], state["out"] = [one], out
    return state


def run(state):
    if "launchers" in state:
        for launch in state["launchers"]:
            launch()
        return state["out"]
    if "packed" in state:
        return ilpm.conv2d_prepacked_epilogue(state["x"], state["packed"], state["c_out"], state["k"], state["b"],
                                              state["stride"], state["pad"], state["epi"], plan=state["plan"])
    if state["epi"]:
        return ilpm.conv2d_epilogue(state["x"], state["w"], state["b"], state["stride"], state["pad"], state["epi"])
    return ilpm.conv2d(state["x"], state["w"], state["b"], state["stride"], state["pad"])


def work(case):
    if case["kind"] == "stack":
        flops, floats = 0.0, 0.0
        scale = (case["hw"] / workloads.VGG16_HW) ** 2
        for _, ci, co, hw, _, _ in workloads.vgg16_layers():
            flops += 2.0 * ci * co * 9 * hw * hw * scale
            floats += co * ci * 9 + co
        return {"bytes": 4.0 * (floats + 3 * case["hw"] ** 2 + 512 * 14 * 14 * scale), "flops": flops}
    _, co, ho, wo = ilpm.epilogue_out_shape(case["c_out"], case["h"], case["w"], case["k"], case["stride"],
                                            case["pad"], EPILOGUES[case["epilogue"]])
    floats = (case["c_in"] * case["h"] * case["w"] + co * case["c_in"] * case["k"] ** 2 + co * ho * wo +
              (co if case["bias"] else 0))
    return {"bytes": 4.0 * floats, "flops": _flops(case)}


def tolerance(case):
    # fp32 products summed in fp32, in any order: a single chain of the longest
    # sums drawn (some 12,800 terms) is 2e-6 off in the 2-norm, the layers here
    # 1e-7 to 6e-7, and the stack of 13 layers 1.2e-6.
    if case["kind"] == "stack":
        return {"rel": 5e-6, "max": 1e-4}
    return {"rel": 5e-6, "max": 5e-5}


def _conv64(x, w, b, stride, pad):
    """conv2d in float64 as one matrix product per band of output rows."""
    c_out, c_in, k, _ = w.shape
    x = F.pad(x.double(), (pad, pad, pad, pad))
    ho, wo = (x.shape[2] - k) // stride + 1, (x.shape[3] - k) // stride + 1
    wm = w.double().reshape(c_out, -1)
    rows = max(1, (1 << 26) // (c_in * k * k * wo))
    bands = []
    for r0 in range(0, ho, rows):
        r1 = min(ho, r0 + rows)
        cols = F.unfold(x[:, :, r0 * stride:(r1 - 1) * stride + k], k, stride=stride)[0]
        bands.append((wm @ cols).reshape(c_out, r1 - r0, wo))
    y = torch.cat(bands, dim=1)[None]
    return y if b is None else y + b.double()[None, :, None, None]


def _epilogue64(y, epi):
    if epi & ilpm.EPI_RELU:
        y = F.relu(y)
    if epi & ilpm.EPI_MAXPOOL2:
        y = F.max_pool2d(y, 2)
    return y


def exact(case, seed):
    if case["kind"] == "stack":
        x, layers = _stack_inputs(case, seed)
        for w, b, _, pool in layers:
            x = _epilogue64(_conv64(x, w, b, 1, 1), EPILOGUES["relu_pool" if pool else "relu"])
        return x
    x, w, b = _layer_inputs(case, seed)
    return _epilogue64(_conv64(x, w, b, case["stride"], case["pad"]), EPILOGUES[case["epilogue"]])

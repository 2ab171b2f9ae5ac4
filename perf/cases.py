"""Performance cases of the library: what is timed, on which inputs, and how far results may differ.

Four kinds of work, all through the Python binding, on float32 and on float16 storage:
  matmul     tfx_matmul / tfx_batch_matmul / tfx_batch_matmul_f16, every transpose
  conv       tfx_conv2d(_f16) with bias and activation: pointwise, 3 x 3, larger filters, strides, both paddings
  depthwise  tfx_depthwise_conv2d(_f16), 3 x 3, stride 1 and 2, with bias and activation
  net        the MobileNet-v1 family: a whole forward pass, or the feature map after a block (end_block > 0)
"""
import math

import torch

import paper_1901_05350_amd as tfx

CHANNELS = (64, 128, 128, 256, 256, 512, 512, 512, 512, 512, 512, 1024, 1024)
STRIDES = (1, 2, 1, 2, 1, 2, 1, 1, 1, 1, 1, 2, 1)
MOST_FLOPS, MOST_BYTES = 6.0e10, 4.0e8  # a drawn case stays below the largest listed ones


def matmul_case(dtype, batch, m, k, n, ta, tb):
    return {"kind": "matmul", "dtype": dtype, "batch": batch, "m": m, "k": k, "n": n, "ta": ta, "tb": tb}


def conv_case(dtype, n, h, w, cin, cout, fh, fw, stride, same, act):
    return {"kind": "conv", "dtype": dtype, "n": n, "h": h, "w": w, "cin": cin, "cout": cout, "fh": fh, "fw": fw,
            "stride": stride, "same": same, "act": act}


def depthwise_case(dtype, n, h, w, c, stride, act):
    return {"kind": "depthwise", "dtype": dtype, "n": n, "h": h, "w": w, "c": c, "stride": stride, "act": act}


def net_case(dtype, batch, size, quarters, classes, end_block):
    return {"kind": "net", "dtype": dtype, "batch": batch, "size": size, "quarters": quarters, "classes": classes,
            "end_block": end_block}


def listed():
    relu6 = tfx.ACT_RELU6
    cases = {
        # the smallest product: one call's launch and host path
        "matmul_f32_64x128x64": matmul_case("f32", 1, 64, 128, 64, False, False),
        # a batch of products that fills the matrix cores
        "matmul_f32_8x1024": matmul_case("f32", 8, 1024, 1024, 1024, False, True),
        # a score matrix over 1001 classes, nothing a multiple of a tile or of a vector load
        "matmul_f16_ragged": matmul_case("f16", 1, 1999, 1023, 1001, False, False),
        # one pointwise layer of one image
        "pointwise_f32_b1": conv_case("f32", 1, 56, 56, 128, 128, 1, 1, 1, True, relu6),
        # 3 x 3 convolution of a batch, few channels
        "conv3x3_f16_b64": conv_case("f16", 64, 56, 56, 64, 64, 3, 3, 1, True, relu6),
        # 3 x 3 convolution with odd maps and channel counts off the powers of two
        "conv3x3_f32_ragged": conv_case("f32", 8, 73, 73, 80, 192, 3, 3, 1, False, tfx.ACT_RELU),
        # the largest depthwise layer of a batch: memory traffic
        "depthwise_f32_b64": depthwise_case("f32", 64, 112, 112, 64, 1, relu6),
        # one image through the network: interactive inference
        "net_f32_b1": net_case("f32", 1, 224, 4, 1000, 0),
        # a small serving batch
        "net_f32_b8": net_case("f32", 8, 224, 4, 1000, 0),
        # throughput
        "net_f32_b64": net_case("f32", 64, 224, 4, 1000, 0),
        # the same two ends on 16-bit storage
        "net_f16_b1": net_case("f16", 1, 224, 4, 1000, 0),
        "net_f16_b64": net_case("f16", 64, 224, 4, 1000, 0),
    }
    return [dict(case, name=name) for name, case in cases.items()]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _extent(rng, lo, hi):
    """Half of the extents are what a user's model has (multiples of 8), the others anything."""
    v = _log(rng, lo, hi)
    return max(8, v // 8 * 8) if rng.random() < 0.5 and v >= 8 else v


def draw(rng):
    dtype = rng.choice(("f32", "f16"))
    while True:
        kind = rng.choice(("matmul", "matmul", "conv", "conv", "depthwise", "net", "net"))
        if kind == "matmul":
            batch = 1 if rng.random() < 0.6 else _log(rng, 2, 32)
            case = matmul_case(dtype, batch, _extent(rng, 16, 4096), _extent(rng, 16, 4096), _extent(rng, 16, 4096),
                               rng.random() < 0.25, rng.random() < 0.5)
        elif kind == "conv":
            f = rng.choice((1, 1, 3, 3, 3, 5))
            cin = 3 if rng.random() < 0.1 else _extent(rng, 8, 512)
            h = _log(rng, 7, 112)
            w = h if rng.random() < 0.7 else _log(rng, 7, 112)
            case = conv_case(dtype, _log(rng, 1, 64), h, w, cin, _extent(rng, 8, 512), f, f, rng.choice((1, 1, 2)),
                             rng.random() < 0.75, rng.choice((tfx.ACT_NONE, tfx.ACT_RELU, tfx.ACT_RELU6)))
        elif kind == "depthwise":
            h = _log(rng, 7, 150)
            case = depthwise_case(dtype, _log(rng, 1, 64), h, h + rng.choice((0, 0, 1, -1)), _extent(rng, 8, 1024),
                                  rng.choice((1, 2)), rng.choice((tfx.ACT_NONE, tfx.ACT_RELU6)))
        else:
            size = rng.choice((128, 160, 192, 224, 224)) if rng.random() < 0.8 else rng.randint(96, 256)
            classes = 1000 if rng.random() < 0.7 else _log(rng, 2, 1024)
            case = net_case(dtype, _log(rng, 1, 64), size, rng.choice((1, 2, 3, 4, 4)), classes,
                            rng.randint(1, 13) if rng.random() < 0.2 else 0)
        cost = work(case)
        if cost["flops"] <= MOST_FLOPS and cost["bytes"] <= MOST_BYTES:
            return case


def _dtype(case):
    return torch.float16 if case["dtype"] == "f16" else torch.float32


def _pad(case):
    return tfx.PAD_SAME if case["same"] else tfx.PAD_VALID


def _net_weights(case, normal):
    """He-normal filters and small biases, as a folded trained network has them in scale."""
    q = case["quarters"]
    c = 32 * q // 4
    w = {"conv0_w": normal((3, 3, 3, c), (2 / 27) ** 0.5), "conv0_b": normal((c,), 0.01)}
    w.update({k: [] for k in ("dw_w", "dw_b", "pw_w", "pw_b")})
    for full in CHANNELS:
        co = full * q // 4
        w["dw_w"].append(normal((3, 3, c, 1), (2 / 9) ** 0.5))
        w["dw_b"].append(normal((c,), 0.01))
        w["pw_w"].append(normal((1, 1, c, co), (2 / c) ** 0.5))
        w["pw_b"].append(normal((co,), 0.01))
        c = co
    w["fc_w"], w["fc_b"] = normal((c, case["classes"]), (2 / c) ** 0.5), normal((case["classes"],), 0.01)
    return w


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    dtype = _dtype(case)

    def normal(shape, std):
        return (torch.randn(shape, generator=gen, device="cuda") * std).to(dtype)

    def uniform(shape):
        return (torch.rand(shape, generator=gen, device="cuda") * 2 - 1).to(dtype)

    state = {"case": case}
    if case["kind"] == "matmul":
        m, k, n = case["m"], case["k"], case["n"]
        state["a"] = normal((case["batch"],) + ((k, m) if case["ta"] else (m, k)), 1.0)
        state["b"] = normal((case["batch"],) + ((n, k) if case["tb"] else (k, n)), 1.0)
        if case["batch"] == 1 and case["dtype"] == "f32":
            state["a"], state["b"] = state["a"][0], state["b"][0]
    elif case["kind"] == "conv":
        taps = case["fh"] * case["fw"] * case["cin"]
        state["x"] = uniform((case["n"], case["h"], case["w"], case["cin"]))
        state["filter"] = normal((case["fh"], case["fw"], case["cin"], case["cout"]), (2 / taps) ** 0.5)
        state["bias"] = normal((case["cout"],), 0.01)
    elif case["kind"] == "depthwise":
        state["x"] = uniform((case["n"], case["h"], case["w"], case["c"]))
        state["filter"] = normal((3, 3, case["c"], 1), (2 / 9) ** 0.5)
        state["bias"] = normal((case["c"],), 0.01)
    else:
        model = tfx.MobileNetV1F16 if case["dtype"] == "f16" else tfx.MobileNetV1
        state["model"] = model(_net_weights(case, normal), batch=case["batch"], image_size=case["size"],
                               width_quarters=case["quarters"])
        state["image"] = uniform((case["batch"], case["size"], case["size"], 3))
    return state


def run(state):
    case = state["case"]
    half = case["dtype"] == "f16"
    if case["kind"] == "matmul":
        if half:
            return tfx.tfx_batch_matmul_f16(state["a"], state["b"], case["ta"], case["tb"])
        if case["batch"] == 1:
            return tfx.tfx_matmul(state["a"], state["b"], case["ta"], case["tb"])
        return tfx.tfx_batch_matmul(state["a"], state["b"], case["ta"], case["tb"])
    if case["kind"] == "conv":
        conv = tfx.tfx_conv2d_f16 if half else tfx.tfx_conv2d
        return conv(state["x"], state["filter"], state["bias"], case["stride"], _pad(case), case["act"])
    if case["kind"] == "depthwise":
        conv = tfx.tfx_depthwise_conv2d_f16 if half else tfx.tfx_depthwise_conv2d
        return conv(state["x"], state["filter"], state["bias"], case["stride"], tfx.PAD_SAME, case["act"])
    if case["end_block"]:
        return state["model"].features(state["image"], case["end_block"])
    return state["model"].forward(state["image"])


def _ceil_div(v, d):
    return -(-v // d)


def work(case):
    size = 2 if case["dtype"] == "f16" else 4
    if case["kind"] == "matmul":
        b, m, k, n = case["batch"], case["m"], case["k"], case["n"]
        return {"bytes": size * b * (m * k + k * n + m * n), "flops": 2 * b * m * n * k}
    if case["kind"] == "conv":
        s, same = case["stride"], case["same"]
        oh, ow = (_ceil_div(e if same else e - f + 1, s) for e, f in ((case["h"], case["fh"]), (case["w"], case["fw"])))
        taps, pixels = case["fh"] * case["fw"] * case["cin"], case["n"] * oh * ow
        return {"bytes": size * (case["n"] * case["h"] * case["w"] * case["cin"] + pixels * case["cout"] +
                                 taps * case["cout"] + case["cout"]),
                "flops": 2 * pixels * taps * case["cout"]}
    if case["kind"] == "depthwise":
        pixels = case["n"] * _ceil_div(case["h"], case["stride"]) * _ceil_div(case["w"], case["stride"])
        return {"bytes": size * case["c"] * (case["n"] * case["h"] * case["w"] + pixels + 10),
                "flops": 18 * pixels * case["c"]}
    # a forward pass reads the image and the weights of the layers that run and writes its result; the feature maps
    # between the layers are not counted
    q, batch = case["quarters"], case["batch"]
    c, hw = 32 * q // 4, _ceil_div(case["size"], 2)
    flops, values = batch * hw * hw * 54 * c, batch * case["size"] ** 2 * 3 + 28 * c
    for i in range(case["end_block"] or 13):
        hw, co = _ceil_div(hw, STRIDES[i]), CHANNELS[i] * q // 4
        flops += batch * hw * hw * (18 * c + 2 * c * co)
        values += 10 * c + (c + 1) * co
        c = co
    if case["end_block"]:
        values += batch * hw * hw * c
    else:
        flops += 2 * batch * c * case["classes"]
        values += (c + 1) * case["classes"] + 2 * batch * case["classes"]
    return {"bytes": size * values, "flops": flops}


def tolerance(case):
    if case["dtype"] == "f32":
        # fp32 products and sums of up to a few thousand terms in another order
        return {"rel": 1e-5}
    if case["kind"] == "net":
        # up to 28 layers, each of which rounds its result to binary16; the last bits differ between implementations
        return {"rel": 1e-2, "max": 0.1}
    # one rounding of an fp32 sum to binary16
    return {"rel": 1e-3, "max": 5e-3}

"""The forward-convolution work a program gives this library, as measurable cases.

A case is one call (or, for the unfused route, one short sequence of calls) through the public entry
points of `paper_1910_00078_amd.cvx`: the create-once / execute-many plan, or for the smallest case the
one-call convenience function.  Sizes are those of the repository's benchmark layers and tests (residual-
network stages, the 224x224 stem, one tiny image) and generic ones between them.  Inputs follow the
benchmark's distributions: activations uniform, filters He-normal, bias uniform[-0.1, 0.1].

`family` names the range a case stands for; `draw` takes other sizes from the same ranges.
"""
import math

import torch

from paper_1910_00078_amd import cvx

TORCH_DTYPE = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
CVX_DTYPE = {"f32": cvx.CVX_F32, "f16": cvx.CVX_F16, "bf16": cvx.CVX_BF16}
ACT = {"identity": cvx.CVX_ACT_IDENTITY, "relu": cvx.CVX_ACT_RELU, "leaky": cvx.CVX_ACT_LEAKY_RELU}
LEAKY_SLOPE = 0.1
BN_EPS = 1e-5

# `route`: "call" conv_fwd_fused on tensors (descriptors, handle and output made by the call),
#          "plan" ConvPlan.run (bias + activation), "bn" ConvPlan.run_bn (bias + batch-norm + activation),
#          "unfused" ConvPlan.run_plain, then bias_add and activation_fwd on its output.


def _case(family, dtype, N, C, H, W, K, R=3, S=3, pad=(1, 1), stride=1, dil=1, groups=1, route="plan", act="relu"):
    return {"family": family, "route": route, "dtype": dtype, "N": N, "C": C, "H": H, "W": W, "K": K, "R": R, "S": S,
            "pad_h": pad[0], "pad_w": pad[1], "stride": stride, "dil": dil, "groups": groups, "act": act}


def listed():
    cases = {
        # the smallest problem of the set through the convenience call: descriptors, kernel choice and launch are all there is
        "tiny_f32_one_call": _case("tiny", "f32", 1, 8, 8, 8, 8, route="call"),
        # one image of a middle stage: latency of an interactive inference request, few blocks, a long reduction
        "single_image_bf16_3x3": _case("single", "bf16", 1, 256, 14, 14, 256),
        # the 56x56 stage of a training or serving batch
        "stage56_bf16_3x3": _case("stage", "bf16", 32, 64, 56, 56, 64),
        # 1x1 reduce in front of a 3x3: input-dominated, bandwidth-bound
        "reduce_bf16_1x1": _case("pointwise", "bf16", 64, 256, 56, 56, 64, 1, 1, (0, 0)),
        # 1x1 expand with the folded batch-norm of inference: output-dominated, bandwidth-bound
        "expand_bf16_1x1_bn": _case("pointwise", "bf16", 64, 64, 56, 56, 256, 1, 1, (0, 0), route="bn"),
        # the stem on RGB images: few channels, store-bound
        "stem_f16_7x7": _case("stem", "f16", 64, 3, 224, 224, 64, 7, 7, (3, 3), 2),
        # the deepest stage: tiny images, the longest reduction, matrix-pipe-bound
        "deep_bf16_3x3": _case("deep", "bf16", 128, 512, 7, 7, 512),
        # the strided convolution between two stages
        "down_bf16_3x3": _case("down", "bf16", 128, 256, 28, 28, 256, stride=2),
        # the 56x56 stage in full precision
        "stage56_f32_3x3": _case("fp32", "f32", 32, 64, 56, 56, 64),
        # another filter size on an odd image with channel counts that fill no tile, in the other 16-bit type
        "wide_f16_5x5_leaky": _case("wide", "f16", 16, 48, 35, 35, 72, 5, 5, (2, 2), act="leaky"),
        # depthwise: one channel per group, a reduction of nine
        "depthwise_bf16_3x3": _case("grouped", "bf16", 32, 128, 28, 28, 128, groups=128),
        # strided 1x1 shortcut as three separate operators: the route of a program that keeps the pre-activations' operators apart
        "shortcut_bf16_1x1_unfused": _case("shortcut", "bf16", 32, 256, 56, 56, 512, 1, 1, (0, 0), 2, route="unfused"),
    }
    return [dict(c, name=n) for n, c in cases.items()]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _channels(rng, lo, hi):
    """Channel counts: mostly multiples of 16 as networks have them, one in four anything."""
    c = _log_int(rng, lo, hi)
    return c if rng.random() < 0.25 else max(lo, (c + 8) // 16 * 16)


def _draw_family(family, rng):
    half = rng.choice(["bf16", "bf16", "f16"])
    act = rng.choice(["relu", "relu", "relu", "leaky", "identity"])
    if family == "tiny":
        return _case(family, rng.choice(["f32", half]), 1, rng.randint(3, 16), rng.randint(5, 12), rng.randint(5, 12), rng.randint(4, 16), route="call")
    if family == "single":
        s = rng.randint(7, 40)
        return _case(family, half, rng.randint(1, 4), _channels(rng, 48, 512), s, s, _channels(rng, 48, 512), act=act)
    if family == "stage":
        h = rng.randint(20, 72)
        return _case(family, half, _log_int(rng, 8, 64), _channels(rng, 32, 192), h, h + rng.choice([0, 0, rng.randint(0, 9)]),
                     _channels(rng, 32, 192), route=rng.choice(["plan", "bn"]), act=act)
    if family == "pointwise":
        s = _log_int(rng, 7, 72)
        return _case(family, half, _log_int(rng, 4, 64), _channels(rng, 32, 1024), s, s, _channels(rng, 32, 1024), 1, 1, (0, 0),
                     route=rng.choice(["plan", "bn"]), act=act)
    if family == "stem":
        s = _log_int(rng, 64, 256)
        return _case(family, half, _log_int(rng, 2, 64), 3, s, s, rng.choice([32, 48, 64, 64, 96]), 7, 7, (3, 3), 2)
    if family == "deep":
        s = rng.randint(6, 17)
        return _case(family, half, _log_int(rng, 16, 128), _channels(rng, 128, 512), s, s, _channels(rng, 128, 512), act=act)
    if family == "down":
        s = rng.randint(14, 57)
        return _case(family, half, _log_int(rng, 8, 128), _channels(rng, 64, 256), s, s, _channels(rng, 64, 320), stride=2,
                     route=rng.choice(["plan", "bn"]))
    if family == "fp32":
        r, s = rng.choice([3, 3, 1, 5]), rng.randint(10, 57)
        return _case(family, "f32", _log_int(rng, 1, 32), _channels(rng, 16, 256), s, s, _channels(rng, 16, 256), r, r, (r // 2, r // 2),
                     rng.choice([1, 1, 2]), act=act)
    if family == "wide":
        s = rng.randint(12, 40)
        r, q, d = rng.choice([(5, 5, 1), (5, 5, 1), (1, 7, 1), (7, 1, 1), (3, 3, 2)])
        return _case(family, half, _log_int(rng, 2, 32), _channels(rng, 16, 160), s, s, _channels(rng, 16, 160), r, q,
                     (r // 2 * d, q // 2 * d), dil=d, act=act)
    if family == "grouped":
        s, n = rng.randint(7, 57), _log_int(rng, 1, 32)
        per = rng.choice([1, 1, 4, 8, 16])
        g = rng.randint(2, 8) * 4 if per > 1 else _log_int(rng, 32, 384)
        return _case(family, half, n, g * per, s, s, g * per, stride=rng.choice([1, 1, 2]), groups=g, act=act)
    s = rng.randint(13, 57)
    return _case("shortcut", half, _log_int(rng, 4, 64), _channels(rng, 64, 512), s, s, _channels(rng, 64, 768), 1, 1, (0, 0), 2, route="unfused")


FAMILIES = ("tiny", "single", "stage", "pointwise", "stem", "deep", "down", "fp32", "wide", "grouped", "shortcut")


def _out_hw(case):
    f = lambda n, p, r: (n + 2 * p - case["dil"] * (r - 1) - 1) // case["stride"] + 1  # noqa: E731
    return f(case["H"], case["pad_h"], case["R"]), f(case["W"], case["pad_w"], case["S"])


def _elems(case):
    ho, wo = _out_hw(case)
    return (case["N"] * case["C"] * case["H"] * case["W"], case["K"] * (case["C"] // case["groups"]) * case["R"] * case["S"],
            case["N"] * case["K"] * ho * wo)


def work(case):
    x, w, y = _elems(case)
    e = 4 if case["dtype"] == "f32" else 2
    per_channel = case["K"] * (e + (16 if case["route"] == "bn" else 0))
    # the unfused operators are separate calls: each reads and writes the whole output again
    passes = 5 if case["route"] == "unfused" else 1
    return {"bytes": e * (x + w + passes * y) + per_channel,
            "flops": 2 * y * (case["C"] // case["groups"]) * case["R"] * case["S"]}


def draw(rng):
    """One more case of the listed ones' ranges, no larger than the largest of them."""
    while True:
        case = _draw_family(rng.choice(FAMILIES), rng)
        w = work(case)
        # fp32, depthwise and filter sizes other than 1x1 / 3x3 / 7x7 have a lower rate: fewer operations for the same time
        flops = 7.4e9 if case["family"] in ("fp32", "wide", "grouped") else 29.6e9
        mbytes = 30e6 if case["family"] == "grouped" else 130e6
        if w["flops"] <= flops and w["bytes"] <= mbytes:
            return case


def tolerance(case):
    # Measured against the same convolution in 64 bits over all families (drawn sizes among them), times about four.
    # Largest 2-norm error seen: fp32 9.4e-7 (sums of 2160), bf16 1.7e-3 and fp16 2.1e-4 (the one rounding of the
    # output), over three separate operators bf16 2.4e-3 and fp16 2.9e-4.  Largest single difference over the
    # root mean square or the value: fp32 7.3e-6, bf16 3.9e-3 (7.6e-3 unfused), fp16 4.9e-4 (9.2e-4).
    if case["dtype"] == "f32":
        return {"rel": 4e-6, "max": 3e-5}
    ops = 2.0 if case["route"] == "unfused" else 1.0
    if case["dtype"] == "bf16":
        return {"rel": 7e-3 if ops == 1.0 else 1e-2, "max": 1.6e-2 * ops}
    return {"rel": 9e-4 if ops == 1.0 else 1.2e-3, "max": 2e-3 * ops}


def prepare(case, seed):
    """What the caller holds before the call: tensors on the GPU, and for the plan routes the plan."""
    dt, dev = TORCH_DTYPE[case["dtype"]], "cuda"
    gen = torch.Generator(device=dev)
    gen.manual_seed(int(seed))
    cg = case["C"] // case["groups"]
    uniform = lambda shape, lo, hi: torch.empty(shape, device=dev).uniform_(lo, hi, generator=gen)  # noqa: E731
    lo = -1.0 if case["family"] in ("tiny", "stem") else 0.0
    st = {"case": case}
    st["x"] = uniform((case["N"], case["C"], case["H"], case["W"]), lo, 1.0).to(dt)
    st["w"] = torch.empty((case["K"], cg, case["R"], case["S"]), device=dev).normal_(0.0, math.sqrt(2.0 / (cg * case["R"] * case["S"])), generator=gen).to(dt)
    st["bias"] = uniform((case["K"],), -0.1, 0.1).to(dt)
    if case["route"] == "bn":
        st["bn"] = (uniform((case["K"],), 0.5, 1.5), uniform((case["K"],), -0.5, 0.5), uniform((case["K"],), -0.3, 0.3), uniform((case["K"],), 0.5, 2.0))
    if case["route"] != "call":
        st["plan"] = cvx.ConvPlan(CVX_DTYPE[case["dtype"]], tuple(st["x"].shape), tuple(st["w"].shape), (case["pad_h"], case["pad_w"]),
                                  case["stride"], case["dil"], case["groups"], stream=torch.cuda.current_stream().cuda_stream)
        st["y"] = torch.empty(st["plan"].y_shape, dtype=dt, device=dev)
    return st


def run(st):
    case = st["case"]
    act, alpha = ACT[case["act"]], LEAKY_SLOPE
    if case["route"] == "call":
        return cvx.conv_fwd_fused(st["x"], st["w"], st["bias"], pad=(case["pad_h"], case["pad_w"]), stride=case["stride"],
                                  dil=case["dil"], groups=case["groups"], act=act, alpha=alpha)
    plan, y = st["plan"], st["y"]
    x_ptr, w_ptr, b_ptr, y_ptr = st["x"].data_ptr(), st["w"].data_ptr(), st["bias"].data_ptr(), y.data_ptr()
    if case["route"] == "bn":
        scale, shift, mean, var = st["bn"]
        plan.run_bn(x_ptr, w_ptr, b_ptr, scale.data_ptr(), shift.data_ptr(), mean.data_ptr(), var.data_ptr(), BN_EPS, y_ptr, act, alpha)
    elif case["route"] == "unfused":
        plan.run_plain(x_ptr, w_ptr, y_ptr)
        cvx.cvx_bias_add(plan.h, plan.bd, b_ptr, plan.yd, y_ptr)
        cvx.cvx_activation_fwd(plan.h, act, alpha, plan.yd, y_ptr)
    else:
        plan.run(x_ptr, w_ptr, b_ptr, y_ptr, act, alpha)
    return y

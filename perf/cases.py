"""The work that the speed of this library is measured on.

Every case is one forward convolution through a public entry point of
``paper_2105_13480_amd.cnn``, as a program that runs a network calls it:

* ``"fwd"``   ``cnn.fwd`` (``cnn_fwd``): the plain call, no plan, no workspace;
* ``"plan"``  ``cnn.plan`` once per layer, then ``cnn.fwd_plan_ws`` with the
  workspace that the plan asks for, kept beside the layer's weights.

Types are the library's three: ``f32``, ``bf16`` (fp32 Out) and
``bf16_obf16`` (bf16 Out).  ``dims`` are (Nb, Nc, Nk, Nw, Nh, Nr, Ns, sw, sh):
the paper's batch, input and output features, output extent, stencil and
strides.

``python3 perf/cases.py`` lists the cases.
"""
from __future__ import annotations

import math

import torch

from paper_2105_13480_amd import cnn

DIMS = ("Nb", "Nc", "Nk", "Nw", "Nh", "Nr", "Ns", "sw", "sh")


def _case(name, api, dtype, *dims):
    case = {"name": name, "api": api, "dtype": dtype}
    case.update(zip(DIMS, dims))
    return case


def listed():
    return [
        # The smallest call: one image of 16 features, where the launch and
        # the host's share count (benchmark workload tiny3x3_f32).
        _case("tiny3x3_f32", "fwd", "f32", 1, 16, 16, 16, 16, 3, 3, 1, 1),
        # Inference on one image, a network's last stage: weights are nearly
        # all of the traffic (benchmark workload late3x3_b1), plain call with
        # the Out type that the next layer reads.
        _case("late3x3_b1", "fwd", "bf16_obf16", 1, 512, 512, 7, 7, 3, 3, 1, 1),
        # The same stage's 1x1 reduction through a kept plan (one of the
        # batch-1 deep layers of the tests).
        _case("late1x1_b1", "plan", "bf16", 1, 2048, 512, 7, 7, 1, 1, 1, 1),
        # The 3x3 layer of a residual network's first stage (benchmark
        # workload conv3x3_b32).
        _case("conv3x3_b32", "fwd", "bf16", 32, 64, 64, 56, 56, 3, 3, 1, 1),
        # The strided 3x3 layer, plan and workspace kept with the layer
        # (benchmark workload conv3x3_s2_b64, the benchmark's default).
        _case("conv3x3_s2_b64", "plan", "bf16", 64, 128, 256, 28, 28, 3, 3, 2, 2),
        # A bottleneck's 1x1 layer at a large batch, a pure matrix product
        # (benchmark workload pointwise_b256), bf16 activations throughout.
        _case("pointwise_b256", "fwd", "bf16_obf16", 256, 1024, 256, 14, 14, 1, 1, 1, 1),
        # The strided projection beside a stage's first block (benchmark
        # workload pointwise_s2_b64).
        _case("pointwise_s2_b64", "fwd", "bf16", 64, 256, 512, 28, 28, 1, 1, 2, 2),
        # The input layer: three channels, large stencil, large Out
        # (benchmark workload stem7x7_s2_b64).
        _case("stem7x7_s2_b64", "fwd", "bf16_obf16", 64, 3, 64, 112, 112, 7, 7, 2, 2),
        # A 3x3 layer at full image resolution, as the first stages of a plain
        # network or a decoder's last ones run it: rows of 226 positions.
        _case("wide3x3_b8", "fwd", "bf16_obf16", 8, 64, 64, 224, 224, 3, 3, 1, 1),
        # The first-stage 3x3 layer in full precision (training or reference
        # runs in fp32).
        _case("conv3x3_b16_f32", "fwd", "f32", 16, 64, 64, 56, 56, 3, 3, 1, 1),
        # A 1x1 layer in full precision.
        _case("pointwise_b16_f32", "fwd", "f32", 16, 256, 128, 28, 28, 1, 1, 1, 1),
        # Odd sizes everywhere: a 5x5 stencil on odd rows, odd feature counts.
        _case("ragged5x5_b8", "fwd", "bf16", 8, 75, 131, 35, 27, 5, 5, 1, 1),
    ]


# What a drawn case may cost at most: the floating-point operations and the
# bytes of the largest listed cases, and for fp32 (whose matrix rate is a
# sixteenth of bf16's) those of the largest listed fp32 case.
_MAX_FLOPS = {"f32": 3.7e9, "bf16": 2.9e10, "bf16_obf16": 2.9e10}
_MAX_BYTES = 2.2e8


def _log(rng, lo, hi):
    """A whole number spread evenly over the logarithm of [lo, hi]."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _features(rng, lo, hi):
    """A feature count: mostly multiples of 16, some of 8, some odd."""
    n = _log(rng, lo, hi)
    kind = rng.random()
    unit = 16 if kind < 0.6 else 8 if kind < 0.75 else 1
    return max(lo, (n + unit // 2) // unit * unit)


def _extent(rng, lo, hi):
    """An output extent: square three times in four."""
    w = _log(rng, lo, hi)
    return (w, w) if rng.random() < 0.75 else (w, _log(rng, lo, hi))


def _draw_small(rng):
    r = rng.choice((1, 3, 3, 5))
    s = rng.choice((1, 1, 2))
    return (1, _features(rng, 8, 64), _features(rng, 8, 64), *_extent(rng, 8, 32), r, r, s, s)


def _draw_deep(rng):
    r = rng.choice((1, 3))
    return (rng.choice((1, 1, 2)), _features(rng, 256, 2048), _features(rng, 128, 1024),
            *_extent(rng, 7, 14), r, r, 1, 1)


def _draw_conv3(rng):
    s = rng.choice((1, 1, 2))
    return (_log(rng, 4, 64), _features(rng, 32, 256), _features(rng, 32, 256),
            *_extent(rng, 14, 112), 3, 3, s, s)


def _draw_pointwise(rng):
    s = rng.choice((1, 1, 2))
    return (_log(rng, 4, 256), _features(rng, 64, 1024), _features(rng, 64, 512),
            *_extent(rng, 7, 56), 1, 1, s, s)


def _draw_stem(rng):
    r = rng.choice((3, 5, 7))
    return (_log(rng, 4, 64), rng.choice((1, 3, 3, 4)), _features(rng, 16, 96),
            *_extent(rng, 56, 160), r, r, 2, 2)


def _draw_wide(rng):
    return (_log(rng, 1, 8), _features(rng, 16, 128), _features(rng, 16, 128),
            *_extent(rng, 112, 256), 3, 3, 1, 1)


def _draw_f32(rng):
    r = rng.choice((1, 3, 3, 5))
    s = rng.choice((1, 1, 2))
    return (_log(rng, 1, 32), _features(rng, 16, 256), _features(rng, 16, 256),
            *_extent(rng, 7, 112), r, r, s, s)


def _draw_ragged(rng):
    nr, ns = rng.choice(((5, 5), (3, 5), (1, 7), (7, 1), (3, 2), (4, 4)))
    return (_log(rng, 1, 32), _features(rng, 9, 200), _features(rng, 9, 200),
            *_extent(rng, 9, 60), nr, ns, rng.choice((1, 1, 2)), rng.choice((1, 1, 2)))


_DRAWS = ((_draw_small, ("f32", "bf16", "bf16_obf16")), (_draw_deep, ("bf16", "bf16_obf16")),
          (_draw_conv3, ("bf16", "bf16_obf16")), (_draw_pointwise, ("bf16", "bf16_obf16")),
          (_draw_stem, ("bf16", "bf16_obf16")), (_draw_wide, ("bf16", "bf16_obf16")),
          (_draw_f32, ("f32",)), (_draw_ragged, ("bf16", "bf16_obf16")))


def draw(rng):
    """One more case: a network layer of one of the kinds listed above."""
    make, dtypes = rng.choice(_DRAWS)
    dims = list(make(rng))
    case = {"api": rng.choice(("fwd", "fwd", "plan")), "dtype": rng.choice(dtypes)}
    while True:
        case.update(zip(DIMS, dims))
        w = work(case)
        if w["flops"] <= _MAX_FLOPS[case["dtype"]] and w["bytes"] <= _MAX_BYTES:
            return case
        # too large: fewer images, then fewer rows
        i = 0 if dims[0] > 1 else 3
        dims[i] = max(1, dims[i] * 3 // 4)


def _dims(case):
    return tuple(case[d] for d in DIMS)


def _in_extent(case):
    return (case["sw"] * (case["Nw"] - 1) + case["Nr"], case["sh"] * (case["Nh"] - 1) + case["Ns"])


def _inputs(case, seed):
    """In uniform on [0, 1) as after an activation, Ker He-normal."""
    Nb, Nc, Nk, Nw, Nh, Nr, Ns, sw, sh = _dims(case)
    gen = torch.Generator(device="cuda").manual_seed(seed)
    In = torch.rand((Nb, Nc, *_in_extent(case)), device="cuda", generator=gen)
    Ker = torch.randn((Nk, Nc, Nr, Ns), device="cuda", generator=gen) * math.sqrt(2.0 / (Nc * Nr * Ns))
    if case["dtype"] != "f32":
        In, Ker = In.bfloat16(), Ker.bfloat16()
    return In, Ker


def prepare(case, seed):
    In, Ker = _inputs(case, seed)
    out_type = torch.bfloat16 if case["dtype"] == "bf16_obf16" else torch.float32
    Out = torch.empty((case["Nb"], case["Nk"], case["Nw"], case["Nh"]), dtype=out_type, device="cuda")
    state = {"In": In, "Ker": Ker, "Out": Out, "sw": case["sw"], "sh": case["sh"], "plan": None}
    if case["api"] == "plan":
        plan = cnn.plan(cnn.problem(*_dims(case)), cnn.DTYPES[case["dtype"]])
        state["plan"] = plan
        state["ws"] = torch.empty(plan.ws_bytes, dtype=torch.uint8, device="cuda") if plan.ws_bytes else None
    return state


def run(state):
    if state["plan"] is None:
        return cnn.fwd(state["In"], state["Ker"], state["Out"], state["sw"], state["sh"])
    return cnn.fwd_plan_ws(state["In"], state["Ker"], state["Out"], state["plan"], state["ws"],
                           state["sw"], state["sh"])


def work(case):
    """In elements that some output reads, Ker and Out once each."""
    Nb, Nc, Nk, Nw, Nh, Nr, Ns, sw, sh = _dims(case)
    Nx, Ny = _in_extent(case)
    rows = Nw * Nr if sw >= Nr else Nx
    cols = Nh * Ns if sh >= Ns else Ny
    e_in = 4 if case["dtype"] == "f32" else 2
    e_out = 2 if case["dtype"] == "bf16_obf16" else 4
    return {"bytes": e_in * (Nb * Nc * rows * cols + Nk * Nc * Nr * Ns) + e_out * Nb * Nk * Nw * Nh,
            "flops": 2 * Nb * Nk * Nc * Nr * Ns * Nw * Nh}


def tolerance(case):
    """About four times the largest error against 64 bits that the path
    showed over the listed and some drawn cases: sums of products in fp32
    (bf16 products are exact in fp32), and one rounding to bf16 where Out is
    bf16."""
    if case["dtype"] == "bf16_obf16":
        return {"rel": 7e-3, "max": 6e-2}
    return {"rel": 4e-6, "max": 4e-5}


def exact(case, seed):
    """The same convolution in 64 bits: one matrix product per stencil tap."""
    Nb, Nc, Nk, Nw, Nh, Nr, Ns, sw, sh = _dims(case)
    In, Ker = _inputs(case, seed)
    Out = torch.zeros((Nb, Nk, Nw * Nh), dtype=torch.float64, device="cuda")
    for r in range(Nr):
        for s in range(Ns):
            taken = In[:, :, r:r + sw * (Nw - 1) + 1:sw, s:s + sh * (Nh - 1) + 1:sh]
            taken = taken.to(torch.float64).reshape(Nb, Nc, Nw * Nh)
            tap = Ker[:, :, r, s].to(torch.float64).contiguous()
            for b in range(Nb):
                Out[b].addmm_(tap, taken[b])
    return Out.reshape(Nb, Nk, Nw, Nh)


if __name__ == "__main__":
    for c in listed():
        w = work(c)
        print(f"{c['name']:20s} {c['api']:5s} {c['dtype']:11s} {_dims(c)} "
              f"{w['flops'] / 1e9:.3f} GFLOP {w['bytes'] / 1e6:.2f} MB")

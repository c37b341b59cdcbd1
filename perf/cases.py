"""Performance cases of the SFC int8 convolution: what a user's program has the library do.

A case is one layer (``kind = "layer"``) or the 13 stride-1 3x3 layers of the ResNet-18-shaped
stack of ``synth`` run back to back (``kind = "stack"``).  The layer is planned, calibrated and
its filter transformed once in ``prepare``, as a program does when it loads a model; ``run`` is
one pass over a batch that lies in device memory, into an output the program keeps, on the
current stream.  The library chooses algorithm and path for 3x3 filters; for 5x5 and 7x7 filters
the caller names the algorithm.

The path is inference only (there is no backward), the operands are int8, and what differs in
use is the shape, the filter size, the mode (requantized transform domain, or exact) and what
comes out: float32 for a layer whose consumer is another library's, int8 + ReLU between layers,
the raw int32 sums in exact mode.
"""
import math

import torch

from paper_2407_02913_amd import binding, layers, synth

X_SCALE = 0.02  # activation scale of the synthetic layers, as in synth.make_layer
ALG_OF_FILTER = {3: "auto", 5: "6x6_5x5_p184", 7: "4x4_7x7_p184"}
TILE = {"6x6_p88": 6, "7x7_p132": 7, "4x4_p46": 4, "6x6_5x5_p184": 6, "4x4_7x7_p184": 4}
POINTS = {"6x6_p88": 88, "7x7_p132": 132, "4x4_p46": 46, "6x6_5x5_p184": 184, "4x4_7x7_p184": 184}


def layer(name, N, Cin, Cout, H, W, R=3, mode="requant", out="f32", bits=8):
    case = {"kind": "layer", "N": N, "Cin": Cin, "Cout": Cout, "H": H, "W": W, "R": R, "mode": mode,
            "out": out, "bits": bits}
    return dict(case, name=name) if name else case


def listed():
    return [
        # The smallest call: synth's tiny32 (one image, few channels); host and launch time count.
        layer("tiny_b1", 1, 16, 16, 32, 32),
        # A whole network's 3x3 layers for a single image, the latency of interactive inference:
        # 13 dependent layers, each too small to fill the chip.
        {"name": "stack_b1", "kind": "stack", "N": 1},
        # The same at the batch the throughput benchmark runs (bench.py's headline).
        {"name": "stack_b64", "kind": "stack", "N": synth.STACK_BATCH},
        # The four ResNet-shaped layers of synth.LAYERS, each at its own batch: wide maps with few
        # channels to 7x7 maps with 512.  resnet28 hands int8 activations on.
        layer("c64_s56_b32", 32, 64, 64, 56, 56),
        layer("c128_s28_b64_i8", 64, 128, 128, 28, 28, out="i8"),
        layer("c256_s14_b128", 128, 256, 256, 14, 14),
        layer("c512_s7_b256", 256, 512, 512, 7, 7),
        # The first 64 -> 64 layer of a VGG-16-shaped network: the largest maps, int8 handed on.
        layer("c64_s224_b32_i8", 32, 64, 64, 224, 224, out="i8"),
        # Odd everything: channel counts that fill no block, a map no tile divides, a small batch.
        layer("ragged_b7", 7, 184, 136, 31, 45),
        # The larger filters on the 28x28 geometry, as bench.py runs them.
        layer("filter5_c128_s28_b64", 64, 128, 128, 28, 28, R=5),
        layer("filter7_c128_s28_b64", 64, 128, 128, 28, 28, R=7),
        # Exact mode (bit-equal to direct convolution), raw sums out.
        layer("exact_c64_s56_b32", 32, 64, 64, 56, 56, mode="exact", out="i32"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _channels(rng, hi):
    """Half the layers have the round counts of real networks, half any count."""
    if rng.random() < 0.5:
        return rng.choice([c for c in (16, 32, 64, 128, 256, 512) if c <= hi])
    return _log_int(rng, 16, hi)


def draw(rng):
    kind = rng.random()
    if kind < 0.15:
        return {"kind": "stack", "N": rng.choice([n for n in range(2, synth.STACK_BATCH)])
                if rng.random() < 0.5 else _log_int(rng, 2, synth.STACK_BATCH - 1)}
    exact, r = kind > 0.9, 3
    if kind > 0.72 and not exact:
        r = 5 if rng.random() < 0.5 else 7
    while True:
        if rng.random() < 0.5:  # the resolutions of a network, else any map
            h = w = rng.choice([7, 14, 28, 56, 112, 224])
        else:
            h = _log_int(rng, 7, 224)
            w = h if rng.random() < 0.3 else max(7, min(224, int(h * rng.uniform(0.5, 2.0))))
        cin, n = _channels(rng, 256 if exact else 512), _log_int(rng, 1, 256)
        cout = cin if rng.random() < 0.5 else _channels(rng, 256 if exact else 512)
        out = "i32" if exact else rng.choice(["f32", "i8"])
        bits = 8 if exact or rng.random() < 0.8 else rng.choice([4, 6])
        case = layer(None, n, cin, cout, h, w, R=r, mode="exact" if exact else "requant", out=out, bits=bits)
        need = work(case)
        if need["bytes"] <= 2.1e8 and need["flops"] <= (2.4e9 if exact else 1.8e10):
            return case


def _algorithm(case):
    """(tile edge, points) of the algorithm that runs the layer; the library's rule where it chooses."""
    if case["R"] != 3:
        alg = ALG_OF_FILTER[case["R"]]
    else:
        plan = binding.Plan(case["N"], case["Cin"], case["Cout"], case["H"], case["W"], alg="auto",
                            mode=case["mode"], out=case["out"], path="auto")
        alg = plan.alg
        plan.close()
    return TILE[alg], POINTS[alg]


def work(case):
    """Activations, transformed filter and output once each; the products of the algorithm."""
    if case["kind"] == "stack":
        total = {"bytes": 0, "flops": 0}
        for shape, out in _stack(case["N"]):
            one = work(layer(None, shape.N, shape.Cin, shape.Cout, shape.H, shape.W, out=out))
            total = {k: total[k] + one[k] for k in total}
        return total
    n, cin, cout, h, w = (case[k] for k in ("N", "Cin", "Cout", "H", "W"))
    m, p = _algorithm(case)
    tiles = n * -(-h // m) * -(-w // m)
    operand = 2 if case["mode"] == "exact" else 1
    y = n * cout * h * w * (1 if case["out"] == "i8" else 4)
    return {"bytes": n * cin * h * w + operand * p * cin * cout + y, "flops": 2 * p * tiles * cin * cout}


def tolerance(case):
    if case["kind"] == "stack":
        # float32 results behind up to three layers of int8 activations: an activation within
        # float32 reach of a rounding boundary may go either way, and a step of one activation
        # (1/32 of their standard deviation) moves those of the layers behind it
        return {"rel": 1e-2}
    if case["out"] == "i32":
        return "exact"
    if case["out"] == "i8":
        return {"rel": 0.0, "differ": 1e-3}  # ties of the final rounding
    return {"rel": 1e-5}


def _stack(batch):
    """The layers of the stack and what each puts out: int8 to the next layer of its resolution,
    float32 from the last one (a stride-2 layer follows, which is not part of this path)."""
    shapes = synth.stack_layers(batch)
    return [(s, "i8" if i + 1 < len(shapes) and shapes[i + 1].H == s.H else "f32")
            for i, s in enumerate(shapes)]


def _activations(shape, gen):
    a = torch.randn(shape, generator=gen, device="cuda").mul_(30.0).abs_()
    return a.round_().clamp_(0, 127).to(torch.int8)


class _Ready:
    """A layer ready to run: plan, scales, transformed filter."""

    def __init__(self, case, gen):
        n, cin, cout, h, w, r = (case[k] for k in ("N", "Cin", "Cout", "H", "W", "R"))
        requant = case["mode"] == "requant"
        bits = case["bits"] if requant and case["bits"] != 8 else 0
        weights = torch.randn((cout, cin, r, r), generator=gen, device="cuda").mul_(20.0)
        weights = weights.round_().clamp_(-127, 127).to(torch.int8)
        wscale = torch.rand(cout, generator=gen, device="cuda").mul_(0.015).add_(0.005).cpu().numpy()
        self.plan = binding.Plan(n, cin, cout, h, w, alg=ALG_OF_FILTER[r], mode=case["mode"],
                                 out=case["out"], path="auto", transform_bits=bits)
        if requant:
            sample = _activations((min(n, 4), cin, h, w), gen)
            calib = binding.Plan(sample.shape[0], cin, cout, h, w, alg=self.plan.alg, mode="requant",
                                 path="staged", transform_bits=bits)
            scratch = binding.device_buffer(calib.workspace_bytes)
            sx = calib.calibrate_act_scales(sample, scratch)
            self.plan.set_point_scales(sx, calib.calibrate_filter_scales(weights, scratch))
            calib.close()
        if case["out"] == "i8":
            self.plan.set_output_scale(layers.output_scale(cin, r, X_SCALE))
        self.filter = binding.device_buffer(self.plan.filter_bytes)
        self.plan.transform_filter(weights, wscale, self.filter)

    def output(self):
        d = self.plan.desc
        dtype = {"f32": torch.float32, "i8": torch.int8, "i32": torch.int32}[self.plan.out]
        return torch.empty((d.N, d.Cout, d.H, d.W), dtype=dtype, device="cuda")


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    if case["kind"] == "layer":
        x = _activations((case["N"], case["Cin"], case["H"], case["W"]), gen)
        one = _Ready(case, gen)
        return {"steps": [(one, x, one.output())], "results": [0],
                "workspace": binding.device_buffer(one.plan.workspace_bytes)}
    steps, results, x = [], [], None
    for shape, out in _stack(case["N"]):
        if x is None:  # the first layer of a resolution
            x = _activations((shape.N, shape.Cin, shape.H, shape.W), gen)
        one = _Ready(layer(None, shape.N, shape.Cin, shape.Cout, shape.H, shape.W, out=out), gen)
        y = one.output()
        steps.append((one, x, y))
        x = y
        if out == "f32":
            results.append(len(steps) - 1)
            x = None
    need = max(one.plan.workspace_bytes for one, _, _ in steps)
    return {"steps": steps, "results": results, "workspace": binding.device_buffer(need)}


def run(state):
    workspace = state["workspace"]
    for one, x, y in state["steps"]:
        one.plan.conv2d(x, X_SCALE, y, workspace)
    return [state["steps"][i][2] for i in state["results"]]

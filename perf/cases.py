"""The work users have libdora do, as cases that can be timed and whose results can be compared.

A case is a dict of plain values.  `kind` says which calls one pass makes:

  infer      dora_forward / dora_forward_fused keeping nothing, with the row norm that a serving program computed
             once (`norm` "kept") or with the norm inside the call ("inside")
  train      dora_forward saving h, inner and w_norm, then dora_backward from them (`fused`: dora_forward_fused)
  recompute  forward of one or several modules in order keeping nothing, then dora_backward of each in reverse
             order with norm, h and inner recomputed: the gradient-checkpointing pattern
  dropout    dora_forward_dropout and dora_backward_dropout: the adapter branch has its own (dropped) input
  norm       dora_norm alone

Inputs follow the recipe of paper_2603_22276_amd/inputs.py (W, A ~ N(0, 1/d_in), x, dy ~ N(0, 1), s = alpha/sqrt(r),
m = ||W||_row (1 + 1e-3 N(0, 1))), drawn on the device, with B at the scale of an adapter some way into training:
the low-rank branch carries a quarter of the frozen layer's standard deviation.
"""
import torch

from paper_2603_22276_amd import binding as D

DEV = "cuda:0"
TORCH_TYPE = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
CODE = {"f32": D.DORA_F32, "bf16": D.DORA_BF16, "f16": D.DORA_F16}
BRANCH = 0.25   # s * sigma_B * sqrt(r): standard deviation of the low-rank branch against the frozen layer's

# (d_out, d_in) of the MLP pair and of the seven adapted modules of a decoder layer that bench.py times
MLP_PAIR = "27648x5120,5120x27648"
DECODER_LAYER = "4096x4096,1024x4096,1024x4096,4096x4096,14336x4096,14336x4096,4096x14336"


def listed():
    return [
        # serving, one sequence: every token of the answer is such a call per adapted module; launches and latency count
        {"name": "decode_one_token", "kind": "infer", "modules": "4096x4096", "r": 384, "tokens": 1, "dtype": "bf16",
         "fused": True, "norm": "kept", "bias": False},
        # serving, a batch of sequences decoded together, fp16 storage, a base layer with bias, a wide MLP module
        {"name": "decode_batch_f16", "kind": "infer", "modules": "14336x4096", "r": 64, "tokens": 27, "dtype": "f16",
         "fused": True, "norm": "kept", "bias": True},
        # the fp32 module of the benchmark (256 x 512, r 16, 64 tokens) as a training step: a dozen tiny launches
        {"name": "f32_small_step", "kind": "train", "modules": "256x512", "r": 16, "tokens": 64, "dtype": "f32", "fused": False,
         "frozen_m": False},
        # fp32 training of an ordinary small layer, no dimension a multiple of a tile
        {"name": "f32_ragged_step", "kind": "train", "modules": "1000x772", "r": 36, "tokens": 1500, "dtype": "f32",
         "fused": False, "frozen_m": False},
        # a short fine-tuning batch through a key / value projection
        {"name": "kv_short_step", "kind": "train", "modules": "1024x4096", "r": 64, "tokens": 512, "dtype": "bf16", "fused": False,
         "frozen_m": False},
        # the 4096-module workload of the benchmark: one forward, norm inside
        {"name": "forward_4096", "kind": "infer", "modules": "4096x4096", "r": 384, "tokens": 4096, "dtype": "bf16", "fused": False,
         "norm": "inside", "bias": False},
        # serving, prompt of a ragged length through a wide MLP module
        {"name": "prefill_ragged", "kind": "infer", "modules": "14336x4096", "r": 64, "tokens": 1999, "dtype": "bf16",
         "fused": True, "norm": "kept", "bias": False},
        # the headline workload: training step of an 8192 x 8192 module
        {"name": "train_8192", "kind": "train", "modules": "8192x8192", "r": 384, "tokens": 8192, "dtype": "bf16", "fused": False,
         "frozen_m": False},
        # the MLP pair of the benchmark under gradient checkpointing: the largest call
        {"name": "mlp_pair_recompute", "kind": "recompute", "modules": MLP_PAIR, "r": 384, "tokens": 8192, "dtype": "bf16",
         "frozen_m": False},
        # one decoder layer of the benchmark's sweep, its seven modules under gradient checkpointing
        {"name": "decoder_layer_recompute", "kind": "recompute", "modules": DECODER_LAYER, "r": 384, "tokens": 4096, "dtype": "bf16",
         "frozen_m": False},
        # training with LoRA dropout, fp16 storage, ragged everywhere
        {"name": "dropout_f16_ragged", "kind": "dropout", "modules": "2056x3000", "r": 72, "tokens": 1501, "dtype": "f16",
         "frozen_m": False},
        # the norm by itself (after an optimiser step, before serving), as in the benchmark's rank sweep
        {"name": "norm_8192", "kind": "norm", "modules": "8192x8192", "r": 128, "tokens": 0, "dtype": "bf16"},
    ]


def _log(rng, lo, hi, mult):
    """A multiple of `mult` between lo and hi, spread evenly over the logarithm."""
    v = lo * (hi / lo) ** rng.random()
    return max(mult, int(round(v / mult)) * mult)


def draw(rng):
    most = max(work(c)["flops"] for c in listed())
    while True:
        case = _draw(rng)
        if work(case)["flops"] <= most:
            return case


def _draw(rng):
    kind = rng.choice(["infer", "infer", "infer", "train", "train", "train", "recompute", "dropout", "norm"])
    half = rng.choice(["bf16", "bf16", "f16"])
    if kind == "infer":
        # decode (a few tokens) as often as prefill; the norm is inside the call now and then
        tokens = _log(rng, 1, 64, 1) if rng.random() < 0.5 else _log(rng, 65, 8192, 1)
        fused = rng.random() < 0.7
        return {"kind": kind, "modules": "%dx%d" % (_log(rng, 512, 16384, 8), _log(rng, 512, 16384, 8)), "r": _log(rng, 8, 768, 8),
                "tokens": tokens, "dtype": half, "fused": fused, "norm": "kept" if rng.random() < 0.7 else "inside",
                "bias": rng.random() < 0.3}
    if kind == "train" and rng.random() < 0.4:
        return {"kind": kind, "modules": "%dx%d" % (_log(rng, 64, 2048, 4), _log(rng, 64, 2048, 4)), "r": _log(rng, 4, 128, 4),
                "tokens": _log(rng, 16, 2048, 1), "dtype": "f32", "fused": False, "frozen_m": rng.random() < 0.2}
    if kind == "train":
        return {"kind": kind, "modules": "%dx%d" % (_log(rng, 512, 14336, 8), _log(rng, 512, 14336, 8)), "r": _log(rng, 8, 768, 8),
                "tokens": _log(rng, 128, 8192, 1), "dtype": half, "fused": rng.random() < 0.4, "frozen_m": rng.random() < 0.2}
    if kind == "recompute":
        modules = ",".join("%dx%d" % (_log(rng, 512, 27648, 8), _log(rng, 512, 14336, 8)) for _ in range(rng.randint(1, 4)))
        return {"kind": kind, "modules": modules, "r": _log(rng, 16, 768, 8), "tokens": _log(rng, 512, 8192, 1), "dtype": half,
                "frozen_m": rng.random() < 0.2}
    if kind == "dropout":
        return {"kind": kind, "modules": "%dx%d" % (_log(rng, 512, 8192, 8), _log(rng, 512, 8192, 8)), "r": _log(rng, 8, 512, 8),
                "tokens": _log(rng, 128, 8192, 1), "dtype": half, "frozen_m": rng.random() < 0.2}
    return {"kind": kind, "modules": "%dx%d" % (_log(rng, 512, 27648, 8), _log(rng, 512, 27648, 8)), "r": _log(rng, 8, 1024, 8),
            "tokens": 0, "dtype": half}


def _shapes(case):
    return [tuple(int(v) for v in m.split("x")) for m in case["modules"].split(",")]


class _Module:
    """One module as a program holds it: weights, inputs, outputs and one workspace per direction, on the GPU."""

    def __init__(self, case, d_out, d_in, gen):
        kind, T, r = case["kind"], case["tokens"], case["r"]
        dt = TORCH_TYPE[case["dtype"]]
        alpha = 16.0 if case["dtype"] == "f32" else 32.0
        s = alpha / r ** 0.5

        def normal(shape, std=1.0, dtype=dt):
            v = torch.randn(shape, generator=gen, device=DEV, dtype=torch.float32)
            return (v * std if std != 1.0 else v).to(dtype)

        def out(*shape, dtype=dt):
            return torch.full(shape, float("nan"), dtype=dtype, device=DEV)

        def scratch(*phases):
            n = max(D.dora_workspace_bytes(self.desc, p) for p in phases)
            return torch.empty(n, dtype=torch.uint8, device=DEV)

        self.desc = D.make_desc(d_out, d_in, r, T, CODE[case["dtype"]], s)
        self.W = normal((d_out, d_in), d_in ** -0.5)
        self.A = normal((r, d_in), d_in ** -0.5)
        self.B = normal((d_out, r), BRANCH / (s * r ** 0.5))
        self.c = out(d_out, dtype=torch.float32)
        if kind == "norm":
            self.ws = scratch(D.PHASE_NORM)
            return
        self.m = torch.linalg.vector_norm(self.W, dim=1, dtype=torch.float32) * (1 + 1e-3 * normal((d_out,), dtype=torch.float32))
        self.x = normal((T, d_in))
        self.y = out(T, d_out)
        self.bias = normal((d_out,)) if case.get("bias") else None
        self.w_norm = self.h = self.inner = None
        if kind == "infer":
            self.ws = scratch(D.PHASE_FORWARD)
            if case["norm"] == "kept":
                self.w_norm = out(d_out, dtype=torch.float32)
                D.dora_norm(self.desc, self.W, self.A, self.B, self.w_norm, scratch(D.PHASE_NORM))
            return
        self.dy = normal((T, d_out))
        if kind != "recompute":
            self.h, self.inner = out(T, r), out(T, d_out)
        if kind == "dropout":
            keep = torch.rand((T, d_in), generator=gen, device=DEV) >= 0.1
            self.x_lora = (self.x * keep / 0.9).to(dt)
            self.dx_lora = out(T, d_in)
        self.dx = out(T, d_in)
        self.dA, self.dB = out(r, d_in, dtype=torch.float32), out(d_out, r, dtype=torch.float32)
        self.dm = None if case["frozen_m"] else out(d_out, dtype=torch.float32)
        self.ws = scratch(D.PHASE_FORWARD_DROPOUT if kind == "dropout" else D.PHASE_FORWARD)
        self.ws_bwd = scratch({"train": D.PHASE_BACKWARD, "recompute": D.PHASE_BACKWARD_RECOMPUTE, "dropout": D.PHASE_BACKWARD_DROPOUT}[kind])


def prepare(case, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    return {"case": case, "modules": [_Module(case, d_out, d_in, gen) for d_out, d_in in _shapes(case)]}


def run(state):
    case, modules = state["case"], state["modules"]
    kind = case["kind"]
    if kind == "norm":
        (q,) = modules
        D.dora_norm(q.desc, q.W, q.A, q.B, q.c, q.ws)
        return {"w_norm": q.c}
    forward = D.dora_forward_fused if case.get("fused") else D.dora_forward
    if kind == "infer":
        (q,) = modules
        forward(q.desc, q.x, q.W, q.A, q.B, q.m, q.w_norm, q.bias, q.y, None, None, None, q.ws)
        return {"y": q.y}
    if kind == "train":
        (q,) = modules
        forward(q.desc, q.x, q.W, q.A, q.B, q.m, None, None, q.y, q.h, q.inner, q.c, q.ws)
        D.dora_backward(q.desc, q.dy, q.x, q.W, q.A, q.B, q.m, q.c, q.h, q.inner, q.dx, q.dA, q.dB, q.dm, q.ws_bwd)
        return {"y": q.y, "w_norm": q.c, "dx": q.dx, "dA": q.dA, "dB": q.dB, "dm": q.dm}
    if kind == "dropout":
        (q,) = modules
        D.dora_forward_dropout(q.desc, q.x, q.x_lora, q.W, q.A, q.B, q.m, None, None, q.y, q.h, q.inner, q.c, q.ws)
        D.dora_backward_dropout(q.desc, q.dy, q.x_lora, q.W, q.A, q.B, q.m, q.c, q.h, q.inner, q.dx, q.dx_lora, q.dA, q.dB, q.dm,
                                q.ws_bwd)
        return {"y": q.y, "w_norm": q.c, "dx": q.dx, "dx_lora": q.dx_lora, "dA": q.dA, "dB": q.dB, "dm": q.dm}
    for q in modules:
        forward(q.desc, q.x, q.W, q.A, q.B, q.m, None, None, q.y, None, None, None, q.ws)
    for q in reversed(modules):
        D.dora_backward(q.desc, q.dy, q.x, q.W, q.A, q.B, q.m, None, None, None, q.dx, q.dA, q.dB, q.dm, q.ws_bwd)
    return [{"y": q.y, "dx": q.dx, "dA": q.dA, "dB": q.dB, "dm": q.dm} for q in modules]


def work(case):
    kind, T, r = case["kind"], case["tokens"], case["r"]
    e = 4 if case["dtype"] == "f32" else 2
    bytes_, flops = 0, 0
    for do, di in _shapes(case):
        weights = e * (do * di + r * di + do * r)
        norm_flops = 2 * do * di * (r + 1) + 2 * r * r * di + 2 * do * r * (r + 1)   # cross and base term, Gram matrix, B G
        if kind == "norm":
            bytes_ += weights + 4 * do
            flops += norm_flops
            continue
        big, low = 2 * T * do * di, 2 * T * r * (do + di)      # x W^T; x A^T and h B^T
        forward = big + low + 6 * T * do
        # forward: weights, m and x in, y out
        bytes_ += weights + 4 * do + e * T * (di + do)
        flops += forward
        if kind == "infer":
            bytes_ += (4 * do if case["norm"] == "kept" else 0) + (e * do if case["bias"] else 0)
            flops += norm_flops if case["norm"] == "inside" else 0
            continue
        flops += norm_flops
        # backward: weights, m, x, dy in, dx and the weight gradients out; dz B, dz W + dh A, dh^T x, dz^T h
        bytes_ += weights + 4 * do + e * T * (2 * di + do) + 4 * (r * di + do * r)
        flops += big + 2 * low + T * do
        if not case["frozen_m"]:
            bytes_ += 4 * do
            flops += 2 * T * do
        if kind == "recompute":
            # h is needed for dB; inner (x W^T, h B^T) only for dm
            flops += norm_flops + (2 * T * r * di if case["frozen_m"] else forward)
            continue
        bytes_ += 2 * e * T * r + 2 * 4 * do                   # h and the norm, written and read
        bytes_ += e * T * do * (1 if case["frozen_m"] else 2)  # inner: written, and read for dm
        if kind == "dropout":
            bytes_ += e * T * (di + di + di)                   # x_lora in both directions, dx_lora
            flops += 2 * big                                   # x_lora W^T; dy W beside ((g-1) dy) W
    return {"bytes": bytes_, "flops": flops}


def tolerance(case):
    # About four times the difference from the same path in 64 bits, over the listed cases and drawn ones:
    # rel / max  bf16 2.4e-3 / 1.4e-2 (2.9e-3 / 1.3e-2 for dx_lora), fp16 3.6e-4 / 1.7e-3, fp32 9.1e-7 / 4.8e-6,
    # the row norm (fp32 for every storage type) 1.0e-6 / 1.4e-6
    if case["kind"] == "norm":
        return {"rel": 4e-6, "max": 8e-6}
    if case["dtype"] == "f32":
        return {"rel": 4e-6, "max": 2e-5}
    if case["dtype"] == "f16":
        return {"rel": 1.5e-3, "max": 7e-3}
    return {"rel": 1.2e-2 if case["kind"] == "dropout" else 1e-2, "max": 5e-2}

"""Input and weight gradients in one launch, in each of its tiles and on both sides of the lines between it and launches of
their own; each gradient left out in turn."""
import pytest
import torch

from paper_2603_22276_amd import binding as D

import gpu_util as G
from test_gpu_rounds import Inputs, close

pytestmark = pytest.mark.gpu

SHAPES = [  # d_out, d_in, r, tokens: tiles of dx and, in 128 x 128, of dA and dB
    (520, 4104, 40, 500),       # 132 of 128 x 128, 33, 5: one to a CU, ragged
    (9728, 2560, 8, 1024),      # 160, 20, 76: 256, every CU
    (9736, 2560, 8, 1024),      # 160, 20, 77: one more than CUs
    (512, 4096, 16, 1500),      # 384, 32, 4: two to a CU
    (1160, 2304, 40, 4090),     # 144 of 256 x 256, 18, 10
    (1160, 2304, 264, 4090),    # 144 of 256 x 256, 54, 30: the same, two and a bit tiles of the rank
    (1032, 4096, 24, 6144),     # 384 of 256 x 256 in two rounds, 32, 9
    (136, 264, 8, 70),          # dx split over K or a single round of a few tiles
]


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("d_out,d_in,r,tokens", SHAPES)
def test_gradients_together(dtype, d_out, d_in, r, tokens):
    q = Inputs(d_out, d_in, r, tokens, dtype)
    dy, xl, W, A, B = (t.double() for t in (q.dy, q.xl, q.W, q.A, q.B))
    h = xl @ A.T
    q.h.copy_(h)
    q.inner.copy_(xl @ W.T + q.s * h @ B.T)
    dz = q.g * dy
    dh = q.s * dz @ B
    every = slice(None)
    ref = {"dx": dz @ W + dh @ A, "dA": dh.T @ xl, "dB": q.s * dz.T @ h}
    ws = q.ws(D.PHASE_BACKWARD)
    for want in (("dx", "dA", "dB"), ("dx", "dA"), ("dx", "dB"), ("dA", "dB")):
        got = {"dx": torch.full_like(q.dx, float("nan")), "dA": G.empty_f32(r, d_in).fill_(float("nan")),
               "dB": G.empty_f32(d_out, r).fill_(float("nan"))}
        got = {k: v if k in want else None for k, v in got.items()}
        D.dora_backward(q.desc, q.dy, q.xl, q.W, q.A, q.B, q.m, q.c, q.h, q.inner, got["dx"], got["dA"], got["dB"], None, ws)
        for k in want:
            close(k, got[k], (ref[k], every), dtype)
    ref["dx_lora"] = ((q.g - 1) * dy) @ W + dh @ A
    ref["dx"] = dy @ W
    ws = q.ws(D.PHASE_BACKWARD_DROPOUT)
    for want in (("dx", "dx_lora", "dA", "dB"), ("dx_lora", "dA", "dB"), ("dx", "dB")):
        got = {"dx": torch.full_like(q.dx, float("nan")), "dx_lora": torch.full_like(q.dx, float("nan")),
               "dA": G.empty_f32(r, d_in).fill_(float("nan")), "dB": G.empty_f32(d_out, r).fill_(float("nan"))}
        got = {k: v if k in want else None for k, v in got.items()}
        D.dora_backward_dropout(q.desc, q.dy, q.xl, q.W, q.A, q.B, q.m, q.c, q.h, q.inner, got["dx"], got["dx_lora"], got["dA"],
                                got["dB"], None, ws)
        for k in want:
            close(k, got[k], (ref[k], every), dtype)


@pytest.mark.parametrize("d_out,d_in,r,tokens,together", [
    (512, 4096, 16, 1500, True),    # 24 steps of tokens, 9 of dx
    (512, 640, 8, 8192, False),     # 128 and 9: by themselves the weight gradients have a ring of four
    (256, 512, 8, 16000, False),
])
def test_many_tokens_leave_the_launch_of_two_to_a_cu(d_out, d_in, r, tokens, together):
    q = Inputs(d_out, d_in, r, tokens, "bf16")
    q.h.normal_(), q.inner.normal_()
    dA, dB = G.empty_f32(r, d_in), G.empty_f32(d_out, r)
    D.dora_trace_reset(), D.dora_trace_select(~0), D.dora_trace_enable(True)
    D.dora_backward(q.desc, q.dy, q.xl, q.W, q.A, q.B, q.m, q.c, q.h, q.inner, q.dx, dA, dB, None, q.ws(D.PHASE_BACKWARD))
    D.dora_trace_enable(False), D.dora_trace_collect()
    launches = {D.dora_trace_name(k): D.dora_trace_get(k)[1] for k in range(20)}
    assert (launches["gemm_dx"], launches["gemm_dA"]) == (1, 0 if together else 1)
    dh = q.s * (q.g * q.dy.double()) @ q.B.double()
    close("dA", dA, (dh.T @ q.xl.double(), slice(None)), "bf16")
    close("dB", dB, (q.s * (q.g * q.dy.double()).T @ q.h.double(), slice(None)), "bf16")

"""Gradients written over the upstream gradient (and dA, in fp32, over A): each output is written after the last reader of what it
covers, whatever launches the same call with buffers of its own would share."""
import pytest
import torch

from paper_2603_22276_amd import binding as D

import gpu_util as G
from test_gpu_rounds import DT, Inputs, close

pytestmark = pytest.mark.gpu
DT["f32"] = torch.float32


def reference(q):
    dy, x, W, A, B = (t.double() for t in (q.dy, q.xl, q.W, q.A, q.B))
    dz, h = q.g * dy, x @ A.T
    dh = q.s * dz @ B
    inner = x @ W.T + q.s * h @ B.T
    return {"h": h, "inner": inner, "dx": dz @ W + dh @ A, "dx_frozen": dy @ W, "dx_lora": ((q.g - 1) * dy) @ W + dh @ A,
            "dA": dh.T @ x, "dB": q.s * dz.T @ h, "dm": (dy * inner).sum(0) / q.c.double()}


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("d,r,tokens", [(512, 16, 64), (776, 40, 1500), (256, 64, 8200), (1032, 24, 1030)])
def test_dx_over_dy(dtype, d, r, tokens):
    q = Inputs(d, d, r, tokens, dtype)
    ref, every = reference(q), slice(None)
    q.h.copy_(ref["h"]), q.inner.copy_(ref["inner"])
    dA, dB, dm, buf = G.empty_f32(r, d), G.empty_f32(d, r), G.empty_f32(d), q.dy.clone()
    D.dora_backward(q.desc, buf, q.xl, q.W, q.A, q.B, q.m, q.c, q.h, q.inner, buf, dA, dB, dm, q.ws(D.PHASE_BACKWARD))
    for name, got in (("dx", buf), ("dA", dA), ("dB", dB), ("dm", dm)):
        close(name, got, (ref[name], every), dtype)
    buf.copy_(q.dy)
    D.dora_backward_dropout(q.desc, buf, q.xl, q.W, q.A, q.B, q.m, q.c, q.h, q.inner, q.dx, buf, dA, dB, dm,
                            q.ws(D.PHASE_BACKWARD_DROPOUT))
    for name, got in (("dx_frozen", q.dx), ("dx_lora", buf), ("dA", dA), ("dB", dB), ("dm", dm)):
        close(name, got, (ref[name], every), dtype)


def test_dA_over_A():
    q = Inputs(776, 520, 40, 300, "f32")
    ref = reference(q)
    q.h.copy_(ref["h"]), q.inner.copy_(ref["inner"])
    dB, buf = G.empty_f32(776, 40), q.A.clone()
    D.dora_backward(q.desc, q.dy, q.xl, q.W, buf, q.B, q.m, q.c, q.h, q.inner, q.dx, buf, dB, None, q.ws(D.PHASE_BACKWARD))
    for name, got in (("dx", q.dx), ("dA", buf), ("dB", dB)):
        close(name, got, (ref[name], slice(None)), "f32")

"""Eq. 5, Eq. 6 and dm's second stage inside the reduce launch of a split product, or as launches of their own where the product
that could carry them is not split: the same norm, and the same results as with the norm given, bit for bit."""
import pytest
import torch

from paper_2603_22276_amd import binding as D

import gpu_util as G
from test_gpu_rounds import DT, Inputs, close

pytestmark = pytest.mark.gpu
DT["f32"] = torch.float32

SHAPES = [  # d_out, d_in, r, tokens
    (1000, 4104, 72, 77),       # h and dh split, the last block of 32 rows not full
    (8, 2048, 8, 130),          # h split, one block; dh of one K step not split
    (4104, 72, 8, 200),         # dh split, h not
    (136, 136, 16, 300),        # neither
    (2056, 3000, 24, 16000),    # 125 tiles each: two slices, and as many slabs of dm as there are
    (512, 1024, 392, 100),      # rank past the norm of one launch
    (8, 12040, 264, 6000),      # h of 141 tiles in three slices: two workgroups to a CU
    (12040, 16, 264, 6000),     # dh the same
]


def same(name, a, b):
    assert torch.equal(a, b), name


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("d_out,d_in,r,tokens", SHAPES)
def test_norm_formed_on_the_way(dtype, d_out, d_in, r, tokens):
    q = Inputs(d_out, d_in, r, tokens, dtype)
    c = G.empty_f32(d_out)
    D.dora_norm(q.desc, q.W, q.A, q.B, c, q.ws(D.PHASE_NORM))
    for call, ins, phase in ((D.dora_forward, (q.x,), D.PHASE_FORWARD), (D.dora_forward_fused, (q.x,), D.PHASE_FORWARD),
                             (D.dora_forward_dropout, (q.x, q.xl), D.PHASE_FORWARD_DROPOUT)):
        got = []
        for given in (c, None):
            y, h, inner, cw = torch.empty_like(q.y), torch.empty_like(q.h), torch.empty_like(q.inner), G.empty_f32(d_out)
            call(q.desc, *ins, q.W, q.A, q.B, q.m, given, q.bias, y, h, inner, cw, q.ws(phase))
            got.append((y, h, inner, cw))
        for name, a, b in zip(("y", "h", "inner", "norm"), *got):
            same(name, a, b)
        same("norm", got[1][3], c)
    dx, dxl = torch.empty_like(q.dx), torch.empty_like(q.dxl)
    for dropout in (False, True):
        got = []
        for given in (c, None):
            dA, dB, dm = G.empty_f32(r, d_in), G.empty_f32(d_out, r), G.empty_f32(d_out)
            if dropout:
                D.dora_backward_dropout(q.desc, q.dy, q.xl, q.W, q.A, q.B, q.m, given, None, None, dx, dxl, dA, dB, dm,
                                        q.ws(D.PHASE_BACKWARD_DROPOUT))
            else:
                D.dora_backward(q.desc, q.dy, q.xl, q.W, q.A, q.B, q.m, given, None, None, dx, dA, dB, dm,
                                q.ws(D.PHASE_BACKWARD_RECOMPUTE))
            got.append((dx.clone(), dA, dB, dm))
        for name, a, b in zip(("dx", "dA", "dB", "dm"), *got):
            same(name, a, b)
        inner = q.xl.double() @ q.W.double().T + q.s * (q.xl.double() @ q.A.double().T) @ q.B.double().T
        close("dm", got[1][3], ((q.dy.double() * inner).sum(0) / c.double(), slice(None)), dtype)
    # dm alone has nothing to ride in
    alone = G.empty_f32(d_out)
    D.dora_backward(q.desc, q.dy, q.xl, q.W, q.A, q.B, q.m, None, None, None, None, None, None, alone, q.ws(D.PHASE_BACKWARD_RECOMPUTE))
    close("dm alone", alone, ((q.dy.double() * inner).sum(0) / c.double(), slice(None)), dtype)


@pytest.mark.parametrize("d_out,d_in,r,tokens,dtype", [
    (1000, 4104, 72, 77, "bf16"),     # dm's second stage in the reduce of dh: as many slabs as tokens / 16
    (2056, 3000, 24, 16000, "f16"),   # the same, of several slabs to a range
    (4104, 72, 8, 200, "bf16"),
    (136, 136, 16, 300, "f32"),       # fp32 launches of sixteen waves, and of four where dm is alone
    (1000, 772, 36, 1500, "f32"),     # of four beside tiles
    (516, 260, 12, 12000, "f32"),     # 188 slabs
])
def test_dm_does_not_depend_on_what_else_is_wanted(d_out, d_in, r, tokens, dtype):
    q = Inputs(d_out, d_in, r, tokens, dtype)
    q.h.normal_(), q.inner.normal_()
    ws = q.ws(D.PHASE_BACKWARD)
    got = []
    for want in (("dx", "dA", "dB"), ("dB",), ()):
        dm = G.empty_f32(d_out)
        out = {"dx": q.dx, "dA": G.empty_f32(r, d_in), "dB": G.empty_f32(d_out, r)}
        out = [v if k in want else None for k, v in out.items()]
        D.dora_backward(q.desc, q.dy, q.xl, q.W, q.A, q.B, q.m, q.c, q.h, q.inner, *out, dm, ws)
        got.append(dm)
    same("dm", got[0], got[1])
    same("dm", got[0], got[2])
    close("dm", got[0], ((q.dy.double() * q.inner.double()).sum(0) / q.c.double(), slice(None)), dtype)

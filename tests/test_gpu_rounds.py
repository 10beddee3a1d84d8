"""Products over the lines where the tiles change: one round of 256 x 256 tiles that is not full, whole rounds of them with
the rest in 128 x 128 ones (cut along rows, along columns, ragged), pairs of products in either tile, K slices up to sixteen."""
import numpy as np
import pytest
import torch

from paper_2603_22276_amd import binding as D

import gpu_util as G

pytestmark = pytest.mark.gpu

DT = {"bf16": torch.bfloat16, "f16": torch.float16}


class Inputs:
    def __init__(self, d_out, d_in, r, tokens, dtype):
        gen = torch.Generator(device=G.DEV)
        gen.manual_seed(d_out + d_in + r + tokens)
        n = lambda rows, cols, std=1.0: (torch.randn((rows, cols), generator=gen, device=G.DEV) * std).to(DT[dtype])
        self.s = float(np.float32(32.0 / r ** 0.5))
        self.desc = D.make_desc(d_out, d_in, r, tokens, G.dtype_code(dtype), self.s)
        self.W, self.A, self.B = n(d_out, d_in, d_in ** -0.5), n(r, d_in, d_in ** -0.5), n(d_out, r, 0.5 / (self.s * r ** 0.5))
        self.x, self.xl, self.dy = n(tokens, d_in), n(tokens, d_in), n(tokens, d_out)
        self.bias = n(1, d_out)[0].contiguous()
        self.c = torch.rand((d_out,), generator=gen, device=G.DEV) + 0.5
        self.m = self.c * (1 + 0.1 * torch.randn((d_out,), generator=gen, device=G.DEV))
        self.g = self.m.double() / self.c.double()
        self.h, self.inner, self.y = G.empty((tokens, r), dtype), G.empty((tokens, d_out), dtype), G.empty((tokens, d_out), dtype)
        self.dx, self.dxl = G.empty((tokens, d_in), dtype), G.empty((tokens, d_in), dtype)
        self.rows = torch.unique(torch.cat([torch.arange(0, tokens, max(1, tokens // 40)), torch.arange(max(0, tokens - 70), tokens)])).to(G.DEV)

    def ws(self, phase):
        return G.workspace(self.desc, phase)


def close(name, got, ref, dtype):
    assert bool(torch.isfinite(got).all()), name       # every element written
    G.assert_close(name, G.to_f64(got[ref[1]]), G.to_f64(ref[0]), G.TOL[dtype]["tensor"])


SHAPES = [  # d_out, d_in, r, tokens
    (4096, 1032, 24, 4352),     # 17 x 16 large tiles: a row of them left over
    (16640, 1024, 8, 1101),     # 5 x 65: columns left over, ragged rows
    (4104, 1096, 16, 4099),     # 17 x 17: a row and a column, both nearly empty
    (2304, 1160, 40, 4090),     # 16 x 9: one round, not full
    (1024, 4104, 72, 77),       # eight tiles of 128 x 128: K in slices
    (136, 16384, 8, 130),       # four tiles: sixteen slices
]


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("d_out,d_in,r,tokens", SHAPES)
def test_forward_and_input_gradient(dtype, d_out, d_in, r, tokens):
    for do, di in ((d_out, d_in), (d_in, d_out)):      # the second way round, dx has the tiles the first gives y
        q = Inputs(do, di, r, tokens, dtype)
        D.dora_forward_fused(q.desc, q.x, q.W, q.A, q.B, q.m, q.c, q.bias, q.y, q.h, q.inner, None, q.ws(D.PHASE_FORWARD))
        D.dora_backward(q.desc, q.dy, q.x, q.W, q.A, q.B, q.m, q.c, q.h, q.inner, q.dx, None, None, None, q.ws(D.PHASE_BACKWARD))
        x, dy = q.x[q.rows].double(), q.dy[q.rows].double()
        inner = x @ q.W.double().T + q.s * (x @ q.A.double().T) @ q.B.double().T
        close("inner", q.inner, (inner, q.rows), dtype)
        close("y", q.y, (q.g * inner + q.bias.double(), q.rows), dtype)
        dz = q.g * dy
        close("dx", q.dx, (dz @ q.W.double() + q.s * (dz @ q.B.double()) @ q.A.double(), q.rows), dtype)


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("d_out,d_in,r,tokens", [(2056, 3000, 72, 1501), (1032, 1096, 16, 1030), (4096, 1032, 24, 2100), (136, 264, 8, 70)])
def test_dropout_products_in_pairs(dtype, d_out, d_in, r, tokens):
    q = Inputs(d_out, d_in, r, tokens, dtype)
    D.dora_forward_dropout(q.desc, q.x, q.xl, q.W, q.A, q.B, q.m, q.c, q.bias, q.y, q.h, q.inner, None, q.ws(D.PHASE_FORWARD_DROPOUT))
    D.dora_backward_dropout(q.desc, q.dy, q.xl, q.W, q.A, q.B, q.m, q.c, q.h, q.inner, q.dx, q.dxl, None, None, None,
                            q.ws(D.PHASE_BACKWARD_DROPOUT))
    x, xl, dy = q.x[q.rows].double(), q.xl[q.rows].double(), q.dy[q.rows].double()
    base, base_l, lora = x @ q.W.double().T, xl @ q.W.double().T, q.s * (xl @ q.A.double().T) @ q.B.double().T
    close("inner", q.inner, (base_l + lora, q.rows), dtype)
    close("y", q.y, (base + (q.g - 1) * base_l + q.g * lora + q.bias.double(), q.rows), dtype)
    close("dx", q.dx, (dy @ q.W.double(), q.rows), dtype)
    dh = q.s * (q.g * dy) @ q.B.double()
    close("dx_lora", q.dxl, (((q.g - 1) * dy) @ q.W.double() + dh @ q.A.double(), q.rows), dtype)

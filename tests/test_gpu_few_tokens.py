"""Forward of a few tokens (the weight-streaming kernels): both forward entry points against the fp64 oracle where
these kernels can go wrong - edges of the 16-token and 16-row blocks, K shorter than one ring slot, ragged K, more
waves than K steps, ranks that end inside a k-step - up to the first token count that takes the tiled path; then every
tile the y launch chooses from: 64 weight rows per workgroup beyond 8192 of them, 32 between 4096 and 8192 with more than
32 tokens, with a ragged last group and token counts that end inside and right before a block of 16."""
import numpy as np
import pytest
import torch

from oracle import dora_oracle as O
from paper_2603_22276_amd import binding as D
from paper_2603_22276_amd import inputs as I

import gpu_util as G

pytestmark = pytest.mark.gpu

CASES = [  # d_out, d_in, r, tokens
    (8, 8, 8, 1), (24, 64, 8, 2), (264, 72, 24, 15), (200, 1000, 40, 16), (520, 392, 136, 17), (72, 2312, 384, 31),
    (1032, 520, 72, 32), (136, 4104, 40, 33), (520, 264, 392, 48), (264, 1032, 8, 64), (264, 392, 40, 65),
    (8200, 72, 24, 1), (8248, 136, 8, 17), (8264, 200, 40, 33), (8256, 64, 8, 64), (4104, 136, 24, 33), (8184, 72, 8, 64),
    (8216, 72, 16, 48), (4112, 200, 8, 49),
]


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("d_out,d_in,r,tokens", CASES)
def test_forward_of_a_few_tokens(dtype, d_out, d_in, r, tokens):
    cfg = I.stress(I.DoraConfig(f"few_{d_out}_{d_in}_{r}_{tokens}", d_out, d_in, r, tokens, dtype, 32.0, 1e-3, seed_offset=9100))
    mod = G.Module(cfg)
    tol = G.TOL[dtype]["tensor"]
    f = O.forward(x=mod.f64("x"), W=mod.f64("W"), A=mod.f64("A"), B=mod.f64("B"), m=mod.inp["m"].astype(np.float64),
                  s=float(mod.inp["s"]), eps=cfg.eps)
    bias = torch.linspace(-1, 1, d_out, device=G.DEV).to(mod.W.dtype)
    for fused in (False, True):
        out = mod.forward(fused=fused)                        # norm inside, everything saved
        G.assert_norm_close(G.to_f64(out["c"]), f["c"], G.TOL[dtype]["norm"])
        for k in ("y", "h", "inner"):
            G.assert_close(k, G.to_f64(out[k]), f[k], tol)
        # norm given, nothing saved, bias: the same y plus the bias, so the bound is the one of y plus one rounding
        kept = mod.forward(w_norm=out["c"], save=False, fused=fused, bias=bias)
        G.assert_close("y+bias", G.to_f64(kept["y"]), f["y"] + G.to_f64(bias), tol)
        assert torch.equal(kept["c"], out["c"])

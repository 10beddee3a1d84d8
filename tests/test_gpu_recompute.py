"""Backward with norm, h and inner recomputed in 16-bit storage (bf16: inner from one K-concatenated product, s h in the
buffer that dh takes later): one row, edges of the tiles in both directions, ranks beside a K step, the large tile, and the
same calls with a frozen magnitude, where inner is not formed."""
import numpy as np
import pytest
import torch

from oracle import dora_oracle as O
from paper_2603_22276_amd import inputs as I

import gpu_util as G

pytestmark = pytest.mark.gpu

CASES = [  # d_out, d_in, r, tokens; the last two have 256 tiles of 256 x 256
    (8, 8, 8, 1), (136, 72, 24, 63), (264, 200, 40, 65), (128, 64, 64, 129), (72, 136, 8, 193), (4088, 72, 8, 3969), (4096, 64, 16, 4096),
]


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("d_out,d_in,r,tokens", CASES)
def test_recomputed_backward(dtype, d_out, d_in, r, tokens):
    cfg = I.stress(I.DoraConfig(f"rec_{d_out}_{d_in}_{r}_{tokens}", d_out, d_in, r, tokens, dtype, 32.0, 1e-3, seed_offset=9300))
    mod = G.Module(cfg)
    tol = G.TOL[dtype]["tensor"]
    b = O.backward(mod.f64("dy"), x=mod.f64("x"), W=mod.f64("W"), A=mod.f64("A"), B=mod.f64("B"),
                   m=mod.inp["m"].astype(np.float64), s=float(mod.inp["s"]), eps=cfg.eps)
    grads, frozen = mod.backward(), mod.backward(want_dm=False)
    for k in ("dx", "dA", "dB", "dm"):
        G.assert_close(k, G.to_f64(grads[k]), b[k], tol)
        if k != "dm":   # dz is rounded once from g * dy on either route
            assert torch.equal(grads[k].view(torch.uint8), frozen[k].view(torch.uint8)), k

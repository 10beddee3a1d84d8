"""Few tokens, one block of them and of weight rows: h comes through LDS, 512 ranks at a time, and B ahead of the weights.  One
item of h per thread and several, ranks that end at, inside and past a piece, tokens that end inside the block, slices 1 to 8.
Ranks up to 256: every wave takes its own 32 of them."""
import numpy as np
import pytest

from oracle import dora_oracle as O
from paper_2603_22276_amd import inputs as I

import gpu_util as G

pytestmark = pytest.mark.gpu

CASES = [(72, 4104, 512, 1), (264, 520, 520, 16), (1032, 264, 1032, 3), (136, 1032, 248, 15), (72, 72, 1544, 16), (8192, 72, 40, 2)]


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("d_out,d_in,r,tokens", CASES)
def test_h_through_lds(dtype, d_out, d_in, r, tokens):
    cfg = I.stress(I.DoraConfig(f"few_lds_{d_out}_{d_in}_{r}_{tokens}", d_out, d_in, r, tokens, dtype, 32.0, 1e-3, seed_offset=9400))
    mod = G.Module(cfg)
    tol = G.TOL[dtype]["tensor"]
    f = O.forward(x=mod.f64("x"), W=mod.f64("W"), A=mod.f64("A"), B=mod.f64("B"), m=mod.inp["m"].astype(np.float64),
                  s=float(mod.inp["s"]), eps=cfg.eps)
    out = mod.forward(fused=True)
    for k in ("y", "h", "inner"):
        G.assert_close(k, G.to_f64(out[k]), f[k], tol)


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("d_out,d_in,r,tokens", [(72, 4104, 8, 1), (264, 520, 40, 16), (8192, 72, 32, 15), (136, 8200, 72, 3),
                                                 (520, 2056, 256, 16), (1032, 264, 248, 1), (136, 4104, 264, 5)])
def test_each_wave_its_own_ranks(dtype, d_out, d_in, r, tokens):
    cfg = I.stress(I.DoraConfig(f"few_own_{d_out}_{d_in}_{r}_{tokens}", d_out, d_in, r, tokens, dtype, 32.0, 1e-3, seed_offset=9450))
    mod = G.Module(cfg)
    tol = G.TOL[dtype]["tensor"]
    f = O.forward(x=mod.f64("x"), W=mod.f64("W"), A=mod.f64("A"), B=mod.f64("B"), m=mod.inp["m"].astype(np.float64),
                  s=float(mod.inp["s"]), eps=cfg.eps)
    out = mod.forward(fused=True)
    for k in ("y", "h", "inner"):
        G.assert_close(k, G.to_f64(out[k]), f[k], tol)
    # nothing saved: the same y
    np.testing.assert_array_equal(G.to_f64(mod.forward(fused=True, save=False)["y"]), G.to_f64(out["y"]))

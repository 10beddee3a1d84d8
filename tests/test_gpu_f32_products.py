"""fp32 products where their two kernels can go wrong: one row or four columns, ranks and K that end inside a group of 16,
fewer groups of k than waves, K around the change from four to sixteen waves, extents around a tile and around the change
from split 32 x 32 tiles to 64 x 64 ones, two problems of unequal size in one launch."""
import numpy as np
import pytest

from oracle import dora_oracle as O
from paper_2603_22276_amd import inputs as I

import gpu_util as G

pytestmark = pytest.mark.gpu

CASES = [  # d_out, d_in, r, tokens
    (4, 4, 4, 1), (36, 20, 4, 3), (32, 252, 8, 33), (260, 256, 12, 31), (64, 260, 20, 257), (132, 1028, 36, 65),
    (512, 68, 4, 1021), (516, 516, 72, 961), (1000, 772, 36, 1500),
    # 195 tiles of 64 x 64 in dA, then in dB: both operands K-strided, K (tokens) shorter and longer than a step, no multiple of four
    (68, 4100, 132, 37), (4100, 68, 132, 37), (68, 4100, 132, 1), (4100, 68, 132, 101),
]


@pytest.mark.parametrize("d_out,d_in,r,tokens", CASES)
def test_fp32_forward_and_backward(d_out, d_in, r, tokens):
    cfg = I.stress(I.DoraConfig(f"f32_{d_out}_{d_in}_{r}_{tokens}", d_out, d_in, r, tokens, "f32", 16.0, 1e-3, seed_offset=9200))
    mod = G.Module(cfg)
    tol = G.TOL["f32"]["tensor"]
    oi = dict(x=mod.f64("x"), W=mod.f64("W"), A=mod.f64("A"), B=mod.f64("B"), m=mod.inp["m"].astype(np.float64),
              s=float(mod.inp["s"]), eps=cfg.eps)
    f, b = O.forward(**oi), O.backward(mod.f64("dy"), **oi)
    out = mod.forward()
    G.assert_norm_close(G.to_f64(out["c"]), f["c"], G.TOL["f32"]["norm"])
    for k in ("y", "h", "inner"):
        G.assert_close(k, G.to_f64(out[k]), f[k], tol)
    for grads in (mod.backward(w_norm=out["c"], h=out["h"], inner=out["inner"]), mod.backward()):
        for k in ("dx", "dA", "dB", "dm"):
            G.assert_close(k, G.to_f64(grads[k]), b[k], tol)


def test_fp32_infinity_stays_in_its_row():
    # rows and k past the end of a tile are clamped to existing elements: an infinity there must not reach other outputs
    cfg = I.DoraConfig("f32_inf", 36, 20, 4, 33, "f32", 16.0, 1e-3, seed_offset=9201)
    inp = I.make_inputs(cfg)
    inp["x"] = inp["x"].copy()
    inp["x"][-1, -1] = np.inf
    y = G.to_f64(G.Module(cfg, inp).forward()["y"])
    assert np.isfinite(y[:-1]).all() and not np.isfinite(y[-1]).any()

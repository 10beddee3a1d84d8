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
    # either side of the lines between these kernels and the tiles
    (72, 72, 1536, 32), (72, 72, 1544, 32), (136, 72, 768, 48), (136, 72, 776, 33), (136, 72, 640, 49), (136, 72, 648, 49), (16384, 72, 24, 64), (16392, 72, 24, 33),
    (16392, 2048, 8, 40), (16392, 72, 256, 17), (16392, 72, 264, 17), (16392, 64, 24, 16), (32776, 64, 1032, 16),
    (136, 72, 1024, 64), (136, 72, 1032, 33), (16392, 72, 512, 17), (16392, 72, 520, 17), (16392, 72, 256, 33), (16392, 72, 264, 33),
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


LINES = [  # d_out, d_in, r, tokens; streamed as the K-concatenated product, streamed as base + lora + compose pass
    (72, 72, 2048, 16, True, True), (72, 72, 1536, 32, True, True), (72, 72, 1544, 32, False, True), (136, 72, 768, 48, True, True),
    (136, 72, 776, 33, False, True), (136, 72, 640, 64, True, True), (136, 72, 648, 49, False, True), (136, 72, 1032, 33, False, False),
    (16384, 8, 640, 64, True, True), (16392, 8, 2048, 16, True, True), (16392, 8, 2056, 16, False, True), (32776, 8, 1032, 16, False, True),
    (16392, 8, 256, 32, True, True), (16392, 8, 264, 32, False, True), (16392, 8, 520, 17, False, False), (16392, 5128, 8, 17, False, False),
    (16392, 2048, 128, 33, True, True), (16392, 2040, 128, 33, False, True), (16392, 2048, 136, 64, False, True), (16392, 2048, 264, 64, False, False),
    (16392, 4104, 8, 33, False, False), (72, 72, 8, 65, False, False),
]


@pytest.mark.parametrize("d_out,d_in,r,tokens,one_product,three_passes", LINES)
def test_streamed_only_where_it_is_the_faster_route(d_out, d_in, r, tokens, one_product, three_passes):
    # the tiled route forms g in a launch of its own when the norm is given, the streaming one inside its second launch
    mag_scale = 5
    for fused, streamed in ((True, one_product), (False, three_passes)):
        desc = D.make_desc(d_out, d_in, r, tokens, D.DORA_F16, 1.0)
        x, W, A, B, y = (torch.zeros(s, dtype=torch.float16, device=G.DEV) for s in
                         ((tokens, d_in), (d_out, d_in), (r, d_in), (d_out, r), (tokens, d_out)))
        m, c = torch.ones(d_out, device=G.DEV), torch.ones(d_out, device=G.DEV)
        ws = torch.empty(D.dora_workspace_bytes(desc, D.PHASE_FORWARD), dtype=torch.uint8, device=G.DEV)
        D.dora_trace_reset()
        D.dora_trace_select(~0)
        D.dora_trace_enable(True)
        try:
            (D.dora_forward_fused if fused else D.dora_forward)(desc, x, W, A, B, m, c, None, y, None, None, None, ws)
            torch.cuda.synchronize()
        finally:
            D.dora_trace_enable(False)
        D.dora_trace_collect()
        assert D.dora_trace_get(mag_scale)[1] == (0 if streamed else 1)
        D.dora_trace_reset()

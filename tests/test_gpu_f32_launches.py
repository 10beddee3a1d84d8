"""fp32 work that shares launches: 32-row and 64-row tiles in each layout, the norm in slices of its columns, and a backward
that leaves pieces out (each gradient alone, the magnitude frozen, the norm given or formed)."""
import numpy as np
import pytest

from oracle import dora_oracle as O
from paper_2603_22276_amd import binding as D
from paper_2603_22276_amd import inputs as I

import gpu_util as G

pytestmark = pytest.mark.gpu

SHAPES = [  # d_out, d_in, r, tokens
    (1000, 772, 36, 1500),      # 384 and 312 tiles of 64 x 64 become 752 and 611 of 32 x 64
    (68, 4100, 300, 37),        # the same for dA, both operands K-strided; norm in 17 slices
    (4100, 68, 300, 101),       # and for dB, whose rows are scaled
    (2052, 1028, 20, 1030),     # 64 x 64
    (20, 2052, 132, 3),         # two row blocks, norm in 17 slices
]


@pytest.mark.parametrize("d_out,d_in,r,tokens", SHAPES)
def test_pieces_of_the_backward(d_out, d_in, r, tokens):
    cfg = I.stress(I.DoraConfig(f"f32_launch_{d_out}_{d_in}_{r}_{tokens}", d_out, d_in, r, tokens, "f32", 16.0, 1e-3, seed_offset=9300))
    mod = G.Module(cfg)
    tol = G.TOL["f32"]["tensor"]
    oi = dict(x=mod.f64("x"), W=mod.f64("W"), A=mod.f64("A"), B=mod.f64("B"), m=mod.inp["m"].astype(np.float64),
              s=float(mod.inp["s"]), eps=cfg.eps)
    f, b = O.forward(**oi), O.backward(mod.f64("dy"), **oi)
    out = mod.forward()
    G.assert_norm_close(G.to_f64(out["c"]), f["c"], 3e-6)
    for k in ("y", "h", "inner"):
        G.assert_close(k, G.to_f64(out[k]), f[k], tol)
    ws = G.workspace(mod.desc, D.PHASE_BACKWARD_RECOMPUTE)
    for want in (("dx", "dA", "dB", "dm"), ("dx", "dA", "dB"), ("dx",), ("dA",), ("dB",), ("dm",), ("dB", "dm")):
        for c in (out["c"], None):
            got = {"dx": G.empty((tokens, d_in), "f32"), "dA": G.empty_f32(r, d_in), "dB": G.empty_f32(d_out, r), "dm": G.empty_f32(d_out)}
            got = {k: v if k in want else None for k, v in got.items()}
            D.dora_backward(mod.desc, mod.dy, mod.x, mod.W, mod.A, mod.B, mod.m, c, out["h"], out["inner"], got["dx"], got["dA"],
                            got["dB"], got["dm"], ws)
            for k in want:
                G.assert_close(k, G.to_f64(got[k]), b[k], tol)


def test_weight_gradients_in_short_sums():
    """dA and dB of few tiles share the launch of dx and its workgroups of four waves: a quarter of K in one chain of additions
    had an error of 3.9e-7 and 5.2e-7 here, in sums of 64 k 2.2e-7 and 2.3e-7 (sixteen waves: 2.5e-7 and 2.9e-7); the bound lies
    between."""
    cfg = I.DoraConfig("f32_short_sums", 704, 1760, 20, 1509, "f32", 16.0, 1e-3, seed_offset=9400)
    mod = G.Module(cfg)
    oi = dict(x=mod.f64("x"), W=mod.f64("W"), A=mod.f64("A"), B=mod.f64("B"), m=mod.inp["m"].astype(np.float64),
              s=float(mod.inp["s"]), eps=cfg.eps)
    out = mod.forward()
    b = O.backward(mod.f64("dy"), **oi)
    dx, dA, dB = G.empty((1509, 1760), "f32"), G.empty_f32(20, 1760), G.empty_f32(704, 20)
    D.dora_backward(mod.desc, mod.dy, mod.x, mod.W, mod.A, mod.B, mod.m, out["c"], out["h"], out["inner"], dx, dA, dB, None,
                    G.workspace(mod.desc, D.PHASE_BACKWARD))
    for name, got, ref in (("dA", dA, b["dA"]), ("dB", dB, b["dB"])):
        err = np.linalg.norm(G.to_f64(got) - ref) / np.linalg.norm(ref)
        assert err < 3.5e-7, (name, err)


@pytest.mark.parametrize("d_out,d_in,r,tokens", [
    (256, 512, 64, 8192),       # dh in 256 tiles of 32 x 64
    (36, 20, 8, 8200),          # in 129 of 64 x 64, the last of eight rows
    (68, 132, 384, 1409),       # in 138, the last of one row
    (68, 132, 384, 1407),       # in 132
])
def test_scale_of_a_tiled_dh(d_out, d_in, r, tokens):
    """g reaches dh as it reaches dx, whether it has to be formed from the norm (given, inner saved or not needed) or is there
    already.  m is two to seven times the norm, so that neither can stand for the other."""
    cfg = I.stress(I.DoraConfig(f"f32_tiled_dh_{d_out}_{d_in}_{r}_{tokens}", d_out, d_in, r, tokens, "f32", 16.0, 1e-3, seed_offset=9500))
    inp = I.make_inputs(cfg)
    inp["m"] = (inp["m"] * np.random.default_rng(5).uniform(2.0, 7.0, d_out)).astype(np.float32)
    mod = G.Module(cfg, inp)
    tol = G.TOL["f32"]["tensor"]
    oi = dict(x=mod.f64("x"), W=mod.f64("W"), A=mod.f64("A"), B=mod.f64("B"), m=inp["m"].astype(np.float64), s=float(inp["s"]), eps=cfg.eps)
    out, b = mod.forward(), O.backward(mod.f64("dy"), **oi)
    for c in (out["c"], None):
        for h, inner, want_dm in ((out["h"], out["inner"], True), (out["h"], None, False), (None, None, True)):
            got = mod.backward(w_norm=c, h=h, inner=inner, want_dm=want_dm)
            for k in ("dx", "dA", "dB") + (("dm",) if want_dm else ()):
                G.assert_close(k, G.to_f64(got[k]), b[k], tol)


@pytest.mark.parametrize("d_out,d_in,r,tokens,launches", [
    (84, 12, 4, 29613, 2),      # dx in tiles, dA and dB over all tokens: by themselves, sixteen waves to a workgroup
    (8196, 20, 12, 90, 2),      # dB in tiles, dx over 8208 k
    (56, 900, 44, 666, 1),      # dx in tiles, dA and dB short enough beside them
    (140, 940, 224, 3001, 1),   # the longer dA and dB ahead of many tiles of dx
])
def test_long_sums_beside_tiles(d_out, d_in, r, tokens, launches):
    cfg = I.stress(I.DoraConfig(f"f32_long_{d_out}_{d_in}_{r}_{tokens}", d_out, d_in, r, tokens, "f32", 16.0, 1e-3, seed_offset=9600))
    mod = G.Module(cfg)
    oi = dict(x=mod.f64("x"), W=mod.f64("W"), A=mod.f64("A"), B=mod.f64("B"), m=mod.inp["m"].astype(np.float64),
              s=float(mod.inp["s"]), eps=cfg.eps)
    out, b = mod.forward(), O.backward(mod.f64("dy"), **oi)
    D.dora_trace_reset(), D.dora_trace_select(~0), D.dora_trace_enable(True)
    got = mod.backward(w_norm=out["c"], h=out["h"], inner=out["inner"])
    D.dora_trace_enable(False), D.dora_trace_collect()
    counts = {D.dora_trace_name(k): D.dora_trace_get(k)[1] for k in range(20)}
    assert counts["gemm_dx"] == launches
    for k in ("dx", "dA", "dB", "dm"):
        G.assert_close(k, G.to_f64(got[k]), b[k], G.TOL["f32"]["tensor"])


@pytest.mark.parametrize("d_out,d_in,r", [
    (36, 20, 4),                # three blocks of 16 rows or two of 32, one group of columns
    (1000, 772, 36),            # one slice, the last group of four columns
    (260, 4100, 132),           # slices, the last of them with fewer groups
    (4100, 260, 68),            # 32 rows, the last block of four
    (5124, 1028, 164),          # 32 rows in slices
    (20, 504, 860),             # more slices than row blocks, ranks far past the columns of a wave
])
def test_norm_in_row_blocks_and_slices(d_out, d_in, r):
    cfg = I.stress(I.DoraConfig(f"f32_norm_{d_out}_{d_in}_{r}", d_out, d_in, r, 1, "f32", 16.0, 1e-3, seed_offset=9700))
    mod = G.Module(cfg)
    ref = O.dense_row_norm(mod.f64("W"), mod.f64("A"), mod.f64("B"), float(mod.inp["s"]))
    c = G.to_f64(mod.norm())
    # a product's own sum over r, then at most 9 groups, 8 lanes and 32 slices one after the other at 2^-24 each, half for the root
    G.assert_norm_close(c, ref, 3e-6)
    # the terms, the cached base term and a row that is not finite beside its neighbours
    terms, base, again = G.empty_f32(3, d_out), G.empty_f32(d_out), G.empty_f32(d_out)
    ws = G.workspace(mod.desc, D.PHASE_NORM)
    D.dora_norm_terms(mod.desc, mod.W, mod.A, mod.B, terms, None, ws)
    D.dora_norm_assemble(mod.desc, terms, again)
    np.testing.assert_array_equal(G.to_f64(again), c)
    D.dora_base_sq(mod.desc, mod.W, base)
    D.dora_norm_cached(mod.desc, base, mod.W, mod.A, mod.B, again, ws)
    G.assert_norm_close(G.to_f64(again), ref, 3e-6)
    row = d_out // 2 + 1
    mod.W[row, 1] = float("nan")
    bad = G.to_f64(mod.norm())
    assert np.isnan(bad[row])
    np.testing.assert_array_equal(np.delete(bad, row), np.delete(c, row))

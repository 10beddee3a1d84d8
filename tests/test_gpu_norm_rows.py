"""The launch that forms the norm's three sums for ranks up to 384: every count of K steps, ranks and columns ragged in the
last one, a single row block and a ragged last one, one column tile per workgroup and a walk over many; rows stay apart."""
import numpy as np
import pytest
import torch

from oracle import dora_oracle as O
from paper_2603_22276_amd import binding as D

import gpu_util as G

pytestmark = pytest.mark.gpu

# (d_out, d_in, r); 33032 rows are 259 row blocks, more than one round of workgroups: each walks over all its column tiles
SHAPES = [(8, 8, 8), (1024, 4096, 64), (33032, 1416, 64), (136, 264, 72), (33032, 1416, 128), (520, 2312, 136), (33032, 648, 192),
          (392, 3000, 200), (33032, 392, 256), (128, 5000, 264), (33032, 264, 320), (1160, 1096, 328), (33032, 1416, 384), (8, 27648, 384)]


def make(d_out, d_in, r, dtype):
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(d_out + d_in + r)
    dt = {"bf16": torch.bfloat16, "f16": torch.float16}[dtype]
    mk = lambda rows, cols, std: (torch.randn((rows, cols), generator=gen, device="cuda:0") * std).to(dt)
    s = 32.0 / r ** 0.5
    # the low-rank part as large as the frozen one, so that each of the three sums counts
    W, A, B = mk(d_out, d_in, d_in ** -0.5), mk(r, d_in, d_in ** -0.5), mk(d_out, r, 1.0 / (s * r ** 0.5))
    desc = D.make_desc(d_out, d_in, r, 0, G.dtype_code(dtype), s)
    return desc, W, A, B, s


def norm(desc, W, A, B):
    c = G.empty_f32(W.shape[0])
    D.dora_norm(desc, W, A, B, c, G.workspace(desc, D.PHASE_NORM))
    return G.to_f64(c)


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("d_out,d_in,r", SHAPES)
def test_norm_of_every_rank_step(dtype, d_out, d_in, r):
    desc, W, A, B, s = make(d_out, d_in, r, dtype)
    rows = np.unique(np.r_[0:min(d_out, 8), np.linspace(0, d_out - 1, 60).astype(int), max(0, d_out - 140):d_out])
    ref = O.dense_row_norm(G.to_f64(W[rows]), G.to_f64(A), G.to_f64(B[rows]), float(np.float32(s)))
    # Each sum meets at most 16 products of a block, 12 tiles, 8 lanes and 11 slices one after the other, 2^-24 of it each
    # time: 2.8e-6, half of that for the root, and as much again for the products' own sums over r.
    G.assert_norm_close(norm(desc, W, A, B)[rows], ref, 3e-6)


@pytest.mark.parametrize("r", [72, 200])
def test_a_row_that_is_not_finite_stays_alone(r):
    # r past a multiple of 64: the masked part of a row of B is its neighbour's; d_in past a multiple of 128: so is W's
    desc, W, A, B, s = make(264, 392, r, "bf16")
    clean = norm(desc, W, A, B)
    W[7, 3], B[9, 0], B[130, r - 1], W[255, 391] = float("nan"), float("inf"), float("nan"), float("inf")
    bad = [7, 9, 130, 255]
    c = norm(desc, W, A, B)
    assert not np.any(np.isfinite(c[bad]))
    keep = np.delete(np.arange(264), bad)
    np.testing.assert_array_equal(c[keep], clean[keep])

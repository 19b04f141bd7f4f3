"""GPU: the fp32 kernels (fp32 operands split into three bf16 planes on their way to the matrix pipes) and
the bf16 shapes they serve, at the edges of their tiles and load modes, against the fp64 oracle; and how
exact the split products are."""
import math

import numpy as np
import pytest
import torch

import paper_2201_13195_amd as rmm
from paper_2201_13195_amd import binding, synth
from test_gpu_parity import check_layer

pytestmark = pytest.mark.gpu
DEV = "cuda"

SHAPES = [
    # (n, d_in, d_out, k): 32x32, 64x64 and 128x128 tiles of the plain products, both sketch tiles
    (33, 36, 31, 5), (500, 129, 127, 40),          # 32 x 32 tiles; contractions around one and two LDS tiles
    (1030, 1028, 1004, 70),                         # 64 x 64 tiles of Y and dX, rows on 16 bytes
    (2049, 516, 1030, 290),                         # the same with rows that start on 8 bytes
    (2050, 2044, 2052, 100),                        # 128 x 128 tiles (a last round of one)
    (4096, 260, 1027, 33),                          # odd rows on one side only
]


@pytest.mark.parametrize("kind", [rmm.GAUSSIAN, rmm.RADEMACHER, rmm.SORS])
@pytest.mark.parametrize("shape", SHAPES)
def test_fp32_tiles_and_load_modes(shape, kind):
    n, d_in, d_out, k = shape
    X, W, dY = synth.layer_inputs(n, d_in, d_out, "f32", (n, d_in + 1, d_out + 2), w_std=1.0 / math.sqrt(d_in))
    bias = synth.to_torch(synth.normal((d_out,), 15), "f32")
    check_layer(X, W, dY, k, kind, 0x5EED0031, 5, "f32", bias=bias, label="f32 %s kind=%d" % (shape, kind))


# dX and dW on 128 x 128 tiles with two sums: contractions of one 16-deep step, one tile, an odd number of tiles and a ragged last one
@pytest.mark.parametrize("shape", [(2041, 1928, 12, 9), (2041, 1928, 36, 9), (1100, 4000, 100, 9), (64, 2052, 1990, 5),
                                   (64, 2052, 1990, 33), (96, 2052, 1990, 90)])
def test_fp32_large_tiles_of_the_gradients(shape):
    n, d_in, d_out, k = shape
    X, W, dY = synth.layer_inputs(n, d_in, d_out, "f32", (n, d_in + 1, d_out + 2), w_std=1.0 / math.sqrt(d_in))
    check_layer(X, W, dY, k, rmm.RADEMACHER, 0x5EED0033, 5, "f32", label="f32 large %s" % (shape,))


# One to five LDS tiles along a contraction, the last one whole, ragged or a single element: dX on 128 x 128 tiles (of 32
# elements) and on 64 x 64 (64) with an odd number of them, Y with an even one, products on 32 x 32 (128) and X_proj on 32 x 128 (64 tokens;
# bf16: most of them in slices).  (LDS_TILES has the others.)
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", [(2041, 1929, 32, 9), (2041, 64, 1929, 9), (2041, 1929, 65, 9), (2041, 128, 1929, 9), (2041, 1929, 129, 9),
                                   (1100, 1031, 64, 9), (1100, 65, 1031, 9), (1100, 1031, 192, 9), (1100, 256, 1031, 9), (1100, 1031, 257, 9),
                                   (300, 311, 128, 9), (300, 129, 311, 9), (384, 311, 385, 300), (512, 64, 65, 30), (513, 63, 70, 30),
                                   (64, 300, 17001, 900), (65, 300, 9001, 900), (129, 300, 9001, 900), (192, 300, 5401, 900),
                                   (257, 300, 5201, 900)])
def test_every_number_of_lds_tiles(shape, dtype):
    n, d_in, d_out, k = shape
    X, W, dY = synth.layer_inputs(n, d_in, d_out, dtype, (n, d_in + 1, d_out + 2), w_std=1.0 / math.sqrt(d_in))
    check_layer(X, W, dY, k, rmm.RADEMACHER if n in (192, 512) else rmm.GAUSSIAN, 0x5EED0034, 7, dtype,
                label="%s %s" % (dtype, shape))


# Two and three LDS tiles along the contraction, whole and ragged, of every product on every tile it can run with, and of the sketch products
# one and four too, in either type (test_launch_plans.py: these shapes have them)
LDS_TILES = [(16, 2049, 1473, 40), (31, 1500, 2049, 65), (32, 1473, 2049, 96), (32, 2041, 1929, 64), (33, 192, 17001, 192),
             (64, 300, 17001, 700), (64, 17001, 300, 700), (65, 95, 17001, 95), (65, 128, 8201, 97), (65, 385, 9001, 500),
             (65, 17001, 40, 129), (97, 5505, 385, 512), (128, 256, 300, 300), (128, 300, 8201, 700), (128, 5505, 512, 512),
             (128, 17001, 65, 96), (140, 300, 5505, 700), (140, 5505, 300, 700), (160, 150, 150, 129), (191, 5505, 192, 128),
             (192, 300, 5505, 700), (192, 5505, 300, 700), (256, 300, 4201, 700), (256, 384, 31, 65), (256, 8201, 33, 95),
             (300, 257, 384, 384), (384, 31, 256, 32), (512, 31, 33, 256), (1473, 64, 2049, 16), (1473, 96, 2049, 96),
             (1473, 2049, 64, 31), (1473, 2049, 96, 16), (1929, 65, 1929, 16), (2041, 2041, 33, 31), (2049, 33, 1500, 33),
             (2049, 500, 128, 40), (5505, 160, 129, 40), (9001, 65, 100, 16), (9001, 384, 65, 16)]


@pytest.mark.parametrize("shape", LDS_TILES)
def test_odd_and_even_numbers_of_lds_tiles(shape):
    n, d_in, d_out, k = shape
    for dtype in ("f32", "bf16"):
        X, W, dY = synth.layer_inputs(n, d_in, d_out, dtype, (n, d_in + 1, d_out + 2), w_std=1.0 / math.sqrt(d_in))
        check_layer(X, W, dY, k, rmm.GAUSSIAN, 0x5EED0035, 7, dtype, label="%s %s" % (dtype, shape))


@pytest.mark.parametrize("kind", [rmm.GAUSSIAN, rmm.RADEMACHER, rmm.SORS])
@pytest.mark.parametrize("shape", [(33, 35, 31, 5), (1030, 1028, 1004, 70), (2049, 515, 1030, 290), (3000, 768, 1001, 300),
                                   (4096, 261, 1032, 33)])
def test_bf16_widths_that_are_no_multiple_of_8(shape, kind):
    n, d_in, d_out, k = shape
    X, W, dY = synth.layer_inputs(n, d_in, d_out, "bf16", (n, d_in + 1, d_out + 2), w_std=1.0 / math.sqrt(d_in))
    bias = synth.to_torch(synth.normal((d_out,), 16), "bf16")
    check_layer(X, W, dY, k, kind, 0x5EED0032, 6, "bf16", bias=bias, label="bf16 %s kind=%d" % (shape, kind))


@pytest.mark.parametrize("kind", [rmm.GAUSSIAN, rmm.RADEMACHER, rmm.SORS])
@pytest.mark.parametrize("shape", [(4001, 512, 77, 33), (4001, 77, 264, 65), (4096, 264, 35, 31)])
def test_bf16_sketch_products_in_token_slices(shape, kind):
    """Slices of unequal length, an odd number of sketch values, tiles with one row or column; the scratch is asked for."""
    n, d_in, d_out, k = shape
    fwd, bwd = (rmm.rmm_workspace_bytes(n, d_in, d_out, k, torch.bfloat16, kind, op) for op in (0, 1))
    assert (fwd > 0) == (d_in % 8 == 0) and bwd > (k * d_out * 2 + 255) // 256 * 256
    X, W, dY = synth.layer_inputs(n, d_in, d_out, "bf16", (n, d_in + 1, d_out + 2), w_std=1.0 / math.sqrt(d_in))
    bias = synth.to_torch(synth.normal((d_out,), 16), "bf16")
    check_layer(X, W, dY, k, kind, 0x5EED0034, 6, "bf16", bias=bias, label="sliced %s kind=%d" % (shape, kind))


def test_an_infinity_in_one_token_slice():
    """It meets every sketch column with the sign of its entry; the other columns do not see it."""
    n, d_in, d_out, k = 4001, 512, 77, 33
    X, W, _ = synth.layer_inputs(n, d_in, d_out, "bf16", (1, 2, 3), w_std=0.02)
    X, W = X.to(DEV), W.to(DEV)
    _, want = rmm.rmm_forward(X, W, None, k, rmm.GAUSSIAN, 9, 4)
    X[3333, 100] = float("inf")
    _, got = rmm.rmm_forward(X, W, None, k, rmm.GAUSSIAN, 9, 4)
    P = rmm.rmm_debug_sketch_tile(rmm.GAUSSIAN, 9, 4, 3333, 0, 1, k)[0]
    assert torch.equal(got[:, 100].float(), torch.copysign(torch.full_like(P, float("inf")), P))
    got[:, 100] = want[:, 100]
    assert torch.equal(got, want)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_rows_beyond_the_descriptor_range(dtype):
    """Rows of 2^22 elements and more are loaded from 64-bit addresses."""
    n, d_in, d_out, k = 3, (1 << 22) + 5, 5, 2
    X, W, dY = synth.layer_inputs(n, d_in, d_out, dtype, (1, 2, 3), w_std=1.0 / math.sqrt(d_in))
    X[:, 3000:-3000] = 0      # (a sum of 2^22 fp32 terms is not exact to 1e-5 in any order)
    check_layer(X, W, dY, k, rmm.GAUSSIAN, 7, 8, dtype, label="long rows %s" % dtype)


@pytest.mark.parametrize("n,d_in,d_out", [(256, 1, 256), (512, 8, 512), (1024, 768, 1024)])
def test_fp32_products_are_as_exact_as_fp32_multiply_adds(n, d_in, d_out):
    """Contractions of one, a few and many terms, entries spread over 40 binades: the error against fp64
    is bounded by the roundings of an fp32 accumulation, relative to the sum of the terms' magnitudes."""
    g = np.random.default_rng(5)
    X = (g.standard_normal((n, d_in)) * np.exp2(g.integers(-20, 20, (n, d_in)))).astype(np.float32)
    W = (g.standard_normal((d_out, d_in)) * np.exp2(g.integers(-20, 20, (d_out, d_in)))).astype(np.float32)
    Y, _ = rmm.rmm_forward(torch.from_numpy(X).to(DEV), torch.from_numpy(W).to(DEV), None, 1, 0, 1, 2, need_xproj=False)
    X64, W64 = X.astype(np.float64), W.astype(np.float64)
    err = np.abs(synth.to_f64(Y) - X64 @ W64.T) / (np.abs(X64) @ np.abs(W64).T)
    print("K=%d: largest error / sum of magnitudes = %.2f * 2^-24" % (d_in, err.max() * 2.0 ** 24), flush=True)
    assert err.max() <= 2.0 ** -24 * (2.0 + math.sqrt(d_in))


@pytest.mark.parametrize("spread", [0, 20])
@pytest.mark.parametrize("n,d_in,d_out", [(256, 128, 256), (1024, 768, 1024), (4096, 768, 3072)])
def test_fp32_products_are_no_further_off_than_a_chain_of_multiply_adds(n, d_in, d_out, spread):
    """Every tile size of the plain products: error against fp64, relative to the sum of the terms' magnitudes,
    beside that of fp32 multiply-adds in order (64 rows), for entries of one size and over 40 binades."""
    g = np.random.default_rng(6)

    def draw(*shape):
        x = g.standard_normal(shape)
        return (x * np.exp2(g.integers(-spread, spread + 1, shape)) if spread else x).astype(np.float32)
    X, W = draw(n, d_in), draw(d_out, d_in)
    Y, _ = rmm.rmm_forward(torch.from_numpy(X).to(DEV), torch.from_numpy(W).to(DEV), None, 1, 0, 1, 2, need_xproj=False)
    rows = np.arange(64) * (n // 64)
    X64, W64 = X[rows].astype(np.float64), W.astype(np.float64)
    want, size = X64 @ W64.T, np.abs(X64) @ np.abs(W64.T)
    chain = np.zeros((64, d_out))
    for j in range(d_in):
        chain = (chain + X64[:, j:j + 1] * W64[:, j]).astype(np.float32).astype(np.float64)
    rms = [float(np.sqrt(np.mean(((a - want) / size) ** 2)) * 2.0 ** 24) for a in (synth.to_f64(Y)[rows], chain)]
    print("%s spread %d: %.3f, chain %.3f (rms, 2^-24 of the sum of magnitudes)" % ((n, d_in, d_out), spread, *rms), flush=True)
    assert rms[0] <= rms[1]


@pytest.mark.parametrize("n,d_out,dtype", [(300, 3080, "bf16"), (257, 24, "bf16"), (700, 1544, "f32"), (1000, 20, "f32"), (513, 1001, "bf16"),
                                           (33, 7, "f32"), (1, 8, "bf16")])
def test_column_sums_of_whole_numbers_are_exact(n, d_out, dtype):
    """Both widths of a work-group's pieces and the element-wise form, in the launch of dW or of the pass (sums below 2^8)."""
    t = torch.bfloat16 if dtype == "bf16" else torch.float32
    dY = torch.randint(-1, 2, (n, d_out), generator=torch.Generator().manual_seed(n)).to(t)
    W, Xp = torch.zeros((d_out, 16), dtype=t, device=DEV), torch.zeros((5, 16), dtype=t, device=DEV)
    for need_dX in (True, False):
        _, _, db = rmm.rmm_backward(dY.to(DEV), W, Xp, rmm.RADEMACHER, 3, 4, need_dX=need_dX, need_dbias=True)
        assert torch.equal(db.float().cpu(), dY.float().sum(dim=0))


# 32 x 32, 64 x 64 and 128 x 128 tiles of the plain product, few and many sketch tiles beside them
@pytest.mark.parametrize("kind", [rmm.GAUSSIAN, rmm.RADEMACHER, rmm.SORS])
@pytest.mark.parametrize("dtype,shape", [("f32", (1000, 600, 700, 500)), ("f32", (300, 2000, 100, 250)), ("f32", (2100, 640, 1350, 90)),
                                         ("bf16", (1800, 640, 1351, 90)), ("bf16", (500, 1001, 300, 300)), ("bf16", (600, 264, 401, 500)),
                                         ("bf16", (2207, 1440, 1019, 110)), ("bf16", (3000, 768, 1001, 300))])
def test_products_one_by_one_give_the_bits_of_one_launch(dtype, shape, kind):
    n, d_in, d_out, k = shape
    X, W, dY = (t.to(DEV) for t in synth.layer_inputs(n, d_in, d_out, dtype, (51, 52, 53), w_std=1.0 / math.sqrt(d_in)))
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    a.record(); b.record()
    torch.cuda.synchronize()
    Y, Xp = rmm.rmm_forward(X, W, None, k, kind, 5, 1)
    for stage in (binding.STAGE_FWD_Y, binding.STAGE_FWD_XPROJ, binding.STAGE_FWD_PAIR):
        got = rmm.rmm_forward(X, W, None, k, kind, 5, 1, profile=(stage, a, b))
        assert torch.equal(Y, got[0]) and torch.equal(Xp, got[1]), stage
    for need_dX in (True, False):
        want = rmm.rmm_backward(dY, W, Xp, kind, 5, 1, need_dX=need_dX, need_dbias=True)
        for stage in (binding.STAGE_BWD_DX, binding.STAGE_BWD_G, binding.STAGE_BWD_DW, binding.STAGE_BWD_DBIAS):
            got = rmm.rmm_backward(dY, W, Xp, kind, 5, 1, need_dX=need_dX, need_dbias=True, profile=(stage, a, b))
            assert all(torch.equal(x, y) for x, y in zip(want, got) if x is not None), stage

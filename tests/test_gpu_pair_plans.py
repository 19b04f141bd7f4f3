"""GPU: paired launches whose work-groups share compute units two by two (128 x 128 tiles in two LDS stages, 64 x 256 sketch
tiles), and passes whose sketch product is cut differently from the same product alone: ragged edges, contractions of few
steps, against the fp64 oracle and bit for bit against the separate launches."""
import math

import pytest
import torch

import paper_2201_13195_amd as rmm
from paper_2201_13195_amd import binding, synth
from oracle import rmm as o_rmm
from parity import assert_close
from test_gpu_parity import check_layer

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,kind", [((4090, 776, 760, 400), rmm.GAUSSIAN),     # two to a compute unit, either pass
                                        ((4090, 776, 760, 400), rmm.RADEMACHER),
                                        ((6365, 632, 576, 318), rmm.GAUSSIAN),
                                        ((4100, 264, 1000, 300), rmm.GAUSSIAN),    # a contraction of five steps
                                        ((1201, 896, 3656, 240), rmm.RADEMACHER),  # 64 sketch work-groups beside 290 tiles
                                        ((3001, 1304, 520, 600), rmm.GAUSSIAN),    # fewer slices than alone
                                        ((1500, 1544, 520, 1400), rmm.RADEMACHER)])
def test_passes_with_plans_of_their_own(shape, kind):
    n, d_in, d_out, k = shape
    X, W, dY = synth.layer_inputs(n, d_in, d_out, "bf16", (n, d_in + 1, d_out + 2), w_std=1.0 / math.sqrt(d_in))
    bias = synth.to_torch(synth.normal((d_out,), 17), "bf16")
    check_layer(X, W, dY, k, kind, 0x5EED0071, 13, "bf16", bias=bias, label="plan %s" % (shape,))
    Xd, Wd, dYd = (t.to("cuda") for t in (X, W, dY))
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    a.record(); b.record()
    torch.cuda.synchronize()
    Y0, Xp0 = rmm.rmm_forward(Xd, Wd, None, k, kind, 5, 1)
    Y1, Xp1 = rmm.rmm_forward(Xd, Wd, None, k, kind, 5, 1, profile=(binding.STAGE_FWD_Y, a, b))
    dX0, dW0, _ = rmm.rmm_backward(dYd, Wd, Xp0, kind, 5, 1)
    dX1, dW1, _ = rmm.rmm_backward(dYd, Wd, Xp0, kind, 5, 1, profile=(binding.STAGE_BWD_DX, a, b))
    assert torch.equal(Y0, Y1) and torch.equal(Xp0, Xp1) and torch.equal(dX0, dX1) and torch.equal(dW0, dW1)


# Every pairing of a plain tile and a sketch tile that passes with 256 to 16384 tokens and widths of 256 to 4096 take:
# (tokens, width of the sketched operand, other width, k), kind, tiles ("split": dX with two wave groups).  (test_launch_plans.py: they take these, and there are no others.)
PAIRS = [((4439, 280, 2776, 222), rmm.GAUSSIAN, "256x256", "128x256"),
         ((4439, 280, 2776, 222), rmm.RADEMACHER, "256x256", "128x256"),
         ((7121, 304, 1320, 356), rmm.GAUSSIAN, "256x256", "128x384"),
         ((7121, 304, 1320, 356), rmm.RADEMACHER, "256x256", "128x384"),
         ((4563, 272, 2632, 228), rmm.GAUSSIAN, "256x256", "128x512"),
         ((4563, 272, 2632, 228), rmm.RADEMACHER, "256x256", "128x512"),
         ((2567, 272, 3736, 128), rmm.GAUSSIAN, "256x256", "64x256"),
         ((2567, 272, 3736, 128), rmm.RADEMACHER, "256x256", "64x256"),
         ((3243, 272, 3992, 162), rmm.GAUSSIAN, "256x256", "64x384"),
         ((3331, 392, 3152, 167), rmm.RADEMACHER, "256x256", "64x384"),
         ((5356, 264, 1928, 268), rmm.GAUSSIAN, "256x256", "64x512"),
         ((5356, 264, 1928, 268), rmm.RADEMACHER, "256x256", "64x512"),
         ((962, 2744, 328, 192), rmm.GAUSSIAN, "128x128 split", "128x256"),
         ((1285, 1872, 272, 257), rmm.RADEMACHER, "128x128 split", "128x256"),
         ((4056, 1576, 264, 406), rmm.GAUSSIAN, "128x128 split", "128x384"),
         ((2604, 1552, 440, 521), rmm.RADEMACHER, "128x128 split", "128x384"),
         ((3865, 1552, 664, 193), rmm.GAUSSIAN, "128x128 split", "128x512"),
         ((904, 1624, 3728, 90), rmm.RADEMACHER, "128x128 split", "128x512"),
         ((330, 1624, 264, 66), rmm.GAUSSIAN, "128x128 split", "64x256"),
         ((330, 1624, 264, 66), rmm.RADEMACHER, "128x128 split", "64x256"),
         ((516, 3920, 280, 103), rmm.GAUSSIAN, "128x128 split", "64x384"),
         ((516, 3920, 280, 103), rmm.RADEMACHER, "128x128 split", "64x384"),
         ((1687, 2120, 312, 337), rmm.GAUSSIAN, "128x128 split", "64x512"),
         ((2819, 2632, 296, 141), rmm.RADEMACHER, "128x128 split", "64x512"),
         ((1456, 520, 2184, 73), rmm.GAUSSIAN, "128x128", "128x256"),
         ((1299, 400, 2480, 65), rmm.RADEMACHER, "128x128", "128x256"),
         ((1550, 344, 2200, 78), rmm.GAUSSIAN, "128x128", "128x384"),
         ((1358, 264, 2696, 68), rmm.RADEMACHER, "128x128", "128x384"),
         ((1352, 392, 2776, 68), rmm.GAUSSIAN, "128x128", "128x512"),
         ((1352, 392, 2776, 68), rmm.RADEMACHER, "128x128", "128x512"),
         ((324, 272, 280, 65), rmm.GAUSSIAN, "128x128", "64x256"),
         ((324, 272, 280, 65), rmm.RADEMACHER, "128x128", "64x256"),
         ((520, 776, 280, 468), rmm.GAUSSIAN, "128x128", "64x384"),
         ((520, 776, 280, 468), rmm.RADEMACHER, "128x128", "64x384"),
         ((1299, 400, 2480, 65), rmm.GAUSSIAN, "128x128", "64x512"),
         ((2840, 400, 1064, 142), rmm.RADEMACHER, "128x128", "64x512"),
         ((1358, 264, 2696, 68), rmm.GAUSSIAN, "128x128 compact", "64x256"),
         ((1411, 264, 2648, 71), rmm.RADEMACHER, "128x128 compact", "64x256"),
         ((7362, 408, 2112, 368), rmm.GAUSSIAN, "128x256", "128x256"),
         ((2428, 840, 2984, 121), rmm.RADEMACHER, "128x256", "128x256"),
         ((921, 2416, 3232, 828), rmm.GAUSSIAN, "128x256", "128x384"),
         ((7823, 344, 2280, 391), rmm.RADEMACHER, "128x256", "128x384"),
         ((2078, 992, 3024, 207), rmm.GAUSSIAN, "128x256", "128x512"),
         ((2078, 992, 3024, 207), rmm.RADEMACHER, "128x256", "128x512"),
         ((1042, 1488, 3928, 65), rmm.GAUSSIAN, "128x256", "64x256"),
         ((1042, 1488, 3928, 65), rmm.RADEMACHER, "128x256", "64x256"),
         ((3360, 1288, 1472, 168), rmm.GAUSSIAN, "128x256", "64x384"),
         ((5481, 360, 3496, 274), rmm.RADEMACHER, "128x256", "64x384"),
         ((2428, 840, 2984, 121), rmm.GAUSSIAN, "128x256", "64x512"),
         ((2070, 1320, 2808, 414), rmm.RADEMACHER, "128x256", "64x512")]


@pytest.mark.parametrize("shape,kind,plain,sketch", PAIRS)
def test_every_pairing_of_tiles(shape, kind, plain, sketch):
    """Forward over A, backward over the same A as dY with W transposed: Y and dX are the same product, X_proj and G too."""
    n, d, d_other, k = shape
    A, W, Xp = (synth.to_torch(synth.normal(s, 0x5EED0080 + sum(s), std), "bf16")
                for s, std in (((n, d), 1.0), ((d_other, d), 1.0 / math.sqrt(d)), ((k, d_other), 1.0)))
    oY, oG = o_rmm.forward(synth.to_f64(A), synth.to_f64(W), None, k, kind, 0x5EED0081, 14)
    Ad, Wd, Wt, Xpd = A.to("cuda"), W.to("cuda"), W.t().contiguous().to("cuda"), Xp.to("cuda")
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    a.record(); b.record()
    Y, G = rmm.rmm_forward(Ad, Wd, None, k, kind, 0x5EED0081, 14)
    dX, dW, _ = rmm.rmm_backward(Ad, Wt, Xpd, kind, 0x5EED0081, 14)
    label = "%s beside %s %s" % (sketch, plain, shape)
    for got, want, what in ((Y, oY, "Y"), (G, oG, "X_proj"), (dX, oY, "dX"), (dW, oG.T @ synth.to_f64(Xp), "dW")):
        assert_close(got, want, what, "bf16", label)
    Y1, G1 = rmm.rmm_forward(Ad, Wd, None, k, kind, 0x5EED0081, 14, profile=(binding.STAGE_FWD_Y, a, b))
    dX1, dW1, _ = rmm.rmm_backward(Ad, Wt, Xpd, kind, 0x5EED0081, 14, profile=(binding.STAGE_BWD_DX, a, b))
    assert torch.equal(Y, Y1) and torch.equal(G, G1) and torch.equal(dX, dX1) and torch.equal(dW, dW1)


# dX on 128 x 256 tiles with the column sums of dY in its launch, behind the plain tiles or behind sketch work-groups in front of them, with and without short last
# slices: (tokens, d_in, d_out, k), kind.  (test_launch_plans.py: they take these.)
WIDE_WITH_BIAS = [((1340, 2864, 2192, 1206), rmm.RADEMACHER), ((1238, 4016, 3768, 247), rmm.GAUSSIAN), ((2486, 1672, 1824, 248), rmm.RADEMACHER),
                  ((1904, 2168, 1704, 952), rmm.GAUSSIAN), ((2582, 4072, 792, 1291), rmm.GAUSSIAN), ((2050, 3088, 1216, 1845), rmm.RADEMACHER),
                  ((2693, 1776, 1832, 134), rmm.GAUSSIAN), ((3364, 1120, 2016, 168), rmm.RADEMACHER)]


@pytest.mark.parametrize("shape,kind", WIDE_WITH_BIAS)
def test_bias_gradient_beside_wide_tiles(shape, kind):
    n, d_in, d_out, k = shape
    dY, W, Xp = (synth.to_torch(synth.normal(s, 0x5EED00B0 + sum(s), std), "bf16")
                 for s, std in (((n, d_out), 1.0), ((d_out, d_in), 1.0 / math.sqrt(d_out)), ((k, d_in), 1.0)))
    odX, odW, odb = o_rmm.backward(synth.to_f64(dY), synth.to_f64(W), synth.to_f64(Xp), kind, 0x5EED00B1, 16)
    dYd, Wd, Xpd = dY.to("cuda"), W.to("cuda"), Xp.to("cuda")
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    a.record(); b.record()
    torch.cuda.synchronize()
    got = rmm.rmm_backward(dYd, Wd, Xpd, kind, 0x5EED00B1, 16, need_dbias=True)
    for x, want, name in zip(got, (odX, odW, odb), ("dX", "dW", "db")):
        assert_close(x, want, name, "bf16", "wide with bias %s" % (shape,))
    for stage in (binding.STAGE_BWD_DX, binding.STAGE_BWD_DBIAS):      # both products apart, the column sums apart
        apart = rmm.rmm_backward(dYd, Wd, Xpd, kind, 0x5EED00B1, 16, need_dbias=True, profile=(stage, a, b))
        assert all(torch.equal(x, y) for x, y in zip(got, apart)), stage
    dW, db = got[1].clone(), got[2].clone()
    again = rmm.rmm_backward(dYd, Wd, Xpd, kind, 0x5EED00B1, 16, dW=dW, dbias=db, need_dbias=True, accumulate=True)
    assert torch.equal(again[0], got[0])
    assert_close(db, odb + synth.to_f64(got[2]), "db", "bf16", "wide with bias, accumulated %s" % (shape,))
    assert_close(dW, odW + synth.to_f64(got[1]), "dW", "bf16", "wide with bias, accumulated %s" % (shape,))


@pytest.mark.parametrize("n,d,d_other", [(4096, 3072, 768), (4090, 776, 760), (2056, 1544, 1032), (16384, 1024, 1024)])
def test_y_has_the_same_bits_beside_any_sketch(n, d, d_other):
    """k, kind and scratch choose how the launch of Y with a sketch product is made up; the bits of Y follow from its sizes."""
    A, W = (synth.to_torch(synth.normal(s, 0x5EED0090 + sum(s), std), "bf16").to("cuda") for s, std in (((n, d), 1.0), ((d_other, d), 0.05)))
    want, few = None, False
    for kind in (rmm.GAUSSIAN, rmm.RADEMACHER, rmm.SORS):
        for k in (1, 7, 25, 33, 64, 65, n // 20, n // 10, n // 5, n // 2, 9 * n // 10):
            if rmm.rmm_uses_paired_launch(n, d, d_other, k, torch.bfloat16, kind, binding.OP_FORWARD):
                Y, _ = rmm.rmm_forward(A, W, None, k, kind, 5, 1)
                want = Y if want is None else want
                assert torch.equal(Y, want), (kind, k)
                few |= k <= 64
    assert few


@pytest.mark.parametrize("shape,kind", [((640, 2056, 512, 25), rmm.GAUSSIAN), ((4099, 264, 1032, 33), rmm.RADEMACHER), ((738, 2656, 384, 64), rmm.GAUSSIAN)])
def test_few_sketch_columns_without_dx_are_made_by_the_streaming_kernel(shape, kind):
    """(tokens, d_in, d_out, k): dW without dX is the product of what rmm_sketch makes of dY, bit for bit and in any scratch; with dX, whose launch it shares, as
    close.  (X_proj = 1 where its row and column meet, d_in >= k: dW's columns are G's rows.)"""
    n, d_in, d_out, k = shape
    assert rmm.rmm_uses_paired_launch(n, d_in, d_out, k, torch.bfloat16, kind, binding.OP_BACKWARD) and d_in >= k
    dY = synth.to_torch(synth.normal((n, d_out), 0x5EED00C0), "bf16").to("cuda")
    W = synth.to_torch(synth.normal((d_out, d_in), 0x5EED00C1, 0.05), "bf16").to("cuda")
    Xp = torch.zeros((k, d_in), dtype=torch.bfloat16, device="cuda")
    Xp[range(k), range(k)] = 1
    G = rmm.rmm_sketch(dY, k, kind, 5, 1)
    _, alone, _ = rmm.rmm_backward(dY, W, Xp, kind, 5, 1, need_dX=False)
    assert torch.equal(alone[:, :k], G.t())
    _, beside, _ = rmm.rmm_backward(dY, W, Xp, kind, 5, 1)
    assert_close(beside[:, :k], synth.to_f64(G.t()), "dW", "bf16", "few columns beside dX %s" % (shape,))


@pytest.mark.parametrize("shape,kind", [((8192, 776, 760, 64), rmm.GAUSSIAN),      # sketch tiles of exactly 64 rows
                                        ((4099, 1032, 264, 33), rmm.RADEMACHER),   # ragged tokens and widths, half a sketch tile
                                        ((640, 512, 2056, 25), rmm.GAUSSIAN),
                                        ((1030, 264, 1000, 1), rmm.RADEMACHER),    # one sketch column
                                        ((60, 48, 520, 3), rmm.GAUSSIAN)])         # fewer tokens than a tile has rows
def test_few_sketch_columns_in_the_paired_launch(shape, kind):
    """k <= 64: against the oracle, bit for bit against the separate launches, and without dX."""
    n, d, d_other, k = shape
    assert rmm.rmm_uses_paired_launch(n, d, d_other, k, torch.bfloat16, kind, binding.OP_FORWARD)
    assert rmm.rmm_uses_paired_launch(n, d_other, d, k, torch.bfloat16, kind, binding.OP_BACKWARD)
    A, W, Xp = (synth.to_torch(synth.normal(s, 0x5EED00A0 + sum(s), std), "bf16")
                for s, std in (((n, d), 1.0), ((d_other, d), 1.0 / math.sqrt(d)), ((k, d_other), 1.0)))
    oY, oG = o_rmm.forward(synth.to_f64(A), synth.to_f64(W), None, k, kind, 0x5EED00A1, 14)
    want = dict(Y=oY, X_proj=oG, dX=oY, dW=oG.T @ synth.to_f64(Xp), db=synth.to_f64(A).sum(0))
    Ad, Wd, Wt, Xpd = A.to("cuda"), W.to("cuda"), W.t().contiguous().to("cuda"), Xp.to("cuda")
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    a.record(); b.record()
    torch.cuda.synchronize()

    def run(profiles=(None, None)):
        Y, G = rmm.rmm_forward(Ad, Wd, None, k, kind, 0x5EED00A1, 14, profile=profiles[0])
        dX, dW, db = rmm.rmm_backward(Ad, Wt, Xpd, kind, 0x5EED00A1, 14, need_dbias=True, profile=profiles[1])
        return dict(Y=Y, X_proj=G, dX=dX, dW=dW, db=db)

    paired = run()
    for name, got in paired.items():
        assert_close(got, want[name], name, "bf16", "few columns %s" % (shape,))
    for name, got in run(((binding.STAGE_FWD_Y, a, b), (binding.STAGE_BWD_DX, a, b))).items():
        assert torch.equal(got, paired[name]), name
    dX, dW, _ = rmm.rmm_backward(Ad, Wt, Xpd, kind, 0x5EED00A1, 14, need_dX=False)
    assert_close(dW, want["dW"], "dW", "bf16", "few columns %s, no dX" % (shape,))

"""GPU: Y of odd widths whose X and W have rows on 16 bytes, on the tiles that write rows that start anywhere: every width modulo 8, ragged rows and
contractions, with and without a bias, alone and beside the sketch product; nothing behind the last row is written."""
import math

import pytest
import torch

import paper_2201_13195_amd as rmm
from paper_2201_13195_amd import binding, synth
from oracle import rmm as o_rmm
from parity import assert_close

pytestmark = pytest.mark.gpu

# (tokens, d_in, d_out, k), kind, tile (test_launch_plans.py: they take these)
SHAPES = [((3000, 768, 1001, 300), rmm.GAUSSIAN, "128x128 compact"), ((2050, 72, 1153, 40), rmm.RADEMACHER, "128x128 compact"),
          ((2050, 200, 1002, 33), rmm.SORS, "128x128 compact"), ((1700, 200, 1001, 33), rmm.SORS, "64x128"), ((1340, 1080, 1217, 134), rmm.RADEMACHER, "64x128"),
          ((772, 1000, 1412, 77), rmm.GAUSSIAN, "64x128"), ((1042, 144, 1027, 997), rmm.RADEMACHER, "64x128"), ((705, 264, 2155, 634), rmm.GAUSSIAN, "64x128"),
          ((1025, 8, 1030, 16), rmm.GAUSSIAN, "64x128"), ((901, 136, 1197, 20), rmm.RADEMACHER, "64x128"), ((1111, 520, 967, 90), rmm.SORS, "64x128")]


@pytest.mark.parametrize("shape,kind,tile", SHAPES)
def test_y_of_any_width(shape, kind, tile):
    n, d_in, d_out, k = shape
    X, W = (synth.to_torch(synth.normal(s, 0x5EED00A0 + sum(s), std), "bf16") for s, std in (((n, d_in), 1.0), ((d_out, d_in), 1.0 / math.sqrt(d_in))))
    bias = synth.to_torch(synth.normal((d_out,), 19), "bf16")
    Xd, Wd, bd = X.to("cuda"), W.to("cuda"), bias.to("cuda")
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    a.record(); b.record()
    for with_bias in (False, True):
        oY, oXp = o_rmm.forward(synth.to_f64(X), synth.to_f64(W), synth.to_f64(bias) if with_bias else None, k, kind, 0x5EED00A1, 15)
        room = torch.full((n * d_out + 64,), 7.0, dtype=torch.bfloat16, device="cuda")
        Y = room[:n * d_out].view(n, d_out)
        got, Xp = rmm.rmm_forward(Xd, Wd, bd if with_bias else None, k, kind, 0x5EED00A1, 15, Y=Y)
        assert got.data_ptr() == Y.data_ptr() and bool((room[n * d_out:] == 7.0).all())
        assert_close(Y, oY, "Y", "bf16", "%s %s" % (tile, shape))
        assert_close(Xp, oXp, "X_proj", "bf16", "%s %s" % (tile, shape))
        alone = rmm.rmm_forward(Xd, Wd, bd if with_bias else None, k, kind, 0x5EED00A1, 15, profile=(binding.STAGE_FWD_Y, a, b))
        assert torch.equal(alone[0], Y) and torch.equal(alone[1], Xp)
        only, _ = rmm.rmm_forward(Xd, Wd, bd if with_bias else None, k, kind, 0, 0, need_xproj=False)
        assert_close(only, oY, "Y", "bf16", "%s %s alone" % (tile, shape))


# beside a sketch product on 64 x 64 tiles, or on another tile than alone (test_launch_plans.py)
BESIDE = [((1200, 264, 1043, 300), rmm.GAUSSIAN), ((455, 520, 2525, 227), rmm.GAUSSIAN), ((351, 2440, 2695, 35), rmm.SORS), ((1835, 512, 2903, 917), rmm.RADEMACHER)]


@pytest.mark.parametrize("shape,kind", BESIDE)
def test_y_keeps_its_tile_when_the_products_of_a_pass_are_launched_one_by_one(shape, kind):
    n, d_in, d_out, k = shape
    X, W = (synth.to_torch(synth.normal(s, 0x5EED00A8 + sum(s), std), "bf16") for s, std in (((n, d_in), 1.0), ((d_out, d_in), 1.0 / math.sqrt(d_in))))
    oY, oXp = o_rmm.forward(synth.to_f64(X), synth.to_f64(W), None, k, kind, 0x5EED00A9, 15)
    Xd, Wd = X.to("cuda"), W.to("cuda")
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    a.record(); b.record()
    Y, Xp = rmm.rmm_forward(Xd, Wd, None, k, kind, 0x5EED00A9, 15)
    only, _ = rmm.rmm_forward(Xd, Wd, None, k, kind, 0, 0, need_xproj=False)
    for got, want, name in ((Y, oY, "Y"), (only, oY, "Y"), (Xp, oXp, "X_proj")):
        assert_close(got, want, name, "bf16", "beside %s" % (shape,))
    alone = rmm.rmm_forward(Xd, Wd, None, k, kind, 0x5EED00A9, 15, profile=(binding.STAGE_FWD_Y, a, b))
    assert torch.equal(alone[0], Y) and torch.equal(alone[1], Xp)

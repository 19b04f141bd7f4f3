"""GPU: plain products on each tile of the menu (64 x 64 to 128 x 256; 256 x 256: test_gpu_large_tiles.py) at contractions
of one step, fewer steps than LDS stages, an odd number and a ragged last one, with ragged edges, against the fp64 oracle.
(test_launch_plans.py: these shapes take these tiles.)"""
import math

import pytest

import paper_2201_13195_amd as rmm
from paper_2201_13195_amd import synth
from oracle import rmm as o_rmm
from parity import assert_close
from test_gpu_parity import check_layer

pytestmark = pytest.mark.gpu

# (n, width across, contractions): the tile that Y (d_in = contraction) and dX (d_out = contraction) take
TILES = [(700, 1032, (8, 64, 72, 136, 200, 328)),   # 64 x 64, four stages
         (1290, 1000, (8, 72, 136, 200)),           # 64 x 128
         (2300, 1544, (136, 192, 264)),             # 128 x 128
         (2100, 1288, (1544, 1608)),                # 128 x 128, two wave groups
         (2500, 1544, (8, 72, 136, 200))]           # 128 x 256
SHAPES = [(n, c, w, 50) for n, w, cs in TILES for c in cs] + [(n, w, c, 50) for n, w, cs in TILES for c in cs]


@pytest.mark.parametrize("shape", SHAPES)
def test_plain_products_on_every_tile(shape):
    n, d_in, d_out, k = shape
    kind = rmm.RADEMACHER if d_in % 3 == 0 else rmm.GAUSSIAN
    X, W, dY = synth.layer_inputs(n, d_in, d_out, "bf16", (n, d_in + 1, d_out + 2), w_std=1.0 / math.sqrt(d_in))
    bias = synth.to_torch(synth.normal((d_out,), 17), "bf16")
    check_layer(X, W, dY, k, kind, 0x5EED0052, 10, "bf16", bias=bias, label="tile %s" % (shape,))


# dW on 64 x 128, 128 x 128, 128 x 128 with two wave groups, 128 x 256 and 64 x 64, with its bias gradient, and once more on
# top of what is there
@pytest.mark.parametrize("d_out,d_in,k", [(1290, 1000, 200), (2304, 1544, 264), (2096, 1288, 1608), (2504, 1544, 136), (704, 1032, 72)])
def test_weight_gradient_on_every_tile(d_out, d_in, k):
    n = 400
    d_out -= d_out % 8
    X, W, dY = synth.layer_inputs(n, d_in, d_out, "bf16", (n, d_in + 1, d_out + 2), w_std=1.0 / math.sqrt(d_in))
    check_layer(X, W, dY, k, rmm.RADEMACHER, 0x5EED0053, 10, "bf16", bias=synth.to_torch(synth.normal((d_out,), 17), "bf16"),
                label="dW tile %s" % ((d_out, d_in, k),))
    Wd, dYd = W.to("cuda"), dY.to("cuda")
    Xp = rmm.rmm_sketch(X.to("cuda"), k, rmm.RADEMACHER, 0x5EED0053, 10)
    _, dW, db = rmm.rmm_backward(dYd, Wd, Xp, rmm.RADEMACHER, 0x5EED0053, 10, need_dX=False, need_dbias=True)
    first = synth.to_f64(dW).copy(), synth.to_f64(db).copy()
    rmm.rmm_backward(dYd, Wd, Xp, rmm.RADEMACHER, 0x5EED0053, 11, need_dX=False, dW=dW, dbias=db, need_dbias=True, accumulate=True)
    _, odW, odb = o_rmm.backward(synth.to_f64(dY), synth.to_f64(W), synth.to_f64(Xp), rmm.RADEMACHER, 0x5EED0053, 11)
    assert_close(dW, first[0] + odW, "dW", "bf16", "dW twice, tile %s" % ((d_out, d_in, k),))
    assert_close(db, first[1] + odb, "db", "bf16", "db twice, tile %s" % ((d_out, d_in, k),))

"""GPU: plain products on 256 x 256 tiles (loads straight into LDS, two stages) at contractions of one step,
two, an odd number and a ragged last one, with ragged edges, against the fp64 oracle."""
import math

import pytest

import paper_2201_13195_amd as rmm
from paper_2201_13195_amd import synth
from test_gpu_parity import check_layer

pytestmark = pytest.mark.gpu

# 160 tiles or more in Y (d_out wide, contraction d_in) or in dX (d_in wide, contraction d_out).
SHAPES = [(2600, c, 4000, 50) for c in (8, 64, 72, 200)] + [(2600, 4000, c, 50) for c in (8, 64, 72, 200)]


@pytest.mark.parametrize("shape", SHAPES)
def test_large_tile_products(shape):
    n, d_in, d_out, k = shape
    kind = rmm.RADEMACHER if d_in % 3 == 0 else rmm.GAUSSIAN
    X, W, dY = synth.layer_inputs(n, d_in, d_out, "bf16", (n, d_in + 1, d_out + 2), w_std=1.0 / math.sqrt(d_in))
    bias = synth.to_torch(synth.normal((d_out,), 17), "bf16")
    check_layer(X, W, dY, k, kind, 0x5EED0051, 10, "bf16", bias=bias, label="large %s" % (shape,))

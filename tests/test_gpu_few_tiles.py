"""GPU: products with few output tiles (contraction split over the waves of a work-group) at the edges of
their tiles, steps and switch points, against the fp64 oracle."""
import math

import pytest

import paper_2201_13195_amd as rmm
from paper_2201_13195_amd import synth
from test_gpu_parity import check_layer

pytestmark = pytest.mark.gpu

SHAPES = [
    # (n, d_in, d_out, k)
    (1, 8, 8, 1), (31, 40, 24, 7), (33, 504, 72, 66),        # less than a tile, a wave with nothing to do
    (64, 512, 520, 512), (65, 520, 512, 520),                 # contractions of one step of every wave and one chunk more
    (512, 1024, 1024, 70), (520, 1032, 1016, 129),            # 512 and 561 tiles of 32 x 32, on 64 x 64 tiles by the contraction
    (1277, 344, 344, 50), (1000, 512, 400, 30),               # 440 and 416 of them, two to a compute unit
    (40, 4104, 24, 300), (1000, 1032, 1000, 1030),            # long contractions, ragged everywhere
]


@pytest.mark.parametrize("shape", SHAPES)
def test_few_tile_products(shape):
    n, d_in, d_out, k = shape
    kind = rmm.GAUSSIAN if n % 2 == 0 else rmm.RADEMACHER
    X, W, dY = synth.layer_inputs(n, d_in, d_out, "bf16", (n, d_in + 1, d_out + 2), w_std=1.0 / math.sqrt(d_in))
    bias = synth.to_torch(synth.normal((d_out,), 17), "bf16")
    check_layer(X, W, dY, k, kind, 0x5EED0041, 9, "bf16", bias=bias, label="few %s" % (shape,))

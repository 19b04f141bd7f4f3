"""GPU: sketch products whose tokens are cut into long slices and one short slice per tile (several short slices to a
work-group), with ragged token counts and edges, against the fp64 oracle."""
import math

import pytest

import paper_2201_13195_amd as rmm
from paper_2201_13195_amd import synth
from test_gpu_parity import check_layer

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,kind", [((7757, 512, 264, 1384), rmm.GAUSSIAN),     # 22 tiles, eleven long slices
                                        ((1827, 2408, 264, 1680), rmm.GAUSSIAN),    # 70 tiles, three
                                        ((1827, 2408, 264, 1680), rmm.RADEMACHER),  # 98 tiles, two
                                        ((2219, 2312, 264, 1616), rmm.RADEMACHER),  # an odd number of tiles
                                        ((4097, 2896, 264, 1063), rmm.RADEMACHER)])  # one token in the last step
def test_long_and_short_slices(shape, kind):
    n, d_in, d_out, k = shape
    X, W, dY = synth.layer_inputs(n, d_in, d_out, "bf16", (n, d_in + 1, d_out + 2), w_std=1.0 / math.sqrt(d_in))
    check_layer(X, W, dY, k, kind, 0x5EED0061, 11, "bf16", label="slices %s" % (shape,))

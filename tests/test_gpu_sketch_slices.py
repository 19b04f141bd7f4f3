"""GPU: sketch products whose tokens are cut into long slices and one short slice per tile (several short slices to a
work-group), with ragged token counts and edges, against the fp64 oracle.  (test_launch_plans.py: these shapes are cut so.)"""
import math

import pytest
import torch

import paper_2201_13195_amd as rmm
from oracle import rmm as o_rmm
from paper_2201_13195_amd import binding, synth
from parity import assert_close
from test_gpu_parity import check_layer

pytestmark = pytest.mark.gpu


# S^T X with long and short slices on its own
@pytest.mark.parametrize("shape,kind", [((1827, 2408, 264, 1680), rmm.GAUSSIAN),     # 70 tiles, three long slices
                                        ((1827, 2408, 264, 1680), rmm.RADEMACHER),   # 98 tiles, two
                                        ((2219, 2312, 264, 1616), rmm.RADEMACHER),   # an odd number of tiles
                                        ((4097, 2896, 264, 1063), rmm.RADEMACHER)])  # one token in the last step
def test_long_and_short_slices_of_a_product_alone(shape, kind):
    n, d, _, k = shape
    X = synth.to_torch(synth.normal((n, d), 21), "bf16")
    got = rmm.rmm_sketch(X.to("cuda"), k, kind, 0x5EED0063, 14)
    _, want = o_rmm.forward(synth.to_f64(X), synth.to_f64(X[:8]), None, k, kind, 0x5EED0063, 14)
    assert_close(got, want, "X_proj", "bf16", "slices alone %s" % (shape,))


# S^T dY with long and short slices beside dX
IN_A_PASS = [((7757, 512, 264, 1384), rmm.GAUSSIAN), ((2183, 304, 1880, 167), rmm.GAUSSIAN), ((2133, 176, 1032, 1056), rmm.GAUSSIAN),
             ((2697, 224, 2704, 182), rmm.RADEMACHER)]


@pytest.mark.parametrize("shape,kind", IN_A_PASS[1:])
def test_long_and_short_slices_in_a_backward_pass(shape, kind):
    n, d_in, d_out, k = shape
    X, W, dY = synth.layer_inputs(n, d_in, d_out, "bf16", (n, d_in + 1, d_out + 2), w_std=1.0 / math.sqrt(d_in))
    check_layer(X, W, dY, k, kind, 0x5EED0064, 15, "bf16", label="slices in a pass %s" % (shape,))


# (as the passes cut them: long slices, one, and in the first backward pass short ones too)
@pytest.mark.parametrize("shape,kind", [((7757, 512, 264, 1384), rmm.GAUSSIAN),
                                        ((1827, 2408, 264, 1680), rmm.GAUSSIAN),
                                        ((1827, 2408, 264, 1680), rmm.RADEMACHER),
                                        ((2219, 2312, 264, 1616), rmm.RADEMACHER),
                                        ((4097, 2896, 264, 1063), rmm.RADEMACHER)])
def test_long_and_short_slices(shape, kind):
    n, d_in, d_out, k = shape
    X, W, dY = synth.layer_inputs(n, d_in, d_out, "bf16", (n, d_in + 1, d_out + 2), w_std=1.0 / math.sqrt(d_in))
    check_layer(X, W, dY, k, kind, 0x5EED0061, 11, "bf16", label="slices %s" % (shape,))


@pytest.mark.parametrize("kind", [rmm.GAUSSIAN, rmm.RADEMACHER])
def test_slices_of_a_pass_with_a_bias_gradient(kind):
    """Short last slices given up for the column sums of dY: G differs from the pass without bias in the order of its
    sums only, and asking for a stage's events (separate launches) changes no bit."""
    n, d_in, d_out, k = 8192, 1000, 4000, 800
    X, W, dY = synth.layer_inputs(n, d_in, d_out, "bf16", (71, 72, 73), w_std=1.0 / math.sqrt(d_in))
    bias = synth.to_torch(synth.normal((d_out,), 17), "bf16")
    check_layer(X, W, dY, k, kind, 0x5EED0062, 12, "bf16", bias=bias, label="slices with bias")
    dev = [t.to("cuda") for t in (dY, W)]
    Xp = rmm.rmm_sketch(X.to("cuda"), k, kind, 0x5EED0062, 12)
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    a.record(); b.record()
    torch.cuda.synchronize()
    one = rmm.rmm_backward(*dev, Xp, kind, 0x5EED0062, 12, need_dbias=True)
    for stage in (binding.STAGE_BWD_DX, binding.STAGE_BWD_G, binding.STAGE_BWD_DW, binding.STAGE_BWD_DBIAS):
        for x, y in zip(one, rmm.rmm_backward(*dev, Xp, kind, 0x5EED0062, 12, need_dbias=True, profile=(stage, a, b))):
            assert torch.equal(x, y), stage
    assert torch.equal(one[1], rmm.rmm_backward(*dev, Xp, kind, 0x5EED0062, 12, need_dX=False, need_dbias=True)[1])

"""GPU: paired launches whose work-groups share compute units two by two (128 x 128 tiles in two LDS stages, 64 x 256 sketch
tiles), and passes whose sketch product is cut differently from the same product alone: ragged edges, contractions of few
steps, against the fp64 oracle and bit for bit against the separate launches."""
import math

import pytest
import torch

import paper_2201_13195_amd as rmm
from paper_2201_13195_amd import binding, synth
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

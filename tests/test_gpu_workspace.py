"""GPU: passes in less scratch than rmm_workspace_bytes() says, down to the least that they run in: the same results
but for the order of fp32 sums, and nothing written behind the scratch that was given."""
import math

import numpy as np
import pytest
import torch

import paper_2201_13195_amd as rmm
from oracle import rmm as o_rmm
from paper_2201_13195_amd import binding, synth
from parity import assert_close

pytestmark = pytest.mark.gpu
SEED, OFFSET, GUARD = 0x5EED0081, 16, 4096


class Scratch:
    """`size` bytes for a call, followed by a guard that has to stay as it is."""

    def __init__(self, size):
        self.all = torch.full((size + GUARD,), 0x5A, dtype=torch.uint8, device="cuda")
        self.ws = self.all[:size] if size > 0 else self.all[:0]

    def untouched(self):
        return bool((self.all[self.ws.numel():] == 0x5A).all())


def inputs(n, d_in, d_out):
    X, W, dY = synth.layer_inputs(n, d_in, d_out, "bf16", (n, d_in + 1, d_out + 2), w_std=1.0 / math.sqrt(d_in))
    return (X, W, dY), [t.to("cuda") for t in (X, W, dY)]


def check_pass(shape, kind, forward_sizes, backward_sizes):
    n, d_in, d_out, k = shape
    (X, W, dY), (Xd, Wd, dYd) = inputs(n, d_in, d_out)
    bf16 = torch.bfloat16
    oY, oXp = o_rmm.forward(synth.to_f64(X), synth.to_f64(W), None, k, kind, SEED, OFFSET)
    for size in forward_sizes:
        s = Scratch(size)
        Y, Xp = rmm.rmm_forward(Xd, Wd, None, k, kind, SEED, OFFSET, ws=s.ws)
        assert s.untouched(), (shape, "forward", size)
        for name, got, want in (("Y", Y, oY), ("X_proj", Xp, oXp)):
            assert_close(got, want, name, "bf16", "%s in %d" % (shape, size))
    odX, odW, odb = o_rmm.backward(synth.to_f64(dY), synth.to_f64(W), synth.to_f64(Xp), kind, SEED, OFFSET)
    for size in backward_sizes:
        s = Scratch(size)
        dX, dW, db = rmm.rmm_backward(dYd, Wd, Xp, kind, SEED, OFFSET, need_dbias=True, ws=s.ws)
        assert s.untouched(), (shape, "backward", size)
        for name, got, want in (("dX", dX, odX), ("dW", dW, odW), ("db", db, odb)):
            assert_close(got, want, name, "bf16", "%s in %d" % (shape, size))
        # the products one by one, in the same scratch: the same bits
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record(); b.record()
        torch.cuda.synchronize()
        again = rmm.rmm_backward(dYd, Wd, Xp, kind, SEED, OFFSET, need_dbias=True, ws=s.ws, profile=(binding.STAGE_BWD_DX, a, b))
        assert torch.equal(dX, again[0]) and torch.equal(dW, again[1]) and torch.equal(db, again[2])
    with pytest.raises(rmm.RmmError) as e:
        rmm.rmm_backward(dYd, Wd, Xp, kind, SEED, OFFSET, ws=torch.empty(backward_sizes[0] - 1, dtype=torch.uint8, device="cuda"))
    assert e.value.status == -3


def up(x):
    return (x + 255) // 256 * 256


@pytest.mark.parametrize("kind", [rmm.GAUSSIAN, rmm.RADEMACHER, rmm.SORS])
@pytest.mark.parametrize("shape", [(3000, 768, 1001, 300), (2048, 1001, 264, 205), (1327, 2672, 313, 1194)])
def test_odd_widths_in_any_scratch_from_none_up(shape, kind):
    """Forward from no scratch on, backward from a G of rows that start anywhere: the sizes these passes took before their
    sketch products were cut, then padded rows of G, two slices, and what the query says."""
    n, d_in, d_out, k = shape
    need = [rmm.rmm_workspace_bytes(n, d_in, d_out, k, torch.bfloat16, kind, op) for op in (binding.OP_FORWARD, binding.OP_BACKWARD)]
    row = (d_out + 7) // 8 * 8
    padded = up(k * row * 2)
    forward = [0] + [s for s in (2 * k * d_in * 4 - 4, 2 * k * d_in * 4, need[0]) if s <= need[0]]
    backward = [up(k * d_out * 2)] + [s for s in (padded, padded + 2 * k * row * 4, need[1]) if s <= need[1]]
    check_pass(shape, kind, forward, backward)


@pytest.mark.parametrize("shape,kind", [((4096, 768, 3072, 410), rmm.GAUSSIAN), ((3001, 520, 1304, 600), rmm.RADEMACHER),
                                        ((2690, 864, 2376, 269), rmm.GAUSSIAN),        # (6 slices of X asked for)
                                        ((8192, 1000, 4000, 800), rmm.RADEMACHER),     # short last slices; column sums in the pair
                                        ((4096, 3072, 768, 2048), rmm.GAUSSIAN)])
def test_token_slices_follow_the_scratch(shape, kind):
    """From two slices up; and with the same scratch the same bits, whichever launches."""
    n, d_in, d_out, k = shape
    need = [rmm.rmm_workspace_bytes(n, d_in, d_out, k, torch.bfloat16, kind, op) for op in (binding.OP_FORWARD, binding.OP_BACKWARD)]
    g = up(k * d_out * 2)
    forward = [s for s in (up(2 * k * d_in * 4), 3 * k * d_in * 4, 5 * k * d_in * 4 - 4, need[0]) if s <= need[0]]
    backward = [g + s for s in (up(2 * k * d_out * 4), 3 * k * d_out * 4, 5 * k * d_out * 4 - 4, need[1] - g) if g + s <= need[1]]
    if not forward:
        forward = [0]
    if not backward:
        backward = [g]
    check_pass(shape, kind, forward, backward)
    if need[0] > 0:
        with pytest.raises(rmm.RmmError) as e:
            check_pass(shape, kind, [forward[0] - 1], [])
        assert e.value.status == -3


@pytest.mark.parametrize("shape,alone", [((4637, 1008, 304, 4173), False), ((2511, 3088, 440, 1255), True)])
def test_one_slice_where_passes_had_one(shape, alone):
    """A pass whose sketch product alone has no slices, for the size of its partial sums, asks for some and runs without; and one
    that had none beside a plain product on half of the compute units."""
    n, d_in, d_out, k = shape
    need = [rmm.rmm_workspace_bytes(n, d_in, d_out, k, torch.bfloat16, rmm.RADEMACHER, op) for op in (binding.OP_FORWARD, binding.OP_BACKWARD)]
    assert need[0] > 0 and (rmm.rmm_workspace_bytes(n, d_in, d_in, k, torch.bfloat16, rmm.RADEMACHER, binding.OP_SKETCH) > 0) == alone
    check_pass(shape, rmm.RADEMACHER, [0, need[0] - 4, need[0]], [up(k * d_out * 2) + up(2 * k * d_out * 4), need[1]])


@pytest.mark.parametrize("shape", [(4099, 1032, 264, 33), (8192, 776, 760, 64), (640, 2056, 512, 25), (100, 264, 520, 5)])
def test_few_sketch_columns_in_any_scratch(shape):
    """k <= 64: from what the streaming kernel of the sketch product takes (none, of few tokens) up to what the query says."""
    n, d_in, d_out, k = shape
    for kind in (rmm.GAUSSIAN, rmm.RADEMACHER):
        need = [rmm.rmm_workspace_bytes(n, d_in, d_out, k, torch.bfloat16, kind, op) for op in (binding.OP_FORWARD, binding.OP_BACKWARD)]
        alone = [rmm.rmm_workspace_bytes(n, d, d, k, torch.bfloat16, kind, binding.OP_SKETCH) for d in (d_in, d_out)]
        check_pass(shape, kind, [alone[0], need[0]], [up(k * d_out * 2) + alone[1], need[1]])


@pytest.mark.parametrize("shape", [(201, 200, 136), (1000, 264, 520), (2100, 1800, 520), (197, 2504, 776)])
def test_variance_monitors_in_less_scratch(shape):
    """Down to what 128 x 128 tiles of X^T dY take, and not below it; the same values but for the order of the sums."""
    n, d_in, d_out = shape
    (X, _, dY), (Xd, _, dYd) = inputs(n, d_in, d_out)
    need = rmm.rmm_workspace_bytes(n, d_in, d_out, 30, torch.bfloat16, rmm.GAUSSIAN, binding.OP_VARIANCE)
    want = rmm.rmm_variance_stats(Xd, dYd, 30, rmm.GAUSSIAN).cpu()
    xty = float(np.sum((synth.to_f64(X).T @ synth.to_f64(dY)) ** 2))
    sizes = []
    for size in range(need, 0, -256):
        s = Scratch(size)
        try:
            got = rmm.rmm_variance_stats(Xd, dYd, 30, rmm.GAUSSIAN, ws=s.ws).cpu()
        except rmm.RmmError as e:
            assert e.status == -3
            break
        assert s.untouched(), (shape, size)
        assert torch.allclose(got, want, rtol=1e-6, atol=0) and abs(float(got[3]) - xty) <= 2e-5 * xty, (shape, size)
        sizes.append(size)
    blocks = min((n + 7) // 8, 1024)                        # work-groups of the row norms: three values each
    assert sizes[-1] == min(need, up(8 * (3 * blocks + -(-d_in // 128) * -(-d_out // 128))))

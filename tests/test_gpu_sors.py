"""GPU parity of the SORS sketch kind (signs, Walsh-Hadamard transform along the tokens, row
selection; the construction is stated in include/rmm.h and oracle/sketch.py and is this build's
own, so parity with the paper is unpinned): every entry of S read back through an identity
operand, the sketch primitive and the whole layer against the fp64 oracle, on the fast-transform
kernel (bf16, width a multiple of 8, at most 32768 tokens) and on the entry-by-entry path that
serves everything else, and unbiasedness of the weight gradient over many states."""
import math

import numpy as np
import pytest
import torch

import paper_2201_13195_amd as rmm
from paper_2201_13195_amd import binding, synth
from oracle import rmm as o_rmm
from oracle import sketch as o_sketch
from parity import assert_close
from test_gpu_parity import check_layer

pytestmark = pytest.mark.gpu
DEV = "cuda"
SORS = rmm.SORS


@pytest.mark.parametrize("n,k", [(256, 40), (300, 64), (1000, 130), (1024, 1024), (4096, 410), (2056, 77), (8, 5), (1, 3)])
def test_every_entry_through_an_identity_operand(n, k):
    """S^T I = S^T: rmm_sketch on an identity returns sigma_i * (-1)^popcount(i AND r_j) / sqrt(k)
    rounded to bf16: signs exact, magnitude within one rounding.  Token counts on both sides of
    powers of two (the transform runs on n_pad) and below the kernel's shortest transform."""
    seed, offset = 0x5EED0020, (1 << 32) | 3
    d = (n + 7) // 8 * 8
    A = torch.zeros((n, d), dtype=torch.bfloat16, device=DEV)
    A[torch.arange(n), torch.arange(n)] = 1.0
    got = synth.to_f64(rmm.rmm_sketch(A, k, SORS, seed, offset))          # k x d
    want = o_sketch.sketch_S(n, k, o_sketch.SORS, seed, offset).T        # k x n
    assert np.array_equal(got[:, n:], np.zeros((k, d - n)))
    got = got[:, :n]
    assert np.array_equal(np.signbit(got), np.signbit(want))
    assert np.abs(np.abs(got) * math.sqrt(k) - 1.0).max() <= 2.0 ** -8


@pytest.mark.parametrize("n,d,k", [(256, 64, 32), (700, 264, 33), (4096, 768, 410), (4096, 3072, 410), (5000, 128, 300),
                                   (16384, 1024, 1638), (32768, 64, 100), (20000, 72, 9),
                                   (2048, 64, 50), (2049, 64, 50), (4097, 64, 50), (8192, 72, 2048),
                                   # more than 2048 sketch columns of more than 2048 tokens: sixteen waves to a strip
                                   (4096, 64, 3686), (3000, 72, 2049), (9000, 64, 2100), (16384, 16, 2304), (30000, 8, 2050)])
def test_sketch_primitive_fast_transform(n, d, k):
    A = synth.to_torch(synth.normal((n, d), 0x5EED0021 + n), "bf16")
    got = rmm.rmm_sketch(A.to(DEV), k, SORS, 0x5EED0022, 5)
    torch.cuda.synchronize()
    want = o_rmm.sketch_apply(synth.to_f64(A), k, o_sketch.SORS, 0x5EED0022, 5)
    err = assert_close(got, want, "X_proj", "bf16", "sors sketch n=%d d=%d k=%d" % (n, d, k))
    print("sors sketch n=%d d=%d k=%d: %.2e" % (n, d, k, err), flush=True)
    assert rmm.rmm_workspace_bytes(n, d, d, k, torch.bfloat16, SORS, binding.OP_SKETCH) == 0


@pytest.mark.parametrize("n,d,k", [(1025, 2056, 90), (2048, 2064, 300), (2049, 2072, 65), (4097, 2056, 2048)])
def test_two_strips_to_a_work_group(n, d, k):
    """More than 256 strips, also an odd number of them; one and several chunks, and the column sums beside them."""
    A = synth.to_torch(synth.normal((n, d), 0x5EED0024 + n), "bf16")
    got = rmm.rmm_sketch(A.to(DEV), k, SORS, 0x5EED0025, 5)
    want = o_rmm.sketch_apply(synth.to_f64(A), k, o_sketch.SORS, 0x5EED0025, 5)
    assert_close(got, want, "X_proj", "bf16", "sors sketch n=%d d=%d k=%d" % (n, d, k))
    W = torch.zeros((d, 8), dtype=torch.bfloat16, device=DEV)
    Xp = torch.zeros((k, 8), dtype=torch.bfloat16, device=DEV)
    _, _, db = rmm.rmm_backward(A.to(DEV), W, Xp, SORS, 0x5EED0025, 5, need_dX=False, need_dbias=True)
    assert_close(db, synth.to_f64(A).sum(axis=0), "db", "bf16", "sors db n=%d d=%d k=%d" % (n, d, k))


@pytest.mark.parametrize("n,d,k", [(2049, 8, 2049), (4096, 24, 8192), (4097, 520, 8193), (5000, 2056, 4100), (6001, 16, 9001), (16384, 24, 4099)])
def test_more_sketch_columns_than_a_strip_has_accumulators(n, d, k):
    """Strips shared by one to eight work-groups, the last of them with fewer sketch columns; waves with some, all and none of theirs."""
    A = synth.to_torch(synth.normal((n, d), 0x5EED0026 + n), "bf16")
    got = rmm.rmm_sketch(A.to(DEV), k, SORS, 0x5EED0027, 5)
    want = o_rmm.sketch_apply(synth.to_f64(A), k, o_sketch.SORS, 0x5EED0027, 5)
    assert_close(got, want, "X_proj", "bf16", "sors sketch n=%d d=%d k=%d" % (n, d, k))
    W = torch.zeros((d, 8), dtype=torch.bfloat16, device=DEV)
    Xp = torch.zeros((k, 8), dtype=torch.bfloat16, device=DEV)
    db = None
    for times in (1, 2):
        _, _, db = rmm.rmm_backward(A.to(DEV), W, Xp, SORS, 0x5EED0027, 5, need_dX=False, need_dbias=True, dbias=db, accumulate=times == 2,
                                    dW=torch.zeros((d, 8), dtype=torch.bfloat16, device=DEV))
        assert_close(db, times * synth.to_f64(A).sum(axis=0), "db", "bf16", "sors db n=%d d=%d k=%d, %d times" % (n, d, k, times))


@pytest.mark.parametrize("dtype,n,d,k", [("f32", 256, 128, 32), ("f32", 333, 50, 77), ("bf16", 333, 52, 20),
                                         ("bf16", 40000, 8, 8)])
def test_sketch_primitive_entry_by_entry_path(dtype, n, d, k):
    """fp32, widths that are not multiples of 8 and more than 32768 tokens: the same S applied densely."""
    A = synth.to_torch(synth.normal((n, d), 77), dtype)
    got = rmm.rmm_sketch(A.to(DEV), k, SORS, 0x5EED0023, 6)
    torch.cuda.synchronize()
    want = o_rmm.sketch_apply(synth.to_f64(A), k, o_sketch.SORS, 0x5EED0023, 6)
    assert_close(got, want, "X_proj", dtype, "sors dense %s n=%d d=%d k=%d" % (dtype, n, d, k))


@pytest.mark.parametrize("dtype,shape", [("f32", (256, 128, 128, 32)), ("bf16", (333, 200, 136, 77)),
                                         ("bf16", (1000, 264, 520, 129)), ("bf16", (130, 72, 264, 300))])
def test_layer_small_and_ragged(dtype, shape):
    n, d_in, d_out, k = shape
    X, W, dY = synth.layer_inputs(n, d_in, d_out, dtype, (811, 812, 813))
    bias = synth.to_torch(synth.normal((d_out,), 814), dtype)
    check_layer(X, W, dY, k, SORS, 0xABCDEF, 43, dtype, bias=bias, label="sors %s %s" % (shape, dtype))


@pytest.mark.parametrize("name", ["c2_base_attn", "c3_base_ffn_up", "c3_base_ffn_down", "c4_large_ffn_up"])
def test_layer_at_the_paper_shapes(name):
    c = synth.CONFIGS[name]
    X, W, dY = synth.layer_inputs(c["n"], c["d_in"], c["d_out"], c["dtype"], c["seeds"])
    check_layer(X, W, dY, c["k"], SORS, c["seed"], 21, "bf16", label="sors %s" % name)


def test_forward_backward_and_sketch_agree_and_are_deterministic():
    X, W, dY = synth.layer_inputs(1500, 264, 520, "bf16", (31, 32, 33))
    Xd, Wd, dYd = X.to(DEV), W.to(DEV), dY.to(DEV)
    Y1, Xp1 = rmm.rmm_forward(Xd, Wd, None, 96, SORS, 5, 6)
    Y2, Xp2 = rmm.rmm_forward(Xd, Wd, None, 96, SORS, 5, 6)
    Xp3 = rmm.rmm_sketch(Xd, 96, SORS, 5, 6)
    assert torch.equal(Y1, Y2) and torch.equal(Xp1, Xp2) and torch.equal(Xp1, Xp3)
    d1 = rmm.rmm_backward(dYd, Wd, Xp1, SORS, 5, 6)
    d2 = rmm.rmm_backward(dYd, Wd, Xp1, SORS, 5, 6)
    assert torch.equal(d1[0], d2[0]) and torch.equal(d1[1], d2[1])
    assert not torch.equal(Xp1, rmm.rmm_sketch(Xd, 96, SORS, 5, 7))
    assert not torch.equal(Xp1, rmm.rmm_sketch(Xd, 96, SORS, 4, 6))
    assert not torch.equal(Xp1, rmm.rmm_sketch(Xd, 96, rmm.RADEMACHER, 5, 6))


def test_weight_gradient_is_unbiased_on_the_device():
    """Mean of dW over 600 states against dY^T X (Eq. 3), at the 1/sqrt(states) rate."""
    n, d_in, d_out, k, states = 512, 64, 72, 64, 600
    X, W, dY = synth.layer_inputs(n, d_in, d_out, "bf16", (41, 42, 43))
    Xd, Wd, dYd = X.to(DEV), W.to(DEV), dY.to(DEV)
    exact = synth.to_f64(dY).T @ synth.to_f64(X)
    acc = np.zeros_like(exact)
    sq = np.zeros_like(exact)
    for t in range(states):
        _, Xp = rmm.rmm_forward(Xd, Wd, None, k, SORS, 77, t)
        _, dW, _ = rmm.rmm_backward(dYd, Wd, Xp, SORS, 77, t, need_dX=False)
        est = synth.to_f64(dW)
        acc += est
        sq += est * est
    mean = acc / states
    sd = np.sqrt(np.maximum(sq / states - mean * mean, 0.0) / states)
    z = np.abs(mean - exact) / (sd + 1e-3 * np.abs(exact).max())
    assert z.max() < 5.5, z.max()
    # and the estimator is not trivially exact: one state is far from the mean
    assert np.linalg.norm(est - exact) > 0.05 * np.linalg.norm(exact)


def test_variance_monitor_refuses_the_kind():
    X, W, dY = synth.layer_inputs(256, 128, 128, "bf16", (1, 2, 3))
    with pytest.raises(rmm.RmmError):
        rmm.rmm_variance_stats(X.to(DEV), dY.to(DEV), 32, SORS)


@pytest.mark.parametrize("name", ["c2_base_attn", "c3_base_ffn_up", "c3_base_ffn_down", "c4_large_attn"])
def test_paired_launch_gives_the_bits_of_the_separate_launches(name):
    """Where the plain product of a pass leaves compute units idle (strips behind its tiles), or
    runs full rounds beside few long strips (strips in front: the third shape), the strips of the
    sketch product share its launch; asking for a single product's stage makes the pass launch
    them one after the other.  Same kernels' arithmetic either way: every output must agree bit for bit."""
    c = synth.CONFIGS[name]
    n, d_in, d_out, k = c["n"], c["d_in"], c["d_out"], c["k"]
    assert rmm.rmm_uses_paired_launch(n, d_in, d_out, k, torch.bfloat16, SORS, binding.OP_FORWARD)
    assert rmm.rmm_uses_paired_launch(n, d_in, d_out, k, torch.bfloat16, SORS, binding.OP_BACKWARD)
    X, W, dY = synth.layer_inputs(n, d_in, d_out, "bf16", c["seeds"])
    Xd, Wd, dYd = X.to(DEV), W.to(DEV), dY.to(DEV)
    Y0, Xp0 = rmm.rmm_forward(Xd, Wd, None, k, SORS, 9, 1)
    dX0, dW0, _ = rmm.rmm_backward(dYd, Wd, Xp0, SORS, 9, 1)
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    Y1, Xp1 = rmm.rmm_forward(Xd, Wd, None, k, SORS, 9, 1, profile=(binding.STAGE_FWD_Y, a, b))
    dX1, dW1, _ = rmm.rmm_backward(dYd, Wd, Xp1, SORS, 9, 1, profile=(binding.STAGE_BWD_DX, a, b))
    torch.cuda.synchronize()
    assert torch.equal(Y0, Y1) and torch.equal(Xp0, Xp1) and torch.equal(dX0, dX1) and torch.equal(dW0, dW1)
    # a width with an odd number of strips: the last work-group of the pair has one live strip
    X2, W2, dY2 = synth.layer_inputs(4096, 776, 3080, "bf16", (7, 8, 9))
    if rmm.rmm_uses_paired_launch(4096, 776, 3080, 300, torch.bfloat16, SORS, binding.OP_FORWARD):
        check_layer(X2, W2, dY2, 300, SORS, 0xFEED, 3, "bf16", label="sors paired, odd strips")


@pytest.mark.parametrize("n,d_out,k", [(1, 8, 1), (100, 24, 40), (300, 40, 70), (700, 136, 64), (2000, 24, 2000), (4000, 16, 2050),
                                       (4097, 776, 300), (5000, 264, 2048), (5000, 24, 2050), (16384, 136, 100)])
def test_bias_gradient_from_the_strips(n, d_out, k):
    """Column sums of dY taken by the strip kernels (every chunk length, one and several chunks, two strips to a
    work-group), by the column-sum kernel where those do not serve, and once more on top of what is there."""
    d_in = 264
    X, W, dY = synth.layer_inputs(n, d_in, d_out, "bf16", (n, d_out, k))
    Xd, Wd, dYd = X.to(DEV), W.to(DEV), dY.to(DEV)
    _, Xp = rmm.rmm_forward(Xd, Wd, None, k, SORS, 3, 4)
    for need_dX in (True, False):
        _, dW, db = rmm.rmm_backward(dYd, Wd, Xp, SORS, 3, 4, need_dX=need_dX, need_dbias=True)
        want = synth.to_f64(dY).sum(axis=0)
        assert_close(db, want, "db", "bf16", label="sors db %s" % ((n, d_out, k),))
        first = synth.to_f64(db).copy()
        rmm.rmm_backward(dYd, Wd, Xp, SORS, 3, 4, need_dX=need_dX, dW=dW, dbias=db, need_dbias=True, accumulate=True)
        assert_close(db, want + first, "db", "bf16", label="sors db twice %s" % ((n, d_out, k),))


@pytest.mark.parametrize("n,d_in,d_out,k", [(4096, 768, 3072, 410),      # paired; by themselves the strips go two to a work-group
                                            (16384, 4096, 1024, 1638),   # paired, several rounds of tiles; alone one strip each
                                            (5000, 264, 2056, 90), (5000, 264, 520, 90),
                                            (4000, 264, 136, 2050), (700, 264, 136, 64), (300, 264, 40, 70)])
def test_bias_gradient_has_the_same_bits_in_every_form_of_the_pass(n, d_in, d_out, k):
    """With dX and without, in one launch with it or with an event pair for any stage.  Every column of dY sums to zero, so
    that db is nothing but the fp32 roundings of the order it was added in."""
    X, W, dY = synth.layer_inputs(n, d_in, d_out, "bf16", (n, d_out, k))
    gen = torch.Generator().manual_seed(n)
    dY *= torch.exp2(-torch.randint(0, 13, (n, 1), generator=gen).float()).to(dY.dtype)     # (exact)
    dY[n // 2:n // 2 * 2] = -dY[:n // 2][torch.randperm(n // 2, generator=gen)]
    dY[n // 2 * 2:] = 0
    Xd, Wd, dYd = X.to(DEV), W.to(DEV), dY.to(DEV)
    _, Xp = rmm.rmm_forward(Xd, Wd, None, k, SORS, 3, 4)
    dX, dW, db = rmm.rmm_backward(dYd, Wd, Xp, SORS, 3, 4, need_dbias=True)
    assert np.abs(synth.to_f64(db)).max() > 0
    _, dW1, db1 = rmm.rmm_backward(dYd, Wd, Xp, SORS, 3, 4, need_dX=False, need_dbias=True)
    assert torch.equal(db, db1) and torch.equal(dW, dW1), "without dX"
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    a.record(); b.record()
    for stage in (binding.STAGE_BWD_DX, binding.STAGE_BWD_G, binding.STAGE_BWD_DW, binding.STAGE_BWD_DBIAS,
                  binding.STAGE_BWD_G_PRODUCT, binding.STAGE_BWD_PAIR):
        dX1, dW1, db1 = rmm.rmm_backward(dYd, Wd, Xp, SORS, 3, 4, need_dbias=True, profile=(stage, a, b))
        assert torch.equal(dX, dX1) and torch.equal(dW, dW1) and torch.equal(db, db1), stage


# Strips that share compute units with 128 x 128 tiles, forward and backward: fewer tokens than a tile, transforms of 1024 and 2048, one
# chunk with more sketch columns than accumulators, several chunks, ragged edges, and where 256 x 256 tiles would be 160 or more.
COMPACT = [(8, 264, 264, 3), (300, 264, 264, 40), (500, 272, 304, 70), (1025, 264, 392, 100), (2000, 264, 392, 2100),
           (2275, 312, 584, 455), (4250, 1232, 864, 425), (10681, 1216, 840, 1068)]


@pytest.mark.parametrize("shape", COMPACT)
def test_strips_beside_tiles_on_a_compute_unit(shape):
    """Against the oracle, and bit for bit against launches of their own; Y also against that beside a dense sketch."""
    n, d_in, d_out, k = shape
    X, W, dY = synth.layer_inputs(n, d_in, d_out, "bf16", (n, d_in + 1, d_out + 2), w_std=1.0 / math.sqrt(d_in))
    bias = synth.to_torch(synth.normal((d_out,), 17), "bf16")
    check_layer(X, W, dY, k, SORS, 0x5EED0091, 15, "bf16", bias=bias, label="compact %s" % (shape,))
    Xd, Wd, dYd = (t.to(DEV) for t in (X, W, dY))
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    a.record(); b.record()
    torch.cuda.synchronize()
    Y0, Xp0 = rmm.rmm_forward(Xd, Wd, None, k, SORS, 9, 1)
    Y1, Xp1 = rmm.rmm_forward(Xd, Wd, None, k, SORS, 9, 1, profile=(binding.STAGE_FWD_Y, a, b))
    assert torch.equal(Y0, Y1) and torch.equal(Xp0, Xp1)
    for need_dbias in (False, True):
        one = rmm.rmm_backward(dYd, Wd, Xp0, SORS, 9, 1, need_dbias=need_dbias)
        two = rmm.rmm_backward(dYd, Wd, Xp0, SORS, 9, 1, need_dbias=need_dbias, profile=(binding.STAGE_BWD_DX, a, b))
        assert all(x is None and y is None or torch.equal(x, y) for x, y in zip(one, two)), need_dbias
    if k > 64:
        assert torch.equal(Y0, rmm.rmm_forward(Xd, Wd, None, k, rmm.RADEMACHER, 9, 1)[0])


@pytest.mark.parametrize("shape,forward,backward", [((4096, 512, 768, 410), True, True), ((2048, 768, 3072, 410), True, False),
                                                    ((4096, 768, 3072, 410), True, True), ((16384, 1024, 4096, 1638), True, False),
                                                    ((16384, 4096, 1024, 1638), False, True)])
def test_events_say_whether_a_pass_is_one_launch(shape, forward, backward):
    """In every form of the launch; with 1, rmm_uses_paired_launch says so too."""
    n, d_in, d_out, k = shape
    X, W, dY = (torch.zeros(s, device=DEV, dtype=torch.bfloat16) for s in ((n, d_in), (d_out, d_in), (n, d_out)))
    _, Xp = rmm.rmm_forward(X, W, None, k, SORS, 9, 1)

    def recorded(call, stage):
        a, b, made = (torch.cuda.Event(enable_timing=True) for _ in range(3))
        for e in (a, b, made):
            e.record()
        torch.cuda.synchronize()
        call((stage, a, b))
        torch.cuda.synchronize()
        return made.elapsed_time(a) > 0

    for call, stage, op, expected in ((lambda p: rmm.rmm_forward(X, W, None, k, SORS, 9, 1, profile=p), binding.STAGE_FWD_PAIR, binding.OP_FORWARD, forward),
                                      (lambda p: rmm.rmm_backward(dY, W, Xp, SORS, 9, 1, profile=p), binding.STAGE_BWD_PAIR, binding.OP_BACKWARD, backward)):
        assert recorded(call, stage) == expected, stage
        assert expected or not rmm.rmm_uses_paired_launch(n, d_in, d_out, k, torch.bfloat16, SORS, op)


@pytest.mark.parametrize("n", [1, 8, 300, 512])
def test_short_passes_have_the_same_bits_on_512_points_and_on_1024(n):
    """Strips beside tiles take 1024 points, those of a launch of their own, and column sums alone, 512."""
    d_in, d_out, k = 264, 520, max(1, n // 7)
    X, W, dY = synth.layer_inputs(n, d_in, d_out, "bf16", (n, d_in + 1, d_out + 2), w_std=1.0 / math.sqrt(d_in))
    check_layer(X, W, dY, k, SORS, 0x5EED0092, 15, "bf16", bias=synth.to_torch(synth.normal((d_out,), 17), "bf16"), label="short %d" % n)
    Xd, Wd, dYd = (t.to(DEV) for t in (X, W, dY))
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    a.record(); b.record()
    torch.cuda.synchronize()
    Xp = rmm.rmm_forward(Xd, Wd, None, k, SORS, 9, 1)[1]
    assert torch.equal(Xp, rmm.rmm_sketch(Xd, k, SORS, 9, 1))
    dX, dW, db = rmm.rmm_backward(dYd, Wd, Xp, SORS, 9, 1, need_dbias=True)
    for stage in (binding.STAGE_BWD_DX, binding.STAGE_BWD_DBIAS):
        dX1, dW1, db1 = rmm.rmm_backward(dYd, Wd, Xp, SORS, 9, 1, need_dbias=True, profile=(stage, a, b))
        assert torch.equal(dX, dX1) and torch.equal(dW, dW1) and torch.equal(db, db1), stage

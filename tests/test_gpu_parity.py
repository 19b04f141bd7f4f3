"""GPU parity: the HIP path, called through the C ABI, against the fp64 oracle on
identical seeded inputs.  Integer work (Philox words, Rademacher signs) must be
bit-exact; Y, X_proj, dX, dW must agree to a relative Frobenius error of 1e-5
(fp32) / 1e-2 (bf16) and entry by entry within the bound stated in tests/parity.py."""
import math

import numpy as np
import pytest
import torch

import paper_2201_13195_amd as rmm
from paper_2201_13195_amd import binding, synth
from oracle import philox as o_philox
from oracle import rmm as o_rmm
from oracle import sketch as o_sketch
from parity import assert_close, elementwise_excess

pytestmark = pytest.mark.gpu

TOL = {"f32": 1e-5, "bf16": 1e-2}
DEV = "cuda"


def rel_fro(got, want):
    got = synth.to_f64(got) if isinstance(got, torch.Tensor) else got
    return float(np.linalg.norm(got - want) / max(np.linalg.norm(want), 1e-300))


def run_layer(X, W, dY, k, kind, seed, offset, bias=None):
    """One forward + backward through the library; returns GPU tensors."""
    Xd, Wd, dYd = X.to(DEV), W.to(DEV), dY.to(DEV)
    bd = None if bias is None else bias.to(DEV)
    Y, Xp = rmm.rmm_forward(Xd, Wd, bd, k, kind, seed, offset)
    dX, dW, db = rmm.rmm_backward(dYd, Wd, Xp, kind, seed, offset, need_dbias=bias is not None)
    torch.cuda.synchronize()
    return Y, Xp, dX, dW, db


def check_layer(X, W, dY, k, kind, seed, offset, dtype, bias=None, label=""):
    Y, Xp, dX, dW, db = run_layer(X, W, dY, k, kind, seed, offset, bias)
    X64, W64, dY64 = synth.to_f64(X), synth.to_f64(W), synth.to_f64(dY)
    b64 = None if bias is None else synth.to_f64(bias)
    oY, oXp = o_rmm.forward(X64, W64, b64, k, kind, seed, offset)
    # the backward oracle gets the X_proj the device layer actually saved, as the real backward call does
    odX, odW, odb = o_rmm.backward(dY64, W64, synth.to_f64(Xp), kind, seed, offset)
    # ... and also the fully chained oracle value, which the saved X_proj must reproduce
    _, odW_chain, _ = o_rmm.backward(dY64, W64, oXp, kind, seed, offset)
    tol = TOL[dtype]
    errs = {"Y": rel_fro(Y, oY), "X_proj": rel_fro(Xp, oXp), "dX": rel_fro(dX, odX), "dW": rel_fro(dW, odW),
            "dW_chain": rel_fro(dW, odW_chain)}
    if bias is not None:
        errs["db"] = rel_fro(db, odb)
    print(label, {k_: "%.2e" % v for k_, v in errs.items()}, flush=True)
    for name, e in errs.items():
        assert e <= tol, (label, name, e)
    # entry by entry (a few wrong entries do not show in a norm)
    for name, got, want in (("Y", Y, oY), ("X_proj", Xp, oXp), ("dX", dX, odX), ("dW", dW, odW)) + \
            ((("db", db, odb),) if bias is not None else ()):
        assert_close(got, want, name, dtype, label)
    return errs


# ----------------------------------------------------------------------------- generator, bit-exact

def test_philox_words_bit_exact():
    cases = [(0, 0, 0, 0, 1000), (0x0123456789ABCDEF, (7 << 32) | 5, 12345, 77, 4099),
             (2 ** 64 - 1, 2 ** 64 - 1, 2 ** 32 - 3, 2 ** 32 - 1, 10)]      # last: c0 wraps past 2^32
    for seed, offset, c0, c1, ncalls in cases:
        got = rmm.rmm_debug_philox(seed, offset, c0, c1, ncalls).cpu().numpy().view(np.uint32)
        t = np.arange(ncalls, dtype=np.uint64)
        want = np.stack(o_philox.philox4x32_10((c0 + t) & 0xFFFFFFFF, c1, offset & 0xFFFFFFFF, offset >> 32,
                                               seed & 0xFFFFFFFF, seed >> 32), axis=1)
        assert np.array_equal(got, want)


def test_philox_known_answers_on_device():
    """Published vector: counter 0, key 0 -> 6627e8d5 e169c58d bc57ac4c 9b00dbd8."""
    got = rmm.rmm_debug_philox(0, 0, 0, 0, 1).cpu().numpy().view(np.uint32)[0]
    assert [hex(int(x)) for x in got] == ["0x6627e8d5", "0xe169c58d", "0xbc57ac4c", "0x9b00dbd8"]


@pytest.mark.parametrize("i0,j0,rows,cols", [(0, 0, 300, 7), (100, 3, 200, 65), (127, 1000, 3, 2), (4090, 0, 6, 410)])
def test_rademacher_signs_bit_exact(i0, j0, rows, cols):
    seed, offset = 0xFEEDFACE12345678, 3
    got = rmm.rmm_debug_sketch_tile(rmm.RADEMACHER, seed, offset, i0, j0, rows, cols).cpu().numpy()
    want = o_sketch.sketch_P(i0 + rows, j0 + cols, o_sketch.RADEMACHER, seed, offset)[i0:, j0:]
    assert np.array_equal(got.astype(np.float64), want)


@pytest.mark.parametrize("i0,j0,rows,cols", [(0, 0, 64, 16), (5, 9, 131, 33), (16380, 1630, 4, 8)])
def test_gaussian_tile_fp32(i0, j0, rows, cols):
    seed, offset = 0xFEEDFACE12345678, 1 << 33
    got = rmm.rmm_debug_sketch_tile(rmm.GAUSSIAN, seed, offset, i0, j0, rows, cols).cpu().numpy().astype(np.float64)
    want = o_sketch.sketch_P(i0 + rows, j0 + cols, o_sketch.GAUSSIAN, seed, offset)[i0:, j0:]
    assert np.abs(got - want).max() < 4e-6
    assert rel_fro(got, want) < 1e-6


def test_gaussian_entries_of_the_fp32_path_are_as_exact_as_library_functions():
    """Error against fp64 in units of the last place, over 2^22 entries (every radius and every angle many
    times).  sqrtf, logf and sincospif give 0.634 rms.  Largest: the factors are within 1.5 and 0.9 ulp, up to
    twice as much in ulps of their product, plus its rounding."""
    seed, offset, n, k = 0x5EED0051, 9, 4096, 1024
    got = rmm.rmm_debug_sketch_tile(rmm.GAUSSIAN, seed, offset, 0, 0, n, k).cpu().numpy().astype(np.float64)
    want = o_sketch.sketch_P(n, k, o_sketch.GAUSSIAN, seed, offset)
    ulp = np.exp2(np.floor(np.log2(np.maximum(np.abs(want), 2.0 ** -60))) - 23)
    some = np.abs(want) > 1e-6                # (at a quarter turn the oracle's own rounded angle gives 1e-16, not 0)
    err = np.abs(got - want)[some] / ulp[some]
    print("rms %.4f ulp, largest %.3f" % (np.sqrt(np.mean(err ** 2)), err.max()), flush=True)
    assert np.all(np.abs(got[~some]) < 1e-6)
    assert np.sqrt(np.mean(err ** 2)) <= 0.60 and err.max() <= 5.3


@pytest.mark.parametrize("kind", [rmm.GAUSSIAN, rmm.RADEMACHER])
@pytest.mark.parametrize("n,k", [(1024, 520), (1024, 200), (768, 600), (768, 100), (520, 130), (1032, 40), (1032, 17),
                                 (4096, 410), (2056, 1638), (392, 65)])
def test_bf16_generator_entry_by_entry_through_identity_operand(n, k, kind):
    """The sketch as the bf16 product kernels generate it (hardware log / sqrt / sin / cos, packed
    to bf16 inside the kernel; not the precise generator the debug hook exports): S^T I = S^T, so
    rmm_sketch on a bf16 identity returns every entry of S, each rounded to bf16 as P, scaled by
    1/sqrt(k) in fp32 and rounded once more.  Shapes reach every product kernel the library chooses
    between (operand widths >= 1024, multiples of 384, others; k <= 64, <= 512, larger), with
    several token slices and ragged edges.  Rademacher signs must be exact."""
    seed, offset = 0x5EED000A, (3 << 32) | 11
    A = torch.eye(n, dtype=torch.bfloat16, device=DEV)
    got = synth.to_f64(rmm.rmm_sketch(A, k, kind, seed, offset))          # k x n
    want = o_sketch.sketch_S(n, k, kind, seed, offset).T
    assert got.shape == want.shape
    if kind == rmm.RADEMACHER:
        assert np.array_equal(np.signbit(got), np.signbit(want))           # the bits, exactly
        assert np.abs(np.abs(got) * math.sqrt(k) - 1.0).max() <= 2.0 ** -8
    else:
        # two roundings to bf16 (at most 2^-8 relative each) plus the absolute error of the
        # hardware sin / cos near their zeros (below 1e-5 of a unit-variance entry)
        bound = 2.0 ** -7 * np.abs(want) + 1e-5 / math.sqrt(k)
        ratio = np.abs(got - want) / bound
        worst = np.unravel_index(int(np.argmax(ratio)), ratio.shape)
        assert ratio[worst] <= 1.0, (n, k, worst, got[worst], want[worst])


# ----------------------------------------------------------------------------- layer parity

def test_config1_fp32():
    c = synth.CONFIGS["c1_fp32_small"]
    X, W, dY = synth.config_inputs("c1_fp32_small")
    check_layer(X, W, dY, c["k"], rmm.GAUSSIAN, c["seed"], 0, "f32", label="c1")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("kind", [rmm.GAUSSIAN, rmm.RADEMACHER])
@pytest.mark.parametrize("shape", [(333, 200, 136, 77), (130, 72, 264, 129), (1, 8, 8, 1), (9, 16, 24, 40),
                                   (257, 101, 67, 19), (1000, 8, 520, 5)])
def test_small_and_ragged(dtype, kind, shape):
    """Several tiles plus ragged tails in every dimension; n not a multiple of the
    generator's block (8 / 128 tokens); k = 1; k > n; odd widths."""
    n, d_in, d_out, k = shape
    X, W, dY = synth.layer_inputs(n, d_in, d_out, dtype, (11, 12, 13), w_std=1.0 / math.sqrt(d_in))
    bias = synth.to_torch(synth.normal((d_out,), 14), dtype)
    check_layer(X, W, dY, k, kind, 0xABCDEF, 42, dtype, bias=bias, label="ragged %s %s %s" % (shape, dtype, kind))


@pytest.mark.parametrize("kind", [rmm.GAUSSIAN, rmm.RADEMACHER])
def test_large_tiles_ragged(kind):
    """Every output (Y, dX, dW) has at least 256 tiles of 256 x 256, the point where the
    library switches to its large tile, and every dimension leaves a ragged tail there."""
    n, d_in, d_out, k = 4100, 3848, 3848, 100
    X, W, dY = synth.layer_inputs(n, d_in, d_out, "bf16", (21, 22, 23), w_std=1.0 / math.sqrt(d_in))
    bias = synth.to_torch(synth.normal((d_out,), 24), "bf16")
    check_layer(X, W, dY, k, kind, 0x5EED, 7, "bf16", bias=bias, label="large ragged kind=%d" % kind)


@pytest.mark.parametrize("kind", [rmm.GAUSSIAN, rmm.RADEMACHER])
def test_long_contractions_few_tiles(kind):
    """Few output tiles and contractions of more than 1536 in all three products (d_in for Y,
    d_out for dX, k for dW; k > n): the shapes where two wave groups split the contraction
    of a tile.  Every dimension is ragged."""
    n, d_in, d_out, k = 300, 1544, 1608, 1550
    X, W, dY = synth.layer_inputs(n, d_in, d_out, "bf16", (41, 42, 43), w_std=1.0 / math.sqrt(d_in))
    bias = synth.to_torch(synth.normal((d_out,), 44), "bf16")
    check_layer(X, W, dY, k, kind, 0xC0FFEE, 3, "bf16", bias=bias, label="long contraction kind=%d" % kind)


def test_config2_base_attention():
    c = synth.CONFIGS["c2_base_attn"]
    X, W, dY = synth.config_inputs("c2_base_attn")
    check_layer(X, W, dY, c["k"], rmm.GAUSSIAN, c["seed"], 0, "bf16", label="c2")


@pytest.mark.parametrize("kind", [rmm.GAUSSIAN, rmm.RADEMACHER])
@pytest.mark.parametrize("rho", [0.1, 0.2, 0.5, 0.9])
@pytest.mark.parametrize("name,offset", [("c3_base_ffn_up", 0), ("c3_base_ffn_down", 1)])
def test_config3_base_ffn_sweep(name, offset, rho, kind):
    c = synth.CONFIGS[name]
    k = synth.sketch_size(rho, c["n"])
    assert k in (410, 819, 2048, 3686)
    X, W, dY = synth.config_inputs(name)
    check_layer(X, W, dY, k, kind, c["seed"], offset, "bf16", label="%s rho=%s kind=%d" % (name, rho, kind))


@pytest.mark.parametrize("name,offset", [("c4_large_attn", 0), ("c4_large_ffn_up", 1), ("c4_large_ffn_down", 2)])
def test_config4_large(name, offset):
    c = synth.CONFIGS[name]
    assert c["k"] == synth.sketch_size(0.1, c["n"]) == 1638
    X, W, dY = synth.config_inputs(name)
    check_layer(X, W, dY, c["k"], rmm.GAUSSIAN, c["seed"], offset, "bf16", label=name)


@pytest.mark.parametrize("kind", [rmm.GAUSSIAN, rmm.RADEMACHER])
@pytest.mark.parametrize("n,d,k", [(4100, 520, 24), (4100, 520, 64), (700, 264, 33), (16384, 4096, 32)])
def test_sketch_primitive_small_k(n, d, k, kind):
    """rmm_sketch alone (Eq. 4) in the regime bound by one pass over A (k <= 64), several token
    slices, ragged tails; the last case is the shape the HBM roofline is quoted on."""
    A = synth.to_torch(synth.normal((n, d), 31), "bf16")
    got = rmm.rmm_sketch(A.to(DEV), k, kind, 0x5EED0006, 9)
    torch.cuda.synchronize()
    want = o_rmm.sketch_apply(synth.to_f64(A), k, kind, 0x5EED0006, 9)
    err = assert_close(got, want, "X_proj", "bf16", "sketch n=%d d=%d k=%d kind=%d" % (n, d, k, kind))
    print("sketch n=%d d=%d k=%d kind=%d: %.2e" % (n, d, k, kind, err), flush=True)


@pytest.mark.parametrize("kind", [rmm.GAUSSIAN, rmm.RADEMACHER])
def test_sketch_primitive_large_k(kind):
    A = synth.to_torch(synth.normal((3000, 392), 32), "bf16")
    got = rmm.rmm_sketch(A.to(DEV), 300, kind, 0x5EED0007, 2)
    torch.cuda.synchronize()
    want = o_rmm.sketch_apply(synth.to_f64(A), 300, kind, 0x5EED0007, 2)
    assert_close(got, want, "X_proj", "bf16", "sketch large k kind=%d" % kind)


# ----------------------------------------------------------------------------- contracts of the boundary

def test_forward_and_sketch_agree_and_are_deterministic():
    X, W, dY = synth.layer_inputs(700, 256, 128, "bf16", (21, 22, 23))
    Xd, Wd, dYd = X.to(DEV), W.to(DEV), dY.to(DEV)
    for kind in (rmm.GAUSSIAN, rmm.RADEMACHER):
        Y1, Xp1 = rmm.rmm_forward(Xd, Wd, None, 96, kind, 5, 6)
        Y2, Xp2 = rmm.rmm_forward(Xd, Wd, None, 96, kind, 5, 6)
        Xp3 = rmm.rmm_sketch(Xd, 96, kind, 5, 6)
        assert torch.equal(Y1, Y2) and torch.equal(Xp1, Xp2) and torch.equal(Xp1, Xp3)
        d1 = rmm.rmm_backward(dYd, Wd, Xp1, kind, 5, 6)
        d2 = rmm.rmm_backward(dYd, Wd, Xp1, kind, 5, 6)
        assert torch.equal(d1[0], d2[0]) and torch.equal(d1[1], d2[1])
        # another offset / seed is another sketch
        assert not torch.equal(Xp1, rmm.rmm_sketch(Xd, 96, kind, 5, 7))
        assert not torch.equal(Xp1, rmm.rmm_sketch(Xd, 96, kind, 4, 6))
        # dX can be skipped
        dX, dW, _ = rmm.rmm_backward(dYd, Wd, Xp1, kind, 5, 6, need_dX=False)
        assert dX is None and torch.equal(dW, d1[1])


def test_saved_bytes_ratio_is_k_over_n():
    """Section 2.4.1: what the layer keeps is X_proj (k x d_in) + 16 bytes."""
    for name in ("c2_base_attn", "c4_large_ffn_down"):
        c = synth.CONFIGS[name]
        Xp = torch.empty((c["k"], c["d_in"]), dtype=torch.bfloat16, device=DEV)
        x_bytes = c["n"] * c["d_in"] * 2
        assert Xp.numel() * Xp.element_size() * c["n"] == x_bytes * c["k"]
        saved, plain = o_rmm.saved_bytes(c["n"], c["d_in"], c["k"], 2)
        assert saved == Xp.numel() * 2 + 16 and plain == x_bytes


def test_workspace_too_small_is_reported():
    X, W, dY = synth.layer_inputs(64, 32, 32, "f32", (1, 2, 3))
    Xd, Wd, dYd = X.to(DEV), W.to(DEV), dY.to(DEV)
    _, Xp = rmm.rmm_forward(Xd, Wd, None, 8, rmm.GAUSSIAN, 0, 0)
    small = torch.empty(16, dtype=torch.uint8, device=DEV)
    with pytest.raises(rmm.RmmError) as e:
        rmm.rmm_backward(dYd, Wd, Xp, rmm.GAUSSIAN, 0, 0, ws=small)
    assert e.value.status == -3


def test_profiled_entry_points_time_one_stage_and_change_nothing():
    """The profiled variants record the caller's events around exactly one stage and
    compute what the plain entry points compute."""
    X, W, dY = synth.layer_inputs(2048, 512, 768, "bf16", (31, 32, 33))
    Xd, Wd, dYd = X.to(DEV), W.to(DEV), dY.to(DEV)
    k, kind = 205, rmm.GAUSSIAN
    Y0, Xp0 = rmm.rmm_forward(Xd, Wd, None, k, kind, 9, 1)
    dX0, dW0, _ = rmm.rmm_backward(dYd, Wd, Xp0, kind, 9, 1)
    ms = {}
    for stage in range(8):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record(); b.record()
        torch.cuda.synchronize()
        Y1, Xp1 = rmm.rmm_forward(Xd, Wd, None, k, kind, 9, 1, profile=(stage, a, b))
        dX1, dW1, _ = rmm.rmm_backward(dYd, Wd, Xp1, kind, 9, 1, profile=(stage, a, b))
        torch.cuda.synchronize()
        ms[stage] = a.elapsed_time(b)
        assert torch.equal(Y0, Y1) and torch.equal(Xp0, Xp1) and torch.equal(dX0, dX1) and torch.equal(dW0, dW1)
    print("stage ms", ms, flush=True)
    for stage in (0, 1, 2, 3, 4, 6, 7):
        assert 0.0 < ms[stage] < 50.0, (stage, ms)
    # a product kernel is part of its stage
    assert ms[6] <= ms[1] * 1.5 + 0.02 and ms[7] <= ms[3] * 1.5 + 0.02
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    a.record(); b.record()
    torch.cuda.synchronize()
    Xp2 = rmm.rmm_sketch(Xd, k, kind, 9, 1, events=(a, b))
    torch.cuda.synchronize()
    assert torch.equal(Xp2, Xp0) and 0.0 < a.elapsed_time(b) < 50.0


@pytest.mark.parametrize("dtype,shape", [("f32", (333, 200, 136, 77)), ("bf16", (333, 200, 136, 77)),
                                         ("bf16", (700, 264, 520, 96)), ("bf16", (300, 1544, 1608, 1550))])
def test_backward_accumulate_over_two_micro_batches(dtype, shape):
    """Gradient accumulation: the second micro-batch's backward adds its dW and dbias to the
    first one's (plain sum of two Algorithm 1 backward results), dX is overwritten."""
    n, d_in, d_out, k = shape
    kind = rmm.GAUSSIAN
    X1, W, dY1 = synth.layer_inputs(n, d_in, d_out, dtype, (71, 72, 73), w_std=1.0 / math.sqrt(d_in))
    X2, _, dY2 = synth.layer_inputs(n, d_in, d_out, dtype, (74, 72, 75), w_std=1.0 / math.sqrt(d_in))
    Wd = W.to(DEV)
    _, Xp1 = rmm.rmm_forward(X1.to(DEV), Wd, None, k, kind, 9, 100)
    _, Xp2 = rmm.rmm_forward(X2.to(DEV), Wd, None, k, kind, 9, 101)
    dX1, dW, db = rmm.rmm_backward(dY1.to(DEV), Wd, Xp1, kind, 9, 100, need_dbias=True)
    dW_first, db_first = synth.to_f64(dW), synth.to_f64(db)
    dX2, dW_b, db_b = rmm.rmm_backward(dY2.to(DEV), Wd, Xp2, kind, 9, 101, need_dbias=True, dW=dW, dbias=db,
                                       accumulate=True)
    assert dW_b is dW and db_b is db
    W64 = synth.to_f64(W)
    odX1, odW1, odb1 = o_rmm.backward(synth.to_f64(dY1), W64, synth.to_f64(Xp1), kind, 9, 100)
    odX2, odW2, odb2 = o_rmm.backward(synth.to_f64(dY2), W64, synth.to_f64(Xp2), kind, 9, 101)
    tol = TOL[dtype]
    errs = {"dW_sum": rel_fro(dW, odW1 + odW2), "dW_step": rel_fro(dW, dW_first + odW2),
            "db_sum": rel_fro(db, odb1 + odb2), "db_step": rel_fro(db, db_first + odb2),
            "dX1": rel_fro(dX1, odX1), "dX2": rel_fro(dX2, odX2)}
    print(shape, dtype, {k_: "%.2e" % v for k_, v in errs.items()}, flush=True)
    for name, e in errs.items():
        assert e <= tol, (name, e)
    # the accumulated result is not just the second estimate
    assert rel_fro(dW, odW2) > 0.3


@pytest.mark.parametrize("dtype,n,d_out", [("bf16", 4096, 3072), ("bf16", 16384, 1024), ("bf16", 16384, 4096),
                                           ("bf16", 5000, 3080), ("bf16", 777, 264), ("bf16", 300, 67),
                                           ("f32", 4096, 1536), ("f32", 1000, 132), ("f32", 300, 50)])
def test_bias_gradient_at_paper_sizes(dtype, n, d_out):
    """db = dY^T 1 (Eq. 3) against column sums in fp64, on the layer's real dY sizes and on ragged
    ones: wide matrices (four 16-byte pieces of a row per work-group), narrow ones (one piece),
    widths that are no multiple of 16 bytes (element-wise kernel); then once more accumulated
    on top of itself.  The other products of the call are kept tiny (d_in = 8, k = 8)."""
    d_in, k = 8, 8
    g = torch.Generator(device="cpu")
    g.manual_seed(1234 + n + d_out)
    tdtype = torch.bfloat16 if dtype == "bf16" else torch.float32
    dY = torch.randn((n, d_out), generator=g).to(tdtype).to(DEV)
    W = torch.randn((d_out, d_in), generator=g).to(tdtype).to(DEV)
    X_proj = torch.randn((k, d_in), generator=g).to(tdtype).to(DEV)
    _, dW, db = rmm.rmm_backward(dY, W, X_proj, rmm.RADEMACHER, 5, 6, need_dX=False, need_dbias=True)
    want = synth.to_f64(dY).sum(axis=0)
    assert_close(db, want, "db", dtype, label="db %s %dx%d" % (dtype, n, d_out))
    first = synth.to_f64(db).copy()  # the accumulated value starts from the stored (rounded) one
    rmm.rmm_backward(dY, W, X_proj, rmm.RADEMACHER, 5, 6, need_dX=False, dW=dW, dbias=db, need_dbias=True, accumulate=True)
    assert_close(db, want + first, "db", dtype, label="db accumulate")


@pytest.mark.parametrize("kind", [rmm.GAUSSIAN, rmm.RADEMACHER])
@pytest.mark.parametrize("name,k_override", [("c2_base_attn", 0), ("c3_base_ffn_up", 0), ("c3_base_ffn_down", 0),
                                             ("c4_large_ffn_up", 0), ("c3_base_ffn_up", 3686), ("c3_base_ffn_down", 3686)])
def test_paired_launch_gives_the_bits_of_the_separate_launches(name, k_override, kind):
    """At these shapes a pass runs its plain product and its sketch product as one launch; asking
    for a single product's stage makes it launch them one after the other, with the same token
    slices.  Same tiles, same order of additions: every output must agree bit for bit.  At
    k = 3686 the sketch product of the 3072-wide operand is unsliced: alone it writes bf16
    directly, in the paired launch it goes through a single fp32 slice."""
    c = synth.CONFIGS[name]
    n, d_in, d_out, k = c["n"], c["d_in"], c["d_out"], k_override or c["k"]
    assert rmm.rmm_uses_paired_launch(n, d_in, d_out, k, torch.bfloat16, kind, binding.OP_FORWARD)
    assert rmm.rmm_uses_paired_launch(n, d_in, d_out, k, torch.bfloat16, kind, binding.OP_BACKWARD)
    X, W, dY = synth.layer_inputs(n, d_in, d_out, "bf16", c["seeds"])
    Xd, Wd, dYd = X.to(DEV), W.to(DEV), dY.to(DEV)
    Y0, Xp0 = rmm.rmm_forward(Xd, Wd, None, k, kind, 9, 1)
    dX0, dW0, _ = rmm.rmm_backward(dYd, Wd, Xp0, kind, 9, 1)
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    a.record(); b.record()
    torch.cuda.synchronize()
    Y1, Xp1 = rmm.rmm_forward(Xd, Wd, None, k, kind, 9, 1, profile=(binding.STAGE_FWD_Y, a, b))
    dX1, dW1, _ = rmm.rmm_backward(dYd, Wd, Xp1, kind, 9, 1, profile=(binding.STAGE_BWD_DX, a, b))
    torch.cuda.synchronize()
    assert torch.equal(Y0, Y1) and torch.equal(Xp0, Xp1) and torch.equal(dX0, dX1) and torch.equal(dW0, dW1)


@pytest.mark.parametrize("shape", [(4096, 768, 3072, 410), (4096, 3072, 768, 410), (2000, 264, 520, 100), (300, 1544, 1608, 1550),
                                   (16384, 1024, 4096, 1638), (16384, 4096, 1024, 1638), (16384, 1024, 1024, 1638)])
def test_weight_and_bias_gradient_in_one_launch_give_the_bits_of_two(shape):
    """With a bias gradient the backward pass takes the column sums of dY in the launch of dW or,
    where dW fills the chip (the last three shapes), in the paired launch of dX and the sketch
    product; asking for the dW stage's events makes it use the kernel of their own.  Same tiles,
    same order of additions."""
    n, d_in, d_out, k = shape
    X, W, dY = synth.layer_inputs(n, d_in, d_out, "bf16", (61, 62, 63))
    Xd, Wd, dYd = X.to(DEV), W.to(DEV), dY.to(DEV)
    _, Xp = rmm.rmm_forward(Xd, Wd, None, k, rmm.GAUSSIAN, 3, 4)
    dX0, dW0, db0 = rmm.rmm_backward(dYd, Wd, Xp, rmm.GAUSSIAN, 3, 4, need_dbias=True)
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    a.record(); b.record()
    torch.cuda.synchronize()
    dX1, dW1, db1 = rmm.rmm_backward(dYd, Wd, Xp, rmm.GAUSSIAN, 3, 4, need_dbias=True, profile=(binding.STAGE_BWD_DW, a, b))
    torch.cuda.synchronize()
    assert torch.equal(dX0, dX1) and torch.equal(dW0, dW1) and torch.equal(db0, db1)
    assert_close(db0, synth.to_f64(dY).sum(axis=0), "db", "bf16", label="db fused %s" % (shape,))
    # accumulated on top of itself, again both ways
    dWa, dba = dW0.clone(), db0.clone()
    rmm.rmm_backward(dYd, Wd, Xp, rmm.GAUSSIAN, 3, 4, dW=dWa, dbias=dba, need_dbias=True, accumulate=True)
    assert_close(dba, synth.to_f64(dY).sum(axis=0) + synth.to_f64(db0), "db", "bf16", label="db fused accumulate")
    assert_close(dWa, 2.0 * synth.to_f64(dW0), "dW", "bf16", label="dW fused accumulate")

"""GPU: the fp32 products over the whole range of fp32: infinities, NaN, the largest numbers and the
smallest, in every operand, against the same products with fp64 multiply-adds."""
import math

import numpy as np
import pytest
import torch

import paper_2201_13195_amd as rmm
from paper_2201_13195_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda"
U, TINY = 2.0 ** -24, 2.0 ** -149
BIG = float(np.finfo(np.float32).max)

# 32 x 32, 64 x 64 and 128 x 128 tiles, rows on 16 bytes and not, rows beyond 32-bit offsets
SHAPES = [(40, 36, 44), (500, 129, 127), (1030, 260, 1004), (2050, 257, 2051)]
LONG = (3, (1 << 22) + 5, 5)


def products(dtype, n, d_in, d_out, X, W, k, kind):
    """(device result, left operand, right operand) of Y = X W^T and X_proj = S^T X."""
    Xd, Wd = torch.from_numpy(X).to(DEV).to(dtype), torch.from_numpy(W).to(DEV).to(dtype)
    Y, Xp = rmm.rmm_forward(Xd, Wd, None, k, kind, 0x5EED0041, 3)
    S = rmm.rmm_debug_sketch_tile(kind, 0x5EED0041, 3, 0, 0, n, k).cpu().numpy()      # (entries of S sqrt(k))
    return [(synth.to_f64(Y), X, W.T, 1.0), (synth.to_f64(Xp), S.T, X, 1.0 / math.sqrt(k))]


def check(got, A, B, alpha, u=U):
    """Every entry against fp64: NaN and infinities where they belong, else within the roundings of an
    fp32 accumulation of K terms (a product below fp32's smallest number is lost)."""
    A, B = A.astype(np.float64), B.astype(np.float64)
    with np.errstate(all="ignore"):
        want, size = alpha * (A @ B), alpha * (np.abs(A) @ np.abs(B))
        assert np.array_equal(np.isnan(got), np.isnan(want))
        inf = np.isinf(want)
        assert np.array_equal(got[inf], want[inf])
        ok = np.isfinite(want)
        bound = u * (2.0 + math.sqrt(A.shape[1])) * size[ok] + A.shape[1] * TINY
        assert np.all(np.abs(got[ok] - want[ok]) <= bound), np.nanmax(np.abs(got[ok] - want[ok]) / bound)


@pytest.mark.parametrize("kind", [rmm.GAUSSIAN, rmm.RADEMACHER])
@pytest.mark.parametrize("shape", SHAPES)
def test_infinities_nan_and_the_largest_numbers(shape, kind):
    n, d_in, d_out = shape
    g = np.random.default_rng(7)
    X = g.standard_normal((n, d_in)).astype(np.float32)
    W = (g.standard_normal((d_out, d_in)) / math.sqrt(d_in)).astype(np.float32)
    W[0, 5] = 0.0                                   # (infinity times zero is NaN)
    for row, col, value in ((0, 5, np.inf), (1, 6, -np.inf), (n // 2, 7, -BIG / 16), (n - 1, 8, BIG / 16), (n - 2, 9, np.nan),
                            (n - 3, d_in - 1, 1e30)):
        X[row, col] = value
    for got, A, B, alpha in products(torch.float32, n, d_in, d_out, X, W, 33, kind):
        check(got, A, B, alpha)
    X[:] = 0                                        # one product to a sum: the largest numbers themselves
    X[3, 4], X[4, 5], W[:, 4], W[:, 5] = BIG, -BIG, 1.0, 1.0
    for got, A, B, alpha in products(torch.float32, n, d_in, d_out, X, W, 1, rmm.RADEMACHER):
        check(got, A, B, alpha)


@pytest.mark.parametrize("kind", [rmm.GAUSSIAN, rmm.RADEMACHER])
@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("ex,ew", [(-125, 0), (-125, 100), (-145, 120), (0, -140), (-60, -70), (-75, -75)])
def test_the_smallest_numbers(shape, kind, ex, ew):
    """Operands down to fp32's smallest, also where their products are large, and products that underflow."""
    n, d_in, d_out = shape
    g = np.random.default_rng(8)
    X = np.ldexp(g.standard_normal((n, d_in)), ex).astype(np.float32)
    W = np.ldexp(g.standard_normal((d_out, d_in)), ew).astype(np.float32)
    for got, A, B, alpha in products(torch.float32, n, d_in, d_out, X, W, 33, kind):
        check(got, A, B, alpha)


def test_long_rows_with_infinities():
    n, d_in, d_out = LONG
    X, W = np.zeros((n, d_in), np.float32), np.zeros((d_out, d_in), np.float32)
    X[0, 7], X[1, d_in - 1], X[2, 9], W[:, 7], W[:, d_in - 1], W[:, 9] = np.inf, -1e-42, BIG, 1.0, 2.0, -0.5
    Y, _ = rmm.rmm_forward(torch.from_numpy(X).to(DEV), torch.from_numpy(W).to(DEV), None, 1, 0, 1, 2, need_xproj=False)
    check(synth.to_f64(Y), X, W.T, 1.0)


@pytest.mark.parametrize("accumulate", [False, True])
def test_infinities_in_the_backward_pass(accumulate):
    """dX, dW (with the old value added, or not) and db with an infinite and a NaN gradient."""
    n, d_in, d_out, k, kind = 300, 132, 140, 37, rmm.RADEMACHER
    g = np.random.default_rng(9)
    dY, W, Xp = (g.standard_normal(s).astype(np.float32) for s in ((n, d_out), (d_out, d_in), (k, d_in)))
    dY[3, 4], dY[5, 6], Xp[2, 7] = np.inf, np.nan, -np.inf
    dev = [torch.from_numpy(a).to(DEV) for a in (dY, W, Xp)]
    old = torch.from_numpy(g.standard_normal((d_out, d_in)).astype(np.float32)).to(DEV) if accumulate else None
    old_b = torch.ones(d_out, device=DEV) if accumulate else None
    want_old = 0.0 if old is None else synth.to_f64(old)
    dX, dW, db = rmm.rmm_backward(*dev, kind, 0x5EED0042, 1, need_dbias=True, dW=old, dbias=old_b, accumulate=accumulate)
    G = rmm.rmm_sketch(dev[0], k, kind, 0x5EED0042, 1).cpu().numpy()
    check(synth.to_f64(dX), dY, W, 1.0)
    with np.errstate(all="ignore"):
        want = G.astype(np.float64).T @ Xp.astype(np.float64) + want_old
        got = synth.to_f64(dW)
        assert np.array_equal(np.isnan(got), np.isnan(want)) and np.array_equal(got[np.isinf(want)], want[np.isinf(want)])
        ok = np.isfinite(want)
        assert np.allclose(got[ok], want[ok], rtol=1e-5, atol=1e-4)
        sums = dY.astype(np.float64).sum(0) + (1.0 if accumulate else 0.0)
    assert np.allclose(synth.to_f64(db), sums, rtol=1e-5, atol=1e-4, equal_nan=True)


def test_bf16_odd_width_gaussian_sketch_of_infinities():
    """The sketch entries are split too: an infinite bf16 activation gives infinities of the entries' signs."""
    n, d_in, d_out, k = 200, 71, 33, 40
    g = np.random.default_rng(10)
    X = torch.from_numpy(g.standard_normal((n, d_in)).astype(np.float32)).bfloat16()
    X[3, 4], X[5, 6] = math.inf, math.nan
    W = torch.ones(d_out, d_in, dtype=torch.bfloat16)
    for got, A, B, alpha in products(torch.bfloat16, n, d_in, d_out, X.float().numpy(), W.float().numpy(), k, rmm.GAUSSIAN)[1:]:
        check(got, A, B, alpha, u=2.0 ** -8)

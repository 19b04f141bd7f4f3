"""GPU: the variance monitors of Section 2.3 (rmm_variance_stats, through the C ABI) against the
fp64 oracle's closed forms and against the paper's worked example."""
import os

import numpy as np
import pytest
import torch

import paper_2201_13195_amd as rmm
from paper_2201_13195_amd import synth
from oracle import variance as o_var

pytestmark = pytest.mark.gpu
DEV = "cuda"
# Inputs are exact in both paths; the device sums products in fp32 inside a tile / a row and in
# fp64 across tiles / rows, the oracle in fp64 throughout: a few 1e-6 relative.
TOL = 2e-5


def oracle_stats(X, dY, k, kind):
    X64, Y64 = synth.to_f64(X), synth.to_f64(dY)
    rows = float(np.sum(np.sum(X64 * X64, axis=1) * np.sum(Y64 * Y64, axis=1)))
    d2_rmm = o_var.rmm_variance_gaussian(X64, Y64, k) if kind == rmm.GAUSSIAN else o_var.rmm_variance_rademacher(X64, Y64, k)
    return dict(x_fro2=float(np.sum(X64 * X64)), y_fro2=float(np.sum(Y64 * Y64)), rows=rows,
                xty_fro2=float(np.sum((X64.T @ Y64) ** 2)), d2_sgd=o_var.d2_sgd(X64, Y64), d2_rmm=d2_rmm,
                alpha=o_var.alpha(X64, Y64), d2_rmm_printed=o_var.d2_rmm_printed(X64, Y64, k))


def check(X, dY, k, kind, label):
    got = rmm.rmm_variance_stats(X.to(DEV), dY.to(DEV), k, kind).cpu().numpy()
    want = oracle_stats(X, dY, k, kind)
    errs = {}
    for i, name in enumerate(rmm.VARIANCE_FIELDS):
        scale = abs(want[name]) if name != "d2_rmm_printed" else abs(want["d2_rmm"])   # a difference of large terms
        errs[name] = abs(got[i] - want[name]) / max(scale, 1e-300)
    print(label, {n_: "%.1e" % e for n_, e in errs.items()}, flush=True)
    for name, e in errs.items():
        assert e <= TOL, (label, name, e, want[name])
    return got


@pytest.mark.parametrize("kind", [rmm.GAUSSIAN, rmm.RADEMACHER])
@pytest.mark.parametrize("dtype,shape", [("f32", (256, 128, 128, 32)), ("f32", (333, 77, 50, 19)),
                                         ("bf16", (333, 200, 136, 77)), ("bf16", (130, 67, 101, 9)),
                                         ("bf16", (4096, 768, 768, 410)), ("bf16", (4096, 768, 3072, 410)),
                                         ("bf16", (2100, 520, 264, 100))])
def test_variance_stats_match_closed_forms(dtype, shape, kind):
    n, d_in, d_out, k = shape
    X, _, dY = synth.layer_inputs(n, d_in, d_out, dtype, (81, 82, 83))
    check(X, dY, k, kind, "variance %s %s kind=%d" % (shape, dtype, kind))


def test_variance_stats_on_correlated_inputs_and_large_tiles():
    """dY correlated with X makes |X^T dY|^2 dominate (alpha far from 0); 4104 x 4104 outputs go
    through the large-tile kernel, ragged in every dimension."""
    n, d = 2056, 4104
    X = synth.to_torch(synth.normal((n, d), 91), "bf16")
    dY = synth.to_torch(synth.to_f64(X) * 0.5 + synth.normal((n, d), 92) * 0.1, "bf16")
    got = check(X, dY, 205, rmm.GAUSSIAN, "variance correlated")
    assert got[6] > 1.3 / n      # independent X, dY would give about 1/n


# (n, d_in, d_out) of each tile that X^T dY runs with, ragged in every dimension (test_launch_plans.py: they are taken)
TILES = [((201, 200, 136), "64x64"), ((201, 1800, 520), "64x128"), ((197, 2504, 776), "128x128"), ((1101, 2312, 776), "128x128 split"),
         ((261, 2552, 1528), "128x128 compact"), ((203, 1672, 2312), "128x256"), ((71, 4104, 4104), "256x256")]


@pytest.mark.parametrize("shape,tile", TILES)
def test_variance_stats_on_every_tile(shape, tile):
    n, d_in, d_out = shape
    X, _, dY = synth.layer_inputs(n, d_in, d_out, "bf16", (87, 88, 89))
    check(X, dY, 30, rmm.RADEMACHER, "variance %s" % tile)


def test_worked_example_of_the_paper(golden_dir):
    """Section 2.3, B = 2: (B-1) D2_SGD = 4 and B_proj D2_RMM = 2 + eps^2 + eps^-2 (X^T Y = 0)."""
    with open(os.path.join(golden_dir, "worked_example_b2.txt")) as f:
        rows = [[float(t) for t in line.split()] for line in f if line.strip() and not line.startswith("#")]
    for eps, sgd, rmm_val in rows:
        X = torch.tensor([[1.0, 0.0], [-eps, 0.0]], dtype=torch.float32)
        Y = torch.tensor([[1.0, 0.0], [1.0 / eps, 0.0]], dtype=torch.float32)
        for kproj in (1, 3, 10):
            got = rmm.rmm_variance_stats(X.to(DEV), Y.to(DEV), kproj, rmm.GAUSSIAN).cpu().numpy()
            assert abs(got[4] - sgd) <= 1e-5 * sgd
            assert abs(kproj * got[5] - rmm_val) <= 1e-5 * rmm_val and abs(kproj * got[7] - rmm_val) <= 1e-5 * rmm_val
            assert abs(got[6]) < 1e-6


def test_variance_stats_are_reproducible_and_check_workspace():
    X, _, dY = synth.layer_inputs(1000, 264, 520, "bf16", (84, 85, 86))
    a = rmm.rmm_variance_stats(X.to(DEV), dY.to(DEV), 100, rmm.RADEMACHER)
    b = rmm.rmm_variance_stats(X.to(DEV), dY.to(DEV), 100, rmm.RADEMACHER)
    assert torch.equal(a, b)
    with pytest.raises(rmm.RmmError) as e:
        rmm.rmm_variance_stats(X.to(DEV), dY.to(DEV), 100, rmm.RADEMACHER, ws=torch.empty(16, dtype=torch.uint8, device=DEV))
    assert e.value.status == -3


def test_hand_cases_with_nonzero_cross_term(golden_dir):
    """Lemma 2.1 and alpha of Theorem 2.3 on the hand-evaluated integer inputs of
    tests/golden/variance_hand_cases.txt (X^T Y != 0), against the literals."""
    n_cases = 0
    with open(os.path.join(golden_dir, "variance_hand_cases.txt")) as f:
        for line in f:
            if not line.strip() or line.startswith("#"):
                continue
            t = [float(v) for v in line.split()]
            B, N, M = int(t[0]), int(t[1]), int(t[2])
            X = torch.tensor(t[3:3 + B * N], dtype=torch.float32).reshape(B, N)
            Y = torch.tensor(t[3 + B * N:3 + B * N + B * M], dtype=torch.float32).reshape(B, M)
            for dtype in (torch.float32, torch.bfloat16):       # small integers are exact in both
                got = rmm.rmm_variance_stats(X.to(DEV).to(dtype), Y.to(DEV).to(dtype), 3, rmm.GAUSSIAN).cpu().numpy()
                assert abs(got[4] - t[-2]) <= 1e-6 * max(1.0, abs(t[-2])), (line, got[4])
                assert abs(got[6] - t[-1]) <= 1e-6, (line, got[6])
            n_cases += 1
    assert n_cases >= 4

"""Float32 product on the matrix cores (kmvm_split.hip) against the float64 oracle.

Bound per output: 2e-6 * sum_j |k_ij v_jc|.  A term's relative error is at most
about (1.5 |log2 k| ln 2 + 2) 2^-24 (roundings of r^2, of the exponent argument
and of the exponential), 1e-6 for every entry above e^-10; a float32 chain
of m steps adds about sqrt(m) 2^-25 of its largest partial sum, below 1e-6 for
the chains here (6 n2 / (32 splits) steps).
"""

import numpy as np
import pytest
import torch

from oracle import kmvm as okmvm
from paper_2207_06856_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda"


def check(lib, X1, X2, V, kind, ls, noise, add_noise, rows=None):
    t1 = torch.from_numpy(X1).to(DEV)
    t2 = t1 if X2 is X1 else torch.from_numpy(X2).to(DEV)
    out = lib.kmvm(t1, t2, torch.from_numpy(V).to(DEV), kind, ls, 1.25, noise, add_noise=add_noise,
                   precision=lib.FP32).cpu().numpy()
    rows = np.arange(0, X1.shape[0], max(1, X1.shape[0] // 400)) if rows is None else rows
    ref = okmvm.kmvm(X1[rows], X2, V, kind, ls, 1.25, 0.0, False)
    mag = okmvm.kmvm(X1[rows], X2, np.abs(V), kind, ls, 1.25, 0.0, False)
    if add_noise:
        ref = ref + float(np.float32(noise)) * V[rows]
        mag = mag + float(np.float32(noise)) * np.abs(V[rows])
    assert np.all(np.abs(out[rows] - ref) <= 2e-6 * mag + 1e-30)
    return out


# operand widths (d + 4 <= 32 slots, then 5 d + 6 in chunks of 32), row and
# column remainders, one and several passes over the right-hand sides
@pytest.mark.parametrize("d,n1,n2,r,kind", [
    (1, 9000, 9000, 1, 0), (5, 5003, 6200, 16, 1), (6, 4353, 6097, 17, 3), (11, 257, 120001, 3, 0),
    (12, 5000, 0, 33, 1), (18, 4700, 0, 8, 3), (19, 4500, 4500, 16, 0), (25, 4097, 4200, 5, 1),
    (28, 4600, 0, 20, 0), (8, 160000, 256, 16, 0), (7, 6100, 0, 4, 1), (4, 7400, 0, 2, 3)])
def test_split_product_matches_oracle(gpu_lib, d, n1, n2, r, kind):
    X1 = synth.random_points(n1, d, 700 + d)
    X2 = synth.random_points(n2, d, 800 + d) if n2 else X1
    V = synth.random_rhs(X2.shape[0], r, 900 + d)
    ls = [0.5 * np.sqrt(d)]
    check(gpu_lib, X1, X2, V, kind, np.asarray(ls, np.float32), 0.3, not n2)


def test_split_product_offset_points_and_ard(gpu_lib):
    # a box far from the origin: coordinates are taken from its centre
    X = synth.random_points(7100, 3, 41) + np.float32(50.0)
    V = synth.random_rhs(7100, 4, 42)
    check(gpu_lib, X, X, V, 0, np.array([0.7, 1.9, 4.0], np.float32), 0.1, True)


def test_split_product_keeps_small_entries(gpu_lib):
    # unit right-hand sides: single kernel values down to 1e-20 keep their digits
    X = synth.random_points(7800, 2, 43, scale=3.0)
    V = np.zeros((7800, 2), np.float32)
    V[7, 0] = 1.0
    V[7799, 1] = 1e-12
    t = torch.from_numpy(X).to(DEV)
    out = gpu_lib.kmvm(t, t, torch.from_numpy(V).to(DEV), 0, [0.8], 1.0, 0.0,
                       precision=gpu_lib.FP32).cpu().numpy()
    ref = okmvm.kmvm(X, X, V, 0, np.array([0.8], np.float32), 1.0, 0.0, False)
    k = ref / np.array([1.0, 1e-12])
    keep = k > 1e-20
    assert keep[:, 0].sum() > 1000
    rel = np.abs(out - ref)[keep] / ref[keep]
    assert np.all(rel <= (2 + 2 * np.abs(np.log2(k[keep]))) * 2.0 ** -23)
    assert np.all(out >= 0)


@pytest.mark.parametrize("what", ["wide", "nan_x", "matern12"])
def test_inputs_outside_the_form_take_the_vector_product(gpu_lib, what):
    X = synth.random_points(7200, 3, 44)
    V = synth.random_rhs(7200, 3, 45)
    kind, ls = 0, np.array([1.0], np.float32)
    if what == "wide":
        X[17] = (400.0, -300.0, 10.0)
    if what == "matern12":
        kind = 2
    if what == "nan_x":
        X[5, 1] = np.nan
        t = torch.from_numpy(X).to(DEV)
        out = gpu_lib.kmvm(t, t, torch.from_numpy(V).to(DEV), kind, ls, 1.0, 0.0,
                           precision=gpu_lib.FP32).cpu().numpy()
        assert np.all(np.isnan(out))
        return
    check(gpu_lib, X, X, V, kind, ls, 0.2, True)


@pytest.mark.parametrize("r", [4, 6])
def test_split_product_non_finite_rhs_stays_in_its_column(gpu_lib, r):
    X = synth.random_points(7100, 3, 46)
    V = synth.random_rhs(7100, r, 47)
    V[100, 1] = np.inf
    V[2000, 2] = np.nan
    t = torch.from_numpy(X).to(DEV)
    out = gpu_lib.kmvm(t, t, torch.from_numpy(V).to(DEV), 0, [1.0], 1.0, 0.0,
                       precision=gpu_lib.FP32).cpu().numpy()
    assert np.all(np.isposinf(out[:, 1])) and np.all(np.isnan(out[:, 2]))
    ref = okmvm.kmvm(X, X, V[:, [0, 3]], 0, np.array([1.0], np.float32), 1.0, 0.0, False)
    mag = okmvm.kmvm(X, X, np.abs(V[:, [0, 3]]), 0, np.array([1.0], np.float32), 1.0, 0.0, False)
    assert np.all(np.abs(out[:, [0, 3]] - ref) <= 2e-6 * mag)

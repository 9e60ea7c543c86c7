"""The gradient's split-operand form (grad_split.hip) and its neighbours below the lines
of its rule against the float64 oracle, at the bound of the other gradient tests:
2e-5 sum |dK~_ij| |W_ij| per component (float32 kernel values and P = G W, 22-bit parts
of U and C, float64 sums; float32 differences of coordinates up to d = 4)."""

import numpy as np
import pytest
import torch

from oracle import train as otrain
from paper_2207_06856_amd import synth

pytestmark = pytest.mark.gpu


def inputs(n, d, r, seed):
    X = synth.random_points(n, d, seed)
    B = synth.random_rhs(n, r, seed + 1, dist="rademacher")
    B[:, 0] = np.sin(X).sum(1)
    U = (0.9 * B + 0.3 * synth.random_rhs(n, r, seed + 2)).astype(np.float32)
    return X, B, U


def check(lib, X, B, U, kind, ls, a2):
    dev = [torch.from_numpy(a).cuda() for a in (X, B, U)]
    got = lib.mll_grad(*dev, kind, ls, a2, 0.4)
    ard = np.size(ls) > 1
    ref = otrain.pseudo_loss_grad(X, U, B, kind, ls, a2, ard)
    scale = otrain.pseudo_loss_grad_scale(X, U, B, kind, ls, a2, ard)
    m = len(ref)
    assert np.all(np.abs(got[:m] - ref) <= 2e-5 * np.asarray(scale) + 1e-12), (got[:m], ref, scale)
    return got


# operand widths and component blocks (d = 5/6, 8/9, 11/12, 16), row and column
# remainders, padded right-hand sides
@pytest.mark.parametrize("n,d,r,kind", [
    (3400, 2, 16, 0), (2753, 5, 16, 1), (2600, 6, 8, 3), (2432, 8, 16, 0), (2303, 9, 5, 1),
    (2177, 11, 2, 3), (2060, 12, 16, 0), (1857, 16, 16, 1), (3001, 8, 16, 0)])
def test_split_gradient_matches_oracle(gpu_lib, n, d, r, kind):
    X, B, U = inputs(n, d, r, 60 + n)
    ls = np.float32(0.5 * np.sqrt(d)) * (1 + np.arange(d, dtype=np.float32) / d)
    check(gpu_lib, X, B, U, kind, ls, 1.3)


# one lengthscale: the whole range (split form) against two row ranges, which
# take the difference form; sampled rows of the oracle give the size of the terms
@pytest.mark.parametrize("n,d,r,kind", [(16384, 1, 2, 0), (16500, 5, 16, 1), (16385, 11, 9, 3),
                                        (17001, 16, 16, 0)])
def test_isotropic_split_gradient_matches_row_ranges(gpu_lib, n, d, r, kind):
    X, B, U = inputs(n, d, r, 30 + d)
    ls = np.array([0.5 * np.sqrt(d)], np.float32)
    dev = [torch.from_numpy(a).cuda() for a in (X, B, U)]
    whole = gpu_lib.mll_grad(*dev, kind, ls, 0.9, 0.4)
    cut = 7000
    parts = sum(gpu_lib.mll_grad(*dev, kind, ls, 0.9, 0.4, rows=rg) for rg in ((0, cut), (cut, n)))
    rows = np.arange(0, n, n // 64)
    scale = otrain.pseudo_loss_grad_scale(X, U, B, kind, ls, 0.9, False, rows=rows) * n / len(rows)
    assert np.all(np.abs(whole - parts)[:3] <= 2e-5 * scale)


def test_wide_points_take_the_difference_form(gpu_lib):
    X, B, U = inputs(3200, 3, 4, 77)
    X[3] = (90.0, -80.0, 5.0)
    check(gpu_lib, X, B, U, 0, np.array([0.8, 1.0, 1.2], np.float32), 1.0)


def test_split_gradient_scales(gpu_lib):
    # right-hand sides and solutions of very different sizes per column
    X, B, U = inputs(3000, 4, 6, 78)
    s = np.float32(10.0) ** np.array([3, -4, 0, 2, -2, 1], np.float32)
    check(gpu_lib, X, B, (U * s).astype(np.float32), 1, np.array([1.1, 0.9, 1.3, 1.0], np.float32), 0.7)

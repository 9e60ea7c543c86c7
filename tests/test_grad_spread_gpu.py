"""The gradient's split-operand form over its dispatch's edges, and on points that lie
close together far from the centre of their box, where the squares of the coordinates
exceed those of the differences by (|a| / |a - b|)^2, against the float64 oracle at the
bound of the other gradient tests, 2e-5 sum |dK~_ij| |W_ij| per component.  The form's
own share: float64 sums, 2^-53 (20 / 0.005)^2 = 2e-9 (float32 differences up to d = 4,
2^-24 20 / 0.007 = 2e-4 of an entry, random per point and in sign over 3400 points);
kernel values, r^2 to 2e-7 at the widest box, i.e. at most 1e-5 of a Matern-3/2 term at
r = 0.01 and random in sign.

W is zero where both solutions and right-hand sides are, so a small set scattered among
points of zero rows has the small set's gradient: the oracle needs the set alone, and
the call is as large as the form asks for."""

import numpy as np
import pytest
import torch

from oracle import train as otrain
from paper_2207_06856_amd import synth

pytestmark = pytest.mark.gpu

# points from which the form is taken (d <= 4, <= 8, above; one lengthscale)
MIN_POINTS = {4: 28672, 8: 6144, 16: 2250}
MIN_ISO = {5: 24576, 16: 16384}


def least(table, d):
    return table[min(k for k in table if d <= k)]


def rhs(X, r, seed):
    B = synth.random_rhs(X.shape[0], r, seed, dist="rademacher")
    B[:, 0] = np.sin(X).sum(1)
    U = (0.9 * B + 0.3 * synth.random_rhs(X.shape[0], r, seed + 1)).astype(np.float32)
    return B, U


def check(lib, X, B, U, kind, ls, n):
    """The set X scattered among n points of its box; B and U are the set's rows."""
    m, d = X.shape
    rng = np.random.default_rng(n)
    Xn = rng.uniform(X.min(0), X.max(0), (n, d)).astype(np.float32)
    Bn, Un = np.zeros((2, n, B.shape[1]), np.float32)
    at = np.sort(rng.choice(n, m, replace=False))
    Xn[at], Bn[at], Un[at] = X, B, U
    got = lib.mll_grad(*[torch.from_numpy(a).cuda() for a in (Xn, Bn, Un)], kind, ls, 1.3, 0.4)
    ard = np.size(ls) > 1
    ref = otrain.pseudo_loss_grad(X, U, B, kind, ls, 1.3, ard)
    scale = np.asarray(otrain.pseudo_loss_grad_scale(X, U, B, kind, ls, 1.3, ard))
    k = len(ref)
    assert np.all(np.abs(got[:k] - ref) <= 2e-5 * scale), (np.abs(got[:k] - ref) / scale)


def lengthscales(d):
    return np.linspace(1.0, 1.2, d).astype(np.float32)


# both sides of every line, operand widths (d = 5/6, 11/12), component blocks (4/5,
# 8/9), row and column remainders, padded right-hand sides
@pytest.mark.parametrize("d,r,kind", [(2, 16, 0), (3, 5, 1), (4, 16, 3), (5, 16, 1), (6, 8, 3),
                                      (8, 16, 0), (9, 5, 1), (11, 2, 3), (12, 16, 0), (16, 16, 1)])
@pytest.mark.parametrize("over", [-1, 0, 77])
def test_gradient_at_the_lines(gpu_lib, d, r, kind, over):
    X = synth.random_points(900, d, 40 + d)
    B, U = rhs(X, r, 41 + d)
    ls = np.float32(0.5 * np.sqrt(d)) * (1 + np.arange(d, dtype=np.float32) / d)
    check(gpu_lib, X, B, U, kind, ls, least(MIN_POINTS, d) + over)


@pytest.mark.parametrize("d,r,kind", [(1, 2, 0), (2, 16, 3), (5, 16, 1), (6, 9, 0), (12, 16, 3)])
def test_isotropic_gradient_above_the_line(gpu_lib, d, r, kind):
    X = synth.random_points(900, d, 45 + d)
    B, U = rhs(X, r, 46 + d)
    check(gpu_lib, X, B, U, kind, np.array([0.5 * np.sqrt(d)], np.float32), least(MIN_ISO, d) + 3)


# clusters just inside the form's radius of 32 lengthscales; d = 2 takes differences,
# 6 and 9 one and two blocks of float64 products
@pytest.mark.parametrize("d,kind", [(2, 0), (2, 1), (2, 3), (6, 0), (6, 1), (6, 3), (9, 0), (9, 1),
                                    (9, 3)])
@pytest.mark.parametrize("sd", [0.1, 0.02, 0.005])
def test_clusters_far_from_the_centre(gpu_lib, d, kind, sd):
    m = 3400 if d == 2 else 2200
    rng = np.random.default_rng(50 + d)
    if d == 2:
        sites = np.stack(np.meshgrid(np.linspace(-20, 20, 6), np.linspace(-20, 20, 6)), -1).reshape(-1, 2)
    else:
        sites = rng.choice([-10.0, 10.0], (36, d)) * (1.2 if d == 6 else 1.0)
    X = (sites[np.arange(m) % 36] + sd * rng.standard_normal((m, d))).astype(np.float32)
    B, U = rhs(X, 16, 51 + d)
    check(gpu_lib, X, B, U, kind, lengthscales(d), least(MIN_POINTS, d) + 100)


# every point thirty times over, and one input whose two values lie six lengthscales apart
@pytest.mark.parametrize("d,kind", [(3, 0), (4, 3), (7, 0), (10, 1)])
def test_repeated_points_and_distant_levels(gpu_lib, d, kind):
    rng = np.random.default_rng(60 + d)
    m = 2220
    X = (3.0 * rng.standard_normal((m // 30 + 1, d))).astype(np.float32)[np.arange(m) // 30]
    X[:, 0] = 6.0 * (np.arange(m) % 2)
    B, U = rhs(X, 8, 61 + d)
    check(gpu_lib, X, B, U, kind, np.linspace(1.0, 1.5, d).astype(np.float32),
          least(MIN_POINTS, d) + 100)


# one target of 10^4 among ordinary ones, on a wide box: entries of W over many orders
@pytest.mark.parametrize("d", [2, 5])
def test_one_large_target(gpu_lib, d):
    m, ls = 2200, lengthscales(d)
    X = np.random.default_rng(70).uniform(-22, 22, (m, d)).astype(np.float32)
    if d == 5:
        X /= 2.0
    B, _ = rhs(X, 8, 71)
    B[m // 2, 0] = 1e4
    U = np.linalg.solve(otrain.ktilde(X, 0, ls, 1.3, 0.4), B.astype(np.float64)).astype(np.float32)
    check(gpu_lib, X, B, U, 0, ls, least(MIN_POINTS, d) + 100)

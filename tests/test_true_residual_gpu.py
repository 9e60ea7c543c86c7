"""The solver's float64 true residual on split operands (kmvm_split64.hip, from 8192 points)
against the float64 oracle: the reported norm at ordinary residuals, and its error where
nearly nothing of the residual is left.

An entry's r^2 carries two float32 roundings, its value |log2 k| 2^-24 and 2^-24 more, as
where the distances are float64, so ordinary residuals agree to 1e-4 with much to spare.
On a box so wide that K is the identity but for entries below 1e-9 the residual of
u = b / (1 + s^2) is u's rounding, 3e-8, and the diagonal must be exactly 1: what T's
roundings leave of a coincident point's distance, 1e-12 R^2, costs 1e-9 (RBF), an r^2 of
1e-10 R^2 would cost 3e-8."""
import numpy as np
import pytest
import torch

from oracle import kmvm as okmvm
from paper_2207_06856_amd import synth

pytestmark = pytest.mark.gpu


def reported(lib, X, B, U, kind, ls, s2, **kw):
    dev = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (X, B, U)]
    V, st = lib.cg_solve(dev[0], dev[1], kind, ls, 1.0, s2, tol=1e-6, x0=dev[2], **kw)
    return V.cpu().numpy(), st


def true_rel(X, B, U, kind, ls, s2):
    K = okmvm.kmvm(X, X, U.astype(np.float64), kind, ls, 1.0, s2, True)
    return np.linalg.norm(B - K, axis=0) / np.linalg.norm(B.astype(np.float64), axis=0)


# one, two to four, five to eight and more right-hand sides, operand widths (d = 5/6,
# 11/12, 16/17, 24/25), ragged rows; x0 as it is and after two iterations
@pytest.mark.parametrize("d,r,kind,prec,iters", [
    (1, 1, 0, "FP32", 0), (5, 3, 1, "FP16", 2), (6, 4, 3, "FP32", 0), (11, 5, 0, "FP16", 0),
    (12, 8, 1, "FP32", 2), (16, 9, 3, "FP16", 0), (17, 17, 0, "FP32", 0), (25, 16, 1, "FP16", 0),
    (28, 2, 0, "FP16", 0)])
def test_reported_residual_matches_oracle(gpu_lib, d, r, kind, prec, iters):
    n, s2 = 8192 + 37 * r + d, float(np.float32(0.3))
    X = synth.random_points(n, d, 300 + d)
    B = synth.random_rhs(n, r, 301 + d)
    U = (0.02 * synth.random_rhs(n, r, 302 + d)).astype(np.float32)
    ls = np.array([0.5 * np.sqrt(d)], np.float32)
    V, st = reported(gpu_lib, X, B, U, kind, ls, s2, max_iter=iters, min_iter=iters,
                     precision=getattr(gpu_lib, prec))
    np.testing.assert_allclose(st["true_rel_res"], true_rel(X, B, V, kind, ls, s2), rtol=1e-4)


def test_periodic_residuals_match_oracle(gpu_lib):
    n, d, r, s2 = 8300, 3, 2, float(np.float32(0.3))
    X, B = synth.random_points(n, d, 310), synth.random_rhs(n, r, 311)
    ls = np.array([0.8], np.float32)
    dev = [torch.from_numpy(a).cuda() for a in (X, B)]
    U, st = gpu_lib.cg_solve(*dev, 0, ls, 1.0, s2, tol=1e-6, max_iter=6, min_iter=6,
                             true_res_every=3, precision=gpu_lib.FP32)
    half, _ = gpu_lib.cg_solve(*dev, 0, ls, 1.0, s2, tol=1e-6, max_iter=3, min_iter=3,
                               precision=gpu_lib.FP32)
    want = [true_rel(X, B, u.cpu().numpy(), 0, ls, s2) for u in (half, U)]
    np.testing.assert_allclose(st["true_history"], want, rtol=1e-4)


# boxes wider than the form's limit, and points that are not finite nowhere but in x0
@pytest.mark.parametrize("prec", ["FP32", "FP16"])
def test_wide_box_takes_the_float64_distances(gpu_lib, prec):
    n, d, r, s2 = 8400, 3, 5, float(np.float32(0.3))
    X = synth.random_points(n, d, 320)
    X[5] = (90.0, -60.0, 10.0)
    B = synth.random_rhs(n, r, 321)
    U = (0.02 * synth.random_rhs(n, r, 322)).astype(np.float32)
    ls = np.array([0.9], np.float32)
    V, st = reported(gpu_lib, X, B, U, 1, ls, s2, max_iter=2, min_iter=2, true_res_every=1,
                     precision=getattr(gpu_lib, prec))
    np.testing.assert_allclose(st["true_rel_res"], true_rel(X, B, V, 1, ls, s2), rtol=1e-4)


def check_little_left(lib, X, kind, r):
    B = synth.random_rhs(X.shape[0], r, 331, dist="rademacher")
    U = (B / np.float32(1.5)).astype(np.float32)
    ls = np.ones(1, np.float32)
    _, st = reported(lib, X, B, U, kind, ls, 0.5, max_iter=0, precision=lib.FP32)
    want = true_rel(X, B, U, kind, ls, 0.5)
    err = np.sqrt(np.abs(np.asarray(st["true_rel_res"]) ** 2 - want ** 2))
    assert want.max() <= 1e-6 and err.max() <= 4e-9, (want.max(), err.max())


@pytest.mark.parametrize("r", [16, 5])
def test_little_left_of_the_residual(gpu_lib, r):
    X = np.random.default_rng(330).uniform(-7.5, 7.5, (8400, 16)).astype(np.float32)   # R = 30
    check_little_left(gpu_lib, X, 0, r)


# the Matern kernels' tails need points further apart: distinct corners of the box
@pytest.mark.parametrize("kind,r", [(1, 16), (3, 4)])
def test_little_left_of_the_residual_matern(gpu_lib, kind, r):
    c = np.random.default_rng(340).permutation(1 << 16)[:8400]
    X = np.where((c[:, None] >> np.arange(16)) & 1, 7.5, -7.5).astype(np.float32)
    check_little_left(gpu_lib, X, kind, r)


# one and five to eight right-hand sides: the diagonal's correction of each sum's form
@pytest.mark.parametrize("kind,r,n", [(1, 8, 8400), (3, 1, 8193), (1, 5, 8447)])
def test_little_left_of_the_residual_matern_few(gpu_lib, kind, r, n):
    c = np.random.default_rng(341).permutation(1 << 16)[:n]
    X = np.where((c[:, None] >> np.arange(16)) & 1, 7.5, -7.5).astype(np.float32)
    check_little_left(gpu_lib, X, kind, r)

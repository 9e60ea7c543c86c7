"""The float32 product's bfloat16 parts: sums of one sign carry no common shortfall, and
right-hand sides at the ends of float32's range keep their value.

The parts of an entry and of a right-hand side leave out products of at most 2^-22 of
the whole whose sign is that of the right-hand side's second and third part, and every
other rounding is to nearest, so the mean error over many rows is near zero: within
2.5e-8 of the sum of magnitudes (parts that are all cut off leave 6e-8 on the low side)."""
import numpy as np
import pytest
import torch

from oracle import kmvm as okmvm
from paper_2207_06856_amd import synth

pytestmark = pytest.mark.gpu


def product(lib, X1, X2, V, ls):
    t = [torch.from_numpy(a).cuda() for a in (X1, X2, V)]
    return lib.kmvm(*t, 0, ls, 1.0, 0.0, precision=lib.FP32).cpu().numpy().astype(np.float64)


@pytest.mark.parametrize("d,n1,n2,r", [(2, 140_000, 256, 16), (8, 60_000, 700, 20), (5, 9000, 9000, 5)])
def test_same_sign_sums_have_no_bias(gpu_lib, d, n1, n2, r):
    X1, X2 = synth.random_points(n1, d, 400 + d), synth.random_points(n2, d, 401 + d)
    V = np.abs(synth.random_rhs(n2, r, 402 + d)) + np.float32(0.1)
    ls = np.array([0.7 * np.sqrt(d)], np.float32)
    rows = np.arange(0, n1, max(1, n1 // 6000))
    ref = okmvm.kmvm(X1[rows], X2, V, 0, ls, 1.0, 0.0, False)
    err = (product(gpu_lib, X1, X2, V, ls)[rows] - ref) / ref
    assert abs(err.mean()) <= 2.5e-8, err.mean()
    assert np.abs(err).max() <= 2e-6


def test_right_hand_sides_at_the_ends_of_the_range(gpu_lib):
    # the largest floats would round to an infinite first part; at most one per column,
    # so that the sums before the outputscale stay finite
    X = synth.random_points(7300, 3, 410)
    big = np.finfo(np.float32).max
    V = np.zeros((7300, 6), np.float32)
    V[:, 0], V[7, 1], V[7, 2] = 1e-30, -big, big
    V[100, 3], V[200, 4] = np.nextafter(big, np.float32(0)), 2.0 ** 127
    V[:, 5] = synth.random_rhs(7300, 1, 411)[:, 0] * np.float32(1e33)
    ls = np.array([2.0], np.float32)
    ref = okmvm.kmvm(X, X, V, 0, ls, 2.0 ** -12, 0.0, False)
    mag = okmvm.kmvm(X, X, np.abs(V), 0, ls, 2.0 ** -12, 0.0, False)
    t = [torch.from_numpy(a).cuda() for a in (X, X, V)]
    out = gpu_lib.kmvm(*t, 0, ls, 2.0 ** -12, 0.0, precision=gpu_lib.FP32).cpu().numpy()
    assert np.isfinite(out).all()
    assert np.all(np.abs(out - ref) <= 2e-6 * mag)

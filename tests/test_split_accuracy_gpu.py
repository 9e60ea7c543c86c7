"""The float32 product's distances at the two ends of their range.

Where little but the diagonal of K is left (a wide box in many dimensions) an output is
its right-hand side, and its error one float32 rounding at most: 2^-24 / sqrt(3) = 3.4e-8
rms, of which an exact diagonal leaves next to nothing; half of that is the bar.

Where far entries make up the sums, an entry carries one rounding of r^2, uniform within
half a unit, and 1.5 units of its exponential, parts and product, independent from entry
to entry: rms 2^-24 / sqrt(12) |ln k| and 2^-24, plus 4e-8 for the sum of the whole.
Several roundings of r^2 per entry (one for each MFMA of a chain) are twice that and more."""
import numpy as np
import pytest
import torch

from oracle import kernels as okern
from oracle import kmvm as okmvm
from paper_2207_06856_amd import synth

pytestmark = pytest.mark.gpu
ONE = np.ones(1, np.float32)


def product(lib, X1, X2, V, kind):
    t1, v = torch.from_numpy(X1).cuda(), torch.from_numpy(V).cuda()
    t2 = t1 if X2 is X1 else torch.from_numpy(X2).cuda()
    return lib.kmvm(t1, t2, v, kind, [1.0], 1.0, 0.0, precision=lib.FP32).cpu().numpy()


# inside the form's radius (R = 19) and beyond it (29); parts and FMAs
@pytest.mark.parametrize("d,R,r", [(28, 19.0, 8), (28, 19.0, 2), (16, 29.0, 16), (16, 29.0, 3)])
def test_little_but_the_diagonal(gpu_lib, d, R, r):
    n = 6500
    X = (np.random.default_rng(420 + d).uniform(-1, 1, (n, d)) * (R / np.sqrt(d))).astype(np.float32)
    V = synth.random_rhs(n, r, 421 + d)
    ref = okmvm.kmvm(X, X, V, 0, ONE, 1.0, 0.0, False)
    err = (product(gpu_lib, X, X, V, 0) - ref) / okmvm.kmvm(X, X, np.abs(V), 0, ONE, 1.0, 0.0, False)
    assert np.sqrt((err ** 2).mean()) <= 1.7e-8, np.sqrt((err ** 2).mean())


@pytest.mark.parametrize("d,n1,n2,kind", [(12, 60_000, 1200, 0), (20, 60_000, 1000, 0),
                                          (28, 40_000, 1200, 0)])
def test_sums_of_far_entries(gpu_lib, d, n1, n2, kind):
    scale = np.float32(4.0 / np.sqrt(d))            # R = 4.4 x 4
    X1, X2 = synth.random_points(n1, d, 430) * scale, synth.random_points(n2, d, 431) * scale
    V = synth.random_rhs(n2, 16, 432)
    rows = np.arange(0, n1, 37)
    out = product(gpu_lib, X1, X2, V, kind)[rows]
    K = okern.kfun(kind, okern.scaled_sqdist(X1[rows].astype(np.float64), X2.astype(np.float64), ONE))
    mag = K @ np.abs(V.astype(np.float64))
    err = (out - K @ V.astype(np.float64)) / mag
    one = K * 2.0 ** -24 * np.hypot(np.log(np.maximum(K, 1e-300)) / np.sqrt(12.0), 1.0)
    want = np.sqrt(((one ** 2) @ (V.astype(np.float64) ** 2)) / mag ** 2)
    bar = np.sqrt((want ** 2).mean()) + 4e-8
    assert np.sqrt((err ** 2).mean()) <= bar, (np.sqrt((err ** 2).mean()), bar)

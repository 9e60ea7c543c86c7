"""Repeated points far from the origin: the pivoted Cholesky factor stops once the distinct
points are used up, as near the origin.  Equal points are at distance 0 exactly, so the
residual diagonal of a used-up point is the rounding of a^2 - l^2, below 1e-15 a^2; a
distance of one rounding of x / l (4e-12 here) would leave a Matern-1/2 diagonal of 8e-12."""
import numpy as np
import pytest
import torch

from oracle import pivchol
from paper_2207_06856_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", [0, 1, 2, 3])
def test_early_stop_on_repeated_points_far_from_the_origin(gpu_lib, kind):
    base = synth.random_points(12, 3, 7) + np.float32(30000.0)
    X = np.repeat(base, 30, axis=0)
    ls = np.array([0.7], np.float32)
    P = gpu_lib.Precond(torch.from_numpy(X).cuda(), kind, ls, 1.0, 0.1, 40)
    Lr, piv, _ = pivchol.pivoted_cholesky(X, kind, ls, 1.0, 40)
    distinct = len(np.unique(base, axis=0))
    assert P.rank == Lr.shape[1] == distinct
    np.testing.assert_array_equal(P.pivots, piv)
    assert P.trace_residual <= 360 * 1e-12
    P.close()

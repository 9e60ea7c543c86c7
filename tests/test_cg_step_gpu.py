"""The one-launch step of small unpreconditioned float32 solves, against the float64 oracle.

Sizes: the smallest, remainders of its rows and columns, the largest it takes
(n = 2048; n times the padded columns = 4096) and the first it does not, and a basis that
outgrows it within the solve, after which the step's separate launches go on.

Bars: re-orthogonalised CG follows the float64 recurrence, so the iteration
count of a column may differ only where its residual passes the tolerance
within rounding: at most one iteration.  With e = 2^-24 ||K~|| ||u|| / ||b||
(the norm by the largest row sum) for one rounding of the entries, the solver's
residual is the oracle's to 4 e, and the tolerance plus float32's attainable
accuracy, sqrt(n) e, bounds it.  Since K~ - s^2 I is positive
semidefinite, ||u - u*|| <= ||residual|| / s^2.
"""
import numpy as np
import pytest
import torch

from oracle import cg as ocg
from oracle import direct
from paper_2207_06856_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def to_dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


@pytest.mark.parametrize("n,r,kind,algo,reorth,lse", [
    (1, 1, 0, 1, True, True),
    (5, 3, 1, 1, True, False),
    (64, 64, 0, 1, True, True),        # every column lane, 16 row lanes
    (61, 17, 2, 1, True, True),
    (500, 3, 0, 1, True, True),
    (255, 8, 0, 1, False, True),
    (256, 8, 1, 1, True, True),        # the most at two entries a thread
    (257, 8, 1, 1, True, True),
    (512, 8, 0, 1, True, True),        # the most at four
    (513, 8, 0, 1, True, True),        # separate launches
    (1024, 2, 0, 0, False, False),
    (1025, 1, 1, 1, True, False),
    (2048, 1, 0, 1, True, True),
    (2049, 1, 0, 1, True, True),       # separate launches
    (2000, 2, 2, 1, True, True),       # more iterations than the basis allows (96)
])
def test_small_solve_matches_oracle(gpu_lib, n, r, kind, algo, reorth, lse):
    print(f"small step n={n} r={r} kind={kind} algo={algo} {reorth} {lse}", flush=True)
    X = synth.random_points(n, 3, n + r)
    B = synth.random_rhs(n, r, n + r)
    B[:, r // 2] *= 1e-3
    if r > 2:
        B[:, -1] = np.cos(np.arange(n))
    ls, s2 = np.array([0.9], np.float32), float(np.float32(0.01 if kind == 2 else 0.25))
    tol = 1e-5
    U, st = gpu_lib.cg_solve(to_dev(X), to_dev(B), kind, ls, 1.0, s2, tol=tol, max_iter=400,
                             min_iter=0, algo=algo, reorth=reorth, use_lse=lse,
                             precision=gpu_lib.FP32)
    U = U.cpu().numpy().astype(np.float64)
    A = direct.ktilde(X, kind, ls, 1.0, s2)
    assert st["converged"].all() and not st["breakdown"].any()
    if reorth:
        _, ref = ocg.solve(lambda V: A @ V, B, tol, 400, algo="enhanced", reorth=True,
                           use_lse=lse)
        print("iterations", st["iters"], ref["iters"], flush=True)
        assert np.abs(np.asarray(ref["iters"]) - st["iters"]).max() <= 1
    tr = ocg.true_relative_residual(lambda V: A @ V, B, U)
    bn, un = np.linalg.norm(B, axis=0), np.linalg.norm(U, axis=0)
    entry = 2.0 ** -24 * A.sum(1).max() * un / bn
    assert (np.abs(st["true_rel_res"] - tr) <= 1e-4 * tr + 4 * entry).all()
    assert (tr <= tol + np.sqrt(max(n, 16)) * entry).all()
    exact = np.linalg.solve(A, B.astype(np.float64))
    assert (np.linalg.norm(U - exact, axis=0) <= 1.0001 * tr * bn / s2 + 1e-9 * un).all()

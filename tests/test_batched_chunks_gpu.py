"""The batched solve at the edges of its row chunks and factor tiles.

Row counts around multiples of the 128-row chunks and of the 32-row steps, more
chunks than a work group has threads, ranks around the 16-wide tiles of the
factor products (and a factorisation that ends early), right-hand sides around
the 16-wide column tiles.  Bars of the batched suite: 1e-3 relative to the
single-problem solver at the same iteration counts, counts within one, the true
residual of the float64 oracle to 1e-4.  The factorisation follows float64
residual diagonals, so that its rank and the applied preconditioner decide the
iteration counts compared here.
"""
import numpy as np
import pytest
import torch

from oracle import cg as ocg
from oracle import direct
from paper_2207_06856_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def rel(a, b):
    b = np.asarray(b, np.float64)
    return float(np.linalg.norm(np.asarray(a, np.float64) - b) / np.linalg.norm(b))


@pytest.mark.parametrize("lse", [True, False])
def test_batched_chunk_edges(gpu_lib, lse):
    shapes = [(1, 1, 0), (33, 1, 1), (127, 3, 15), (128, 8, 16), (129, 8, 17), (255, 16, 31),
              (257, 17, 33), (385, 33, 48), (1000, 64, 49), (2049, 1, 128), (70, 2, 60)]
    probs = []
    for i, (n, r, rank) in enumerate(shapes):
        X = synth.random_points(n, 3, 900 + i)
        if n == 70:
            X = np.repeat(X[:7], 10, axis=0)       # seven distinct points: rank 7
        B = synth.random_rhs(n, r, 900 + i)
        probs.append(dict(X=torch.from_numpy(X).to(DEV), B=torch.from_numpy(B).to(DEV), kind=i % 4,
                          lengthscale=np.array([0.8], np.float32), outputscale=1.0,
                          noise=float(np.float32(0.5)), precond_rank=rank, Xn=X, Bn=B))
    Us, sts = gpu_lib.cg_solve_batched(probs, tol=1e-2, max_iter=60, min_iter=0, use_lse=lse)
    for i, p in enumerate(probs):
        print(f"chunks n={shapes[i][0]} r={shapes[i][1]} rank={shapes[i][2]}", flush=True)
        P = (gpu_lib.Precond(p["X"], p["kind"], p["lengthscale"], 1.0, p["noise"],
                             p["precond_rank"]) if p["precond_rank"] else None)
        U, st = gpu_lib.cg_solve(p["X"], p["B"], p["kind"], p["lengthscale"], 1.0, p["noise"],
                                 tol=1e-2, max_iter=60, min_iter=0, precond=P, use_lse=lse)
        print(sts[i]["iters"], st["iters"], flush=True)
        assert sts[i]["converged"].all() and not sts[i]["breakdown"].any()
        assert np.abs(sts[i]["iters"] - st["iters"]).max() <= 1
        if (sts[i]["iters"] == st["iters"]).all():
            assert rel(Us[i].cpu().numpy(), U.cpu().numpy()) <= 1e-3
        A = direct.ktilde(p["Xn"], p["kind"], p["lengthscale"], 1.0, p["noise"])
        tr = ocg.true_relative_residual(lambda V: A @ V, p["Bn"], Us[i].cpu().numpy())
        np.testing.assert_allclose(sts[i]["true_rel_res"], tr, rtol=1e-4, atol=1e-7)


def test_batched_many_chunks(gpu_lib):
    # 269 chunks: more than the 256 threads that merge them
    n = 34_321
    X = torch.from_numpy(synth.random_points(n, 4, 77)).to(DEV)
    B = torch.from_numpy(synth.random_rhs(n, 3, 77)).to(DEV)
    ls, s2 = np.array([1.0], np.float32), float(np.float32(1.0))
    Us, sts = gpu_lib.cg_solve_batched(
        [dict(X=X, B=B, kind=0, lengthscale=ls, outputscale=1.0, noise=s2, precond_rank=20)],
        tol=1.0, max_iter=60, min_iter=10)
    P = gpu_lib.Precond(X, 0, ls, 1.0, s2, 20)
    U, st = gpu_lib.cg_solve(X, B, 0, ls, 1.0, s2, tol=1.0, max_iter=60, min_iter=10, precond=P)
    assert (sts[0]["iters"] == st["iters"]).all()
    assert rel(Us[0].cpu().numpy(), U.cpu().numpy()) <= 1e-3

"""Float64 sums of the one-launch step.  With all points equal K = 1 1^T, and with powers of
two in the direction and the noise every float32 product and sum of the first iteration
but d^T K~ d is exact: sum_i d_i (4 + s^2 d_i) = 16 + s^2 ||d||^2 = 144.002 from terms of
+-32,768.  In float32 each merge of the large terms rounds by up to 2^-9 (1.4e-5 of the
result), in float64 by nothing; alpha then carries ||b||^2's float32 roundings (2e-7)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,r", [(2048, 1), (1024, 2), (256, 16)])
def test_first_step_length_without_logsumexp(gpu_lib, n, r):
    s2, big = 2.0 ** -20, 8192.0
    b = np.ones(n, np.float32)
    b[1:-1][np.random.default_rng(n).permutation(n - 2)[:n // 2 - 3]] = -1.0
    b[0], b[-1] = big, -big
    S, b2 = float(b.sum()), float((b.astype(np.float64) ** 2).sum())
    assert S == 4.0
    B = torch.from_numpy(np.repeat(b[:, None], r, axis=1)).cuda()
    U, _ = gpu_lib.cg_solve(torch.zeros((n, 1), device="cuda"), B, 0, [1.0], 1.0, s2, tol=0.0,
                            max_iter=1, min_iter=1, algo=0, reorth=False, use_lse=False,
                            precision=gpu_lib.FP32, true_res_every=-1)
    alpha = b2 / (S * S + s2 * b2)
    got = U.cpu().numpy().astype(np.float64) / b[:, None]
    assert np.abs(got / alpha - 1.0).max() <= 1e-6, np.abs(got / alpha - 1.0).max()

"""The gradient with little device memory left: the split form's operands do not fit and
the difference form, which needs a fifth of the scratch, runs in its place."""

import numpy as np
import pytest
import torch

from oracle import train as otrain
from paper_2207_06856_amd import synth

pytestmark = pytest.mark.gpu


def test_gradient_without_room_for_the_split_operands(gpu_lib):
    # scratch: 121 MB for the difference form, 460 MB more for the split operands
    n, d, m, r, left = 600_000, 16, 900, 16, 320 << 20
    rng = np.random.default_rng(5)
    ls = (2.0 + np.arange(d) / d).astype(np.float32)
    X = synth.random_points(m, d, 6)
    B = synth.random_rhs(m, r, 7, dist="rademacher")
    U = (0.9 * B + 0.3 * synth.random_rhs(m, r, 8)).astype(np.float32)
    at = torch.from_numpy(np.sort(rng.choice(n, m, replace=False))).cuda()
    Xn = torch.randn((n, d), device="cuda", generator=torch.Generator("cuda").manual_seed(9))
    Bn, Un = torch.zeros((n, r), device="cuda"), torch.zeros((n, r), device="cuda")
    for full, part in ((Xn, X), (Bn, B), (Un, U)):
        full[at] = torch.from_numpy(part).cuda()
    torch.cuda.synchronize()
    gpu_lib.release_cached_memory()
    torch.cuda.empty_cache()
    fill = []
    while (more := torch.cuda.mem_get_info()[0] - left) > 4 << 20:
        fill.append(torch.empty(more, dtype=torch.uint8, device="cuda"))
    try:
        got = gpu_lib.mll_grad(Xn, Bn, Un, 0, ls, 1.3, 0.4)
    finally:
        del fill
        gpu_lib.release_cached_memory()
        torch.cuda.empty_cache()
    ref = otrain.pseudo_loss_grad(X, U, B, 0, ls, 1.3, True)
    scale = np.asarray(otrain.pseudo_loss_grad_scale(X, U, B, 0, ls, 1.3, True))
    assert np.all(np.abs(got[:len(ref)] - ref) <= 2e-5 * scale)

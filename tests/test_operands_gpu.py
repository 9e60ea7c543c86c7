"""The operands of the 16-bit products, bit for bit.

The points lie so far apart that every kernel value of two distinct points
rounds to zero and that of a point with itself to one (binary16: exp(-18) is
below half the least subnormal; bfloat16: exp(-112) is below its least value;
the argument's error, at most a few 2^-22 of the squared norms, is below half an
ulp of one).  The product is then the rounded right-hand sides themselves:
a column times the power of two that brings its largest entry to [2^14, 2^15)
(or 1/sqrt(n)), rounded to the format, divided by it again.  Every sum has one
non-zero term, so that equality is exact, at every remainder of the operand
rows, the row blocks, the stages and the groups of the column maxima.
"""
import numpy as np
import pytest
import torch

from paper_2207_06856_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def spread_points(n, d, step):
    i = np.arange(n)[:, None] // 3 ** np.arange(d)[None, :] % 3
    return ((i - 1) * step).astype(np.float32)


def round_to(x, bf16):
    t = torch.from_numpy(np.ascontiguousarray(x, dtype=np.float32))
    return t.to(torch.bfloat16 if bf16 else torch.float16).float().numpy()


@pytest.mark.parametrize("n,d,r", [
    (1, 1, 1), (2, 1, 3), (31, 4, 16), (32, 4, 17), (33, 4, 63), (127, 5, 64), (128, 5, 65),
    (129, 5, 130), (255, 6, 1), (256, 6, 7), (257, 30, 5), (2187, 7, 16), (6561, 9, 2),
    (19683, 9, 16),                     # the symmetric form (binary16), 154 groups of maxima
    (19683, 9, 64),                     # 256 groups
])
@pytest.mark.parametrize("bf16", [False, True])
def test_operands_exact(gpu_lib, n, d, r, bf16):
    print(f"operands n={n} d={d} r={r} bf16={bf16}", flush=True)
    X = torch.from_numpy(spread_points(n, d, 15.0 if bf16 else 6.0)).to(DEV)
    g = np.random.Generator(np.random.PCG64(n + r))
    V = (synth.random_rhs(n, r, n + r) * 2.0 ** g.integers(-9, 0, (n, r))).astype(np.float32)
    V *= (2.0 ** g.integers(-30, 30, r)).astype(np.float32)
    V[g.integers(0, n, r), np.arange(r)] *= 100.0           # one row sets a column's scale
    if r > 2:
        V[:, r // 2] = 0.0
    prec = gpu_lib.BF16 if bf16 else gpu_lib.FP16
    for scale_mode in (0, 1):
        if scale_mode == 0:
            m = np.abs(V).max(0)
            s = np.where(m > 0, np.ldexp(1.0, 15 - np.frexp(np.where(m > 0, m, 1.0))[1]), 1.0)
            inv = 1.0 / s
        else:
            s = np.full(r, np.float32(1.0 / np.sqrt(n)))
            inv = np.full(r, np.float32(np.sqrt(n)))
        s, inv = s.astype(np.float32), inv.astype(np.float32)
        if scale_mode == 1 and not bf16:
            V = np.clip(V, -6e4, 6e4)                       # a fixed scale may overflow binary16
        ref = round_to(V * s, bf16) * inv
        out = gpu_lib.kmvm(X, X, torch.from_numpy(V).to(DEV), 0, [1.0], 1.0, 0.0, add_noise=False,
                           precision=prec, scale_mode=scale_mode)
        np.testing.assert_array_equal(out.cpu().numpy(), ref)

"""GPU: the dense inverse of the coarsest level at the sizes where its forms
change (32 rows a register; 192 rows, above which the matrix is in global
memory), through the preconditioner of a one-level hierarchy, which is the
dense solve: equal to the oracle's (LU with partial pivoting) to the 1e-12 of
the cycle's comparisons where the matrix is scaled (no row is interchanged),
and to 1e-11 where it is not: nearly every row is interchanged then, and
nd eps cond = 270 x 2.2e-16 x 130 = 8e-12 at the largest.
"""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def gpu():
    import torch
    import paper_2608_09102_amd as llg
    assert torch.cuda.is_available()
    return llg


@pytest.mark.parametrize("left_scale,tol", [(1, 1e-12), (0, 1e-11)])
@pytest.mark.parametrize("n", [(2, 2), (2, 5), (3, 7), (4, 8), (5, 9), (6, 7), (6, 9), (8, 8), (5, 13), (9, 10)])
def test_dense_inverse(gpu, orc, n, left_scale, tol):
    import torch
    N = n[0] * n[1]
    say("[dense]", n, 3 * N, left_scale)
    rng = np.random.default_rng(N)
    m = rng.standard_normal((N, 3))
    m /= np.linalg.norm(m, axis=1, keepdims=True)
    kw = dict(max_levels=1, max_coarse=N, left_scale=left_scale)
    S = gpu.Solver(gpu.make_grid(2, n, 1.0 / n[0]), gpu.default_opts(precision="fp64", **kw))
    H = orc.Hierarchy(orc.make_grid(2, n, 1.0 / n[0]), orc.default_opts(**kw), m, 0.1, 1e-1)
    assert S.setup(torch.from_numpy(m).cuda(), 0.1, 1e-1) == gpu.OK
    assert S.num_levels == 1 and H.num_levels == 1
    v = rng.standard_normal((N, 3))
    z = S.precond(torch.from_numpy(v).cuda()).cpu().numpy()
    ref = H.precond(v)
    d = np.abs(z - ref).max() / np.abs(ref).max()
    say("  diff %.2e" % d)
    assert d <= tol

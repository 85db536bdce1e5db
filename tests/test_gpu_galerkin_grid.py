"""GPU: level 1 from a grid level stored as BSR, with one block K_i a row.

The coarse blocks are bit-identical to the oracle's at the edges of the
kernel's forms: a slice of 64 coarse rows and one row more, rows scaled and
not (the diagonal block the identity and not), up to four members a row and
up to eight, and a level 1 that is the coarsest.
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


CASES = [(2, (2, 2, 1), dict(max_coarse=1, max_levels=2)), (2, (15, 14, 1), dict()), (2, (17, 13, 1), dict(npass=1)),
         (2, (40, 33, 1), dict(npass=3)), (3, (13, 11, 9), dict(npass=3, max_coarse=300)), (3, (9, 14, 12), dict())]


@pytest.mark.parametrize("left_scale", [1, 0])
@pytest.mark.parametrize("dim,n,kw", CASES, ids=["x".join(map(str, c[1])) for c in CASES])
def test_galerkin_grid_bsr(gpu, orc, dim, n, kw, left_scale):
    import torch
    say("[galerkin_grid]", n, kw, left_scale)
    rng = np.random.default_rng(2)
    m = rng.standard_normal((int(np.prod(n)), 3))
    m /= np.linalg.norm(m, axis=1, keepdims=True)
    kw = dict(kw, left_scale=left_scale)
    S = gpu.Solver(gpu.make_grid(dim, n, 1.0 / n[0]), gpu.default_opts(precision="fp64", fine_operator="bsr", **kw))
    H = orc.Hierarchy(orc.make_grid(dim, n, 1.0 / n[0]), orc.default_opts(**kw), m, 0.1, 1e-3)
    assert S.setup(torch.from_numpy(m).cuda(), 0.1, 1e-3) == gpu.OK
    assert S.num_levels == H.num_levels
    for l in range(H.num_levels):
        rp, ci, val = S.level(l)
        R = H.level(l)
        assert np.array_equal(rp, R.rp) and np.array_equal(ci, R.ci) and np.array_equal(val, R.val), l

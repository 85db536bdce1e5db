"""GPU: the structure of the small levels built by one launch of a team.

The team takes the decisions and orders of the per-pass kernels, so aggregates
and patterns equal the oracle's and FP64 values are bit-identical to it, after
several rebuilds, at grids around the largest pass matched in LDS (640 nodes)
and the largest level built by a team (24576 nodes), for every number of
passes, with long rows, and beside the solve or in line with it.
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


CASES = [
    (2, (2, 3, 1), dict(max_coarse=1)),
    (2, (32, 20, 1), dict(max_coarse=4)),
    (2, (641, 2, 1), dict(max_coarse=1, npass=1)),
    (2, (67, 59, 1), dict(npass=3, max_coarse=2, overlap_rebuild=0)),
    (2, (192, 128, 1), dict(overlap_rebuild=0)),
    (2, (193, 128, 1), dict()),
    (3, (29, 29, 29), dict(npass=3)),
    (3, (17, 16, 15), dict(npass=1, max_coarse=3, beta_num=1, beta_den=1)),
    (3, (24, 23, 22), dict(smoother=1, overlap_rebuild=0)),
    (2, (130, 70, 1), dict(beta_num=0, max_coarse=2, max_levels=4)),
]


@pytest.mark.parametrize("case", CASES, ids=["%dd-%s-%d" % (c[0], "x".join(map(str, c[1])), k)
                                             for k, c in enumerate(CASES)])
def test_team_build_is_the_oracles(gpu, orc, case):
    import torch
    dim, n, kw = case
    say("[team_build]", dim, n, kw)
    rng = np.random.default_rng(3)
    m = rng.standard_normal((int(np.prod(n)), 3))
    m /= np.linalg.norm(m, axis=1, keepdims=True)
    S = gpu.Solver(gpu.make_grid(dim, n, 1.0 / n[0]), gpu.default_opts(precision="fp64", **kw))
    mt = torch.from_numpy(m).cuda()
    okw = {k: v for k, v in kw.items() if k != "overlap_rebuild"}
    H = orc.Hierarchy(orc.make_grid(dim, n, 1.0 / n[0]), orc.default_opts(**okw), m, 0.1, 1e-4)
    assert S.num_levels == H.num_levels
    for rebuild in range(3):
        assert S.setup(mt, 0.1, 1e-4) == gpu.OK
        for l in range(H.num_levels):
            rp, ci, val = S.level(l)
            R = H.level(l)
            assert np.array_equal(rp, R.rp) and np.array_equal(ci, R.ci), (rebuild, l)
            assert np.array_equal(val, R.val), (rebuild, l)
            if l + 1 < H.num_levels:
                assert np.array_equal(S.aggregates(l), R.agg), (rebuild, l)

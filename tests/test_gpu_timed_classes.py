"""GPU: what the kernel classes of set_kernel_timing hold.

The residual class is the residuals and their restriction.  Where a team runs
the small levels' cycle, the class holds those of the levels above it only, so
it is never more than with the levels one by one.
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


KT_RESIDUAL = 3


@pytest.mark.parametrize("smoother", ("jacobi", "mcgs"))
def test_residual_class_without_the_team(gpu, smoother):
    import torch
    say("[residual_class_without_the_team]", smoother)
    n = (96, 96, 1)
    m = np.random.default_rng(2).standard_normal((n[0] * n[1], 3))
    m = torch.from_numpy(m / np.linalg.norm(m, axis=1, keepdims=True)).cuda()
    ms = {}
    for t in (128, 0):
        S = gpu.Solver(gpu.make_grid(2, n, 1.0 / n[0]), gpu.default_opts(tail_nodes=t, smoother=smoother,
                                                                         kcycle_depth=1))
        S.set_kernel_timing(KT_RESIDUAL)
        best = []
        for _ in range(5):
            _, s, st = S.step(m, 0.05, 2e-4)
            assert s == gpu.OK and st.kernel_launches > 0
            best.append(st.kernel_ms / st.iters)
        ms[t] = min(best)
        say("  tail_nodes %d: %.1f us an iteration in %d intervals" % (t, 1e3 * ms[t], st.kernel_launches))
        S.close()
    assert ms[128] <= ms[0]

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


KT_OUTER_SPMV, KT_RESIDUAL = 1, 3


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


def test_product_class_is_the_product(gpu):
    """Unpreconditioned iterations form the scaled basis vector in the
    product's launch; with the product timed they are two launches."""
    import torch
    from torch.profiler import ProfilerActivity, profile
    say("[product_class_is_the_product]")
    n = (96, 96, 1)
    m = np.random.default_rng(2).standard_normal((n[0] * n[1], 3))
    m = torch.from_numpy(m / np.linalg.norm(m, axis=1, keepdims=True)).cuda()
    out, runs = [], []
    for cls in (0, KT_OUTER_SPMV):
        S = gpu.Solver(gpu.make_grid(2, n, 1.0 / n[0]), gpu.default_opts(krylov="gmres", max_iters=20))
        S.set_kernel_timing(cls)
        with profile(activities=[ProfilerActivity.CUDA]) as p:
            u, _, st = S.step(m, 0.1, 4e-4, check=False)
            torch.cuda.synchronize()
        names = [e.name for e in p.events()]
        count = [sum(k in x for x in names) for k in ("k_spmv_scaled", "k_spmv_outer")]
        say("  class %d: %d iterations, %s scaled and plain products" % (cls, st.iters, count))
        assert st.kernel_launches == (st.iters if cls else 0)
        out.append(u.cpu().numpy())
        runs.append(count)
        S.close()
    # (the trace may lose records, it invents none)
    assert runs[0][0] > 0 and runs[0][1] == 0
    assert runs[1][0] == 0 and runs[1][1] > 0
    assert np.array_equal(out[0], out[1])

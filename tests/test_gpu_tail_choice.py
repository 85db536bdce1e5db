"""GPU: which of the fused coarse cycles runs (opts.tail_nodes, stats.tail_level).

At the default bound the small levels go to a team and no level is the first
of a one-workgroup cycle; at any other bound the one-workgroup cycle runs up to
it (block Jacobi; Gauss-Seidel levels go to the team); and where the K-cycle makes the team's list too long it runs at the default
bound too.  Each is bit-identical to the levels one by one.
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


# (grid, options, bound, whether the one-workgroup cycle runs)
CASES = [
    ((64, 64, 1), dict(kcycle_depth=1, fine_operator="factored"), 128, False),
    ((64, 64, 1), dict(kcycle_depth=1, fine_operator="factored"), 127, True),
    ((64, 64, 1), dict(kcycle_depth=1, fine_operator="factored"), 129, True),
    ((64, 64, 1), dict(precision="fp32_amg"), 300, True),
    ((64, 64, 1), dict(smoother="mcgs"), 300, False),
    # six K-cycle levels by halves: about 1400 steps, past the longest list (1024)
    ((64, 64, 1), dict(npass=1, max_coarse=8, kcycle_depth=6), 128, True),
    ((64, 64, 1), dict(npass=1, max_coarse=8, kcycle_depth=6, precision="fp32_amg", nu_pre=0, nu_post=2), 128, True),
]


@pytest.mark.parametrize("case", CASES, ids=["%d-bound%d" % (k, c[2]) for k, c in enumerate(CASES)])
def test_one_workgroup_cycle_where_asked(gpu, case):
    import torch
    n, kw, bound, runs = case
    say("[one_workgroup_cycle_where_asked]", kw, bound)
    m = np.random.default_rng(17).standard_normal((n[0] * n[1], 3))
    m = torch.from_numpy(m / np.linalg.norm(m, axis=1, keepdims=True)).cuda()
    v = torch.from_numpy(np.random.default_rng(18).standard_normal(m.shape)).cuda()
    got = []
    for t in (bound, 0):
        S = gpu.Solver(gpu.make_grid(2, n, 1.0 / n[0]), gpu.default_opts(tail_nodes=t, **kw))
        u, s, st = S.step(m, 0.05, 2e-4)
        nodes = list(st.level_nodes[:st.levels])
        say("  bound %d: nodes %s, one workgroup from %d" % (t, nodes, st.tail_level))
        assert s == gpu.OK
        # the first level below the K-cycle levels (and level 1 of the per-node
        # grid level) from which none but the coarsest has more nodes
        first = max(kw.get("kcycle_depth", 0) + 1, 2 if "fine_operator" in kw else 1)
        while first < len(nodes) - 1 and nodes[first] > t:
            first += 1
        assert first <= len(nodes) - 2 or not t
        assert st.tail_level == (first if t and runs else 0)
        got.append((u.cpu().numpy(), S.precond(v).cpu().numpy()))
        S.close()
    assert np.isfinite(got[0][1]).all()
    assert np.array_equal(got[0][0], got[1][0]) and np.array_equal(got[0][1], got[1][1])

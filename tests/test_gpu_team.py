"""GPU: the small levels' cycle as one launch of a team of workgroups.

The team takes the steps of the per-level kernels with the same row products,
lane groups and orders of additions, so the preconditioner is bit-identical to
the one with the levels one by one (tail_nodes = 0), for every smoother, sweep
count and cycle, at level sizes around the wavefront, the lane group and the
team's size; also when two contexts launch teams at the same time.
"""
import sys
import threading

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


def _rough(n, seed):
    rng = np.random.default_rng(seed)
    m = rng.standard_normal((int(np.prod(n)), 3))
    return m / np.linalg.norm(m, axis=1, keepdims=True)


def _cuda(x):
    import torch
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


# (dim, n, options): one small coarse level above the coarsest; ragged grids; a
# level of about 2 MB; Gauss-Seidel; deep K-cycles, the deepest past the longest list
CASES = [
    (2, (16, 13, 1), dict(precision="fp64", nu_pre=0, nu_post=1)),
    (2, (16, 13, 1), dict(precision="fp32_amg", nu_pre=0, nu_post=0, kcycle_depth=1)),
    (2, (97, 61, 1), dict(precision="fp32_amg", nu_pre=2, nu_post=3, kcycle_depth=2)),
    (2, (320, 300, 1), dict(precision="fp64", kcycle_depth=1, fine_operator="factored", nu_pre=0, nu_post=2)),
    (3, (40, 37, 41), dict(precision="fp32_amg", fine_operator="factored", nu_pre=0, nu_post=2)),
    (3, (33, 17, 9), dict(precision="fp64", smoother="mcgs", kcycle_depth=1)),
    (2, (65, 64, 1), dict(precision="fp32_amg", smoother="mcgs", nu_pre=2, nu_post=0)),
    (2, (96, 96, 1), dict(precision="fp64", kcycle_depth=8, tail_nodes=1 << 20)),
    (2, (700, 650, 1), dict(precision="fp64", kcycle_depth=8, max_coarse=8)),
]


@pytest.mark.parametrize("case", CASES, ids=["%dd-%s-%d" % (c[0], "x".join(map(str, c[1])), k)
                                             for k, c in enumerate(CASES)])
def test_team_cycle_bit_identical(gpu, case):
    dim, n, kw = case
    say("[team_cycle_bit_identical]", n, kw)
    m = _rough(n, 11)
    g = gpu.make_grid(dim, n, 1.0 / n[0])
    S = [gpu.Solver(g, gpu.default_opts(**{**kw, "tail_nodes": t})) for t in (kw.get("tail_nodes", 128), 0)]
    for s in S:
        assert s.setup(_cuda(m), 0.05, 2e-4) == gpu.OK
    rng = np.random.default_rng(5)
    for _ in range(3):
        v = _cuda(rng.standard_normal(m.shape))
        a, b = (s.precond(v).cpu().numpy() for s in S)
        assert np.isfinite(a).all()
        assert np.array_equal(a, b), np.abs(a - b).max() / np.abs(b).max()
    for s in S:
        s.close()


def test_teams_at_the_same_time(gpu):
    """Nine contexts (more than XCDs) in threads of their own, each on its own
    stream: every one gives what it gives alone."""
    import torch
    say("[teams_at_the_same_time]")
    n, out, want = (48, 52, 1), {}, {}
    ms = [_rough(n, 100 + k) for k in range(9)]

    def one(k, res):
        st = torch.cuda.Stream()
        with torch.cuda.stream(st):
            S = gpu.Solver(gpu.make_grid(2, n), gpu.default_opts(rtol=1e-9, kcycle_depth=1), stream=st)
            m, nxt = torch.from_numpy(ms[k]).cuda(), None
            st.synchronize()
            for _ in range(4):
                nxt, s, _ = S.step(m, 0.1, 1e-3)
                assert s == gpu.OK
                m = nxt
            st.synchronize()
            res[k] = m.cpu().numpy()
            S.close()
    for k in range(9):
        one(k, want)
    th = [threading.Thread(target=one, args=(k, out)) for k in range(9)]
    for t in th:
        t.start()
    for t in th:
        t.join(60)
    assert sorted(out) == list(range(9))
    for k in range(9):
        assert np.array_equal(out[k], want[k]), k

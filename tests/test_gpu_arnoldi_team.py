"""GPU: the orthogonalization of short vectors in one launch of a team.

A step with it agrees with the step of the two-pass Gram-Schmidt (whose
kernels it does not touch): at odd and tiny lengths, at the length up to which
the team is taken (30720 entries) and past it, through restarts at the largest
restart length, preconditioned and not.  Both solve to a relative residual of
1e-11 of matrices of condition below 35 (1 + 8 dt / h^2), so the fields agree to 1e-9 and
iteration counts to one a cycle.
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
    ((2, 3, 1), "fgmres_amg", 32, 1e-2), ((9, 5, 1), "gmres", 32, 1e-2), ((9, 5, 1), "gmres", 3, 1e-2),
    ((33, 31, 1), "gmres", 32, 3e-3), ((64, 64, 1), "fgmres_amg", 30, 1e-3), ((160, 64, 1), "gmres", 32, 1e-4),
    ((161, 64, 1), "gmres", 32, 1e-4), ((21, 19, 23), "fgmres_amg", 5, 1e-3),
]


@pytest.mark.parametrize("n,krylov,restart,dt", CASES, ids=["%s-%s-%d" % ("x".join(map(str, c[0])), c[1], c[2])
                                                            for c in CASES])
def test_arnoldi_team(gpu, n, krylov, restart, dt):
    import torch
    say("[arnoldi_team]", n, krylov, restart)
    rng = np.random.default_rng(5)
    m = rng.standard_normal((int(np.prod(n)), 3))
    m /= np.linalg.norm(m, axis=1, keepdims=True)
    res = []
    for arnoldi in ("dcgs2", "cgs2"):
        S = gpu.Solver(gpu.make_grid(2 if n[2] == 1 else 3, n, 1.0 / n[0]),
                       gpu.default_opts(precision="fp64", krylov=krylov, restart=restart, arnoldi=arnoldi, rtol=1e-11,
                                        max_iters=400))
        out, s, st = S.step(torch.from_numpy(m).cuda(), 0.1, dt)
        assert s == gpu.OK
        res.append((out.cpu().numpy(), st.iters))
        S.close()
    d = np.abs(res[0][0] - res[1][0]).max()
    say("  iters", res[0][1], res[1][1], "diff %.2e" % d)
    assert d <= 1e-9
    assert abs(res[0][1] - res[1][1]) <= 1 + res[1][1] // restart


@pytest.mark.parametrize("n", [(3, 2, 1), (13, 5, 1), (64, 1, 1), (33, 31, 1), (9, 8, 7)],
                         ids=lambda n: "x".join(map(str, n)))
def test_scaled_product(gpu, n):
    """The unpreconditioned iteration's product with the scaling in it: the
    same values as the copy and the product apart (which captured graphs keep),
    so the steps are bit-identical, at rows around the wavefront."""
    import torch
    n = (n[0], max(n[1], 2), n[2])
    say("[scaled_product]", n)
    rng = np.random.default_rng(6)
    m = rng.standard_normal((int(np.prod(n)), 3))
    m /= np.linalg.norm(m, axis=1, keepdims=True)
    res = []
    for graphs in (0, 1):
        S = gpu.Solver(gpu.make_grid(2 if n[2] == 1 else 3, n, 1.0 / n[0]),
                       gpu.default_opts(precision="fp64", krylov="gmres", fine_operator="bsr", graphs=graphs, rtol=1e-10))
        for _ in range(2):
            out, s, st = S.step(torch.from_numpy(m).cuda(), 0.1, 1e-3)
            assert s == gpu.OK
        res.append((out.cpu().numpy(), st.iters))
        S.close()
    assert res[0][1] == res[1][1] and np.array_equal(res[0][0], res[1][0])

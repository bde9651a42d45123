"""Small particle counts of the particle model (fb_small.hip): the row forward,
the split adjoint and the rings cut into segments with halos, against the FP64
oracle at the edges of their rows, batches and segments, and against the
one-particle-per-lane kernels across the count where the choice changes."""
import numpy as np
import pytest

from oracle import ref
from paper_2505_04328_amd import workloads as wl
from tests.parity_util import (TOL, assert_grad, dump_to_paths, gpu_device, per_path_error, rel_err)

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev(oracle_lib):
    return gpu_device()


def _track(N, T):
    t = np.arange(N + 1) * (T / N)
    return np.stack([0.5 * np.sin(t), 0.3 * np.cos(t)], axis=1)


def _problem(N, **kw):
    T = kw.pop("T", 0.1 * N)
    return wl.feedback_problem(N=N, T=T, zd=_track(N, T), alpha=0.2, **kw)


# independent particles: rows of 16 lanes (batches of 16 steps, 16 particles per
# workgroup); rings: whole rings up to 32, segments of 16 own particles and 16
# steps beyond (forward), of 128 own and 128 steps beyond 256 (recursion)
SHAPES = [
    (17, 33, dict(nx=11, nv=3)), (1, 1, dict()), (16, 16, dict(init="uniform", nx=10, nv=9)),
    (255, 17, dict(nx=16, nv=16, eps=0.8)), (60, 12, dict(T=6.0, gamma=-0.6)),
    (7, 17, dict(np_=32, omega=0.7)), (5, 33, dict(np_=33, omega=0.7)),
    (3, 31, dict(np_=49, omega=0.7, cost="ellipse", init="ellipse")),
    (3, 16, dict(np_=256, omega=0.6, nx=12, nv=7)), (2, 140, dict(np_=257, omega=0.5)),
    (9, 20, dict(np_=300, omega=0.5, T=8.0, gamma=-0.5)),
]


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("case", range(len(SHAPES)))
def test_small_counts_match_oracle(dev, case, precision):
    from paper_2505_04328_amd import binding as B
    M, N, kw = SHAPES[case]
    p = _problem(N, **kw)
    print(case, precision, M, N, kw, flush=True)
    mu = wl.random_feedback_control(p, 4, 0.5)
    P = M * p.np
    z, lam, _, _, C = ref.fb_paths(p, 21, 2, 0, M, mu)
    J_ref, g_ref = ref.fb_cost_grad(p, M, 21, 2, mu)
    scale = ref.fb_grad_scale(p, M, 21, 2, mu)
    eng = B.FbEngine(p, M=M, seed=21, precision=precision, device=dev)
    dp, d = eng.path_dump(0, P)
    J = float(eng.forward(mu, it=2, dump=dp))
    eng.adjoint(mu, it=2, dump=dp)
    J2, g = eng.cost_grad(mu, it=2)
    Jc = float(eng.forward(mu, it=2, store=False))
    tol = TOL[precision]
    assert J == float(J2) == Jc
    assert rel_err(J, J_ref) <= tol["J"]
    assert_grad(g.cpu().numpy(), g_ref, scale, tol["g"])
    assert per_path_error(dump_to_paths(d["X"], P), z) <= tol["path"]
    assert per_path_error(dump_to_paths(d["lam"], P)[:, 1:], lam[:, 1:]) <= tol["path"]


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("M,more,kw", [(32768, 70000, dict()), (40, 400, dict(np_=300, omega=0.5)),
                                       (300, 3000, dict(np_=30, omega=0.5))])
def test_small_and_large_counts_agree_bitwise(dev, M, more, kw, precision):
    """The states and adjoint sources of the same particles do not depend on
    how many others run beside them: the trajectory of the first M of `more`
    realizations (lane kernels) is bitwise that of M alone (row kernels).  The
    adjoints do not depend on the count either."""
    from paper_2505_04328_amd import binding as B
    p = _problem(18, **kw)
    mu = wl.random_feedback_control(p, 3, 0.5)
    out = []
    for m in (M, more):
        eng = B.FbEngine(p, M=m, seed=5, precision=precision, device=dev)
        dp, d = eng.path_dump(0, M * p.np)
        eng.forward(mu, dump=dp)
        eng.adjoint(mu, dump=dp)
        out.append((d["X"].cpu().numpy(), d["lam"].cpu().numpy()[1:], d["cost"].cpu().numpy(),
                    eng.trajectory()[:, :, :M * p.np].cpu().numpy()))
    for a, b in zip(*out):
        np.testing.assert_array_equal(a, b)

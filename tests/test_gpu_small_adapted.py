"""Small particle counts on the jump-adapted grid (the row forward and the split
adjoint): against the FP64 oracle at the edges of their rows and batches, with
many jumps in an interval and particles past the jump stack, and bitwise against
the kernels of larger counts."""
import numpy as np
import pytest

from oracle import ref
from paper_2505_04328_amd import workloads as wl
from tests.parity_util import TOL, assert_grad, dump_to_paths, gpu_device, per_path_error, rel_err

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev(oracle_lib):
    return gpu_device()


def _problem(N, **kw):
    T = kw.pop("T", 0.1 * N)
    t = np.arange(N + 1) * (T / N)
    zd = np.stack([0.5 * np.sin(t), 0.3 * np.cos(t)], axis=1)
    return wl.feedback_problem(N=N, T=T, zd=zd, alpha=0.2, grid="adapted", **kw)


# batches of 16 intervals and 16 particles per workgroup (forward), batches of 8
# sub-steps (recursion); up to 16 expected jumps are split, and at 15.9 about one
# particle of 20000 is past the stack's 32
SHAPES = [
    (1, 1, dict()), (17, 16, dict(init="uniform")), (16, 17, dict(nx=11, nv=3)),
    (255, 33, dict(nx=16, nv=16, eps=0.8)), (20000, 8, dict(T=3.0, beta=88.0, gamma=0.9)),
    (2000, 50, dict(T=5.0)), (257, 7, dict(T=2.0, gamma=-0.6, nx=4, nv=10)),
]


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("case", range(len(SHAPES)))
def test_small_adapted_counts_match_oracle(dev, case, precision):
    from paper_2505_04328_amd import binding as B
    M, N, kw = SHAPES[case]
    p = _problem(N, **kw)
    print(case, precision, M, N, kw, f"jumps per particle {p.rate * p.T:.2f}", flush=True)
    mu = wl.random_feedback_control(p, 4, 0.5)
    z, lam, _, _, _ = ref.fb_paths(p, 21, 2, 0, M, mu)
    J_ref, g_ref = ref.fb_cost_grad(p, M, 21, 2, mu)
    scale = ref.fb_grad_scale(p, M, 21, 2, mu)
    eng = B.FbEngine(p, M=M, seed=21, precision=precision, device=dev)
    dp, d = eng.path_dump(0, M)
    J = float(eng.forward(mu, it=2, dump=dp))
    ga = eng.adjoint(mu, it=2, dump=dp).cpu().numpy()
    J2, g = eng.cost_grad(mu, it=2)
    g = g.cpu().numpy()
    Jc = float(eng.forward(mu, it=2, store=False))
    tol = TOL[precision]
    assert J == float(J2) == Jc
    np.testing.assert_array_equal(g, ga)
    assert rel_err(J, J_ref) <= tol["J"]
    assert_grad(g, g_ref, scale, tol["g"])
    assert per_path_error(dump_to_paths(d["X"], M), z) <= tol["path"]
    assert per_path_error(dump_to_paths(d["lam"], M)[:, 1:], lam[:, 1:]) <= tol["path"]


# (the larger count: the forward with the sub-steps after a jump in rows)
@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("M,N,T", [(28672, 18, 1.8), (28673, 2, 0.1), (49152, 1, 0.05),
                                   (20000, 30, 1.0)])
def test_small_and_large_adapted_counts_agree_bitwise(dev, M, N, T, precision):
    from paper_2505_04328_amd import binding as B
    p = _problem(N, T=T)
    mu = wl.random_feedback_control(p, 3, 0.5)
    out = []
    for m in (M, 140000):
        eng = B.FbEngine(p, M=m, seed=5, precision=precision, device=dev)
        dp, d = eng.path_dump(0, M)
        eng.forward(mu, dump=dp)
        eng.adjoint(mu, dump=dp)
        out.append((d["X"].cpu().numpy(), d["lam"].cpu().numpy()[1:], d["cost"].cpu().numpy(),
                    eng.trajectory()[:, :, :M].cpu().numpy()))
    for a, b in zip(*out):
        np.testing.assert_array_equal(a, b)

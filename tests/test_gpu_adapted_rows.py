"""The jump-adapted adjoint that evaluates the sub-steps after a jump in rows of
16 lanes, against the FP64 oracle: blocks with and without a particle past the
jump stack in one launch, several jumps in an interval, shape-function grids
narrower and wider than a row's compiled widths, the shortest sweeps."""
import numpy as np
import pytest

from oracle import ref
from paper_2505_04328_amd import workloads as wl
from tests.parity_util import TOL, assert_grad, dump_to_paths, gpu_device, per_path_error, rel_err

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev(oracle_lib):
    return gpu_device()


# (particles, steps, problem): jumps per interval rate T / N <= 0.1 in both precisions but
# for the last, which FP64 alone takes in rows
CASES = [
    (2000, 500, dict(T=10.5)),  # 19 jumps per particle: some blocks past the stack's 32
    (700, 300, dict(T=12.0, nx=13, nv=7, eps=0.7, gamma=-0.7)),
    (300, 1, dict(T=0.05)), (257, 2, dict(T=0.1, nx=4, nv=12)),
    (300, 60, dict(T=9.0, nx=9, nv=10)),
]


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_adapted_adjoint_in_rows_matches_oracle(dev, case, precision):
    from paper_2505_04328_amd import binding as B
    M, N, kw = CASES[case]
    kw = dict(kw)
    T = kw["T"]
    t = np.arange(N + 1) * (T / N)
    zd = np.stack([0.5 * np.sin(t), 0.3 * np.cos(t)], axis=1)
    p = wl.feedback_problem(N=N, zd=zd, alpha=0.2, grid="adapted", **kw)
    print(case, precision, M, N, kw, f"jumps per interval {p.rate * p.dt:.3f}", flush=True)
    mu = wl.random_feedback_control(p, 4, 0.5)
    z, lam, _, _, _ = ref.fb_paths(p, 31, 2, 0, M, mu)
    J_ref, g_ref = ref.fb_cost_grad(p, M, 31, 2, mu)
    scale = ref.fb_grad_scale(p, M, 31, 2, mu)
    eng = B.FbEngine(p, M=M, seed=31, precision=precision, device=dev)
    dp, d = eng.path_dump(0, M)
    eng.forward(mu, it=2, dump=dp)
    ga = eng.adjoint(mu, it=2, dump=dp).cpu().numpy()
    J, g = eng.cost_grad(mu, it=2)
    g = g.cpu().numpy()
    tol = TOL[precision]
    np.testing.assert_array_equal(g, ga)
    assert rel_err(float(J), J_ref) <= tol["J"]
    assert_grad(g, g_ref, scale, tol["g"])
    assert per_path_error(dump_to_paths(d["X"], M), z) <= tol["path"]
    assert per_path_error(dump_to_paths(d["lam"], M)[:, 1:], lam[:, 1:]) <= tol["path"]

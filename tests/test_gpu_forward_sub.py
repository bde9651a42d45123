"""The jump-adapted forward that evaluates the sub-steps after a jump in rows of
16 lanes, four particles at a time: against the FP64 oracle at few and many jumps
per interval (more than four of a wave, several of one particle, past the jump
stack), grids narrower and wider than the compiled widths, the shortest sweeps."""
import numpy as np
import pytest

from oracle import ref
from paper_2505_04328_amd import workloads as wl
from tests.parity_util import TOL, dump_to_paths, gpu_device, per_path_error, rel_err

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev(oracle_lib):
    return gpu_device()


# (precision, particles, dumped from, problem): FP64 above the small counts, FP32 from
# 131072 particles on
CASES = [
    ("fp64", 28673, 28600, dict(N=20, T=1.0, nx=4, nv=10)),
    ("fp64", 28800, 28000, dict(N=8, T=3.0, beta=88.0)),
    ("fp64", 30000, 0, dict(N=50, T=9.0, beta=50.0, nx=16, nv=13, eps=0.8)),
    ("fp64", 28700, 28672, dict(N=1, T=0.3)),
    ("fp32", 131073, 130900, dict(N=12, T=2.0, gamma=-0.6)),
    ("fp32", 131072, 131000, dict(N=2, T=0.2, nx=12, nv=7, eps=0.8)),
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_forward_sub_steps_in_rows_match_oracle(dev, case):
    from paper_2505_04328_amd import binding as B
    precision, M, m0, kw = CASES[case]
    N, T = kw["N"], kw["T"]
    t = np.arange(N + 1) * (T / N)
    zd = np.stack([0.5 * np.sin(t), 0.3 * np.cos(t)], axis=1)
    p = wl.feedback_problem(zd=zd, alpha=0.2, grid="adapted", **kw)
    print(case, precision, M, kw, f"jumps per interval {p.rate * p.dt:.3f}", flush=True)
    mu = wl.random_feedback_control(p, 4, 0.5)
    count = min(M - m0, 500)
    z, _, _, _, C = ref.fb_paths(p, 31, 2, m0, count, mu)
    J_ref, _ = ref.fb_cost_grad(p, M, 31, 2, mu, grad=False)
    eng = B.FbEngine(p, M=M, seed=31, precision=precision, device=dev)
    dp, d = eng.path_dump(m0, count)
    J = float(eng.forward(mu, it=2, dump=dp))
    Jc = float(eng.forward(mu, it=2, store=False))
    tol = TOL[precision]
    assert J == Jc
    assert rel_err(J, J_ref) <= tol["J"]
    assert per_path_error(dump_to_paths(d["X"], count), z) <= tol["path"]
    np.testing.assert_allclose(d["cost"].cpu().numpy(), C, rtol=0, atol=tol["path"] * np.abs(C).max())

"""The particle model's line search where several trials share a launch: the
iterates against the FP64 oracle with more trials than one launch takes, the
limit on the trials inside a launch, and the same decisions whatever the number
of particles lets a launch take."""
import numpy as np
import pytest

from oracle import ref
from paper_2505_04328_amd import workloads as wl
from tests.parity_util import TOL, gpu_device, norm_err, rel_err

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev(oracle_lib):
    return gpu_device()


# particles: 4, 3, 2 trials of a launch, and one
@pytest.mark.parametrize("M,grid,zeta0", [(400, "fixed", 3000.0), (2500, "adapted", 400.0),
                                          (3000, "fixed", 400.0), (6000, "adapted", 400.0)])
def test_trials_sharing_a_launch_match_oracle(dev, M, grid, zeta0):
    from paper_2505_04328_amd import binding as B
    p = wl.feedback_problem(N=20, T=2.0, alpha=0.05, grid=grid)
    mu0 = np.zeros((p.N, p.L))
    mu_ref, logs_ref, n_ref = ref.fb_optimize(p, M, 9, 0, mu0, n_max=3, zeta0=zeta0)
    print(M, grid, [b["backtracks"] for b in logs_ref], flush=True)
    assert n_ref == 3 and logs_ref[0]["backtracks"] >= 4
    eng = B.FbEngine(p, M=M, seed=9, precision="fp64", device=dev)
    mu, logs = eng.optimize(mu0, n_max=3, zeta0=zeta0)
    tol = TOL["fp64"]
    assert len(logs) == 3
    for a, b in zip(logs, logs_ref):
        assert a["backtracks"] == b["backtracks"] and a["zeta"] == b["zeta"]
        assert rel_err(a["J"], b["J"]) <= tol["J"]
    assert norm_err(mu.cpu().numpy(), mu_ref) <= 10 * tol["g"]
    # one trial fewer than the first iteration needs fails, exactly as many succeed
    need = logs[0]["backtracks"] + 1
    with pytest.raises(B.JdError):
        eng.optimize(mu0, n_max=1, zeta0=zeta0, max_backtracks=need - 1)
    _, one = eng.optimize(mu0, n_max=1, zeta0=zeta0, max_backtracks=need)
    assert one[0]["backtracks"] == logs[0]["backtracks"]
    assert one[0]["J_new"] == logs[0]["J_new"] and one[0]["E"] == logs[0]["E"]

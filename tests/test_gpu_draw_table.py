"""The FP64 Box-Muller transform by tables (jd_device.hpp: bm_radius, bm_cos,
bm_sin) against the transform in extended precision, over every subinterval of
the logarithm table and every tabulated angle, the ends of the unit interval
among them."""
import numpy as np
import pytest

from paper_2505_04328_amd import workloads as wl
from tests.parity_util import gpu_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [1, 2])
def test_fp64_normals_match_extended_precision(d):
    dev = gpu_device()
    from paper_2505_04328_amd import binding as B
    M, K, seed = 20000, 60, 77
    p = wl.general_problem(d, K, seed=d, lam=5.0)
    eng = B.Engine(p, M=M, seed=seed, precision="fp64", device=dev)
    zw, zj, _ = (t.cpu().numpy() for t in eng.draws(0, M, 0, K))
    ctr = np.zeros((M * K, 4), np.uint32)
    ctr[:, 0] = np.repeat(np.arange(M), K)
    ctr[:, 1] = np.tile(np.arange(K), M)
    w = B.philox(seed, ctr, device=dev).reshape(-1, 4) >> 8 | 1
    ld = np.longdouble
    pi = ld("3.14159265358979323846264338327950288")
    for i in range(d):
        a, b = w[:, 2 * i], w[:, 2 * i + 1]
        # every table entry is used: exponents and subintervals of the uniform's
        # binary form, angles by their nearest of 256
        hi = (a.astype(np.float64).view(np.uint64) >> np.uint64(32)).astype(np.int64) - 0x3FE60000
        assert len(np.unique(hi >> 13 & 127)) == 128 and len(np.unique((b + 0x8000) >> 16 & 255)) == 256
        r = np.sqrt(-2 * np.log(a.astype(ld) / 2 ** 24))
        th = 2 * pi * (b.astype(ld) / 2 ** 24)
        for z, ref in ((zw, r * np.cos(th)), (zj, r * np.sin(th))):
            err = np.abs(z[:, :, i].reshape(-1).astype(ld) - ref)
            # radius, branch and product are each within 1.6 units of 2^-53 of
            # their value, and |Z| <= r <= 5.8: 4.8 2^-53 r
            assert np.all(err <= 4.8 * 2.0 ** -53 * r), float(np.max(err / r))
            # a rounding error per factor, uniform: an RMS of about 2^-53 |r| / sqrt(3) each
            assert np.sqrt(np.mean(err ** 2)) <= 1.2e-16

// Device side of the gradient iteration's line search (Section 5, eq.
// Stochastic_Armijo, Algorithm 5.4), run by the cost reductions of both models.
#pragma once

#include "jd_device.hpp"
#include "jd_launch.hpp"

namespace jd {

// Sufficient decrease J(u - zeta g) <= J(u) - c zeta ||g||^2_L2 on the same
// draws (a non-finite trial cost is rejected), trial by trial in their order; the
// first that holds records ||u' - u||^2_L2, moves u to u', writes the iteration's
// log entry and opens the next phase of the device-driven iteration (see LsArmijo).
// All TPB threads of one block; Jt: the trials' costs, in LDS, as thread 0 wrote
// them; sh: TPB doubles of LDS.
template <int TPB>
__device__ __forceinline__ void armijo_step(WsHeader* hdr, const LsTail& t, const double* Jt,
                                            double* sh) {
    __shared__ int acc;
    const LsArmijo& ls = t.ls;
    if (threadIdx.x == 0) {
        const double J = hdr->J, g2 = hdr->gnorm2;
        int i = 0;
        while (i < t.trials && !(isfinite(Jt[i]) && Jt[i] <= J - ls.c_armijo * t.zeta[i] * g2))
            ++i;
        acc = i;
        hdr->accept = i < t.trials;
        hdr->J_trial = Jt[i < t.trials ? i : t.trials - 1];
        if (i == t.trials) {
            if (ls.j + i >= ls.max_backtracks) {
                hdr->ls_status = JD_ELINESEARCH;
                hdr->ls_phase = kLsStop;
            } else {
                hdr->ls_phase = ls_phase(ls.n, ls.j + i);
            }
        }
    }
    __syncthreads();
    const int i = acc;
    if (i == t.trials)
        return;
    const double* ut = t.ut + (size_t)i * t.nd;
    double e = 0.0;
    for (int q = threadIdx.x; q < t.nd; q += TPB) {
        const double x = ut[q], r = x - t.u[q];
        e += r * r;
        t.u[q] = x;
    }
    e = block_sum<TPB>(e, sh);
    if (threadIdx.x == 0) {
        const double E2 = ls.dt * e;
        hdr->E2 = E2;
        LsLog& L = t.ring[ls.n % kLsLogCap];
        L.J = hdr->J;
        L.gnorm2 = hdr->gnorm2;
        L.zeta = t.zeta[i];
        L.J_new = Jt[i];
        L.E2 = E2;
        L.iter = ls.iter;
        L.backtracks = ls.j + i;
        L.n = ls.n;
        hdr->ls_done = ls.n + 1;
        if (ls.n + 1 >= ls.n_max || sqrt(E2) <= ls.tol) {
            hdr->ls_status = kLsDone;
            hdr->ls_phase = kLsStop;
        } else {
            hdr->ls_phase = ls_phase(ls.n + 1, -1);
        }
    }
}

// After the gradient of iteration n (one thread): on to trial (n, 0), or stop
// with JD_ENONFINITE.
__device__ __forceinline__ void ls_after_grad_step(WsHeader* hdr, int n) {
    if (hdr->ls_phase == ls_phase(n, -1)) {
        if (hdr->nonfinite) {
            hdr->ls_status = JD_ENONFINITE;
            hdr->ls_phase = kLsStop;
        } else {
            hdr->ls_phase = ls_phase(n, 0);
        }
    }
}

}  // namespace jd

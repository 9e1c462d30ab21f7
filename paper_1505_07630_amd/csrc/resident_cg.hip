// The resident standard-CG kernels (resident.hpp) and their choice.
#include "resident.hpp"
#include "resident_host.hpp"

namespace fvpcg {

namespace {

// A team on its own launch: member r is workgroup r.
template <int RPT, int WT, typename CI, bool JAC, bool ONE>
__global__ __launch_bounds__(kResBsCg) void k_res_cg(ResSystem sys, ResTeam t, ResOut* out) {
    __shared__ double lds[ResLds<kResBsCg, RPT, ONE>::doubles];
    __shared__ int s_ok;
    if (threadIdx.x == 0) s_ok = 1;
    t.rank = (int)blockIdx.x;
    t.ok = &s_ok;
    if (ONE) {
        t.size = 1;
        __syncthreads();
    } else if (!team_meet(t)) {
        return;
    }
    resident_cg<RPT, WT, CI, JAC, ONE>(sys, t, lds, out);
}

template <int RPT, int WT, bool ONE>
ResKernel pick_form(bool col16, bool jac) {
    if constexpr (RPT <= 3)
        if (!col16) return jac ? k_res_cg<RPT, WT, int, true, ONE> : k_res_cg<RPT, WT, int, false, ONE>;
    return jac ? k_res_cg<RPT, WT, int16_t, true, ONE> : k_res_cg<RPT, WT, int16_t, false, ONE>;
}

template <int WT>
ResKernel pick_rpt(const ResPlan& p, bool col16, bool jac) {
    if (p.one) return p.rpt == 1 ? pick_form<1, WT, true>(col16, jac) : pick_form<2, WT, true>(col16, jac);
    if (p.rpt == 1) return pick_form<1, WT, false>(col16, jac);
    if constexpr (WT <= 6) {
        if (p.rpt == 3) return pick_form<3, WT, false>(col16, jac);
        if (p.rpt == 4) return pick_form<4, WT, false>(col16, jac);
    }
    return pick_form<2, WT, false>(col16, jac);
}

}  // namespace

ResKernel res_kernel_cg(const ResPlan& p, int wt, bool col16, bool jac) {
    if (wt == 4) return pick_rpt<4>(p, col16, jac);
    if (wt == 6) return pick_rpt<6>(p, col16, jac);
    return pick_rpt<8>(p, col16, jac);
}

}  // namespace fvpcg

// The resident mixed-precision kernels (resident.hpp) and their choice.
#include "resident.hpp"
#include "resident_host.hpp"

namespace fvpcg {

namespace {

// A team on its own launch.
template <int RPT, int WT, typename CI>
__global__ __launch_bounds__(kResBsMixed) void k_res_pipe32(PipeVec<float> a, int n, int iters, ResTeam t, DevState* st,
                                                            DevState* st_skip) {
    __shared__ float lds[4 * RPT * kResBsMixed];
    __shared__ int s_ok;
    if (threadIdx.x == 0) s_ok = 1;
    t.rank = (int)blockIdx.x;  // numbered by XCD (res_rank) 3% slower here
    t.ok = &s_ok;
    t.queued = false;
    if (st->done || st_skip->done) return;  // as every member sees them
    if (!team_meet(t)) {
        if (threadIdx.x == 0) st_skip->done = kResNoTeam;
        return;
    }
    resident_pipe32<RPT, WT, CI>(a, n, iters, t, st, st_skip, lds);
}

template <int WT, typename CI>
ResMixedKernel pick_rpt(int rpt) {
    switch (rpt) {
        case 1: return k_res_pipe32<1, WT, CI>;
        case 2: return k_res_pipe32<2, WT, CI>;
        case 4: return k_res_pipe32<4, WT, CI>;
        default: break;
    }
    if constexpr (WT <= 6 && sizeof(CI) == 2) return rpt == 6 ? k_res_pipe32<6, WT, CI> : k_res_pipe32<8, WT, CI>;
    return nullptr;
}

}  // namespace

ResMixedKernel res_kernel_mixed(int rpt, int wt, bool col16) {
    if (wt == 4) return col16 ? pick_rpt<4, int16_t>(rpt) : pick_rpt<4, int>(rpt);
    if (wt == 6) return col16 ? pick_rpt<6, int16_t>(rpt) : pick_rpt<6, int>(rpt);
    return col16 ? pick_rpt<8, int16_t>(rpt) : pick_rpt<8, int>(rpt);
}

}  // namespace fvpcg

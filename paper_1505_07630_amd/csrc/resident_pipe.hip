// The resident pipelined-CG kernels (resident.hpp) and their choice.
#include "resident.hpp"
#include "resident_host.hpp"

namespace fvpcg {

namespace {

// A team on its own launch.
template <int RPT, int WT, typename CI, bool JAC, bool LIT, bool ONE>
__global__ __launch_bounds__(kResBsPipe) void k_res_pipe(ResSystem sys, ResTeam t, ResOut* out) {
    __shared__ double lds[ResLds<kResBsPipe, RPT, ONE>::doubles];
    __shared__ int s_ok;
    if (threadIdx.x == 0) s_ok = 1;
    t.rank = res_rank((int)blockIdx.x, t.size);
    t.ok = &s_ok;
    t.queued = false;
    if (ONE) {
        t.rank = 0;
        t.size = 1;
        __syncthreads();
    } else if (!team_meet(t)) {
        return;
    }
    resident_pipe<RPT, WT, CI, JAC, LIT, ONE>(sys, t, lds, out);
}

// Many systems in one launch: workgroup b works through its list of (system,
// rank, team size, slot offset), all lists in one global order, so the first
// unfinished system always has its whole team.
template <int RPT, int WT, typename CI, bool JAC>
__global__ __launch_bounds__(kResBsPipe) void k_res_batch_pipe(ResSystem sys, ResTeam t, ResBatch bt) {
    __shared__ double lds[ResLds<kResBsPipe, RPT, false>::doubles];
    __shared__ int s_ok;
    if (threadIdx.x == 0) s_ok = 1;
    t.rank = (int)blockIdx.x;
    t.ok = &s_ok;
    if (!team_meet(t)) return;
    const int end = bt.list[blockIdx.x + 1];
    for (int i = bt.list[blockIdx.x]; i < end; ++i) {
        const int4 task = bt.tasks[i];
        ResTeam tm = t;
        tm.rank = task.y;
        tm.size = task.z;
        tm.slots = t.slots + (size_t)kResBufs * kResSums * task.w;
        tm.k = 0;
        tm.queued = true;
        sys.c0 = bt.cell_off[task.x];
        sys.c1 = bt.cell_off[task.x + 1];
        if (sys.c0 == sys.c1) {  // no rows: b = 0
            if (threadIdx.x == 0) bt.out[task.x] = ResOut{0.0, 0.0, 0.0, 0.0, 0, 0, 0, FVPCG_OK, 1, 1};
            continue;
        }
        resident_pipe<RPT, WT, CI, JAC, false, false>(sys, tm, lds, bt.out + task.x);
        __syncthreads();
        if (!s_ok) return;
    }
}

template <int RPT, int WT, bool ONE>
ResKernel pick_form(bool col16, bool jac, bool lit) {
    if constexpr (RPT <= 4)
        if (lit) return col16 ? k_res_pipe<RPT, WT, int16_t, true, true, ONE> : k_res_pipe<RPT, WT, int, true, true, ONE>;
    if constexpr (RPT <= 6)
        if (!col16) return jac ? k_res_pipe<RPT, WT, int, true, false, ONE> : k_res_pipe<RPT, WT, int, false, false, ONE>;
    return jac ? k_res_pipe<RPT, WT, int16_t, true, false, ONE> : k_res_pipe<RPT, WT, int16_t, false, false, ONE>;
}

template <int WT>
ResKernel pick_rpt(const ResPlan& p, bool col16, bool jac, bool lit) {
    if (p.one) {
        if (p.rpt == 1) return pick_form<1, WT, true>(col16, jac, lit);
        if (p.rpt == 2) return pick_form<2, WT, true>(col16, jac, lit);
        return pick_form<4, WT, true>(col16, jac, lit);
    }
    if (p.rpt == 1) return pick_form<1, WT, false>(col16, jac, lit);
    if (p.rpt == 2) return pick_form<2, WT, false>(col16, jac, lit);
    if (p.rpt == 3) return pick_form<3, WT, false>(col16, jac, lit);
    if constexpr (WT <= 6) {
        if (p.rpt == 6) return pick_form<6, WT, false>(col16, jac, lit);
        if (p.rpt == 8) return pick_form<8, WT, false>(col16, jac, lit);
    }
    return pick_form<4, WT, false>(col16, jac, lit);
}

}  // namespace

ResKernel res_kernel_pipe(const ResPlan& p, int wt, bool col16, bool jac) {
    const bool lit = p.method == FVPCG_PIPECG_LITERAL;
    if (wt == 4) return pick_rpt<4>(p, col16, jac, lit);
    if (wt == 6) return pick_rpt<6>(p, col16, jac, lit);
    return pick_rpt<8>(p, col16, jac, lit);
}

namespace {

template <int WT>
ResBatchKernel pick_batch(int rpt, bool col16, bool jac) {
    if constexpr (WT <= 6)
        if (rpt == 8) return jac ? k_res_batch_pipe<8, WT, int16_t, true> : k_res_batch_pipe<8, WT, int16_t, false>;
    if (rpt == 4) {
        if (col16) return jac ? k_res_batch_pipe<4, WT, int16_t, true> : k_res_batch_pipe<4, WT, int16_t, false>;
        return jac ? k_res_batch_pipe<4, WT, int, true> : k_res_batch_pipe<4, WT, int, false>;
    }
    if (col16) return jac ? k_res_batch_pipe<2, WT, int16_t, true> : k_res_batch_pipe<2, WT, int16_t, false>;
    return jac ? k_res_batch_pipe<2, WT, int, true> : k_res_batch_pipe<2, WT, int, false>;
}

}  // namespace

ResBatchKernel res_batch_pipe(int rpt, int wt, bool col16, bool jac) {
    if (wt == 4) return pick_batch<4>(rpt, col16, jac);
    if (wt == 6) return pick_batch<6>(rpt, col16, jac);
    return pick_batch<8>(rpt, col16, jac);
}

}  // namespace fvpcg

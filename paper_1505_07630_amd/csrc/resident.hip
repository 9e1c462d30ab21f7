// Host side of the resident solves (resident.hpp): which systems take that
// path, its launch, and what to do when the team does not come together.
#include <cstdlib>

#include <mutex>

#include "resident.hpp"
#include "resident_host.hpp"

namespace fvpcg {

namespace {

// A team on its own launch: member r is workgroup r.
template <int RPT, int WT, typename CI, bool JAC, bool ONE>
__global__ __launch_bounds__(kResBs) void k_res_pipe(ResSystem sys, ResTeam t, ResOut* out) {
    __shared__ double lds[ResLds<RPT, ONE>::doubles];
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
    resident_pipe<RPT, WT, CI, JAC, ONE>(sys, t, lds, out);
}

// Sentinels into the slots, the rendezvous word, abort flag and result cleared.
__global__ void k_res_reset(double* slots, int count, unsigned* meet, int* abort_flag, ResOut* out) {
    const int i = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (i < count) slots[i] = __longlong_as_double((long long)kResSentinel);
    if (i == 0) {
        *meet = 0u;
        *abort_flag = 0;
        out->ok = 0;
    }
}

using ResKernel = void (*)(ResSystem, ResTeam, ResOut*);

template <int RPT, int WT, bool ONE>
ResKernel pick_pipe(bool col16, bool jac) {
    if (col16) return jac ? k_res_pipe<RPT, WT, int16_t, true, ONE> : k_res_pipe<RPT, WT, int16_t, false, ONE>;
    return jac ? k_res_pipe<RPT, WT, int, true, ONE> : k_res_pipe<RPT, WT, int, false, ONE>;
}

template <int WT>
ResKernel pick_pipe_rpt(const ResPlan& p, bool col16, bool jac) {
    if (p.one) {
        if (p.rpt == 1) return pick_pipe<1, WT, true>(col16, jac);
        if (p.rpt == 2) return pick_pipe<2, WT, true>(col16, jac);
        return pick_pipe<4, WT, true>(col16, jac);
    }
    switch (p.rpt) {
        case 1: return pick_pipe<1, WT, false>(col16, jac);
        case 2: return pick_pipe<2, WT, false>(col16, jac);
        case 3: return pick_pipe<3, WT, false>(col16, jac);
        case 4: return pick_pipe<4, WT, false>(col16, jac);
        default: break;
    }
    if constexpr (WT <= 6) {
        if (p.rpt == 6) return pick_pipe<6, WT, false>(col16, jac);
        return pick_pipe<8, WT, false>(col16, jac);
    }
    return nullptr;
}

ResKernel pick_kernel(const ResPlan& p, int wt, bool col16, bool jac) {
    if (wt == 4) return pick_pipe_rpt<4>(p, col16, jac);
    if (wt == 6) return pick_pipe_rpt<6>(p, col16, jac);
    return pick_pipe_rpt<8>(p, col16, jac);
}

constexpr int kMaxDevices = 64;
struct DeviceInfo {
    std::once_flag once;
    std::mutex teams;
    int cus = 0;
    double ticks_per_ms = 0;
};
DeviceInfo g_dev[kMaxDevices];

const DeviceInfo& device_info(int dev) {
    DeviceInfo& d = g_dev[dev];
    std::call_once(d.once, [&] {
        int khz = 0;
        if (hipDeviceGetAttribute(&d.cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) d.cus = 0;
        if (hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, dev) != hipSuccess) khz = 0;
        (void)hipGetLastError();
        d.ticks_per_ms = (double)khz;
    });
    return d;
}

}  // namespace

std::mutex* resident_teams(int device) {
    return device >= 0 && device < kMaxDevices ? &g_dev[device].teams : nullptr;
}

// Up to 2,048 cells one workgroup holds the system and exchanges through LDS
// (no rendezvous, no device-wide reduction).  Above that a team takes the
// tiles of the launch-per-iteration kernels, at most kResMaxTeam workgroups
// of up to kResMaxRpt rows per thread: 1,048,576 cells, as many as registers
// and LDS hold.  Unpacked int32 columns leave room for 6 rows per thread,
// rows of more than 6 slots for 4, rows of more than 8 slots for none.
ResPlan resident_plan(const fvpcg_mesh* m) {
    ResPlan p;
    const char* env = getenv("FVPCG_RESIDENT");
    if (env && env[0] == '0') return p;
    if (m->WT > 8 || m->n < 1 || m->device < 0 || m->device >= kMaxDevices) return p;
    const int tiles = (m->n + kResBs - 1) / kResBs;
    if (tiles <= 4) {
        p.one = true;
        p.size = 1;
        p.rpt = tiles <= 2 ? tiles : 4;
        return p;
    }
    const int g = std::min(tiles, kResMaxTeam);  // geom_for's workgroups
    int rpt = (tiles + g - 1) / g;
    if (rpt == 5 || rpt == 7) ++rpt;
    if (rpt > (m->WT > 6 ? 4 : m->col16 ? kResMaxRpt : 6) || g > device_info(m->device).cus) return p;
    p.size = g;
    p.rpt = rpt;
    return p;
}

int resident_solve(const fvpcg_matrix* A, const ResPlan& plan, const ResWork& w, const double* b, double* x, double tol,
                   int maxit, bool jac, hipStream_t s, fvpcg_stats* stats, bool* done) {
    *done = false;
    const fvpcg_mesh* m = A->mesh;
    const DeviceInfo& info = device_info(m->device);
    if (info.ticks_per_ms <= 0) return FVPCG_OK;
    std::unique_lock<std::mutex> lock(g_dev[m->device].teams, std::defer_lock);
    if (!plan.one && !lock.try_lock()) return FVPCG_OK;  // another team has the GPU
    ResSystem sys{m->col16 ? (const void*)m->col16 : (const void*)m->col, A->val, jac ? A->val_cs : A->val, A->d, b, x,
                  w.e0, w.e1, (size_t)m->n, 0, m->n, tol, maxit};
    ResOut host{};
    ResOut* out = w.pinned ? w.pinned : w.out;
    if (w.pinned) w.pinned->ok = 0;
    if (!plan.one) {
        const int count = (int)res_slots(plan.size);
        hipLaunchKernelGGL(k_res_reset, dim3((count + 255) / 256), dim3(256), 0, s, w.slots, count, w.meet, w.abort_flag,
                           out);
    }
    const char* env = getenv("FVPCG_RESIDENT_MEET_MS");
    const double meet_ms = env && *env ? std::max(0.0, atof(env)) : kResMeetMs;
    ResTeam t{0, plan.size, w.slots, w.meet, w.abort_flag, nullptr,
              (unsigned long long)(info.ticks_per_ms * meet_ms), (unsigned long long)(info.ticks_per_ms * kResSpinMs),
              0};
    ResKernel k = pick_kernel(plan, m->WT, m->col16 != nullptr, jac);
    hipLaunchKernelGGL(k, dim3(plan.size), dim3(kResBs), 0, s, sys, t, out);
    FV_LAUNCHED();
    if (!w.pinned) FV_HIP(hipMemcpyAsync(&host, w.out, sizeof(ResOut), hipMemcpyDeviceToHost, s));
    FV_HIP(hipStreamSynchronize(s));
    if (w.pinned) host = *w.pinned;
    if (!host.ok) return FVPCG_OK;  // the team did not come together: x holds a valid start
    *done = true;
    if (stats) {
        stats->iters = host.iter;
        stats->outer_iters = 0;
        stats->status = host.status;
        stats->b_norm = host.bnorm;
        stats->r0_norm = host.r0norm;
        stats->rel_res = host.bnorm > 0 ? sqrt(host.rho) / host.bnorm : 0.0;
        stats->true_rel_res = host.bnorm > 0 ? sqrt(host.true_rr) / host.bnorm : 0.0;
        stats->device_ms = (double)host.ticks / info.ticks_per_ms;
        stats->iter_ms = (double)host.it_ticks / info.ticks_per_ms;
    }
    return host.status;
}

}  // namespace fvpcg

// Host side of the resident solves (resident.hpp): which systems take that
// path, its launch, and what to do when the team does not come together.
#include <atomic>
#include <chrono>
#include <cstdlib>
#include <mutex>

#include "resident.hpp"
#include "resident_host.hpp"

namespace fvpcg {

namespace {

// Sentinels into the slots, the rendezvous word, abort flag and results cleared.
__global__ void k_res_reset(double* slots, size_t count, unsigned* meet, int* abort_flag, ResOut* out, int nout) {
    const size_t first = (size_t)blockIdx.x * blockDim.x + threadIdx.x, step = (size_t)gridDim.x * blockDim.x;
    for (size_t i = first; i < count; i += step) slots[i] = __longlong_as_double((long long)kResSentinel);
    for (size_t i = first; i < (size_t)nout; i += step) out[i].ok = 0;
    if (first == 0) {
        *meet = 0u;
        *abort_flag = 0;
    }
}

constexpr int kMaxDevices = 64;
struct DeviceInfo {
    std::once_flag once;
    std::mutex teams;
    std::atomic<long long> quiet_until{0};  // steady clock, ns: no team before (resident_missed)
    int cus = 0;
    double ticks_per_ms = 0;
};
DeviceInfo g_dev[kMaxDevices];

long long now_ns() {
    return std::chrono::duration_cast<std::chrono::nanoseconds>(std::chrono::steady_clock::now().time_since_epoch())
        .count();
}

// A missed rendezvous has cost the call its whole limit.  What holds the CUs (a
// second process, a stream with a CU mask, long kernels) is likely to hold
// them in the next call too, so the device's solves go by launches for
// kQuiet times that limit: at most 2% of the time goes into teams that do not
// meet.  20 solves of 1M cells and 20 iterations on a stream with half of the
// CUs, after the first: 826 ms when every call waits (twice), 24 without.
constexpr double kQuiet = 50.0;
bool quiet(int device) {
    const long long until = g_dev[device].quiet_until.load(std::memory_order_relaxed);
    return until && now_ns() < until;
}

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

void resident_device(int device, int* cus, double* ticks_per_ms) {
    if (device < 0 || device >= kMaxDevices) {
        *cus = 0;
        *ticks_per_ms = 0;
        return;
    }
    const DeviceInfo& d = device_info(device);
    *cus = d.cus;
    *ticks_per_ms = d.ticks_per_ms;
}

double resident_meet_ms() {
    const char* env = getenv("FVPCG_RESIDENT_MEET_MS");
    return env && *env ? std::max(0.0, atof(env)) : kResMeetMs;
}

double resident_spin_ms() {
    const char* env = getenv("FVPCG_RESIDENT_SPIN_MS");
    return env && *env ? std::max(0.0, atof(env)) : kResSpinMs;
}

void resident_missed(int device) {
    if (device < 0 || device >= kMaxDevices) return;
    g_dev[device].quiet_until.store(now_ns() + (long long)(kQuiet * 1e6 * resident_meet_ms()), std::memory_order_relaxed);
}

int resident_no_result(int device, const int* abort_flag, const char* what, hipStream_t s) {
    int gave_up = 0;
    FV_HIP(hipMemcpyAsync(&gave_up, abort_flag, sizeof(int), hipMemcpyDeviceToHost, s));
    FV_HIP(hipStreamSynchronize(s));
    if (gave_up) return set_error(FVPCG_DEVICE_ERROR, "%s: a wait between workgroups timed out (x is invalid)", what);
    resident_missed(device);
    return FVPCG_OK;
}

bool resident_quiet(int device) { return device >= 0 && device < kMaxDevices && quiet(device); }

int resident_reset(double* slots, size_t count, unsigned* meet, int* abort_flag, ResOut* out, int nout, hipStream_t s) {
    const size_t work = std::max(count, (size_t)nout);
    hipLaunchKernelGGL(k_res_reset, dim3((unsigned)std::min<size_t>((work + 255) / 256, 256)), dim3(256), 0, s, slots, count,
                       meet, abort_flag, out, nout);
    FV_LAUNCHED();
    return FVPCG_OK;
}

// Up to 2,048 cells one workgroup holds the system and exchanges through LDS
// (no rendezvous, no device-wide reduction).  Above that a team takes the
// tiles of the launch-per-iteration kernels, at most kMaxGrid workgroups of up
// to 4,096 rows: 1,048,576 cells, as many as registers and LDS hold.  Unpacked
// int32 columns leave room for 3,072 rows, rows of more than 6 slots for
// 2,048, rows of more than 8 slots for none; the literal recurrences' two more
// vectors leave room for 2,048.
//
// Standard CG gathers two vectors, past the L2 caches; every line of a gather
// is fetched by itself.  On a mesh whose cells are in no order a product
// fetches a line per slot, which the launches' single vector finds in the L2
// caches.  Launches against one launch, by the lines of a product: 1.09x at
// 1.3M (60^3 shuffled), 1.13x at 1.3M (91^3, blocks of 16 cells shuffled), 1.05x at
// 1.6M (200,000 cells with 8 neighbours, shuffled), 0.86x at 2.1M (70^3 shuffled),
// 0.92x at 2.2M (91^3 by blocks of 8), 0.53x at 4.5M (91^3 shuffled); in order 91^3
// has 0.6M, 2.0x.  Past the line k_res_cg_stream takes the system, which gathers
// one vector through the caches: 0.99x to 1.09x in these.  Pipelined CG gathers
// one vector and gains past the caches, too (1.4x to 2.3x).
constexpr long long kCgLines = 1700000;

ResPlan resident_plan(const fvpcg_mesh* m, int method) {
    ResPlan p;
    const char* env = getenv("FVPCG_RESIDENT");
    if (env && env[0] == '0') return p;
    if (m->WT > 8 || m->n < 1 || m->device < 0 || m->device >= kMaxDevices) return p;
    const int bs = method == FVPCG_CG ? kResBsCg : kResBsPipe;
    const int tiles = (m->n + bs - 1) / bs;
    p.method = method;
    p.block = bs;
    if (tiles * bs <= 2048) {
        p.one = true;
        p.size = 1;
        p.rpt = tiles <= 2 ? tiles : 4;
        return p;
    }
    const int g = std::min(tiles, kMaxGrid);  // geom_for's workgroups
    int rpt = (tiles + g - 1) / g;
    if (rpt == 5 || rpt == 7) ++rpt;
    const int rows = m->WT > 6 || method == FVPCG_PIPECG_LITERAL ? 2048 : m->col16 ? 4096 : 3072;
    if (rpt * bs > rows || g > device_info(m->device).cus || quiet(m->device)) return p;
    if (method == FVPCG_CG && m->lines > kCgLines) return p;
    p.size = g;
    p.rpt = rpt;
    return p;
}

ResPlan resident_plan_stream(const fvpcg_mesh* m, int method) {
    ResPlan p;
    const char* env = getenv("FVPCG_RESIDENT");
    if (env && env[0] == '0') return p;
    if (m->WT > 8 || m->n < 1 || m->device < 0 || m->device >= kMaxDevices) return p;
    const DeviceInfo& info = device_info(m->device);
    const int bs = method == FVPCG_CG ? kResBsCg : kResBsPipe;
    const int tiles = (m->n + bs - 1) / bs;
    const int g = std::min(tiles, kMaxGrid);  // geom_for's workgroups
    const int per = (tiles + g - 1) / g;
    if (per > (method == FVPCG_CG ? 16 : kStreamTiles) || g > info.cus || info.ticks_per_ms <= 0 ||
        quiet(m->device))
        return p;
    p.method = method;
    p.block = bs;
    p.size = g;
    if (method == FVPCG_CG)
        p.rpt = per <= 8 ? 8 : 16;
    else
        p.rpt = per <= 16 ? 16 : per <= 32 ? 32 : 64;
    return p;
}

int resident_stream_run(const fvpcg_mesh* m, const ResPlan& plan, const ResWork& w, const PipeVec<double>& a, bool jac,
                        DevState* st, hipStream_t s, bool* done) {
    *done = false;
    const DeviceInfo& info = device_info(m->device);
    std::unique_lock<std::mutex> lock(g_dev[m->device].teams, std::try_to_lock);
    if (!lock.owns_lock()) return FVPCG_OK;  // another team has the GPU
    int rc;
    w.pinned->ok = 0;
    if ((rc = resident_reset(w.slots, res_slots(plan.size), w.meet, w.abort_flag, nullptr, 0, s))) return rc;
    ResTeam t{0, plan.size, w.slots, w.meet, w.abort_flag, nullptr,
              (unsigned long long)(info.ticks_per_ms * resident_meet_ms()),
              (unsigned long long)(info.ticks_per_ms * resident_spin_ms()), 0};
    const auto pick = plan.method == FVPCG_CG ? res_kernel_cg_stream : res_kernel_stream;
    hipLaunchKernelGGL(pick(plan.rpt, m->WT, m->col16 != nullptr, jac), dim3(plan.size), dim3(plan.block), 0, s, a, m->n, t,
                       st, w.pinned);
    FV_LAUNCHED();
    FV_HIP(hipStreamSynchronize(s));
    if (w.pinned->ok) {
        *done = true;
        return FVPCG_OK;
    }
    return resident_no_result(m->device, w.abort_flag, "CG", s);
}

ResPlan resident_plan32(const fvpcg_mesh* m) {
    ResPlan p;
    const char* env = getenv("FVPCG_RESIDENT");
    if (env && env[0] == '0') return p;
    if (m->WT > 8 || m->n < 1 || m->device < 0 || m->device >= kMaxDevices) return p;
    const DeviceInfo& info = device_info(m->device);
    const int tiles = (m->n + kResBsMixed - 1) / kResBsMixed;
    const int g = std::min(tiles, kMaxGrid);  // geom_for's workgroups
    int rpt = (tiles + g - 1) / g;
    rpt = rpt <= 2 ? rpt : rpt <= 4 ? 4 : rpt <= 6 ? 6 : rpt;
    if (rpt == 7) rpt = 8;
    if (rpt > (m->WT > 6 || !m->col16 ? 4 : 8) || g > info.cus || info.ticks_per_ms <= 0 ||
        quiet(m->device))
        return p;
    p.block = kResBsMixed;
    p.size = g;
    p.rpt = rpt;
    return p;
}

int resident_run32(const fvpcg_mesh* m, const ResPlan& plan, const ResWork& w, const PipeVec<float>& a, int iters,
                   DevState* st, DevState* st_skip, hipStream_t s) {
    const DeviceInfo& info = device_info(m->device);
    int rc;
    if ((rc = resident_reset(w.slots, res_slots(plan.size), w.meet, w.abort_flag, nullptr, 0, s))) return rc;
    ResTeam t{0, plan.size, w.slots, w.meet, w.abort_flag, nullptr,
              (unsigned long long)(info.ticks_per_ms * resident_meet_ms()),
              (unsigned long long)(info.ticks_per_ms * resident_spin_ms()), 0};
    hipLaunchKernelGGL(res_kernel_mixed(plan.rpt, m->WT, m->col16 != nullptr), dim3(plan.size), dim3(plan.block), 0, s, a,
                       m->n, iters, t, st, st_skip);
    FV_LAUNCHED();
    return FVPCG_OK;
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
    int rc;
    if (!plan.one && (rc = resident_reset(w.slots, res_slots(plan.size), w.meet, w.abort_flag, out, 1, s))) return rc;
    ResTeam t{0, plan.size, w.slots, w.meet, w.abort_flag, nullptr,
              (unsigned long long)(info.ticks_per_ms * resident_meet_ms()), (unsigned long long)(info.ticks_per_ms * resident_spin_ms()),
              0};
    ResKernel k = plan.method == FVPCG_CG ? res_kernel_cg(plan, m->WT, m->col16 != nullptr, jac)
                                          : res_kernel_pipe(plan, m->WT, m->col16 != nullptr, jac);
    hipLaunchKernelGGL(k, dim3(plan.size), dim3(plan.block), 0, s, sys, t, out);
    FV_LAUNCHED();
    if (!w.pinned) FV_HIP(hipMemcpyAsync(&host, w.out, sizeof(ResOut), hipMemcpyDeviceToHost, s));
    FV_HIP(hipStreamSynchronize(s));
    if (w.pinned) host = *w.pinned;
    if (!host.ok) return resident_no_result(m->device, w.abort_flag, "CG", s);
    *done = true;
    if (stats) {
        stats->iters = host.iter;
        stats->outer_iters = 0;
        stats->status = host.status;
        stats->one_launch = 1;
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

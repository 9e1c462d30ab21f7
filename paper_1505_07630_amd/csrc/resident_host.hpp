// The resident solves' host interface (resident.hip).
#pragma once

#include <mutex>

#include "handles.hpp"

namespace fvpcg {

struct ResOut;
struct ResSystem;
struct ResTeam;
struct ResBatch;
template <typename T>
struct PipeVec;
using ResStreamKernel = void (*)(PipeVec<double>, int, ResTeam, DevState*, ResOut*);
using ResMixedKernel = void (*)(PipeVec<float>, int, int, ResTeam, DevState*, DevState*);
using ResBatchKernel = void (*)(ResSystem, ResTeam, ResBatch);
using ResKernel = void (*)(ResSystem, ResTeam, ResOut*);

// Rendezvous limit: past it (other work holds the GPU's CUs) the launch-per-
// iteration path runs instead (FVPCG_RESIDENT_MEET_MS sets another;
// FVPCG_RESIDENT=0 always takes that path).  Limit of any later wait, which
// ends by itself (FVPCG_RESIDENT_SPIN_MS sets another; past it the call is a
// device error: members may have written x by then, so no other path goes on
// from it).
constexpr double kResMeetMs = 20.0, kResSpinMs = 5000.0;

struct ResPlan {
    int rpt = 0;   // rows per thread; 0: not resident
    int size = 0;  // workgroups
    int block = 0; // threads per workgroup
    int method = 0;
    bool one = false;
};

// Buffers of a resident solve: exchange vectors, slots for kResMaxTeam
// members, rendezvous word, abort flag, result (device, or pinned).
struct ResWork {
    double *e0, *e1, *slots;
    unsigned* meet;
    int* abort_flag;
    ResOut* out;
    ResOut* pinned;
};

// Held while a launch whose workgroups wait for each other is on the device:
// two such launches side by side could each hold half of the CUs and wait.
std::mutex* resident_teams(int device);

ResPlan resident_plan(const fvpcg_mesh* m, int method);
ResKernel res_kernel_pipe(const ResPlan& p, int wt, bool col16, bool jac);
ResKernel res_kernel_cg(const ResPlan& p, int wt, bool col16, bool jac);
ResMixedKernel res_kernel_mixed(int rpt, int wt, bool col16);
ResStreamKernel res_kernel_stream(int nt, int wt, bool col16, bool jac);
ResStreamKernel res_kernel_cg_stream(int nt, int wt, bool col16, bool jac);
ResBatchKernel res_batch_pipe(int rpt, int wt, bool col16, bool jac);
ResBatchKernel res_batch_cg(int rpt, int wt, bool col16, bool jac);
double resident_meet_ms();
double resident_spin_ms();
// After a launch whose result is missing: FVPCG_OK if the team did not come
// together (nothing was written), FVPCG_DEVICE_ERROR if a later wait was given up.
int resident_no_result(int device, const int* abort_flag, const char* what, hipStream_t s);
// A rendezvous was missed on the device; whether one was missed so recently
// that no team is tried (the plans ask it by themselves).
void resident_missed(int device);
bool resident_quiet(int device);
// CUs, and wall-clock ticks per ms (0: unknown) of a device.
void resident_device(int device, int* cus, double* ticks_per_ms);
// Enqueues the reset of `count` slot doubles, the rendezvous word, the abort
// flag and nout results.
int resident_reset(double* slots, size_t count, unsigned* meet, int* abort_flag, ResOut* out, int nout, hipStream_t s);

// A run of `iters` FP32 pipelined iterations (resident_pipe32): up to 2,097,152
// cells (8 rows per thread; int32 columns or rows of more than 6 slots leave
// room for 4).  The caller holds resident_teams() from the launch until it has
// seen what became of it in st_skip.
ResPlan resident_plan32(const fvpcg_mesh* m);
int resident_run32(const fvpcg_mesh* m, const ResPlan& plan, const ResWork& w, const PipeVec<float>& a, int iters,
                   DevState* st, DevState* st_skip, hipStream_t s);

// The iterations of a larger folded pipelined or standard solve in one launch
// (resident_stream, k_res_cg_stream), the initial residual and first reduction
// done (st, a).
// *done = false with FVPCG_OK: nothing was done, iterate by launches.
ResPlan resident_plan_stream(const fvpcg_mesh* m, int method = FVPCG_PIPECG);
int resident_stream_run(const fvpcg_mesh* m, const ResPlan& plan, const ResWork& w, const PipeVec<double>& a, bool jac,
                        DevState* st, hipStream_t s, bool* done);

// *done = false with FVPCG_OK: not solved here, solve by launches (x is still
// a valid starting vector); a negative code is an error.
int resident_solve(const fvpcg_matrix* A, const ResPlan& plan, const ResWork& w, const double* b, double* x, double tol,
                   int maxit, bool jac, hipStream_t s, fvpcg_stats* stats, bool* done);

}  // namespace fvpcg

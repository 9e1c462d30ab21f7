// The streaming resident pipelined-CG kernels (resident.hpp) and their choice.
#include "resident.hpp"
#include "resident_host.hpp"

namespace fvpcg {

namespace {

template <int NT, int WT, typename CI, bool JAC>
__global__ __launch_bounds__(kResBsPipe) void k_res_stream(PipeVec<double> a, int n, ResTeam t, DevState* st, ResOut* out) {
    __shared__ double lds[(NT == 64 ? kStreamLdsTiles : 32) * kResBsPipe];
    __shared__ int s_ok;
    if (threadIdx.x == 0) s_ok = 1;
    t.rank = res_rank((int)blockIdx.x, t.size);
    t.ok = &s_ok;
    t.queued = false;
    if (!team_meet(t)) return;
    resident_stream<NT, WT, CI, JAC>(a, n, t, lds, st, out);
}

template <int NT, int WT>
ResStreamKernel pick_form(bool col16, bool jac) {
    if (col16) return jac ? k_res_stream<NT, WT, int16_t, true> : k_res_stream<NT, WT, int16_t, false>;
    return jac ? k_res_stream<NT, WT, int, true> : k_res_stream<NT, WT, int, false>;
}

template <int WT>
ResStreamKernel pick_tiles(int nt, bool col16, bool jac) {
    if (nt == 16) return pick_form<16, WT>(col16, jac);
    if (nt == 32) return pick_form<32, WT>(col16, jac);
    return pick_form<64, WT>(col16, jac);
}

}  // namespace

ResStreamKernel res_kernel_stream(int nt, int wt, bool col16, bool jac) {
    if (wt == 4) return pick_tiles<4>(nt, col16, jac);
    if (wt == 6) return pick_tiles<6>(nt, col16, jac);
    return pick_tiles<8>(nt, col16, jac);
}

}  // namespace fvpcg

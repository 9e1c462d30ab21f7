// Standard CG beyond what the chip holds whole, all iterations in one launch
// (solve.hip's k_cg_spmv, k_cg_update_r and k_cg_update_xp, whose results these
// are bit for bit), with the matrix streamed and the vectors on chip as far as
// they fit at 1,024 threads (tiles of 1,024 rows per member):
//   up to 8 tiles (2.1M cells)  q, r and x in registers, p and d in LDS;
//   up to 16 tiles (4.2M)       q and r in registers, p in LDS.
// Bound by memory, and by the round trips of one row at a time per thread in
// the product: 76 and 116 bytes per row and iteration against 164 by launches.
// us per iteration, launches and here (columns of level-ordered cubes): 39.9 and 30.2 at
// 1.05M cells, 67.4 and 49.2 at 2.1M, 101 and 87 at 3.4M, 117 and 98 at 4.1M.
// With 32 tiles (q in registers, r in LDS for 16) 171 against 155 at 5.4M and 206
// against 202 at 7.1M: larger systems stay with the launches.  p is stored with agent scope and gathered through the caches,
// which every member invalidates after the meeting that follows.
#include "resident.hpp"
#include "resident_host.hpp"

namespace fvpcg {

namespace {

// N doubles of a thread in registers, indexed by the (uniform) tile number.
template <int N>
using RegTiles = double __attribute__((ext_vector_type(N)));

template <int NT, int WT, typename CI, bool JAC>
__global__ __launch_bounds__(kResBsCg) void k_res_cg_stream(PipeVec<double> a, int n, ResTeam t, DevState* st, ResOut* out) {
    constexpr int BS = kResBsCg;
    constexpr bool kX = NT == 8, kD = NT == 8;  // x in registers, d in LDS
    __shared__ double lds[16 * BS];
    __shared__ int s_ok;
    if (threadIdx.x == 0) s_ok = 1;
    t.rank = res_rank((int)blockIdx.x, t.size);
    t.ok = &s_ok;
    t.queued = false;
    if (!team_meet(t)) return;
    const CI* __restrict__ col = (const CI*)a.col;
    const double* __restrict__ val = a.val;
    const double* __restrict__ d = a.d;
    double* const p = a.p;
    double* const x = a.x;
    const double* __restrict__ r = a.r;
    double* const lp = lds + threadIdx.x;           // p
    double* const ld = lds + 8 * BS + threadIdx.x;  // d
    const int G = t.size, tiles = (n + BS - 1) / BS;
    const int mine = t.rank < tiles ? (tiles - t.rank + G - 1) / G : 0;
    const int first = t.rank * BS + (int)threadIdx.x;
    RegTiles<NT> q = 0.0, rr = 0.0;
    RegTiles<8> xr = 0.0;
    for (int k = 0; k < mine; ++k) {
        const int c = first + k * G * BS;
        if (c >= n) continue;
        rr[k] = r[c];
        lp[k * BS] = p[c];
        if (kD) ld[k * BS] = d[c];
        if (kX) xr[k & 7] = x[c];
    }
    double gamma = st->gamma, alpha = 0.0, beta = 0.0, rho = st->rho, delta = st->delta;
    const double tol_abs = st->tol_abs;
    const int maxit = st->maxit;
    int iter = st->iter, status = FVPCG_NOT_CONVERGED;
    bool done = false;
    const unsigned long long t0 = (unsigned long long)wall_clock64();
    for (;;) {
        // q = A p
        double s1[1] = {0.0};
        for (int k = 0; k < mine; ++k) {
            const int c = first + k * G * BS;
            if (c >= n) continue;
            CI j[WT];
            double m[WT], g[WT];
            load_slots_raw<double, WT, CI>(col, val, n, c, j, m);
            const double dc = kD ? ld[k * BS] : d[c], pc = lp[k * BS];
#pragma unroll
            for (int i = 0; i < WT; ++i) g[i] = p[slot_abs(j[i], c)];
            double qc = dc * pc;
#pragma unroll
            for (int i = 0; i < WT; ++i) qc = fma(m[i], g[i], qc);
            q[k] = qc;
            s1[0] += pc * qc;
        }
        if (!team_sum<BS, 1>(s1, t)) return;
        delta = s1[0];
        if (!(delta > 0.0) || !isfinite(delta) || !isfinite(gamma)) {
            done = true;
            status = FVPCG_BREAKDOWN;
            break;
        }
        alpha = gamma / delta;
        // r -= alpha q, z = M^-1 r
        double s2[2] = {0.0, 0.0};
        for (int k = 0; k < mine; ++k) {
            const int c = first + k * G * BS;
            if (c >= n) continue;
            const double dc = !JAC ? 1.0 : kD ? ld[k * BS] : d[c];
            const double rc = rr[k] - alpha * q[k];
            rr[k] = rc;
            const double zc = JAC ? rc / dc : rc;
            s2[0] += rc * zc;
            s2[1] += rc * rc;
        }
        if (!team_sum<BS, 2>(s2, t)) return;
        iter += 1;
        rho = s2[1];
        if (sqrt(rho) <= tol_abs) {
            done = true;
            status = FVPCG_OK;
        } else if (iter >= maxit) {
            done = true;
        } else {
            beta = s2[0] / gamma;
            gamma = s2[0];
        }
        // x += alpha p, p = z + beta p
        for (int k = 0; k < mine; ++k) {
            const int c = first + k * G * BS;
            if (c >= n) continue;
            const double dc = !JAC ? 1.0 : kD ? ld[k * BS] : d[c];
            const double pc = lp[k * BS];
            const double xc = (kX ? xr[k & 7] : ld_once(x + c)) + alpha * pc;
            if (kX) xr[k & 7] = xc;
            else st_once(x + c, xc);
            if (!done) {
                const double rc = rr[k];
                const double zc = JAC ? rc / dc : rc;
                const double pn = zc + beta * pc;
                lp[k * BS] = pn;
                st_agent(p + c, pn);
            }
        }
        if (done) break;
        double none[1] = {0.0};
        if (!team_sum<BS, 1>(none, t)) return;
        team_acquire();
    }
    if (kX) {
        for (int k = 0; k < mine; ++k) {
            const int c = first + k * G * BS;
            if (c < n) x[c] = xr[k & 7];
        }
    }
    if (t.rank == 0 && threadIdx.x == 0) {
        st->gamma = gamma;
        st->delta = delta;
        st->alpha = alpha;
        st->beta = beta;
        st->rho = rho;
        st->iter = iter;
        st->status = status;
        st->done = done ? 1 : 0;
        out->it_ticks = (unsigned long long)wall_clock64() - t0;
        out->ok = 1;
    }
}

template <int NT, int WT>
ResStreamKernel pick_form(bool col16, bool jac) {
    if (col16) return jac ? k_res_cg_stream<NT, WT, int16_t, true> : k_res_cg_stream<NT, WT, int16_t, false>;
    return jac ? k_res_cg_stream<NT, WT, int, true> : k_res_cg_stream<NT, WT, int, false>;
}

template <int WT>
ResStreamKernel pick_tiles(int nt, bool col16, bool jac) {
    return nt == 8 ? pick_form<8, WT>(col16, jac) : pick_form<16, WT>(col16, jac);
}

}  // namespace

ResStreamKernel res_kernel_cg_stream(int nt, int wt, bool col16, bool jac) {
    if (wt == 4) return pick_tiles<4>(nt, col16, jac);
    if (wt == 6) return pick_tiles<6>(nt, col16, jac);
    return pick_tiles<8>(nt, col16, jac);
}

}  // namespace fvpcg

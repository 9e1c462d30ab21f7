// BiCGSTAB's iterations in one launch (bicgstab.hip states the method and the
// launch-per-iteration form, whose results these are bit for bit).
//
// Per iteration and row the launches move, for three components, 536 bytes:
// v and t are written once and read back. Here a team (resident.hpp) keeps v
// in registers (vectors of 16 indexed by the tile number) and t in LDS (two
// components, the third in registers too): 416 bytes, 40 fewer per component (v
// is read twice, t once), and four meetings of the team instead of four
// launches:
//   v = A M^-1 p, (rhat, v)                       -> alpha
//   s = r - alpha v in r's place
//   t = A M^-1 s and its five sums                -> omega, rho', beta
//   x, r', p' and (r', r')                        -> the stopping test
// Up to 16 tiles of 512 rows per member (2,097,152 cells).  p and s are stored
// with agent scope and gathered through the caches, which every member
// invalidates after the meetings they follow.  Bound by the passes over
// memory: at 128^3 and three components 872 MB in 187 us, 4.67 TB/s (by
// launches 1,124 MB in 245 us).
#include "bicgstab.hpp"
#include "resident.hpp"
#include "resident_host.hpp"

namespace fvpcg {

namespace {

constexpr int kBiSums = 16;  // slots: up to 5 sums for each of 3 components
constexpr int kBiTiles = 16;

__device__ __forceinline__ double uniform(double v) {
    return __hiloint2double(__builtin_amdgcn_readfirstlane(__double2hiint(v)),
                            __builtin_amdgcn_readfirstlane(__double2loint(v)));
}

template <int NR, int WT, typename CI, bool JAC>
__global__ __launch_bounds__(kResBsPipe) void k_res_bicg(const CI* __restrict__ col, const double* __restrict__ val,
                                                         const double* __restrict__ d, int n, double* x, double* r,
                                                         const double* __restrict__ rhat, double* p, ResTeam t,
                                                         BiState* st, ResOut* out) {
    constexpr int BS = kResBsPipe, NL = NR < 2 ? NR : 2;  // NL: components of t in LDS
    static_assert(NR <= 3, "the third component's t in registers, a fourth has no place");
    __shared__ double lds[NL * kBiTiles * BS];
    __shared__ BiState s_st[NR];
    __shared__ int s_ok;
    if (threadIdx.x == 0) s_ok = 1;
    t.rank = res_rank((int)blockIdx.x, t.size);
    t.ok = &s_ok;
    t.queued = false;
    if (!team_meet(t)) return;
    const int G = t.size, tiles = (n + BS - 1) / BS;
    const int mine = t.rank < tiles ? (tiles - t.rank + G - 1) / G : 0;
    double* const lt = lds + threadIdx.x;
    if ((int)threadIdx.x < NR) s_st[threadIdx.x] = st[threadIdx.x];
    __syncthreads();
    Tile16 v[NR], t2;
    t2 = 0.0;
#pragma unroll
    for (int k = 0; k < NR; ++k) v[k] = 0.0;
    const unsigned long long t0 = (unsigned long long)wall_clock64();
    bool act[NR];
    auto active = [&]() {
        bool any = false;
#pragma unroll
        for (int k = 0; k < NR; ++k) {
            act[k] = __builtin_amdgcn_readfirstlane(s_st[k].done) == 0;
            any |= act[k];
        }
        return any;
    };
    while (active()) {
        // v = A M^-1 p
        double a1[NR];
#pragma unroll
        for (int k = 0; k < NR; ++k) a1[k] = 0.0;
        for (int q = 0; q < mine; ++q) {
            const int c = (q * G + t.rank) * BS + (int)threadIdx.x;
            if (c >= n) continue;
            CI j[WT];
            double m[WT], vc[NR], h[NR];
            load_slots_raw<double, WT, CI>(col, val, n, c, j, m);
            const double dc = JAC ? 1.0 : ld_once(d + c);
#pragma unroll
            for (int k = 0; k < NR; ++k) {
                h[k] = ld_once(rhat + (size_t)k * n + c);
                const double pc = p[(size_t)k * n + c];
                vc[k] = JAC ? pc : dc * pc;
            }
            gather_v<WT, CI, NR>(j, m, n, c, p, act, vc);
#pragma unroll
            for (int k = 0; k < NR; ++k) {
                if (!act[k]) continue;
                v[k][q] = vc[k];
                a1[k] += h[k] * vc[k];
            }
        }
        if (!team_sum<BS, NR, kBiSums>(a1, t)) return;
        if (threadIdx.x == 0) {
#pragma unroll
            for (int k = 0; k < NR; ++k)
                if (act[k]) bi_step_pv(&s_st[k], a1[k]);
        }
        __syncthreads();
        if (!active()) break;
        double alpha[NR];
#pragma unroll
        for (int k = 0; k < NR; ++k) alpha[k] = uniform(s_st[k].alpha);
        // s = r - alpha v in r's place
        for (int q = 0; q < mine; ++q) {
            const int c = (q * G + t.rank) * BS + (int)threadIdx.x;
            if (c >= n) continue;
            double rc[NR];
#pragma unroll
            for (int k = 0; k < NR; ++k) rc[k] = ld_once(r + (size_t)k * n + c);
#pragma unroll
            for (int k = 0; k < NR; ++k)
                if (act[k]) st_agent(r + (size_t)k * n + c, bi_half(rc[k], v[k][q], alpha[k]));
        }
        double none[1] = {0.0};
        if (!team_sum<BS, 1, kBiSums>(none, t)) return;
        team_acquire();
        // t = A M^-1 s
        double a2[5 * NR];
#pragma unroll
        for (int k = 0; k < 5 * NR; ++k) a2[k] = 0.0;
        for (int q = 0; q < mine; ++q) {
            const int c = (q * G + t.rank) * BS + (int)threadIdx.x;
            if (c >= n) continue;
            CI j[WT];
            double m[WT], sc[NR], tc[NR], h[NR];
            load_slots_raw<double, WT, CI>(col, val, n, c, j, m);
            const double dc = JAC ? 1.0 : ld_once(d + c);
#pragma unroll
            for (int k = 0; k < NR; ++k) {
                h[k] = ld_once(rhat + (size_t)k * n + c);
                sc[k] = r[(size_t)k * n + c];
                tc[k] = JAC ? sc[k] : dc * sc[k];
            }
            gather_v<WT, CI, NR>(j, m, n, c, r, act, tc);
#pragma unroll
            for (int k = 0; k < NR; ++k) {
                if (!act[k]) continue;
                const double tk = tc[k], sk = sc[k], hk = h[k];
                if (k < NL)
                    lt[(k * kBiTiles + q) * BS] = tk;
                else
                    t2[q] = tk;
                a2[5 * k] += tk * sk;
                a2[5 * k + 1] += tk * tk;
                a2[5 * k + 2] += sk * sk;
                a2[5 * k + 3] += hk * sk;
                a2[5 * k + 4] += hk * tk;
            }
        }
        if (!team_sum<BS, 5 * NR, kBiSums>(a2, t)) return;
        if (threadIdx.x == 0) {
#pragma unroll
            for (int k = 0; k < NR; ++k)
                if (act[k]) bi_step_st(&s_st[k], a2 + 5 * k);
        }
        __syncthreads();
        if (!active()) break;
        double omega[NR], beta[NR];
#pragma unroll
        for (int k = 0; k < NR; ++k) {
            alpha[k] = uniform(s_st[k].alpha);
            omega[k] = uniform(s_st[k].omega);
            beta[k] = uniform(s_st[k].beta);
        }
        // x, r' and p'
        double a3[NR];
#pragma unroll
        for (int k = 0; k < NR; ++k) a3[k] = 0.0;
        for (int q = 0; q < mine; ++q) {
            const int c = (q * G + t.rank) * BS + (int)threadIdx.x;
            if (c >= n) continue;
            double sc[NR], pc[NR], xc[NR];
            const double dc = JAC ? ld_once(d + c) : 1.0;
#pragma unroll
            for (int k = 0; k < NR; ++k) {
                const size_t e = (size_t)k * n + c;
                sc[k] = r[e];
                pc[k] = p[e];
                xc[k] = ld_once(x + e);
            }
#pragma unroll
            for (int k = 0; k < NR; ++k) {
                if (!act[k]) continue;
                const size_t e = (size_t)k * n + c;
                const double tc = k < NL ? lt[(k * kBiTiles + q) * BS] : t2[q];
                const double dx = fma(alpha[k], pc[k], omega[k] * sc[k]);
                st_once(x + e, xc[k] + (JAC ? dx / dc : dx));
                const double rn = fma(-omega[k], tc, sc[k]);
                st_once(r + e, rn);
                st_agent(p + e, fma(beta[k], fma(-omega[k], v[k][q], pc[k]), rn));
                a3[k] += rn * rn;
            }
        }
        if (!team_sum<BS, NR, kBiSums>(a3, t)) return;
        if (threadIdx.x == 0) {
#pragma unroll
            for (int k = 0; k < NR; ++k)
                if (act[k]) bi_step_update(&s_st[k], a3[k]);
        }
        team_acquire();
    }
    if (t.rank == 0 && (int)threadIdx.x < NR) st[threadIdx.x] = s_st[threadIdx.x];
    if (t.rank == 0 && threadIdx.x == 0) {
        out->it_ticks = (unsigned long long)wall_clock64() - t0;
        out->ok = 1;
    }
}

template <int NR, bool JAC>
int launch(const fvpcg_matrix* A, BiWork& w, const double* val, double* x, const ResPlan& plan, const ResTeam& t,
           hipStream_t s) {
    const fvpcg_mesh* m = A->mesh;
#define FV_BICG(W, CI, cols)                                                                                         \
    hipLaunchKernelGGL((k_res_bicg<NR, W, CI, JAC>), dim3(plan.size), dim3(plan.block), 0, s, cols, val, A->d, m->n, x, w.r, \
                       w.rhat, w.p, t, w.st, w.out)
    if (m->WT == 4) {
        if (m->col16) FV_BICG(4, int16_t, m->col16);
        else FV_BICG(4, int, m->col);
    } else if (m->WT == 6) {
        if (m->col16) FV_BICG(6, int16_t, m->col16);
        else FV_BICG(6, int, m->col);
    } else {
        if (m->col16) FV_BICG(8, int16_t, m->col16);
        else FV_BICG(8, int, m->col);
    }
#undef FV_BICG
    FV_LAUNCHED();
    return FVPCG_OK;
}

}  // namespace

size_t bicg_slots() { return res_slots(kResMaxTeam, kBiSums); }

int resident_bicg_run(const fvpcg_matrix* A, BiWork& w, int nr, const double* val, double* x, bool jac, hipStream_t s,
                      bool* done) {
    *done = false;
    const fvpcg_mesh* m = A->mesh;
    const ResPlan plan = resident_plan_stream(m);
    // More tiles per member than v and t have room for, or a fourth component:
    // by launches.  One component past a tile per member too: its launches
    // gather r and v in the second product and so have three kernels against
    // four meetings (us per iteration, launches and team: 19.1 and 14.0 at
    // 32^3, 25.3 and 24.3 at 48^3, 32.9 and 34.7 at 64^3, 58 and 61 at 96^3).
    // Two and three always gain: 31 and 18 us at 16^3, 59 and 49-51 at 64^3,
    // 122 and 98 at 96^3, 245 and 190 at 128^3 for three.
    if (plan.rpt != kBiTiles || nr > 3 || (nr == 1 && m->n > plan.size * plan.block)) return FVPCG_OK;
    std::unique_lock<std::mutex> lock(*resident_teams(m->device), std::try_to_lock);
    if (!lock.owns_lock()) return FVPCG_OK;  // another team has the GPU
    int cus = 0, rc;
    double ticks = 0;
    resident_device(m->device, &cus, &ticks);
    int* abort_flag = reinterpret_cast<int*>(w.meet + 1);
    w.out->ok = 0;
    if ((rc = resident_reset(w.slots, res_slots(plan.size, kBiSums), w.meet, abort_flag, nullptr, 0, s))) return rc;
    const ResTeam t{0, plan.size, w.slots, w.meet, abort_flag, nullptr, (unsigned long long)(ticks * resident_meet_ms()),
                    (unsigned long long)(ticks * resident_spin_ms()), 0};
    switch (nr) {
        case 1: rc = jac ? launch<1, true>(A, w, val, x, plan, t, s) : launch<1, false>(A, w, val, x, plan, t, s); break;
        case 2: rc = jac ? launch<2, true>(A, w, val, x, plan, t, s) : launch<2, false>(A, w, val, x, plan, t, s); break;
        default: rc = jac ? launch<3, true>(A, w, val, x, plan, t, s) : launch<3, false>(A, w, val, x, plan, t, s); break;
    }
    if (rc) return rc;
    FV_HIP(hipStreamSynchronize(s));
    if (w.out->ok) {
        *done = true;
        return FVPCG_OK;
    }
    return resident_no_result(m->device, abort_flag, "BiCGSTAB", s);
}

}  // namespace fvpcg

// BiCGSTAB's state, workspace and the pieces its launch-per-iteration and
// one-launch forms share (bicgstab.hip states the method).
#pragma once

#include "handles.hpp"
#include "rows.hpp"

namespace fvpcg {

// Scalars of one component's recurrences, written by the last workgroup of
// each kernel.
struct alignas(128) BiState {
    double rho;      // (rhat, r) of the current iterate
    double rho_next; // (rhat, r') of the iterate being formed
    double alpha;    // alpha, omega, beta are 0 once the component has stopped
    double omega;    // 0 after a half-step exit
    double beta;
    double rr;       // (r, r)
    double bnorm;
    double tol_abs;  // tol * ||b||
    double r0norm;
    double true_rr;  // ||b - A x||^2 at exit
    int32_t iter;    // iterations that formed alpha
    int32_t maxit;
    int32_t done;
    int32_t status;
    int32_t zero_b;
    int32_t half;    // ||s|| met the tolerance: x += alpha phat ends the solve
    uint32_t ticket; // reduction ticket (component 0's serves all)
    uint32_t pad;
};

constexpr int kBiMaxRhs = 4;

struct BiWork {
    int n = 0;
    int nr = 0;                  // components the vectors are sized for
    double* r = nullptr;         // [nr][n] each
    double* rhat = nullptr;
    double* p = nullptr;
    double* v = nullptr;
    double* t = nullptr;
    double* partials = nullptr;  // [5 kBiMaxRhs][kBiMaxGrid]
    double* slots = nullptr;     // of the one-launch iterations (resident.hpp), with the rendezvous words
    unsigned* meet = nullptr;    // [2]
    ResOut* out = nullptr;       // pinned
    BiState* st = nullptr;       // [kBiMaxRhs]
    BiState* hst = nullptr;      // pinned [3][kBiMaxRhs]: two chunk slots and the reset image
    hipEvent_t ev[2] = {nullptr, nullptr};
    hipEvent_t t_begin = nullptr, t_end = nullptr, t_it0 = nullptr, t_it1 = nullptr;
};

// s = r - alpha v with one rounding: the row that owns an entry and every
// row that gathers it compute the same bits.
__device__ __forceinline__ double bi_half(double r, double v, double alpha) { return fma(-alpha, v, r); }

// The component's exit: status, and zero scalars so later launches leave it
// untouched.
__device__ __forceinline__ void bi_stop(BiState* st, int status) {
    st->done = 1;
    st->status = status;
    st->alpha = 0.0;
    st->omega = 0.0;
    st->beta = 0.0;
}

// alpha from (rhat, v).
__device__ __forceinline__ void bi_step_pv(BiState* sk, double rv) {
    const double alpha = sk->rho / rv;
    if (rv == 0.0 || !isfinite(alpha)) {
        bi_stop(sk, FVPCG_BREAKDOWN);
        return;
    }
    sk->alpha = alpha;
}

// omega, rho' and beta from q = (t, s), (t, t), (s, s), (rhat, s), (rhat, t), or
// the half-step exit.
__device__ __forceinline__ void bi_step_st(BiState* sk, const double* q) {
    if (sqrt(q[2]) <= sk->tol_abs) {
        sk->omega = 0.0;
        sk->beta = 0.0;
        sk->half = 1;
        return;
    }
    const double omega = q[0] / q[1];
    if (q[1] == 0.0 || omega == 0.0 || !isfinite(omega)) {
        sk->iter = sk->iter + 1;
        bi_stop(sk, FVPCG_BREAKDOWN);
        return;
    }
    const double rho_next = fma(-omega, q[4], q[3]);
    sk->omega = omega;
    sk->rho_next = rho_next;
    sk->beta = (rho_next / sk->rho) * (sk->alpha / omega);
}

// The stopping test on (r', r') and the next rho.
__device__ __forceinline__ void bi_step_update(BiState* sk, double rr) {
    const int it = sk->iter + 1;
    sk->iter = it;
    sk->rr = rr;
    if (sk->half || sqrt(rr) <= sk->tol_abs) {
        bi_stop(sk, FVPCG_OK);
        return;
    }
    if (it >= sk->maxit) {
        bi_stop(sk, FVPCG_NOT_CONVERGED);
        return;
    }
    const double rho = sk->rho_next;
    if (rho == 0.0 || !isfinite(rho) || !isfinite(sk->beta)) {
        bi_stop(sk, FVPCG_BREAKDOWN);
        return;
    }
    sk->rho = rho;
}

// acc[k] += sum_i m[i] * v[k][col_i] over the WT slots (j, m) of row c for
// the components still iterating (v component-major).  Every component's
// values are loaded before any is used, so all the row's gathers are in
// flight at once; the loads of a stopped component are made and discarded.
template <int WT, typename CI, int NR>
__device__ __forceinline__ void gather_v(const CI (&j)[WT], const double (&m)[WT], int n, int c,
                                         const double* __restrict__ v, const bool (&act)[NR], double (&acc)[NR]) {
    double g[NR][WT];
#pragma unroll
    for (int k = 0; k < NR; ++k)
#pragma unroll
        for (int i = 0; i < WT; ++i) g[k][i] = v[(size_t)k * n + slot_abs(j[i], c)];
#pragma unroll
    for (int k = 0; k < NR; ++k) {
        if (!act[k]) continue;
#pragma unroll
        for (int i = 0; i < WT; ++i) acc[k] = fma(m[i], g[k][i], acc[k]);
    }
}

// All iterations in one launch where the system fits (resident_bicg.hip).
// *done = false with FVPCG_OK: nothing was done, iterate by launches.
size_t bicg_slots();
int resident_bicg_run(const fvpcg_matrix* A, BiWork& w, int nr, const double* val, double* x, bool jac, hipStream_t s,
                      bool* done);

}  // namespace fvpcg

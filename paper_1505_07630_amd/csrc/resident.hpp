// Resident solves: a whole Krylov solve in one launch, with a system's matrix
// rows and vectors held in registers and LDS by a team of workgroups from the
// first iteration to the last.
//
// What bounds a small system is not memory but the chain of one iteration:
// a launch, the slot -> gather loads, the reduction's ticket and the scalars.
// With one launch per iteration that chain is 6.3 us at 1.7k cells, 6.8 us at
// 32k and 33 us at 1M (where every array is read again from the last-level
// cache).  Here an iteration reads nothing but the neighbours' exchanged
// vector, and its only synchronisation is the reduction itself:
//
//   * member r of a team of G takes the system's row tiles r, r + G, ...
//     (tiles of BS rows, the launch-per-iteration kernels' order), thread t
//     the t-th row of each: RPT rows per thread, in registers; with RPT > 4
//     four of the vectors in LDS;
//   * the exchanged vector (w, or p and z) goes through device memory with
//     agent-scope relaxed stores and loads, which pass the per-XCD L2 caches,
//     so no cache is written back or invalidated.  Before a workgroup
//     publishes its sums every one of its waves waits for its stores to
//     complete (vmcnt 0), so a member that has seen all sums sees all rows;
//   * a reduction is all-to-all: each member stores its partial sums in its
//     slots, and reads everybody's until none holds the sentinel, a NaN bit
//     pattern no sum is stored with.  The slots are their own flags.  There
//     are four buffers of them; in reduction k a member puts the sentinel
//     back into its slots of reduction k - 2 (nobody reads those any more:
//     everybody has published k - 1, hence read k - 2), which every member
//     sees before it can reach reduction k + 2.
//
// Pipelined CG on MI355X takes 2.3 us per iteration at 1.7k cells (one workgroup),
// 3.1 at 8k, 3.2 at 32k, 5.6 at 262k and 9.9 at 1M.  Acquire fences with cached gathers instead, and a
// two-level reduction, were slower at every size (1M rows: 12.4 us for the
// former when this took 10.9); own tiles of the exchanged vector in LDS as
// well, for the neighbours within the tile, 6.2 us at 262k and 15 at 1M.
//
// The team must be resident together.  It meets once at the start (rendezvous)
// with a short time limit; a team that does not come together there leaves
// without having touched x, and the host takes the launch-per-iteration path.
// Past the rendezvous every member holds its place until it ends, so every
// wait ends; the waits are bounded by a clock all the same (but a queued team's
// first, which lasts as long as its members' earlier systems: team_sum).  A
// wait that is given up ends the call with an error: members may have written
// x by then.
//
// Sums are formed in the launch-per-iteration kernels' order (rows per
// thread, wave, workgroup, workgroups in index order) from the same
// expressions, so both paths give the same bits.
#pragma once

#include "rows.hpp"

namespace fvpcg {

constexpr int kResBsPipe = 512, kResBsCg = 1024, kResBsMixed = 1024;  // threads per workgroup: the launch path's tiles
static_assert(kResBsPipe == kBsPipe && kResBsCg == kBsCg && kResBsMixed == kBsMixed, "the same tiles, the same sums");
constexpr int kResMaxTeam = kMaxGrid;  // members of a team at most
constexpr int kResBufs = 4;           // slot buffers
constexpr int kResSums = 3;           // sums per reduction
constexpr unsigned long long kResSentinel = 0x7ff8f1c3a5965e17ull;
constexpr unsigned kResAbort = 0x80000000u;

// Doubles of slots a team of `size` needs.
inline __host__ __device__ size_t res_slots(int size, int sums = kResSums) { return (size_t)kResBufs * sums * size; }

// What one system's solve reports.
struct ResOut {
    double bnorm, r0norm, rho, true_rr;
    unsigned long long ticks, it_ticks;  // wall clock: the whole solve, the iterations
    int32_t iter, status, zero_b, ok;    // ok = 0: left without a result (see above)
};

// One system as its team sees it.  Columns, values and vectors are indexed
// by the global row; rows [c0, c1) are the system's.
struct ResSystem {
    const void* col;
    const double* val;     // plain values (residuals)
    const double* val_it;  // values of the iterations' product (column-scaled with Jacobi)
    const double* d;
    const double* b;
    double* x;
    double *e0, *e1;  // exchange vectors
    size_t n;         // slot stride
    int c0, c1;
    double tol;
    int maxit;
};

struct ResBatch {
    const int* cell_off;
    const int4* tasks;  // (system, rank, team size, slot offset in members)
    const int* list;    // [grid + 1] each workgroup's range of tasks
    ResOut* out;        // [systems]
};

struct ResTeam {
    int rank, size;
    double* slots;            // [kResBufs][kResSums][size], sentinels at the start
    unsigned* meet;           // rendezvous word, 0 at the start
    int* abort_flag;          // any member's timeout
    int* ok;                  // LDS: 1 until this workgroup has given up a wait
    unsigned long long meet_ticks, spin_ticks;
    int k;                    // reductions so far
    bool queued = false;      // members may still be solving an earlier system of their lists (batches)
};

// Agent-scope accesses of exchanged data.
__device__ __forceinline__ void st_agent(double* p, double v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ double ld_agent(const double* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// The same at element i of an exchanged vector below 4 GiB: a scalar base and
// one address register per access.
template <typename T>
__device__ __forceinline__ void put_agent(T* p, int i, T v) {
    __hip_atomic_store((T*)((char*)p + (unsigned)i * (unsigned)sizeof(T)), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ T get_agent(const T* p, int i) {
    return __hip_atomic_load((const T*)((const char*)p + (unsigned)i * (unsigned)sizeof(T)), __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_AGENT);
}
// Plain accesses (own rows) addressed alike.
template <typename T>
__device__ __forceinline__ void put_plain(T* p, int i, T v) {
    *(T*)((char*)p + (unsigned)i * (unsigned)sizeof(T)) = v;
}
template <typename T>
__device__ __forceinline__ T get_plain(const T* p, int i) {
    return *(const T*)((const char*)p + (unsigned)i * (unsigned)sizeof(T));
}
// The wave's earlier stores have completed.
__device__ __forceinline__ void stores_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Member number of workgroup b of G.  The hardware deals workgroups to the 8
// XCDs in turn; the members of one XCD take consecutive numbers, hence
// consecutive tiles, so most entries a row gathers were stored by its own XCD
// (levels order: 11.3 -> 9.8 us per iteration at 1M cells, 6.6 -> 5.6 at 262k;
// the sums are taken by member number either way).
__device__ __forceinline__ int res_rank(int b, int G) {
    const int x = b & 7, q = G >> 3, rem = G & 7;
    return x * q + (x < rem ? x : rem) + (b >> 3);
}

// True once the whole team runs; false if it did not come together in time.
// The word counts arrivals; a member whose time is up sets the abort bit
// unless the last one has arrived meanwhile, so all members agree.  With no
// time at all (0 ticks) no team comes together: the arrivals of a whole team
// take about as long as a member's first look at the clock and the exchange
// that sets the bit, which fails while the word still moves.
__device__ __forceinline__ bool team_meet(const ResTeam& t) {
    __shared__ int s_go;
    if (t.meet_ticks == 0) return false;
    if (threadIdx.x == 0) {
        unsigned w = __hip_atomic_fetch_add(t.meet, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1u;
        const unsigned long long t0 = (unsigned long long)wall_clock64();
        while (!(w & kResAbort) && w != (unsigned)t.size) {
            if ((unsigned long long)wall_clock64() - t0 > t.meet_ticks) {
                unsigned seen = w;
                if (__hip_atomic_compare_exchange_strong(t.meet, &seen, w | kResAbort, __ATOMIC_RELAXED,
                                                         __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
                    seen = w | kResAbort;
                w = seen;
                continue;
            }
            __builtin_amdgcn_s_sleep(2);
            w = __hip_atomic_load(t.meet, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        s_go = !(w & kResAbort);
    }
    __syncthreads();
    const bool go = s_go != 0;
    __syncthreads();
    return go;
}

// v from lane l ^ X of the same 16 lanes (X = 1, 2, 4 or 8; 4 as 7 then 3).
template <int X>
__device__ __forceinline__ double lane_xor(double v) {
    constexpr int c0 = X == 1 ? 0xB1 : X == 2 ? 0x4E : X == 8 ? 0x128 : 0x141;
    int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), c0, 0xf, 0xf, false);
    int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), c0, 0xf, 0xf, false);
    if (X == 4) {
        lo = __builtin_amdgcn_update_dpp(0, lo, 0x1B, 0xf, 0xf, false);
        hi = __builtin_amdgcn_update_dpp(0, hi, 0x1B, 0xf, 0xf, false);
    }
    return __hiloint2double(hi, lo);
}

// One step of row_sums: of each pair of values a lane keeps the one its bit X
// names and gives the other to lane ^ X.
template <int X, int P>
__device__ __forceinline__ void sums_step(double (&v)[P], int n, int lane) {
    const bool odd = (lane & X) != 0;
#pragma unroll
    for (int i = 0; i < P / 2; ++i)
        if (i < n / 2) {
            const double keep = odd ? v[2 * i + 1] : v[2 * i], give = odd ? v[2 * i] : v[2 * i + 1];
            v[i] = keep + lane_xor<X>(give);
        }
}

// The sums of N values over each row of 16 lanes at once: lane l returns the
// sum of value l mod P (P = N rounded up to a power of two, at most 16) over
// its row.  The tree is that of wave_sum (adjacent pairs, pairs of pairs, ...),
// whose total is (row 0 + row 1) + (row 2 + row 3): the same bits, for 12 values
// in a third of the instructions (1,728 cells, 99 iterations: a solve 307 -> 251 us;
// for the 3 values of a team wave_sum is the quicker).
template <int N>
struct RowSums {
    static constexpr int P = N <= 1 ? 1 : N <= 2 ? 2 : N <= 4 ? 4 : N <= 8 ? 8 : 16;
    static __device__ __forceinline__ double of(const double* x) {
        const int lane = (int)threadIdx.x & 63;
        double v[P < 2 ? 2 : P];
#pragma unroll
        for (int i = 0; i < (P < 2 ? 2 : P); ++i) v[i] = i < N ? x[i] : 0.0;
        int n = P;
        if (n > 1) {
            sums_step<1>(v, n, lane);
            n /= 2;
        } else {
            v[0] += lane_xor<1>(v[0]);
        }
        if (n > 1) {
            sums_step<2>(v, n, lane);
            n /= 2;
        } else {
            v[0] += lane_xor<2>(v[0]);
        }
        if (n > 1) {
            sums_step<4>(v, n, lane);
            n /= 2;
        } else {
            v[0] += lane_xor<4>(v[0]);
        }
        if (n > 1)
            sums_step<8>(v, n, lane);
        else
            v[0] += lane_xor<8>(v[0]);
        return v[0];
    }
};

// v[0..NV) summed over the team, the totals in every thread; false when a
// wait was given up.  Every earlier agent-scope store of any member is
// visible to every member afterwards.
// KS: sums the team's slots have room for.
template <int BS, int NV, int KS = kResSums>
__device__ __forceinline__ bool team_sum(double (&v)[NV], ResTeam& t) {
    constexpr int kW = BS / 64;
    static_assert(NV <= KS && NV <= 16 && KS <= 64, "room in the slots, a lane per sum");
    __shared__ double s_part[NV][kW];
    __shared__ double s_tot[NV];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    if constexpr (NV > 4) {
        double a = RowSums<NV>::of(v);
        a += __shfl_xor(a, 16, 64);
        a += __shfl_xor(a, 32, 64);
        if (lane < NV) s_part[lane][wid] = a;
    } else {
#pragma unroll
        for (int k = 0; k < NV; ++k) v[k] = wave_sum(v[k]);
        if (lane == 0) {
#pragma unroll
            for (int k = 0; k < NV; ++k) s_part[k][wid] = v[k];
        }
    }
    stores_done();
    __syncthreads();
    double mine = 0.0;
    if ((int)threadIdx.x < NV) {
#pragma unroll
        for (int w = 0; w < kW; ++w) mine += s_part[threadIdx.x][w];
    }
    double* buf = t.slots + (size_t)(t.k & (kResBufs - 1)) * KS * t.size;
    if ((int)threadIdx.x < NV) {
        if (__double_as_longlong(mine) == (long long)kResSentinel)
            mine = __longlong_as_double((long long)(kResSentinel ^ 1ull));
        st_agent(buf + (size_t)threadIdx.x * t.size + t.rank, mine);
    }
    if ((int)threadIdx.x < KS) {
        double* old = t.slots + (size_t)((t.k + 2) & (kResBufs - 1)) * KS * t.size;
        st_agent(old + (size_t)threadIdx.x * t.size + t.rank, __longlong_as_double((long long)kResSentinel));
    }
    for (int sum = wid; sum < NV; sum += kW) {
        const double* q = buf + (size_t)sum * t.size;
        constexpr int kC = kResMaxTeam / 64;
        double g[kC];
        // A queued team's first sums come when its last member has finished
        // its earlier systems, which takes as long as these do (every member
        // is resident and each list is in the same order, so it ends); from
        // the second reduction on all members are at work on this system.
        const unsigned long long limit = t.queued && t.k == 0 ? ~0ull : t.spin_ticks;
        unsigned spins = limit ? 0u : 63u;  // a limit of 0: given up at the first poll that finds a sum missing
        const unsigned long long t0 = (unsigned long long)wall_clock64();
        for (;;) {
            bool wait = false;
#pragma unroll
            for (int i = 0; i < kC; ++i) {
                g[i] = 0.0;
                if (i * 64 + lane < t.size) {
                    g[i] = ld_agent(q + i * 64 + lane);
                    wait |= __double_as_longlong(g[i]) == (long long)kResSentinel;
                }
            }
            if (!__any(wait)) break;
            if ((++spins & 63u) == 0 &&
                ((unsigned long long)wall_clock64() - t0 > limit ||
                 __hip_atomic_load(t.abort_flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))) {
                if (lane == 0) {
                    __hip_atomic_store(t.abort_flag, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    *t.ok = 0;
                }
                break;
            }
            __builtin_amdgcn_s_sleep(1);
        }
        double s = 0.0;
#pragma unroll
        for (int i = 0; i < kC; ++i)
            if (i * 64 < t.size) s += wave_sum(g[i]);
        if (lane == 0) s_tot[sum] = s;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NV; ++k) v[k] = s_tot[k];
    t.k += 1;
    return *t.ok != 0;
}

// The members' stores before their last reduction, seen by this workgroup's
// plain loads.
__device__ __forceinline__ void team_acquire() {
    if (threadIdx.x < 64) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    __syncthreads();
}

// Sums of a workgroup on its own (ONE): each tile of BS rows is summed as the
// member of a team that held it would, then the tiles as the members.
template <int BS, int NV, int RPT>
__device__ __forceinline__ void tile_sums(double (&v)[RPT][NV], double (&tot)[NV]) {
    constexpr int kW = BS / 64;
    static_assert(NV <= kW && RPT * NV <= 16, "a wave per sum, a lane of each row per tile and sum");
    __shared__ double s_part[RPT * NV][kW];
    __shared__ double s_tot[NV];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    if constexpr (RPT * NV > 4) {
        double a = RowSums<RPT * NV>::of(&v[0][0]);
        a += __shfl_xor(a, 16, 64);
        a += __shfl_xor(a, 32, 64);
        if (lane < RPT * NV) s_part[lane][wid] = a;
    } else {
#pragma unroll
        for (int q = 0; q < RPT; ++q)
#pragma unroll
            for (int k = 0; k < NV; ++k) {
                const double a = wave_sum(v[q][k]);
                if (lane == 0) s_part[q * NV + k][wid] = a;
            }
    }
    __syncthreads();
    if (wid < NV) {
        double mine = 0.0;
        if (lane < RPT) {
#pragma unroll
            for (int w = 0; w < kW; ++w) mine += s_part[lane * NV + wid][w];
        }
        mine = wave_sum(mine);
        if (lane == 0) s_tot[wid] = mine;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NV; ++k) tot[k] = s_tot[k];
}

// A thread's partial sums of one reduction, kept per row for tile_sums.
template <int BS, int NV, int RPT, bool ONE>
struct Sums {
    static constexpr int kR = ONE ? RPT : 1;
    double a[kR][NV] = {};
    __device__ __forceinline__ void add(int k, int i, double v) { a[ONE ? k : 0][i] += v; }
    __device__ __forceinline__ bool finish(ResTeam& t, double (&tot)[NV]) {
        if constexpr (ONE) {
            tile_sums<BS, NV, RPT>(a, tot);
            return true;
        } else {
#pragma unroll
            for (int i = 0; i < NV; ++i) tot[i] = a[0][i];
            return team_sum<BS, NV>(tot, t);
        }
    }
};

// Columns of RPT rows: int16 offsets two to a register, int32 columns one.
template <int WT, typename CI>
struct RowCols;
template <int WT>
struct RowCols<WT, int16_t> {
    int v[(WT + 1) / 2];
    __device__ __forceinline__ void load(const void* col, size_t n, int c) {
        const int16_t* p = (const int16_t*)col;
        int16_t t[WT];
#pragma unroll
        for (int i = 0; i < WT; ++i) t[i] = ld_once(p + (size_t)i * n + c);
#pragma unroll
        for (int i = 0; i < WT; i += 2)
            v[i / 2] = (int)(uint16_t)t[i] | (i + 1 < WT ? (int)((unsigned)(uint16_t)t[i + 1] << 16) : 0);
    }
    __device__ __forceinline__ int at(int i, int c) const { return c + (int)(int16_t)(v[i / 2] >> (16 * (i & 1))); }
    // Keeps the packed form live across the iterations: the compiler would
    // otherwise unpack every column once before the loop, for twice the
    // registers.
    __device__ __forceinline__ void pin() {
#pragma unroll
        for (int i = 0; i < (WT + 1) / 2; ++i) asm volatile("" : "+v"(v[i]));
    }
};
template <int WT>
struct RowCols<WT, int> {
    int v[WT];
    __device__ __forceinline__ void load(const void* col, size_t n, int c) {
        const int* p = (const int*)col;
#pragma unroll
        for (int i = 0; i < WT; ++i) v[i] = ld_once(p + (size_t)i * n + c);
    }
    __device__ __forceinline__ int at(int i, int) const { return v[i]; }
    __device__ __forceinline__ void pin() {
#pragma unroll
        for (int i = 0; i < WT; ++i) asm volatile("" : "+v"(v[i]));
    }
};

// RPT values per thread in registers, or in LDS.
template <int BS, int RPT, bool LDS, typename T = double>
struct Store;
template <int BS, int RPT, typename T>
struct Store<BS, RPT, false, T> {
    T v[RPT];
    __device__ __forceinline__ Store(T*) {}
    __device__ __forceinline__ T get(int k) const { return v[k]; }
    __device__ __forceinline__ void set(int k, T a) { v[k] = a; }
};
template <int BS, int RPT, typename T>
struct Store<BS, RPT, true, T> {
    T* p;
    __device__ __forceinline__ Store(T* base) : p(base + threadIdx.x) {}
    __device__ __forceinline__ T get(int k) const { return p[k * BS]; }
    __device__ __forceinline__ void set(int k, T a) { p[k * BS] = a; }
};

// The exchanged vectors: device memory with agent scope, or, for a system one
// workgroup solves alone (ONE), LDS.
template <int BS, int RPT, bool ONE>
struct Exchange;
template <int BS, int RPT>
struct Exchange<BS, RPT, false> {
    double* v[2];
    __device__ __forceinline__ Exchange(const ResSystem& sys, double*) : v{sys.e0, sys.e1} {}
    __device__ __forceinline__ void put(int buf, int c, double a) { put_agent(buf ? v[1] : v[0], c, a); }
    __device__ __forceinline__ double get(int buf, int c) const { return get_agent(buf ? v[1] : v[0], c); }
};
template <int BS, int RPT>
struct Exchange<BS, RPT, true> {
    double* v;
    __device__ __forceinline__ Exchange(const ResSystem& sys, double* lds) : v(lds - sys.c0) {}
    __device__ __forceinline__ void put(int buf, int c, double a) { v[buf * RPT * BS + c] = a; }
    __device__ __forceinline__ double get(int buf, int c) const { return v[buf * RPT * BS + c]; }
};

// acc + sum_i val[i][c] v(col_i), the values streamed once (the residuals at
// the start and the end).
template <int WT, typename CI, typename V>
__device__ __forceinline__ double res_gather(const RowCols<WT, CI>& col, const double* __restrict__ val, size_t n, int c,
                                             V&& v, double acc) {
    double a[WT], g[WT];
#pragma unroll
    for (int i = 0; i < WT; ++i) {
        a[i] = ld_once(val + (size_t)i * n + c);
        g[i] = v(col.at(i, c));
    }
#pragma unroll
    for (int i = 0; i < WT; ++i) acc = fma(a[i], g[i], acc);
    return acc;
}

// Scalars of the recurrences, the same in every thread of the team.
struct ResScalars {
    double gamma = 0, alpha = 0, beta = 0, tol_abs = 0, r0norm = 0, rho = 0;
    double delta = 0, gamma_old = 0, alpha_old = 0;
    int iter = 0, status = FVPCG_NOT_CONVERGED;
    bool done = false;
};

// pipe_scalars' steps (rows.hpp).
__device__ __forceinline__ void res_pipe_step(ResScalars& y, double gamma, double delta, double rho, bool first,
                                              int maxit) {
    if (first)
        y.r0norm = sqrt(rho);
    else
        y.iter += 1;
    y.rho = rho;
    if (sqrt(rho) <= y.tol_abs) {
        y.done = true;
        y.status = FVPCG_OK;
        return;
    }
    if (y.iter >= maxit) {
        y.done = true;
        y.status = FVPCG_NOT_CONVERGED;
        return;
    }
    double beta, den;
    if (first) {
        beta = 0.0;
        den = delta;
    } else {
        beta = gamma / y.gamma;
        den = delta - beta * gamma / y.alpha;
    }
    const double alpha = gamma / den;
    if (!(den > 0.0) || !isfinite(den) || !isfinite(alpha) || !isfinite(beta)) {
        y.done = true;
        y.status = FVPCG_BREAKDOWN;
        return;
    }
    y.gamma_old = y.gamma;
    y.alpha_old = y.alpha;
    y.gamma = gamma;
    y.delta = delta;
    y.alpha = alpha;
    y.beta = beta;
}

// A row index the compiler does not keep in a register from one pass to the
// next.
__device__ __forceinline__ int res_row(int c) {
    asm volatile("" : "+v"(c));
    return c;
}

// The k-th row of this thread and whether the system has it.
#define RES_ROWS(k, c)                                              \
    _Pragma("unroll") for (int k = 0; k < RPT; ++k)                 \
        if (const int c = res_row(sys.c0 + (k * t.size + t.rank) * BS + (int)threadIdx.x); c < sys.c1)

// Rows of an iteration are taken GR at a time: the gathers of a group are issued
// together, before any of its arithmetic and outside any branch (a row past
// the system's end reads the last row's entries and is then left out), so a
// wave waits for memory once per group and not once per row.
// RES_BASE starts a pass over the rows: the thread's first row, opaque to the
// compiler, which would otherwise form every row's indices and addresses once
// before the iterations and keep them in registers.
#define RES_BASE                                                             \
    const int base_ = res_row(sys.c0 + t.rank * BS + (int)threadIdx.x)
#define RES_ROW(k, c, cx)                                                    \
    const int c = base_ + (k) * t.size * BS;                                  \
    const int cx = c < sys.c1 ? c : sys.c1 - 1
constexpr int res_group(int rpt) { return rpt % 2 ? 1 : 2; }

// LDS of a resident solve: four vectors where registers cannot hold them
// (above 4 rows per thread at 512 threads, 2 at 1024), or the two exchange
// vectors of a workgroup on its own.
template <int BS, int RPT, bool ONE>
struct ResLds {
    static constexpr bool vectors = BS * RPT > 2048;
    static_assert(!(vectors && ONE), "a single workgroup's rows stay in registers");
    static constexpr int doubles = ONE ? 2 * RPT * BS : vectors ? 4 * RPT * BS : 1;
};

__device__ __forceinline__ void res_report(const ResTeam& t, ResOut* out, const ResScalars& y, double bnorm,
                                           double true_rr, bool zero_b, unsigned long long t0, unsigned long long t_it0,
                                           unsigned long long t_it1) {
    if (t.rank != 0 || threadIdx.x != 0) return;
    ResOut o;
    o.bnorm = bnorm;
    o.r0norm = y.r0norm;
    o.rho = y.rho;
    o.true_rr = true_rr;
    o.it_ticks = t_it1 - t_it0;
    o.ticks = (unsigned long long)wall_clock64() - t0;
    o.iter = y.iter;
    o.status = y.status;
    o.zero_b = zero_b ? 1 : 0;
    o.ok = 1;
    *out = o;
}

// Pipelined CG, folded or with its literal recurrences (LIT; see solve.hip):
// registers hold the iteration values, the columns, d, r and the row's own w;
// z, s, p and x are in LDS with RPT > 4.
template <int RPT, int WT, typename CI, bool JAC, bool LIT, bool ONE>
__device__ __forceinline__ void resident_pipe(const ResSystem& sys, ResTeam& t, double* lds, ResOut* out) {
    constexpr int BS = kResBsPipe;
    constexpr bool L = ResLds<BS, RPT, ONE>::vectors;
    const unsigned long long t_begin = (unsigned long long)wall_clock64();
    Exchange<BS, RPT, ONE> e(sys, lds);
    RowCols<WT, CI> col[RPT];
    double d[RPT], r[RPT], w[RPT];
    [[maybe_unused]] double u[LIT ? RPT : 1], qv[LIT ? RPT : 1];
    Store<BS, RPT, L> z(lds), s(lds + RPT * BS), p(lds + 2 * RPT * BS), x(lds + 3 * RPT * BS);
    // r = b - A x through buffer 1, (b, b)
    Sums<BS, 1, RPT, ONE> sb;
    RES_BASE;
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
        RES_ROW(k, c, cx);
        col[k].load(sys.col, sys.n, cx);
        d[k] = sys.d[cx];
    }
    RES_ROWS(k, c) {
        const double bc = sys.b[c], dc = d[k], xc = sys.x[c];
        const double rc = bc - res_gather<WT, CI>(col[k], sys.val, sys.n, c, [&](int j) { return sys.x[j]; }, dc * xc);
        r[k] = rc;
        x.set(k, xc);
        z.set(k, 0.0);
        s.set(k, 0.0);
        p.set(k, 0.0);
        if constexpr (LIT) {
            u[k] = JAC ? rc / dc : rc;
            qv[k] = 0.0;
        }
        e.put(1, c, rc);
        sb.add(k, 0, bc * bc);
    }
    double bb[1];
    bool ok = sb.finish(t, bb);
    ResScalars y;
    const double bnorm = sqrt(bb[0]);
    y.tol_abs = sys.tol * bnorm;
    const bool zero_b = bb[0] == 0.0;
    double val[RPT][WT];
    if (zero_b) {
        y.done = true;
        y.status = FVPCG_OK;
    } else if (ok) {
        // w = A M^-1 r
        Sums<BS, 3, RPT, ONE> sa;
        RES_ROWS(k, c) {
            double g[WT];
#pragma unroll
            for (int i = 0; i < WT; ++i) {
                val[k][i] = ld_once(sys.val_it + (size_t)i * sys.n + c);
                g[i] = e.get(1, col[k].at(i, c));
            }
            const double rc = r[k], dc = d[k];
            double wc = JAC ? rc : dc * rc;
#pragma unroll
            for (int i = 0; i < WT; ++i) wc = fma(val[k][i], g[i], wc);
            w[k] = wc;
            e.put(0, c, wc);
            const double uc = JAC ? rc / dc : rc;
            sa.add(k, 0, rc * uc);
            sa.add(k, 1, wc * uc);
            sa.add(k, 2, rc * rc);
        }
        double a[3];
        ok = sa.finish(t, a);
        res_pipe_step(y, a[0], a[1], a[2], true, sys.maxit);
    }
    const unsigned long long t_it0 = (unsigned long long)wall_clock64();
    for (int it = 0; ok && !y.done; ++it) {
        const int in = it & 1;
        const double alpha = y.alpha, beta = y.beta;
        Sums<BS, 3, RPT, ONE> sa;
        constexpr int GR = res_group(RPT);
        RES_BASE;
#pragma unroll
        for (int k0 = 0; k0 < RPT; k0 += GR) {
        double g[GR][WT];
#pragma unroll
        for (int q = 0; q < GR; ++q) {
            RES_ROW(k0 + q, c, cx);
            if (RPT > 3) col[k0 + q].pin();
#pragma unroll
            for (int i = 0; i < WT; ++i) g[q][i] = e.get(in, col[k0 + q].at(i, cx));
        }
#pragma unroll
        for (int k = k0; k < k0 + GR; ++k) {
            RES_ROW(k, c, cx);
            (void)cx;
            const double wc = w[k], dc = d[k];
            double nv = JAC ? wc : dc * wc;
#pragma unroll
            for (int i = 0; i < WT; ++i) nv = fma(val[k][i], g[k - k0][i], nv);
            const double zc = nv + beta * z.get(k);
            const double wn = wc - alpha * zc;
            if (c < sys.c1) e.put(in ^ 1, c, wn);
            const double sc = wc + beta * s.get(k);
            double rc = r[k];
            double uc;
            if constexpr (LIT) {
                const double mc = JAC ? wc / dc : wc;
                qv[k] = mc + beta * qv[k];
                uc = u[k];
            } else {
                uc = JAC ? rc / dc : rc;
            }
            const double pc = uc + beta * p.get(k);
            p.set(k, pc);
            x.set(k, x.get(k) + alpha * pc);
            rc -= alpha * sc;
            z.set(k, zc);
            s.set(k, sc);
            r[k] = rc;
            w[k] = wn;
            if constexpr (LIT) {
                uc -= alpha * qv[k];
                u[k] = uc;
            } else {
                uc = JAC ? rc / dc : rc;
            }
            if (c < sys.c1) {
                sa.add(k, 0, rc * uc);
                sa.add(k, 1, wn * uc);
                sa.add(k, 2, rc * rc);
            }
        }
        }
        double a[3];
        ok = sa.finish(t, a);
        res_pipe_step(y, a[0], a[1], a[2], false, sys.maxit);
    }
    const unsigned long long t_it1 = (unsigned long long)wall_clock64();
    if (!ok) return;
    // x, also through buffer 0 (all reads of it were done before the last
    // reduction), and ||b - A x||^2
    RES_ROWS(k, c) {
        if (zero_b) x.set(k, 0.0);
        sys.x[c] = x.get(k);
        e.put(0, c, x.get(k));
    }
    double rr[1];
    if (!Sums<BS, 1, RPT, ONE>().finish(t, rr)) return;
    Sums<BS, 1, RPT, ONE> sr;
    RES_ROWS(k, c) {
        const double rc = sys.b[c] - res_gather<WT, CI>(col[k], sys.val, sys.n, c, [&](int j) { return e.get(0, j); }, d[k] * x.get(k));
        sr.add(k, 0, rc * rc);
    }
    if (!sr.finish(t, rr)) return;
    res_report(t, out, y, bnorm, rr[0], zero_b, t_begin, t_it0, t_it1);
}

// Standard preconditioned CG.  Its two reductions per iteration are the only
// synchronisations: p = z + beta p is formed by the row that owns an entry and
// again, from the same z and p with the same rounding, by every row that
// gathers it, so no third one is needed between the new direction and the
// product.  Registers hold the values, the columns and q; x, r, p and d are
// in LDS with RPT > 2.  e0 carries z, e1 the previous p; both are stored after
// the first reduction (everybody has gathered the old ones) and read after the
// second.
template <int RPT, int WT, typename CI, bool JAC, bool ONE>
__device__ __forceinline__ void resident_cg(const ResSystem& sys, ResTeam& t, double* lds, ResOut* out) {
    constexpr int BS = kResBsCg;
    constexpr bool L = ResLds<BS, RPT, ONE>::vectors;
    const unsigned long long t_begin = (unsigned long long)wall_clock64();
    Exchange<BS, RPT, ONE> e(sys, lds);
    RowCols<WT, CI> col[RPT];
    double val[RPT][WT], q[RPT];
    Store<BS, RPT, L> x(lds), r(lds + RPT * BS), p(lds + 2 * RPT * BS), d(lds + 3 * RPT * BS);
    // r = b - A x, z = M^-1 r, p = z
    Sums<BS, 3, RPT, ONE> s0;
    RES_BASE;
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
        RES_ROW(k, c, cx);
        col[k].load(sys.col, sys.n, cx);
    }
    RES_ROWS(k, c) {
        const double bc = sys.b[c], dc = sys.d[c], xc = sys.x[c];
        double g[WT];
#pragma unroll
        for (int i = 0; i < WT; ++i) {
            val[k][i] = ld_once(sys.val + (size_t)i * sys.n + c);
            g[i] = sys.x[col[k].at(i, c)];
        }
        double ax = dc * xc;
#pragma unroll
        for (int i = 0; i < WT; ++i) ax = fma(val[k][i], g[i], ax);
        const double rc = bc - ax;
        const double zc = JAC ? rc / dc : rc;
        x.set(k, xc);
        r.set(k, rc);
        p.set(k, zc);
        d.set(k, dc);
        e.put(0, c, zc);
        e.put(1, c, 0.0);
        s0.add(k, 0, rc * zc);
        s0.add(k, 1, rc * rc);
        s0.add(k, 2, bc * bc);
    }
    double a0[3];
    bool ok = s0.finish(t, a0);
    ResScalars y;
    const double bnorm = sqrt(a0[2]);
    const bool zero_b = a0[2] == 0.0;
    if (zero_b) {
        y.done = true;
        y.status = FVPCG_OK;
    } else {
        y.tol_abs = sys.tol * bnorm;
        y.gamma = a0[0];
        y.rho = a0[1];
        y.r0norm = sqrt(a0[1]);
        if (y.r0norm <= y.tol_abs) {
            y.done = true;
            y.status = FVPCG_OK;
        } else if (sys.maxit <= 0) {
            y.done = true;
        }
    }
    const unsigned long long t_it0 = (unsigned long long)wall_clock64();
    for (int it = 0; ok && !y.done; ++it) {
        const double beta = y.beta;
        const bool first = it == 0;
        // q = A p; delta = (p, q)
        Sums<BS, 1, RPT, ONE> s1;
        RES_BASE;
#pragma unroll
        for (int k = 0; k < RPT; ++k) {
            RES_ROW(k, c, cx);
            double gz[WT], gp[WT];
            if (RPT > 1) col[k].pin();
#pragma unroll
            for (int i = 0; i < WT; ++i) {
                const int j = col[k].at(i, cx);
                gz[i] = e.get(0, j);
                gp[i] = e.get(1, j);  // zeros before the first iteration
            }
            const double pc = p.get(k);
            double qc = d.get(k) * pc;
#pragma unroll
            for (int i = 0; i < WT; ++i) qc = fma(val[k][i], first ? gz[i] : fma(beta, gp[i], gz[i]), qc);
            q[k] = qc;
            if (c < sys.c1) s1.add(k, 0, pc * qc);
        }
        double a1[1];
        ok = s1.finish(t, a1);
        if (!ok) break;
        const double delta = a1[0];
        if (!(delta > 0.0) || !isfinite(delta) || !isfinite(y.gamma)) {
            y.done = true;
            y.status = FVPCG_BREAKDOWN;
            break;
        }
        const double alpha = y.gamma / delta;
        // x += alpha p, r -= alpha q, z = M^-1 r
        Sums<BS, 2, RPT, ONE> s2;
        RES_ROWS(k, c) {
            const double pc = p.get(k), dc = d.get(k);
            const double rc = r.get(k) - alpha * q[k];
            r.set(k, rc);
            const double zc = JAC ? rc / dc : rc;
            e.put(0, c, zc);
            e.put(1, c, pc);
            x.set(k, x.get(k) + alpha * pc);
            s2.add(k, 0, rc * zc);
            s2.add(k, 1, rc * rc);
        }
        double a2[2];
        ok = s2.finish(t, a2);
        y.iter += 1;
        y.rho = a2[1];
        if (sqrt(a2[1]) <= y.tol_abs) {
            y.done = true;
            y.status = FVPCG_OK;
        } else if (y.iter >= sys.maxit) {
            y.done = true;
        } else {
            y.beta = a2[0] / y.gamma;
            y.gamma = a2[0];
            RES_ROWS(k, c) {
                const double rc = r.get(k);
                const double zc = JAC ? rc / d.get(k) : rc;
                p.set(k, fma(y.beta, p.get(k), zc));
            }
        }
    }
    const unsigned long long t_it1 = (unsigned long long)wall_clock64();
    if (!ok) return;
    // x, also through buffer 0 (see resident_pipe; a breakdown ends on the
    // first reduction, after which nobody reads it either), and ||b - A x||^2
    RES_ROWS(k, c) {
        if (zero_b) x.set(k, 0.0);
        sys.x[c] = x.get(k);
        e.put(0, c, x.get(k));
    }
    double rr[1];
    if (!Sums<BS, 1, RPT, ONE>().finish(t, rr)) return;
    Sums<BS, 1, RPT, ONE> sr;
    RES_ROWS(k, c) {
        double g[WT];
#pragma unroll
        for (int i = 0; i < WT; ++i) g[i] = e.get(0, col[k].at(i, c));
        double ax = d.get(k) * x.get(k);
#pragma unroll
        for (int i = 0; i < WT; ++i) ax = fma(val[k][i], g[i], ax);
        const double rc = sys.b[c] - ax;
        sr.add(k, 0, rc * rc);
    }
    if (!sr.finish(t, rr)) return;
    res_report(t, out, y, bnorm, rr[0], zero_b, t_begin, t_it0, t_it1);
}

// A run of FP32 folded pipelined iterations of the mixed-precision solve
// (solve.hip, between two FP64 updates): the recurrence vectors are read from
// memory at the start and written back at the end, the iterations between
// keep them on chip, w, the values and the columns in registers, z, s, p and r
// in LDS.  d and the correction, which only its own row reads, come from the L2
// (4 and 8 bytes a row).  The scalars
// are those of `st`, as pipe_scalars steps them; member 0 writes them back.
// A team that does not come together sets st_skip->done = kResNoTeam, which
// makes the update kernels that follow do nothing; a wait given up sets
// kResLost.
constexpr int32_t kResNoTeam = 2, kResLost = 3;

template <int RPT, int WT, typename CI>
__device__ __forceinline__ void resident_pipe32(const PipeVec<float>& a, int n, int iters, ResTeam& t, DevState* st,
                                                DevState* st_skip, float* lds) {
    constexpr int BS = kResBsMixed;
    struct {
        int c0, c1;
    } sys{0, n};
    RowCols<WT, CI> col[RPT];
    float val[RPT][WT], w[RPT];
    Store<BS, RPT, true, float> z(lds), s(lds + RPT * BS), p(lds + 2 * RPT * BS), r(lds + 3 * RPT * BS);
    RES_BASE;
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
        RES_ROW(k, c, cx);
        (void)c;
        col[k].load(a.col, (size_t)n, cx);
#pragma unroll
        for (int i = 0; i < WT; ++i) val[k][i] = ld_once(a.val + (size_t)i * n + cx);
        w[k] = a.w_in[cx];
        r.set(k, a.r[cx]);
        z.set(k, a.z[cx]);
        s.set(k, a.s[cx]);
        p.set(k, a.p[cx]);
    }
    ResScalars y;
    y.gamma = st->gamma;
    y.delta = st->delta;
    y.alpha = st->alpha;
    y.beta = st->beta;
    y.gamma_old = st->gamma_old;
    y.alpha_old = st->alpha_old;
    y.tol_abs = st->tol_abs;
    y.rho = st->rho;
    y.iter = st->iter;
    y.status = st->status;
    const int maxit = st->maxit;
    float* const e0 = const_cast<float*>(a.w_in);
    bool ok = true;
    for (int it = 0; it < iters && !y.done; ++it) {
        const float* w_in = (it & 1) ? a.w_out : e0;
        float* w_out = (it & 1) ? e0 : a.w_out;
        const float alpha = (float)y.alpha, beta = (float)y.beta;
        Sums<BS, 3, RPT, false> sa;
        constexpr int GR = res_group(RPT);
        RES_BASE;
#pragma unroll
        for (int k0 = 0; k0 < RPT; k0 += GR) {
        float g[GR][WT], dg[GR], xg[GR];
#pragma unroll
        for (int q = 0; q < GR; ++q) {
            RES_ROW(k0 + q, c, cx);
            (void)c;
            col[k0 + q].pin();
#pragma unroll
            for (int i = 0; i < WT; ++i) g[q][i] = get_agent(w_in, col[k0 + q].at(i, cx));
            dg[q] = get_plain(a.d, cx);
            xg[q] = get_plain(a.x, cx);
        }
#pragma unroll
        for (int k = k0; k < k0 + GR; ++k) {
            RES_ROW(k, c, cx);
            (void)cx;
            const float dc = dg[k - k0];
            const float wc = w[k];
            float nv = wc;
#pragma unroll
            for (int i = 0; i < WT; ++i) nv = fma(val[k][i], g[k - k0][i], nv);
            const float zc = nv + beta * z.get(k);
            const float wn = wc - alpha * zc;
            const float sc = wc + beta * s.get(k);
            float rc = r.get(k);
            float uc = rc / dc;
            const float pc = uc + beta * p.get(k);
            p.set(k, pc);
            rc -= alpha * sc;
            z.set(k, zc);
            s.set(k, sc);
            r.set(k, rc);
            w[k] = wn;
            uc = rc / dc;
            if (c < sys.c1) {
                put_agent(w_out, c, wn);
                put_plain(a.x, c, xg[k - k0] + alpha * pc);
                sa.add(k, 0, (double)rc * (double)uc);
                sa.add(k, 1, (double)wn * (double)uc);
                sa.add(k, 2, (double)rc * (double)rc);
            }
        }
        }
        double q[3];
        ok = sa.finish(t, q);
        if (!ok) break;
        res_pipe_step(y, q[0], q[1], q[2], false, maxit);
    }
    if (!ok) {
        if (threadIdx.x == 0) st_skip->done = kResLost;
        return;
    }
    // w lies where the launches would have left it (a stopped run leaves w as
    // its last iteration's; nobody reads it then)
    RES_ROWS(k, c) {
        a.r[c] = r.get(k);
        a.z[c] = z.get(k);
        a.s[c] = s.get(k);
        a.p[c] = p.get(k);
    }
    if (t.rank == 0 && threadIdx.x == 0) {
        st->gamma = y.gamma;
        st->delta = y.delta;
        st->alpha = y.alpha;
        st->beta = y.beta;
        st->gamma_old = y.gamma_old;
        st->alpha_old = y.alpha_old;
        st->rho = y.rho;
        st->iter = y.iter;
        st->status = y.status;
        st->done = y.done ? 1 : 0;
    }
}

// Folded pipelined CG of systems beyond what the chip holds whole (up to 64
// tiles per member, 8.4M cells): the iterations of k_pipe_iter (solve.hip) in
// one launch, with the matrix streamed and as many of the recurrence vectors
// on chip as fit.  A thread has 64 doubles of registers for them, as four
// vectors of 16 indexed by the (uniform) tile number, and 32 in LDS:
//   up to 16 tiles (2.1M cells)  z, s, p and r in registers, x and d in LDS;
//   up to 32 tiles (4.2M)        z and s in registers, p in LDS;
//   up to 64 tiles (8.4M)        z in registers, s in LDS for 32 tiles.
// Every resident vector saves its read and its write.  Per iteration, against
// the launches (bandwidth-bound at 6.3 TB/s): 35.5 us against 62.7 at 2.1M
// cells, 75 against 109 at 4.1M, 143-146 against 182 at 7.1M.  A row's loads are all
// issued before its gathers are waited for: with r and p read after them 209 us
// at 7.1M.  w is stored with agent
// scope; its gathers go through the L2 caches (uncached they would fetch every
// entry six times), so each member invalidates them after the reduction.  x in
// memory is updated every second iteration (PairX), pending updates at the
// end.  The scalars are those of `st`, read at the start and written back by
// member 0, with out->ok = 1.
using Tile16 = double __attribute__((ext_vector_type(16)));
constexpr int kStreamTiles = 64, kStreamLdsTiles = 32;

template <int NT, int WT, typename CI, bool JAC>
__device__ __forceinline__ void resident_stream(const PipeVec<double>& a, int n, ResTeam& t, double* lds, DevState* st,
                                                ResOut* out) {
    constexpr int BS = kResBsPipe, CH = NT / 16;
    static_assert(NT == 16 || NT == 32 || NT == 64, "16 tiles to a register vector");
    constexpr bool kSReg = NT <= 32, kPR = NT == 16;  // s in registers; p, r in registers and x, d in LDS
    // What the 256 MB last-level cache keeps from one iteration to the next: w
    // and d, and the columns if they are int16 (85 MB at 7.08M cells), else r
    // (57 MB, read and written; with int32 columns kept 172 us against 157).
    constexpr bool kKeepCol = sizeof(CI) == 2;
    Tile16 z[CH], s[kSReg ? CH : 1], p[kPR ? CH : 1], r[kPR ? CH : 1];
    double* const l0 = lds + threadIdx.x;               // x | p | s
    double* const l1 = lds + NT * BS + threadIdx.x;     // d (16 tiles only)
    const int G = t.size, tiles = (n + BS - 1) / BS;
    const int mine = t.rank < tiles ? (tiles - t.rank + G - 1) / G : 0;
    const CI* __restrict__ col = (const CI*)a.col;
#pragma unroll
    for (int h = 0; h < CH; ++h) {
        z[h] = 0.0;
        if constexpr (kSReg) s[h] = 0.0;
        if constexpr (kPR) p[h] = 0.0;
    }
    for (int k = 0; k < mine; ++k) {
        const int c = (k * G + t.rank) * BS + (int)threadIdx.x;
        const int cx = c < n ? c : n - 1;
        if constexpr (kPR) {
            r[0][k] = a.r[cx];
            l0[k * BS] = a.x[cx];
            l1[k * BS] = a.d[cx];
        } else if constexpr (kSReg) {
            l0[k * BS] = 0.0;
        } else {
            if (k < kStreamLdsTiles) l0[k * BS] = 0.0;
        }
    }
    ResScalars y;
    y.gamma = st->gamma;
    y.alpha = st->alpha;
    y.beta = st->beta;
    y.alpha_old = st->alpha_old;
    y.gamma_old = st->gamma_old;
    y.tol_abs = st->tol_abs;
    y.r0norm = st->r0norm;
    y.rho = st->rho;
    y.iter = st->iter;
    const int maxit = st->maxit;
    double* const e0 = const_cast<double*>(a.w_in);
    const unsigned long long t0 = (unsigned long long)wall_clock64();
    bool ok = true;
    for (int it = 0; !y.done; ++it) {
        const double* w_in = (it & 1) ? a.w_out : e0;
        double* w_out = (it & 1) ? e0 : a.w_out;
        const double alpha = y.alpha, beta = y.beta, alpha_prev = y.alpha_old;
        const bool odd = (it & 1) != 0;
        double q[3] = {0.0, 0.0, 0.0};
#pragma unroll
        for (int h = 0; h < CH; ++h) {
            const int m = min(16, mine - 16 * h);
            for (int j = 0; j < m; ++j) {
                const int k = 16 * h + j;
                const int c = (k * G + t.rank) * BS + (int)threadIdx.x;
                if (c >= n) continue;
                // every load of the row before the gather's wait
                const bool s_lds = !kSReg && 16 * h < kStreamLdsTiles;  // known per h
                const double wc = w_in[c];
                const double dc = kPR ? l1[k * BS] : a.d[c];
                double rc = kPR ? r[h][j] : kKeepCol ? ld_once(a.r + c) : a.r[c];
                const double pold = kPR ? p[h][j] : kSReg ? l0[k * BS] : ld_once(a.p + c);
                const double so = kSReg ? s[h][j] : s_lds ? l0[k * BS] : ld_once(a.s + c);
                double xc = 0.0;
                if constexpr (!kPR)
                    if (odd) xc = ld_once(a.x + c);
                const double nv = row_gather<double, WT, CI, kKeepCol>(col, a.val, n, c, w_in, JAC ? wc : dc * wc);
                const double zc = nv + beta * z[h][j];
                z[h][j] = zc;
                const double sc = wc + beta * so;
                if constexpr (kSReg)
                    s[h][j] = sc;
                else if (s_lds)
                    l0[k * BS] = sc;
                else
                    st_once(a.s + c, sc);
                double uc = JAC ? rc / dc : rc;
                const double pc = uc + beta * pold;
                if constexpr (kPR) {
                    p[h][j] = pc;
                    l0[k * BS] = l0[k * BS] + alpha * pc;
                } else {
                    if constexpr (kSReg)
                        l0[k * BS] = pc;
                    else
                        st_once(a.p + c, pc);
                    if (odd) {
                        const double xa = xc + alpha_prev * pold;
                        st_once(a.x + c, xa + alpha * pc);
                    }
                }
                rc -= alpha * sc;
                const double wn = wc - alpha * zc;
                if constexpr (kPR)
                    r[h][j] = rc;
                else if constexpr (kKeepCol)
                    st_once(a.r + c, rc);
                else
                    a.r[c] = rc;
                st_agent(w_out + c, wn);
                uc = JAC ? rc / dc : rc;
                q[0] += rc * uc;
                q[1] += wn * uc;
                q[2] += rc * rc;
            }
        }
        ok = team_sum<BS, 3>(q, t);
        if (!ok) return;
        // the members' w: no stale copy in this XCD's caches
        if (threadIdx.x < 64) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        __syncthreads();
        res_pipe_step(y, q[0], q[1], q[2], false, maxit);
    }
    for (int k = 0; k < mine; ++k) {
        const int c = (k * G + t.rank) * BS + (int)threadIdx.x;
        if (c >= n) continue;
        if constexpr (kPR)
            a.x[c] = l0[k * BS];
        else if (y.iter & 1)
            a.x[c] += y.alpha * (kSReg ? l0[k * BS] : a.p[c]);
    }
    if (t.rank == 0 && threadIdx.x == 0) {
        st->rho = y.rho;
        st->iter = y.iter;
        st->status = y.status;
        st->done = 1;
        out->it_ticks = (unsigned long long)wall_clock64() - t0;
        out->ok = 1;
    }
}

}  // namespace fvpcg

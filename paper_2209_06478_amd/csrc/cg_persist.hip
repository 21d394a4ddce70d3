// The CG loop in one launch: workgroups that stay, each with a run of rows.
//
// The three-kernel iteration pays for its launches and for streaming x, r, q
// and p through memory.  Here every workgroup of one launch (at most one per
// CU) keeps the x, r, q and p of its rows in LDS for the whole
// solve; between iterations only r crosses workgroups, through memory.  An
// iteration has two grid-wide meetings: the p.q sum, and the r.r sum, with
// which the new r goes out.  p = r + beta p is formed by every workgroup for
// its own rows and for the columns its rows reach, from the r of their owners
// and the p it had there before (one fused multiply-add on both sides: the
// same bits), so p needs no meeting of its own.  The columns a workgroup's
// rows reach have to fit in LDS with its rows.  Where they do not (HPCG 104^3
// in FP64), a form that published p in a third meeting and staged it per tile
// and cluster of diagonals ran 57-65 us an iteration against 58 us for the
// launch-per-step loop, and 110 against 47 at 128^3 with BF16 values (a CU's
// one workgroup keeps too few loads in flight behind two barriers per tile):
// not kept, those systems take the other loop.
//
// A meeting: every workgroup stores its sum (one 64-bit word) in its slot and
// then reads the slots of all, so the meeting itself carries the reduction,
// each workgroup forms the same total in the same order, and no counter is
// contended.  A slot holds a NaN pattern that no sum has (EMPTY) until it is
// written; four sets of slots take turns, and a workgroup clears its slot of
// the set after next: it has seen everyone's word of the set before, so
// everyone has finished reading the set two before.  Words and r are stored
// and loaded past the L2s, which are not coherent between XCDs within a
// launch; each wave waits for its stores before its workgroup's word goes
// out.  The words lie in the memory of q, which the launch keeps in LDS.
// Measured alone: 2.4 us over 8 workgroups, 4.5 us over 256 (an
// agent-scope fence per wave instead of the plain stores past the L2: 38 us).
//
// Whole solves to 1e-10, launch-per-step loop -> now: HPCG 16^3 CSR 774 -> 340
// us (9.8 -> 6.8 us an iteration, 292 -> 51 us beside them: no captures, no
// launches past convergence, x0's product and the true residual in the same
// launch), 32^3 CSR 1460 -> 900, 48^3 CSR 2878 -> 1830, 64^3 ELL 4206 -> 3064,
// 64^3 DIA 3602 -> 2962; SPD bands, CSR: 20k rows 746 -> 357, 200k rows 1309
// -> 714.  256 rows a workgroup at least: 512 cost 16^3 1.3 us an iteration
// (a CU is fed at 60 GB/s), fewer only add words to the meetings.
//
// All workgroups of a launch have to be on the device together.  A launch has
// no more of them than there are CUs, each fits on a CU by itself, and the
// launches in flight share the CUs out among them (CuShare: a solve waits for
// its turn), so whatever else runs only has to finish.  (hipLaunchCooperative-
// Kernel gives the same guarantee, but after such launches from several
// threads' streams, kernels of different streams no longer overlapped on the
// device: four-stream serving went from 8 to 26 ms.)  Should a workgroup not
// show up within WAIT_TICKS all the same (kernels of other processes that
// wait like this, CUs masked off), whoever waits gives the launch up and
// everybody leaves.  Results are stored after the last meeting, by all
// workgroups or by none (outcome.hpp): a launch's time may also be up in that
// meeting, when others are past it.  The solve then goes on from the last
// launch that was kept, a step per launch instead of a meeting (PHASE_*): the
// same workgroups with the same rows and sums in the same order, so its bits
// do not depend on what else the device was doing.
#include <condition_variable>
#include <cmath>
#include <cstdlib>
#include <mutex>
#include <type_traits>

#include "cg_common.hpp"
#include "outcome.hpp"
#include "wg_kernels.hpp"

namespace dsm {

constexpr int PG = 256;                   // workgroups at most
constexpr int SETS = 4, SUMS = 2;         // slot sets, sums per meeting at most
constexpr int MAX_DIAGS = 1024;           // DIA offsets kept in LDS
constexpr u64 EMPTY = 0x7ff4dead7ff4deadull;
constexpr u64 NAN_WORD = 0x7ff8000000000000ull;
constexpr long long WAIT_TICKS = 10000000;  // of the 100 MHz clock: 0.1 s
constexpr int ALONE = 64;                 // solves that go by steps after one that was given up

// The steps of a solve between meetings, as launches of their own.
enum { PHASE_INIT, PHASE_PQ, PHASE_RR, PHASE_TRUE };

struct CgpArgs {
    int n, rpw;  // rows, rows per workgroup (a multiple of 64)
    int win;     // columns a row reaches at most on each side
    // the matrix
    const i32 *rp, *col;
    int lanes;
    const void *val;
    const i32 *offs;
    int nd;  // ELL: nd slots
    i64 pitch;
    const i32 *ecol;
    // vectors
    const void *b, *x_in;
    void *x_out, *x_work;  // where x goes when the solve is done, and before
    void *p[2];  // p of iteration k, after it in p[(k + par) & 1]; an unfinished launch leaves r in the other
    void *r;
    int par;
    const double *dinv;
    u64 *slots;
    u32 *outcome;
    CgState *st, *host;
    double tol, pcont;
    long long maxit;
    int steps;    // iterations of this launch at most
    int resume;   // x_work, r, p and *st hold an unfinished solve
    int x0_zero;  // x_in is zero (and not read)
    int want_true;
    // a solve by steps
    void *q;
    double *part;  // the workgroups' sums: PG of each of three
    int phase;
};

template <class T>
__device__ __forceinline__ T ld_agent(const T *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <class T>
__device__ __forceinline__ void st_agent(T *p, T v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__global__ void k_slots_clear(u64 *slots, int n, u32 *outcome, u32 open) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) slots[i] = EMPTY;
    if (i == 0) *outcome = open;
}

// The launch's outcome (outcome.hpp).
struct OutcomeWord {
    u32 *p;
    __device__ __forceinline__ u32 load() const { return ld_agent(p); }
    __device__ __forceinline__ u32 swap(u32 from, u32 to) const {
        __hip_atomic_compare_exchange_strong(p, &from, to, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT);
        return from;
    }
};

struct Meeting {
    u64 *slots;
    u32 *outcome;
    int *ok;  // LDS: [0] is 1 until the launch has been given up, [1] the end of kept()
    WgSum<> total;
    int set = 0;

    // v[k]: this thread's part of sum k on entry, the grid's sum on return.
    // What the workgroup stored before is visible to the others' loads past
    // the L2 afterwards.  False: give up.
    template <int N>
    __device__ __forceinline__ bool operator()(double (&v)[N]) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
        for (int k = 0; k < N; k++) v[k] = total(v[k]);
        const u32 G = gridDim.x;
        u64 *now = slots + (size_t)set * SUMS * G, *clear = slots + (size_t)((set + 2) % SETS) * SUMS * G;
        if (threadIdx.x == 0) {
#pragma unroll
            for (int k = 0; k < N; k++)
                st_agent(now + k * G + blockIdx.x, v[k] == v[k] ? __builtin_bit_cast(u64, v[k]) : NAN_WORD);
#pragma unroll
            for (int k = 0; k < SUMS; k++) st_agent(clear + k * G + blockIdx.x, EMPTY);
        }
        u64 w[N];
#pragma unroll
        for (int k = 0; k < N; k++) w[k] = 0;
        if (threadIdx.x < G) {
            const long long t0 = wall_clock64();
            for (u32 tries = 1;; tries++) {
                bool all = true;
#pragma unroll
                for (int k = 0; k < N; k++) {
                    w[k] = ld_agent(now + k * G + threadIdx.x);
                    all = all && w[k] != EMPTY;
                }
                if (all) break;
                if (tries % 64 == 0 && outcome_gives_up(OutcomeWord{outcome}, wall_clock64() - t0 > WAIT_TICKS)) {
                    *ok = 0;
                    break;
                }
            }
        }
#pragma unroll
        for (int k = 0; k < N; k++) v[k] = total(__builtin_bit_cast(double, w[k]));
        set = (set + 1) % SETS;
        asm volatile("" ::: "memory");
        return *ok != 0;
    }

    // After the launch's last meeting: whether the results may be stored.
    __device__ __forceinline__ bool kept() {
        if (threadIdx.x == 0) ok[1] = outcome_keeps(OutcomeWord{outcome});
        __syncthreads();
        return ok[1] != 0;
    }
};

// FMT: DSM_CSR, DSM_ELL or DSM_DIA.  STEP: one step of the solve (A.phase)
// instead of its loop, its vectors in memory between steps.
template <class V, class X, int FMT, bool JAC, bool STEP>
__global__ void __launch_bounds__(BB) k_cg_persist(const CgpArgs A) {
    extern __shared__ __align__(16) char dyn[];
    __shared__ double sums[2 * NW];
    __shared__ int ok[2];
    __shared__ i32 offs[FMT == DSM_DIA ? MAX_DIAGS : 1];
    __shared__ WaveRows wrows[NW];  // CSR: held in registers they cost spills
    const int tid = threadIdx.x;
    const int r0 = blockIdx.x * A.rpw, rows = min(A.rpw, A.n - r0);
    // LDS: x, r, q of the rows, p of the columns [r0 - win, r0 + rpw + win) and
    // a zero word
    X *xs = (X *)dyn, *rs = xs + A.rpw, *qs = rs + A.rpw, *pw = qs + A.rpw;
    const int win = A.win, W = A.rpw + 2 * win;
    X *ps = pw + win;
    const X *pc = pw - (r0 - win);  // p by column
    const int zero = r0 - win + W;  // pc[zero] = 0
    X *prod = pw + W + 2;           // CSR: products, then row pointers
    i32 *rps = (i32 *)(prod + NW * WCH);
    const X *b = (const X *)A.b;
    X *r = (X *)A.r, *const pb[2] = {(X *)A.p[0], (X *)A.p[1]};

    if (tid == 0) {
        ok[0] = 1;
        pw[W] = 0;
    }
    if (FMT == DSM_CSR)
        for (int i = tid; i <= rows; i += BB) rps[i] = A.rp[r0 + i];
    if (FMT == DSM_DIA)  // zero-padded to a multiple of 16
        for (int i = tid; i < (A.nd + 15) / 16 * 16; i += BB) offs[i] = A.offs[i];
    __syncthreads();
    if (FMT == DSM_CSR) {
        const WaveRows w = wave_rows(rows, rps);
        if (tid % WAVE == 0) wrows[tid / WAVE] = w;
    }
    Meeting meet{A.slots, A.outcome, ok, WgSum<>{sums}};

    // The vector of a product, by column: src as it is, or the direction p =
    // z + beta src (z + nothing where there is no src), z = r or D^-1 r.
    struct Vec {
        const X *src;
        bool dir;
        X beta;
    };
    auto dinv = [&](int j) { return JAC ? A.dinv[j] : 1.0; };
    auto direction = [&](const Vec &v, X z, X old) { return v.src ? (X)fma(v.beta, old, z) : z; };
    auto precond = [&](X ri, int j) { return JAC ? (X)(ri * dinv(j)) : ri; };

    // q = A (v); the workgroup's rows of v are in ps
    auto product = [&](const Vec v) {
        // the columns around the workgroup's rows
        const X *from = v.dir ? r : v.src;
        auto around = [&](auto hu) {
            constexpr int HU = decltype(hu)::value;  // loads in flight
            for (int i0 = tid; i0 < 2 * win; i0 += HU * BB) {
                X z[HU];
                int t[HU], j[HU];
#pragma unroll
                for (int u = 0; u < HU; u++) {
                    const int i = i0 + u * BB;
                    t[u] = i < win ? i : rows + i;
                    j[u] = i < 2 * win ? r0 - win + t[u] : -1;
                    z[u] = ld_agent(from + (j[u] >= 0 && j[u] < A.n ? j[u] : 0));
                }
#pragma unroll
                for (int u = 0; u < HU; u++) {
                    if (i0 + u * BB >= 2 * win) break;
                    const bool in = j[u] >= 0 && j[u] < A.n;
                    const X e = v.dir ? direction(v, precond(z[u], in ? j[u] : 0), pw[t[u]]) : z[u];
                    pw[t[u]] = in ? e : (X)0;
                }
            }
        };
        if (2 * win <= BB) around(std::integral_constant<int, 1>());
        else around(std::integral_constant<int, 8>());
        __syncthreads();
        if constexpr (FMT == DSM_CSR) {
            const WaveRows &w = wrows[tid / WAVE];
            const WaveRows mine{
                __builtin_amdgcn_readfirstlane(w.r), __builtin_amdgcn_readfirstlane(w.r1),
                __builtin_amdgcn_readfirstlane(w.e), __builtin_amdgcn_readfirstlane(w.e1)};
            wg_spmv_csr<X>(mine, A.lanes, A.col, (const V *)A.val, pc, zero, qs, rps, prod);
            __syncthreads();
        } else if constexpr (FMT == DSM_ELL) {
            if (rows <= BB)
                wg_spmv_ell<X, 1, 16, false>(rows, A.nd, (int)A.pitch, A.ecol + r0, (const V *)A.val + r0, pc, zero,
                                             qs);
            else
                wg_spmv_ell<X, 2, 8, false>(rows, A.nd, (int)A.pitch, A.ecol + r0, (const V *)A.val + r0, pc, zero,
                                            qs);
        } else {
            if (rows <= BB)
                wg_spmv_dia<X, 1, 16>(rows, r0, A.n, A.nd, A.pitch, offs, (const V *)A.val + r0, pc, zero, qs);
            else
                wg_spmv_dia<X, 2, 8>(rows, r0, A.n, A.nd, A.pitch, offs, (const V *)A.val + r0, pc, zero, qs);
        }
    };
    auto publish = [&](X *to, int i, X v) { st_agent(to + r0 + i, v); };

    if constexpr (STEP) {
        WgSum<> total{sums};
        auto put = [&](int k, double v) {
            v = total(v);
            if (tid == 0) A.part[k * PG + blockIdx.x] = v;
        };
        X *const xw = (X *)A.x_work, *const q = (X *)A.q;
        double s[2] = {0, 0};
        if (A.phase == PHASE_INIT) {
            if (!A.x0_zero) {
                for (int i = tid; i < rows; i += BB) ps[i] = xs[i] = ((const X *)A.x_in)[r0 + i];
                product(Vec{(const X *)A.x_in, false, (X)0});
            }
            for (int i = tid; i < rows; i += BB) {
                const X ri = A.x0_zero ? b[r0 + i] : b[r0 + i] - qs[i];
                xw[r0 + i] = A.x0_zero ? (X)0 : xs[i];
                r[r0 + i] = ri;
                s[0] += JAC ? (double)ri * ((double)ri * dinv(r0 + i)) : (double)ri * (double)ri;
                s[1] += (double)ri * (double)ri;
            }
            put(0, s[0]);
            put(1, s[1]);
            return;
        }
        if (A.phase == PHASE_TRUE) {
            for (int i = tid; i < rows; i += BB) ps[i] = xw[r0 + i];
            product(Vec{xw, false, (X)0});
            for (int i = tid; i < rows; i += BB) {
                const double bi = (double)b[r0 + i], d = bi - (double)qs[i];
                s[0] += d * d;
                s[1] += bi * bi;
            }
            put(0, s[0]);
            put(1, s[1]);
            return;
        }
        if (A.st->done) return;  // (the steps' kernels do not write it)
        const long long k = A.st->iters;
        if (A.phase == PHASE_PQ) {
            Vec v{nullptr, true, (X)0};
            if (k > 0) v = Vec{pb[(k + A.par) & 1], true, (X)(A.st->rho[k & 1] / A.st->rho[(k & 1) ^ 1])};
            else if (A.pcont != 0) v = Vec{pb[A.par & 1], true, (X)A.pcont};
            for (int t = tid; v.src && t < W; t += BB) {
                const int j = r0 - win + t;
                pw[t] = j >= 0 && j < A.n ? v.src[j] : (X)0;
            }
            __syncthreads();
            for (int i = tid; i < rows; i += BB) ps[i] = direction(v, precond(r[r0 + i], r0 + i), ps[i]);
            product(v);
            X *const pn = pb[(k + 1 + A.par) & 1];
            for (int i = tid; i < rows; i += BB) {
                pn[r0 + i] = ps[i];
                q[r0 + i] = qs[i];
                s[0] += (double)ps[i] * (double)qs[i];
            }
            put(2, s[0]);
        } else {  // PHASE_RR
            const X alpha = (X)(A.st->rho[(k & 1) ^ 1] / A.st->pq);
            const X *const p = pb[(k + A.par) & 1];
            for (int i = tid; i < rows; i += BB) {
                xw[r0 + i] = xw[r0 + i] + alpha * p[r0 + i];
                const X ri = r[r0 + i] - alpha * q[r0 + i];
                r[r0 + i] = ri;
                s[0] += JAC ? (double)ri * ((double)ri * dinv(r0 + i)) : (double)ri * (double)ri;
                s[1] += (double)ri * (double)ri;
            }
            put(0, s[0]);
            if (JAC) put(1, s[1]);
        }
        return;
    }

    double rho, nr0, relres;
    double rho_last = 0, pq_last = 0;  // rho before the last iteration
    long long k = 0;
    int done = 0;
    Vec v{nullptr, true, (X)0};  // the next direction
    if (A.resume) {
        k = A.st->iters;
        rho = A.st->rho[k & 1];
        rho_last = A.st->rho[(k & 1) ^ 1];
        nr0 = A.st->nr0;
        relres = A.st->relres;
        v = Vec{pb[(k + A.par) & 1], true, (X)(rho / rho_last)};
        for (int i = tid; i < rows; i += BB) {
            xs[i] = ((const X *)A.x_work)[r0 + i];
            rs[i] = r[r0 + i];
        }
    } else {
        double s[2] = {0, 0};
        if (A.x0_zero) {
            for (int i = tid; i < rows; i += BB) {
                xs[i] = 0;
                rs[i] = b[r0 + i];
            }
        } else {
            for (int i = tid; i < rows; i += BB) {
                ps[i] = xs[i] = ((const X *)A.x_in)[r0 + i];
                publish(pb[0], i, xs[i]);
            }
            double none[1] = {0};
            if (!meet(none)) return;
            product(Vec{pb[0], false, (X)0});
            for (int i = tid; i < rows; i += BB) rs[i] = b[r0 + i] - qs[i];
        }
        for (int i = tid; i < rows; i += BB) {
            const X ri = rs[i];
            publish(r, i, ri);
            s[0] += JAC ? (double)ri * ((double)ri * dinv(r0 + i)) : (double)ri * (double)ri;
            s[1] += (double)ri * (double)ri;
        }
        if (!meet(s)) return;
        rho = s[0];
        nr0 = sqrt(s[1]);
        relres = s[1] > 0 ? 1.0 : 0.0;
        done = s[1] == 0 ? 1 : ((!isfinite(s[1]) || !isfinite(s[0])) ? 3 : (A.maxit <= 0 ? 2 : 0));
        if (A.pcont != 0) v = Vec{pb[A.par & 1], true, (X)A.pcont};
    }
    if (v.src) {  // the direction before lies in memory (written by an earlier launch)
        for (int t = tid; t < W; t += BB) {
            const int j = r0 - win + t;
            pw[t] = j >= 0 && j < A.n ? v.src[j] : (X)0;
        }
        __syncthreads();
    }
    for (int step = 0; done == 0 && step < A.steps; step++) {
        for (int i = tid; i < rows; i += BB) ps[i] = direction(v, precond(rs[i], r0 + i), ps[i]);
        product(v);
        k++;
        rho_last = rho;
        double s[1] = {0};
        for (int i = tid; i < rows; i += BB) s[0] += (double)ps[i] * (double)qs[i];
        if (!meet(s)) return;
        const double pq = s[0];
        pq_last = pq;
        if (!(pq > 0) || !isfinite(pq)) {
            done = 3;
            break;
        }
        const X alpha = (X)(rho / pq);
        double t[JAC ? 2 : 1] = {};
        for (int i = tid; i < rows; i += BB) {
            xs[i] = xs[i] + alpha * ps[i];
            const X ri = rs[i] - alpha * qs[i];
            rs[i] = ri;
            publish(r, i, ri);
            if constexpr (JAC) {
                t[0] += (double)ri * ((double)ri * dinv(r0 + i));
                t[1] += (double)ri * (double)ri;
            } else {
                t[0] += (double)ri * (double)ri;
            }
        }
        if (!meet(t)) return;
        const double rho1 = t[0], nr = sqrt(t[JAC ? 1 : 0]);
        relres = nr0 > 0 ? nr / nr0 : 0.0;
        if (!isfinite(rho1) || !isfinite(nr)) done = 3;
        else if (nr <= A.tol * nr0) done = 1;
        else if (k >= A.maxit) done = 2;
        rho = rho1;
        v = Vec{pb[(k + A.par) & 1], true, (X)(rho1 / rho_last)};
    }
    double rel_true = 0;
    if (done && A.want_true) {
        // x goes out in r's place, which nobody reads any more
        for (int i = tid; i < rows; i += BB) {
            ps[i] = xs[i];
            publish(r, i, xs[i]);
        }
        double none[1] = {0};
        if (!meet(none)) return;
        product(Vec{r, false, (X)0});
        double s[2] = {0, 0};
        for (int i = tid; i < rows; i += BB) {
            const double bi = (double)b[r0 + i], d = bi - (double)qs[i];
            s[0] += d * d;
            s[1] += bi * bi;
        }
        if (!meet(s)) return;
        rel_true = s[1] > 0 ? sqrt(s[0]) / sqrt(s[1]) : sqrt(s[0]);
    }
    if (!meet.kept()) return;
    X *xo = (X *)(done ? A.x_out : A.x_work);
    for (int i = tid; i < rows; i += BB) {
        xo[r0 + i] = xs[i];
        if (!(done && A.want_true)) pb[(k + A.par) & 1][r0 + i] = ps[i];
        if (!done) pb[(k + 1 + A.par) & 1][r0 + i] = rs[i];  // a launch that is given up leaves r overwritten
    }
    if (blockIdx.x == 0 && tid == 0) {
        CgState v;
        v.rho[k & 1] = rho;
        v.rho[(k & 1) ^ 1] = rho_last;
        v.nr0 = nr0;
        v.pq = pq_last;
        v.relres = relres;
        v.tol = A.tol;
        v.iters = k;
        v.maxit = A.maxit;
        v.done = done;
        v.pad = 0;
        *A.st = v;
        A.host[0] = v;
        v.relres = rel_true;
        A.host[1] = v;
        __threadfence_system();
    }
}

// What a workgroup makes of the sums of a meeting, for a solve by steps (one
// workgroup; the sums are formed as in a meeting).
template <bool JAC>
__global__ void __launch_bounds__(BB) k_cgp_scalars(const CgpArgs A, int groups, int phase) {
    __shared__ double sums[2 * NW];
    WgSum<> total{sums};
    auto grid = [&](int k) { return total((int)threadIdx.x < groups ? A.part[k * PG + threadIdx.x] : 0.0); };
    CgState *const st = A.st;
    const bool first = threadIdx.x == 0;
    if (phase == PHASE_INIT) {
        const double rho = grid(0), rr = grid(1);
        if (!first) return;
        st->rho[0] = rho;
        st->rho[1] = 0;
        st->nr0 = sqrt(rr);
        st->pq = 0;
        st->relres = rr > 0 ? 1.0 : 0.0;
        st->tol = A.tol;
        st->iters = 0;
        st->maxit = A.maxit;
        st->done = rr == 0 ? 1 : ((!isfinite(rr) || !isfinite(rho)) ? 3 : (A.maxit <= 0 ? 2 : 0));
        st->pad = 0;
        return;
    }
    if (phase == PHASE_TRUE) {
        const double rr = grid(0), bb = grid(1);
        if (first) A.part[0] = bb > 0 ? sqrt(rr) / sqrt(bb) : sqrt(rr);
        return;
    }
    if (st->done) return;  // (thread 0 writes it after the sums' barriers)
    const long long k = st->iters;
    if (phase == PHASE_PQ) {
        const double pq = grid(2), rho = st->rho[k & 1];
        if (!first) return;
        st->iters = k + 1;
        st->pq = pq;
        if (!(pq > 0) || !isfinite(pq)) {
            st->done = 3;
            st->rho[(k + 1) & 1] = rho;
        }
    } else {  // PHASE_RR
        const double rho1 = grid(0), nr = sqrt(JAC ? grid(1) : rho1), nr0 = st->nr0;
        if (!first) return;
        st->relres = nr0 > 0 ? nr / nr0 : 0.0;
        if (!isfinite(rho1) || !isfinite(nr)) st->done = 3;
        else if (nr <= st->tol * nr0) st->done = 1;
        else if (k >= st->maxit) st->done = 2;
        st->rho[k & 1] = rho1;
    }
}

// ---------------------------------------------------------------- how far rows reach
// max |column - row| of a CSR (first and last entry of each row) or ELL part
__global__ void __launch_bounds__(256) k_reach_csr(i64 n, const i32 *rp, const i32 *col, int *out) {
    __shared__ int m;
    if (threadIdx.x == 0) m = 0;
    __syncthreads();
    int v = 0;
    for (i64 i = (i64)blockIdx.x * 256 + threadIdx.x; i < n; i += (i64)gridDim.x * 256) {
        const i32 a = rp[i], z = rp[i + 1];
        if (a < z) v = max(v, max((int)i - col[a], col[z - 1] - (int)i));
    }
    atomicMax(&m, v);
    __syncthreads();
    if (threadIdx.x == 0 && m > 0) atomicMax(out, m);
}
__global__ void __launch_bounds__(256) k_reach_ell(i64 n, i64 K, i64 pitch, const i32 *ecol, int *out) {
    __shared__ int m;
    if (threadIdx.x == 0) m = 0;
    __syncthreads();
    int v = 0;
    for (i64 i = (i64)blockIdx.x * 256 + threadIdx.x; i < n; i += (i64)gridDim.x * 256)
        for (i64 k = 0; k < K; k++) {
            const i32 c = ecol[k * pitch + i];
            if (c >= 0) v = max(v, abs(c - (int)i));
        }
    atomicMax(&m, v);
    __syncthreads();
    if (threadIdx.x == 0 && m > 0) atomicMax(out, m);
}

// d: an int of scratch
static i64 reach_of(dsm_matrix m, int *d, hipStream_t s) {
    Payload &P = m->P;
    if (P.reach >= 0) return P.reach;
    int h = 0;
    DSM_HIP(hipMemsetAsync(d, 0, sizeof(int), s));
    const unsigned g = std::min<unsigned>(512, grid_for(m->nrows, 256));
    if (P.fmt == DSM_CSR)
        hipLaunchKernelGGL(k_reach_csr, dim3(g), dim3(256), 0, s, m->nrows, P.rp, P.col, d);
    else
        hipLaunchKernelGGL(k_reach_ell, dim3(g), dim3(256), 0, s, m->nrows, P.K, P.pitch, P.ecol, d);
    DSM_HIP(hipGetLastError());
    DSM_HIP(hipMemcpyAsync(&h, d, sizeof(int), hipMemcpyDeviceToHost, s));
    DSM_HIP(hipStreamSynchronize(s));
    return P.reach = h;
}

// ---------------------------------------------------------------- host side
// The CUs of one device that launches of this kernel hold, given out in the
// order of asking.
class CuShare {
    std::mutex mu;
    std::condition_variable cv;
    int used = 0;
    u64 asked = 0, served = 0;

public:
    void take(int cus, int all) {
        std::unique_lock<std::mutex> lk(mu);
        const u64 mine = asked++;
        cv.wait(lk, [&] { return served == mine && used + cus <= all; });
        used += cus;
        served++;
        cv.notify_all();
    }
    void give(int cus) {
        std::lock_guard<std::mutex> lk(mu);
        used -= cus;
        cv.notify_all();
    }
};
constexpr int MAX_DEVICES = 64;
static CuShare cu_share[MAX_DEVICES];

constexpr size_t LDS_MAX = (160 << 10) - 1024 - sizeof(i32) * MAX_DIAGS;

template <class X>
static size_t lds_need(int fmt, i64 rpw, i64 win) {
    size_t w = 4 * (size_t)rpw + 2 * (size_t)win + 2;
    if (fmt == DSM_CSR) w += NW * WCH;
    return w * sizeof(X) + (fmt == DSM_CSR ? sizeof(i32) * (size_t)(rpw + 2) : 0);
}

template <class V, class X, bool JAC, bool STEP>
static const void *kernel_of(int fmt) {
    if (fmt == DSM_CSR) return (const void *)&k_cg_persist<V, X, DSM_CSR, JAC, STEP>;
    if (fmt == DSM_ELL) return (const void *)&k_cg_persist<V, X, DSM_ELL, JAC, STEP>;
    return (const void *)&k_cg_persist<V, X, DSM_DIA, JAC, STEP>;
}
template <class X, bool JAC, bool STEP>
static const void *kernel_of(int fmt, int vdt) {
    if constexpr (std::is_same<X, double>::value) {
        if (vdt == DSM_F64) return kernel_of<double, X, JAC, STEP>(fmt);
    }
    return vdt == DSM_F32 ? kernel_of<float, X, JAC, STEP>(fmt) : kernel_of<bf16, X, JAC, STEP>(fmt);
}
template <class X, bool STEP>
static const void *kernel_of(int fmt, int vdt, bool jacobi) {
    if constexpr (std::is_same<X, double>::value) {
        if (jacobi) return kernel_of<X, true, STEP>(fmt, vdt);
    }
    return kernel_of<X, false, STEP>(fmt, vdt);
}

// The solve, or what is left of it after the launches that were kept (A.resume;
// `last`: the state they ended with), by steps; waits.
template <class X>
static void cgp_steps(CgpArgs A, const CgState &last, const void *kernel, int groups, size_t lds, CgState *out,
                      double *rel_true, hipStream_t s) {
    constexpr int CHUNK = 16;  // iterations between looks at the state
    const bool jac = A.dinv != nullptr;
    auto step = [&](int phase) {
        A.phase = phase;
        void *args[] = {&A};
        DSM_HIP(hipLaunchKernel(kernel, dim3(groups), dim3(BB), args, lds, s));
        if (jac) hipLaunchKernelGGL(k_cgp_scalars<true>, dim3(1), dim3(BB), 0, s, A, groups, phase);
        else hipLaunchKernelGGL(k_cgp_scalars<false>, dim3(1), dim3(BB), 0, s, A, groups, phase);
        DSM_HIP(hipGetLastError());
    };
    const size_t bytes = sizeof(X) * (size_t)A.n;
    if (A.resume)
        DSM_HIP(hipMemcpyAsync(A.r, A.p[(last.iters + 1 + A.par) & 1], bytes, hipMemcpyDeviceToDevice, s));
    else
        step(PHASE_INIT);
    do {
        for (int i = 0; i < CHUNK; i++) {
            step(PHASE_PQ);
            step(PHASE_RR);
        }
        DSM_HIP(hipMemcpyAsync(out, A.st, sizeof(CgState), hipMemcpyDeviceToHost, s));
        DSM_HIP(hipStreamSynchronize(s));
    } while (!out->done);
    if (rel_true) {
        step(PHASE_TRUE);
        DSM_HIP(hipMemcpyAsync(rel_true, A.part, sizeof(double), hipMemcpyDeviceToHost, s));
    }
    DSM_HIP(hipMemcpyAsync(A.x_out, A.x_work, bytes, hipMemcpyDeviceToDevice, s));
    DSM_HIP(hipStreamSynchronize(s));
}

template <class X>
bool cg_persist(dsm_matrix m, const CgpSolve<X> &S, hipStream_t s, Workspace &cgws, CgState *out, double *rel_true) {
    const char *env = getenv("DSM_CG_RESIDENT");
    if (env && env[0] == '0') return false;
    const Payload &P = m->P;
    const i64 n = m->nrows;
    int fmt = P.fmt;
    if (fmt == DSM_HDC && P.csr_nnz == 0) fmt = DSM_DIA;
    if (fmt == DSM_HYB && P.coo_nnz == 0) fmt = DSM_ELL;
    if ((fmt != DSM_CSR && fmt != DSM_DIA && fmt != DSM_ELL) || n < 1 || m->nrows != m->ncols) return false;
    if (fmt == DSM_DIA && (P.ndiag == 0 || P.ndiag > MAX_DIAGS || P.reach < 0)) return false;
    if (m->ctx->device >= MAX_DEVICES) return false;
    int ncu = 0;
    DSM_HIP(hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, m->ctx->device));
    const i64 most = std::min(ncu, PG);
    // rows per workgroup: PROWS or more, so that small systems meet in small
    // groups
    constexpr i64 PROWS = 256;
    const i64 rpw = (std::max<i64>(PROWS, (n + most - 1) / most) + 63) / 64 * 64;
    const int G = (int)((n + rpw - 1) / rpw);
    if (lds_need<X>(fmt, rpw, 0) > LDS_MAX) return false;
    const i64 win = std::min<i64>(fmt == DSM_DIA ? P.reach : reach_of(m, (int *)S.part, s), n);
    const size_t lds = lds_need<X>(fmt, rpw, win);
    if (lds > LDS_MAX) return false;
    if (!cgws.host)
        DSM_HIP(hipHostMalloc(&cgws.host, 2 * sizeof(CgState), hipHostMallocCoherent | hipHostMallocMapped));
    CgState *host = (CgState *)cgws.host, *host_dev = nullptr;
    DSM_HIP(hipHostGetDevicePointer((void **)&host_dev, cgws.host, 0));

    CgpArgs A{};
    A.n = (int)n;
    A.rpw = (int)rpw;
    A.win = (int)win;
    A.rp = P.rp;
    A.col = P.col;
    A.val = fmt == DSM_CSR ? P.val : (fmt == DSM_DIA ? P.dval : P.evl);
    const double mean = (double)P.csr_nnz / (double)n;
    A.lanes = 1;
    while (A.lanes < 32 && 16 * A.lanes <= mean) A.lanes <<= 1;
    A.offs = P.offs;
    A.nd = (int)(fmt == DSM_DIA ? P.ndiag : P.K);
    A.pitch = P.pitch;
    A.ecol = P.ecol;
    A.b = S.b;
    A.x_in = S.x_in;
    A.x_out = S.x_out;
    A.x_work = S.x_work;
    A.p[0] = S.p[0];
    A.p[1] = S.p[1];
    A.par = S.par;
    A.r = S.r;
    A.dinv = S.dinv;
    // 64 G + 4 bytes of the 8 n, rounded up to 256: n > 256 (G - 1)
    static_assert(sizeof(u64) * SETS * SUMS < 8 * PROWS, "the words of the meetings lie in q");
    A.slots = (u64 *)S.q;
    A.outcome = (u32 *)(A.slots + SETS * SUMS * G);
    A.st = S.st;
    A.host = host_dev;
    A.tol = S.tol;
    A.pcont = S.pcont;
    A.maxit = S.maxit;
    A.x0_zero = S.x0_zero;
    A.want_true = rel_true != nullptr;
    A.q = S.q;
    A.part = S.part;
    // iterations per launch: about 20 ms, so that other streams get their turn
    const double us = 8.0 + spmv_bytes(m, P, std::is_same<X, double>::value ? DSM_F64 : DSM_F32) / 5e6;
    A.steps = S.every > 0 ? S.every : (int)std::max(16.0, 20000.0 / us);
    if (P.vdt == DSM_F64 && !std::is_same<X, double>::value) return false;
    const void *loop = kernel_of<X, false>(fmt, P.vdt, S.dinv != nullptr);
    const char *up = getenv("DSM_CG_GIVE_UP");  // the launch of a solve that is given up, for tests
    const int give_up = up ? atoi(up) : -1;
    CgState last{};
    bool by_steps = cgws.alone_wait > 0;  // a solve before this one did not get the device
    if (by_steps) cgws.alone_wait--;
    // (what the stream still has to do is done before CUs are asked for)
    else if (!S.waited) DSM_HIP(hipStreamSynchronize(s));
    for (int launch = 0; !by_steps; launch++) {
        struct Cus {
            CuShare &share;
            int n;
            Cus(CuShare &c, int n_, int all) : share(c), n(n_) { share.take(n, all); }
            ~Cus() { share.give(n); }
        } cus(cu_share[m->ctx->device], G, ncu);
        host[0].done = -1;
        hipLaunchKernelGGL(k_slots_clear, dim3(grid_for(SETS * SUMS * G, 256)), dim3(256), 0, s, A.slots,
                           SETS * SUMS * G, A.outcome,
                           (u32)(launch == give_up ? OUTCOME_GIVEN_UP : OUTCOME_OPEN));
        void *args[] = {&A};
        DSM_HIP(hipLaunchKernel(loop, dim3(G), dim3(BB), args, lds, s));
        DSM_HIP(hipStreamSynchronize(s));
        if (host[0].done < 0) {  // given up
            cgws.alone_wait = ALONE;
            by_steps = true;
            break;
        }
        last = host[0];
        if (last.done) break;
        A.resume = 1;
    }
    if (by_steps) {
        cgp_steps<X>(A, last, kernel_of<X, true>(fmt, P.vdt, S.dinv != nullptr), G, lds, out, rel_true, s);
        return true;
    }
    *out = last;
    if (rel_true) *rel_true = host[1].relres;
    return true;
}

template bool cg_persist<double>(dsm_matrix, const CgpSolve<double> &, hipStream_t, Workspace &, CgState *, double *);
template bool cg_persist<float>(dsm_matrix, const CgpSolve<float> &, hipStream_t, Workspace &, CgState *, double *);

}  // namespace dsm

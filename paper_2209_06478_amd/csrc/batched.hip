// Batched CG: many independent small systems in one persistent launch.
//
// A fixed grid of workgroups pulls request indices from an integer counter;
// each workgroup then runs one request's whole CG loop by itself, with
// workgroup barriers as the only synchronisation (no inter-workgroup waits,
// so every workgroup finishes once the counter passes the request count).
// Every reduction inside a request uses the same thread-to-element map and
// the same fixed combination order, so a request's iterates and iteration
// count do not depend on which workgroup runs it or on what else is in the
// batch.
//
// Supported in-workgroup formats: CSR (a power-of-two lane group per row,
// the "tile" the batched tuner picks), DIA and ELL, with FP64 values.
// Anything else, or systems above the size threshold, is solved by the
// device-wide solver on a side stream while the batch kernel runs.
#include <algorithm>
#include <thread>
#include <vector>

#include "core.hpp"
#include "wg_kernels.hpp"

namespace dsm {

constexpr i64 BATCH_SMALL_ROWS = 40000;  // largest system solved by one workgroup

struct BReq {
    int fmt;
    int lanes;
    i64 n;
    const i32 *rp;
    const i32 *col;
    const double *val;
    const i32 *offs;
    i64 ndiag;
    i64 pitch;
    const double *dval;
    const i32 *ecol;
    const double *evl;
    i64 K;
    const double *b;
    double *x;
    double *r;
    double *p;
    double *q;
    double tol;
    i64 maxit;
};

struct BRes {
    i64 iters;
    double relres;
    double relres_true;
    int status;
    int pad;
};

// ---- one workgroup's q = A p
// What bounds it is the rate at which one CU is fed, about 60 GB/s (a
// 4096-row system of 60 ELL slots a row: 2.95 MB in 45 us per iteration, the
// same with twice the loads in flight), and close behind it VALU
// instructions per stored slot (4 cycles each per wave and SIMD).  So loads
// are issued in batches whose addresses are a scalar base plus one offset
// per lane, bounds tests sit on whole batches, and padding columns (-1) read
// the zero word kept just below p[0] in LDS.  Measured per iteration, before (512
// threads; a chain of dependent round trips per 512 / lanes rows, p and all
// else through the L2) and now: 4096 rows, CSR SPD band of 39 entries a row
// 336 -> 47-57 us, HPCG 16^3 CSR 337 -> 32-39 us, ELL 42 -> 26 us, DIA 50 ->
// 28 us; HPCG 24^3 ELL 156 -> 95 us; HPCG 8^3 ELL 7.4 -> 5.6 us.  128 systems
// of up to 4096 rows in one call: 17.6 -> 2.0 ms.
// q = A p for one descriptor, the zero word at p[zero]
template <class PP, class QQ, class RPP>
__device__ __forceinline__ void csr_spmv(const BReq &R, const WaveRows &rows, PP p, int zero, QQ q, RPP rp,
                                         double *prod) {
    wg_spmv_csr(rows, R.lanes, R.col, R.val, p, zero, q, rp, prod);
}
template <int U, int B, class PP, class QQ>
__device__ __forceinline__ void dia_spmv(const BReq &R, PP p, int zero, QQ q) {
    wg_spmv_dia<double, U, B>((int)R.n, 0, (int)R.n, (int)R.ndiag, R.pitch, R.offs, R.dval, p, zero, q);
}
template <int U, int B, bool ZERO_BELOW, class PP, class QQ>
__device__ __forceinline__ void ell_spmv(const BReq &R, PP p, int zero, QQ q) {
    wg_spmv_ell<double, U, B, ZERO_BELOW>((int)R.n, (int)R.K, (int)R.pitch, R.ecol, R.evl, p, zero, q);
}

// ---- where a system's vectors live
// Up to 19000 rows (CSR: 8000): p (below it the zero word) in LDS, for CSR
// the row pointers in LDS, and q in LDS where it still fits; an iteration
// then reads nothing from memory but the matrix, x and r (x and r stay in
// memory: held in registers, they cost the products 70-120 spilled ones).
// Larger systems keep all vectors in memory, and share a zero word in the
// arena's fixed part.
constexpr i64 WL_ROWS = 19000;       // 8 bytes a row
constexpr i64 WL_Q_ROWS = 9500;      // q in LDS too: 16 bytes a row
constexpr i64 WL_CSR_ROWS = 8000;    // 12 bytes a row beside the 64 KB of products
constexpr i64 WL_CSR_Q_ROWS = 4800;  // q in LDS too: 20 bytes a row

// Threads of a launch: 1024, or as many as the largest of its systems has rows,
// rounded up to a power of two; the barriers of idle waves, and their place on
// the CU, cost small systems more than their work.  One call, CSR, DIA and ELL:
// 2000 systems of 64 rows 519, 341 and 250 us with 1024 threads, 106, 88 and 81
// with 64; 1000 of 512 rows 767, 468 and 417, now 451, 312 and 334; one of 64
// rows 59.7, 42.3 and 30.8, now 38.2, 34.2 and 22.5.  A system's bits do not
// depend on it: the waves that take part in a CSR product go by its rows.
static __host__ __device__ int csr_waves(i64 n) { return n <= 64 ? 1 : n <= 128 ? 2 : n <= 256 ? 4 : n <= 512 ? 8 : NW; }
static __host__ __device__ size_t prod_bytes(int threads) { return sizeof(double) * (threads / WAVE) * WCH; }

static __host__ __device__ size_t lds_vec(i64 n) { return (size_t)(n + (n & 1)) * sizeof(double); }
static __host__ __device__ bool on_cu(int fmt, i64 n) { return n <= (fmt == DSM_CSR ? WL_CSR_ROWS : WL_ROWS); }
static __host__ __device__ bool lds_q(int fmt, i64 n) { return n <= (fmt == DSM_CSR ? WL_CSR_Q_ROWS : WL_Q_ROWS); }
static __host__ __device__ size_t lds_bytes(int fmt, i64 n, int threads) {
    size_t b = fmt == DSM_CSR ? prod_bytes(threads) : 0;
    if (!on_cu(fmt, n)) return b;
    b += 2 * sizeof(double) + lds_vec(n) + (lds_q(fmt, n) ? lds_vec(n) : 0);
    return b + (fmt == DSM_CSR ? (size_t)(n + 2) * sizeof(i32) : 0);
}

// One system, start to end, by T threads (T < BB: of at most T rows).  ONCU: p
// on the CU as above.  A solve is a
// sequence of products q = A p: the first with x0 in p's place, the last
// with the final x (for the true residual).
// zero_word: the zero word of the other systems.
template <int T, bool ONCU>
__device__ __forceinline__ void solve_one(const BReq *req, BRes *out, double *lds, char *dyn,
                                          const double *zero_word) {
    const BReq &R = *req;
    const int tid = threadIdx.x;
    const int n = (int)R.n;
    double *prod = (double *)dyn;
    if (R.fmt == DSM_CSR) dyn += prod_bytes(T);
    double *ps = (double *)dyn + 2, *qs = ps + (n + (n & 1));
    i32 *rps = (i32 *)(lds_q(R.fmt, n) ? qs + (n + (n & 1)) : qs);
    const bool ql = ONCU && lds_q(R.fmt, n);
    WgSum<T> total{lds};
    // element access of the two places p and q can live in
    auto getp = [&](int i) { return ONCU ? ps[i] : R.p[i]; };
    auto setp = [&](int i, double t) {
        if (ONCU) ps[i] = t;
        else R.p[i] = t;
    };
    auto getq = [&](int i) {
        if (ONCU && ql) return qs[i];
        return R.q[i];
    };
    if (ONCU && tid == 0) ps[-1] = 0.0;
    if (ONCU && R.fmt == DSM_CSR)
        for (int i = tid; i <= n; i += T) rps[i] = R.rp[i];
    for (int i = tid; i < n; i += BB) setp(i, R.x[i]);
    WaveRows wrows{};
    if (R.fmt == DSM_CSR) {
        if (ONCU) {
            __syncthreads();  // rps
            wrows = wave_rows(n, rps, csr_waves(n));
        } else {
            wrows = wave_rows(n, R.rp);
        }
    }
    // x and r of the thread's first row stay in registers (a system of up to
    // BB rows then waits for no vector; more rows would spill)
    double x0 = tid < n ? R.x[tid] : 0.0, r0 = 0;
    double rho = 0, nr0 = 0, nb = 0, relres = 0;
    int status = 1;  // running
    i64 k = -1;      // products of the loop so far; -1: the product with x0
    for (;;) {
        __syncthreads();
        // The product reads its descriptor anew through a pointer the
        // compiler cannot trace: it had moved every address of the three
        // products out of this loop, at 580 spilled registers per lane.
        const BReq *again = req;
        asm volatile("" : "+s"(again));
        const BReq &R = *again;
        const int zero = ONCU ? -1 : (int)(zero_word - R.p);
        if (R.fmt == DSM_CSR) {
            if (T < BB || (ONCU && ql)) csr_spmv(R, wrows, ps, zero, qs, rps, prod);
            else if (ONCU) csr_spmv(R, wrows, ps, zero, R.q, rps, prod);
            else csr_spmv(R, wrows, R.p, zero, R.q, R.rp, prod);
        } else if (R.fmt == DSM_DIA) {
            if (T < BB || (ONCU && n <= BB)) dia_spmv<1, 16>(R, ps, zero, qs);
            else if (ONCU && ql) dia_spmv<2, 8>(R, ps, zero, qs);
            else if (ONCU) dia_spmv<2, 8>(R, ps, zero, R.q);
            else dia_spmv<2, 8>(R, R.p, zero, R.q);
        } else {
            if (T < BB || (ONCU && n <= BB)) ell_spmv<1, 16, true>(R, ps, zero, qs);
            else if (ONCU && ql) ell_spmv<2, 8, true>(R, ps, zero, qs);
            else if (ONCU) ell_spmv<2, 8, true>(R, ps, zero, R.q);
            else ell_spmv<2, 8, false>(R, R.p, zero, R.q);
        }
        if (R.fmt == DSM_CSR) __syncthreads();  // DIA and ELL: a thread reads its own q only
        double a = 0, c = 0;
        if (k < 0) {
            __syncthreads();  // p is about to be overwritten
            for (int i = tid; i < n; i += BB) {
                const double bi = R.b[i], ri = bi - getq(i);
                if (i == tid) r0 = ri;
                else R.r[i] = ri;
                setp(i, ri);
                a += ri * ri;
                c += bi * bi;
            }
            rho = total(a);
            nb = sqrt(total(c));
            nr0 = sqrt(rho);
            status = rho == 0 ? DSM_OK : (!isfinite(rho) ? DSM_E_BREAKDOWN : 1);
            relres = rho > 0 ? 1.0 : 0.0;
            k = 0;
        } else if (status != 1) {
            for (int i = tid; i < n; i += BB) {
                const double t = R.b[i] - getq(i);
                a += t * t;
            }
            const double nrt = sqrt(total(a));
            if (tid == 0) {
                out->iters = k;
                out->relres = relres;
                out->relres_true = nb > 0 ? nrt / nb : nrt;
                out->status = status;
            }
            __syncthreads();
            return;
        } else {
            k++;
            for (int i = tid; i < n; i += BB) a += getp(i) * getq(i);
            const double pq = total(a);
            if (!(pq > 0) || !isfinite(pq)) {
                status = DSM_E_BREAKDOWN;
            } else {
                const double alpha = rho / pq;
                a = 0;
                if (tid < n) {
                    x0 = x0 + alpha * getp(tid);
                    r0 = r0 - alpha * getq(tid);
                    a = r0 * r0;
                }
#pragma unroll 4
                for (int i = tid + BB; i < n; i += BB) {
                    const double xi = R.x[i], ri = R.r[i] - alpha * getq(i);
                    R.x[i] = xi + alpha * getp(i);
                    R.r[i] = ri;
                    a += ri * ri;
                }
                const double rho1 = total(a);
                relres = nr0 > 0 ? sqrt(rho1) / nr0 : 0.0;
                if (!isfinite(rho1)) {
                    status = DSM_E_BREAKDOWN;
                } else if (sqrt(rho1) <= R.tol * nr0) {
                    status = DSM_OK;
                } else {
                    const double beta = rho1 / rho;
                    if (tid < n) setp(tid, r0 + beta * getp(tid));
#pragma unroll 4
                    for (int i = tid + BB; i < n; i += BB) setp(i, R.r[i] + beta * getp(i));
                    rho = rho1;
                }
            }
        }
        if (status == 1 && k >= R.maxit) status = DSM_E_NOT_CONVERGED;
        if (status != 1) {
            if (tid < n) R.x[tid] = x0;
            for (int i = tid; i < n; i += BB) setp(i, R.x[i]);
        }
    }
}

template <int T>
__global__ void __launch_bounds__(T, BB / WAVE / 4) k_cg_batched(const BReq *__restrict__ reqs, BRes *__restrict__ res, int count,
                                                   int *next, const double *zero_word) {
    __shared__ double lds[2 * T / WAVE];
    __shared__ int sidx;
    extern __shared__ char dyn[];  // lds_bytes of the launch's largest system
    for (;;) {
        if (threadIdx.x == 0) sidx = atomicAdd(next, 1);
        __syncthreads();
        // uniform, so that the descriptor is read into scalar registers
        const int idx = __builtin_amdgcn_readfirstlane(sidx);
        __syncthreads();
        if (idx >= count) return;
        const BReq *req = reqs + idx;
        if (T < BB || on_cu(req->fmt, req->n)) solve_one<T, true>(req, &res[idx], lds, dyn, zero_word);
        else solve_one<T, false>(req, &res[idx], lds, dyn, zero_word);
    }
}

// ---------------------------------------------------------------- host side
bool batch_eligible(const dsm_matrix_s *m, i64 small_rows) {
    const Payload &P = m->P;
    return m->nrows == m->ncols && m->nrows <= small_rows && P.vdt == DSM_F64 &&
           (P.fmt == DSM_CSR || P.fmt == DSM_DIA || P.fmt == DSM_ELL);
}

// Lanes that sum a CSR row: 8 to 16 products each, so that one pass of a
// wave covers the rows of a WCH-entry batch (the loads do not depend on it).
static int default_lanes(const dsm_matrix_s *m, const Payload &P) {
    if (P.fmt != DSM_CSR) return 1;
    const double mean = m->nrows ? (double)P.csr_nnz / (double)m->nrows : 1.0;
    int L = 1;
    while (L < 32 && 16 * L <= mean) L <<= 1;
    return L;
}

static size_t vec_bytes(i64 n) { return ((size_t)std::max<i64>(n, 1) * 8 + 255) & ~(size_t)255; }

// Arena bytes of one batch: a fixed part (the work counter, the zero word and
// the 256-byte rounding of the descriptor and result arrays) plus one share per
// request.
size_t batch_request_bytes(i64 n) { return 3 * vec_bytes(n) + sizeof(BReq) + sizeof(BRes); }
size_t batch_arena_fixed() { return 1536; }

static BReq make_req(const dsm_matrix_s *m, const Payload &P, int lanes) {
    BReq R{};
    R.fmt = P.fmt;
    R.lanes = lanes;
    R.n = m->nrows;
    R.rp = P.rp;
    R.col = P.col;
    R.val = (const double *)P.val;
    R.offs = P.offs;
    R.ndiag = P.ndiag;
    R.pitch = P.pitch;
    R.dval = (const double *)P.dval;
    R.ecol = P.ecol;
    R.evl = (const double *)P.evl;
    R.K = P.K;
    return R;
}

// Lays out descriptors, results, counter and per-request vectors in `arena`,
// launches the persistent kernel on s and waits.
static void launch_reqs(dsm_ctx ctx, std::vector<BReq> &hreq, std::vector<BRes> &hres, Workspace &arena,
                        hipStream_t s) {
    const int count = (int)hreq.size();
    if (count == 0) return;
    size_t bytes = batch_arena_fixed();
    for (auto &R : hreq) bytes += batch_request_bytes(R.n);
    char *base = (char *)ws_get(ctx, arena, bytes, s);
    auto take = [&](size_t sz) {
        char *p = base;
        base += (sz + 255) & ~(size_t)255;
        return (void *)p;
    };
    int *next = (int *)take(2 * sizeof(double));
    double *zero_word = (double *)next + 1;
    BReq *dreq = (BReq *)take(sizeof(BReq) * count);
    BRes *dres = (BRes *)take(sizeof(BRes) * count);
    for (auto &R : hreq) {
        R.r = (double *)take(vec_bytes(R.n));
        R.p = (double *)take(vec_bytes(R.n));
        R.q = (double *)take(vec_bytes(R.n));
    }
    hres.resize(count);
    DSM_HIP(hipMemcpyAsync(dreq, hreq.data(), sizeof(BReq) * count, hipMemcpyHostToDevice, s));
    DSM_HIP(hipMemsetAsync(next, 0, 2 * sizeof(double), s));
    int ncu = 256;
    DSM_HIP(hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, ctx->device));
    i64 most = 0;
    for (auto &R : hreq) most = std::max(most, R.n);
    const int threads = most <= 64 ? 64 : most <= 128 ? 128 : most <= 256 ? 256 : most <= 512 ? 512 : BB;
    const unsigned grid = (unsigned)std::min(count, ncu * 4 * (BB / threads));
    size_t dyn = 0;
    for (auto &R : hreq) dyn = std::max(dyn, lds_bytes(R.fmt, R.n, threads));
    auto kernel = threads == 64 ? k_cg_batched<64> : threads == 128 ? k_cg_batched<128> : threads == 256 ? k_cg_batched<256> : threads == 512 ? k_cg_batched<512> : k_cg_batched<BB>;
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(threads), dyn, s, dreq, dres, count, next, zero_word);
    DSM_HIP(hipGetLastError());
    DSM_HIP(hipMemcpyAsync(hres.data(), dres, sizeof(BRes) * count, hipMemcpyDeviceToHost, s));
    DSM_HIP(hipStreamSynchronize(s));
}

static void to_result(const BRes &r, dsm_cg_result *out) {
    dsm_cg_result R{};
    R.iters = r.iters;
    R.outer_iters = 0;
    R.relres = r.relres;
    R.relres_true = r.relres_true;
    R.status = r.status;
    *out = R;
}

void run_batch(dsm_ctx ctx, const BatchJob &job, dsm_cg_result *results, Workspace &arena, hipStream_t s) {
    const size_t count = job.mats.size();
    // most stored slots first (what an iteration reads), so the tail of the
    // batch is short systems
    std::vector<size_t> order(count);
    for (size_t k = 0; k < count; k++) order[k] = k;
    auto slots = [&](size_t k) {
        const Payload &P = job.mats[k]->P;
        return P.fmt == DSM_CSR ? P.csr_nnz : (P.fmt == DSM_DIA ? P.ndiag : P.K) * P.pitch;
    };
    std::stable_sort(order.begin(), order.end(), [&](size_t a, size_t c) { return slots(a) > slots(c); });
    std::vector<BReq> hreq;
    for (size_t k : order) {
        dsm_matrix m = job.mats[k];
        BReq R = make_req(m, m->P, m->P.fmt == DSM_CSR && m->batch_lanes > 0 ? m->batch_lanes
                                                                             : default_lanes(m, m->P));
        R.b = job.b[k];
        R.x = job.x[k];
        R.tol = job.opts[k].tol;
        R.maxit = job.opts[k].maxit > 0 ? job.opts[k].maxit : std::min<i64>(10 * std::max<i64>(m->nrows, 1), 20000);
        hreq.push_back(R);
    }
    std::vector<BRes> hres;
    launch_reqs(ctx, hreq, hres, arena, s);
    for (size_t i = 0; i < count; i++) to_result(hres[i], &results[order[i]]);
}

__global__ void k_ones(i64 n, double *v) {
    i64 i = (i64)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) v[i] = 1.0;
}

double time_batched_solve(dsm_matrix m, const Payload &P, int lanes, int iters, hipStream_t s) {
    dsm_ctx ctx = m->ctx;
    const i64 n = m->nrows;
    void *v = dev_alloc(ctx, 2 * vec_bytes(n));
    double *b = (double *)v, *x = (double *)((char *)v + vec_bytes(n));
    Workspace arena;
    double us = 0;
    try {
        hipLaunchKernelGGL(k_ones, dim3(grid_for(n, 256)), dim3(256), 0, s, n, b);
        std::vector<BReq> hreq(1, make_req(m, P, lanes));
        hreq[0].b = b;
        hreq[0].x = x;
        hreq[0].tol = 0.0;  // run exactly `iters` iterations
        hreq[0].maxit = iters;
        std::vector<BRes> hres;
        hipEvent_t e0, e1;
        DSM_HIP(hipEventCreate(&e0));
        DSM_HIP(hipEventCreate(&e1));
        for (int rep = 0; rep < 3; rep++) {
            DSM_HIP(hipMemsetAsync(x, 0, 8 * (size_t)n, s));
            std::vector<BReq> r = hreq;
            DSM_HIP(hipEventRecord(e0, s));
            launch_reqs(ctx, r, hres, arena, s);
            DSM_HIP(hipEventRecord(e1, s));
            DSM_HIP(hipEventSynchronize(e1));
            float ms = 0;
            DSM_HIP(hipEventElapsedTime(&ms, e0, e1));
            us = rep == 0 ? ms * 1e3 : std::min(us, (double)ms * 1e3);
        }
        (void)hipEventDestroy(e0);
        (void)hipEventDestroy(e1);
    } catch (...) {
        ws_release(ctx, arena);
        dev_free(ctx, v, 2 * vec_bytes(n));
        throw;
    }
    ws_release(ctx, arena);
    dev_free(ctx, v, 2 * vec_bytes(n));
    return us;
}

}  // namespace dsm

using namespace dsm;

DSM_API dsm_status dsm_cg_solve_batched(int32_t count, const dsm_matrix *mats, const double *const *b,
                                        double *const *x, const dsm_cg_opts *opts, dsm_cg_result *results,
                                        void *stream) {
    return guard([&] {
        DSM_CHECK(count >= 0, DSM_E_INVALID, "negative count");
        if (count == 0) return;
        DSM_CHECK(mats && b && x && opts && results, DSM_E_INVALID, "null argument");
        dsm_ctx ctx = nullptr;
        for (int k = 0; k < count; k++) {
            DSM_CHECK(mats[k] && mats[k]->ctx, DSM_E_INVALID, "null matrix handle");
            DSM_CHECK(mats[k]->nrows == mats[k]->ncols, DSM_E_UNSUPPORTED, "CG needs square matrices");
            DSM_CHECK(opts[k].mode == DSM_CG_F64, DSM_E_UNSUPPORTED, "batched solves are FP64 only");
            DSM_CHECK(opts[k].tol >= 0, DSM_E_INVALID, "negative tolerance");
            DSM_CHECK((b[k] && x[k]) || mats[k]->nrows == 0, DSM_E_INVALID, "null vector");
            if (!ctx) ctx = mats[k]->ctx;
            DSM_CHECK(mats[k]->ctx == ctx, DSM_E_INVALID, "all matrices must share one context");
        }
        DSM_HIP(hipSetDevice(ctx->device));
        hipStream_t s = (hipStream_t)stream;
        BatchJob job;
        std::vector<int> small, large;
        for (int k = 0; k < count; k++) {
            if (batch_eligible(mats[k], BATCH_SMALL_ROWS)) {
                small.push_back(k);
                job.mats.push_back(mats[k]);
                job.b.push_back(b[k]);
                job.x.push_back(x[k]);
                job.opts.push_back(opts[k]);
            } else {
                large.push_back(k);
            }
        }
        // large systems on a side stream, overlapping the batch
        hipStream_t side = nullptr;
        Workspace arena, cgws, spws;
        std::vector<dsm_cg_result> sres(small.size());
        auto cleanup = [&] {
            if (side) {
                (void)hipStreamSynchronize(side);
                (void)hipStreamDestroy(side);
            }
            (void)hipStreamSynchronize(s);
            ws_release(ctx, arena);
            ws_release(ctx, cgws);
            ws_release(ctx, spws);
        };
        try {
            if (!large.empty()) DSM_HIP(hipStreamCreateWithFlags(&side, hipStreamNonBlocking));
            if (!small.empty()) {
                // enqueue the batch first, then drive the large solves while it runs
                std::exception_ptr err;
                std::thread th([&] {
                    try {
                        DSM_HIP(hipSetDevice(ctx->device));
                        run_batch(ctx, job, sres.data(), arena, s);
                    } catch (...) {
                        err = std::current_exception();
                    }
                });
                try {
                    for (int k : large) cg_solve_ws(mats[k], b[k], x[k], opts[k], &results[k], side, cgws, spws, false);
                } catch (...) {
                    th.join();
                    throw;
                }
                th.join();
                if (err) std::rethrow_exception(err);
            } else {
                for (int k : large) cg_solve_ws(mats[k], b[k], x[k], opts[k], &results[k], side, cgws, spws, false);
            }
        } catch (...) {
            cleanup();
            throw;
        }
        cleanup();
        for (size_t i = 0; i < small.size(); i++) results[small[i]] = sres[i];
    });
}

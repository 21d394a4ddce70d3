// Format selection by profiling runs: the paper's naive auto-tuner
// (Section V-E) times SpMV in every candidate format and keeps the fastest.
// Here it runs per matrix handle on the GPU, also picks the kernel variant
// (CSR lane grouping, XCD-aware tile order), prunes candidates that cannot
// win on bytes or that pad too much, and caches the decision per context
// under a fingerprint of the row structure.
#include <algorithm>
#include <cmath>
#include <sstream>
#include <vector>

#include "core.hpp"

namespace dsm {

Payload build_format(dsm_matrix m, int fmt, const dsm_convert_opts &o, hipStream_t s);

constexpr int BATCH_TUNE_ITERS = 20;  // CG iterations one batched-solver timing runs

template <class T>
__global__ void k_fill_value(i64 n, T *y, T v) {
    i64 i = (i64)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) y[i] = v;
}

static std::string fingerprint(dsm_matrix m, int vdt, int vec) {
    i64 st[38];
    row_stats(m, st, m->last_stream);
    std::ostringstream os;
    os << m->nrows << "x" << m->ncols << ":" << m->nnz << ":v" << vdt << ":x" << vec;
    for (int i = 0; i < 38; i++) os << "," << st[i];
    return os.str();
}

// Device buffer that cold timing reads before every timed SpMV.
struct Flush {
    void *buf = nullptr;
    double *part = nullptr;
    i64 bytes = 0;
};

// Median time (us) of `reps` SpMVs after `warmup` untimed ones: back to back
// with an event pair around each (warm), or, with a flush buffer, each SpMV
// started after a read of the whole buffer and timed by the events its own
// launches carry (cold, kernel-only).
static double time_spmv(dsm_matrix m, const Payload &P, int variant, const void *x, void *y, int vec, int warmup,
                        int reps, hipStream_t s, const Flush *flush = nullptr) {
    for (int i = 0; i < warmup; i++) spmv(m, P, x, y, vec, variant, s);
    if (flush && flush->bytes > 0) {
        // the kernel-only timer runs the handle's active payload and variant
        const Payload keep = m->P;
        const int keep_v = m->variant;
        m->P = P;
        m->variant = variant;
        std::vector<double> t(reps);
        try {
            for (int i = 0; i < reps; i++) {
                flush_read(flush->buf, flush->bytes, flush->part, s);
                t[i] = spmv_kernel_us(m, x, y, vec, s);
            }
        } catch (...) {
            m->P = keep;
            m->variant = keep_v;
            throw;
        }
        m->P = keep;
        m->variant = keep_v;
        std::sort(t.begin(), t.end());
        return reps ? t[reps / 2] : 0.0;
    }
    std::vector<hipEvent_t> ev(2 * reps);
    for (auto &e : ev) DSM_HIP(hipEventCreate(&e));
    for (int i = 0; i < reps; i++) {
        DSM_HIP(hipEventRecord(ev[2 * i], s));
        spmv(m, P, x, y, vec, variant, s);
        DSM_HIP(hipEventRecord(ev[2 * i + 1], s));
    }
    DSM_HIP(hipStreamSynchronize(s));
    std::vector<double> t(reps);
    for (int i = 0; i < reps; i++) {
        float ms = 0;
        DSM_HIP(hipEventElapsedTime(&ms, ev[2 * i], ev[2 * i + 1]));
        t[i] = ms * 1000.0;
    }
    for (auto &e : ev) (void)hipEventDestroy(e);
    std::sort(t.begin(), t.end());
    return reps ? t[reps / 2] : 0.0;
}

// ---------------------------------------------------------------- model
// Time of one SpMV predicted from the structure features: every format is
// a sum of sweeps of four kernel classes (COO, CSR, DIA, ELL; HYB = ELL +
// COO, HDC = DIA + CSR).  A sweep costs its traffic over the class's learned
// bandwidth, at least its critical path, plus a launch overhead per kernel.
// Traffic is the format's bytes (as spmv_bytes, from the features alone)
// plus one 64-byte sector for each x gather that leaves the cache window
// around the diagonal.  A CSR sweep's critical path is the longest row: one
// workgroup takes it in passes of 1024 entries, each pass two dependent
// memory round trips (1.2 us: rows of 4096 in an 8.7 us launch, 3.9 us of it
// the launch of a tiny matrix).
constexpr i64 NEAR_WINDOW = 1 << 16;
constexpr double FAR_BYTES = 64.0;
constexpr double LAUNCH_US = 3.0;
constexpr double ROW_PASS_US = 1.2;
constexpr double LEARN_MIN_BYTES = 16e6;  // smaller sweeps are latency-bound
enum { KC_COO = 0, KC_CSR = 1, KC_DIA = 2, KC_ELL = 3 };

struct Sweep {
    int kc = KC_CSR;
    double traffic = 0, crit_us = 0;
    int launches = 1;
};

struct Prediction {
    double bytes[6] = {0, 0, 0, 0, 0, 0};
    int feasible[6] = {0, 0, 0, 0, 0, 0};
    Sweep part[6][2];
    int nparts[6] = {1, 1, 1, 1, 2, 2};
};

static double csr_crit(i64 max_len) { return ROW_PASS_US * (double)std::max<i64>(1, (max_len + 1023) / 1024); }

static Prediction predict(const dsm_matrix_s *m, const StructFeatures &F, int vdt, int vec, double max_pad_ratio) {
    Prediction P;
    const double v = (double)dtype_size(vdt), i = 4.0, X = (double)dtype_size(vec);
    const double N = (double)m->nrows, nnz = (double)F.nnz, xy = (double)m->ncols * X + N * X;
    const double far = (double)(F.nnz - F.near);
    const double ratio = max_pad_ratio > 0 ? max_pad_ratio : 16.0;
    auto farof = [&](double part_nnz) { return nnz > 0 ? FAR_BYTES * far * part_nnz / nnz : 0.0; };
    P.bytes[DSM_COO] = nnz * (v + 2 * i) + xy;
    P.bytes[DSM_CSR] = nnz * (v + i) + (N + 1) * i + xy;
    P.bytes[DSM_DIA] = (double)F.ndiag * N * v + (double)F.ndiag * i + xy;
    P.bytes[DSM_ELL] = (double)F.max_len * N * (v + i) + xy;
    const double coo_part = (double)F.hyb_coo, ell_part = nnz - coo_part;
    P.bytes[DSM_HYB] = (double)F.hyb_width * N * (v + i) + coo_part * (v + 2 * i) + xy;
    const double rem = nnz - (double)F.hdc_dia_nnz;
    P.bytes[DSM_HDC] = (double)F.hdc_ndiag * N * v + (double)F.hdc_ndiag * i + rem * (v + i) + (N + 1) * i + xy;

    P.part[DSM_COO][0] = {KC_COO, P.bytes[DSM_COO] + farof(nnz), 0, 2};
    P.part[DSM_CSR][0] = {KC_CSR, P.bytes[DSM_CSR] + farof(nnz), csr_crit(F.max_len), 1};
    P.part[DSM_DIA][0] = {KC_DIA, P.bytes[DSM_DIA], 0, 1};
    P.part[DSM_ELL][0] = {KC_ELL, P.bytes[DSM_ELL] + farof(nnz), 0, 1};
    // the second part of HYB/HDC reads x again and updates the y rows it holds
    P.part[DSM_HYB][0] = {KC_ELL, (double)F.hyb_width * N * (v + i) + xy + farof(ell_part), 0, 1};
    P.part[DSM_HYB][1] = {KC_COO, coo_part * (v + 2 * i) + (double)m->ncols * X + 2 * std::min(coo_part, N) * X +
                                      farof(coo_part), 0, 2};
    P.part[DSM_HDC][0] = {KC_DIA, (double)F.hdc_ndiag * N * v + (double)F.hdc_ndiag * i + xy, 0, 1};
    P.part[DSM_HDC][1] = {KC_CSR, rem * (v + i) + (N + 1) * i + (double)m->ncols * X + 2 * N * X + farof(rem),
                          rem > 0 ? csr_crit(F.max_len) : 0.0, 1};
    if (coo_part == 0) P.nparts[DSM_HYB] = 1;
    for (int f = 0; f < 6; f++) P.feasible[f] = 1;
    if ((double)F.ndiag * N > ratio * std::max(nnz, 1.0)) P.feasible[DSM_DIA] = 0;
    if ((double)F.max_len * N > ratio * std::max(nnz, 1.0)) P.feasible[DSM_ELL] = 0;
    return P;
}

static double sweep_us(const Sweep &w, const double *bw) {
    return std::max(w.traffic / (bw[w.kc] * 1e3), w.crit_us) + w.launches * LAUNCH_US;
}

static double predict_us(const Prediction &P, int f, const double *bw) {
    double t = 0;
    for (int k = 0; k < P.nparts[f]; k++) t += sweep_us(P.part[f][k], bw);
    return t;
}

// Feeds one timed selection back into the context's bandwidth table: the
// single-sweep formats give their class's bandwidth directly, when the sweep
// was large enough to be bandwidth-bound.
static void learn(dsm_ctx ctx, const Prediction &P, const dsm_select_report &R, const int *best_variant) {
    std::lock_guard<std::mutex> lk(ctx->cache_mu);
    for (int f = 0; f < 6; f++) {
        if (R.status[f] != DSM_OK || R.median_us[f] <= 0) continue;
        if (best_variant[f] >= 0) ctx->model_variant[f] = best_variant[f];
        if (P.nparts[f] != 1 || f == DSM_HYB || f == DSM_HDC) continue;
        const Sweep &w = P.part[f][0];
        const double t = R.median_us[f] - w.launches * LAUNCH_US;
        if (w.traffic < LEARN_MIN_BYTES || t <= 2.0 * w.crit_us) continue;
        const double bw = w.traffic / (t * 1e3);  // GB/s
        ctx->model_bw[w.kc] = 0.5 * ctx->model_bw[w.kc] + 0.5 * bw;
    }
}

// preference order for exact ties: CSR, DIA, ELL, HYB, HDC, COO
static int rank_of(int f) {
    static const int r[6] = {5, 0, 1, 2, 3, 4};
    return r[f];
}

void select_format(dsm_matrix m, uint32_t mask, const dsm_select_opts &o, dsm_select_report *rep, hipStream_t s) {
    dsm_ctx ctx = m->ctx;
    dsm_select_report R{};
    for (int f = 0; f < DSM_NUM_FORMATS; f++) R.status[f] = DSM_E_UNSUPPORTED;
    const int vec = o.vec_dtype;
    DSM_CHECK(vec == DSM_F64 || vec == DSM_F32, DSM_E_INVALID, "vec_dtype must be F64 or F32");
    DSM_CHECK(o.target == 0 || o.target == 1, DSM_E_INVALID, "target must be 0 or 1");
    mask &= (1u << DSM_NUM_FORMATS) - 1;
    if (o.target == 1) {
        DSM_CHECK(m->nrows == m->ncols, DSM_E_UNSUPPORTED, "the batched solver needs a square matrix");
        DSM_CHECK(o.value_dtype == DSM_F64, DSM_E_UNSUPPORTED, "the batched solver uses FP64 values");
        mask &= (1u << DSM_CSR) | (1u << DSM_DIA) | (1u << DSM_ELL);
    }
    DSM_CHECK(mask != 0, DSM_E_INVALID, "empty candidate mask");
    m->last_stream = s;
    const std::string key =
        fingerprint(m, o.value_dtype, vec) + ":m" + std::to_string(mask) + ":t" + std::to_string(o.target) +
        (o.flush_bytes > 0 && o.target == 0 ? ":cold" : "");

    dsm_convert_opts co;
    dsm_convert_opts_default(&co);
    co.value_dtype = o.value_dtype;
    co.max_pad_ratio = o.max_pad_ratio;

    if (o.use_cache) {
        std::pair<int, int> hit{-1, 0};
        {
            std::lock_guard<std::mutex> lk(ctx->cache_mu);
            auto it = ctx->select_cache.find(key);
            if (it != ctx->select_cache.end()) hit = it->second;
        }
        if (hit.first >= 0) {
            if (!(m->P.fmt == hit.first && m->P.vdt == o.value_dtype)) {
                Payload np = build_format(m, hit.first, co, s);
                DSM_HIP(hipStreamSynchronize(s));
                m->P.release(ctx);
                m->P = np;
            }
            if (o.target == 1) {
                m->batch_lanes = hit.first == DSM_CSR ? hit.second : 0;
            } else {
                m->variant = hit.second;
                m->variant_set = true;
            }
            R.chosen = hit.first;
            R.chosen_variant = hit.second;
            R.cache_hit = 1;
            R.status[hit.first] = DSM_OK;
            R.bytes[hit.first] = spmv_bytes(m, m->P, vec);
            if (rep) *rep = R;
            return;
        }
    }

    // structure features of the matrix (through a CSR copy when the active
    // format is another one); they give the model's exact byte counts
    StructFeatures F;
    {
        Payload tmp;
        const Payload *C = &m->P;
        if (m->P.fmt != DSM_CSR) {
            tmp = to_csr(m, m->P, s);
            C = &tmp;
        }
        try {
            F = structure_features(m, *C, 0.5, NEAR_WINDOW, s);
        } catch (...) {
            tmp.release(ctx);
            throw;
        }
        tmp.release(ctx);
    }
    const Prediction PR = predict(m, F, o.value_dtype, vec, o.max_pad_ratio);

    if (o.reps == 0 && o.target == 0) {
        // online choice: no profiling runs, the model picks
        int best = -1;
        double bt = 0;
        {
            std::lock_guard<std::mutex> lk(ctx->cache_mu);
            for (int f : {DSM_CSR, DSM_DIA, DSM_ELL, DSM_HYB, DSM_HDC, DSM_COO}) {
                if (!(mask & (1u << f))) continue;
                R.bytes[f] = PR.bytes[f];
                if (!PR.feasible[f]) {
                    R.status[f] = DSM_E_INFEASIBLE;
                    continue;
                }
                R.status[f] = DSM_OK;
                R.median_us[f] = predict_us(PR, f, ctx->model_bw);
                if (best < 0 || R.median_us[f] < bt) {
                    best = f;
                    bt = R.median_us[f];
                }
            }
        }
        DSM_CHECK(best >= 0, DSM_E_INFEASIBLE, "no candidate format is feasible");
        hipEvent_t c0, c1;
        DSM_HIP(hipEventCreate(&c0));
        DSM_HIP(hipEventCreate(&c1));
        DSM_HIP(hipEventRecord(c0, s));
        if (!(m->P.fmt == best && m->P.vdt == o.value_dtype)) {
            Payload np = build_format(m, best, co, s);
            DSM_HIP(hipStreamSynchronize(s));
            m->P.release(ctx);
            m->P = np;
        }
        DSM_HIP(hipEventRecord(c1, s));
        DSM_HIP(hipEventSynchronize(c1));
        float cms = 0;
        DSM_HIP(hipEventElapsedTime(&cms, c0, c1));
        (void)hipEventDestroy(c0);
        (void)hipEventDestroy(c1);
        R.convert_us[best] = cms * 1e3;
        {
            std::lock_guard<std::mutex> lk(ctx->cache_mu);
            m->variant = ctx->model_variant[best];
            m->variant_set = true;
        }
        if (m->P.fmt == DSM_COO) m->variant = 0;
        R.chosen = best;
        R.chosen_variant = m->variant;
        if (rep) *rep = R;
        return;
    }

    const size_t xs = dtype_size(vec);
    void *x = dev_alloc(ctx, xs * (size_t)std::max<i64>(m->ncols, 1));
    void *y = nullptr;
    try {
        y = dev_alloc(ctx, xs * (size_t)std::max<i64>(m->nrows, 1));
    } catch (...) {
        dev_free(ctx, x, xs * (size_t)std::max<i64>(m->ncols, 1));
        throw;
    }
    Flush flush;
    if (o.flush_bytes > 0 && o.target == 0) {
        flush.bytes = (o.flush_bytes + 15) / 16 * 16;
        try {
            flush.buf = dev_alloc(ctx, (size_t)flush.bytes);
            flush.part = (double *)dev_alloc(ctx, sizeof(double) * DSM_PROBE_PARTIALS);
        } catch (...) {
            if (flush.buf) dev_free(ctx, flush.buf, (size_t)flush.bytes);
            dev_free(ctx, x, xs * (size_t)std::max<i64>(m->ncols, 1));
            dev_free(ctx, y, xs * (size_t)std::max<i64>(m->nrows, 1));
            throw;
        }
    }
    const unsigned gx = grid_for(m->ncols, 256);
    if (vec == DSM_F64) hipLaunchKernelGGL(k_fill_value<double>, dim3(gx), dim3(256), 0, s, m->ncols, (double *)x, 1.0);
    else hipLaunchKernelGGL(k_fill_value<float>, dim3(gx), dim3(256), 0, s, m->ncols, (float *)x, 1.0f);

    Payload best;
    int best_variant_per_fmt[6] = {-1, -1, -1, -1, -1, -1};
    bool have_best = false, best_is_current = false;
    double best_t = 0, best_bytes = 0, min_bytes = 0;
    int best_f = -1, best_v = 0;
    static const int order[6] = {DSM_CSR, DSM_DIA, DSM_ELL, DSM_HYB, DSM_HDC, DSM_COO};
    auto cleanup = [&] {
        (void)hipStreamSynchronize(s);
        dev_free(ctx, x, xs * (size_t)std::max<i64>(m->ncols, 1));
        dev_free(ctx, y, xs * (size_t)std::max<i64>(m->nrows, 1));
        if (flush.buf) {
            dev_free(ctx, flush.buf, (size_t)flush.bytes);
            dev_free(ctx, flush.part, sizeof(double) * DSM_PROBE_PARTIALS);
        }
    };
    try {
        for (int f : order) {
            if (!(mask & (1u << f))) continue;
            // candidate payload: the current one if it already matches
            Payload cand;
            bool is_current = m->P.fmt == f && m->P.vdt == o.value_dtype;
            hipEvent_t c0, c1;
            DSM_HIP(hipEventCreate(&c0));
            DSM_HIP(hipEventCreate(&c1));
            DSM_HIP(hipEventRecord(c0, s));
            if (!is_current) {
                try {
                    cand = build_format(m, f, co, s);
                } catch (const Error &e) {
                    (void)hipEventDestroy(c0);
                    (void)hipEventDestroy(c1);
                    if (e.status == DSM_E_INFEASIBLE || e.status == DSM_E_NOMEM) {
                        R.status[f] = e.status;
                        continue;
                    }
                    throw;
                }
            }
            DSM_HIP(hipEventRecord(c1, s));
            DSM_HIP(hipStreamSynchronize(s));
            float cms = 0;
            DSM_HIP(hipEventElapsedTime(&cms, c0, c1));
            (void)hipEventDestroy(c0);
            (void)hipEventDestroy(c1);
            R.convert_us[f] = is_current ? 0.0 : cms * 1000.0;
            const Payload &P = is_current ? m->P : cand;
            const double bytes = spmv_bytes(m, P, vec);
            R.bytes[f] = bytes;
            if (min_bytes > 0 && bytes > o.bytes_prefilter * min_bytes) {
                R.status[f] = DSM_E_UNSUPPORTED;  // pruned: cannot win on bytes
                if (!is_current) cand.release(ctx);
                continue;
            }
            min_bytes = min_bytes > 0 ? std::min(min_bytes, bytes) : bytes;
            // kernel variants of this format (target 1: CSR lanes per row)
            std::vector<int> variants{0};
            if (o.target == 1) {
                variants = f == DSM_CSR ? std::vector<int>{1, 2, 4, 8, 16, 32} : std::vector<int>{1};
            } else if (o.tune_variant) {
                if (f == DSM_CSR) variants = {0, 7, 8, 15, 2, 3, 4, 5, 6};
                else if (f == DSM_DIA || f == DSM_HDC)
                    variants = {0, 1, 2, 4, 8, 10, 12, 16, 18, 20, 19, 21, 32, 40, 48, 56, 50, 58};
                else if (f == DSM_ELL || f == DSM_HYB) variants = {0, 1, 2, 4, 8, 10, 12};
            }
            double tf = 0;
            int vf = 0;
            for (int v : variants) {
                double t = o.target == 1 ? time_batched_solve(m, P, v, BATCH_TUNE_ITERS, s)
                                         : time_spmv(m, P, v, x, y, vec, o.warmup, o.reps, s, &flush);
                // a later variant must be clearly faster (1%) to displace an
                // earlier one, so the choice does not flip on timing noise
                if (v == variants[0] || t < 0.99 * tf) {
                    tf = t;
                    vf = v;
                }
            }
            R.status[f] = DSM_OK;
            R.median_us[f] = tf;
            best_variant_per_fmt[f] = vf;
            bool better = !have_best;
            if (have_best) {
                if (tf < best_t * 0.98) better = true;
                else if (tf <= best_t * 1.02) {
                    if (bytes < best_bytes) better = true;
                    else if (bytes == best_bytes && rank_of(f) < rank_of(best_f)) better = true;
                }
            }
            if (better) {
                if (have_best && !best_is_current) best.release(ctx);
                if (is_current) {
                    best_is_current = true;
                } else {
                    best = cand;
                    best_is_current = false;
                }
                have_best = true;
                best_t = tf;
                best_bytes = bytes;
                best_f = f;
                best_v = vf;
            } else if (!is_current) {
                cand.release(ctx);
            }
        }
    } catch (...) {
        if (have_best && !best_is_current) best.release(ctx);
        cleanup();
        throw;
    }
    cleanup();
    DSM_CHECK(have_best, DSM_E_INFEASIBLE, "no candidate format is feasible");
    // the cost model learns warm bandwidths only (what back-to-back use sees)
    if (o.target == 0 && flush.bytes == 0) learn(ctx, PR, R, best_variant_per_fmt);
    if (!best_is_current) {
        m->P.release(ctx);
        m->P = best;
    }
    if (o.target == 1) {
        m->batch_lanes = best_f == DSM_CSR ? best_v : 0;
        m->variant = 0;
        m->variant_set = false;
    } else {
        m->variant = best_v;
        m->variant_set = true;
    }
    R.chosen = best_f;
    R.chosen_variant = best_v;
    {
        std::lock_guard<std::mutex> lk(ctx->cache_mu);
        ctx->select_cache[key] = {best_f, best_v};
    }
    if (rep) *rep = R;
}

}  // namespace dsm

using namespace dsm;

DSM_API void dsm_select_opts_default(dsm_select_opts *o) {
    if (!o) return;
    o->warmup = 3;
    o->reps = 20;
    o->use_cache = 1;
    o->tune_variant = 1;
    o->vec_dtype = DSM_F64;
    o->value_dtype = DSM_F64;
    o->max_pad_ratio = 16.0;
    o->bytes_prefilter = 2.0;
    o->target = 0;
    o->flush_bytes = 0;
}

DSM_API dsm_status dsm_select(dsm_matrix m, uint32_t candidate_mask, const dsm_select_opts *opts,
                              dsm_select_report *report, void *stream) {
    return guard([&] {
        DSM_CHECK(m && m->ctx, DSM_E_INVALID, "null matrix handle");
        DSM_HIP(hipSetDevice(m->ctx->device));
        dsm_select_opts o;
        dsm_select_opts_default(&o);
        if (opts) o = *opts;
        DSM_CHECK(o.reps >= 0 && o.warmup >= 0, DSM_E_INVALID, "reps and warmup must be >= 0");
        DSM_CHECK(o.reps >= 1 || o.target == 0, DSM_E_INVALID, "the batched target needs timed runs");
        DSM_CHECK(o.value_dtype >= DSM_F64 && o.value_dtype <= DSM_BF16, DSM_E_INVALID, "bad value dtype");
        if (o.bytes_prefilter <= 0) o.bytes_prefilter = 2.0;
        DSM_CHECK(o.flush_bytes >= 0, DSM_E_INVALID, "flush_bytes must be >= 0");
        select_format(m, candidate_mask, o, report, (hipStream_t)stream);
    });
}

DSM_API dsm_status dsm_time_spmv(dsm_matrix m, const void *x, void *y, dsm_dtype vec_dtype, int32_t warmup,
                                 int32_t reps, double *median_us, void *stream) {
    return guard([&] {
        DSM_CHECK(m && m->ctx && median_us, DSM_E_INVALID, "null argument");
        DSM_CHECK((x || m->ncols == 0) && (y || m->nrows == 0), DSM_E_INVALID, "null vector");
        DSM_CHECK(x != y || m->nrows == 0, DSM_E_INVALID, "x and y must not alias");
        DSM_CHECK(reps >= 1 && warmup >= 0, DSM_E_INVALID, "reps must be >= 1 and warmup >= 0");
        DSM_HIP(hipSetDevice(m->ctx->device));
        hipStream_t s = (hipStream_t)stream;
        *median_us = time_spmv(m, m->P, m->variant, x, y, vec_dtype, warmup, reps, s);
        m->last_stream = s;
    });
}

DSM_API dsm_status dsm_spmv_kernel_time(dsm_matrix m, const void *x, void *y, dsm_dtype vec_dtype, double *us,
                                        void *stream) {
    return guard([&] {
        DSM_CHECK(m && m->ctx && us, DSM_E_INVALID, "null argument");
        DSM_CHECK((x || m->ncols == 0) && (y || m->nrows == 0), DSM_E_INVALID, "null vector");
        DSM_CHECK(x != y || m->nrows == 0, DSM_E_INVALID, "x and y must not alias");
        DSM_HIP(hipSetDevice(m->ctx->device));
        hipStream_t s = (hipStream_t)stream;
        *us = spmv_kernel_us(m, x, y, vec_dtype, s);
        m->last_stream = s;
    });
}

DSM_API dsm_status dsm_select_cache_clear(dsm_ctx ctx) {
    return guard([&] {
        DSM_CHECK(ctx, DSM_E_INVALID, "null context");
        std::lock_guard<std::mutex> lk(ctx->cache_mu);
        ctx->select_cache.clear();
    });
}

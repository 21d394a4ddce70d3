// On-device format conversions (the "convert" operation: an element-wise
// copy between storage formats in the same memory space).
//
// Canonical CSR is the hub: every format is built from CSR and turned back
// into CSR with prefix scans, so each conversion is a handful of coalesced
// sweeps plus one scan and needs no sort.  Values are moved as raw bit
// patterns (64/32/16-bit words); the only arithmetic on values is the
// explicit narrowing cast (FP64 -> FP32 -> BF16, round to nearest even).
// Results are canonical encodings, identical bit for bit whatever the launch
// shape:
//   COO  sorted by (row, col)
//   DIA  offsets = ascending distinct (col - row); slot (k, i) holds
//        A(i, i + off_k) or +0; diagonal-major with a padded pitch
//   ELL  K = longest row; slot (k, i) = k-th entry of row i, empty slots
//        col -1 / value +0
//   HYB  ELL of width K_h (largest k reached by >= ceil(nrows/3) rows) plus
//        the remaining entries as sorted COO
//   HDC  DIA over diagonals with count >= theta * length, CSR for the rest
#include <algorithm>
#include <vector>

#include "clusters.hpp"
#include "core.hpp"

namespace dsm {

constexpr int CB = 256;        // threads per workgroup
constexpr int EB_ROWS = 256;   // rows per workgroup when walking entries
constexpr int CB_U = 8;        // entries a row-per-thread kernel loads per batch
constexpr int RB_T = 1024;     // adaptive CSR: nnz bucket per row block
constexpr int RB_RCAP = 256;   // adaptive CSR: max rows per block

static i64 pitch_for(i64 nrows) { return ((nrows + 63) / 64) * 64; }

// Raw storage word for a value dtype.
template <int DT> struct Word;
template <> struct Word<DSM_F64> { using T = u64; };
template <> struct Word<DSM_F32> { using T = u32; };
template <> struct Word<DSM_BF16> { using T = uint16_t; };

// +0 and -0 have all bits but the sign clear.
template <class W>
__device__ __forceinline__ bool word_is_zero(W w) {
    return (W)(w << 1) == 0;
}

// Calls f(row, entry) for every entry of rows [blockIdx.x*EB_ROWS, +EB_ROWS).
template <class F>
__device__ __forceinline__ void for_each_entry(i64 nrows, const i32 *rp, F f) {
    __shared__ i32 srp[EB_ROWS + 1];
    const i64 r0 = (i64)blockIdx.x * EB_ROWS;
    const int nr = (int)min((i64)EB_ROWS, nrows - r0);
    for (int t = threadIdx.x; t <= nr; t += blockDim.x) srp[t] = rp[r0 + t];
    __syncthreads();
    const i64 e0 = srp[0], e1 = srp[nr];
    for (i64 e = e0 + threadIdx.x; e < e1; e += blockDim.x) {
        int lo = 0, hi = nr;  // invariant: srp[lo] <= e < srp[hi]
        while (hi - lo > 1) {
            int mid = (lo + hi) >> 1;
            if ((i64)srp[mid] <= e) lo = mid;
            else hi = mid;
        }
        f(r0 + lo, e);
    }
}

static unsigned entry_grid(i64 nrows) { return grid_for(nrows, EB_ROWS); }

// Privatised counting for histograms whose keys repeat heavily inside a
// workgroup (the diagonals of a banded matrix, the row lengths of a regular
// one): one global atomic per entry on a handful of bins serialises at the
// memory side (about 15 ms for the 29.8M entries of HPCG 104^3).  Counts go
// to an open-addressing table in LDS instead and reach the global bins once
// per workgroup and key; a key that finds no free slot within HT_PROBES goes
// straight to its global bin.  Keys are non-negative int32 (-1 = empty).
constexpr int HT_LOG = 11, HT = 1 << HT_LOG, HT_PROBES = 8;

__device__ __forceinline__ void ht_init(i32 *hk, i32 *hv) {
    for (int t = threadIdx.x; t < HT; t += blockDim.x) {
        hk[t] = -1;
        hv[t] = 0;
    }
    __syncthreads();
}

__device__ __forceinline__ void ht_add(i32 *hk, i32 *hv, i32 key, i32 *global) {
    unsigned h = ((unsigned)key * 2654435761u) >> (32 - HT_LOG);
    for (int probe = 0; probe < HT_PROBES; probe++, h = (h + 1) & (HT - 1)) {
        i32 k = __atomic_load_n(&hk[h], __ATOMIC_RELAXED);
        if (k == -1) {
            k = atomicCAS(&hk[h], -1, key);
            if (k == -1) k = key;
        }
        if (k == key) {
            atomicAdd(&hv[h], 1);
            return;
        }
    }
    atomicAdd(&global[key], 1);
}

// after a barrier that follows every ht_add of the workgroup
__device__ __forceinline__ void ht_flush(const i32 *hk, const i32 *hv, i32 *global) {
    for (int t = threadIdx.x; t < HT; t += blockDim.x)
        if (hk[t] >= 0 && hv[t] > 0) atomicAdd(&global[hk[t]], hv[t]);
}

// ---------------------------------------------------------------- validation
// err: bit 0 row_ptr[0] != 0, bit 1 row_ptr[n] != nnz, bit 2 decreasing or
// out-of-range pointers, bit 3 column out of range, bit 4 columns not
// strictly ascending (duplicates included).
__global__ void k_validate_csr(i64 nrows, i64 ncols, i64 nnz, const i32 *rp, const i32 *col, int *err) {
    i64 i = (i64)blockIdx.x * blockDim.x + threadIdx.x;
    if (i == 0) {
        if (rp[0] != 0) atomicOr(err, 1);
        if ((i64)rp[nrows] != nnz) atomicOr(err, 2);
    }
    if (i >= nrows) return;
    i64 a = rp[i], b = rp[i + 1];
    if (a < 0 || b < a || b > nnz) {
        atomicOr(err, 4);
        return;
    }
    // CB_U columns loaded together (indices clamped into the row, so every
    // load is unconditional), then checked in order
    i32 prev = -1;
    int bad = 0;
    for (i64 k0 = a; k0 < b; k0 += CB_U) {
        i32 c[CB_U];
#pragma unroll
        for (int u = 0; u < CB_U; u++) c[u] = col[min(k0 + u, b - 1)];
#pragma unroll
        for (int u = 0; u < CB_U; u++)
            if (k0 + u < b) {
                if (c[u] < 0 || (i64)c[u] >= ncols) bad |= 8;
                if (c[u] <= prev) bad |= 16;
                prev = c[u];
            }
    }
    if (bad) atomicOr(err, bad);
}

static int read_flag(int *d, hipStream_t s) {
    int h = 0;
    DSM_HIP(hipMemcpyAsync(&h, d, sizeof(int), hipMemcpyDeviceToHost, s));
    DSM_HIP(hipStreamSynchronize(s));
    return h;
}

// RAII scratch allocation; every use is ordered on `s`.
struct Tmp {
    dsm_ctx ctx;
    void *p = nullptr;
    size_t n = 0;
    hipStream_t s;
    Tmp(dsm_ctx c, size_t bytes, hipStream_t st) : ctx(c), n(bytes ? bytes : 16), s(st) { p = dev_alloc(ctx, n, s); }
    ~Tmp() {
        if (p) dev_free(ctx, p, n, s);
    }
    Tmp(const Tmp &) = delete;
    Tmp &operator=(const Tmp &) = delete;
    template <class T> T *as() { return (T *)p; }
};

void validate_csr(dsm_ctx ctx, i64 nrows, i64 ncols, i64 nnz, const i32 *rp, const i32 *col, hipStream_t s) {
    Tmp err(ctx, sizeof(int), s);
    DSM_HIP(hipMemsetAsync(err.p, 0, sizeof(int), s));
    hipLaunchKernelGGL(k_validate_csr, dim3(grid_for(nrows, CB)), dim3(CB), 0, s, nrows, ncols, nnz, rp, col,
                       err.as<int>());
    DSM_HIP(hipGetLastError());
    int f = read_flag(err.as<int>(), s);
    if (f) {
        std::string why;
        if (f & 1) why += " row_ptr[0] != 0;";
        if (f & 2) why += " row_ptr[nrows] != nnz;";
        if (f & 4) why += " row pointers decrease or leave [0, nnz];";
        if (f & 8) why += " column index out of range;";
        if (f & 16) why += " columns not strictly ascending within a row (unsorted or duplicate);";
        fail(DSM_E_INVALID, "invalid CSR:" + why);
    }
}

// ---------------------------------------------------------------- row blocks
// Row i opens a block when its first entry falls in another RB_T-bucket than
// row i-1's, when row i or row i-1 is longer than RB_T (long rows stand
// alone), or at every multiple of RB_RCAP.  Every block therefore holds fewer
// than 2*RB_T entries and at most RB_RCAP rows, or is one long row.
__global__ void k_rowblock_flags(i64 nrows, const i32 *rp, i32 *flag) {
    i64 i = (i64)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nrows) return;
    int f = 1;
    if (i > 0) {
        i32 a = rp[i - 1], b = rp[i], c = rp[i + 1];
        f = (b / RB_T != a / RB_T) || (b - a > RB_T) || (c - b > RB_T) || (i % RB_RCAP == 0);
    }
    flag[i] = f;
}

__global__ void k_rowblock_scatter(i64 nrows, const i32 *flag, const i32 *pos, i32 *blocks, i64 nblocks) {
    i64 i = (i64)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < nrows && flag[i]) blocks[pos[i]] = (i32)i;
    if (i == 0) blocks[nblocks] = (i32)nrows;
}

// What decides how a large matrix' row blocks are swept, in parts per
// workgroup.  out[0]: entries of rows of more than 32 and four times the mean;
// out[1], out[2]: of 4096 pairs of neighbouring rows, spread over the matrix,
// those with entries, and those whose first columns lie more than STRUCT_FAR
// apart.  A few workgroups, and no atomics (one per wave took 155 us on a Zipf
// matrix of 1M rows).
constexpr int STRUCT_GROUPS = 512, STRUCT_PAIRS = 4096 / STRUCT_GROUPS, STRUCT_FAR = 1024;
__global__ void __launch_bounds__(CB) k_row_structure(i64 nrows, const i32 *rp, const i32 *col, i32 *out) {
    __shared__ i32 lds[CB / WAVE];
    const i64 t = (i64)blockIdx.x * CB + threadIdx.x, threads = (i64)STRUCT_GROUPS * CB;
    bool pair = false;
    i32 apart = 0;
    if (threadIdx.x < STRUCT_PAIRS) {
        const i64 i = ((i64)blockIdx.x * STRUCT_PAIRS + threadIdx.x) * (nrows - 1) / 4096;  // below nrows - 1
        const i32 a = rp[i], b = rp[i + 1];
        pair = a < b && b < rp[i + 2];
        apart = pair ? abs(col[b] - col[a]) : 0;
    }
    const i64 long_row = max(32ll, 4 * (i64)rp[nrows] / nrows);
    i32 heavy = 0;
    for (i64 r = t; r < nrows; r += threads) {
        const i32 len = rp[r + 1] - rp[r];
        heavy += len > long_row ? len : 0;
    }
    const i32 n[3] = {heavy, pair, apart > STRUCT_FAR};
    for (int k = 0; k < 3; k++) {
        const i32 sum = block_sum<CB>(n[k], lds);
        if (threadIdx.x == 0) out[k * STRUCT_GROUPS + blockIdx.x] = sum;
    }
}

void build_row_blocks(dsm_ctx ctx, Payload &P, i64 nrows, hipStream_t s) {
    if (nrows == 0) {
        P.nrblocks = 0;
        P.rblocks = (i32 *)P.alloc(ctx, sizeof(i32));
        DSM_HIP(hipMemsetAsync(P.rblocks, 0, sizeof(i32), s));
        return;
    }
    Tmp flag(ctx, sizeof(i32) * (size_t)nrows, s), pos(ctx, sizeof(i32) * (size_t)(nrows + 1), s);
    hipLaunchKernelGGL(k_rowblock_flags, dim3(grid_for(nrows, CB)), dim3(CB), 0, s, nrows, P.rp, flag.as<i32>());
    DSM_HIP(hipGetLastError());
    i64 nb = exclusive_scan_i32(ctx, flag.as<i32>(), pos.as<i32>(), nrows, s, true);
    P.nrblocks = nb;
    P.rblocks = (i32 *)P.alloc(ctx, sizeof(i32) * (size_t)(nb + 1));
    const bool big = nb >= 4096;
    i32 h[3 * STRUCT_GROUPS] = {};
    hipLaunchKernelGGL(k_rowblock_scatter, dim3(grid_for(nrows, CB)), dim3(CB), 0, s, nrows, flag.as<i32>(),
                       pos.as<i32>(), P.rblocks, nb);
    if (big)  // (the flags have been read; 4096 blocks are 4096 rows and more)
        hipLaunchKernelGGL(k_row_structure, dim3(STRUCT_GROUPS), dim3(CB), 0, s, nrows, P.rp, P.col, flag.as<i32>());
    DSM_HIP(hipGetLastError());
    if (big) DSM_HIP(hipMemcpyAsync(h, flag.p, sizeof(h), hipMemcpyDeviceToHost, s));
    DSM_HIP(hipStreamSynchronize(s));
    i64 sum[3] = {0, 0, 0};
    for (int k = 0; k < 3 * STRUCT_GROUPS; k++) sum[k / STRUCT_GROUPS] += h[k];
    P.skewed = sum[0] > P.csr_nnz / 8;
    P.scattered = sum[2] > sum[1] / 2;
}

// ---------------------------------------------------------------- small kernels
__global__ void k_row_len(i64 nrows, const i32 *rp, i32 *len) {
    i64 i = (i64)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < nrows) len[i] = rp[i + 1] - rp[i];
}

template <class Wi, class Wo, int DTI, int DTO>
__global__ void k_cast(i64 n, const Wi *in, Wo *out) {
    i64 i = (i64)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    Wi w = in[i];
    double d;
    float f;
    if constexpr (DTI == DSM_F64) {
        memcpy(&d, &w, 8);
    } else if constexpr (DTI == DSM_F32) {
        memcpy(&f, &w, 4);
        d = (double)f;
    } else {
        bf16 h;
        h.bits = w;
        d = (double)bf16_to_float(h);
    }
    Wo o;
    if constexpr (DTO == DSM_F64) {
        memcpy(&o, &d, 8);
    } else if constexpr (DTO == DSM_F32) {
        f = (float)d;  // round to nearest even (exact when widening)
        memcpy(&o, &f, 4);
    } else {
        // narrowing goes through FP32; from FP32 or BF16 sources it is exact
        f = (float)d;
        o = float_to_bf16(f).bits;
    }
    out[i] = o;
}

// Flags a value whose cast to DTO (the cast k_cast applies), widened back,
// differs from it bit for bit (NaN payloads and the sign of zero included).
template <class Wi, int DTI, int DTO>
__global__ void k_values_exact(i64 first, i64 n, const Wi *in, int *bad) {
    i64 i = (first + blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= n) return;
    Wi w = in[i];
    double d;
    if constexpr (DTI == DSM_F64) {
        memcpy(&d, &w, 8);
    } else {
        float f;
        memcpy(&f, &w, 4);
        d = (double)f;
    }
    const float f = (float)d;
    const double back = DTO == DSM_F32 ? (double)f : (double)bf16_to_float(float_to_bf16(f));
    u64 a, b;
    memcpy(&a, &d, 8);
    memcpy(&b, &back, 8);
    if (a != b) *bad = 1;
}

// Dispatch helpers over the value storage width.
#define DSM_BY_DTYPE(dt, ...)                                                            \
    switch (dt) {                                                                        \
    case DSM_F64: { using W = u64; __VA_ARGS__; break; }                                 \
    case DSM_F32: { using W = u32; __VA_ARGS__; break; }                                 \
    default: { using W = uint16_t; __VA_ARGS__; break; }                                 \
    }

static void cast_values(int dti, const void *in, int dto, void *out, i64 n, hipStream_t s) {
    if (n == 0) return;
    if (dti == dto) {
        DSM_HIP(hipMemcpyAsync(out, in, (size_t)n * dtype_size(dti), hipMemcpyDeviceToDevice, s));
        return;
    }
    dim3 g(grid_for(n, CB)), b(CB);
#define CASTK(WI, WO, A, B) hipLaunchKernelGGL((k_cast<WI, WO, A, B>), g, b, 0, s, n, (const WI *)in, (WO *)out)
    if (dti == DSM_F64 && dto == DSM_F32) CASTK(u64, u32, DSM_F64, DSM_F32);
    else if (dti == DSM_F64 && dto == DSM_BF16) CASTK(u64, uint16_t, DSM_F64, DSM_BF16);
    else if (dti == DSM_F32 && dto == DSM_F64) CASTK(u32, u64, DSM_F32, DSM_F64);
    else if (dti == DSM_F32 && dto == DSM_BF16) CASTK(u32, uint16_t, DSM_F32, DSM_BF16);
    else if (dti == DSM_BF16 && dto == DSM_F64) CASTK(uint16_t, u64, DSM_BF16, DSM_F64);
    else CASTK(uint16_t, u32, DSM_BF16, DSM_F32);
#undef CASTK
    DSM_HIP(hipGetLastError());
}

Payload cast_csr(dsm_matrix m, const Payload &src, int vdt, hipStream_t s) {
    Payload P;
    P.fmt = DSM_CSR;
    P.vdt = vdt;
    P.csr_nnz = src.csr_nnz;
    try {
        P.rp = (i32 *)P.alloc(m->ctx, sizeof(i32) * (size_t)(m->nrows + 1));
        P.col = (i32 *)P.alloc(m->ctx, sizeof(i32) * (size_t)src.csr_nnz);
        P.val = P.alloc(m->ctx, dtype_size(vdt) * (size_t)src.csr_nnz);
        DSM_HIP(hipMemcpyAsync(P.rp, src.rp, sizeof(i32) * (size_t)(m->nrows + 1), hipMemcpyDeviceToDevice, s));
        DSM_HIP(hipMemcpyAsync(P.col, src.col, sizeof(i32) * (size_t)src.csr_nnz, hipMemcpyDeviceToDevice, s));
        cast_values(src.vdt, src.val, vdt, P.val, src.csr_nnz, s);
        build_row_blocks(m->ctx, P, m->nrows, s);
    } catch (...) {
        P.release(m->ctx);
        throw;
    }
    return P;
}

// ---------------------------------------------------------------- CSR <-> COO
__global__ void __launch_bounds__(CB) k_csr_expand_rows(i64 nrows, const i32 *rp, i32 *row) {
    for_each_entry(nrows, rp, [&](i64 r, i64 e) { row[e] = (i32)r; });
}

// Sorted COO rows -> row pointers; flags unsorted/duplicate/out-of-range.
__global__ void k_coo_rowptr(i64 nnz, i64 nrows, i64 ncols, const i32 *row, const i32 *col, i32 *rp, int *err) {
    i64 k = (i64)blockIdx.x * blockDim.x + threadIdx.x;
    if (k > nnz) return;
    i64 prev = k == 0 ? -1 : (i64)row[k - 1];
    i64 cur = k == nnz ? nrows : (i64)row[k];
    if (k < nnz) {
        if (cur < 0 || cur >= nrows || col[k] < 0 || (i64)col[k] >= ncols) {
            if (err) atomicOr(err, 8);
            return;
        }
        if (k > 0 && (cur < prev || (cur == prev && col[k] <= col[k - 1]))) {
            if (err) atomicOr(err, 16);
            return;
        }
    }
    if (prev < -1 || prev >= nrows) return;  // reported by the previous entry
    for (i64 r = prev + 1; r <= cur; r++) rp[r] = (i32)k;
}

// ---------------------------------------------------------------- DIA
// MARK_L lanes per row, so that no entry has to look its row up; a flag is
// read (from cache, for all but the first entries of a diagonal) before it is
// set.  HPCG 104^3: 107 us with a search of the row per entry and a store
// each, now 40 us.
constexpr int MARK_L = 8;
__global__ void __launch_bounds__(CB) k_diag_mark(i64 first, i64 nrows, const i32 *rp, const i32 *col, i32 *flag) {
    const i64 r = ((first + blockIdx.x) * CB + threadIdx.x) / MARK_L;
    if (r >= nrows) return;
    const i64 e1 = rp[r + 1];
    i32 *f = flag + (nrows - 1 - r);
    for (i64 e = rp[r] + threadIdx.x % MARK_L; e < e1; e += 4 * MARK_L) {
        i32 c[4], t[4];
#pragma unroll
        for (int u = 0; u < 4; u++) c[u] = col[min(e + u * MARK_L, e1 - 1)];
#pragma unroll
        for (int u = 0; u < 4; u++) t[u] = f[c[u]];
#pragma unroll
        for (int u = 0; u < 4; u++)
            if (t[u] == 0) f[c[u]] = 1;
    }
}

static void diag_mark(i64 nrows, const i32 *rp, const i32 *col, i32 *flag, hipStream_t s) {
    in_launches((nrows + CB / MARK_L - 1) / (CB / MARK_L), [&](i64 first, unsigned g) {
        hipLaunchKernelGGL(k_diag_mark, dim3(g), dim3(CB), 0, s, first, nrows, rp, col, flag);
    });
}

// Entries per diagonal (index col - row + nrows - 1).  `table`: the span of
// indices fits int32 keys, so the counts are privatised in LDS.
__global__ void __launch_bounds__(CB) k_diag_count(i64 nrows, const i32 *rp, const i32 *col, i32 *cnt, int table) {
    __shared__ i32 hk[HT], hv[HT];
    if (!table) {
        for_each_entry(nrows, rp, [&](i64 r, i64 e) { atomicAdd(&cnt[(i64)col[e] - r + nrows - 1], 1); });
        return;
    }
    ht_init(hk, hv);
    for_each_entry(nrows, rp, [&](i64 r, i64 e) { ht_add(hk, hv, (i32)((i64)col[e] - r + nrows - 1), cnt); });
    __syncthreads();
    ht_flush(hk, hv, cnt);
}

static void diag_count(i64 n, i64 span, const i32 *rp, const i32 *col, i32 *cnt, hipStream_t s) {
    if (n > 0)
        hipLaunchKernelGGL(k_diag_count, dim3(entry_grid(n)), dim3(CB), 0, s, n, rp, col, cnt,
                           span <= (i64)INT32_MAX ? 1 : 0);
}

__global__ void k_offsets_compact(i64 span, i64 nrows, const i32 *flag, const i32 *slot, i32 *offs) {
    i64 d = (i64)blockIdx.x * blockDim.x + threadIdx.x;
    if (d < span && flag[d]) offs[slot[d]] = (i32)(d - (nrows - 1));
}

// Diagonal d (index d + nrows - 1) is "true" for HDC when its count reaches
// theta times the number of in-range positions on it (decided in FP64).
__global__ void k_hdc_true(i64 span, i64 nrows, i64 ncols, double theta, const i32 *cnt, i32 *flag) {
    i64 s = (i64)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= span) return;
    i64 d = s - (nrows - 1);
    i64 lo = d < 0 ? -d : 0;
    i64 hi = min(nrows, ncols - d);
    i64 L = hi > lo ? hi - lo : 0;
    i32 c = cnt[s];
    flag[s] = (c > 0 && (double)c >= theta * (double)L) ? 1 : 0;
}

// ---- 64 rows through LDS
// CSR keeps a row's entries together, DIA and ELL keep slot k of consecutive
// rows together.  The kernels that go between them take 64 rows per workgroup
// and turn them around in LDS, so that both sides are read and written in
// runs: thread t has row t % 64 of the group and the t / 64-th quarter of the
// slots.  A group with more entries than the launch's LDS holds (`cap`)
// works on memory directly.
constexpr int RG = 64;            // rows per workgroup
constexpr int RGP = CB / RG;      // threads per row
constexpr int RG_MAX_CAP = 8192;  // 96 KB with FP64 values

// LDS entries for groups of average size, with a quarter of slack.
static int rg_cap(i64 nnz, i64 nrows) {
    const i64 mean = nrows > 0 ? (nnz * RG + nrows - 1) / nrows : 0;
    return (int)std::min<i64>(RG_MAX_CAP, std::max<i64>(512, (mean * 5 / 4 + 63) / 64 * 64));
}
template <class W>
static size_t rg_bytes(int cap) { return (size_t)cap * (sizeof(W) + sizeof(i32)); }

template <class W>
struct RowGroup {
    i32 *srp;  // RG + 1 row pointers, relative to e0
    const i32 *c;
    const W *v;  // entry e of the group: c[e], v[e]
    i64 r0, e0;

    // Loads the row pointers and, where they fit, the entries of the group's rows
    // [r0, r0 + RG); rows past nrows are empty.  Ends with a barrier.
    __device__ __forceinline__ RowGroup(i64 group, i64 nrows, const i32 *rp, const i32 *col, const W *val, int cap,
                                        char *lds, i32 *srp_)
        : srp(srp_) {
        r0 = group * RG;
        e0 = rp[min(r0, nrows)];
        for (int t = threadIdx.x; t <= RG; t += CB) srp[t] = (i32)(rp[min(r0 + t, nrows)] - e0);
        __syncthreads();
        const int ne = srp[RG];
        if (ne <= cap) {
            W *sv = (W *)lds;
            i32 *sc = (i32 *)(sv + cap);
            for (int e = threadIdx.x; e < ne; e += CB) {
                sc[e] = col[e0 + e];
                sv[e] = val[e0 + e];
            }
            c = sc;
            v = sv;
        } else {
            c = col + e0;
            v = val + e0;
        }
        __syncthreads();
    }
};

// CSR -> DIA: every slot of rows [0, pitch) of the diagonals offs (entries
// on other diagonals, HDC's remainder, are passed over), zero where the row
// has no entry.  Bound by its 360 MB read and 243 MB written at HPCG 104^3:
// 265 us + 32 us of clearing for a scatter of single entries, now 135 us (4.5 TB/s).
template <class W>
__global__ void __launch_bounds__(CB) k_dia_fill(i64 group0, i64 nrows, const i32 *rp, const i32 *col,
                                                 const W *val, i64 ndiag, const i32 *offs, i64 pitch, W *dval,
                                                 int cap) {
    extern __shared__ __align__(16) char rg_lds[];
    __shared__ i32 srp[RG + 1];
    const RowGroup<W> G(group0 + blockIdx.x, nrows, rp, col, val, cap, rg_lds, srp);
    const int row = threadIdx.x % RG, part = __builtin_amdgcn_readfirstlane(threadIdx.x / RG);  // a wave per part
    const i64 i = G.r0 + row;
    const int k0 = (int)(ndiag * part / RGP), k1 = (int)(ndiag * (part + 1) / RGP);
    if (k0 == k1) return;
    int e = srp[row], hi = srp[row + 1];
    const int end = hi;
    const i64 first = i + offs[k0];
    while (e < hi) {
        const int mid = (e + hi) >> 1;
        if ((i64)G.c[mid] < first) e = mid + 1;
        else hi = mid;
    }
    i64 cur = e < end ? (i64)G.c[e] : INT64_MAX;
    for (int k = k0; k < k1; k++) {
        const i64 j = i + offs[k];
        while (cur < j) {
            e++;
            cur = e < end ? (i64)G.c[e] : INT64_MAX;
        }
        dval[k * pitch + i] = cur == j ? G.v[e] : (W)0;
    }
}

// Per row: entries not on a true diagonal (HDC remainder).  Column loads of
// CB_U entries, then their flag loads, are issued together (entries past the
// row read the sentinel column, then the sentinel as their flag: nonzero, so
// they count nothing).
__global__ void __launch_bounds__(CB) k_rest_count(i64 nrows, const i32 *rp, const i32 *col, const i32 *flag,
                                                   i32 *cnt) {
    const i64 i = (i64)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nrows) return;
    const i64 a = rp[i], b = rp[i + 1];
    i32 n_rest = 0;
    for (i64 e0 = a; e0 < b; e0 += CB_U) {
        i32 c[CB_U], f[CB_U];
#pragma unroll
        for (int u = 0; u < CB_U; u++) c[u] = *(e0 + u < b ? col + e0 + u : sentinel_ptr<i32>());
#pragma unroll
        for (int u = 0; u < CB_U; u++) f[u] = *(c[u] >= 0 ? flag + ((i64)c[u] - i + nrows - 1) : sentinel_ptr<i32>());
#pragma unroll
        for (int u = 0; u < CB_U; u++) n_rest += f[u] ? 0 : 1;
    }
    cnt[i] = n_rest;
}

template <class W>
__global__ void k_rest_fill(i64 nrows, const i32 *rp, const i32 *col, const W *val, const i32 *flag,
                            const i32 *orp, i32 *ocol, W *oval) {
    i64 i = (i64)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nrows) return;
    i64 o = orp[i];
    for (i64 e = rp[i]; e < rp[i + 1]; e++) {
        if (flag[(i64)col[e] - i + nrows - 1]) continue;
        ocol[o] = col[e];
        oval[o] = val[e];
        o++;
    }
}

// DIA -> CSR: count, then fill in ascending offset order, dropping +-0.
template <class W>
__global__ void k_dia_rowcount(i64 nrows, i64 ncols, i64 ndiag, const i32 *offs, const W *dval, i64 pitch,
                               const i32 *extra_rp, i32 *cnt) {
    i64 i = (i64)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nrows) return;
    i32 c = 0;
    for (i64 k = 0; k < ndiag; k++) {
        i64 j = i + offs[k];
        if (j >= 0 && j < ncols && !word_is_zero(dval[k * pitch + i])) c++;
    }
    if (extra_rp) c += extra_rp[i + 1] - extra_rp[i];
    cnt[i] = c;
}

// Slot arrays -> CSR rows, 64 rows per workgroup, RGB slots of a row per
// thread and pass; a row's entries keep their slot order.
constexpr int RGB = 8;

// DIA slots: +-0 is no entry.
template <class W>
struct DiaSlots {
    i64 ncols;
    const i32 *offs;
    const W *val;
    i64 pitch;
    __device__ __forceinline__ bool get(i64 k, i64 i, i32 *c, W *v) const {
        *v = val[k * pitch + i];
        const i64 j = i + offs[k];
        *c = (i32)j;
        return j >= 0 && j < ncols && !word_is_zero(*v);
    }
};
// ELL slots: column -1 is none.
template <class W>
struct EllSlots {
    const i32 *col;
    const W *val;
    i64 pitch;
    __device__ __forceinline__ bool get(i64 k, i64 i, i32 *c, W *v) const {
        *c = col[k * pitch + i];
        *v = val[k * pitch + i];
        return *c >= 0;
    }
};

// xrp, xcol, xval: a row's further entries (HDC's CSR part, HYB's COO part),
// in ascending columns.  MERGE: they lie between the slots' columns, and such
// a row is merged entry by entry by one thread; else they follow them.
// Bound by its 243 MB read and 360 MB written at HPCG 104^3 from DIA: 1031 us
// with a row per thread, each load behind the last test, now 148 us (4.1 TB/s).
template <class W, class Slots, bool MERGE>
__global__ void __launch_bounds__(CB) k_slots_to_csr(i64 group0, i64 nrows, i64 nk, Slots S, const i32 *xrp,
                                                     const i32 *xcol, const W *xval, const i32 *orp, i32 *ocol, W *oval, int cap) {
    extern __shared__ __align__(16) char rg_lds[];
    __shared__ i32 srp[RG + 1];
    __shared__ i32 cnt[2][RGP][RG];
    const i64 r0 = (group0 + blockIdx.x) * RG;
    const i64 e0 = orp[r0];
    for (int t = threadIdx.x; t <= RG; t += CB) srp[t] = (i32)(orp[min(r0 + t, nrows)] - e0);
    __syncthreads();
    const int ne = srp[RG];
    const bool staged = ne <= cap;
    W *sv = (W *)rg_lds;
    i32 *sc = (i32 *)(sv + cap);
    const int row = threadIdx.x % RG, part = __builtin_amdgcn_readfirstlane(threadIdx.x / RG);  // a wave per part
    const i64 i = r0 + row;
    const bool live = i < nrows;
    const i64 x0 = live && xrp ? xrp[i] : 0, x1 = live && xrp ? xrp[i + 1] : 0;
    const bool serial = MERGE && x1 > x0;
    int o = srp[row];
    auto put = [&](int at, i32 c, W v) {
        if (staged) {
            sc[at] = c;
            sv[at] = v;
        } else {
            ocol[e0 + at] = c;
            oval[e0 + at] = v;
        }
    };
    for (i64 k0 = 0, pass = 0; k0 < nk; k0 += RGP * RGB, pass ^= 1) {
        i32 c[RGB];
        W v[RGB];
        bool on[RGB];
        int n = 0;
#pragma unroll
        for (int u = 0; u < RGB; u++) {
            const i64 k = k0 + part * RGB + u;
            on[u] = S.get(min(k, nk - 1), live ? i : nrows - 1, &c[u], &v[u]);
            on[u] = on[u] && k < nk && live && !serial;
            n += on[u];
        }
        cnt[pass][part][row] = n;
        __syncthreads();
        int at = o;
#pragma unroll
        for (int p = 0; p < RGP; p++) {
            const int t = cnt[pass][p][row];
            at += p < part ? t : 0;
            o += t;
        }
#pragma unroll
        for (int u = 0; u < RGB; u++)
            if (on[u]) put(at++, c[u], v[u]);
    }
    if (serial) {
        if (part == 0) {
            i64 k = 0, e = x0;
            i32 c = 0;
            W v = 0;
            for (;;) {
                bool slot = false;
                for (; k < nk && !(slot = S.get(k, i, &c, &v)); k++) {}
                if (!slot && e >= x1) break;
                if (slot && (e >= x1 || c < xcol[e])) {
                    put(o++, c, v);
                    k++;
                } else {
                    put(o++, xcol[e], xval[e]);
                    e++;
                }
            }
        }
    } else {
        for (i64 e = x0 + part; e < x1; e += RGP) put(o + (int)(e - x0), xcol[e], xval[e]);
    }
    if (!staged) return;
    __syncthreads();
    for (int e = threadIdx.x; e < ne; e += CB) {
        ocol[e0 + e] = sc[e];
        oval[e0 + e] = sv[e];
    }
}

// ---------------------------------------------------------------- ELL / HYB
// Every slot of rows [0, pitch): the k-th entry of the row for k < len, the
// -1 column sentinel and a zero value after the row's end and in the pitch
// padding rows (so no memset is needed first).
template <class W>
__global__ void __launch_bounds__(CB) k_ell_fill(i64 group0, i64 nrows, i64 pitch, const i32 *rp, const i32 *col,
                                                 const W *val, i64 K, i32 *ecol, W *eval, int cap) {
    extern __shared__ __align__(16) char rg_lds[];
    __shared__ i32 srp[RG + 1];
    const RowGroup<W> G(group0 + blockIdx.x, nrows, rp, col, val, cap, rg_lds, srp);
    const int row = threadIdx.x % RG, part = __builtin_amdgcn_readfirstlane(threadIdx.x / RG);  // a wave per part
    const i64 i = G.r0 + row;
    const int a = srp[row], len = srp[row + 1] - a;
    for (i64 k = part; k < K; k += RGP) {
        const bool in = k < len;
        ecol[k * pitch + i] = in ? G.c[a + k] : -1;
        eval[k * pitch + i] = in ? G.v[a + k] : (W)0;
    }
}

// Row-length histogram (bins privatised in LDS per workgroup).
__global__ void __launch_bounds__(CB) k_len_hist(i64 nrows, const i32 *rp, i32 *hist) {
    __shared__ i32 hk[HT], hv[HT];
    ht_init(hk, hv);
    for (i64 i = (i64)blockIdx.x * blockDim.x + threadIdx.x; i < nrows; i += (i64)gridDim.x * blockDim.x)
        ht_add(hk, hv, rp[i + 1] - rp[i], hist);
    __syncthreads();
    ht_flush(hk, hv, hist);
}

constexpr unsigned STATS_GRID = 1024;  // workgroups of the grid-stride statistics kernels

static void len_hist(i64 n, const i32 *rp, i32 *hist, hipStream_t s) {
    if (n > 0)
        hipLaunchKernelGGL(k_len_hist, dim3(std::min<unsigned>(grid_for(n, CB), STATS_GRID)), dim3(CB), 0, s, n, rp,
                           hist);
}

// K_h = largest k with #{rows : len >= k} >= need (single thread; maxlen is
// the longest row).
__global__ void k_hyb_width(const i32 *hist, i64 maxlen, i64 need, i32 *out) {
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    i64 ge = 0;
    i64 k = maxlen;
    for (; k > 0; k--) {
        ge += hist[k];
        if (ge >= need) break;
    }
    *out = (i32)k;
}

__global__ void k_overflow_blocks(i64 n, i64 nblk, const i32 *orp, i32 *blk) {
    const i64 b = (i64)blockIdx.x * blockDim.x + threadIdx.x;
    if (b <= nblk) blk[b] = orp[min(b * 256, n)];
}

__global__ void k_overflow_count(i64 nrows, const i32 *rp, i64 K, i32 *cnt) {
    i64 i = (i64)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nrows) return;
    i64 len = rp[i + 1] - rp[i];
    cnt[i] = (i32)(len > K ? len - K : 0);
}

template <class W>
__global__ void k_overflow_fill(i64 nrows, const i32 *rp, const i32 *col, const W *val, i64 K, const i32 *orp,
                                i32 *crow, i32 *ccol, W *cval) {
    i64 i = (i64)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nrows) return;
    i64 o = orp[i];
    for (i64 e = rp[i] + K; e < rp[i + 1]; e++, o++) {
        crow[o] = (i32)i;
        ccol[o] = col[e];
        cval[o] = val[e];
    }
}

// ELL (+ optional COO part with row pointers crp) -> CSR counts and fill.
__global__ void k_ell_rowcount(i64 nrows, i64 K, i64 pitch, const i32 *ecol, const i32 *crp, i32 *cnt) {
    i64 i = (i64)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nrows) return;
    i32 c = 0;
    for (i64 k = 0; k < K; k++) c += ecol[k * pitch + i] >= 0 ? 1 : 0;
    if (crp) c += crp[i + 1] - crp[i];
    cnt[i] = c;
}

// ---------------------------------------------------------------- stats
__global__ void __launch_bounds__(CB) k_row_stats(i64 nrows, const i32 *rp, unsigned long long *acc) {
    // acc: [0] max, [1] min, [2] sum, [3] sumsq, [4] empty, [5..37] histogram
    // of floor(log2(len)) + 1 (0 for empty rows); reduced per workgroup in
    // LDS, then one global atomic per field and workgroup
    __shared__ unsigned long long sh[5];
    __shared__ unsigned hb[33];
    if (threadIdx.x < 5) sh[threadIdx.x] = threadIdx.x == 1 ? ~0ull : 0ull;
    if (threadIdx.x < 33) hb[threadIdx.x] = 0;
    __syncthreads();
    unsigned long long mx = 0, mn = ~0ull, sum = 0, sq = 0, empty = 0;
    for (i64 i = (i64)blockIdx.x * blockDim.x + threadIdx.x; i < nrows; i += (i64)gridDim.x * blockDim.x) {
        const unsigned long long len = (unsigned long long)(rp[i + 1] - rp[i]);
        mx = max(mx, len);
        mn = min(mn, len);
        sum += len;
        sq += len * len;
        empty += len == 0 ? 1 : 0;
        int b = len == 0 ? 0 : 64 - __clzll(len);  // floor(log2(len)) + 1
        if (b > 32) b = 32;
        atomicAdd(&hb[b], 1u);
    }
    atomicMax(&sh[0], mx);
    atomicMin(&sh[1], mn);
    atomicAdd(&sh[2], sum);
    atomicAdd(&sh[3], sq);
    atomicAdd(&sh[4], empty);
    __syncthreads();
    const int t = threadIdx.x;
    if (t == 0) atomicMax(&acc[0], sh[0]);
    else if (t == 1) atomicMin(&acc[1], sh[1]);
    else if (t < 5) {
        if (sh[t]) atomicAdd(&acc[t], sh[t]);
    } else if (t < 38) {
        if (hb[t - 5]) atomicAdd(&acc[t], (unsigned long long)hb[t - 5]);
    }
}

__global__ void k_stats_init(unsigned long long *acc) {
    int t = threadIdx.x;
    if (t < 38) acc[t] = t == 1 ? ~0ull : 0ull;
}

// ================================================================ host side
static void sync(hipStream_t s) { DSM_HIP(hipStreamSynchronize(s)); }

static void check_pad(double slots, double nnz, double ratio, const char *what) {
    if (ratio <= 0) ratio = 16.0;
    if (slots > ratio * std::max(nnz, 1.0))
        fail(DSM_E_INFEASIBLE, std::string(what) + ": " + std::to_string((long long)slots) +
                                   " stored slots exceed max_pad_ratio * nnz");
}

// row lengths of a CSR part -> longest row
static i64 max_row_len(dsm_ctx ctx, i64 nrows, const i32 *rp, hipStream_t s) {
    if (nrows == 0) return 0;
    Tmp len(ctx, sizeof(i32) * (size_t)nrows, s);
    hipLaunchKernelGGL(k_row_len, dim3(grid_for(nrows, CB)), dim3(CB), 0, s, nrows, rp, len.as<i32>());
    DSM_HIP(hipGetLastError());
    return reduce_max_i32(ctx, len.as<i32>(), nrows, s);
}

template <class W>
static void dia_from_csr(dsm_matrix m, const Payload &C, Payload &P, const i32 *flag_true, bool hdc,
                         const dsm_convert_opts &o, hipStream_t s) {
    dsm_ctx ctx = m->ctx;
    const i64 n = m->nrows, nc = m->ncols, span = n + nc - 1;
    Tmp flag(ctx, sizeof(i32) * (size_t)span, s), slot(ctx, sizeof(i32) * (size_t)(span + 1), s);
    const i32 *use_flag = flag_true;
    if (!flag_true) {
        DSM_HIP(hipMemsetAsync(flag.p, 0, sizeof(i32) * (size_t)span, s));
        diag_mark(n, C.rp, C.col, flag.as<i32>(), s);
        DSM_HIP(hipGetLastError());
        use_flag = flag.as<i32>();
    }
    i64 nd = exclusive_scan_i32(ctx, use_flag, slot.as<i32>(), span, s, true);
    P.pitch = pitch_for(n);
    if (!hdc) check_pad((double)nd * (double)n, (double)C.csr_nnz, o.max_pad_ratio, "DIA");
    P.ndiag = nd;
    // offsets padded with zeros to a multiple of 16 entries: the sweep reads
    // them in batches of up to 16 without a bound check
    const i64 offs_len = (std::max<i64>(nd, 1) + 15) / 16 * 16;
    P.offs = (i32 *)P.alloc(ctx, sizeof(i32) * (size_t)offs_len);
    DSM_HIP(hipMemsetAsync(P.offs, 0, sizeof(i32) * (size_t)offs_len, s));
    P.dval = P.alloc(ctx, sizeof(W) * (size_t)std::max<i64>(nd * P.pitch, 1));
    hipLaunchKernelGGL(k_offsets_compact, dim3(grid_for(span, CB)), dim3(CB), 0, s, span, n, use_flag,
                       slot.as<i32>(), P.offs);
    // diagonal clusters for the LDS-staged sweep (host pass over the offsets)
    if (nd > 0) {
        std::vector<i32> ho((size_t)nd);
        DSM_HIP(hipMemcpyAsync(ho.data(), P.offs, sizeof(i32) * (size_t)nd, hipMemcpyDeviceToHost, s));
        sync(s);
        P.reach = std::max(std::abs((i64)ho.front()), std::abs((i64)ho.back()));
        const std::vector<i32> hc = diagonal_clusters(ho, DIA_CLUSTER_K, DIA_CLUSTER_SPAN);
        P.nclu = (i64)hc.size() / CLU_REC;
        P.clu = (i32 *)P.alloc(ctx, sizeof(i32) * hc.size());
        DSM_HIP(hipMemcpyAsync(P.clu, hc.data(), sizeof(i32) * hc.size(), hipMemcpyHostToDevice, s));
        sync(s);  // hc is a host temporary
    }
    if (n > 0 && nd > 0) {
        const int cap = rg_cap(C.csr_nnz, n);
        in_launches(P.pitch / RG, [&](i64 group0, unsigned g) {
            hipLaunchKernelGGL((k_dia_fill<W>), dim3(g), dim3(CB), rg_bytes<W>(cap), s, group0, n, C.rp, C.col,
                               (const W *)C.val, nd, P.offs, P.pitch, (W *)P.dval, cap);
        });
    }
    DSM_HIP(hipGetLastError());
    sync(s);
}

template <class W>
static Payload from_csr_typed(dsm_matrix m, const Payload &C, int fmt, const dsm_convert_opts &o, hipStream_t s) {
    dsm_ctx ctx = m->ctx;
    const i64 n = m->nrows, nc = m->ncols, nnz = C.csr_nnz;
    Payload P;
    P.fmt = fmt;
    P.vdt = C.vdt;
    try {
        switch (fmt) {
        case DSM_COO: {
            P.coo_nnz = nnz;
            P.crow = (i32 *)P.alloc(ctx, sizeof(i32) * (size_t)nnz);
            P.ccol = (i32 *)P.alloc(ctx, sizeof(i32) * (size_t)nnz);
            P.cval = P.alloc(ctx, sizeof(W) * (size_t)nnz);
            if (n > 0)
                hipLaunchKernelGGL(k_csr_expand_rows, dim3(entry_grid(n)), dim3(CB), 0, s, n, C.rp, P.crow);
            DSM_HIP(hipGetLastError());
            DSM_HIP(hipMemcpyAsync(P.ccol, C.col, sizeof(i32) * (size_t)nnz, hipMemcpyDeviceToDevice, s));
            DSM_HIP(hipMemcpyAsync(P.cval, C.val, sizeof(W) * (size_t)nnz, hipMemcpyDeviceToDevice, s));
            sync(s);
            break;
        }
        case DSM_DIA:
            dia_from_csr<W>(m, C, P, nullptr, false, o, s);
            break;
        case DSM_ELL:
        case DSM_HYB: {
            i64 K, longest = -1;
            if (fmt == DSM_ELL) {
                K = max_row_len(ctx, n, C.rp, s);
                check_pad((double)K * (double)n, (double)nnz, o.max_pad_ratio, "ELL");
            } else if (o.hyb_width >= 0) {
                K = o.hyb_width;
            } else {
                i64 mx = max_row_len(ctx, n, C.rp, s);
                longest = mx;
                Tmp hist(ctx, sizeof(i32) * (size_t)(mx + 2), s);
                DSM_HIP(hipMemsetAsync(hist.p, 0, sizeof(i32) * (size_t)(mx + 2), s));
                len_hist(n, C.rp, hist.as<i32>(), s);
                i32 *kout = hist.as<i32>() + mx + 1;
                hipLaunchKernelGGL(k_hyb_width, dim3(1), dim3(64), 0, s, hist.as<i32>(), mx, (n + 2) / 3, kout);
                DSM_HIP(hipGetLastError());
                i32 kh = 0;
                DSM_HIP(hipMemcpyAsync(&kh, kout, sizeof(i32), hipMemcpyDeviceToHost, s));
                sync(s);
                K = n > 0 ? kh : 0;
            }
            P.K = K;
            P.pitch = pitch_for(n);
            P.ecol = (i32 *)P.alloc(ctx, sizeof(i32) * (size_t)(K * P.pitch));
            P.evl = P.alloc(ctx, sizeof(W) * (size_t)(K * P.pitch));
            // every slot, the pitch padding rows included (sentinel columns,
            // so any sweep stays valid)
            if (P.pitch > 0 && K > 0) {
                const int cap = rg_cap(nnz, n);
                in_launches(P.pitch / RG, [&](i64 group0, unsigned g) {
                    hipLaunchKernelGGL((k_ell_fill<W>), dim3(g), dim3(CB), rg_bytes<W>(cap), s, group0, n, P.pitch,
                                       C.rp, C.col, (const W *)C.val, K, P.ecol, (W *)P.evl, cap);
                });
            }
            DSM_HIP(hipGetLastError());
            if (fmt == DSM_HYB) {
                Tmp cnt(ctx, sizeof(i32) * (size_t)std::max<i64>(n, 1), s), orp(ctx, sizeof(i32) * (size_t)(n + 1), s);
                if (n > 0)
                    hipLaunchKernelGGL(k_overflow_count, dim3(grid_for(n, CB)), dim3(CB), 0, s, n, C.rp, K,
                                       cnt.as<i32>());
                i64 nco = exclusive_scan_i32(ctx, cnt.as<i32>(), orp.as<i32>(), n, s, true);
                P.coo_nnz = nco;
                P.crow = (i32 *)P.alloc(ctx, sizeof(i32) * (size_t)nco);
                P.ccol = (i32 *)P.alloc(ctx, sizeof(i32) * (size_t)nco);
                P.cval = P.alloc(ctx, sizeof(W) * (size_t)nco);
                if (n > 0 && nco > 0)
                    hipLaunchKernelGGL((k_overflow_fill<W>), dim3(grid_for(n, CB)), dim3(CB), 0, s, n, C.rp,
                                       C.col, (const W *)C.val, K, orp.as<i32>(), P.crow, P.ccol, (W *)P.cval);
                // (memory that only makes products faster is none of a budget's)
                const i64 nblk = (n + 255) / 256;
                if (n > 0 && nco > 0 && longest >= 0 && !ctx->budget)
                    P.cblk = (i32 *)P.try_alloc(ctx, sizeof(i32) * (size_t)(nblk + 1));
                if (P.cblk) {
                    P.coo_row_max = longest - K;
                    hipLaunchKernelGGL(k_overflow_blocks, dim3(grid_for(nblk + 1, CB)), dim3(CB), 0, s, n, nblk,
                                       orp.as<i32>(), P.cblk);
                }
                DSM_HIP(hipGetLastError());
            }
            sync(s);
            break;
        }
        case DSM_HDC: {
            const i64 span = n + nc - 1;
            double theta = o.hdc_theta > 0 ? o.hdc_theta : 0.5;
            P.theta = theta;
            Tmp cnt(ctx, sizeof(i32) * (size_t)std::max<i64>(span, 1), s),
                flag(ctx, sizeof(i32) * (size_t)std::max<i64>(span, 1), s);
            DSM_HIP(hipMemsetAsync(cnt.p, 0, sizeof(i32) * (size_t)span, s));
            diag_count(n, span, C.rp, C.col, cnt.as<i32>(), s);
            if (span > 0)
                hipLaunchKernelGGL(k_hdc_true, dim3(grid_for(span, CB)), dim3(CB), 0, s, span, n, nc, theta,
                                   cnt.as<i32>(), flag.as<i32>());
            DSM_HIP(hipGetLastError());
            dia_from_csr<W>(m, C, P, flag.as<i32>(), true, o, s);
            // CSR remainder
            Tmp rc(ctx, sizeof(i32) * (size_t)std::max<i64>(n, 1), s);
            P.rp = (i32 *)P.alloc(ctx, sizeof(i32) * (size_t)(n + 1));
            if (n > 0)
                hipLaunchKernelGGL(k_rest_count, dim3(grid_for(n, CB)), dim3(CB), 0, s, n, C.rp, C.col,
                                   flag.as<i32>(), rc.as<i32>());
            i64 nr = exclusive_scan_i32(ctx, rc.as<i32>(), P.rp, n, s, true);
            P.csr_nnz = nr;
            P.col = (i32 *)P.alloc(ctx, sizeof(i32) * (size_t)nr);
            P.val = P.alloc(ctx, sizeof(W) * (size_t)nr);
            if (n > 0 && nr > 0)
                hipLaunchKernelGGL((k_rest_fill<W>), dim3(grid_for(n, CB)), dim3(CB), 0, s, n, C.rp, C.col,
                                   (const W *)C.val, flag.as<i32>(), P.rp, P.col, (W *)P.val);
            DSM_HIP(hipGetLastError());
            build_row_blocks(ctx, P, n, s);
            sync(s);
            break;
        }
        default:
            fail(DSM_E_INVALID, "unknown format");
        }
    } catch (...) {
        (void)hipStreamSynchronize(s);
        P.release(ctx);
        throw;
    }
    return P;
}

Payload from_csr(dsm_matrix m, const Payload &csr, int fmt, int vdt, const dsm_convert_opts &o, hipStream_t s) {
    DSM_CHECK(csr.fmt == DSM_CSR, DSM_E_INVALID, "from_csr needs a CSR payload");
    if (fmt == DSM_CSR) return cast_csr(m, csr, vdt, s);
    Payload casted;
    const Payload *src = &csr;
    if (vdt != csr.vdt) {
        casted = cast_csr(m, csr, vdt, s);
        src = &casted;
    }
    Payload out;
    try {
        DSM_BY_DTYPE(vdt, out = from_csr_typed<W>(m, *src, fmt, o, s));
    } catch (...) {
        if (src == &casted) casted.release(m->ctx);
        throw;
    }
    if (src == &casted) casted.release(m->ctx);
    return out;
}

template <class W>
static Payload to_csr_typed(dsm_matrix m, const Payload &S, hipStream_t s) {
    dsm_ctx ctx = m->ctx;
    const i64 n = m->nrows, nc = m->ncols;
    Payload P;
    P.fmt = DSM_CSR;
    P.vdt = S.vdt;
    try {
        P.rp = (i32 *)P.alloc(ctx, sizeof(i32) * (size_t)(n + 1));
        Tmp cnt(ctx, sizeof(i32) * (size_t)std::max<i64>(n, 1), s);
        i64 nnz = 0;
        switch (S.fmt) {
        case DSM_COO: {
            hipLaunchKernelGGL(k_coo_rowptr, dim3(grid_for(S.coo_nnz + 1, CB)), dim3(CB), 0, s, S.coo_nnz, n, nc,
                               S.crow, S.ccol, P.rp, (int *)nullptr);
            DSM_HIP(hipGetLastError());
            nnz = S.coo_nnz;
            P.col = (i32 *)P.alloc(ctx, sizeof(i32) * (size_t)nnz);
            P.val = P.alloc(ctx, sizeof(W) * (size_t)nnz);
            DSM_HIP(hipMemcpyAsync(P.col, S.ccol, sizeof(i32) * (size_t)nnz, hipMemcpyDeviceToDevice, s));
            DSM_HIP(hipMemcpyAsync(P.val, S.cval, sizeof(W) * (size_t)nnz, hipMemcpyDeviceToDevice, s));
            break;
        }
        case DSM_DIA:
        case DSM_HDC: {
            const i32 *xrp = S.fmt == DSM_HDC ? S.rp : nullptr;
            if (n > 0)
                hipLaunchKernelGGL((k_dia_rowcount<W>), dim3(grid_for(n, CB)), dim3(CB), 0, s, n, nc, S.ndiag,
                                   S.offs, (const W *)S.dval, S.pitch, xrp, cnt.as<i32>());
            DSM_HIP(hipGetLastError());
            nnz = exclusive_scan_i32(ctx, cnt.as<i32>(), P.rp, n, s, true);
            P.col = (i32 *)P.alloc(ctx, sizeof(i32) * (size_t)nnz);
            P.val = P.alloc(ctx, sizeof(W) * (size_t)nnz);
            if (n > 0) {
                const int cap = rg_cap(nnz, n);
                in_launches(grid_for(n, RG), [&](i64 group0, unsigned g) {
                    hipLaunchKernelGGL((k_slots_to_csr<W, DiaSlots<W>, true>), dim3(g), dim3(CB), rg_bytes<W>(cap), s,
                                       group0, n, S.ndiag, DiaSlots<W>{nc, S.offs, (const W *)S.dval, S.pitch}, xrp,
                                       S.col, (const W *)S.val, P.rp, P.col, (W *)P.val, cap);
                });
            }
            DSM_HIP(hipGetLastError());
            break;
        }
        case DSM_ELL:
        case DSM_HYB: {
            Tmp crp(ctx, sizeof(i32) * (size_t)(n + 1), s);
            const i32 *cr = nullptr;
            if (S.fmt == DSM_HYB) {
                hipLaunchKernelGGL(k_coo_rowptr, dim3(grid_for(S.coo_nnz + 1, CB)), dim3(CB), 0, s, S.coo_nnz, n,
                                   nc, S.crow, S.ccol, crp.as<i32>(), (int *)nullptr);
                cr = crp.as<i32>();
            }
            if (n > 0)
                hipLaunchKernelGGL(k_ell_rowcount, dim3(grid_for(n, CB)), dim3(CB), 0, s, n, S.K, S.pitch, S.ecol,
                                   cr, cnt.as<i32>());
            DSM_HIP(hipGetLastError());
            nnz = exclusive_scan_i32(ctx, cnt.as<i32>(), P.rp, n, s, true);
            P.col = (i32 *)P.alloc(ctx, sizeof(i32) * (size_t)nnz);
            P.val = P.alloc(ctx, sizeof(W) * (size_t)nnz);
            if (n > 0) {
                const int cap = rg_cap(nnz, n);
                in_launches(grid_for(n, RG), [&](i64 group0, unsigned g) {
                    hipLaunchKernelGGL((k_slots_to_csr<W, EllSlots<W>, false>), dim3(g), dim3(CB), rg_bytes<W>(cap), s,
                                       group0, n, S.K, EllSlots<W>{S.ecol, (const W *)S.evl, S.pitch}, cr, S.ccol,
                                       (const W *)S.cval, P.rp, P.col, (W *)P.val, cap);
                });
            }
            DSM_HIP(hipGetLastError());
            sync(s);
            break;
        }
        default:
            fail(DSM_E_INVALID, "to_csr: unknown source format");
        }
        P.csr_nnz = nnz;
        build_row_blocks(ctx, P, n, s);
        sync(s);
    } catch (...) {
        (void)hipStreamSynchronize(s);
        P.release(ctx);
        throw;
    }
    return P;
}

Payload to_csr(dsm_matrix m, const Payload &src, hipStream_t s) {
    if (src.fmt == DSM_CSR) return cast_csr(m, src, src.vdt, s);
    Payload out;
    DSM_BY_DTYPE(src.vdt, out = to_csr_typed<W>(m, src, s));
    return out;
}

// ---------------------------------------------------------------- structure features
// Entries whose column lies within `w` of the row (x gathers that stay in a
// cache-sized window around the diagonal).
__global__ void __launch_bounds__(CB) k_near_count(i64 nrows, const i32 *rp, const i32 *col, i64 w,
                                                   unsigned long long *out) {
    __shared__ unsigned long long lds[CB / WAVE];
    unsigned long long c = 0;
    for_each_entry(nrows, rp, [&](i64 r, i64 e) {
        const i64 d = (i64)col[e] - r;
        c += (d <= w && d >= -w) ? 1ull : 0ull;
    });
    c = block_sum(c, lds);
    if (threadIdx.x == 0) atomicAdd(out, c);
}

// Entries on diagonals whose flag is set (HDC's DIA part).
__global__ void k_masked_count(i64 span, const i32 *cnt, const i32 *flag, unsigned long long *out) {
    const i64 d = (i64)blockIdx.x * blockDim.x + threadIdx.x;
    if (d < span && flag[d]) atomicAdd(out, (unsigned long long)cnt[d]);
}

StructFeatures structure_features(dsm_matrix m, const Payload &C, double theta, i64 window, hipStream_t s) {
    DSM_CHECK(C.fmt == DSM_CSR, DSM_E_INVALID, "structure_features needs a CSR payload");
    dsm_ctx ctx = m->ctx;
    const i64 n = m->nrows, nc = m->ncols, span = n + nc - 1;
    StructFeatures F{};
    F.nnz = C.csr_nnz;
    if (n == 0) return F;
    F.max_len = max_row_len(ctx, n, C.rp, s);
    // HYB width from the row-length histogram
    {
        Tmp hist(ctx, sizeof(i32) * (size_t)(F.max_len + 2), s);
        DSM_HIP(hipMemsetAsync(hist.p, 0, sizeof(i32) * (size_t)(F.max_len + 2), s));
        len_hist(n, C.rp, hist.as<i32>(), s);
        i32 *kout = hist.as<i32>() + F.max_len + 1;
        hipLaunchKernelGGL(k_hyb_width, dim3(1), dim3(64), 0, s, hist.as<i32>(), F.max_len, (n + 2) / 3, kout);
        Tmp cnt(ctx, sizeof(i32) * (size_t)n, s), orp(ctx, sizeof(i32) * (size_t)(n + 1), s);
        i32 kh = 0;
        DSM_HIP(hipMemcpyAsync(&kh, kout, sizeof(i32), hipMemcpyDeviceToHost, s));
        DSM_HIP(hipStreamSynchronize(s));
        F.hyb_width = kh;
        hipLaunchKernelGGL(k_overflow_count, dim3(grid_for(n, CB)), dim3(CB), 0, s, n, C.rp, (i64)kh, cnt.as<i32>());
        DSM_HIP(hipGetLastError());
        F.hyb_coo = exclusive_scan_i32(ctx, cnt.as<i32>(), orp.as<i32>(), n, s, true);
    }
    // diagonals: all of them (DIA) and the well-filled ones (HDC)
    {
        Tmp cnt(ctx, sizeof(i32) * (size_t)span, s), flag(ctx, sizeof(i32) * (size_t)span, s),
            acc(ctx, 2 * sizeof(unsigned long long), s);
        DSM_HIP(hipMemsetAsync(cnt.p, 0, sizeof(i32) * (size_t)span, s));
        DSM_HIP(hipMemsetAsync(acc.p, 0, 2 * sizeof(unsigned long long), s));
        diag_count(n, span, C.rp, C.col, cnt.as<i32>(), s);
        hipLaunchKernelGGL(k_hdc_true, dim3(grid_for(span, CB)), dim3(CB), 0, s, span, n, nc, theta, cnt.as<i32>(),
                           flag.as<i32>());
        hipLaunchKernelGGL(k_masked_count, dim3(grid_for(span, CB)), dim3(CB), 0, s, span, cnt.as<i32>(),
                           flag.as<i32>(), acc.as<unsigned long long>());
        hipLaunchKernelGGL(k_near_count, dim3(entry_grid(n)), dim3(CB), 0, s, n, C.rp, C.col, window,
                           acc.as<unsigned long long>() + 1);
        DSM_HIP(hipGetLastError());
        Tmp slot(ctx, sizeof(i32) * (size_t)(span + 1), s);
        F.hdc_ndiag = exclusive_scan_i32(ctx, flag.as<i32>(), slot.as<i32>(), span, s, true);
        // every diagonal with at least one entry: mark then count
        DSM_HIP(hipMemsetAsync(flag.p, 0, sizeof(i32) * (size_t)span, s));
        diag_mark(n, C.rp, C.col, flag.as<i32>(), s);
        F.ndiag = exclusive_scan_i32(ctx, flag.as<i32>(), slot.as<i32>(), span, s, true);
        unsigned long long h[2];
        DSM_HIP(hipMemcpyAsync(h, acc.p, sizeof(h), hipMemcpyDeviceToHost, s));
        DSM_HIP(hipStreamSynchronize(s));
        F.hdc_dia_nnz = (i64)h[0];
        F.near = (i64)h[1];
    }
    return F;
}

// ---------------------------------------------------------------- COO ingest
// Unsorted triplets are split into buckets of consecutive rows with about
// BK_TARGET entries each, and one workgroup brings a bucket into canonical
// order; the result is unique, so the order in which entries reach their
// bucket does not matter.  Every entry is read and written twice, in runs,
// instead of going to its row's end one by one (two random atomics and two
// random stores an entry) and through an insertion sort by a single lane per
// row.  8.1M triplets in random order, 400k rows: kernels 2.70 -> 0.27 ms (split
// 126 us, 195 while a tile loaded columns and values after its counting and all
// tiles asked for their places in the same order; bucket rows 106: 128 MB read
// and written by each).
// Without room for the split copy (16 bytes an entry), and beyond 33M rows,
// the entries go to their rows one by one.
constexpr int BK_T = 1024;              // threads
constexpr int BK_PER = 16;              // entries per thread of a split tile
constexpr i64 BK_TILE = (i64)BK_T * BK_PER;
constexpr int BK_MAX = 4096;            // buckets (LDS counters of a split tile)
constexpr int BK_ROWS_LOG = 13;         // rows of a bucket (LDS counters), at most 2^13
constexpr int BK_RPT = 8;               // entries per thread of a bucket in registers
constexpr i64 BK_CAP = (i64)BK_T * BK_RPT;
constexpr i64 BK_TARGET = BK_CAP / 2;
constexpr int COO_ERR_RANGE = 8, COO_ERR_ORDER = 16, COO_ERR_ROW = 32, COO_UNSORTED = 64;

struct CooRec {
    i32 row, col;
    double val;
};

// entries per bucket (row >> shift); rows out of range are flagged and left out
__global__ void __launch_bounds__(BK_T) k_bucket_count(i64 nnz, i64 nrows, const i32 *row, int shift, int nb, i32 *tot,
                                                       int *err) {
    __shared__ i32 cnt[BK_MAX];
    for (int t = threadIdx.x; t < nb; t += BK_T) cnt[t] = 0;
    __syncthreads();
    const i64 e0 = (i64)blockIdx.x * BK_TILE + threadIdx.x;
    i32 r[BK_PER];
#pragma unroll
    for (int u = 0; u < BK_PER; u++) r[u] = row[min(e0 + (i64)u * BK_T, nnz - 1)];
    bool bad = false;
#pragma unroll
    for (int u = 0; u < BK_PER; u++) {
        if (e0 + (i64)u * BK_T >= nnz) continue;
        if (r[u] < 0 || (i64)r[u] >= nrows) bad = true;
        else atomicAdd(&cnt[r[u] >> shift], 1);
    }
    if (bad) atomicOr(err, COO_ERR_ROW);
    __syncthreads();
    for (int t = threadIdx.x; t < nb; t += BK_T)
        if (cnt[t]) atomicAdd(&tot[t], cnt[t]);
}

// off[0 .. nb] = exclusive prefix of tot, cur = off (one workgroup)
__global__ void __launch_bounds__(BK_T) k_bucket_offsets(int nb, const i32 *tot, i32 *off, i32 *cur) {
    __shared__ i32 lds[BK_T / WAVE];
    constexpr int PER = BK_MAX / BK_T;
    i32 v[PER], sum = 0;
#pragma unroll
    for (int u = 0; u < PER; u++) {
        const int b = threadIdx.x * PER + u;
        v[u] = b < nb ? tot[b] : 0;
        sum += v[u];
    }
    i32 incl = sum;
    const int lane = threadIdx.x % WAVE, w = threadIdx.x / WAVE;
#pragma unroll
    for (int d = 1; d < WAVE; d <<= 1) {
        const i32 t = __shfl_up(incl, d, WAVE);
        incl += lane >= d ? t : 0;
    }
    if (lane == WAVE - 1) lds[w] = incl;
    __syncthreads();
    i32 p = incl - sum;
    for (int i = 0; i < w; i++) p += lds[i];
#pragma unroll
    for (int u = 0; u < PER; u++) {
        const int b = threadIdx.x * PER + u;
        if (b <= nb) off[b] = p;
        if (b < nb) cur[b] = p;
        p += v[u];
    }
    if (nb == BK_MAX && threadIdx.x == BK_T - 1) off[nb] = p;
}

// A tile counts its entries per bucket (an entry's count is its place), takes
// that many places of each bucket at once, and writes its entries there.
__global__ void __launch_bounds__(BK_T) k_bucket_split(i64 nnz, i64 nrows, const i32 *row, const i32 *col,
                                                       const double *val, int shift, int nb, i32 *cur, CooRec *out) {
    __shared__ i32 cnt[BK_MAX];
    for (int t = threadIdx.x; t < nb; t += BK_T) cnt[t] = 0;
    __syncthreads();
    // all of an entry is loaded before the counting, which it overlaps
    const i64 e0 = (i64)blockIdx.x * BK_TILE;
    const int ne = (int)min(nnz - e0, BK_TILE);
    row += e0;
    col += e0;
    val += e0;
    i32 r[BK_PER], at[BK_PER], c[BK_PER];
    double v[BK_PER];
#pragma unroll
    for (int u = 0; u < BK_PER; u++) r[u] = row[(u32)min((int)threadIdx.x + u * BK_T, ne - 1)];
#pragma unroll
    for (int u = 0; u < BK_PER; u++) {
        const u32 e = min((int)threadIdx.x + u * BK_T, ne - 1);
        c[u] = col[e];
        v[u] = val[e];
    }
#pragma unroll
    for (int u = 0; u < BK_PER; u++) {
        const bool in = (int)threadIdx.x + u * BK_T < ne && r[u] >= 0 && (i64)r[u] < nrows;
        if (!in) r[u] = -1;
        at[u] = in ? atomicAdd(&cnt[r[u] >> shift], 1) : 0;
    }
    __syncthreads();
    // (tiles start at different buckets: all of them run at once)
    const int turn = (int)((i64)nb * blockIdx.x / gridDim.x);
    for (int k = threadIdx.x; k < nb; k += BK_T) {
        const int t = k + turn < nb ? k + turn : k + turn - nb;
        const i32 m = cnt[t];
        if (m) cnt[t] = atomicAdd(&cur[t], m);
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < BK_PER; u++)
        if (r[u] >= 0) out[cnt[r[u] >> shift] + at[u]] = CooRec{r[u], c[u], v[u]};
}

// One bucket: row pointers from LDS counts, then each entry to its place in
// its row, the number of smaller columns there (read from LDS).  A bucket of
// more than BK_CAP entries is left grouped by row, unsorted, and flagged.
__global__ void __launch_bounds__(BK_T) k_bucket_rows(i64 nrows, i64 ncols, int shift, int nb, const i32 *off,
                                                      const CooRec *in, i32 *rp, i32 *ocol, double *oval, int *err) {
    __shared__ i32 cnt[(1 << BK_ROWS_LOG) + 1];
    __shared__ i32 cols[BK_CAP];
    __shared__ i32 wsum[BK_T / WAVE];
    const int b = blockIdx.x, nr = (int)min((i64)1 << shift, nrows - ((i64)b << shift));
    const i64 row0 = (i64)b << shift;
    const i64 e0 = off[b];
    const int ne = off[b + 1] - off[b];
    for (int t = threadIdx.x; t < nr; t += BK_T) cnt[t] = 0;
    __syncthreads();
    const bool small = ne <= BK_CAP;
    CooRec r[BK_RPT];
    i32 at[BK_RPT];
    if (small) {
#pragma unroll
        for (int u = 0; u < BK_RPT; u++) {
            const int e = threadIdx.x + u * BK_T;
            if (e < ne) r[u] = in[e0 + e];
        }
#pragma unroll
        for (int u = 0; u < BK_RPT; u++)
            if (threadIdx.x + u * BK_T < ne) at[u] = atomicAdd(&cnt[r[u].row - row0], 1);
    } else {
        for (int e = threadIdx.x; e < ne; e += BK_T) atomicAdd(&cnt[in[e0 + e].row - row0], 1);
    }
    __syncthreads();
    // counts -> starts, each thread a run of rows
    const int per = (nr + BK_T - 1) / BK_T, t0 = min((int)threadIdx.x * per, nr), t1 = min(t0 + per, nr);
    i32 sum = 0;
    for (int t = t0; t < t1; t++) sum += cnt[t];
    i32 incl = sum;
    const int lane = threadIdx.x % WAVE, w = threadIdx.x / WAVE;
#pragma unroll
    for (int d = 1; d < WAVE; d <<= 1) {
        const i32 t = __shfl_up(incl, d, WAVE);
        incl += lane >= d ? t : 0;
    }
    if (lane == WAVE - 1) wsum[w] = incl;
    __syncthreads();
    i32 p = incl - sum;
    for (int i = 0; i < w; i++) p += wsum[i];
    for (int t = t0; t < t1; t++) {
        const i32 c = cnt[t];
        cnt[t] = p;
        rp[row0 + t] = (i32)(e0 + p);
        p += c;
    }
    if (threadIdx.x == 0) {
        cnt[nr] = ne;
        if (b == nb - 1) rp[nrows] = off[nb];
    }
    __syncthreads();
    int bad = 0;
    if (small) {
#pragma unroll
        for (int u = 0; u < BK_RPT; u++)
            if (threadIdx.x + u * BK_T < ne) cols[cnt[r[u].row - row0] + at[u]] = r[u].col;
        __syncthreads();
#pragma unroll
        for (int u = 0; u < BK_RPT; u++)
            if (threadIdx.x + u * BK_T < ne) {
                const i32 c = r[u].col, a = cnt[r[u].row - row0], z = cnt[r[u].row - row0 + 1];
                int rank = 0, same = 0;
                for (int k = a; k < z; k++) {
                    rank += cols[k] < c;
                    same += cols[k] == c;
                }
                if (c < 0 || (i64)c >= ncols) bad |= COO_ERR_RANGE;
                if (same > 1) bad |= COO_ERR_ORDER;
                ocol[e0 + a + rank] = c;
                oval[e0 + a + rank] = r[u].val;
            }
    } else {
        // cnt becomes the rows' cursors
        for (int e = threadIdx.x; e < ne; e += BK_T) {
            const CooRec t = in[e0 + e];
            const int k = atomicAdd(&cnt[t.row - row0], 1);
            ocol[e0 + k] = t.col;
            oval[e0 + k] = t.val;
        }
        if (threadIdx.x == 0) bad = COO_UNSORTED;
    }
    if (bad) atomicOr(err, bad);
}

// entries to their rows one by one (the path without a split copy)
__global__ void k_row_hist(i64 nnz, i64 nrows, const i32 *row, i32 *cnt, int *err) {
    i64 k = (i64)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= nnz) return;
    i32 r = row[k];
    if (r < 0 || (i64)r >= nrows) {
        atomicOr(err, COO_ERR_ROW);
        return;
    }
    atomicAdd(&cnt[r], 1);
}

__global__ void k_row_bucket(i64 nnz, const i32 *row, const i32 *col, const double *val, i32 *cursor, i32 *ocol,
                             double *oval) {
    i64 k = (i64)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= nnz) return;
    i32 p = atomicAdd(&cursor[row[k]], 1);
    ocol[p] = col[k];
    oval[p] = val[k];
}

// Sorts the rows of one row block in place (fewer than 2 * RB_T entries, or
// one row): by counting smaller columns in LDS up to RS_CAP entries, beyond
// that by a bitonic network over memory (every step compares the two ends of
// a pair, smaller index first, so pairs past the end need no padding).
constexpr int RS_T = 256, RS_PER = 16;
constexpr int RS_CAP = RS_T * RS_PER;
static_assert(RS_CAP >= 2 * RB_T, "a row block's entries fit the counting sort");
__global__ void __launch_bounds__(RS_T) k_row_sort(const i32 *blocks, i64 ncols, const i32 *rp, i32 *col, double *val,
                                                   int *err) {
    __shared__ i32 cols[RS_CAP];
    __shared__ i32 srp[RB_RCAP + 1];
    const i64 r0 = blocks[blockIdx.x];
    const int nr = (int)(blocks[blockIdx.x + 1] - r0);
    const i64 e0 = rp[r0];
    const i64 len = rp[r0 + nr] - e0;
    int bad = 0;
    if (len <= RS_CAP) {
        for (int t = threadIdx.x; t <= nr; t += RS_T) srp[t] = (i32)(rp[r0 + t] - e0);
        i32 c[RS_PER];
        double v[RS_PER];
#pragma unroll
        for (int u = 0; u < RS_PER; u++) {
            const int e = threadIdx.x + u * RS_T;
            if (e < len) {
                c[u] = col[e0 + e];
                v[u] = val[e0 + e];
                cols[e] = c[u];
            }
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < RS_PER; u++) {
            const int e = threadIdx.x + u * RS_T;
            if (e >= len) continue;
            int lo = 0, hi = nr;  // srp[lo] <= e < srp[hi]
            while (hi - lo > 1) {
                const int mid = (lo + hi) >> 1;
                if (srp[mid] <= e) lo = mid;
                else hi = mid;
            }
            int rank = 0, same = 0;
            for (int k = srp[lo]; k < srp[lo + 1]; k++) {
                rank += cols[k] < c[u];
                same += cols[k] == c[u];
            }
            if (c[u] < 0 || (i64)c[u] >= ncols) bad |= COO_ERR_RANGE;
            if (same > 1) bad |= COO_ERR_ORDER;
            col[e0 + srp[lo] + rank] = c[u];
            val[e0 + srp[lo] + rank] = v[u];
        }
    } else {
        col += e0;
        val += e0;
        auto order = [&](i64 i, i64 j) {
            if (j >= len) return;
            const i32 a = col[i], b = col[j];
            if (a <= b) return;
            const double x = val[i], y = val[j];
            col[i] = b;
            col[j] = a;
            val[i] = y;
            val[j] = x;
        };
        i64 half = 1;
        while (half < len) half <<= 1;
        half >>= 1;  // pairs of the padded length
        for (i64 k = 1; k <= half; k <<= 1) {
            for (i64 t = threadIdx.x; t < half; t += RS_T) {
                const i64 base = t / k * 2 * k, q = t % k;
                order(base + q, base + 2 * k - 1 - q);
            }
            __syncthreads();
            for (i64 d = k >> 1; d > 0; d >>= 1) {
                for (i64 t = threadIdx.x; t < half; t += RS_T) {
                    const i64 i = t / d * 2 * d + t % d;
                    order(i, i + d);
                }
                __syncthreads();
            }
        }
        for (i64 e = threadIdx.x; e < len; e += RS_T) {
            if (col[e] < 0 || (i64)col[e] >= ncols) bad |= COO_ERR_RANGE;
            if (e > 0 && col[e] == col[e - 1]) bad |= COO_ERR_ORDER;
        }
    }
    if (bad) atomicOr(err, bad);
}

// Row pointers and grouped rows of unsorted triplets, in P's arrays, with
// the device flags in *err; true when no row has been sorted.
static bool coo_group_rows(dsm_matrix m, Payload &P, const i32 *row, const i32 *col, const double *val, i64 nnz,
                           int *err, hipStream_t s) {
    dsm_ctx ctx = m->ctx;
    const i64 n = m->nrows;
    // rows of a bucket: as many (a power of two) as keep it at BK_TARGET
    // entries on average, and enough that there are at most BK_MAX buckets
    int shift = 0;
    while (((n - 1) >> shift) >= BK_MAX || (shift < BK_ROWS_LOG && nnz * ((i64)2 << shift) <= BK_TARGET * n)) shift++;
    if (nnz > 0 && n > 0 && shift <= BK_ROWS_LOG) {
        const int nb = (int)(((n - 1) >> shift) + 1);
        struct Scratch {
            dsm_ctx ctx;
            size_t bytes;
            hipStream_t s;
            void *p = nullptr;
            ~Scratch() { dev_free(ctx, p, bytes, s); }
        } w{ctx, sizeof(CooRec) * (size_t)nnz + sizeof(i32) * (size_t)(3 * nb + 1), s};
        try {
            w.p = dev_alloc(ctx, w.bytes, s);
        } catch (const Error &) {  // no room: one by one
            clear_error();
        }
        if (w.p) {
            CooRec *rec = (CooRec *)w.p;
            i32 *tot = (i32 *)(rec + nnz), *cur = tot + nb, *off = cur + nb;
            const dim3 tiles((unsigned)((nnz + BK_TILE - 1) / BK_TILE));
            DSM_HIP(hipMemsetAsync(tot, 0, sizeof(i32) * (size_t)nb, s));
            hipLaunchKernelGGL(k_bucket_count, tiles, dim3(BK_T), 0, s, nnz, n, row, shift, nb, tot, err);
            hipLaunchKernelGGL(k_bucket_offsets, dim3(1), dim3(BK_T), 0, s, nb, tot, off, cur);
            hipLaunchKernelGGL(k_bucket_split, tiles, dim3(BK_T), 0, s, nnz, n, row, col, val, shift, nb, cur, rec);
            hipLaunchKernelGGL(k_bucket_rows, dim3((unsigned)nb), dim3(BK_T), 0, s, n, m->ncols, shift, nb, off, rec,
                               P.rp, P.col, (double *)P.val, err);
            DSM_HIP(hipGetLastError());
            return false;
        }
    }
    Tmp cnt(ctx, sizeof(i32) * (size_t)std::max<i64>(n, 1), s), cur(ctx, sizeof(i32) * (size_t)(n + 1), s);
    DSM_HIP(hipMemsetAsync(cnt.p, 0, sizeof(i32) * (size_t)std::max<i64>(n, 1), s));
    if (nnz > 0)
        hipLaunchKernelGGL(k_row_hist, dim3(grid_for(nnz, CB)), dim3(CB), 0, s, nnz, n, row, cnt.as<i32>(), err);
    DSM_HIP(hipGetLastError());
    if (read_flag(err, s)) return false;  // rows out of range
    exclusive_scan_i32(ctx, cnt.as<i32>(), P.rp, n, s, false);
    DSM_HIP(hipMemcpyAsync(cur.p, P.rp, sizeof(i32) * (size_t)(n + 1), hipMemcpyDeviceToDevice, s));
    if (nnz > 0) {
        hipLaunchKernelGGL(k_row_bucket, dim3(grid_for(nnz, CB)), dim3(CB), 0, s, nnz, row, col, val, cur.as<i32>(),
                           P.col, (double *)P.val);
    }
    DSM_HIP(hipGetLastError());
    return nnz > 0;
}

Payload coo_to_csr_payload(dsm_matrix m, const i32 *row, const i32 *col, const double *val, i64 nnz, bool sorted,
                           hipStream_t s) {
    dsm_ctx ctx = m->ctx;
    const i64 n = m->nrows, nc = m->ncols;
    Payload P;
    P.fmt = DSM_CSR;
    P.vdt = DSM_F64;
    P.csr_nnz = nnz;
    try {
        P.rp = (i32 *)P.alloc(ctx, sizeof(i32) * (size_t)(n + 1));
        P.col = (i32 *)P.alloc(ctx, sizeof(i32) * (size_t)nnz);
        P.val = P.alloc(ctx, sizeof(double) * (size_t)nnz);
        Tmp err(ctx, sizeof(int), s);
        DSM_HIP(hipMemsetAsync(err.p, 0, sizeof(int), s));
        bool unsorted = false;
        if (sorted) {
            hipLaunchKernelGGL(k_coo_rowptr, dim3(grid_for(nnz + 1, CB)), dim3(CB), 0, s, nnz, n, nc, row, col, P.rp,
                               err.as<int>());
            DSM_HIP(hipGetLastError());
            DSM_HIP(hipMemcpyAsync(P.col, col, sizeof(i32) * (size_t)nnz, hipMemcpyDeviceToDevice, s));
            DSM_HIP(hipMemcpyAsync(P.val, val, sizeof(double) * (size_t)nnz, hipMemcpyDeviceToDevice, s));
        } else {
            unsorted = coo_group_rows(m, P, row, col, val, nnz, err.as<int>(), s);
        }
        auto check = [&](int f) {
            if (f & COO_ERR_ROW) fail(DSM_E_INVALID, "invalid COO: row index out of range");
            if (f & COO_ERR_RANGE) fail(DSM_E_INVALID, "invalid COO: index out of range");
            if (f & COO_ERR_ORDER) fail(DSM_E_INVALID, "invalid COO: unsorted or duplicate (row, col) entries");
        };
        const int f = read_flag(err.as<int>(), s);
        check(f);
        build_row_blocks(ctx, P, n, s);
        if (unsorted || (f & COO_UNSORTED)) {
            hipLaunchKernelGGL(k_row_sort, dim3((unsigned)P.nrblocks), dim3(RS_T), 0, s, P.rblocks, nc, P.rp, P.col,
                               (double *)P.val, err.as<int>());
            DSM_HIP(hipGetLastError());
            check(read_flag(err.as<int>(), s));
        }
    } catch (...) {
        (void)hipStreamSynchronize(s);
        P.release(ctx);
        throw;
    }
    return P;
}

// ---------------------------------------------------------------- stats
bool values_exact(dsm_matrix m, int to, hipStream_t s) {
    const Payload &P = m->P;
    // widening (or keeping) the value type is exact; narrowing order F64, F32, BF16
    if (to <= P.vdt) return true;
    Tmp flag(m->ctx, sizeof(int), s);
    DSM_HIP(hipMemsetAsync(flag.p, 0, sizeof(int), s));
    auto check = [&](const void *v, i64 n) {
        if (!v || n <= 0) return;
        in_launches((n + CB - 1) / CB, [&](i64 first, unsigned g) {
            auto launch = [&](auto kernel, auto *words) {
                hipLaunchKernelGGL(kernel, dim3(g), dim3(CB), 0, s, first, n, words, flag.as<int>());
            };
            if (P.vdt == DSM_F64 && to == DSM_F32) launch(k_values_exact<u64, DSM_F64, DSM_F32>, (const u64 *)v);
            else if (P.vdt == DSM_F64) launch(k_values_exact<u64, DSM_F64, DSM_BF16>, (const u64 *)v);
            else launch(k_values_exact<u32, DSM_F32, DSM_BF16>, (const u32 *)v);
        });
        DSM_HIP(hipGetLastError());
    };
    // every stored value of the active format (padding slots hold +0, exact)
    switch (P.fmt) {
    case DSM_CSR: check(P.val, P.csr_nnz); break;
    case DSM_COO: check(P.cval, P.coo_nnz); break;
    case DSM_DIA: check(P.dval, P.ndiag * P.pitch); break;
    case DSM_ELL: check(P.evl, P.K * P.pitch); break;
    case DSM_HYB: check(P.evl, P.K * P.pitch); check(P.cval, P.coo_nnz); break;
    case DSM_HDC: check(P.dval, P.ndiag * P.pitch); check(P.val, P.csr_nnz); break;
    }
    int h = 0;
    DSM_HIP(hipMemcpyAsync(&h, flag.p, sizeof(int), hipMemcpyDeviceToHost, s));
    DSM_HIP(hipStreamSynchronize(s));
    return h == 0;
}

void row_stats(dsm_matrix m, i64 *out, hipStream_t s) {
    dsm_ctx ctx = m->ctx;
    const i64 n = m->nrows;
    Payload tmp;
    const i32 *rp = nullptr;
    if (m->P.fmt == DSM_CSR) {
        rp = m->P.rp;
    } else {
        tmp = to_csr(m, m->P, s);
        rp = tmp.rp;
    }
    try {
        Tmp acc(ctx, sizeof(unsigned long long) * 38, s);
        hipLaunchKernelGGL(k_stats_init, dim3(1), dim3(64), 0, s, acc.as<unsigned long long>());
        if (n > 0)
            hipLaunchKernelGGL(k_row_stats, dim3(std::min<unsigned>(grid_for(n, CB), STATS_GRID)), dim3(CB), 0, s, n, rp,
                               acc.as<unsigned long long>());
        DSM_HIP(hipGetLastError());
        unsigned long long h[38];
        DSM_HIP(hipMemcpyAsync(h, acc.p, sizeof(h), hipMemcpyDeviceToHost, s));
        sync(s);
        if (n == 0) h[1] = 0;
        for (int i = 0; i < 38; i++) out[i] = (i64)h[i];
    } catch (...) {
        tmp.release(ctx);
        throw;
    }
    tmp.release(ctx);
}

}  // namespace dsm

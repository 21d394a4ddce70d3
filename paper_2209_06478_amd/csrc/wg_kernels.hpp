// Products and sums of one workgroup of BB threads, for the kernels in which a
// workgroup keeps a system, or its share of one, from iteration to iteration.
#pragma once

#include "core.hpp"

namespace dsm {

constexpr int BB = 1024;        // threads of the workgroups below
constexpr int NW = BB / WAVE;   // waves
constexpr int WB = 8;           // CSR entries a lane loads per batch
constexpr int WCH = WB * WAVE;  // entries of one wave's batch (CSR)

// base[lane offset]: a scalar base and a 32-bit byte offset per lane, the
// addressing form that needs no 64-bit address per load.
template <class T>
__device__ __forceinline__ T at_off(const T *base, u32 bytes) {
    return *(const T *)((const char *)base + bytes);
}

__device__ __forceinline__ void wave_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// CSR: each of `parts` waves owns a run of rows with about as many entries and
// streams them WCH at a time, coalesced whatever the row lengths; the
// products go to the wave's LDS buffer, where groups of `lanes` lanes sum
// the rows, and the next batch's loads are in flight meanwhile.  A row cut by
// batch ends is summed batch by batch, in order.
// rp: row pointers of the n rows (rp[0] need not be 0); col, val: the
// matrix's arrays; p[zero] = 0; prod: NW * WCH words of LDS.
struct WaveRows {
    int r, r1, e, e1;  // rows [r, r1) and their entries [e, e1)
};
template <class RPP>
__device__ __forceinline__ WaveRows wave_rows(int n, RPP rp, int parts = NW) {
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
    // first row whose entries end past the target share
    auto row_at = [&](int t) {
        const i64 target = rp[0] + (i64)(rp[n] - rp[0]) * t / parts;
        int lo = 0, hi = n;
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if ((i64)rp[mid] < target) lo = mid + 1;
            else hi = mid;
        }
        return __builtin_amdgcn_readfirstlane(lo);
    };
    WaveRows R;
    R.r = w == 0 ? 0 : w < parts ? row_at(w) : n;
    R.r1 = w >= parts - 1 ? n : row_at(w + 1);
    R.e = __builtin_amdgcn_readfirstlane(rp[R.r]);
    R.e1 = __builtin_amdgcn_readfirstlane(rp[R.r1]);
    return R;
}
template <class X, class V, class PP, class QQ, class RPP>
__device__ __forceinline__ void wg_spmv_csr(const WaveRows &R, int L, const i32 *col, const V *val, PP p, int zero,
                                            QQ q, RPP rp, X *prod_all) {
    const int lane = threadIdx.x % WAVE, w = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
    const int per = WAVE / L;
    X *prod = prod_all + w * WCH;
    int r = R.r, e = R.e;
    const int r1 = R.r1, e1 = R.e1;
    i32 c[2][WB];
    V v[2][WB];
    auto load = [&](int base, i32 (&cc)[WB], V (&vv)[WB]) {
        const i32 *pc = col + base;
        const V *pv = val + base;
        // the last batch loads its last entry again past the end, then drops it
        const int last = e1 - 1 - base;
#pragma unroll
        for (int k = 0; k < WB; k++) {
            const u32 i = (u32)min(lane + k * WAVE, last);
            cc[k] = at_off(pc, i * 4);
            vv[k] = at_off(pv, i * (u32)sizeof(V));
        }
        if (last < WCH - 1) {
#pragma unroll
            for (int k = 0; k < WB; k++) {
                const bool in = lane + k * WAVE <= last;
                cc[k] = in ? cc[k] : zero;
                vv[k] = in ? vv[k] : V{};
            }
        }
    };
    auto step = [&](i32 (&cc)[WB], V (&vv)[WB], i32 (&cn)[WB], V (&vn)[WB]) {
        const int end = batch_end(e, e1, WCH);
        if (end < e1) load(end, cn, vn);
#pragma unroll
        for (int k = 0; k < WB; k++) prod[lane + k * WAVE] = widen<X>(vv[k]) * p[cc[k]];
        wave_fence();
        for (;;) {
            const int row = r + lane / L;
            const int a = row < r1 ? rp[row] : end, z = row < r1 ? rp[row + 1] : end + 1;
            const bool on = row < r1 && (a < end || z <= end);
            // four products in flight per lane (a serial chain of LDS reads was
            // most of a batch's time)
            X s4[4] = {0, 0, 0, 0};
            if (on) {
                int i = max(a, e) - e + lane % L;
                const int hi = min(z, end) - e;
                for (; i + 3 * L < hi; i += 4 * L) {
#pragma unroll
                    for (int t = 0; t < 4; t++) s4[t] += prod[i + t * L];
                }
                for (; i < hi; i += L) s4[0] += prod[i];
            }
            X s = (s4[0] + s4[1]) + (s4[2] + s4[3]);
            for (int off = L >> 1; off > 0; off >>= 1) s += __shfl_xor(s, off, WAVE);
            if (on && lane % L == 0) q[row] = a >= e ? s : q[row] + s;
            const int whole = __popcll(__ballot(on && lane % L == 0 && z <= end));
            r += whole;
            if (whole < per) break;
        }
        wave_fence();
        e = end;
    };
    if (e < e1) load(e, c[0], v[0]);
    while (e < e1) {
        step(c[0], v[0], c[1], v[1]);
        if (e >= e1) break;
        step(c[1], v[1], c[0], v[0]);
    }
    for (int row = r + lane; row < r1; row += WAVE) q[row] = 0;  // no entries left: empty rows
}

// DIA: a lane sweeps the diagonals of U rows, B at a time in ascending order
// (16 loads in flight: 8 of two rows, or 16 of one where the system has no
// more rows than threads); a zero slot is no entry (as in the device-wide
// sweep).  Loads past the last diagonal or
// row group repeat a valid one and are dropped; the rows of a wave past the
// matrix but below the pitch hold padding.  (One row at a time with the next
// batch prefetched measured 10% slower.)
// n rows from row r0 of a matrix of N columns; dval: slot of row r0 on the
// first diagonal; p is indexed by column, p[zero] = 0; q by row - r0.
template <class X, int U, int B, class V, class OP, class PP, class QQ>
__device__ __forceinline__ void wg_spmv_dia(int n, int r0, int N, int nd, i64 pitch, OP offs, const V *dval, PP p,
                                            int zero, QQ q) {
    const int w0 = __builtin_amdgcn_readfirstlane(threadIdx.x & ~(WAVE - 1));
    for (int b0 = 0; b0 + w0 < n; b0 += U * BB) {
        const int i0 = b0 + (int)threadIdx.x;
        const bool both = U == 1 || b0 + w0 + BB < n;  // uniform in the wave
        const int up = both ? BB : 0, wlo = b0 + w0, whi = wlo + (U - 1) * up + WAVE - 1;
        X s[U];
#pragma unroll
        for (int u = 0; u < U; u++) s[u] = 0;
        for (int k0 = 0; k0 < nd; k0 += B) {
            V v[U][B];
            int j[U][B];
#pragma unroll
            for (int k = 0; k < B; k++)
#pragma unroll
                for (int u = 0; u < U; u++)
                    v[u][k] = at_off(dval + min(k0 + k, nd - 1) * pitch + b0 + u * up,
                                     threadIdx.x * (u32)sizeof(V));
            // the offsets are zero-padded to a multiple of 16 entries
            i32 o[B];
#pragma unroll
            for (int k = 0; k < B; k++) o[k] = __builtin_amdgcn_readfirstlane(offs[k0 + k]);
            if (k0 + B <= nd && both && whi < n && r0 + wlo + o[0] >= 0 && r0 + whi + o[B - 1] < N) {
#pragma unroll
                for (int k = 0; k < B; k++)
#pragma unroll
                    for (int u = 0; u < U; u++) j[u][k] = r0 + i0 + u * BB + o[k];
            } else {
#pragma unroll
                for (int k = 0; k < B; k++)
#pragma unroll
                    for (int u = 0; u < U; u++) {
                        const int i = i0 + u * BB, jj = r0 + i + o[k];
                        const bool on = k0 + k < nd && (u == 0 || both);
                        j[u][k] = on && i < n && jj >= 0 && jj < N ? jj : zero;
                        v[u][k] = on ? v[u][k] : V{};
                    }
            }
#pragma unroll
            for (int k = 0; k < B; k++)
#pragma unroll
                for (int u = 0; u < U; u++) {
                    const X pv = p[j[u][k]], wv = widen<X>(v[u][k]);
                    s[u] += wv * (wv != (X)0 ? pv : (X)0);
                }
        }
#pragma unroll
        for (int u = 0; u < U; u++)
            if (i0 + u * BB < n) q[i0 + u * BB] = s[u];
    }
}

// ELL: a lane sweeps the slots of U rows, as above.
// ecol, evl: first slot of the n rows; p[zero] = 0 (the padding column -1 when
// ZERO_BELOW says that p[-1] is that word).
template <class X, int U, int B, bool ZERO_BELOW, class V, class PP, class QQ>
__device__ __forceinline__ void wg_spmv_ell(int n, int K, int pitch, const i32 *ecol, const V *evl, PP p, int zero,
                                            QQ q) {
    const int w0 = __builtin_amdgcn_readfirstlane(threadIdx.x & ~(WAVE - 1));
    for (int b0 = 0; b0 + w0 < n; b0 += U * BB) {
        const int i0 = b0 + (int)threadIdx.x;
        const bool both = U == 1 || b0 + w0 + BB < n;  // uniform in the wave
        const int up = both ? BB : 0;
        X s[U];
#pragma unroll
        for (int u = 0; u < U; u++) s[u] = 0;
        for (int k0 = 0; k0 < K; k0 += B) {
            i32 c[U][B];
            V v[U][B];
#pragma unroll
            for (int k = 0; k < B; k++)
#pragma unroll
                for (int u = 0; u < U; u++) {
                    const i64 at = (i64)min(k0 + k, K - 1) * pitch + b0 + u * up;
                    c[u][k] = at_off(ecol + at, threadIdx.x * 4);
                    v[u][k] = at_off(evl + at, threadIdx.x * (u32)sizeof(V));
                }
            if (k0 + B > K || !both) {
#pragma unroll
                for (int k = 0; k < B; k++)
#pragma unroll
                    for (int u = 0; u < U; u++) {
                        const bool on = k0 + k < K && (u == 0 || both);
                        c[u][k] = on ? c[u][k] : -1;
                        v[u][k] = on ? v[u][k] : V{};
                    }
            }
#pragma unroll
            for (int k = 0; k < B; k++)
#pragma unroll
                for (int u = 0; u < U; u++) {
                    const int j = ZERO_BELOW || c[u][k] >= 0 ? c[u][k] : zero;
                    s[u] += widen<X>(v[u][k]) * p[j];
                }
        }
#pragma unroll
        for (int u = 0; u < U; u++)
            if (i0 + u * BB < n) q[i0 + u * BB] = s[u];
    }
}

// Workgroup sum with one barrier: every wave reduces the waves' sums, kept in
// the half of `lds` (2 * T / WAVE doubles) that the sum before did not use.
// Waves that bring zeros do not change its bits: a sum over fewer threads is
// the same.
template <int T = BB>
struct WgSum {
    static constexpr int WAVES = T / WAVE;
    static_assert(WAVES <= 16 && (WAVES & (WAVES - 1)) == 0, "the waves' sums are a part of one DPP row");
    double *lds;
    int half = 0;
    __device__ __forceinline__ double operator()(double v) {
        v = row_sum(v);
        double *h = lds + (half ^= WAVES);
        if (threadIdx.x % WAVE == 0) h[threadIdx.x / WAVE] = v;
        __syncthreads();
        return lanes_sum<WAVES>(h[threadIdx.x % WAVES]);
    }
    // sum over groups of N lanes of a DPP row, in every lane
    template <int N>
    static __device__ __forceinline__ double lanes_sum(double v) {
        if constexpr (N > 1) v += dpp<0xB1>(v);       // lane ^ 1
        if constexpr (N > 2) v += dpp<0x4E>(v);       // lane ^ 2
        if constexpr (N > 4) v += dpp<0x141>(v);      // the other quad of the half row
        if constexpr (N > 8) v += dpp<0x140>(v);      // the other half row
        return v;
    }
    static __device__ __forceinline__ double row_sum(double v) {
        v = lanes_sum<16>(v);
        return (lane_of(v, 0) + lane_of(v, 16)) + (lane_of(v, 32) + lane_of(v, 48));
    }
    template <int CTRL>
    static __device__ __forceinline__ double dpp(double v) {
        const u64 w = __builtin_bit_cast(u64, v);
        const u32 lo = (u32)__builtin_amdgcn_mov_dpp((int)(u32)w, CTRL, 0xf, 0xf, true);
        const u32 hi = (u32)__builtin_amdgcn_mov_dpp((int)(u32)(w >> 32), CTRL, 0xf, 0xf, true);
        return __builtin_bit_cast(double, (u64)hi << 32 | lo);
    }
    static __device__ __forceinline__ double lane_of(double v, int l) {
        const u64 w = __builtin_bit_cast(u64, v);
        const u32 lo = (u32)__builtin_amdgcn_readlane((int)(u32)w, l);
        const u32 hi = (u32)__builtin_amdgcn_readlane((int)(u32)(w >> 32), l);
        return __builtin_bit_cast(double, (u64)hi << 32 | lo);
    }
};
}  // namespace dsm

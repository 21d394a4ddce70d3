// Device prefix sums and reductions used by the format conversions
// (row pointers, diagonal slot maps, compaction offsets).
//
// Exclusive scan is reduce-then-scan: per-tile totals, a scan of the
// totals (recursively), then a tile-local scan plus the tile's offset.  All
// sums are formed in 64-bit integers, so results are exact and independent
// of the launch shape.
#include "core.hpp"

namespace dsm {

constexpr int SCAN_BLOCK = 256;
constexpr int SCAN_ITEMS = 4;
constexpr int SCAN_ROUNDS = 4;  // of SCAN_BLOCK * SCAN_ITEMS consecutive items
// 4096 items a tile: one level of tile sums up to 16.7M items
constexpr int SCAN_TILE = SCAN_BLOCK * SCAN_ITEMS * SCAN_ROUNDS;
constexpr int SCAN_WAVES = SCAN_BLOCK / WAVE;

template <class T>
__device__ __forceinline__ T wave_incl_scan(T v) {
    const int lane = threadIdx.x % WAVE;
#pragma unroll
    for (int off = 1; off < WAVE; off <<= 1) {
        T t = __shfl_up(v, off, WAVE);
        if (lane >= off) v += t;
    }
    return v;
}

template <class InT>
__global__ void __launch_bounds__(SCAN_BLOCK) k_tile_sums(const InT *in, i64 n, i64 *sums) {
    __shared__ i64 lds[SCAN_WAVES];
    const i64 base = (i64)blockIdx.x * SCAN_TILE + threadIdx.x;
    i64 s = 0;
#pragma unroll
    for (int k = 0; k < SCAN_ITEMS * SCAN_ROUNDS; k++)
        if (base + (i64)k * SCAN_BLOCK < n) s += (i64)in[base + (i64)k * SCAN_BLOCK];
    s = block_sum(s, lds);
    if (threadIdx.x == 0) sums[blockIdx.x] = s;
}

// Each thread scans SCAN_ITEMS items of every round; the rounds' wave totals
// are combined behind one barrier.
template <class InT, class OutT>
__global__ void __launch_bounds__(SCAN_BLOCK) k_tile_scan(const InT *in, OutT *out, i64 n,
                                                          const i64 *tile_off) {
    __shared__ i64 tot[SCAN_ROUNDS][SCAN_WAVES];
    const int lane = threadIdx.x % WAVE, w = threadIdx.x / WAVE;
    const i64 base = (i64)blockIdx.x * SCAN_TILE + (i64)threadIdx.x * SCAN_ITEMS;
    i64 v[SCAN_ROUNDS][SCAN_ITEMS], pre[SCAN_ROUNDS];
#pragma unroll
    for (int r = 0; r < SCAN_ROUNDS; r++)
#pragma unroll
        for (int k = 0; k < SCAN_ITEMS; k++) {
            const i64 i = base + (i64)r * SCAN_BLOCK * SCAN_ITEMS + k;
            v[r][k] = i < n ? (i64)in[i] : 0;
        }
#pragma unroll
    for (int r = 0; r < SCAN_ROUNDS; r++) {
        i64 s = 0;
#pragma unroll
        for (int k = 0; k < SCAN_ITEMS; k++) s += v[r][k];
        const i64 incl = wave_incl_scan(s);
        pre[r] = incl - s;
        if (lane == WAVE - 1) tot[r][w] = incl;
    }
    __syncthreads();
    i64 run = tile_off ? tile_off[blockIdx.x] : 0;
#pragma unroll
    for (int r = 0; r < SCAN_ROUNDS; r++) {
        i64 p = run + pre[r];
#pragma unroll
        for (int i = 0; i < SCAN_WAVES; i++) {
            p += i < w ? tot[r][i] : 0;
            run += tot[r][i];
        }
#pragma unroll
        for (int k = 0; k < SCAN_ITEMS; k++) {
            const i64 i = base + (i64)r * SCAN_BLOCK * SCAN_ITEMS + k;
            if (i < n) out[i] = (OutT)p;
            p += v[r][k];
            // the last element writes the grand total at out[n]
            if (i == n - 1) out[n] = (OutT)p;
        }
    }
}

template <class T>
__global__ void k_store_total(T *out, i64 n) {
    if (threadIdx.x == 0 && blockIdx.x == 0 && n == 0) out[0] = 0;
}

template <class InT, class OutT>
static i64 scan_impl(dsm_ctx ctx, const InT *in, OutT *out, i64 n, hipStream_t s, bool want_total) {
    if (n == 0) {
        hipLaunchKernelGGL(k_store_total<OutT>, dim3(1), dim3(64), 0, s, out, (i64)0);
        DSM_HIP(hipGetLastError());
        return 0;
    }
    i64 ntiles = (n + SCAN_TILE - 1) / SCAN_TILE;
    i64 *offs = nullptr;
    size_t obytes = 0;
    if (ntiles > 1) {
        obytes = sizeof(i64) * (size_t)(2 * ntiles + 1);
        offs = (i64 *)dev_alloc(ctx, obytes, s);
        i64 *sums = offs + ntiles + 1;
        hipLaunchKernelGGL(k_tile_sums<InT>, dim3((unsigned)ntiles), dim3(SCAN_BLOCK), 0, s, in, n, sums);
        DSM_HIP(hipGetLastError());
        try {
            scan_impl<i64, i64>(ctx, sums, offs, ntiles, s, false);
        } catch (...) {
            dev_free(ctx, offs, obytes);
            throw;
        }
    }
    hipLaunchKernelGGL((k_tile_scan<InT, OutT>), dim3((unsigned)ntiles), dim3(SCAN_BLOCK), 0, s, in, out, n,
                       offs);
    DSM_HIP(hipGetLastError());
    i64 total = 0;
    if (want_total) {
        OutT t;
        DSM_HIP(hipMemcpyAsync(&t, out + n, sizeof(OutT), hipMemcpyDeviceToHost, s));
        DSM_HIP(hipStreamSynchronize(s));
        total = (i64)t;
    }
    if (offs) dev_free(ctx, offs, obytes, s);
    return total;
}

i64 exclusive_scan_i32(dsm_ctx ctx, const i32 *in, i32 *out, i64 n, hipStream_t s, bool want_total) {
    return scan_impl<i32, i32>(ctx, in, out, n, s, want_total);
}

i64 exclusive_scan_i64(dsm_ctx ctx, const i64 *in, i64 *out, i64 n, hipStream_t s, bool want_total) {
    return scan_impl<i64, i64>(ctx, in, out, n, s, want_total);
}

__global__ void __launch_bounds__(256) k_reduce_max(const i32 *in, i64 n, i32 *partial) {
    __shared__ i32 lds[256 / WAVE];
    i32 m = INT32_MIN;
    for (i64 i = (i64)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (i64)gridDim.x * blockDim.x)
        m = max(m, in[i]);
#pragma unroll
    for (int off = WAVE / 2; off > 0; off >>= 1) m = max(m, __shfl_xor(m, off, WAVE));
    if (threadIdx.x % WAVE == 0) lds[threadIdx.x / WAVE] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int i = 1; i < 256 / WAVE; i++) m = max(m, lds[i]);
        partial[blockIdx.x] = m;
    }
}

i32 reduce_max_i32(dsm_ctx ctx, const i32 *in, i64 n, hipStream_t s) {
    if (n == 0) return 0;
    unsigned g = (unsigned)std::min<i64>(1024, (n + 255) / 256);
    i32 *part = (i32 *)dev_alloc(ctx, sizeof(i32) * (g + 1), s);
    i32 h = 0;
    try {
        hipLaunchKernelGGL(k_reduce_max, dim3(g), dim3(256), 0, s, in, n, part);
        hipLaunchKernelGGL(k_reduce_max, dim3(1), dim3(256), 0, s, part, (i64)g, part + g);
        DSM_HIP(hipGetLastError());
        DSM_HIP(hipMemcpyAsync(&h, part + g, sizeof(i32), hipMemcpyDeviceToHost, s));
        DSM_HIP(hipStreamSynchronize(s));
    } catch (...) {
        dev_free(ctx, part, sizeof(i32) * (g + 1));
        throw;
    }
    dev_free(ctx, part, sizeof(i32) * (g + 1), s);
    return h;
}

}  // namespace dsm

// Pieces of the init kernels shared by the solver forms: keys and weight range.
#pragma once
#include <hip/hip_runtime.h>
#include <limits.h>

#include "sssp_device.hpp"

namespace {

constexpr int INIT_WG = 256;
constexpr int INIT_MAX_BLOCKS = 1024;

// The longest row of a block, in LDS, 0 where none is longer than the smallest
// row chunk: a thread's share.
constexpr long long NOTED_ROW = 64;
__device__ __forceinline__ void note_row(unsigned* longest, long long deg) {
    if (deg > NOTED_ROW) atomicMax(longest, deg < (long long)UINT_MAX ? (unsigned)deg : UINT_MAX);
}

// Keys of a new solve, in 16-byte stores after a scalar head up to 16-byte
// alignment and with a scalar tail (the caller's array needs only its
// element alignment).
__device__ __forceinline__ void init_keys(long long* key, int n, int src, unsigned shift,
                                          long long tid, long long stride) {
    const long long srckey = pack_key(0, (1u << (shift - 1u)) - 1u, shift);
    const long long head = (((uintptr_t)key & 15u) && n > 0) ? 1 : 0;
    const long long n2 = (n - head) >> 1;
    for (long long v = tid; v < head; v += stride) key[v] = (v == src) ? srckey : KEY_INF;
    longlong2* k2 = (longlong2*)(key + head);
    for (long long i = tid; i < n2; i += stride) {
        const long long v0 = head + 2 * i;
        longlong2 x;
        x.x = (v0 == src) ? srckey : KEY_INF;
        x.y = (v0 + 1 == src) ? srckey : KEY_INF;
        k2[i] = x;
    }
    for (long long v = head + 2 * n2 + tid; v < n; v += stride)
        key[v] = (v == src) ? srckey : KEY_INF;
}

// A thread's share of the weight range, in 16-byte loads (head and tail as
// above).
__device__ __forceinline__ void weight_range(const int* w, long long m, long long tid,
                                             long long stride, int& lo, int& hi) {
    lo = INT_MAX;
    hi = INT_MIN;
    long long wh = (long long)(((16u - ((uintptr_t)w & 15u)) & 15u) >> 2);
    if (wh > m) wh = m;
    const long long m4 = (m - wh) >> 2;
    for (long long e = tid; e < wh; e += stride) {
        const int x = w[e];
        lo = x < lo ? x : lo;
        hi = x > hi ? x : hi;
    }
    const int4* w4 = (const int4*)(w + wh);
    for (long long i = tid; i < m4; i += stride) {
        const int4 x = w4[i];
        const int l01 = x.x < x.y ? x.x : x.y, l23 = x.z < x.w ? x.z : x.w;
        const int h01 = x.x > x.y ? x.x : x.y, h23 = x.z > x.w ? x.z : x.w;
        const int l = l01 < l23 ? l01 : l23, h = h01 > h23 ? h01 : h23;
        lo = l < lo ? l : lo;
        hi = h > hi ? h : hi;
    }
    for (long long e = wh + 4 * m4 + tid; e < m; e += stride) {
        const int x = w[e];
        lo = x < lo ? x : lo;
        hi = x > hi ? x : hi;
    }
}

// The block's weight range into its pair of `wrange` (synchronizes).
__device__ __forceinline__ void block_weight_range(int lo, int hi, int* wrange) {
    for (int off = 32; off > 0; off >>= 1) {
        const int a2 = __shfl_xor(lo, off, 64), b2 = __shfl_xor(hi, off, 64);
        lo = a2 < lo ? a2 : lo;
        hi = b2 > hi ? b2 : hi;
    }
    __shared__ int slo[INIT_WG / 64], shi[INIT_WG / 64];
    if (bq::lane_id() == 0) {
        slo[threadIdx.x >> 6] = lo;
        shi[threadIdx.x >> 6] = hi;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int i = 1; i < INIT_WG / 64; ++i) {
            lo = slo[i] < lo ? slo[i] : lo;
            hi = shi[i] > hi ? shi[i] : hi;
        }
        wrange[2 * blockIdx.x] = lo;
        wrange[2 * blockIdx.x + 1] = hi;
    }
}

}  // namespace

// Wavefront (64 lanes) and workgroup primitives for gfx950.
#pragma once

#include "internal.h"

namespace spg {

// Device memory named through a pointer read from memory (a problem's arrays)
// is reached with flat instructions unless the type says it is global. Flat
// loads and stores also count against the LDS wait counter, so every LDS read
// after them waits for them to complete; through a gmem pointer they are
// global memory instructions, and LDS work overlaps the gathers in flight.
template <typename T>
using gmem = __attribute__((address_space(1))) T;

template <typename T>
__device__ __forceinline__ gmem<T> *to_gmem(T *p) {
    return (gmem<T> *)p;
}

// two consecutive ints at 4-byte alignment (a column pointer and the next one)
typedef int int2a __attribute__((ext_vector_type(2), aligned(4)));

// p[i] and p[i + 1] in one 8-byte load; the caller keeps i + 1 inside the array
__device__ __forceinline__ int2a load_pair(const int32_t *p, long long i) {
    return *(const gmem<const int2a> *)((const gmem<const int32_t> *)p + i);
}

__device__ __forceinline__ int lane_id() {
    return __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
}

__device__ __forceinline__ unsigned long long ballot(bool p) {
    return __builtin_amdgcn_ballot_w64(p);
}

// lanes below this one
__device__ __forceinline__ unsigned long long mask_lt() {
    int l = lane_id();
    return l == 0 ? 0ull : (~0ull >> (64 - l));
}

__device__ __forceinline__ int popc64(unsigned long long x) { return __builtin_popcountll(x); }

// value of lane `src` (any lane pattern) through the LDS crossbar
__device__ __forceinline__ int shfl_idx(int v, int src) {
    return __builtin_amdgcn_ds_bpermute(src << 2, v);
}

// Exchange inside the wavefront with the lane whose number differs in the bits
// of M. 1, 2 and 3 stay in a quad (DPP quad_perm), 7 and 15 mirror half a row
// and a row, 8 rotates a row by 8 lanes (all DPP); 4, 16 and 31 use
// ds_swizzle's bit-mask mode inside 32-lane halves, 32 and 63 cross halves
// through ds_bpermute.
template <int M>
__device__ __forceinline__ int shfl_xor_c(int v) {
    static_assert(M == 1 || M == 2 || M == 3 || M == 4 || M == 7 || M == 8 || M == 15 || M == 16 ||
                      M == 31 || M == 32 || M == 63, "exchange masks in use");
    if constexpr (M == 1) return __builtin_amdgcn_mov_dpp(v, 0xB1, 0xF, 0xF, true);
    else if constexpr (M == 2) return __builtin_amdgcn_mov_dpp(v, 0x4E, 0xF, 0xF, true);
    else if constexpr (M == 3) return __builtin_amdgcn_mov_dpp(v, 0x1B, 0xF, 0xF, true);
    else if constexpr (M == 7) return __builtin_amdgcn_mov_dpp(v, 0x141, 0xF, 0xF, true);
    else if constexpr (M == 8) return __builtin_amdgcn_mov_dpp(v, 0x128, 0xF, 0xF, true);
    else if constexpr (M == 15) return __builtin_amdgcn_mov_dpp(v, 0x140, 0xF, 0xF, true);
    else if constexpr (M < 32)
        // bit-mask mode: and_mask = 0x1f, or_mask = 0, xor_mask = M
        return __builtin_amdgcn_ds_swizzle(v, (M << 10) | 0x1F);
    else return __builtin_amdgcn_ds_bpermute((lane_id() ^ M) << 2, v);
}

template <int J>
__device__ __forceinline__ unsigned long long shfl_xor_c64(unsigned long long v) {
    int lo = (int)(unsigned)v, hi = (int)(unsigned)(v >> 32);
    lo = shfl_xor_c<J>(lo);
    hi = shfl_xor_c<J>(hi);
    return ((unsigned long long)(unsigned)hi << 32) | (unsigned)lo;
}

// value of the lane below / above (lane 0 / lane 63: `edge`), one DPP move
__device__ __forceinline__ int wave_shr1(int v, int edge) {
    return __builtin_amdgcn_update_dpp(edge, v, 0x138, 0xF, 0xF, false);
}
__device__ __forceinline__ int wave_shl1(int v, int edge) {
    return __builtin_amdgcn_update_dpp(edge, v, 0x130, 0xF, 0xF, false);
}
__device__ __forceinline__ double wave_shr1_v(double v) {
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    const int lo = wave_shr1((int)(unsigned)b, 0), hi = wave_shr1((int)(unsigned)(b >> 32), 0);
    return __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
}
__device__ __forceinline__ float wave_shr1_v(float v) {
    return __int_as_float(wave_shr1(__float_as_int(v), 0));
}

// Inclusive prefix sum and maximum over the wavefront: four DPP row shifts
// scan every row of 16 lanes, two row broadcasts carry the rows on. (A scan by
// LDS permutes waits on the LDS six times.)
__device__ __forceinline__ int wave_incl_scan(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);
    return v;
}
__device__ __forceinline__ int wave_incl_max(int v) {
    v = max(v, __builtin_amdgcn_update_dpp(v, v, 0x111, 0xF, 0xF, false));
    v = max(v, __builtin_amdgcn_update_dpp(v, v, 0x112, 0xF, 0xF, false));
    v = max(v, __builtin_amdgcn_update_dpp(v, v, 0x114, 0xF, 0xF, false));
    v = max(v, __builtin_amdgcn_update_dpp(v, v, 0x118, 0xF, 0xF, false));
    v = max(v, __builtin_amdgcn_update_dpp(v, v, 0x142, 0xA, 0xF, false));
    v = max(v, __builtin_amdgcn_update_dpp(v, v, 0x143, 0xC, 0xF, false));
    return v;
}

// 64-bit prefix sum (values and sums of 0 .. 2^63 - 1) over the wavefront, and
// its last value: three scans of 21-bit pieces, whose sums stay below 2^27
__device__ __forceinline__ long long wave_incl_scan64(long long v) {
    constexpr int B = 21, M = (1 << B) - 1;
    const long long a = wave_incl_scan((int)v & M), b = wave_incl_scan((int)(v >> B) & M),
                    c = wave_incl_scan((int)(v >> (2 * B)) & M);
    return a + (b << B) + (c << (2 * B));
}
__device__ __forceinline__ long long wave_last64(long long v) {
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)v, 63);
    const unsigned hi =
        (unsigned)__builtin_amdgcn_readlane((int)(unsigned)((unsigned long long)v >> 32), 63);
    return (long long)(((unsigned long long)hi << 32) | lo);
}
__device__ __forceinline__ long long wave_sum64(long long v) {
    return wave_last64(wave_incl_scan64(v));
}

// the sum over the wavefront, in every lane
__device__ __forceinline__ int wave_sum(int v) {
    return __builtin_amdgcn_readlane(wave_incl_scan(v), 63);
}

// Exclusive prefix sum over a workgroup of kBlock threads. `tmp` holds
// kBlock / 64 + 1 ints of LDS. Returns the exclusive prefix; `total` gets the
// workgroup sum. Contains barriers: every thread must call it.
__device__ __forceinline__ int block_excl_scan(int v, int *tmp, int &total) {
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
    int inc = wave_incl_scan(v);
    if (l == 63) tmp[w] = inc;
    __syncthreads();
    if (threadIdx.x == 0) {
        int run = 0;
        for (int i = 0; i < kBlock / 64; ++i) {
            int x = tmp[i];
            tmp[i] = run;
            run += x;
        }
        tmp[kBlock / 64] = run;
    }
    __syncthreads();
    int ex = tmp[w] + inc - v;
    total = tmp[kBlock / 64];
    __syncthreads();
    return ex;
}

// Exclusive prefix over a workgroup of T threads; `tmp` holds T / 64 + 1 ints
// of LDS; `total` gets the workgroup sum. Contains barriers: every thread must
// call it.
template <int T>
__device__ __forceinline__ int wg_excl_scan(int v, int *tmp, int &total) {
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
    int inc = wave_incl_scan(v);
    if (l == 63) tmp[w] = inc;
    __syncthreads();
    if (threadIdx.x == 0) {
        int run = 0;
        for (int i = 0; i < T / 64; ++i) {
            int x = tmp[i];
            tmp[i] = run;
            run += x;
        }
        tmp[T / 64] = run;
    }
    __syncthreads();
    int ex = tmp[w] + inc - v;
    total = tmp[T / 64];
    __syncthreads();
    return ex;
}

// the same for 64-bit values (`tmp` holds T / 64 + 1 of them)
template <int T>
__device__ __forceinline__ long long wg_excl_scan64(long long v, long long *tmp, long long &total) {
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
    const long long inc = wave_incl_scan64(v);
    if (l == 63) tmp[w] = inc;
    __syncthreads();
    if (threadIdx.x == 0) {
        long long run = 0;
        for (int i = 0; i < T / 64; ++i) {
            const long long x = tmp[i];
            tmp[i] = run;
            run += x;
        }
        tmp[T / 64] = run;
    }
    __syncthreads();
    const long long ex = tmp[w] + inc - v;
    total = tmp[T / 64];
    __syncthreads();
    return ex;
}

// Largest index i in [0, n) with a[i] <= x, for non-decreasing a with a[0] <= x.
__device__ __forceinline__ int last_le(const int *a, int n, int x) {
    int lo = 0, hi = n;
    while (hi - lo > 1) {
        int mid = (lo + hi) >> 1;
        if (a[mid] <= x) lo = mid;
        else hi = mid;
    }
    return lo;
}

__device__ __forceinline__ int ceil_log2(int x) {  // x >= 1
    return x <= 1 ? 0 : 32 - __builtin_clz((unsigned)(x - 1));
}

}  // namespace spg

// Single-launch scans with decoupled look-back (Merrill and Garland, "Single-pass Parallel Prefix Scan
// with Decoupled Look-back", 2016): a workgroup takes the next tile by a ticket, sums it, publishes the sum and
// adds up the sums of the tiles before it (wavefront 0, 64 tiles at a look) until it meets one that
// has published its inclusive sum.  It only ever waits for tiles whose tickets were drawn before its
// own, so their workgroups are running and every wait ends.  A tile's word holds its state and its sum
// together, so no other ordering is needed.  (The three launches of a reduce-then-scan cost a small
// graph more than the work: a build of 2,000 nodes took seven scans, 21 of its 47 launches.)
// Workgroups have kScanThreads threads unless said otherwise; the words are zero before the launch.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace scan {

constexpr uint32_t kScanThreads = 256;

struct Look {
    uint32_t* ticket;
    unsigned long long* tile;  // state << 62 | sum; 0: nothing yet
};
constexpr unsigned long long kTileSum = 1ull << 62, kTileIncl = 2ull << 62, kTileMask = kTileSum - 1;

__device__ __forceinline__ uint32_t look_ticket(const Look& L) {
    __shared__ uint32_t t;
    __syncthreads();
    if (threadIdx.x == 0) t = atomicAdd(L.ticket, 1u);
    __syncthreads();
    return t;
}

// the sum of all tiles before `t`, given this tile's sum (T: uint32_t, or uint64_t for sums below 2^62)
template <typename T>
__device__ T look_back(const Look& L, uint32_t t, T sum) {
    __shared__ T before;
    const int lane = threadIdx.x & 63;
    if (threadIdx.x < 64) {
        if (lane == 0 && t)
            __hip_atomic_store(&L.tile[t], kTileSum | sum, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        T acc = 0;
        for (int64_t at = (int64_t)t - 1; at >= 0;) {
            const int64_t i = at - lane;
            const unsigned long long w =
                i >= 0 ? __hip_atomic_load(&L.tile[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : kTileIncl;
            const unsigned long long incl = __ballot(w >= kTileIncl), none = __ballot(w < kTileSum);
            const int first = incl ? __builtin_ctzll(incl) : 63;  // the lanes 0 .. first are added up
            if (none & (~0ull >> (63 - first))) {
                __builtin_amdgcn_s_sleep(1);
                continue;
            }
            T v = lane <= first ? (T)(w & kTileMask) : (T)0;
#pragma unroll
            for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
            acc += v;
            if (incl) break;
            at -= 64;
        }
        if (lane == 0) {
            __hip_atomic_store(&L.tile[t], kTileIncl | (T)(acc + sum), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            before = acc;
        }
    }
    __syncthreads();
    return before;
}

// exclusive scan over a workgroup of THREADS threads; `total` in every thread
template <typename T, uint32_t THREADS = kScanThreads>
__device__ __forceinline__ T block_excl_scan(T v, T& total) {
    __shared__ T ws[THREADS / 64];
    const uint32_t lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    T inc = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const T o = __shfl_up(inc, d, 64);
        if ((int)lane >= d) inc += o;
    }
    if (lane == 63) ws[w] = inc;
    __syncthreads();
    T base = 0, tot = 0;
#pragma unroll
    for (uint32_t i = 0; i < THREADS / 64; ++i) {
        if (i < w) base += ws[i];
        tot += ws[i];
    }
    __syncthreads();
    total = tot;
    return base + inc - v;
}

}  // namespace scan

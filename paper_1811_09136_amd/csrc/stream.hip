// Incremental streaming (Section II: the stream arrives over time; REPT's sets are built on the
// fly): the stream is taken in chunks, and after every chunk the counters hold Algorithm 1's
// updates of every edge seen so far.
//
// State on the device: the whole adjacency of the edges seen so far, both directions, as one
// array of keys (x << 32 | y) sorted by (x, y) with the arrival time of each edge beside it,
// and the node offsets into it.  An append:
//   1. turns the chunk into keys (both directions, times T .. T+W-1), checks ids and self-loops,
//      copies the edges to the stream in arrival order, and sorts the keys: a small chunk by
//      comparing every pair of keys, others by a stable LSD radix sort over the id bits;
//   2. finds each node's run in the sorted chunk, which gives the merged offsets (in a second array);
//   3. merges the chunk into the other copy of the adjacency: every old and every new entry computes
//      its merged position by one binary search in the other side's run of the same node, so the
//      merge is one pass.  A new entry's search also shows whether its pair is there already; its
//      neighbour in the sorted chunk, whether the pair is in the chunk twice;
//   4. scans the chunk's work items (below).  The host then reads the validation word and the number
//      of items together (the one synchronisation) and, if the chunk is valid, takes the merged copy
//      and offsets as the current ones.  A refused chunk has written nothing that is read again;
//   5. counts the chunk's edges: for the edge (u, v) at time t, the entries w of the shorter of
//      the two lists that arrived before t are searched in the other list (arrived before t as
//      well); each common neighbour is a triangle whose last edge is (u, v), and every group
//      whose hash puts {u, w} and {v, w} in the same active slot adds it to that processor's
//      counters (Algorithm 1's UpdateTriangleCNT).  The work is one item per (edge, entry of
//      its shorter list), spread evenly over the grid through an inclusive scan of the lengths.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "common.h"
#include "edge_hash.h"
#include "scan.h"

namespace {

constexpr uint32_t kThreads = 256;
constexpr uint32_t kHist = 1024;  // processors aggregated in LDS by the counting kernel

__device__ __forceinline__ uint32_t hi32(uint64_t k) { return (uint32_t)(k >> 32); }
__device__ __forceinline__ uint32_t lo32(uint64_t k) { return (uint32_t)k; }

// orders a wavefront's LDS accesses
__device__ __forceinline__ void wave_fence() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// first index in [lo, hi) with key >= x (keys sorted ascending)
__device__ __forceinline__ uint64_t lower_bound64(const uint64_t* __restrict__ k, uint64_t lo, uint64_t hi,
                                                  uint64_t x) {
    while (lo < hi) {
        const uint64_t mid = (lo + hi) >> 1;
        if (k[mid] < x) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

__device__ __forceinline__ uint32_t edge_flags(uint2& e, uint32_t n) {
    if (e.x >= n || e.y >= n) {  // replaced by node 0: every later index stays in range (the append is refused)
        e = make_uint2(0u, 0u);
        return RF_RANGE;
    }
    return e.x == e.y ? (uint32_t)RF_SELFLOOP : 0u;
}
__device__ __forceinline__ uint64_t edge_key(uint2 e, bool rev) {
    return rev ? ((uint64_t)e.y << 32) | e.x : ((uint64_t)e.x << 32) | e.y;
}

// 1a. A small chunk's sort, one launch: a key's position is the number of keys below it, equal keys in
// order of arrival.  A workgroup takes 64 entries, one per lane; its wavefronts share the chunk's
// edges, whose keys they make from scalar loads.  Bound by the compares, (2W)^2 of them over all SIMDs.
// 1,000 edges: 11 us (the radix sort's 20 launches, four digits of 8 bits: 120 us).
constexpr uint32_t kRankThreads = 1024, kRankWaves = kRankThreads / 64;
__global__ void __launch_bounds__(kRankThreads) k_inc_rank(const uint2* __restrict__ edges, IncChunk a) {
    __shared__ uint32_t below[kRankWaves][64];
    const uint32_t lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const uint32_t W = (uint32_t)a.W, i0 = blockIdx.x * 64, i = i0 + lane;
    for (uint32_t k = blockIdx.x * kRankThreads + threadIdx.x; k < a.look_words; k += gridDim.x * kRankThreads)
        a.look[k] = 0ull;
    uint32_t f = 0;
    uint2 own = edges[(i >> 1) < W ? i >> 1 : W - 1];
    if (w == 0 && i < 2 * W) {
        if (!(i & 1u)) a.eall[i >> 1] = own;
        f = edge_flags(own, a.n);
    } else {
        (void)edge_flags(own, a.n);
    }
    const uint64_t key = edge_key(own, i & 1u);
    const uint32_t share = (W + kRankWaves - 1) / kRankWaves;
    const uint32_t e0 = __builtin_amdgcn_readfirstlane(w * share < W ? w * share : W);
    const uint32_t e1 = W - e0 < share ? W : e0 + share;
    const uint32_t o0 = i0 >> 1, o1 = o0 + 32;  // the workgroup's own edges
    uint32_t lt = 0;
    const uint32_t b1 = e1 < o0 ? e1 : o0;
#pragma unroll 8
    for (uint32_t j = e0; j < b1; ++j) {  // arrived before: equal keys count
        uint2 e = edges[j];
        (void)edge_flags(e, a.n);
        lt += edge_key(e, false) <= key;
        lt += edge_key(e, true) <= key;
    }
    const uint32_t m0 = e0 > o0 ? e0 : o0, m1 = e1 < o1 ? e1 : o1;
    for (uint32_t j = m0; j < m1; ++j) {
        uint2 e = edges[j];
        (void)edge_flags(e, a.n);
        const uint64_t k0 = edge_key(e, false), k1 = edge_key(e, true);
        lt += k0 < key || (k0 == key && 2 * j < i);
        lt += k1 < key || (k1 == key && 2 * j + 1 < i);
    }
    const uint32_t a0 = e0 > o1 ? e0 : o1;
#pragma unroll 8
    for (uint32_t j = a0; j < e1; ++j) {
        uint2 e = edges[j];
        (void)edge_flags(e, a.n);
        lt += edge_key(e, false) < key;
        lt += edge_key(e, true) < key;
    }
    below[w][lane] = lt;
    __syncthreads();
    if (w == 0 && i < 2 * W) {
        uint32_t at = 0;
#pragma unroll
        for (uint32_t v = 0; v < kRankWaves; ++v) at += below[v][lane];
        a.ckey[at] = key;
        a.ctim[at] = a.T + (i >> 1);
    }
    if (f) atomicOr(a.flags, f);
}

// 2. noff[x] = off[x] + the first chunk position with node >= x, for x in [0, n]
__global__ void __launch_bounds__(kThreads) k_inc_noff(const uint64_t* __restrict__ ck, uint64_t N2, uint32_t n,
                                                       const uint32_t* __restrict__ off, uint32_t* __restrict__ noff) {
    for (uint64_t x = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; x <= n; x += (uint64_t)gridDim.x * blockDim.x)
        noff[x] = off[x] + (uint32_t)lower_bound64(ck, 0, N2, x << 32);
}

// 3. Entries [0, N) are the old ones: an entry moves up by the number of chunk entries of its node
// with a smaller key.  Entries [N, N + N2) are the chunk's, which land after the old entries of their
// node with a smaller key; a pair twice in the chunk or already in the adjacency is flagged.
__global__ void __launch_bounds__(kThreads) k_inc_merge(const uint64_t* __restrict__ akey,
                                                        const uint32_t* __restrict__ atim, uint64_t N,
                                                        const uint64_t* __restrict__ ck,
                                                        const uint32_t* __restrict__ ct, uint64_t N2,
                                                        const uint32_t* __restrict__ off,
                                                        const uint32_t* __restrict__ noff, uint64_t* __restrict__ okey,
                                                        uint32_t* __restrict__ otim, uint32_t* __restrict__ flags) {
    uint32_t f = 0;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < N + N2;
         i += (uint64_t)gridDim.x * blockDim.x) {
        if (i < N) {
            const uint64_t k = akey[i];
            const uint32_t x = hi32(k), c0 = noff[x] - off[x], c1 = noff[x + 1] - off[x + 1];
            // off[x] + c0 + (i - off[x]) + (chunk entries of x with a smaller key)
            const uint64_t q = i + lower_bound64(ck, c0, c1, k);
            okey[q] = k;
            otim[q] = atim[i];
        } else {
            const uint64_t p = i - N, k = ck[p];
            const uint32_t x = hi32(k);
            const uint64_t e = off[x + 1], r = lower_bound64(akey, off[x], e, k);
            if ((p && ck[p - 1] == k) || (r < e && akey[r] == k)) f |= RF_DUP;
            okey[p + r] = k;  // off[x] + c0 + (p - c0) + (r - off[x])
            otim[p + r] = ct[p];
        }
    }
    if (f) atomicOr(flags, f);
}

// 4. end[p] = items of the chunk entries 0 .. p: the shorter list's length for the entry (u, v) with
// u < v (each chunk edge once), 0 for the other direction
constexpr uint32_t kItems = 8, kItemTile = kThreads * kItems;
static_assert(kThreads == scan::kScanThreads, "workgroups of the scans");
__global__ void __launch_bounds__(kThreads) k_inc_items(const uint64_t* __restrict__ ck, uint64_t N2,
                                                        const uint32_t* __restrict__ noff, uint64_t* __restrict__ end,
                                                        uint64_t* __restrict__ total, scan::Look L) {
    const uint32_t t = scan::look_ticket(L);
    const uint64_t b0 = (uint64_t)t * kItemTile + (uint64_t)threadIdx.x * kItems;
    uint32_t len[kItems];
    uint64_t sum = 0;
#pragma unroll
    for (uint32_t r = 0; r < kItems; ++r) {
        const uint64_t k = b0 + r < N2 ? ck[b0 + r] : 0ull;
        const uint32_t u = hi32(k), v = lo32(k);
        len[r] = 0;
        if (u < v) {
            const uint32_t du = noff[u + 1] - noff[u], dv = noff[v + 1] - noff[v];
            len[r] = du < dv ? du : dv;
        }
        sum += len[r];
    }
    uint64_t tot;
    uint64_t run = scan::block_excl_scan<uint64_t>(sum, tot);
    run += scan::look_back<uint64_t>(L, t, tot);
#pragma unroll
    for (uint32_t r = 0; r < kItems; ++r) {
        run += len[r];
        if (b0 + r < N2) end[b0 + r] = run;
    }
    if (t == gridDim.x - 1 && threadIdx.x == kThreads - 1) *total = run;
}

// first p in [lo, hi) with end[p] > i (end ascending)
__device__ __forceinline__ uint64_t upper_item(const uint64_t* __restrict__ end, uint64_t lo, uint64_t hi, uint64_t i) {
    while (lo < hi) {
        const uint64_t mid = (lo + hi) >> 1;
        if (end[mid] <= i) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

// the same by a wavefront: 64 places tried at a time
__device__ __forceinline__ uint64_t wave_upper_item(const uint64_t* __restrict__ end, uint64_t lo, uint64_t hi,
                                                    uint64_t i) {
    const uint32_t lane = threadIdx.x & 63;
    while (hi - lo > 64) {
        const uint64_t step = (hi - lo + 63) / 64, q = lo + (lane + 1) * step - 1;
        lo += (uint64_t)__popcll(__ballot(q < hi && end[q] <= i)) * step;
        hi = hi < lo + step ? hi : lo + step;
    }
    return lo + (uint64_t)__popcll(__ballot(lo + lane < hi && end[lo + lane] <= i));
}

// 5. the count: item i belongs to the chunk entry p with end[p - 1] <= i < end[p].  A workgroup
// takes a run of consecutive items; the slice of `end` they fall in is staged in LDS when it is
// short enough (entries without items, the reverse direction of each edge, also sit in it),
// so that each item finds its entry there.
//   The counters' atomics would set the time: all triangles of an edge add to its two nodes, and the
// third nodes of many edges are the same few large ones, while the memory side takes one atomic per
// 64-byte line and 12 ns.  So a wavefront, whose items are consecutive, queues its triangles and takes
// them 64 at a time, adds up each edge's and each first node's, and a workgroup collects its additions
// in LDS, in a table that keeps the first node to come to an entry (large nodes come first) and is
// written out at the end; an addition that finds its entry taken goes to memory.  The rest is waiting
// for the searches: eight wavefronts per SIMD (64 VGPRs, 40 KB of LDS for eight) hide it better than
// five, a few spilled registers included.  An append of 200k edges to 1.8M (26M items), all of it:
// 2,890 us with an atomic per addition, 1,353 with the sums, 1,121 with the queues, 903 with 16-bit
// ends and 64 registers, 877 with searches of the keys' low words alone.
constexpr uint32_t kRun = 4096;       // items per workgroup run, at most
constexpr uint32_t kCountThreads = 512;
constexpr uint32_t kStage = 2048;     // entries of `end` staged per run, at most
constexpr uint32_t kNodeBits = 11;    // the table of additions has 2^11 entries
constexpr uint32_t kNoNode = 0xffffffffu;

struct NodeSums {
    uint32_t key[1u << kNodeBits], sum[1u << kNodeBits];
};
// add c to local[k] (kept: k is below kNoNode for every counter)
__device__ __forceinline__ void node_add(NodeSums& T, bool kept, int64_t* local, uint64_t k, uint32_t c) {
    if (kept) {
        const uint32_t key = (uint32_t)k, s = (key * 0x9E3779B1u) >> (32 - kNodeBits);
        uint32_t have = *(volatile uint32_t*)&T.key[s];
        if (have == kNoNode) have = atomicCAS(&T.key[s], kNoNode, key);
        if (have == kNoNode || have == key) {
            atomicAdd(&T.sum[s], c);
            return;
        }
    }
    atomicAdd((unsigned long long*)local + k, (unsigned long long)c);
}
// the lanes of `heads`' segment that starts at this lane
__device__ __forceinline__ uint64_t segment(uint64_t heads, uint32_t lane) {
    const uint64_t later = heads & ~((2ull << lane) - 1ull);
    return (later ? (later & (0ull - later)) - 1ull : ~0ull) & ~((1ull << lane) - 1ull);
}

struct Triangles {  // {u, v, w} with last edge (u, v), in the order of the edges
    uint32_t u[128], v[128], w[128];
};
// The first n <= 64 triangles of a wavefront's queue: per group, the processor that stored both {u, w}
// and {v, w}, if one did, counts the triangle.
__device__ __forceinline__ void count_triangles(const IncCount& a, const Triangles& q, uint32_t n, uint32_t* hist,
                                                bool use_hist, NodeSums& sums, bool kept) {
    const uint32_t lane = threadIdx.x & 63;
    const bool valid = lane < n;
    const uint32_t u = valid ? q.u[lane] : kNoNode, v = valid ? q.v[lane] : kNoNode, w = valid ? q.w[lane] : 0u;
    // (an edge changes where v does, or u)
    const uint32_t pu = __shfl_up(u, 1, 64), pv = __shfl_up(v, 1, 64);
    const bool head_u = lane == 0 || pu != u, head_v = head_u || pv != v;
    const uint64_t seg_u = segment(__ballot(head_u), lane), seg_v = segment(__ballot(head_v), lane);
    for (uint32_t g = 0; g < a.G; ++g) {
        const uint64_t* c4 = a.hp + 4 * g;
        const uint32_t s1 = rept_hash::slot_of(c4, a.m, u, w), s2 = rept_hash::slot_of(c4, a.m, v, w);
        const uint32_t active = (g + 1 < a.G) ? a.ck_full : a.last_ck;
        const bool counted = valid && s1 == s2 && s1 < active;
        const uint32_t proc = g * a.pstride + s1;
        const uint64_t bal = __ballot(counted);
        if (!bal) continue;
        const uint64_t row = (uint64_t)(a.per_proc ? proc : g) * a.n;
        if (counted) {
            if (use_hist) atomicAdd(&hist[proc], 1u);
            else atomicAdd((unsigned long long*)a.global + proc, 1ull);
            node_add(sums, kept, a.local, row + w, 1u);
            if (a.per_proc) {  // (a row per lane)
                node_add(sums, kept, a.local, row + u, 1u);
                node_add(sums, kept, a.local, row + v, 1u);
            }
        }
        if (!a.per_proc) {
            const uint32_t cu = (uint32_t)__popcll(bal & seg_u), cv = (uint32_t)__popcll(bal & seg_v);
            if (head_u && cu) node_add(sums, kept, a.local, row + u, cu);
            if (head_v && cv) node_add(sums, kept, a.local, row + v, cv);
        }
    }
}

__global__ void __launch_bounds__(kCountThreads, 8) k_inc_count(IncCount a) {
    __shared__ unsigned int hist[kHist];
    __shared__ uint16_t s_end[kStage];  // from the run's start on; kRun: past the run
    __shared__ NodeSums sums;
    __shared__ Triangles queues[kCountThreads / 64];
    __shared__ uint64_t s_lo, s_hi;
    const uint32_t lane = threadIdx.x & 63;
    Triangles& queue = queues[threadIdx.x >> 6];
    uint32_t queued = 0;  // (the same in all lanes, below 64 between passes)
    const bool use_hist = a.c <= kHist, kept = a.rows * a.n < kNoNode;
    for (uint32_t i = threadIdx.x; i < kHist; i += blockDim.x) hist[i] = 0u;
    for (uint32_t i = threadIdx.x; i < 1u << kNodeBits; i += blockDim.x) {
        sums.key[i] = kNoNode;
        sums.sum[i] = 0u;
    }
    const uint64_t total = a.N2 ? a.end[a.N2 - 1] : 0;
    const auto flush = [&] {
        if (use_hist)
            for (uint32_t i = threadIdx.x; i < a.c; i += blockDim.x) {
                if (hist[i]) atomicAdd((unsigned long long*)a.global + i, (unsigned long long)hist[i]);
                hist[i] = 0u;
            }
        for (uint32_t i = threadIdx.x; i < 1u << kNodeBits; i += blockDim.x) {
            if (sums.sum[i]) atomicAdd((unsigned long long*)a.local + sums.key[i], (unsigned long long)sums.sum[i]);
            sums.sum[i] = 0u;
        }
    };
    // items taken since the last flush: each adds at most one to a processor's counter and to a
    // node's (the few queued ones later), so flushing once this reaches 2^31 keeps every LDS
    // counter below 2^32
    uint64_t since = 0;
    for (uint64_t i0 = (uint64_t)blockIdx.x * a.run; i0 < total; i0 += (uint64_t)gridDim.x * a.run) {
        const uint64_t i1 = (i0 + a.run) < total ? (i0 + a.run) : total;
        if (since + (i1 - i0) > (1ull << 31)) {  // uniform over the workgroup
            __syncthreads();
            flush();
            since = 0;
        }
        since += i1 - i0;
        __syncthreads();  // the previous run's readers of s_end are done (and the flush's)
        if (threadIdx.x < 128) {  // entries [lo, hi) hold the run
            const bool up = threadIdx.x >= 64;
            const uint64_t at = wave_upper_item(a.end, 0, a.N2, up ? i1 - 1 : i0);
            if (lane == 0) {
                if (up) s_hi = at + 1;
                else s_lo = at;
            }
        }
        __syncthreads();
        const uint64_t plo = s_lo, phi = s_hi;
        const bool staged = phi - plo <= kStage;
        if (staged)
            for (uint64_t k = threadIdx.x; k < phi - plo; k += blockDim.x) {
                const uint64_t e = a.end[plo + k] - i0;
                s_end[k] = (uint16_t)(e < kRun ? e : kRun);
            }
        __syncthreads();
        for (uint64_t ib = i0 + (threadIdx.x & ~63u); ib < i1; ib += blockDim.x) {
            const uint64_t i = ib + lane;
            uint32_t u = kNoNode, v = kNoNode, w = 0;
            bool hit = false;
            if (i < i1) {
                uint64_t p;
                if (staged) {
                    uint32_t lo = 0, hi = (uint32_t)(phi - plo);
                    while (lo < hi) {
                        const uint32_t mid = (lo + hi) >> 1;
                        if (s_end[mid] <= i - i0) lo = mid + 1;
                        else hi = mid;
                    }
                    p = plo + lo;
                } else {
                    p = upper_item(a.end, plo, phi, i);
                }
                const uint64_t k = a.ck[p];
                const uint32_t t = a.ct[p];
                u = hi32(k);
                v = lo32(k);
                const uint32_t su = a.off[u], du = a.off[u + 1] - su, sv = a.off[v], dv = a.off[v + 1] - sv;
                const uint64_t before = p ? (staged && p > plo ? i0 + s_end[p - 1 - plo] : a.end[p - 1]) : 0;
                const uint64_t j = i - before;
                // A: the shorter list (ties: u's), B: the other
                const bool au = du <= dv;
                const uint32_t sa = au ? su : sv;
                const uint32_t sb = au ? sv : su, db = au ? dv : du;
                if (a.tim[sa + j] < t) {  // (else {x, w} is not yet in any set)
                    w = lo32(a.key[sa + j]);
                    // (within a node's run the keys' low words ascend)
                    const uint32_t* low = (const uint32_t*)a.key + 2 * (uint64_t)sb;
                    uint32_t q = 0, hi = db;
                    while (q < hi) {
                        const uint32_t mid = (q + hi) >> 1;
                        if (low[2 * (uint64_t)mid] < w) q = mid + 1;
                        else hi = mid;
                    }
                    // triangle {u, v, w} with last edge (u, v)
                    hit = q < db && low[2 * (uint64_t)q] == w && a.tim[sb + q] < t;
                }
            }
            const uint64_t bal = __ballot(hit);
            if (hit) {
                const uint32_t at = queued + (uint32_t)__popcll(bal & ((1ull << lane) - 1ull));
                queue.u[at] = u;
                queue.v[at] = v;
                queue.w[at] = w;
            }
            queued += (uint32_t)__popcll(bal);
            if (queued < 64) continue;
            wave_fence();
            count_triangles(a, queue, 64, hist, use_hist, sums, kept);
            queued -= 64;
            if (lane < queued) {  // (reads of the upper half, writes of the lower)
                queue.u[lane] = queue.u[64 + lane];
                queue.v[lane] = queue.v[64 + lane];
                queue.w[lane] = queue.w[64 + lane];
            }
            wave_fence();
        }
    }
    wave_fence();
    if (queued) count_triangles(a, queue, queued, hist, use_hist, sums, kept);
    __syncthreads();
    flush();
}

__global__ void k_inc_zero64(uint64_t* p, uint64_t words) {
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < words; i += (uint64_t)gridDim.x * blockDim.x)
        p[i] = 0ull;
}

uint32_t grid_of(uint64_t items, uint32_t cap) {
    uint64_t b = (items + kThreads - 1) / kThreads;
    if (b > cap) b = cap;
    return b ? (uint32_t)b : 1u;
}

// ---- stable LSD radix sort of (key, time) pairs.  The digits are cut from the key's two ids put
// together (x << id_bits | y), at most kDigit bits each and as even as they come, so that ids of 17
// bits take four passes.  A workgroup takes a tile of RS_TILE pairs, each wavefront a contiguous part
// of it, held in registers; a pass counts the digits per tile, scans the counts digit-major (all
// tiles' 0s, then all tiles' 1s, ...), and scatters each tile stably: a wavefront ranks its lanes
// among the lanes of the same digit (a ballot per bit) behind its running count of the digit, and the
// wavefronts' counts, summed from the tile's base, place them.  The first pass's counts come from the
// kernel that makes the keys.  Short of pairs in flight at these sizes (a chunk of 200k edges is 98
// tiles), so the workgroups are large: 16 wavefronts to a tile and wider digits, with one launch per
// scan, take 97 us for that chunk with 17-bit ids, where four wavefronts, digits of 8 bits and three
// launches per scan took 250.
constexpr uint32_t RS_THREADS = 1024, RS_WAVES = RS_THREADS / 64;
constexpr uint32_t RS_TILE = 4096, RS_WAVE = RS_TILE / RS_WAVES, RS_ITEMS = RS_WAVE / 64;
constexpr uint32_t kDigit = 9;
constexpr uint32_t kScanItems = 16, kScanTile = kThreads * kScanItems;

struct Digit {
    uint32_t id_bits, shift, bits;
};
__device__ __forceinline__ uint32_t digit_of(const Digit& d, uint64_t k) {
    return (uint32_t)((((uint64_t)hi32(k) << d.id_bits) | lo32(k)) >> d.shift) & ((1u << d.bits) - 1u);
}

// 1b. chunk edges -> keys of both directions and times, a tile of RS_TILE keys per workgroup
__global__ void __launch_bounds__(RS_THREADS) k_inc_keys(const uint2* __restrict__ edges, IncChunk a, Digit dg,
                                                         uint32_t* __restrict__ hist) {
    __shared__ uint32_t h[1u << kDigit];
    for (uint32_t i = threadIdx.x; i < 1u << kDigit; i += RS_THREADS) h[i] = 0;
    for (uint32_t k = blockIdx.x * RS_THREADS + threadIdx.x; k < a.look_words; k += gridDim.x * RS_THREADS)
        a.look[k] = 0ull;
    __syncthreads();
    uint32_t f = 0;
#pragma unroll
    for (uint32_t r = 0; r < RS_TILE / 2; r += RS_THREADS) {
        const uint64_t i = (uint64_t)blockIdx.x * (RS_TILE / 2) + r + threadIdx.x;
        if (i < a.W) {
            uint2 e = edges[i];
            a.eall[i] = e;
            f |= edge_flags(e, a.n);
            const uint64_t k0 = edge_key(e, false), k1 = edge_key(e, true);
            *(ulonglong2*)(a.ckey + 2 * i) = make_ulonglong2(k0, k1);
            *(uint2*)(a.ctim + 2 * i) = make_uint2(a.T + (uint32_t)i, a.T + (uint32_t)i);
            atomicAdd(&h[digit_of(dg, k0)], 1u);
            atomicAdd(&h[digit_of(dg, k1)], 1u);
        }
    }
    if (f) atomicOr(a.flags, f);
    __syncthreads();
    for (uint32_t d = threadIdx.x; d < 1u << dg.bits; d += RS_THREADS) hist[(uint64_t)d * gridDim.x + blockIdx.x] = h[d];
}

__global__ void __launch_bounds__(RS_THREADS) k_rs_hist(const uint64_t* __restrict__ keys, uint64_t N, Digit dg,
                                                        uint32_t* __restrict__ hist) {
    __shared__ uint32_t h[1u << kDigit];
    for (uint32_t i = threadIdx.x; i < 1u << kDigit; i += RS_THREADS) h[i] = 0;
    __syncthreads();
    const uint64_t b0 = (uint64_t)blockIdx.x * RS_TILE;
#pragma unroll
    for (uint32_t r = 0; r < RS_TILE; r += RS_THREADS) {
        const uint64_t i = b0 + r + threadIdx.x;
        if (i < N) atomicAdd(&h[digit_of(dg, keys[i])], 1u);
    }
    __syncthreads();
    for (uint32_t d = threadIdx.x; d < 1u << dg.bits; d += RS_THREADS) hist[(uint64_t)d * gridDim.x + blockIdx.x] = h[d];
}

// exclusive scan of c[0, N) in place
__global__ void __launch_bounds__(kThreads) k_rs_scan(uint32_t* c, uint32_t N, scan::Look L) {
    const uint32_t t = scan::look_ticket(L);
    const uint32_t b0 = t * kScanTile + threadIdx.x * kScanItems;
    uint32_t v[kScanItems], s = 0;
#pragma unroll
    for (uint32_t r = 0; r < kScanItems; ++r) {
        v[r] = b0 + r < N ? c[b0 + r] : 0u;
        s += v[r];
    }
    uint32_t tot;
    uint32_t run = scan::block_excl_scan<uint32_t>(s, tot);
    run += scan::look_back<uint32_t>(L, t, tot);
#pragma unroll
    for (uint32_t r = 0; r < kScanItems; ++r) {
        if (b0 + r < N) c[b0 + r] = run;
        run += v[r];
    }
}

__global__ void __launch_bounds__(RS_THREADS) k_rs_scatter(const uint64_t* __restrict__ kin,
                                                           const uint32_t* __restrict__ vin, uint64_t N, Digit dg,
                                                           const uint32_t* __restrict__ base,
                                                           uint64_t* __restrict__ kout, uint32_t* __restrict__ vout) {
    __shared__ uint32_t wc[RS_WAVES][1u << kDigit];  // per wavefront: digit counts, then bases
    const uint32_t lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const uint64_t t0 = (uint64_t)blockIdx.x * RS_TILE + (uint64_t)w * RS_WAVE;
    uint64_t k[RS_ITEMS];
    uint32_t t[RS_ITEMS], at[RS_ITEMS];
#pragma unroll
    for (uint32_t r = 0; r < RS_ITEMS; ++r) {
        const uint64_t i = t0 + r * 64 + lane;
        k[r] = i < N ? kin[i] : 0ull;
        t[r] = i < N ? vin[i] : 0u;
    }
    for (uint32_t i = threadIdx.x; i < RS_WAVES << kDigit; i += RS_THREADS) (&wc[0][0])[i] = 0;
    __syncthreads();
    const uint64_t below = lane ? (~0ull >> (64 - lane)) : 0ull;
#pragma unroll
    for (uint32_t r = 0; r < RS_ITEMS; ++r) {
        const bool valid = t0 + r * 64 + lane < N;
        const uint32_t dig = digit_of(dg, k[r]);
        uint64_t peers = __ballot(valid);
        for (uint32_t bit = 0; bit < dg.bits; ++bit) {
            const bool one = (dig >> bit) & 1u;
            const uint64_t bb = __ballot(valid && one);
            peers &= one ? bb : ~bb;
        }
        at[r] = wc[w][dig] + (uint32_t)__popcll(peers & below);
        wave_fence();  // every lane has read its digit's count
        if (valid && (int)lane == 63 - __clzll(peers)) wc[w][dig] += (uint32_t)__popcll(peers);
        wave_fence();
    }
    __syncthreads();
    for (uint32_t d = threadIdx.x; d < 1u << dg.bits; d += RS_THREADS) {
        uint32_t run = base[(uint64_t)d * gridDim.x + blockIdx.x];
#pragma unroll
        for (uint32_t v = 0; v < RS_WAVES; ++v) {
            const uint32_t c = wc[v][d];
            wc[v][d] = run;
            run += c;
        }
    }
    __syncthreads();
#pragma unroll
    for (uint32_t r = 0; r < RS_ITEMS; ++r)
        if (t0 + r * 64 + lane < N) {
            const uint32_t q = wc[w][digit_of(dg, k[r])] + at[r];
            kout[q] = k[r];
            vout[q] = t[r];
        }
}

// temporary storage of an append: the digit counts, then the scans' words (one scan per digit and the
// items' scan, which comes first), which the append's first kernel clears
struct SortTemp {
    size_t hist, look, total;
    uint32_t nb, digit_words, item_words;  // tiles; words of a digit's scan and of the items' scan
};
SortTemp sort_temp(uint64_t N) {
    SortTemp T;
    T.nb = (uint32_t)((N + RS_TILE - 1) / RS_TILE);
    if (T.nb == 0) T.nb = 1;
    const uint64_t nh = (uint64_t)T.nb << kDigit;
    T.digit_words = 1 + (uint32_t)((nh + kScanTile - 1) / kScanTile);
    T.item_words = 1 + (uint32_t)((N + kItemTile - 1) / kItemTile);
    constexpr uint32_t passes = (2 * 29 + kDigit - 1) / kDigit;  // ids below 2^29
    size_t p = 0;
    T.hist = p; p = (p + 4 * nh + 255) & ~(size_t)255;
    T.look = p; p = (p + 8 * ((uint64_t)T.item_words + passes * T.digit_words) + 255) & ~(size_t)255;
    T.total = p;
    return T;
}
scan::Look look_at(unsigned long long* words) { return scan::Look{(uint32_t*)words, words + 1}; }

// Chunks of at most this many edges are sorted by k_inc_rank, whose compares grow with the square of
// the chunk (up to here it has a workgroup per CU at most), while the radix sort's launches hardly grow.
// A whole append to 100k nodes by either: 1,000 edges 68 and 124 us, 4,000 95 and 149, 8,000 125 and
// 155, 12,000 238 and 158; to 3,000 nodes (three digits instead of four) 8,000 edges 131 and 139.
constexpr uint64_t kRankEdges = 8192;

}  // namespace

// ---------------------------------------------------------------------------- launchers ----

size_t rept_inc_sort_temp_bytes(uint64_t entries) { return sort_temp(entries).total; }

hipError_t rept_inc_zero64(void* p, uint64_t words, hipStream_t s) {
    (void)hipGetLastError();
    hipLaunchKernelGGL(k_inc_zero64, dim3(grid_of(words, 4096)), dim3(kThreads), 0, s, (uint64_t*)p, words);
    return hipGetLastError();
}

hipError_t rept_inc_prepare(IncState& st, const uint32_t* edges, uint64_t W, uint32_t* eall, hipStream_t s) {
    (void)hipGetLastError();
    const uint64_t N2 = 2 * W, N = 2 * st.T;
    const SortTemp L = sort_temp(N2);
    uint32_t* hist = (uint32_t*)((uint8_t*)st.temp + L.hist);
    unsigned long long* look = (unsigned long long*)((uint8_t*)st.temp + L.look);
    if (!st.flags_clear)
        hipLaunchKernelGGL(k_inc_zero64, dim3(1), dim3(64), 0, s, (uint64_t*)st.flags, (uint64_t)1);
    st.flags_clear = false;  // until the host has read them as zero
    IncChunk a{W, st.n, (uint32_t)st.T, st.ckey_b, st.ctim_b, (uint2*)eall, st.flags, look, L.item_words};
    if (W <= kRankEdges) {
        hipLaunchKernelGGL(k_inc_rank, dim3((uint32_t)((N2 + 63) / 64)), dim3(kRankThreads), 0, s, (const uint2*)edges, a);
    } else {
        const uint32_t id_bits = st.id_bits, passes = (2 * id_bits + kDigit - 1) / kDigit;
        uint64_t *src_k = st.ckey_b, *dst_k = st.ckey_a;  // the last pass ends in b
        uint32_t *src_t = st.ctim_b, *dst_t = st.ctim_a;
        if (passes & 1u) {
            src_k = st.ckey_a; dst_k = st.ckey_b;
            src_t = st.ctim_a; dst_t = st.ctim_b;
        }
        a.ckey = src_k;
        a.ctim = src_t;
        a.look_words = L.item_words + passes * L.digit_words;
        Digit dg{id_bits, 0, 0};
        for (uint32_t p = 0; p < passes; ++p) {
            dg.shift += dg.bits;
            dg.bits = (2 * id_bits - dg.shift + passes - p - 1) / (passes - p);
            if (p == 0)
                hipLaunchKernelGGL(k_inc_keys, dim3(L.nb), dim3(RS_THREADS), 0, s, (const uint2*)edges, a, dg, hist);
            else
                hipLaunchKernelGGL(k_rs_hist, dim3(L.nb), dim3(RS_THREADS), 0, s, src_k, N2, dg, hist);
            const uint32_t nh = L.nb << dg.bits;
            hipLaunchKernelGGL(k_rs_scan, dim3((nh + kScanTile - 1) / kScanTile), dim3(kThreads), 0, s, hist, nh,
                               look_at(look + L.item_words + p * L.digit_words));
            hipLaunchKernelGGL(k_rs_scatter, dim3(L.nb), dim3(RS_THREADS), 0, s, src_k, src_t, N2, dg, hist, dst_k,
                               dst_t);
            uint64_t* tk = src_k; src_k = dst_k; dst_k = tk;
            uint32_t* tt = src_t; src_t = dst_t; dst_t = tt;
        }
    }
    const int nxt = st.cur ^ 1;
    hipLaunchKernelGGL(k_inc_noff, dim3(grid_of((uint64_t)st.n + 1, 8192)), dim3(kThreads), 0, s, st.ckey_b, N2, st.n,
                       st.off, st.noff);
    hipLaunchKernelGGL(k_inc_merge, dim3(grid_of(N + N2, 8192)), dim3(kThreads), 0, s, st.key[st.cur], st.tim[st.cur],
                       N, st.ckey_b, st.ctim_b, N2, st.off, st.noff, st.key[nxt], st.tim[nxt], st.flags);
    hipLaunchKernelGGL(k_inc_items, dim3((uint32_t)((N2 + kItemTile - 1) / kItemTile)), dim3(kThreads), 0, s,
                       st.ckey_b, N2, st.noff, st.end, (uint64_t*)st.flags + 1, look_at(look));
    return hipGetLastError();
}

void rept_inc_accept(IncState& st, uint64_t W) {
    uint32_t* o = st.off;
    st.off = st.noff;
    st.noff = o;
    st.cur ^= 1;
    st.T += W;
    st.flags_clear = true;
}

hipError_t rept_inc_count(const IncState& st, uint64_t W, uint64_t items, const IncCount& base, hipStream_t s) {
    (void)hipGetLastError();
    const uint64_t N2 = 2 * W;
    IncCount a = base;
    a.key = st.key[st.cur];
    a.tim = st.tim[st.cur];
    a.off = st.off;
    a.ck = st.ckey_b;
    a.ct = st.ctim_b;
    a.end = st.end;
    a.N2 = N2;
    if (items == 0) return hipSuccess;
    // Few items are spread over the grid (90k items in runs of 4096 are 22 workgroups: 91 us, in runs of
    // their threads 18)
    uint64_t run = (items / st.count_blocks + kCountThreads) / kCountThreads * kCountThreads;
    if (run > kRun) run = kRun;
    a.run = (uint32_t)run;
    const uint64_t runs = (items + run - 1) / run;
    const uint32_t blocks = runs < st.count_blocks ? (uint32_t)runs : st.count_blocks;
    hipLaunchKernelGGL(k_inc_count, dim3(blocks), dim3(kCountThreads), 0, s, a);
    return hipGetLastError();
}

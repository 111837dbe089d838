// The counting pass of REPT (Algorithm 1, Section III-A; groups of Section III-B) for every
// processor at once.
//
// What is counted.  For the stream edge (u, v) arriving at time t, processor i adds
// |N_u^(i) ∩ N_v^(i)| to tau^(i), tau_u^(i) and tau_v^(i) and one to tau_w^(i) for each common
// neighbour w, where N_x^(i) holds the neighbours of x through edges processor i stored
// before t.  So every triangle {x, y, z} of the stream graph is counted exactly once per
// processor that stored its first two edges -- at the update of its last edge -- and then
// adds one to tau^(i) and one to the local counter of each of its three nodes (the
// semi-triangles of Section III; Theorem 2).
//
// How it is counted here.  The build stores each edge once, at its lower-ranked endpoint
// (the "apex" side).  A triangle a < b < w (by rank) is found exactly once: from apex a, as
// the entry w of b's list that is also in a's list.  The three arrival times give its last
// edge; the hash of its first two edges gives, per group, whether one processor stored both.
// One pass therefore serves all c processors, and a window [t0, t1) of stream updates is the
// set of triangles whose last edge arrived in the window.
//
// Kernel.  k_count is persistent and drains a device work queue over all jobs of a batch, in
// two phases: apexes with long lists (or many lists to walk) one per workgroup, then the rest, several
// to a wavefront.  A team (workgroup or wavefront) stages a's list in LDS (W side): its entries, a
// filter of one bit per hashed node, and a hash table of their indices.  Its wavefronts then walk
// the lists of a's out-neighbours b (B side) in chunks of up to 64 lists: each walked entry is one
// global load and one filter test; the entries that pass go to a per-wavefront LDS queue and are
// looked up in the exact table and attributed in full-wave batches.  Local counts are aggregated per
// staged entry (and a graph's hubs per workgroup) and global counts per processor in LDS before the
// 64-bit global atomics.
//
// What bounds it.  On the 1M/20M power-law stream (m = 10, c = 40) the heavy phase takes 3.5 ms and the
// light one 0.85 ms, 1.24e9 entries walked.  The vector pipes are busy half of that time; the rest
// is latency: a unit is a chain of dependent loads (its list; the lists' bounds; their entries; the
// candidates' times and slots), with four wavefronts per SIMD to hide it.  Hence the loads issued a
// step ahead, the units counted together by a light wavefront, the workgroup's next tile fetched
// during the current one.  Before these, with an exact table probed per entry, the two phases took
// 4.6 and 1.5 ms.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdio.h>

#include <mutex>
#include <type_traits>

#include "common.h"
#include "edge_hash.h"

namespace {

constexpr uint32_t kHashMul = 0x9E3779B1u;  // table index: Fibonacci hashing of the node id
constexpr uint32_t kFiltMul = 0x9E3779u;     // filter position: 24-bit product of the node id
constexpr uint32_t kGranHeavy = 16;          // entries of one list walked by one lane group
constexpr uint32_t kGranLight = 8;           // (light units' lists are shorter)
constexpr uint32_t kStepHeavy = 4;           // windows of 64 entries loaded together
constexpr uint32_t kStepLight = 2;           // (a light unit has few, and its registers cost waves)
constexpr uint32_t kStepEta = 2;             // (with pair counters, four would spill)
constexpr uint32_t kWalk = 2;                // windows tested between looks at the queue
constexpr uint32_t kQueue = 64 * (kWalk + 1);  // per-wavefront queue: < 64 left + those windows'

__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <bool BLOCK>
__device__ __forceinline__ void team_sync() {
    if (BLOCK) __syncthreads();
    else wave_sync();
}

__device__ __forceinline__ uint32_t lane_id() { return threadIdx.x & 63; }

// A value that is the same in every active lane, in a scalar register.  The compiler cannot
// see that a value read from LDS or exchanged between lanes is uniform; in a scalar register,
// the loops and branches on it take scalar instructions instead of exec-mask control flow.
// (Applied only where it was measured to pay: scalar registers are scarce in k_count, and
// their spills cost vector instructions.)
__device__ __forceinline__ uint32_t wave_uni(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }
// lane u's value (u uniform), in a scalar register
__device__ __forceinline__ uint32_t lane_val(uint32_t v, uint32_t u) {
    return (uint32_t)__builtin_amdgcn_readlane((int)v, (int)u);
}

// Inclusive prefix sum over the 64 lanes with DPP: shifts by 1, 2, 4, 8 within rows of 16
// lanes, then row 0's and row 2's last lanes broadcast into rows 1 and 3 (row_bcast:15), then
// lane 31 into rows 2 and 3 (row_bcast:31).  Lanes without a source add zero.
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v) {
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false);  // row_shr:1
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false);  // row_shr:2
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false);  // row_shr:4
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false);  // row_shr:8
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false);  // row_bcast:15
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false);  // row_bcast:31
    return v;
}

__device__ __forceinline__ uint32_t wave_sum(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_readlane((int)wave_incl_scan(v), 63);
}

__host__ __device__ inline uint32_t pow2_at_least(uint32_t x) {
    uint32_t p = 64;
    while (p < x) p <<= 1;
    return p;
}
__host__ __device__ inline uint32_t log2u(uint32_t p) {
    uint32_t l = 0;
    while ((1u << l) < p) ++l;
    return l;
}
__host__ __device__ inline uint32_t up16(uint32_t x) { return (x + 15u) & ~15u; }
// 16-bit slots per staged edge: G padded to 1, 2, 4 or 8 (the slot table's row width)
__host__ __device__ inline uint32_t slot_width(uint32_t G) { return G <= 1 ? 1u : (G <= 2 ? 2u : (G <= 4 ? 4u : 8u)); }

// ---- LDS layout (shared by host sizing and device carving) --------------------------------
// [per-wave misc] x nwaves, then one union region: the workgroup's heavy team area or the
// wavefronts' light team areas (the heavy phase finishes before the light phase starts).
struct WArea {  // a's list: hash filter, hash table and entries
    uint32_t filt, table, ew, et, wslot, cntw, ownl, ewe;
    uint32_t red;  // 64 words of team scratch (reductions, the next chunk of lists)
    uint32_t bytes;
};
constexpr uint32_t kPack = 16;  // light units counted together by a wavefront, at most
struct UArea {  // the units of a wavefront's pass
    uint32_t w0, l0, s, r0, a, own;
    uint32_t bytes;
};
struct BArea {  // one wavefront's chunk of lists to walk
    uint32_t eb, etb, bslot, cntb, bpos, bgr, ebe;
    uint32_t bytes;
};
// RW: slots per staged row (the widest slot-table row of the launch's jobs: the padded group
// count, or one keep mask for parallel MASCOT); G: groups of per-entry counters
// eta: also Algorithm 2's per-edge counts, (s, L) packed 16 + 16 bits per group
__host__ __device__ inline WArea w_layout(uint32_t DW, uint32_t G, uint32_t RW, bool eta) {
    WArea A;
    uint32_t p = 0;
    A.filt = p; p = up16(p + 4 * pow2_at_least(DW));
    A.table = p; p = up16(p + 4 * pow2_at_least(2 * DW));
    A.ew = p; p = up16(p + 4 * DW);
    A.et = p; p = up16(p + 4 * DW);
    A.wslot = p; p = up16(p + 2 * RW * DW);
    A.cntw = p; p = up16(p + 2 * slot_width(G) * DW);
    A.ownl = p; p = up16(p + 2 * DW);  // the W entries whose own lists are walked
    A.ewe = p; p = eta ? up16(p + 4 * G * DW) : p;
    A.red = p; p = up16(p + 4 * 64);
    A.bytes = p;
    return A;
}
__host__ __device__ inline UArea u_layout(uint32_t G) {
    UArea A;
    uint32_t p = 0;
    A.w0 = p; p += 4 * (kPack + 1);   // first W entry of each unit (and their number)
    A.l0 = p; p += 4 * (kPack + 1);   // first reverse list of each unit (and their number)
    A.s = p; p += 4 * kPack;          // offset of its list
    A.r0 = p; p += 4 * kPack;         // offset of its reverse list
    A.a = p; p += 4 * kPack;          // its node
    A.own = p; p = up16(p + 4 * G * kPack);  // its own counts
    A.bytes = p;
    return A;
}
__host__ __device__ inline BArea b_layout(uint32_t DB, uint32_t G, uint32_t RW, bool eta) {
    BArea A;
    uint32_t p = 0;
    A.eb = p; p = up16(p + 4 * DB);
    A.etb = p; p = up16(p + 4 * DB);
    A.bslot = p; p = up16(p + 2 * RW * DB);
    A.cntb = p; p = up16(p + 2 * slot_width(G) * DB);
    A.bpos = p; p = up16(p + 8 * DB);        // (offset, length | unit << 28) of each staged list
    A.bgr = p; p = up16(p + 4 * (DB + 1));   // its first granule in the chunk's walk
    A.ebe = p; p = eta ? up16(p + 4 * G * DB) : p;
    A.bytes = p;
    return A;
}
struct Misc {  // per wavefront
    uint32_t mark, desc, qe, qo, hist, bytes;
};
__host__ __device__ inline Misc misc_layout(uint32_t HC) {
    Misc M;
    uint32_t p = 0;
    M.mark = M.desc = p; p = up16(p + 8 * 64);  // a batch's granules; before them, a byte mark each
    M.qe = p; p = up16(p + 8 * kQueue);
    M.qo = p; p = up16(p + 2 * kQueue);
    M.hist = p; p = up16(p + 4 * HC);
    M.bytes = p;
    return M;
}
// A workgroup's hub counters: a hash table of the hubs' nodes (linear probing), and per group one
// 64-bit count per table slot.
constexpr uint32_t kHubSlots = 2 * kHubs;
constexpr uint32_t kHubShift = 32 - __builtin_ctz(kHubSlots);
static_assert((kHubSlots & (kHubSlots - 1)) == 0, "indexed by the top bits of a hash");
__host__ __device__ inline uint32_t hub_bytes(uint32_t G) { return 4 * kHubSlots + 8 * kHubSlots * G; }
struct Layout {
    Misc misc;
    WArea hw, lw;  // the heavy team's, a light wavefront's
    BArea hb, lb;  // a wavefront's in the heavy and in the light phase
    UArea lu;
    uint32_t misc_off, union_off, total;
};
// lists per chunk of a heavy team's wavefront: its share of the workgroup's, one per lane at most
__host__ __device__ inline uint32_t wave_lists(uint32_t DB, uint32_t nwaves) {
    const uint32_t x = (DB + nwaves - 1) / nwaves;
    return x < 64u ? x : 64u;
}
__host__ __device__ inline Layout count_layout(uint32_t nwaves, uint32_t DL, uint32_t DW, uint32_t DB,
                                               uint32_t G, uint32_t RW, uint32_t HC, uint32_t DLB, bool eta,
                                               bool heavy, bool light) {
    Layout L;
    L.misc = misc_layout(HC);
    L.hw = w_layout(DW, G, RW, eta);
    L.hb = b_layout(wave_lists(DB, nwaves), G, RW, eta);
    L.lw = w_layout(DL, G, RW, eta);
    L.lb = b_layout(wave_lists(DLB, 1), G, RW, eta);
    L.lu = u_layout(G);
    L.misc_off = up16(hub_bytes(G));
    L.union_off = L.misc_off + nwaves * L.misc.bytes;
    // a launch holds only the areas of the phases it runs
    const uint32_t hb = heavy ? L.hw.bytes + nwaves * L.hb.bytes : 0u;
    const uint32_t lb = light ? nwaves * (L.lw.bytes + L.lb.bytes + L.lu.bytes) : 0u;
    const uint32_t u = hb > lb ? hb : lb;
    L.total = L.union_off + u;
    return L;
}

// ---- views ---------------------------------------------------------------------------------
struct TeamView {
    uint32_t* filt;  // one bit per hashed key position, DW words (a power of two of at least 64)
    uint32_t* table;  // of the keys' indices, pow2_at_least(2 DW) slots
    uint32_t* ew;
    uint32_t* et;
    uint16_t* wslot;  // [DW][gs] slot rows of the W entries
    uint16_t* cntw;  // [DW][gp] local counts of the W entries since the last flush, by group
    uint16_t* ownl;  // W entries i of the pairs whose lists the unit walks (| unit << 12 in a light pass)
    uint32_t* eb;
    uint32_t* etb;
    uint16_t* bslot;  // [DB][gs] slot rows of the B entries
    uint16_t* cntb;  // [DB][gp] of the B entries
    uint2* bpos;    // offset of b's list, its length (below 2^16) | its unit << 28
    uint32_t* bgr;  // index of its first granule in the chunk's walk; after the last list, their number
    uint32_t* ewe;   // [G][DW] pair counts (s | L << 16) of the W entries since the last flush
    uint32_t* ebe;   // [G][DB] the same for the B entries
    uint32_t* red;
    uint32_t *uw0, *ul0, *us, *ur0, *ua, *uown;  // the units of a light pass (UArea)
    uint32_t DW, DB;
};
__device__ inline TeamView team_view(uint8_t* base, uint8_t* bbase, const WArea& A, const BArea& B, uint32_t DW,
                                     uint32_t DB) {
    TeamView T;
    T.filt = (uint32_t*)(base + A.filt);
    T.table = (uint32_t*)(base + A.table);
    T.ew = (uint32_t*)(base + A.ew);
    T.et = (uint32_t*)(base + A.et);
    T.wslot = (uint16_t*)(base + A.wslot);
    T.cntw = (uint16_t*)(base + A.cntw);
    T.eb = (uint32_t*)(bbase + B.eb);
    T.etb = (uint32_t*)(bbase + B.etb);
    T.bslot = (uint16_t*)(bbase + B.bslot);
    T.cntb = (uint16_t*)(bbase + B.cntb);
    T.bpos = (uint2*)(bbase + B.bpos);
    T.bgr = (uint32_t*)(bbase + B.bgr);
    T.ownl = (uint16_t*)(base + A.ownl);
    T.ewe = (uint32_t*)(base + A.ewe);
    T.ebe = (uint32_t*)(bbase + B.ebe);
    T.red = (uint32_t*)(base + A.red);
    T.DW = DW;
    T.DB = DB;
    return T;
}
__device__ inline void unit_view(TeamView& T, uint8_t* base, const UArea& A) {
    T.uw0 = (uint32_t*)(base + A.w0);
    T.ul0 = (uint32_t*)(base + A.l0);
    T.us = (uint32_t*)(base + A.s);
    T.ur0 = (uint32_t*)(base + A.r0);
    T.ua = (uint32_t*)(base + A.a);
    T.uown = (uint32_t*)(base + A.own);
}
struct WaveView {
    uint8_t* mark;
    uint2* desc;   // granules of a batch: position of the first entry, entries | list << 16 | unit << 28
    uint2* qe;     // queued candidates: list position, node id
    uint16_t* qo;  // and their list | unit << 12
    uint32_t* hist;
    uint32_t* hub;  // the workgroup's hub table, or null if it holds another job's
    uint32_t hits;  // candidates drained since the histogram's last flush (uniform)
};
__device__ inline WaveView wave_view(uint8_t* base, const Misc& M) {
    WaveView V;
    V.mark = base + M.mark;
    V.desc = (uint2*)(base + M.desc);
    V.qe = (uint2*)(base + M.qe);
    V.qo = (uint16_t*)(base + M.qo);
    V.hist = (uint32_t*)(base + M.hist);
    V.hits = 0;
    V.hub = nullptr;
    return V;
}

// ---- per-job constants held while a wavefront works on that job ----------------------------
struct JobRegs {
    const JobDev* __restrict__ jd;  // what is not used per walked entry is read from there
    const uint32_t* off;
    const uint32_t* nbr;
    const uint32_t* tim;
    const uint4* rrec;
    const uint32_t* rpos;
    int64_t* local;
    const uint16_t* tab;  // slot table of the stored edges, gs slots per edge
    uint32_t* pairs;      // Algorithm 2's counters (null: none), es edges to a group
    uint32_t n, G, gs, gp, per_proc, t0, t1, ck, last_ck, pstride, use_hist, mask, es;
};

__device__ inline void load_job(const JobDev* __restrict__ j, uint32_t HC, JobRegs& r) {
    r.jd = j;
    r.off = j->off;
    r.pairs = j->pairs;  // (read per hit: from the job they cost 20M edges 13.0 ms instead of 9.0)
    r.es = j->es;
    r.nbr = j->nbr;
    r.tim = j->tim;
    r.rrec = j->rrec;
    r.rpos = j->rpos;
    r.local = j->local;
    r.n = j->n;
    r.tab = j->tab;
    r.gs = j->gs;
    r.G = j->G;
    r.gp = slot_width(j->G);
    r.per_proc = j->per_proc;
    r.t0 = j->t0;
    r.t1 = j->t1;
    r.ck = j->ck;
    r.last_ck = j->last_ck;
    r.pstride = j->pstride;
    r.mask = j->mask;
    r.use_hist = (HC != 0 && j->c <= HC) ? 1u : 0u;
}

using rept_hash::slot_of;

__device__ __forceinline__ void add64(int64_t* p, uint64_t v) {
    atomicAdd((unsigned long long*)p, (unsigned long long)v);
}

// ---- hub counters.  A hub's local counter is updated by almost every unit; one address takes about
// 9 ns per 64-bit atomic, so on a 2M-edge power-law stream (largest degree 5e4) the queue of the
// largest hub's updates alone outlasted the light units' work.  A workgroup therefore gathers its
// hub updates in LDS and adds them once per job: at most one update per workgroup and hub.
__device__ __forceinline__ uint32_t hub_find(const uint32_t* key, uint32_t node) {  // slot, or kHubSlots
    uint32_t h = (node * kHashMul) >> kHubShift;
    for (;;) {
        const uint32_t k = key[h];
        if (k == node + 1u) return h;
        if (k == 0u) return kHubSlots;
        h = (h + 1u) & (kHubSlots - 1u);
    }
}
// the slot of a node whose counts go to the hub table, kHubSlots otherwise
__device__ __forceinline__ uint32_t hub_slot(const uint32_t* hub, uint32_t node) {
    return hub ? hub_find(hub, node) : kHubSlots;
}
__device__ __forceinline__ void add_local(int64_t* local, uint32_t n, uint32_t* hub, uint32_t slot, uint32_t g,
                                          uint32_t node, uint64_t v) {
    if (slot < kHubSlots)
        atomicAdd((unsigned long long*)(hub + kHubSlots) + g * kHubSlots + slot, (unsigned long long)v);
    else
        add64(local + (uint64_t)g * n + node, v);
}
// bind the table to a job (whole workgroup; the table is empty or flushed)
__device__ __forceinline__ void hub_bind(const JobDev& J, uint32_t* hub, uint32_t G) {
    for (uint32_t i = threadIdx.x; i < kHubSlots + 2 * kHubSlots * G; i += blockDim.x) hub[i] = 0u;
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < J.n_hub; i += blockDim.x) {
        const uint32_t v = J.hubs[i];
        uint32_t h = (v * kHashMul) >> kHubShift;
        while (atomicCAS(&hub[h], 0u, v + 1u) != 0u) h = (h + 1u) & (kHubSlots - 1u);
    }
    __syncthreads();
}
// add the table's counts to the job's outputs (whole workgroup)
__device__ __forceinline__ void hub_flush(const JobDev& J, const uint32_t* hub) {
    __syncthreads();
    if (!J.per_proc)
        for (uint32_t i = threadIdx.x; i < kHubSlots * J.G; i += blockDim.x) {
            const uint32_t k = hub[i % kHubSlots];
            const uint64_t v = ((const uint64_t*)(hub + kHubSlots))[i];
            if (k && v) add64(J.local + (uint64_t)(i / kHubSlots) * J.n + (k - 1u), v);
        }
    __syncthreads();
}

// loads from the graph arrays (global memory: lets the compiler emit global, not flat, loads)
template <typename T>
__device__ __forceinline__ T ldg(const T* p) {
    return *(const __attribute__((address_space(1))) T*)p;
}

// Slots of the edge stored at position p for every group, 16 bits per group: groups 0-3 in
// `lo`, groups 4-7 in `hi`.  gs (1, 2, 4 or 8) is uniform over the wavefront.
__device__ __forceinline__ void load_slots(const uint16_t* tab, uint32_t gs, uint32_t p, uint64_t& lo,
                                           uint64_t& hi) {
    hi = 0;
    if (gs == 1) {
        lo = ldg(tab + p);
    } else if (gs == 2) {
        lo = ldg((const uint32_t*)tab + p);
    } else if (gs == 4) {
        lo = ldg((const uint64_t*)tab + p);
    } else {
        lo = ldg((const uint64_t*)tab + 2 * (uint64_t)p);
        hi = ldg((const uint64_t*)tab + 2 * (uint64_t)p + 1);
    }
}
// staged slot rows in LDS, in the slot table's format; GS: row width known at compile time
template <uint32_t GS>
__device__ __forceinline__ void lds_row_t(const uint16_t* rows, uint32_t i, uint64_t& lo, uint64_t& hi) {
    hi = 0;
    if (GS == 1) {
        lo = rows[i];
    } else if (GS == 2) {
        lo = ((const uint32_t*)rows)[i];
    } else if (GS == 4) {
        lo = ((const uint64_t*)rows)[i];
    } else {
        const uint4 r = ((const uint4*)rows)[i];
        lo = ((uint64_t)r.y << 32) | r.x;
        hi = ((uint64_t)r.w << 32) | r.z;
    }
}
template <uint32_t GS>
__device__ __forceinline__ void load_slots_t(const uint16_t* tab, uint32_t p, uint64_t& lo, uint64_t& hi) {
    hi = 0;
    if (GS == 1) {
        lo = ldg(tab + p);
    } else if (GS == 2) {
        lo = ldg((const uint32_t*)tab + p);
    } else if (GS == 4) {
        lo = ldg((const uint64_t*)tab + p);
    } else {
        lo = ldg((const uint64_t*)tab + 2 * (uint64_t)p);
        hi = ldg((const uint64_t*)tab + 2 * (uint64_t)p + 1);
    }
}
__device__ __forceinline__ void lds_row(const uint16_t* rows, uint32_t gs, uint32_t i, uint64_t& lo, uint64_t& hi) {
    hi = 0;
    if (gs == 1) {
        lo = rows[i];
    } else if (gs == 2) {
        lo = ((const uint32_t*)rows)[i];
    } else if (gs == 4) {
        lo = ((const uint64_t*)rows)[i];
    } else {
        lo = ((const uint64_t*)rows)[2 * i];
        hi = ((const uint64_t*)rows)[2 * i + 1];
    }
}
__device__ __forceinline__ void store_row(uint16_t* rows, uint32_t gs, uint32_t i, uint64_t lo, uint64_t hi) {
    if (gs == 1) {
        rows[i] = (uint16_t)lo;
    } else if (gs == 2) {
        ((uint32_t*)rows)[i] = (uint32_t)lo;
    } else if (gs == 4) {
        ((uint64_t*)rows)[i] = lo;
    } else {
        ((uint64_t*)rows)[2 * i] = lo;
        ((uint64_t*)rows)[2 * i + 1] = hi;
    }
}
// A light wavefront holds the lists of several units at once, so its filter and table are keyed by
// node and unit (< kPack).
__device__ __forceinline__ uint32_t unit_key_of(uint32_t w, uint32_t unit) { return w ^ (unit << 13); }

// ---- LDS hash table of a's list: 2-slot buckets probed linearly.  A slot holds i + 1 for the W
// entry i (13 bits) under the low 19 bits of its key; 0 = empty.  Slot 0 of a bucket fills
// before slot 1, so an empty slot ends a probe sequence.  kbits is log2 of the bucket count (at
// least the number of keys: load factor <= 1/2).
constexpr uint32_t kTagShift = 13;
__device__ __forceinline__ void hash_insert(uint32_t* table, uint32_t kbits, uint32_t key, uint32_t i) {
    const uint32_t mask = (1u << kbits) - 1u, slot = (key << kTagShift) | (i + 1u);
    uint32_t b = (key * kHashMul) >> (32 - kbits);
    for (;;) {
        if (atomicCAS(&table[2 * b], 0u, slot) == 0u) return;
        if (atomicCAS(&table[2 * b + 1], 0u, slot) == 0u) return;
        b = (b + 1u) & mask;
    }
}
// the W entry of node w among the entries [lo, hi) (of its unit), or NO_SLOT
constexpr uint32_t NO_SLOT = 0xffffffffu;
__device__ __forceinline__ uint32_t hash_find(const uint32_t* table, const uint32_t* ew, uint32_t kbits, uint32_t key,
                                              uint32_t w, uint32_t lo, uint32_t hi) {
    const uint32_t mask = (1u << kbits) - 1u, tag = key << kTagShift;
    uint32_t b = (key * kHashMul) >> (32 - kbits);
    for (;;) {
        const uint2 k2 = *(const uint2*)(table + 2 * b);
        // (an empty slot's low bits are 0, so its distance from the tag is never an index)
        const uint32_t x = k2.x - tag - 1u, y = k2.y - tag - 1u;
        if (x - lo < hi - lo && ew[x] == w) return x;
        if (y - lo < hi - lo && ew[y] == w) return y;
        if (k2.y == 0u) return NO_SLOT;
        b = (b + 1u) & mask;
    }
}

// Filter of a's list: one bit per key in a table of 2^fbits words (32 bits per key or more), tested
// for every walked entry before the exact table is looked up.  The word comes from the top bits of a
// 24-bit product (one full-rate instruction; ids above 2^24 keep their low bits, which only lets
// more candidates through), the bit from its low five: bit 31 - (h & 31), so that a test is a shift
// by h into the sign.
__device__ __forceinline__ uint32_t filt_hash(uint32_t w) { return __umul24(w, kFiltMul); }
__device__ __forceinline__ void filt_insert(uint32_t* filt, uint32_t fbits, uint32_t w) {
    const uint32_t h = filt_hash(w);
    atomicOr(&filt[h >> (32 - fbits)], 0x80000000u >> (h & 31u));
}
__device__ __forceinline__ bool filt_test(const uint32_t* filt, uint32_t fshift, uint32_t w) {
    const uint32_t h = filt_hash(w);
    const uint32_t word = *(const uint32_t*)((const uint8_t*)filt + ((h >> fshift) & ~3u));
    return (int32_t)(word << (h & 31u)) < 0;
}

// find the job owning queue position `tile` (largest j with prefix[j] <= tile)
__device__ __forceinline__ uint32_t find_job(const JobDev* jobs, uint32_t njobs, uint32_t tile, bool heavy) {
    uint32_t lo = 0, hi = njobs;
    while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) >> 1;
        const uint32_t p = heavy ? jobs[mid].heavy_prefix : jobs[mid].light_prefix;
        if (p <= tile) lo = mid; else hi = mid;
    }
    return lo;
}

// exclusive scan over the wavefront
__device__ __forceinline__ uint32_t wave_excl_scan(uint32_t v, uint32_t& total) {
    const uint32_t inc = wave_incl_scan(v);
    total = lane_val(inc, 63);
    return inc - v;
}

// sum over the team, 64-bit (the per-thread parts may exceed 32 bits together).  Within a
// wavefront the part is summed with the DPP scan, which needs no LDS permutes (unlike lane
// shuffles): in one 32-bit pass if the caller knows the wavefront's sum is below 2^32
// (`narrow`), else in three pieces of 26, 26 and 12 bits, whose 64-lane sums stay below 2^32
// and so are exact in 32 bits.
template <bool BLOCK>
__device__ __forceinline__ uint64_t team_sum64(uint64_t v, uint32_t* red, bool narrow) {
    if (narrow)
        v = wave_sum((uint32_t)v);
    else
        v = (uint64_t)wave_sum((uint32_t)v & 0x3ffffffu) + ((uint64_t)wave_sum((uint32_t)(v >> 26) & 0x3ffffffu) << 26) +
            ((uint64_t)wave_sum((uint32_t)(v >> 52)) << 52);
    if (!BLOCK) return v;
    const uint32_t lane = lane_id(), wid = threadIdx.x >> 6, nw = blockDim.x >> 6;
    uint64_t* red64 = (uint64_t*)(red + 16);  // words 16..47: up to 16 wavefronts
    if (lane == 0) red64[wid] = v;
    __syncthreads();
    uint64_t t = 0;
    for (uint32_t w = 0; w < nw; ++w) t += red64[w];
    __syncthreads();
    return t;
}

// Local counts: rows of gp 16-bit counters per staged entry, gp the group count padded to 1, 2, 4 or
// 8 (the callers flush before a counter can pass 2^16 - 1).
__device__ __forceinline__ void count16(uint16_t* cnt, uint32_t i) {
    atomicAdd((uint32_t*)cnt + (i >> 1), 1u << (16u * (i & 1u)));
}
__device__ __forceinline__ void clear_row(uint16_t* cnt, uint32_t gp, uint32_t i) {
    if (gp == 1) {
        cnt[i] = 0;
    } else if (gp == 2) {
        ((uint32_t*)cnt)[i] = 0u;
    } else if (gp == 4) {
        ((uint64_t*)cnt)[i] = 0ull;
    } else {
        ((uint64_t*)cnt)[2 * i] = 0ull;
        ((uint64_t*)cnt)[2 * i + 1] = 0ull;
    }
}
// f(group, count) for the nonzero counts of a row
template <typename F>
__device__ __forceinline__ void for_counts(const uint16_t* cnt, uint32_t gp, uint32_t i, const F& f) {
    if (gp == 1) {
        const uint32_t v = cnt[i];
        if (v) f(0u, v);
        return;
    }
    for (uint32_t h = 0; h < gp; h += 2) {
        const uint32_t v = ((const uint32_t*)cnt)[(gp * i + h) >> 1];
        if (v & 0xffffu) f(h, v & 0xffffu);
        if (v >> 16) f(h + 1u, v >> 16);
    }
}
// 16-bit field g of a slot row
template <uint32_t GS>
__device__ __forceinline__ uint32_t row_field(uint64_t lo, uint64_t hi, uint32_t g) {
    return (uint32_t)((GS == 8 && g >= 4 ? hi >> (16 * (g - 4)) : lo >> (16 * g)) & 0xffffu);
}

// A batch of up to 64 candidates, one per lane, taken off the queue: the loads of the walked edge's
// time and slots are issued when it is taken and used when it is drained, one step later.
template <uint32_t GS>
struct HitBatch {
    uint32_t n = 0;  // candidates (uniform)
    uint32_t ib, unit, w, p, t;
    uint64_t lo, hi;
};
// the queue's last `n` candidates, from index `at` on
template <uint32_t GS>
__device__ __forceinline__ void take_batch(const JobRegs& J, const WaveView& V, uint32_t at, uint32_t n, HitBatch<GS>& D) {
    const uint32_t q = at + (lane_id() < n ? lane_id() : 0u);
    const uint2 e = V.qe[q];
    D.n = n;
    const uint32_t o = V.qo[q];
    D.ib = o & 0xfffu;
    D.unit = o >> 12;
    D.p = e.x;
    D.w = e.y;
    D.t = ldg(J.tim + e.x) & ~REPT_REV_BIT;
    load_slots_t<GS>(J.tab, e.x, D.lo, D.hi);
}

// Attribute a batch.  A candidate is (B index ib, node w, list position p); it is a hit if the table
// holds w, at W entry k: the triangle (a, b = eb[ib], w = ew[k]) with times t_ab = etb[ib], t_aw =
// et[k], t_bw = tim[p].  Its first two edges by time decide the processor per group: edges at a
// have their slots staged; the slots of {b, w} come from the slot table.
// PACK: the list belongs to one of several units, a0 is not used.
template <bool ETA, bool PACK, uint32_t GS>
__device__ __forceinline__ void drain_batch(const JobRegs& J, const TeamView& T, const WaveView& V, uint32_t a0,
                                            uint32_t kbits, const HitBatch<GS>& D) {
    if (lane_id() >= D.n) return;
    const uint32_t w = D.w, ib = D.ib, p = D.p, tbw = D.t;
    const uint64_t blo = D.lo, bhi = D.hi;
    const uint32_t k = hash_find(T.table, T.ew, kbits, PACK ? unit_key_of(w, D.unit) : w, w, PACK ? T.uw0[D.unit] : 0u,
                                 PACK ? T.uw0[D.unit + 1] : T.DW);
    if (k == NO_SLOT) return;
    const uint32_t a = PACK && J.per_proc ? T.ua[D.unit] : a0;
    const uint32_t b = T.eb[ib], tab = T.etb[ib], taw = T.et[k];
    uint64_t alo, ahi, wlo, whi;
    lds_row_t<GS>(T.bslot, ib, alo, ahi);
    lds_row_t<GS>(T.wslot, k, wlo, whi);
    // which edge arrived last: 0 = {a,b}, 1 = {a,w}, 2 = {b,w} (times are distinct)
    const uint32_t last = (tab > taw && tab > tbw) ? 0u : (taw > tbw ? 1u : 2u);
    const uint32_t tl = last == 0 ? tab : (last == 1 ? taw : tbw);
    // slot rows of the first two edges; the groups where their slots agree, all at once
    const uint64_t xlo = last == 0 ? wlo : alo, xhi = last == 0 ? whi : ahi;
    const uint64_t ylo = last == 2 ? wlo : blo, yhi = last == 2 ? whi : bhi;
    if (GS == 1 && J.mask) {
        // parallel MASCOT: the processors that kept both earlier edges
        uint32_t mm = (uint32_t)(xlo & ylo) & ((1u << J.G) - 1u);
        if (!(tl >= J.t0 && tl < J.t1)) mm = 0;
        while (mm) {
            const uint32_t g = (uint32_t)__builtin_ctz(mm);  // processor g, its own group
            mm &= mm - 1u;
            if (J.use_hist) atomicAdd(&V.hist[g], 1u);
            else add64(J.jd->global + g, 1);
            if (J.per_proc) {
                int64_t* row = J.local + (uint64_t)g * J.n;
                add64(row + a, 1);
                add64(row + b, 1);
                add64(row + w, 1);
            } else {
                count16(T.cntb, J.gp * ib + g);
                count16(T.cntw, J.gp * k + g);
            }
        }
        return;
    }
    if (!(tl >= J.t0 && tl < J.t1)) return;
    // group by group: a loop over a lane's agreeing groups would run, for the whole wavefront, as
    // often as its worst lane's, with the group's counters found at run time
#pragma unroll
    for (uint32_t g = 0; g < GS; ++g) {
        if (g >= J.G) break;
        const uint32_t s1 = row_field<GS>(xlo, xhi, g), ck = (g + 1 < J.G) ? J.ck : J.last_ck;
        if (s1 == row_field<GS>(ylo, yhi, g) && s1 < ck) {
            const uint32_t proc = g * J.pstride + s1;
            if (J.use_hist) atomicAdd(&V.hist[proc], 1u);
            else add64(J.jd->global + proc, 1);
            if (J.per_proc) {
                int64_t* row = J.local + (uint64_t)proc * J.n;
                add64(row + a, 1);
                add64(row + b, 1);
                add64(row + w, 1);
            } else {
                count16(T.cntb, GS * ib + g);
                count16(T.cntw, GS * k + g);
            }
            if (ETA && J.pairs) {
                // Algorithm 2's per-edge counts (Section III-B): the first two edges gain a
                // non-last occurrence (s), the last edge a last-edge occurrence (L) when the
                // same processor stores it.  {a, w} and {a, b} are staged entries, counted in
                // LDS; {b, w} (list position p) in global memory.
                const uint32_t sl = last == 0   ? row_field<GS>(alo, ahi, g)
                                    : last == 1 ? row_field<GS>(wlo, whi, g)
                                                : row_field<GS>(blo, bhi, g);
                const uint32_t lw = sl == s1 ? (1u << 16) : 0u;  // the last edge's L step
                const uint32_t we = last == 1 ? lw : 1u;  // {a, w}: last (L) or not (s)
                const uint32_t be = last == 0 ? lw : 1u;  // {a, b}
                if (we) atomicAdd(&T.ewe[g * T.DW + k], we);
                if (be) atomicAdd(&T.ebe[g * T.DB + ib], be);
                uint32_t* cp = J.pairs + 2 * ((uint64_t)g * J.es + p);
                if (last != 2) atomicAdd(cp, 1u);
                else if (lw) atomicAdd(cp + 1, 1u);
            }
        }
    }
}

// Add the wavefront's histogram of global counts to the outputs and clear it (c counters, or none where
// c is larger than the histogram; looked up here, not per drain: R-MAT scale 24 197.6 and 198.6 ms).
__device__ __forceinline__ void flush_hist_now(const JobRegs& J, WaveView& V) {
    const uint32_t lane = lane_id(), c = J.use_hist ? J.jd->c : 0u;
    wave_sync();
    for (uint32_t p = lane; p < c; p += 64) {
        const uint32_t v = V.hist[p];
        if (v) {
            add64(J.jd->global + p, v);
            V.hist[p] = 0;
        }
    }
    V.hits = 0;
    wave_sync();
}

// A histogram counter gains at most one per drained hit (a hit is one triangle, and it is a
// semi-triangle of at most one processor per group), so it cannot pass kHistFlushHits + one
// drain's hits (< 2^32) if the histogram is flushed whenever the wavefront's hits since the
// last flush reach kHistFlushHits.
constexpr uint32_t kHistFlushHits = 1u << 31;

// drain a batch and count its candidates
template <bool ETA, bool PACK, uint32_t GS>
__device__ __forceinline__ void drain_hits(const JobRegs& J, const TeamView& T, WaveView& V, uint32_t a, uint32_t kbits,
                                           HitBatch<GS>& D, std::integral_constant<bool, PACK>) {
    drain_batch<ETA, PACK, GS>(J, T, V, a, kbits, D);
    const uint32_t h = V.hits + D.n;
    if (h >= kHistFlushHits) flush_hist_now(J, V);
    else V.hits = h;
    D.n = 0;
}

// add packed pair counts (s | L << 16) to the stored edge at adjacency position pos, group g
__device__ __forceinline__ void flush_pair(const JobRegs& J, uint32_t g, uint32_t pos, uint32_t v) {
    uint32_t* cp = J.pairs + 2 * ((uint64_t)g * J.es + pos);
    if (v & 0xffffu) atomicAdd(cp, v & 0xffffu);
    if (v >> 16) atomicAdd(cp + 1, v >> 16);
}

// popcount of the bits of `m` below this lane
__device__ __forceinline__ uint32_t lanes_below(uint64_t m) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Walk granules [0, g_end) of the staged B chunk.  A granule is up to kGran consecutive entries of
// one list: list i holds the granules bgr[i] .. bgr[i + 1) (staged lists are not empty,
// so list starts are distinct).  Granules are taken 64 at a time, one per lane: a lane's list is i0
// (the list of the batch's first granule) plus the number of list starts after the first granule
// and at or before its own.  The lanes leave (position, entries, list) in LDS; then windows of 64
// entries take kWinGran granules each, kGran lanes to a granule, so that finding an entry's list
// costs a window one LDS read.  Lanes past a granule's end load the entries that follow it (in the
// graph's buffer: the times come after the neighbours) and are masked out of the test.
// An entry that passes the filter is queued as (position, node, list); whole batches of 64 are
// looked up in the exact table and attributed by drain_hits.
// The walk is bound by memory latency: the bytes a wavefront has in flight.  So the loads of the
// next step's windows are issued before this step's are tested, and a batch's loads one step before
// it is drained.
// late(): run once after the first loads are issued (it stores what the drains need and the walk
// does not).
template <bool ETA, bool PACK, uint32_t GS, typename Late>
__device__ __forceinline__ void walk_items(const JobRegs& J, const TeamView& T, WaveView& V, uint32_t a, uint32_t kbits,
                                           uint32_t fshift, uint32_t bn, uint32_t g_end, const Late& late) {
    constexpr uint32_t kGran = PACK ? kGranLight : kGranHeavy, kWinGran = 64 / kGran;
    constexpr uint32_t kStep = PACK ? kStepLight : (ETA ? kStepEta : kStepHeavy);
    const uint32_t lane = lane_id(), sub = lane % kGran;
    const uint2* const dp = V.desc + lane / kGran;
    uint32_t qn = 0;
    uint32_t i0 = 0, g0 = 0;  // the batch of granules after the last one prepared, and its first list
    uint32_t gw = 64;         // next step's first granule within the prepared ones
    uint2 dn[kStep];
    uint32_t wn[kStep];
    HitBatch<GS> D;
    const std::integral_constant<bool, PACK> pack{};
    // prepare the next 64 granules if the prepared ones are used up, and issue a step's loads
    auto issue = [&]() {
        if (gw >= 64) {
            V.mark[lane] = 0;
            wave_sync();
            const uint32_t idx = i0 + 1 + lane;
            if (idx < bn) {
                const uint32_t st = T.bgr[idx];
                if (st - g0 < 64u) V.mark[st - g0] = 1;
            }
            wave_sync();
            const uint32_t f = V.mark[lane];
            const uint64_t bal = __ballot(f != 0);
            const uint32_t own = i0 + lanes_below(bal) + f, g = g0 + lane;
            const uint2 oe = T.bpos[own];
            const uint32_t pos = oe.x + kGran * (g - T.bgr[own]);
            const uint32_t left = g < g_end ? oe.x + (oe.y & 0xffffu) - pos : 0u;
            wave_sync();
            V.desc[lane] = make_uint2(g < g_end ? pos : 0u, (left < kGran ? left : kGran) | (own << 16) |
                                                                (PACK ? oe.y & 0xf0000000u : 0u));
            wave_sync();
            // list of the next batch's first granule
            const uint32_t last = i0 + (uint32_t)__popcll(bal), nx = last + 1;
            g0 += 64;
            i0 = (nx < bn && wave_uni(T.bgr[nx < bn ? nx : bn]) <= g0) ? nx : last;
            gw = 0;
        }
#pragma unroll
        for (uint32_t j = 0; j < kStep; ++j) {
            dn[j] = dp[gw + j * kWinGran];
            dn[j].x += sub;
            wn[j] = ldg(J.nbr + dn[j].x);
        }
        gw += kStep * kWinGran;
    };
    issue();
    late();
    for (uint32_t done = 0; done < g_end; done += kStep * kWinGran) {
        uint2 dsc[kStep];
        uint32_t w[kStep];
#pragma unroll
        for (uint32_t j = 0; j < kStep; ++j) {
            dsc[j] = dn[j];
            w[j] = wn[j];
        }
        if (done + kStep * kWinGran < g_end) issue();
#pragma unroll
        for (uint32_t j0 = 0; j0 < kStep; j0 += kWalk) {
            bool hit[kWalk];
#pragma unroll
            for (uint32_t j = 0; j < kWalk; ++j)
                hit[j] = filt_test(T.filt, fshift, PACK ? unit_key_of(w[j0 + j], dsc[j0 + j].y >> 28) : w[j0 + j]) &&
                         sub < (dsc[j0 + j].y & 0xffffu);
#pragma unroll
            for (uint32_t j = 0; j < kWalk; ++j) {
                const uint64_t hm = __ballot(hit[j]);
                if (hit[j]) {
                    const uint32_t q = qn + lanes_below(hm);
                    V.qe[q] = make_uint2(dsc[j0 + j].x, w[j0 + j]);
                    V.qo[q] = (uint16_t)(dsc[j0 + j].y >> 16);
                }
                qn += (uint32_t)__popcll(hm);
            }
            wave_sync();
            while (qn >= 64) {
                if (D.n) drain_hits<ETA>(J, T, V, a, kbits, D, pack);
                qn -= 64;
                take_batch<GS>(J, V, qn, 64, D);
                wave_sync();
            }
        }
    }
    // the batch in flight, then the rest of the queue
    for (uint32_t last = 0; last < 2; ++last) {
        if (D.n) drain_hits<ETA>(J, T, V, a, kbits, D, pack);
        if (qn) take_batch<GS>(J, V, 0, qn, D);
        qn = 0;
    }
    wave_sync();
}

// Walk one chunk of lists, one per lane, and flush its entries' counts.  The lane's list: out(b) at
// offset bo, bd entries (0: no list); tb, pab, (lo, hi): arrival time, adjacency position and slot
// row of its pair; u: its unit in a light pass.
template <bool ETA, bool PACK>
__device__ __forceinline__ void walk_chunk(const JobRegs& J, const TeamView& T, WaveView& V, uint32_t a, uint32_t kbits,
                                           uint32_t fshift, uint32_t b, uint32_t bo, uint32_t bd, uint32_t tb,
                                           uint32_t pab, uint32_t u, uint64_t lo, uint64_t hi) {
    constexpr uint32_t kGran = PACK ? kGranLight : kGranHeavy;
    uint32_t nb, grans;  // lists and granules
    const uint32_t pos = wave_excl_scan(bd ? 1u : 0u, nb);
    const uint32_t sc = wave_excl_scan((bd + kGran - 1u) / kGran, grans);
    if (!nb) return;
    if (bd) {
        T.eb[pos] = b;
        T.etb[pos] = tb;
        T.bpos[pos] = make_uint2(bo, PACK ? bd | (u << 28) : bd);
        T.bgr[pos] = sc;
        clear_row(T.cntb, J.gp, pos);
        if (ETA)
            for (uint32_t g = 0; g < J.G; ++g) T.ebe[g * T.DB + pos] = 0;
    }
    wave_sync();
    // the slot rows, needed only by the drains, are stored once the walk's first loads are on their way
    auto late = [&]() {
        if (bd) store_row(T.bslot, J.gs, pos, lo, hi);
        wave_sync();
    };
    if (J.gs == 1) walk_items<ETA, PACK, 1>(J, T, V, a, kbits, fshift, nb, grans, late);
    else if (J.gs == 2) walk_items<ETA, PACK, 2>(J, T, V, a, kbits, fshift, nb, grans, late);
    else if (J.gs == 4) walk_items<ETA, PACK, 4>(J, T, V, a, kbits, fshift, nb, grans, late);
    else walk_items<ETA, PACK, 8>(J, T, V, a, kbits, fshift, nb, grans, late);
    if (bd) {
        if (!J.per_proc) {
            const uint32_t hs = hub_slot(V.hub, b);
            for_counts(T.cntb, J.gp, pos, [&](uint32_t g, uint32_t v) { add_local(J.local, J.n, V.hub, hs, g, b, v); });
        }
        // this chunk's pair counts of the B entries: at most one per W entry each
        if (ETA && J.pairs)
            for (uint32_t g = 0; g < J.G; ++g) {
                const uint32_t v = T.ebe[g * T.DB + pos];
                if (v) flush_pair(J, g, pab, v);
            }
    }
    wave_sync();
}

// Apexes with this many out-neighbours and more have long lists to walk (the b's rank above a), so
// that a chunk's walk outlasts the taking of it: their chunks shrink to kChunkMin lists towards the
// unit's end, so that its wavefronts end together.  Below it the smaller chunks cost more than the
// wait: with every unit split so, R-MAT scale 24 gains the same 6% (209.7 to 197.7 ms), but the
// 20M-edge power law loses 1.2% (7.84 to 7.94 ms) and 32 jobs of 500k edges 3% (1.17 to 1.21 ms);
// from 384 on, 209.7 to 199.7 ms and neither of the others moves.
constexpr uint32_t kLong = 384, kChunkMin = 16;
constexpr uint32_t kRoundLists = 1u << 15;  // lists walked between flushes of the W entries' counts

// Count every triangle whose lowest-ranked node is a.  The team is the workgroup (BLOCK) or
// this wavefront.  a's list is hashed into LDS in chunks of DW entries (W side); for each W
// chunk the unit's lists are walked in chunks of up to DB lists (B side), each by one wavefront of
// the team: the wavefronts take chunks from a counter and share nothing but the W side, so they
// meet only before the first chunk and after the last.
// (s, d): offset and length of a's list; (r0, rn): offset and length of a's reverse list.  Only the
// lists [e0, e1) of the unit's d + rn are walked (a part of the unit; counts add over parts).
// ahead(): run once by the team's last wavefront after the list is staged, while the others start on
// the chunks (a workgroup claims its next tile there).
template <bool BLOCK, bool ETA, typename Ahead>
__device__ __forceinline__ void count_apex(const JobRegs& J, const TeamView& T, WaveView& V, uint32_t a, uint32_t s,
                                           uint32_t d, uint32_t r0, uint32_t rn, uint32_t e0, uint32_t e1,
                                           const Ahead& ahead) {
    const uint32_t nt = BLOCK ? blockDim.x : 64, lane = lane_id();
    const uint32_t tid = BLOCK ? threadIdx.x : lane;
    const uint32_t nw = nt >> 6;
    const uint32_t nbtot = d + rn;
    const uint32_t G = J.G;
    uint32_t *const next = T.red + 63, *const nown = T.red + 62;  // the team's next chunk; own lists
    // B lists: first those of a's own pairs a -> b whose out(b) is not longer than out(a) (walk
    // out(b)), then the reverse pairs y -> a with out(y) shorter than out(a) (walk out(y)): every
    // triangle is found once, from its lowest pair, walking the shorter list.  The own pairs are
    // picked while a's list is staged, if that is all at once.
    const bool whole = d <= T.DW;
    const uint32_t o0 = e0 < d ? e0 : d, o1 = e1 < d ? e1 : d;  // own entries [o0, o1) of this part
    const uint32_t rb = r0 + (e0 > d ? e0 - d : 0u), nr = (e1 - e0) - (o1 - o0);
    for (uint32_t ws = 0; ws < d; ws += T.DW) {
        const uint32_t wn = (d - ws) < T.DW ? (d - ws) : T.DW;
        // the whole table (sized for DW keys) is used whatever wn is: a sparser table ends more
        // probes at their first bucket
        const uint32_t slots = pow2_at_least(2 * T.DW), kbits = log2u(slots) - 1;
        const uint32_t fwords = pow2_at_least(T.DW), fbits = log2u(fwords), fshift = 30 - fbits;
        for (uint32_t i = tid; i < slots; i += nt) T.table[i] = 0;
        for (uint32_t i = tid; i < fwords; i += nt) T.filt[i] = 0;
        if (tid == 0) *nown = 0;
        team_sync<BLOCK>();
        for (uint32_t i = tid; i < wn; i += nt) {
            const uint32_t w = ldg(J.nbr + s + ws + i), t = ldg(J.tim + s + ws + i);
            uint64_t lo, hi;
            load_slots(J.tab, J.gs, s + ws + i, lo, hi);
            T.ew[i] = w;
            T.et[i] = t & ~REPT_REV_BIT;
            const bool own = whole && !(t & REPT_REV_BIT) && i >= o0 && i < o1;
            const uint64_t bal = __ballot(own);
            uint32_t at = 0;
            if (lane == 0 && bal) at = atomicAdd(nown, (uint32_t)__popcll(bal));
            at = lane_val(at, 0);
            if (own) T.ownl[at + lanes_below(bal)] = (uint16_t)i;
            store_row(T.wslot, J.gs, i, lo, hi);
            clear_row(T.cntw, J.gp, i);
            if (ETA)
                for (uint32_t g = 0; g < G; ++g) T.ewe[g * T.DW + i] = 0;
            filt_insert(T.filt, fbits, w);
            hash_insert(T.table, kbits, w, i);
        }
        if (BLOCK && tid == 0) *next = 0;
        team_sync<BLOCK>();
        if (BLOCK && ws == 0 && (threadIdx.x >> 6) == nw - 1u) ahead();
        const uint32_t no = whole ? wave_uni(*nown) : o1 - o0, lists = no + nr;
        // Lists per chunk: a few lists are spread over all wavefronts, 16 to a chunk at least; under a
        // long apex (kLong), half a wavefront's share of what is left
        const uint32_t even = ((lists + nw - 1u) / nw + 15u) & ~15u;
        // A W entry's 16-bit counts gain at most one per list, so they are flushed every kRoundLists.
        for (uint32_t es = 0; es < lists; ) {
            const uint32_t ee = lists - es > kRoundLists ? es + kRoundLists : lists;
            if (es) {
                if (BLOCK && tid == 0) *next = 0;
                team_sync<BLOCK>();
            }
            for (uint32_t at = es;;) {
                uint32_t db = T.DB;  // (at most 64: one list per lane)
                if (BLOCK) {
                    if (lane == 0) {
                        db = even;
                        if (d >= kLong) {
                            const uint32_t seen = *(volatile uint32_t*)next, all = ee - es;
                            db = (all > seen ? all - seen : 0u) / (2u * nw);
                            db = db < kChunkMin ? kChunkMin : db;
                        }
                        db = db < T.DB ? db : T.DB;
                        at = es + atomicAdd(next, db);
                    }
                    at = lane_val(at, 0);
                    db = lane_val(db, 0);
                }
                if (at >= ee) break;
                const uint32_t x = at + lane;
                if (!BLOCK) at += db;
                uint32_t b = 0, bo = 0, bd = 0, tb = 0, pab = 0;
                uint64_t lo = 0, hi = 0;
                if (lane < db && x < ee) {
                    if (x < no) {
                        if (whole) {
                            const uint32_t i = T.ownl[x];
                            b = T.ew[i];
                            tb = T.et[i];
                            pab = s + i;
                            lds_row(T.wslot, J.gs, i, lo, hi);
                        } else {
                            pab = s + o0 + x;
                            tb = ldg(J.tim + pab);
                            b = ldg(J.nbr + pab);
                            load_slots(J.tab, J.gs, pab, lo, hi);
                        }
                        if (!(tb & REPT_REV_BIT)) {  // (else out(a) is shorter: counted at b)
                            bo = ldg(J.off + b);
                            bd = ldg(J.off + b + 1) - bo;
                        }
                    } else {
                        const uint32_t q = rb + (x - no);
                        const uint4 r = J.rrec[q];
                        pab = ldg(J.rpos + q);
                        b = r.x;
                        tb = r.y;
                        bo = r.z;
                        bd = r.w;
                        load_slots(J.tab, J.gs, pab, lo, hi);
                    }
                }
                walk_chunk<ETA, false>(J, T, V, a, kbits, fshift, b, bo, bd, tb, pab, 0u, lo, hi);
            }
            team_sync<BLOCK>();
            if (ETA && J.pairs) {
                for (uint32_t x = tid; x < G * wn; x += nt) {
                    const uint32_t g = x / wn, i = x - g * wn;
                    const uint32_t v = T.ewe[g * T.DW + i];
                    if (v) {
                        flush_pair(J, g, s + ws + i, v);
                        T.ewe[g * T.DW + i] = 0;
                    }
                }
            }
            if (!J.per_proc) {
                // flush the w-side counts; their sum per group is a's own count for this chunk.  A W
                // entry gains at most one per list walked against it, so that sum is at most
                // wn * nbtot: a light unit's is below 2^32 and one 32-bit pass sums it.  A team of a
                // heavy unit always takes the three-piece sum (a few instructions per unit there), so
                // every graph with heavy and light units runs both forms.
                const bool narrow = !BLOCK && (uint64_t)wn * nbtot < (1ull << 32);
                for (uint32_t g = 0; g < G; ++g) {
                    uint64_t part = 0;
                    for (uint32_t i = tid; i < wn; i += nt) {
                        const uint32_t v = T.cntw[J.gp * i + g];
                        if (v) {
                            const uint32_t w = T.ew[i];
                            add_local(J.local, J.n, V.hub, hub_slot(V.hub, w), g, w, v);
                            part += v;
                            if (ee < e1) T.cntw[J.gp * i + g] = 0;
                        }
                    }
                    const uint64_t tot = team_sum64<BLOCK>(part, T.red, narrow);
                    if (tid == 0 && tot) add64(J.local + (uint64_t)g * J.n + a, tot);
                }
            }
            es = ee;
        }
        team_sync<BLOCK>();
    }
}

// Unit of entry i0 + lane of a pass whose units start at start[0..k) (start[0] = 0, increasing: every
// unit has entries): the number of starts at or before it, less one.
__device__ __forceinline__ uint32_t pass_unit(const uint32_t* start, uint32_t k, uint32_t i0, const WaveView& V) {
    const uint32_t lane = lane_id();
    V.mark[lane] = 0;
    wave_sync();
    const uint32_t st = lane < k ? start[lane] : 0xffffffffu;
    if (st - i0 < 64u) V.mark[st - i0] = 1;
    const uint32_t before = (uint32_t)__popcll(__ballot(st < i0));
    wave_sync();
    const uint32_t f = V.mark[lane];
    const uint32_t u = before + lanes_below(__ballot(f != 0)) + f - 1u;
    wave_sync();
    return u;
}

// Count several light units in one pass of a wavefront: lanes [f, f + k) hold their nodes `ta`, list
// offsets and lengths `ts`, `td` and reverse-list offsets and lengths `tr`, `trn`, with at most T.DW
// list entries together (wpre: those before the lane's, from lane f on).  A light unit is too small
// to fill the wavefront, and counting it is a chain of dependent loads (its list, the lists'
// bounds, their entries, the candidates' times); a pass pays the chain once for all its units, in
// fuller steps.  The units' entries and lists are concatenated; filter and table are keyed by
// (node, unit).
template <bool ETA>
__device__ __forceinline__ void count_pack(const JobRegs& J, const TeamView& T, WaveView& V, uint32_t f, uint32_t k,
                                           uint32_t ta, uint32_t ts, uint32_t td, uint32_t tr, uint32_t trn,
                                           uint32_t wpre) {
    const uint32_t lane = lane_id(), G = J.G;
    const bool mine = lane >= f && lane < f + k;
    uint32_t nr;  // reverse lists
    const uint32_t rpre = wave_excl_scan(mine ? trn : 0u, nr);
    if (mine) {
        T.uw0[lane - f] = wpre;
        T.ul0[lane - f] = rpre;
        T.us[lane - f] = ts;
        T.ur0[lane - f] = tr;
        T.ua[lane - f] = ta;
    }
    const uint32_t wn = lane_val(wpre + td, f + k - 1);
    if (lane == 0) {
        T.uw0[k] = wn;
        T.ul0[k] = nr;
    }
    for (uint32_t x = lane; x < G * kPack; x += 64) T.uown[x] = 0;
    const uint32_t slots = pow2_at_least(2 * T.DW), kbits = log2u(slots) - 1;
    const uint32_t fwords = pow2_at_least(T.DW), fbits = log2u(fwords), fshift = 30 - fbits;
    for (uint32_t i = lane; i < slots; i += 64) T.table[i] = 0;
    for (uint32_t i = lane; i < fwords; i += 64) T.filt[i] = 0;
    wave_sync();
    uint32_t no = 0;  // own lists
    for (uint32_t i0 = 0; i0 < wn; i0 += 64) {
        const uint32_t i = i0 + lane, u = pass_unit(T.uw0, k, i0, V);
        bool own = false;
        if (i < wn) {
            const uint32_t p = T.us[u] + (i - T.uw0[u]);
            const uint32_t w = ldg(J.nbr + p), t = ldg(J.tim + p);
            uint64_t lo, hi;
            load_slots(J.tab, J.gs, p, lo, hi);
            T.ew[i] = w;
            T.et[i] = t & ~REPT_REV_BIT;
            own = !(t & REPT_REV_BIT);
            store_row(T.wslot, J.gs, i, lo, hi);
            clear_row(T.cntw, J.gp, i);
            if (ETA)
                for (uint32_t g = 0; g < G; ++g) T.ewe[g * T.DW + i] = 0;
            filt_insert(T.filt, fbits, unit_key_of(w, u));
            hash_insert(T.table, kbits, unit_key_of(w, u), i);
        }
        const uint64_t bal = __ballot(own);
        if (own) T.ownl[no + lanes_below(bal)] = (uint16_t)(i | (u << 12));
        no += (uint32_t)__popcll(bal);
    }
    wave_sync();
    const uint32_t lists = no + nr, db = T.DB;
    for (uint32_t bs = 0; bs < lists; bs += db) {
        const uint32_t x = bs + lane;
        uint32_t u = 0, b = 0, bo = 0, bd = 0, tb = 0, pab = 0;
        uint64_t lo = 0, hi = 0;
        if (lane < db && x < lists) {
            if (x < no) {
                const uint32_t o = T.ownl[x], i = o & 0xfffu;
                u = o >> 12;
                b = T.ew[i];
                tb = T.et[i];
                pab = T.us[u] + (i - T.uw0[u]);
                lds_row(T.wslot, J.gs, i, lo, hi);
                bo = ldg(J.off + b);
                bd = ldg(J.off + b + 1) - bo;
            } else {
                // the unit: the last whose first reverse list is at or before this one
                uint32_t last = k;
                while (last - u > 1) {
                    const uint32_t mid = (u + last) >> 1;
                    if (T.ul0[mid] <= x - no) u = mid; else last = mid;
                }
                const uint32_t q = T.ur0[u] + (x - no - T.ul0[u]);
                const uint4 r = J.rrec[q];
                pab = ldg(J.rpos + q);
                b = r.x;
                tb = r.y;
                bo = r.z;
                bd = r.w;
                load_slots(J.tab, J.gs, pab, lo, hi);
            }
        }
        walk_chunk<ETA, true>(J, T, V, 0u, kbits, fshift, b, bo, bd, tb, pab, u, lo, hi);
    }
    // the w-side counts (at most one per list of the unit each); their sum per group and unit is the
    // unit's own count (below 2^32: at most its entries times its lists)
    for (uint32_t i0 = 0; i0 < wn; i0 += 64) {
        const uint32_t i = i0 + lane, u = pass_unit(T.uw0, k, i0, V);
        if (i < wn) {
            const uint32_t w = T.ew[i], hs = hub_slot(V.hub, w);
            if (!J.per_proc)
                for_counts(T.cntw, J.gp, i, [&](uint32_t g, uint32_t v) {
                    add_local(J.local, J.n, V.hub, hs, g, w, v);
                    atomicAdd(&T.uown[g * kPack + u], v);
                });
            if (ETA && J.pairs)  // a W entry gains at most one per list of its unit: 16 bits each suffice
                for (uint32_t g = 0; g < G; ++g) {
                    const uint32_t v = T.ewe[g * T.DW + i];
                    if (v) flush_pair(J, g, T.us[u] + (i - T.uw0[u]), v);
                }
        }
    }
    wave_sync();
    if (!J.per_proc)
        for (uint32_t x = lane; x < G * kPack; x += 64) {
            const uint32_t v = T.uown[x];
            if (v) add64(J.local + (uint64_t)(x / kPack) * J.n + T.ua[x % kPack], v);
        }
    wave_sync();
}

__device__ __forceinline__ void flush_hist(const JobRegs& J, WaveView& V, int cur) {
    if (cur < 0 || !J.use_hist) return;
    flush_hist_now(J, V);
}

// ======================================================================= setup / zero ====

// Slot table of each job whose launch writes it: tab[p * gs + k] = h_k of the edge stored at
// position p, i.e. {b, nbr[p]} for the node b whose list holds p (Section III-A's hash, one
// independent function per group as in Section III-B).  Grid (X, njobs) of 256 threads.  A
// workgroup takes FILL_CHUNK consecutive positions (so a range of long lists is spread over
// many workgroups), finds the nodes owning its first and last positions, stages the offsets of
// that node range in LDS, FILL_NODES at a time, and hashes one position per thread (coalesced),
// finding each position's node by binary search over the staged offsets.
constexpr uint32_t FILL_CHUNK = 4096;
constexpr uint32_t FILL_NODES = 1024;

// the node whose list holds position p (the largest b < n with off[b] <= p), for p < off[n]:
// each round samples the candidate node range at 256 evenly spaced nodes, one per thread, and
// keeps the interval between the last sample at or below p and the next
__device__ uint32_t fill_owner(const uint32_t* off, uint32_t n, uint32_t p) {
    uint32_t L = 0, R = n;  // off[L] <= p < off[R]
    while (R - L > 1) {
        const uint32_t step = (R - L + 255u) / 256u;
        const uint32_t b = L + threadIdx.x * step;
        const uint32_t k = (uint32_t)__syncthreads_count(b < R && ldg(off + b) <= p);  // >= 1
        const uint32_t L2 = L + (k - 1u) * step;
        R = (L2 + step) < R ? (L2 + step) : R;
        L = L2;
    }
    return L;
}

// Everything a counting launch needs done before it, for one job (256 threads, gridDim.x
// workgroups): its outputs cleared if it overwrites them, its slot table written if it asks for it.
__device__ void prepare_job(const JobDev& J) {
    __shared__ uint32_t so[FILL_NODES + 1];
    if (!J.accumulate) {
        const uint64_t nglob = J.c, nloc = (uint64_t)J.rows * J.n, stride = (uint64_t)gridDim.x * blockDim.x;
        for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nglob + nloc; i += stride) {
            if (i < nglob) J.global[i] = 0;
            else J.local[i - nglob] = 0;
        }
    }
    if (!J.fill) return;
    const uint32_t G = J.G, gs = J.gs, m = J.m, n = J.n;
    const uint32_t* __restrict__ off = J.off;
    const uint32_t* __restrict__ nbr = J.nbr;
    uint16_t* __restrict__ tab = J.tab;
    uint64_t cf[4 * REPT_GMAX];  // coefficients read once (the table stores cannot change them)
#pragma unroll
    for (uint32_t i = 0; i < 4 * REPT_GMAX; ++i) cf[i] = i < 4 * G ? J.hp[i] : 0;
    const uint32_t Es = ldg(off + n);
    // a small graph's positions are spread over the whole grid, 256 per workgroup at least
    const uint32_t even = (((Es + gridDim.x - 1u) / gridDim.x) + 255u) & ~255u;
    const uint32_t chunk = even < 256u ? 256u : (even < FILL_CHUNK ? even : FILL_CHUNK);
    for (uint64_t c0 = (uint64_t)blockIdx.x * chunk; c0 < Es; c0 += (uint64_t)gridDim.x * chunk) {
        const uint32_t p0 = (uint32_t)c0, p1 = (c0 + chunk) < Es ? (uint32_t)(c0 + chunk) : Es;
        const uint32_t bf = fill_owner(off, n, p0), bl = fill_owner(off, n, p1 - 1u);
        for (uint32_t w0 = bf; w0 <= bl; w0 += FILL_NODES) {
            const uint32_t cnt = (bl + 1u - w0) < FILL_NODES ? (bl + 1u - w0) : FILL_NODES;
            __syncthreads();  // the previous window's offsets are no longer read
            for (uint32_t i = threadIdx.x; i <= cnt; i += 256u) so[i] = ldg(off + w0 + i);
            __syncthreads();
            const uint32_t q0 = so[0] > p0 ? so[0] : p0, q1 = so[cnt] < p1 ? so[cnt] : p1;
            for (uint32_t p = q0 + threadIdx.x; p < q1; p += 256u) {
                uint32_t lo = 0, hi = cnt;  // so[lo] <= p < so[hi]
                while (hi - lo > 1) {
                    const uint32_t mid = (lo + hi) >> 1;
                    if (so[mid] <= p) lo = mid; else hi = mid;
                }
                const uint32_t b = w0 + lo, w = ldg(nbr + p);
                uint32_t wd[4] = {0u, 0u, 0u, 0u};
                if (J.mask) {  // parallel MASCOT: bit g = processor g keeps the edge (h_g = 0)
#pragma unroll
                    for (uint32_t g = 0; g < REPT_GMAX; ++g)
                        if (g < G) wd[0] |= (slot_of(cf + 4 * g, m, b, w) == 0u ? 1u : 0u) << g;
                } else {
#pragma unroll
                    for (uint32_t g = 0; g < REPT_GMAX; ++g)
                        if (g < G) wd[g >> 1] |= slot_of(cf + 4 * g, m, b, w) << (16 * (g & 1));
                }
                if (gs == 1) tab[p] = (uint16_t)wd[0];
                else if (gs == 2) ((uint32_t*)tab)[p] = wd[0];
                else if (gs == 4) ((uint2*)tab)[p] = make_uint2(wd[0], wd[1]);
                else ((uint4*)tab)[p] = make_uint4(wd[0], wd[1], wd[2], wd[3]);
            }
        }
    }
}

__device__ __forceinline__ void reset_queues(BatchHeader* hdr) {
    for (uint32_t i = threadIdx.x; i < kQueues * kQueueStride; i += blockDim.x) hdr->queues[i] = 0u;
}

// One launch before the counting kernel: grid (workgroups per job, njobs).  The single-job form
// takes its shape and job by value and writes them to the control block that k_count reads.
__global__ void __launch_bounds__(256) k_prep(BatchHeader* hdr, const JobDev* __restrict__ jobs) {
    if (blockIdx.x == 0 && blockIdx.y == 0) reset_queues(hdr);
    const JobDev job = jobs[blockIdx.y];  // (a copy: the stores below cannot change it)
    prepare_job(job);
}
__global__ void __launch_bounds__(256) k_prep_one(uint8_t* ctrl, BatchShape shape, JobDev job) {
    if (blockIdx.x == 0) {
        BatchHeader* hdr = (BatchHeader*)ctrl;
        reset_queues(hdr);
        if (threadIdx.x == 0) {
            *(BatchShape*)hdr = shape;
            *(JobDev*)(ctrl + sizeof(BatchHeader)) = job;
        }
    }
    prepare_job(job);
}

// Algorithm 2's triangle-pair counts from the per-edge counters (Section III-B).  For a stored
// edge g of processor i (group k, slot h_k(g)): s = semi-triangles of i with g as a non-last
// edge, L = those with g as the last edge.  The definition of eta^(i) counts C(s, 2) pairs at
// g; Algorithm 2 as printed, whose counter starts at |N| when g is inserted, counts
// s L + C(s, 2).  Both go to eta[0][i], eta[1][i]; each edge's share also goes to both of its
// endpoints in eta_v[0][.], eta_v[1][.] (summed over processors).  Work split as in prepare_job.
// 16 wavefronts to a chunk: with four, the 489 chunks of 2M edges keep two wavefronts per SIMD in
// flight on a chain of 16 dependent loads and probes each (149 us, now 121; the rest is the searches
// for the chunk's first and last node and the atomics of the largest nodes).
constexpr uint32_t ETA_THREADS = 1024;
constexpr uint32_t ETA_LDS_PROCS = 512;  // processors accumulated in LDS per workgroup
constexpr uint32_t ETA_HASH = 1024;      // neighbour shares aggregated per workgroup (open addressing)
constexpr uint32_t ETA_PROBES = 16;      // probes before a share goes to global memory directly
__global__ void __launch_bounds__(ETA_THREADS) k_eta(const uint32_t* __restrict__ off, const uint32_t* __restrict__ nbr,
                                             uint32_t n, const uint16_t* __restrict__ tab, uint32_t gs, uint32_t G,
                                             uint32_t m, uint32_t c, const uint32_t* __restrict__ pairs, uint32_t es,
                                             uint32_t proc0, uint32_t stride,
                                             int64_t* __restrict__ eta, int64_t* __restrict__ eta_v) {
    __shared__ uint32_t so[FILL_NODES + 1];
    __shared__ unsigned long long acc[2][ETA_LDS_PROCS];
    __shared__ unsigned long long own[2][FILL_NODES];  // shares of the owners in the node window
    __shared__ uint32_t hkey[ETA_HASH];                 // neighbour id + 1, 0 = empty
    __shared__ unsigned long long hval[2][ETA_HASH];
    const bool in_lds = c <= ETA_LDS_PROCS;
    for (uint32_t i = threadIdx.x; i < ETA_LDS_PROCS; i += ETA_THREADS) acc[0][i] = acc[1][i] = 0ull;
    for (uint32_t i = threadIdx.x; i < ETA_HASH; i += ETA_THREADS) {
        hkey[i] = 0u;
        hval[0][i] = hval[1][i] = 0ull;
    }
    const uint32_t Es = ldg(off + n);
    for (uint64_t c0 = (uint64_t)blockIdx.x * FILL_CHUNK; c0 < Es; c0 += (uint64_t)gridDim.x * FILL_CHUNK) {
        const uint32_t p0 = (uint32_t)c0, p1 = (c0 + FILL_CHUNK) < Es ? (uint32_t)(c0 + FILL_CHUNK) : Es;
        const uint32_t bf = fill_owner(off, n, p0), bl = fill_owner(off, n, p1 - 1u);
        for (uint32_t w0 = bf; w0 <= bl; w0 += FILL_NODES) {
            const uint32_t cnt = (bl + 1u - w0) < FILL_NODES ? (bl + 1u - w0) : FILL_NODES;
            __syncthreads();
            for (uint32_t i = threadIdx.x; i <= cnt; i += ETA_THREADS) so[i] = ldg(off + w0 + i);
            for (uint32_t i = threadIdx.x; i < cnt; i += ETA_THREADS) own[0][i] = own[1][i] = 0ull;
            __syncthreads();
            const uint32_t q0 = so[0] > p0 ? so[0] : p0, q1 = so[cnt] < p1 ? so[cnt] : p1;
            for (uint32_t p = q0 + threadIdx.x; p < q1; p += ETA_THREADS) {
                unsigned long long fd = 0, fl = 0;
                for (uint32_t k = 0; k < G; ++k) {
                    const uint64_t w2 = ldg((const uint64_t*)pairs + (uint64_t)k * es + p);  // (s, L)
                    const uint32_t sx = (uint32_t)w2, ly = (uint32_t)(w2 >> 32);
                    const uint32_t slot = ldg(tab + (uint64_t)p * gs + k);
                    // an edge counts only for an active processor (inactive slots stay at zero)
                    if (sx == 0 || k * m + slot >= c) continue;
                    const unsigned long long d = (unsigned long long)sx * (sx - 1u) / 2u;
                    const unsigned long long l = d + (unsigned long long)sx * ly;
                    const uint32_t proc = k * m + slot;
                    if (in_lds) {
                        atomicAdd(&acc[0][proc], d);
                        atomicAdd(&acc[1][proc], l);
                    } else {
                        atomicAdd((unsigned long long*)eta + proc0 + proc, d);
                        atomicAdd((unsigned long long*)eta + stride + proc0 + proc, l);
                    }
                    fd += d;
                    fl += l;
                }
                if (eta_v && (fd | fl)) {
                    uint32_t lo = 0, hi = cnt;  // so[lo] <= p < so[hi]
                    while (hi - lo > 1) {
                        const uint32_t mid = (lo + hi) >> 1;
                        if (so[mid] <= p) lo = mid; else hi = mid;
                    }
                    atomicAdd(&own[0][lo], fd);  // the owner a = w0 + lo
                    atomicAdd(&own[1][lo], fl);
                    // the neighbour b: its slot in the workgroup's table, or global memory
                    const uint32_t b = ldg(nbr + p), key = b + 1u;
                    uint32_t h = (b * kHashMul) >> (32 - 10), probes = 0;
                    bool done = false;
                    for (; probes < ETA_PROBES; ++probes, h = (h + 1u) & (ETA_HASH - 1u)) {
                        const uint32_t cur = hkey[h];
                        if (cur == key || (cur == 0u && atomicCAS(&hkey[h], 0u, key) == 0u) || hkey[h] == key) {
                            atomicAdd(&hval[0][h], fd);
                            atomicAdd(&hval[1][h], fl);
                            done = true;
                            break;
                        }
                    }
                    if (!done) {
                        atomicAdd((unsigned long long*)eta_v + b, fd);
                        atomicAdd((unsigned long long*)eta_v + n + b, fl);
                    }
                }
            }
            __syncthreads();
            if (eta_v) {
                for (uint32_t i = threadIdx.x; i < cnt; i += ETA_THREADS) {
                    if (own[0][i]) atomicAdd((unsigned long long*)eta_v + w0 + i, own[0][i]);
                    if (own[1][i]) atomicAdd((unsigned long long*)eta_v + n + w0 + i, own[1][i]);
                }
            }
        }
        // the neighbour shares of this run of positions
        __syncthreads();
        if (eta_v) {
            for (uint32_t i = threadIdx.x; i < ETA_HASH; i += ETA_THREADS) {
                const uint32_t key = hkey[i];
                if (key) {
                    if (hval[0][i]) atomicAdd((unsigned long long*)eta_v + (key - 1u), hval[0][i]);
                    if (hval[1][i]) atomicAdd((unsigned long long*)eta_v + n + (key - 1u), hval[1][i]);
                    hkey[i] = 0u;
                    hval[0][i] = hval[1][i] = 0ull;
                }
            }
        }
    }
    __syncthreads();
    if (in_lds) {
        for (uint32_t i = threadIdx.x; i < c; i += ETA_THREADS) {
            if (acc[0][i]) atomicAdd((unsigned long long*)eta + proc0 + i, acc[0][i]);
            if (acc[1][i]) atomicAdd((unsigned long long*)eta + stride + proc0 + i, acc[1][i]);
        }
    }
}

// zero n 32-bit words (a kernel rather than a memset, so the sequence stays capture-safe)
__global__ void k_zero_u32(uint32_t* p, uint64_t words) {
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < words; i += (uint64_t)gridDim.x * blockDim.x)
        p[i] = 0u;
}

// ======================================================================= count kernel ====

// Claim the next tile of a phase's queue (counters at ctr[q * kQueueStride]; called by a whole
// wavefront, uniform result).  Tiles below `base` went out without a claim, one per team; the rest
// are claimed from the caller's sub-queue `q` until it is exhausted, then from the next one that is
// not.  `done` marks the sub-queues known to be exhausted: finding one so, the wavefront reads all
// counters at once, so that the end of the kernel costs a team one such look rather than a failing
// claim per sub-queue.  Returns `total` when every sub-queue is exhausted.
__device__ __forceinline__ uint32_t claim_tile(uint32_t* ctr, uint32_t base, uint32_t total, uint32_t& q, uint32_t& done) {
    const uint32_t lane = lane_id(), dyn = total > base ? total - base : 0u;
    constexpr uint32_t kAll = (1u << kQueues) - 1u;
    if (dyn == 0) return total;
    while (done != kAll) {
        const uint32_t cnt = dyn > q ? (dyn - q + kQueues - 1u) / kQueues : 0u;  // tiles of sub-queue q
        uint32_t k = cnt;
        if (cnt && lane == 0) k = atomicAdd(&ctr[q * kQueueStride], 1u);
        k = lane_val(k, 0);
        if (k < cnt) return base + q + kQueues * k;
        uint32_t seen = 0, have = 0;
        if (lane < kQueues) {
            seen = __hip_atomic_load(&ctr[lane * kQueueStride], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            have = dyn > lane ? (dyn - lane + kQueues - 1u) / kQueues : 0u;
        }
        done |= ((uint32_t)__ballot(seen >= have) & kAll) | (1u << q);
        const uint32_t open = ~done & kAll, up = q + 1u < kQueues ? open >> (q + 1u) : 0u;
        if (open) q = up ? q + 1u + (uint32_t)__builtin_ctz(up) : (uint32_t)__builtin_ctz(open);
    }
    return total;
}

// Unit and part of tile t of a queue whose units of at least 2^k parts number cls[k] (cls[0]: all
// of the queue's, descending in k; the units of most parts come first).  Returns k; for k = 0 the
// unit is the tile's position among the units of one part.
__device__ __forceinline__ uint32_t tile_part(const uint32_t* cls, uint32_t classes, uint32_t t, uint32_t& first,
                                              uint32_t& unit, uint32_t& part) {
    uint32_t more = 0;  // units of more parts
    for (uint32_t k = classes - 1; k > 0; --k) {
        const uint32_t c = cls[k];
        const uint32_t tiles = (c - more) << k;
        if (t < tiles) {
            first = more;
            unit = t >> k;
            part = t & ((1u << k) - 1u);
            return k;
        }
        t -= tiles;
        more = c;
    }
    first = more;
    unit = t;
    part = 0;
    return 0;
}

// Tile t of a light queue: units [first, first + count) of the job's light units, or part `part` of
// 2^k of one unit
__device__ __forceinline__ uint32_t light_tile_of(const uint32_t* cls, uint32_t t, uint32_t& first, uint32_t& count,
                                                  uint32_t& part) {
    uint32_t more = 0;  // units of higher classes
    for (uint32_t i = kLightClasses - 1; i > kLightOne; --i) {
        const uint32_t c = cls[i], k = i - kLightOne, tiles = (c - more) << k;
        if (t < tiles) {
            first = more + (t >> k);
            count = 1;
            part = t & ((1u << k) - 1u);
            return k;
        }
        t -= tiles;
        more = c;
    }
    part = 0;
    for (uint32_t q = 0; q < kLightOne; ++q) {
        const uint32_t c = cls[kLightOne - q], tiles = (c - more + (1u << q) - 1u) >> q;
        if (t < tiles) {
            first = more + (t << q);
            count = (c - first) < (1u << q) ? c - first : 1u << q;
            return 0;
        }
        t -= tiles;
        more = c;
    }
    first = more + (t << kLightOne);
    count = (cls[0] - first) < (1u << kLightOne) ? cls[0] - first : 1u << kLightOne;
    return 0;
}

// ETA: the form that also counts Algorithm 2's per-edge pair counters for jobs that ask for
// them (a separate instance, so the plain kernel's registers are not spent on them)
// phases: 1 the heavy phase, 2 the light phase, 3 both (one launch).  An instance each: the light
// phase's registers then do not hold the heavy team's, and more of its wavefronts fit a CU.
template <bool ETA, uint32_t phases>
__global__ void __launch_bounds__(phases == 2u ? kLightThreads : 1024u, phases == 2u ? (ETA ? 3u : 5u) : 4u)
    k_count(BatchHeader* hdr, const JobDev* __restrict__ jobs) {
    extern __shared__ __align__(16) uint8_t lds[];
    const uint32_t lane = lane_id(), wid = threadIdx.x >> 6, nw = blockDim.x >> 6;
    const uint32_t DL = hdr->wave_cap, DW = hdr->block_cap, DB = hdr->b_chunk;
    const uint32_t GM = hdr->G_max, HC = hdr->hist_c, njobs = hdr->njobs;
    const uint32_t DLB = hdr->light_b, RW = hdr->gs_max;
    const Layout L = count_layout(nw, DL, DW, DB, GM, RW, HC, DLB, ETA, (phases & 1u) != 0, (phases & 2u) != 0);
    uint32_t* const hub = (uint32_t*)lds;
    WaveView V = wave_view(lds + L.misc_off + wid * L.misc.bytes, L.misc);
    uint8_t* uni = lds + L.union_off;
    __shared__ uint32_t s_tile[2][9];

    for (uint32_t i = lane; i < HC; i += 64) V.hist[i] = 0;
    JobRegs J;
    int cur = -1;
    int hub_job = -1;  // the job whose hubs the workgroup gathers (uniform)

    // phase 1: long lists, one apex per workgroup
    if (phases & 1u) {
        const TeamView T =
            team_view(uni, uni + L.hw.bytes + wid * L.hb.bytes, L.hw, L.hb, DW, wave_lists(DB, nw));
        const uint32_t total = hdr->heavy_total;
        uint32_t q = blockIdx.x % kQueues, done = 0;  // used by the last wavefront
        // A tile's unit and part, in LDS: found by the last wavefront, for the next tile while the
        // workgroup counts the current one, so that the claim and the loads that follow it (a chain
        // of three) cost no time of their own.
        auto fetch = [&](uint32_t tile, uint32_t* to) {
            if (tile < total) {
                const uint32_t j = find_job(jobs, njobs, tile, true);
                const JobDev& JD = jobs[j];
                uint32_t before, unit, part;
                const uint32_t k = tile_part(JD.hcls, kHeavyClasses, tile - JD.heavy_prefix, before, unit, part);
                const uint32_t a = ldg(JD.apex + JD.unit0 + before + unit);
                const uint32_t s0 = ldg(JD.off + a), r0 = ldg(JD.roff + a);
                const uint32_t d = ldg(JD.off + a + 1) - s0, rn = ldg(JD.roff + a + 1) - r0;
                const uint64_t lists = (uint64_t)d + rn;
                if (lane == 0) {
                    to[1] = j;
                    to[2] = a;
                    to[3] = s0;
                    to[4] = d;
                    to[5] = r0;
                    to[6] = rn;
                    to[7] = (uint32_t)((lists * part) >> k);
                    to[8] = (uint32_t)((lists * (part + 1)) >> k);
                }
            }
            if (lane == 0) to[0] = tile;
        };
        if (wid == nw - 1) fetch(blockIdx.x, s_tile[0]);  // a workgroup's first tile needs no claim
        for (uint32_t at = 0;; at ^= 1u) {
            __syncthreads();
            const uint32_t* const cu = s_tile[at];
            if (wave_uni(cu[0]) >= total) break;
            const uint32_t j = wave_uni(cu[1]);
            if ((int)j != cur) {
                flush_hist(J, V, cur);
                load_job(jobs + j, HC, J);
                cur = (int)j;
                if (hub_job >= 0) hub_flush(jobs[hub_job], hub);
                hub_bind(jobs[j], hub, GM);
                hub_job = (int)j;
                V.hub = hub;
            }
            auto ahead = [&]() {
                fetch(claim_tile(hdr->queues + kHeavyQueue, gridDim.x, total, q, done), s_tile[at ^ 1u]);
            };
            const uint32_t e0 = wave_uni(cu[7]), e1 = wave_uni(cu[8]);
            if (e0 < e1) {
                count_apex<true, ETA>(J, T, V, wave_uni(cu[2]), wave_uni(cu[3]), wave_uni(cu[4]), wave_uni(cu[5]),
                                      wave_uni(cu[6]), e0, e1, ahead);
            } else if (wid == nw - 1) {  // an empty part
                ahead();
            }
        }
    }
    __syncthreads();  // the union area changes owners

    // phase 2: short lists, several apexes to a wavefront
    if (phases & 2u) {
        uint8_t* const mine = uni + wid * (L.lw.bytes + L.lb.bytes + L.lu.bytes);
        TeamView T = team_view(mine, mine + L.lw.bytes, L.lw, L.lb, DL, wave_lists(DLB, 1));
        unit_view(T, mine + L.lw.bytes + L.lb.bytes, L.lu);
        const uint32_t total = hdr->light_total;
        // a wavefront's first tile needs no claim, unless it comes to the light tiles only after
        // heavy ones (those would keep its tile waiting)
        const uint32_t own = (phases & 1u) && hdr->heavy_total ? 0u : gridDim.x * nw;
        if (hub_job < 0 && total) {
            // the job of the workgroup's first tile; its other jobs' hubs are updated directly
            const uint32_t t = blockIdx.x < total ? blockIdx.x : total - 1;
            hub_job = (int)find_job(jobs, njobs, t, false);
            hub_bind(jobs[hub_job], hub, GM);
        }
        V.hub = hub_job == cur && cur >= 0 ? hub : nullptr;
        uint32_t q = (blockIdx.x * nw + wid) % kQueues, done = 0;
        for (bool first = own != 0;; first = false) {
            const uint32_t tile = wave_uni(first ? wid * gridDim.x + blockIdx.x
                                                 : claim_tile(hdr->queues + kLightQueue, own, total, q, done));
            if (tile >= total) {
                if (first) continue;
                break;
            }
            const uint32_t j = find_job(jobs, njobs, tile, false);
            if ((int)j != cur) {
                flush_hist(J, V, cur);
                load_job(jobs + j, HC, J);
                cur = (int)j;
                V.hub = cur == hub_job ? hub : nullptr;
                wave_sync();
            }
            const JobDev& JD = jobs[j];
            uint32_t first_unit, un, part;
            const uint32_t k = light_tile_of(JD.lcls, tile - JD.light_prefix, first_unit, un, part);
            const uint32_t ub = JD.unit0 + JD.hcls[0] + first_unit;
            // the tile's apexes and their list bounds, loaded together (lane i: unit ub + i), then
            // handed to the unit loop in scalar registers
            uint32_t ta = 0, ts = 0, td = 0, tr = 0, trn = 0;
            if (lane < un) {
                ta = ldg(J.jd->apex + ub + lane);
                ts = ldg(J.off + ta);
                td = ldg(J.off + ta + 1) - ts;
                tr = ldg(J.jd->roff + ta);
                trn = ldg(J.jd->roff + ta + 1) - tr;
            }
            if (k) {  // a part of one unit
                const uint32_t d = lane_val(td, 0), rn = lane_val(trn, 0), lists = d + rn;
                const uint32_t e0 = (lists * part) >> k, e1 = (lists * (part + 1)) >> k;
                if (e0 < e1)
                    count_apex<false, ETA>(J, T, V, lane_val(ta, 0), lane_val(ts, 0), d, lane_val(tr, 0), rn, e0, e1,
                                           [] {});
                continue;
            }
            // whole units: passes of as many as fit the table (a light unit's list fits by itself)
            const uint32_t winc = wave_incl_scan(td);
            for (uint32_t f = 0; f < un;) {
                const uint32_t wpre = winc - td - lane_val(winc - td, f);
                const uint32_t fit = (uint32_t)__popcll(
                    __ballot(lane >= f && lane < un && lane < f + kPack && wpre + td <= T.DW));
                count_pack<ETA>(J, T, V, f, fit, ta, ts, td, tr, trn, wpre);
                f += fit;
            }
        }
    }
    if (njobs == 1) {
        // one job: the wavefronts' counts are summed first (one update per workgroup and processor)
        __syncthreads();
        if (HC)
            for (uint32_t p = threadIdx.x; p < jobs[0].c; p += blockDim.x) {
                uint64_t v = 0;
                for (uint32_t w = 0; w < nw; ++w)
                    v += ((const uint32_t*)(lds + L.misc_off + w * L.misc.bytes + L.misc.hist))[p];
                if (v) add64(jobs[0].global + p, v);
            }
    } else {
        flush_hist(J, V, cur);
    }
    if (hub_job >= 0) hub_flush(jobs[hub_job], hub);
}

// ======================================================================= hash slots ======

struct HashParams {
    uint64_t hp[4 * REPT_GMAX];
};

__global__ void k_slots(HashParams P, uint32_t G, uint32_t m, const uint2* __restrict__ edges, uint64_t E,
                        uint32_t* __restrict__ slots) {
    for (uint64_t t = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; t < E;
         t += (uint64_t)gridDim.x * blockDim.x) {
        const uint2 e = edges[t];
        for (uint32_t g = 0; g < G; ++g) slots[(uint64_t)g * E + t] = slot_of(P.hp + 4 * g, m, e.x, e.y);
    }
}

// sums[v] = sum over the rows of local[r][v] (exact int64).  Each thread reads every row at its
// own v before writing sums[v], so sums may be local's first row.
__global__ void k_reduce_rows(const int64_t* local, uint32_t rows, uint32_t n, int64_t* sums) {
    for (uint32_t v = blockIdx.x * blockDim.x + threadIdx.x; v < n; v += gridDim.x * blockDim.x) {
        int64_t acc = 0;
        for (uint32_t r = 0; r < rows; ++r) acc += local[(uint64_t)r * n + v];
        sums[v] = acc;
    }
}

bool g_attr_set = false;

// Second stream of the current device for the light-phase launch, and the fork and join
// events around it (created on first use, default priority, kept for the process).  One
// enqueue sequence at a time: the events are re-recorded by every launch.
struct AuxStream {
    int device = -1;
    hipStream_t stream = nullptr;
    hipEvent_t fork = nullptr, join = nullptr;
};
std::mutex g_aux_mu;
AuxStream g_aux[16];
hipError_t aux_for_current(AuxStream** out) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= 16) return hipErrorInvalidDevice;
    AuxStream& a = g_aux[dev];
    if (a.device != dev) {
        if ((e = hipStreamCreateWithFlags(&a.stream, hipStreamNonBlocking)) != hipSuccess) return e;
        if ((e = hipEventCreateWithFlags(&a.fork, hipEventDisableTiming)) != hipSuccess) return e;
        if ((e = hipEventCreateWithFlags(&a.join, hipEventDisableTiming)) != hipSuccess) return e;
        a.device = dev;
    }
    *out = &a;
    return hipSuccess;
}

hipError_t report(hipError_t e, const char* what) {
    if (e != hipSuccess) fprintf(stderr, "rept: %s failed: %s\n", what, hipGetErrorString(e));
    return e;
}

using CountKernel = void (*)(BatchHeader*, const JobDev*);
CountKernel count_kernel(bool eta, uint32_t phases) {
    if (eta) return phases == 1 ? k_count<true, 1> : (phases == 2 ? k_count<true, 2> : k_count<true, 3>);
    return phases == 1 ? k_count<false, 1> : (phases == 2 ? k_count<false, 2> : k_count<false, 3>);
}

hipError_t set_attrs() {
    if (g_attr_set) return hipSuccess;
    // the kernel's static LDS (a few bytes) and the dynamic part share the CU's 160 KB
    for (uint32_t i = 0; i < 6; ++i) {
        const hipError_t e = hipFuncSetAttribute((const void*)count_kernel(i >= 3, 1u + i % 3u),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024 - 256);
        if (e != hipSuccess) return report(e, "hipFuncSetAttribute(k_count)");
    }
    g_attr_set = true;
    return hipSuccess;
}

// `one`: the single job of a control block, written there by the preparing kernel; null: the job
// table is in `ws` already
hipError_t launch_common(uint8_t* ws, const BatchHeader& h, const JobDev* one, hipStream_t s) {
    (void)hipGetLastError();  // launch errors below are this call's own
    // a grid of 2^32 threads or more cannot be launched: refused before anything is enqueued (below it
    // the kernel's counts of workgroups and wavefronts fit 32 bits)
    auto fits = [](uint32_t blocks, uint32_t threads) { return (uint64_t)blocks * threads <= UINT32_MAX; };
    if (!fits(h.blocks, h.threads) || (h.split && !fits(h.light_blocks, kLightThreads)))
        return report(hipErrorInvalidConfiguration, "counting kernel grid");
    hipError_t e = set_attrs();
    if (e != hipSuccess) return e;
    BatchHeader* hdr = (BatchHeader*)ws;
    JobDev* jobs = (JobDev*)(ws + sizeof(BatchHeader));
    if (one) hipLaunchKernelGGL(k_prep_one, dim3(h.prep_blocks), dim3(256), 0, s, ws, (const BatchShape&)h, *one);
    else hipLaunchKernelGGL(k_prep, dim3(h.prep_blocks, h.njobs), dim3(256), 0, s, hdr, jobs);
    // heavy and light phases in one launch, or the light phase in a launch of its own (a
    // light-only workgroup needs no heavy team area, so more wavefronts fit per CU)
    // (split: the light launch on a second stream, forked after the setup kernels and joined
    // back, so that it runs beside the heavy launch as workgroups free the CUs)
    // A phase without tiles is not launched.
    const bool heavy = h.heavy_total != 0, light = h.light_total != 0;
    auto launch = [&](uint32_t blocks, uint32_t threads, uint32_t lds, hipStream_t on, uint32_t phases) {
        hipLaunchKernelGGL(count_kernel(h.any_eta != 0, phases), dim3(blocks), dim3(threads), lds, on, hdr,
                           (const JobDev*)jobs);
    };
    std::unique_lock<std::mutex> lk(g_aux_mu, std::defer_lock);
    AuxStream* aux = nullptr;
    hipStream_t ls = s;
    if (h.split && h.split_streams && heavy && light) {
        lk.lock();
        if ((e = aux_for_current(&aux)) != hipSuccess) return report(e, "second stream");
        if ((e = hipEventRecord(aux->fork, s)) != hipSuccess) return report(e, "fork event");
        if ((e = hipStreamWaitEvent(aux->stream, aux->fork, 0)) != hipSuccess) return report(e, "fork wait");
        ls = aux->stream;
    }
    if (!h.split) {
        if (heavy || light) launch(h.blocks, h.threads, h.lds_bytes, s, 3u);
    } else {
        if (heavy) launch(h.blocks, h.threads, h.lds_bytes, s, 1u);
        if (light) launch(h.light_blocks, kLightThreads, h.light_lds, ls, 2u);
    }
    if ((e = hipGetLastError()) != hipSuccess) return report(e, "counting kernel launch");
    if (aux) {
        if ((e = hipEventRecord(aux->join, aux->stream)) != hipSuccess) return report(e, "join event");
        if ((e = hipStreamWaitEvent(s, aux->join, 0)) != hipSuccess) return report(e, "join wait");
    }
    return hipSuccess;
}

}  // namespace

uint32_t rept_count_lds(uint32_t threads, uint32_t wave_cap, uint32_t block_cap, uint32_t b_chunk, uint32_t G,
                        uint32_t gs, uint32_t hist_c, uint32_t light_b, bool eta, bool heavy, bool light) {
    return count_layout(threads / 64, wave_cap, block_cap, b_chunk, G, gs, hist_c, light_b, eta, heavy, light).total;
}

uint32_t rept_count_blocks_per_cu(uint32_t threads, uint32_t lds_bytes, bool eta, uint32_t phases) {
    // the query's last answers (every call of one shape asks for the same two)
    struct Last {
        uint32_t threads, lds, form, nb;
    };
    static thread_local Last last[4] = {};
    const uint32_t form = 4u * phases + (eta ? 1u : 0u);
    Last& l = last[phases & 3u];
    if (l.nb && l.threads == threads && l.lds == lds_bytes && l.form == form) return l.nb;
    if (set_attrs() != hipSuccess) return 0;
    int nb = 0;
    const void* fn = (const void*)count_kernel(eta, phases);
    hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, fn, (int)threads, (size_t)lds_bytes);
    if (e != hipSuccess) {
        (void)report(e, "hipOccupancyMaxActiveBlocksPerMultiprocessor(k_count)");
        (void)hipGetLastError();
        return 0;
    }
    l = Last{threads, lds_bytes, form, nb > 0 ? (uint32_t)nb : 0u};
    return l.nb;
}

hipError_t rept_launch_batch(void* ws, const BatchHeader& h, hipStream_t s) {
    return launch_common((uint8_t*)ws, h, nullptr, s);
}

hipError_t rept_launch_single(uint8_t* ctrl, const BatchHeader& hdr, const JobDev& job, hipStream_t s) {
    return launch_common(ctrl, hdr, &job, s);
}

hipError_t rept_launch_reduce(const int64_t* local, uint32_t rows, uint32_t n, int64_t* sums, hipStream_t s) {
    (void)hipGetLastError();
    uint32_t blocks = (n + 255) / 256;
    if (blocks > 8192) blocks = 8192;
    hipLaunchKernelGGL(k_reduce_rows, dim3(blocks), dim3(256), 0, s, local, rows, n, sums);
    return hipGetLastError();
}

hipError_t rept_launch_zero(void* p, uint64_t bytes, hipStream_t s) {
    (void)hipGetLastError();
    const uint64_t words = bytes / 4;
    uint64_t blocks = (words + 255) / 256;
    if (blocks > 8192) blocks = 8192;
    if (blocks < 1) blocks = 1;
    hipLaunchKernelGGL(k_zero_u32, dim3((uint32_t)blocks), dim3(256), 0, s, (uint32_t*)p, words);
    return hipGetLastError();
}

hipError_t rept_launch_eta(const rept_graph* g, const JobDev& d, int64_t* eta, int64_t* eta_v, uint32_t proc0,
                           uint32_t stride, hipStream_t s) {
    (void)hipGetLastError();
    uint64_t blocks = (g->E + FILL_CHUNK - 1) / FILL_CHUNK;
    if (blocks > 8192) blocks = 8192;
    if (blocks < 1) blocks = 1;
    hipLaunchKernelGGL(k_eta, dim3((uint32_t)blocks), dim3(ETA_THREADS), 0, s, g->off, g->nbr, g->n, (const uint16_t*)d.tab,
                       d.gs, d.G, d.m, d.c, (const uint32_t*)d.pairs, d.es, proc0, stride, eta, eta_v);
    return hipGetLastError();
}

hipError_t rept_launch_slots(const uint64_t* hp, uint32_t G, uint32_t m, const uint32_t* edges, uint64_t E,
                             uint32_t* slots, hipStream_t s) {
    HashParams P{};
    for (uint32_t i = 0; i < 4 * G && i < 4 * REPT_GMAX; ++i) P.hp[i] = hp[i];
    uint64_t blocks = (E + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    if (blocks < 1) blocks = 1;
    hipLaunchKernelGGL(k_slots, dim3((uint32_t)blocks), dim3(256), 0, s, P, G, m, (const uint2*)edges, E, slots);
    return hipGetLastError();
}

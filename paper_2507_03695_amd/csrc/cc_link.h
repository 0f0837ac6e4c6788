// cc_link.h — device helpers shared by the single-graph kernels: the key order,
// the finds, the link, membership marks and wave reductions.
#pragma once

#include "cc_internal.h"

namespace ccm {

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint64_t u64x2 __attribute__((ext_vector_type(2)));

// Entry i of a COO list as 32-bit IDs, streamed past the caches' reuse. A 64-bit
// ID above 2^32 - 2 reads as 2^32 - 1, which is out of range for every n here.
__device__ __forceinline__ u32x2 load_entry(const uint32_t* edges, uint64_t i) {
    return __builtin_nontemporal_load(reinterpret_cast<const u32x2*>(edges) + i);
}
__device__ __forceinline__ u32x2 load_entry(const uint64_t* edges, uint64_t i) {
    const u64x2 x = __builtin_nontemporal_load(reinterpret_cast<const u64x2*>(edges) + i);
    return u32x2{x.x < kEmpty ? (uint32_t)x.x : kEmpty, x.y < kEmpty ? (uint32_t)x.y : kEmpty};
}

// Position i of a CSR graph as an entry: its row by a search between the first row
// of i's tile and the next tile's (consecutive lanes search the same few rows, so
// the steps are L1 hits). Clamped like the CSR hook's rows, so that offsets that are
// no row index keep every access in its array.
__device__ __forceinline__ u32x2 load_entry(const CsrList& g, uint64_t i) {
    const uint64_t t = i / kCsrTile;
    const uint32_t v = __builtin_nontemporal_load(g.adj + i);
    uint32_t lo = g.tstart[t], hi = t + 1 < g.ntiles ? g.tstart[t + 1] : g.n - 1;
    if (lo >= g.n) lo = g.n - 1;
    if (hi >= g.n || hi < lo) hi = lo;
    while (lo < hi) {
        const uint32_t mid = lo + (hi - lo + 1) / 2;
        if (g.off[mid] <= i) lo = mid;
        else hi = mid - 1;
    }
    return u32x2{lo, v};
}

__device__ __forceinline__ bool gated_off(Gate g) { return g.word && ld_agent(g.word) != g.want; }

// ---- keys: Formula 1's R used as an order while P stores vertex IDs ----------
// key(x) = x on the plain path; with a zero root z, key(z) = 0 and key(x) = x+1.
template <bool ZR>
__device__ __forceinline__ bool key_less(uint32_t a, uint32_t b, uint32_t z) {
    if (ZR) return (a == z) | ((b != z) & (a < b));
    return a < b;
}

// Root of x, given px = a value read from P[x]. SPLIT = 1: path splitting (each
// visited vertex takes its grandparent); SPLIT = 0: plain walk; SPLIT = k > 1:
// splitting from the k-th step on, for young trees and small arrays: their few levels
// cost less to walk than to split, but entries in an unlucky order can still form
// chains as long as a component, which nothing else would shorten.
constexpr int kLateSplit = 16;
// The splitting writes are device-coherent stores. A plain store would leave a
// dirty line in the writing XCD's L2 whose other words are that XCD's copies;
// links are CASes performed at the memory side, which that copy does not see,
// so the line's write-back can undo a link made meanwhile in the same line (a
// whole-device batch lost links this way). Each store is issued after the next
// step's load, so that its latency overlaps the walk instead of adding to it.
template <int SPLIT>
__device__ __forceinline__ uint32_t find_root(uint32_t* P, uint32_t x, uint32_t px) {
    if (px == x) return x;
    uint32_t gp = P[px];
    int level = 0;
    while (gp != px) {
        const uint32_t ggp = P[gp];
        if (SPLIT == 1 || (SPLIT > 1 && ++level >= SPLIT)) {
            stress_delay(x);
            st_agent(&P[x], gp);
        }
        x = px;
        px = gp;
        gp = ggp;
    }
    return px;
}

// The check before each link's CAS. Global atomics are performed at the memory
// side, past the XCD's L2, and leave the L2's copy of the word as it was; a
// walk that reads P through the L2 can therefore end at a root that has since
// been linked. A CAS on such an entry fails, but only after its round trip, and
// every CAS on one word waits for the ones before it: a giant component's
// former root collects thousands (ER n = 2^16, 2^20 entries: 16,000 CAS on one
// word, a 1.6 ms hook). The entry is read coherently first (a load, which does
// not wait behind the CASes) and a changed entry continues the walk from its
// new value; the CAS is issued only on an entry that still reads as a root.
// ER n = 2^16, 2^20 entries: 1.7 M CAS -> 0.11 M, 1.6-3.4 ms -> 0.16 ms.
// Algorithm 1 / 3 hooking of one entry whose endpoints u, v have parents pu, pv.
// Returns the root under which both endpoints ended up (the surviving root of
// the link, or the common root found). When it is the zero root z, both
// endpoints are certainly in z's tree: z has the smallest key and is never
// linked under anything. If this call's CAS is the one that links, *linked
// (when given) receives the root that was linked; the return value is then its
// new parent.
template <bool ZR, int SPLIT>
__device__ __forceinline__ uint32_t link(uint32_t* P, uint32_t u, uint32_t pu, uint32_t v,
                                         uint32_t pv, uint32_t z, uint32_t* linked = nullptr) {
    while (true) {
        const uint32_t ru = find_root<SPLIT>(P, u, pu);
        const uint32_t rv = find_root<SPLIT>(P, v, pv);
        if (ru == rv) return ru;
        const bool u_low = key_less<ZR>(ru, rv, z);
        const uint32_t hi = u_low ? rv : ru;
        const uint32_t lo = u_low ? ru : rv;
        stress_delay(hi);
        // hi's entry read coherently first (the check described above)
        const uint32_t cur = ld_agent(&P[hi]);
        if (cur != hi) {
            u = hi; pu = cur;
            v = lo; pv = lo;
            continue;
        }
        const uint32_t old = atomicCAS(&P[hi], hi, lo);
        if (old == hi) {
            if (linked) *linked = hi;
            return lo;
        }
        // hi was linked by someone else: its current parent is `old`
        u = hi; pu = old;
        v = lo; pv = lo;
    }
}

// Sets x's bit. The word is read coherently first and the atomic (performed at
// the memory side, where the atomics on one word wait for each other) is issued
// only if the bit is still clear: most of a giant component's members are
// reached by many entries, and their word would otherwise take an atomic for
// each (bits only go from 0 to 1, so a set bit read anywhere stays set).
__device__ __forceinline__ void zbit_set(uint32_t* zbits, uint32_t x) {
    const uint32_t b = 1u << (x & 31);
    if (!(ld_agent(&zbits[x >> 5]) & b)) atomicOr(&zbits[x >> 5], b);
}

__device__ __forceinline__ uint64_t wave_max_u64(uint64_t x) {
    for (int off = 32; off > 0; off >>= 1) {
        uint64_t y = __shfl_xor(x, off, 64);
        x = y > x ? y : x;
    }
    return x;
}

__device__ __forceinline__ uint32_t wave_min_u32(uint32_t x) {
    for (int off = 32; off > 0; off >>= 1) {
        uint32_t y = __shfl_xor(x, off, 64);
        x = y < x ? y : x;
    }
    return x;
}


// ---- per-wave queues of the hooks that test a bitmap in LDS -----------------------
// Entries that are not dropped at once gather in a wave's first queue and are
// looked at again together, one per lane, when the next ones would not fit: most
// then only mark an endpoint (settle). The few with neither endpoint marked
// gather in the second queue, so that the walks and CASes of up to 64 of them
// overlap; linked where they are found, a handful of lanes would hold the wave
// for several memory round trips at nearly every settling (R-MAT n = 2^22,
// 2^26 entries: filter 472 -> 330 us).
constexpr uint32_t kQueueCap = 64;
struct WaveQueues {
    u32x2 *pq, *lq;          // kQueueCap slots each, in LDS
    uint32_t pn = 0, ln = 0; // wave-uniform
};

// Keeps the compiler from moving LDS accesses across it; the lanes of a wave
// execute together and its LDS operations complete in issue order.
__device__ __forceinline__ void wave_order() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// settle(x): marks the other endpoint when exactly one is marked; true when
// neither is. hook(x): hooks x in P. Both are called for one entry per lane;
// every function here is called by the whole wave.
template <class Settle, class Hook>
__device__ __forceinline__ void queue_hook(WaveQueues& q, int lane, const Settle& settle,
                                           const Hook& hook) {
    wave_order();
    if ((uint32_t)lane < q.ln) {
        const u32x2 x = q.lq[lane];
        if (settle(x)) hook(x);      // it may have been marked since
    }
    q.ln = 0;
    wave_order();
}
// direct: hook only notes the entry, and is called at once.
template <class Settle, class Hook>
__device__ __forceinline__ void queue_settle(WaveQueues& q, int lane, const Settle& settle,
                                             const Hook& hook, bool direct = false) {
    wave_order();
    const bool act = (uint32_t)lane < q.pn;
    const u32x2 x = act ? q.pq[lane] : u32x2{0u, 0u};
    const bool keep = act && settle(x);
    if (direct) {
        q.pn = 0;
        if (keep) hook(x);
        wave_order();
        return;
    }
    const uint64_t ball = __ballot(keep);
    const uint32_t c = (uint32_t)__popcll(ball);
    q.pn = 0;
    if (c) {
        if (q.ln + c > kQueueCap) queue_hook(q, lane, settle, hook);
        if (keep) q.lq[q.ln + (uint32_t)__popcll(ball & ((1ull << lane) - 1ull))] = x;
        q.ln += c;
    }
    wave_order();
}
template <class Settle, class Hook>
__device__ __forceinline__ void queue_push(WaveQueues& q, int lane, bool pend, u32x2 x,
                                           const Settle& settle, const Hook& hook,
                                           bool direct = false) {
    const uint64_t ball = __ballot(pend);
    if (!ball) return;
    const uint32_t c = (uint32_t)__popcll(ball);
    if (q.pn + c > kQueueCap) queue_settle(q, lane, settle, hook, direct);
    if (pend) q.pq[q.pn + (uint32_t)__popcll(ball & ((1ull << lane) - 1ull))] = x;
    q.pn += c;
}
template <class Settle, class Hook>
__device__ __forceinline__ void queue_finish(WaveQueues& q, int lane, const Settle& settle,
                                             const Hook& hook, bool direct = false) {
    if (q.pn) queue_settle(q, lane, settle, hook, direct);
    if (q.ln) queue_hook(q, lane, settle, hook);
}

}  // namespace ccm

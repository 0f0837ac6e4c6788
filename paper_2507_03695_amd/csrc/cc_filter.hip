// cc_filter.hip — hooks that test the entries against a membership bitmap held
// in LDS.
//
// Most entries of a graph with a giant component join two vertices already
// known to be connected, and need no parent at all, only one bit per endpoint.
// The hooks here first hook a sample of the entries, flatten the forest and
// write the bitmap of the component of one root (k_giant_bits); then every entry
// is tested against a copy of the bitmap in LDS (random reads at LDS rate
// instead of one L2 line each), and only the entries with an unmarked endpoint
// go further.
#include <algorithm>

#include "cc_internal.h"
#include "cc_link.h"

namespace ccm {

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// ---- the sample -------------------------------------------------------------------------
// Algorithm 1 / 3 on every tstride-th run of kWBlock entries (so that a list in
// any order, sorted rows for instance, is sampled evenly), without the bitmap.
// One entry per thread: the pass is a chain of dependent reads and CASes per
// entry, and a thread with four would take four times as long.
constexpr int kWBlock = 256;

template <bool ZR, int SPLIT>
__global__ __launch_bounds__(kWBlock) void k_warm(const uint32_t* __restrict__ edges, uint64_t m,
                                                  uint32_t n, uint64_t tstride, uint32_t* P,
                                                  DevState* st, uint32_t sym) {
    const uint32_t z = ZR ? ld_agent(&st->zroot) : 0u;
    const uint64_t i = (uint64_t)blockIdx.x * tstride * kWBlock + threadIdx.x;
    if (i >= m) return;
    const u32x2 e = __builtin_nontemporal_load(reinterpret_cast<const u32x2*>(edges) + i);
    if (e.x >= n || e.y >= n) { atomicOr(&st->status, kStatusRange); return; }
    if (sym ? e.x >= e.y : e.x == e.y) return;
    const uint32_t pu = P[e.x], pv = P[e.y];
    if (pu == pv || pu == e.y || pv == e.x) return;
    (void)link<ZR, SPLIT>(P, e.x, pu, e.y, pv, z);
}

// ---- the bitmap of one root's component -------------------------------------------
// Runs on a flat forest (after compress). The root is, on a zero-root solve, the
// zero root z: a vertex is a member when its root is z, or it or its root is
// marked. On a plain solve (PICK) it is the root most often seen above kGSample
// entries' endpoints (ties to the lowest ID), found by every block for itself
// from the same reads, so that no launch of its own is needed; block 0 records
// it in DevState, where the kernels after this one read it as the zero root.
// Each wave writes the two words of 64 consecutive vertices from a ballot.
constexpr int kGBlock = 1024;
constexpr uint32_t kGSample = kGBlock;        // one sampled entry per thread
constexpr uint32_t kGTable = 2 * kGSample;

template <bool PICK>
__global__ __launch_bounds__(kGBlock) void k_giant_bits(const uint32_t* __restrict__ edges,
                                                        uint64_t m, const uint32_t* P, uint64_t n,
                                                        uint32_t* zbits, DevState* st) {
    uint32_t g;
    if (PICK) {
        __shared__ uint32_t s_key[kGTable], s_cnt[kGTable];
        __shared__ uint64_t s_best[kGBlock / 64];
        for (uint32_t i = threadIdx.x; i < kGTable; i += kGBlock) { s_key[i] = kEmpty; s_cnt[i] = 0; }
        __syncthreads();
        const uint64_t cnt = m < kGSample ? m : kGSample;
        if (threadIdx.x < cnt) {
            const uint64_t q = m / cnt, r = m % cnt;
            const uint64_t i = threadIdx.x * q + threadIdx.x * r / cnt;
            const uint32_t x = edges[2 * i + (threadIdx.x & 1)];
            if (x < n) {
                const uint32_t root = ld_agent(&P[x]);
                uint32_t h = (root * 0x9E3779B1u) >> (32 - 11);
                while (true) {
                    const uint32_t k = atomicCAS(&s_key[h], kEmpty, root);
                    if (k == kEmpty || k == root) break;
                    h = (h + 1) & (kGTable - 1);
                }
                atomicAdd(&s_cnt[h], 1u);
            }
        }
        static_assert(kGTable == 1u << 11, "the hash above yields 11 bits");
        __syncthreads();
        uint64_t best = 0;
        for (uint32_t i = threadIdx.x; i < kGTable; i += kGBlock)
            if (s_cnt[i]) best = max(best, ((uint64_t)s_cnt[i] << 32) | (0xFFFFFFFFu - s_key[i]));
        best = wave_max_u64(best);
        if ((threadIdx.x & 63) == 0) s_best[threadIdx.x >> 6] = best;
        __syncthreads();
        best = s_best[0];
        for (int w = 1; w < kGBlock / 64; ++w) best = max(best, s_best[w]);
        g = best ? 0xFFFFFFFFu - (uint32_t)best : ld_agent(&P[0]);
        if (blockIdx.x == 0 && threadIdx.x == 0) st_agent(&st->zroot, g);
    } else {
        g = ld_agent(&st->zroot);
    }
    const uint64_t words = (n + 31) / 32;
    const int lane = threadIdx.x & 63;
    constexpr int kR = 4;
    const uint64_t stride = (uint64_t)gridDim.x * kGBlock;
    for (uint64_t v0 = (uint64_t)blockIdx.x * kGBlock + threadIdx.x; v0 - lane < n;
         v0 += kR * stride) {
        uint32_t p[kR], b[kR];
#pragma unroll
        for (int k = 0; k < kR; ++k) {
            const uint64_t v = v0 + k * stride;
            p[k] = v < n ? ld_agent(&P[v]) : kEmpty;
            b[k] = (!PICK && v < n) ? ld_agent(&zbits[v >> 5]) >> (v & 31) & 1u : 0u;
        }
#pragma unroll
        for (int k = 0; k < kR; ++k) {
            const uint64_t v = v0 + k * stride;
            bool in = v < n && (p[k] == g || b[k]);
            if (!PICK && v < n && !in && p[k] != (uint32_t)v)
                in = ld_agent(&zbits[p[k] >> 5]) >> (p[k] & 31) & 1u;
            const uint64_t ball = __ballot(in);
            const uint64_t w = (v - lane) >> 5;
            if (lane == 0 && w < words) st_agent(&zbits[w], (uint32_t)ball);
            if (lane == 32 && w + 1 < words) st_agent(&zbits[w + 1], (uint32_t)(ball >> 32));
        }
    }
}

// ---- the whole bitmap in LDS ----------------------------------------------------------
// A bitmap of up to kLdsBitsWords words fits in a workgroup's LDS beside the
// waves' queues, so the entries need no regrouping: persistent workgroups stream
// them once, each thread keeping kLEPT loads in flight (an entry's register is
// reloaded with the next round's as soon as it is tested).
//  - both endpoints marked: dropped;
//  - otherwise the entry goes to its wave's queue, and each time 64 are queued
//    they are settled together, one per lane: one endpoint marked, the other is
//    marked too (LDS, and the global word when this set the bit); neither, the
//    entry is hooked in P as in the direct hook.
// The bits set since by other workgroups are not seen; a clear bit only sends an
// entry to P.
constexpr int kLBlock = 1024;
constexpr int kLWaves = kLBlock / 64;
constexpr int kLQueue = 127;
constexpr uint32_t kLdsBitsWords = 36864;      // 144 KB; the queues take 15.9 KB of the 160

template <int SPLIT, int kLEPT>
__global__ __launch_bounds__(kLBlock) void k_hook_lds(const uint32_t* __restrict__ edges, uint64_t m,
                                                      uint32_t n, uint32_t* P, uint32_t* zbits,
                                                      DevState* st, uint32_t sym) {
    extern __shared__ uint32_t bits[];
    __shared__ u32x2 s_q[kLWaves * kLQueue];
    const uint32_t z = ld_agent(&st->zroot);
    const uint32_t words = (n + 31) / 32;
    for (uint32_t i = threadIdx.x; i < words; i += kLBlock) bits[i] = ld_agent(&zbits[i]);
    const int lane = threadIdx.x & 63;
    u32x2* q = s_q + (threadIdx.x >> 6) * kLQueue;
    const u32x2* E = reinterpret_cast<const u32x2*>(edges);
    constexpr uint64_t kTile = (uint64_t)kLBlock * kLEPT;
    const uint64_t step = (uint64_t)gridDim.x * kTile;
    auto bit = [&](uint32_t x) { return (bits[x >> 5] >> (x & 31)) & 1u; };
    auto mark = [&](uint32_t x) {
        const uint32_t b = 1u << (x & 31);
        if (!(atomicOr(&bits[x >> 5], b) & b)) atomicOr(&zbits[x >> 5], b);
    };
    auto settle = [&](uint32_t cnt) {
        if ((uint32_t)lane < cnt) {
            const u32x2 e = q[lane];
            const uint32_t mu = bit(e.x), mv = bit(e.y);
            if (mu != mv) {
                mark(mu ? e.y : e.x);
            } else if (!mu) {
                const uint32_t pu = P[e.x], pv = P[e.y];
                uint32_t r;
                if (pu == pv) r = pu;
                else if (pu == e.y) r = e.y;
                else if (pv == e.x) r = e.x;
                else r = link<true, SPLIT>(P, e.x, pu, e.y, pv, z);
                if (r == z) { mark(e.x); mark(e.y); }
            }
        }
    };
    auto wsync = [] {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    u32x2 e[kLEPT];
    const uint64_t t0 = (uint64_t)blockIdx.x * kTile + threadIdx.x;
#pragma unroll
    for (int k = 0; k < kLEPT; ++k) {
        const uint64_t i = t0 + (uint64_t)k * kLBlock;
        e[k] = __builtin_nontemporal_load(E + (i < m ? i : m - 1));
    }
    __syncthreads();
    uint32_t qn = 0;                                   // wave-uniform
    bool bad = false;
    for (uint64_t t = t0; t - threadIdx.x < m; t += step) {
        // the last round reloads the last entry: an in-bounds address, never tested
        const bool full = t - threadIdx.x + step + kTile <= m;
#pragma unroll
        for (int k = 0; k < kLEPT; ++k) {
            const u32x2 x = e[k];
            const uint64_t i = t + (uint64_t)k * kLBlock;
            const uint64_t j = i + step;
            e[k] = __builtin_nontemporal_load(E + (full || j < m ? j : m - 1));
            const bool ok = (x.x < n) & (x.y < n), in = i < m;
            bad |= in & !ok;
            const uint32_t u = ok ? x.x : 0u, v = ok ? x.y : 0u;
            const bool live = in & (sym ? u < v : u != v);
            const bool pend = live & !(bit(u) & bit(v));
            const uint64_t ball = __ballot(pend);
            if (ball) {
                if (pend) q[qn + (uint32_t)__popcll(ball & ((1ull << lane) - 1ull))] = x;
                qn += (uint32_t)__popcll(ball);
                if (qn >= 64) {
                    wsync();
                    settle(64);
                    const u32x2 rest = (uint32_t)lane < qn - 64 ? q[64 + lane] : u32x2{0u, 0u};
                    wsync();
                    if ((uint32_t)lane < qn - 64) q[lane] = rest;
                    qn -= 64;
                    wsync();
                }
            }
        }
    }
    if (qn) {
        wsync();
        settle(qn);
    }
    if (bad) atomicOr(&st->status, kStatusRange);
}

// ---- host side --------------------------------------------------------------------

uint64_t lds_bits_max_n() { return (uint64_t)kLdsBitsWords * 32; }

int run_warm(uint64_t n, uint64_t m, const uint32_t* edges, uint32_t* P, DevState* st, bool zr,
             bool split, bool sym, uint64_t want, hipStream_t stream) {
    const uint64_t tiles = (m + kWBlock - 1) / kWBlock;
    const uint64_t ts = std::max<uint64_t>(m / std::max<uint64_t>(want, 1), 1);
    const uint64_t g = (tiles + ts - 1) / ts;
    if (g > 0x7FFFFFFFull) return fail(CC_EINVAL, "edge count too large for one launch");
    const uint32_t n32 = (uint32_t)n, sy = sym ? 1u : 0u;
    if (zr && split) k_warm<true, 1><<<(uint32_t)g, kWBlock, 0, stream>>>(edges, m, n32, ts, P, st, sy);
    else if (zr) k_warm<true, 0><<<(uint32_t)g, kWBlock, 0, stream>>>(edges, m, n32, ts, P, st, sy);
    else if (split) k_warm<false, 1><<<(uint32_t)g, kWBlock, 0, stream>>>(edges, m, n32, ts, P, st, sy);
    else k_warm<false, 0><<<(uint32_t)g, kWBlock, 0, stream>>>(edges, m, n32, ts, P, st, sy);
    CCM_HIP(hipGetLastError());
    return CC_OK;
}

int run_giant_bits(uint64_t n, uint64_t m, const uint32_t* edges, const uint32_t* P, uint32_t* zbits,
                   DevState* st, bool pick, hipStream_t stream) {
    const uint64_t blocks = (n + 4 * kGBlock - 1) / (4 * kGBlock);
    const uint32_t g = (uint32_t)std::min<uint64_t>(blocks, 2048);
    if (pick) k_giant_bits<true><<<g, kGBlock, 0, stream>>>(edges, m, P, n, zbits, st);
    else k_giant_bits<false><<<g, kGBlock, 0, stream>>>(edges, m, P, n, zbits, st);
    CCM_HIP(hipGetLastError());
    return CC_OK;
}

int run_hook_lds(uint64_t n, uint64_t m, const uint32_t* edges, uint32_t* P, uint32_t* zbits,
                 DevState* st, bool split, bool sym, int device, hipStream_t stream) {
    const size_t lds = 4 * ((n + 31) / 32);
    const uint64_t cus = device_cu_count(device);
    // two workgroups per CU where two bitmaps fit; on short lists fewer entries
    // per thread, so that every CU has a tile
    const uint64_t wgs = (lds <= (60u << 10) ? 2 : 1) * cus;
    const bool wide = m >= wgs * kLBlock * 8;
    const uint64_t tile = (uint64_t)kLBlock * (wide ? 8 : 2);
    const uint32_t g = (uint32_t)std::min<uint64_t>((m + tile - 1) / tile, wgs);
    const uint32_t n32 = (uint32_t)n, sy = sym ? 1u : 0u;
    auto launch = [&](auto kernel) -> int {
        // the largest size, whatever this call needs: the attribute belongs to the
        // kernel, and another thread's call may need more than this one
        CCM_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                    hipFuncAttributeMaxDynamicSharedMemorySize,
                                    4 * (int)kLdsBitsWords));
        kernel<<<g, kLBlock, lds, stream>>>(edges, m, n32, P, zbits, st, sy);
        CCM_HIP(hipGetLastError());
        return CC_OK;
    };
    if (split) return wide ? launch(&k_hook_lds<1, 8>) : launch(&k_hook_lds<1, 2>);
    return wide ? launch(&k_hook_lds<0, 8>) : launch(&k_hook_lds<0, 2>);
}

}  // namespace ccm

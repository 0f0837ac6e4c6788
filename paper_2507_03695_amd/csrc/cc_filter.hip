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
#include <type_traits>

#include "cc_internal.h"
#include "cc_link.h"

namespace ccm {

// ---- the sample -------------------------------------------------------------------------
// Algorithm 1 / 3 on every tstride-th run of kWBlock entries (so that a list in
// any order, sorted rows for instance, is sampled evenly), without the bitmap
// and with path splitting only in long walks: the trees are young, and the splitting
// stores of all entries would meet on the words just below the few large roots (R-MAT
// n = 2^22, 2^21 entries sampled: 389 us with splitting, 125 without or late). One entry per
// thread: the pass is a chain of dependent reads and CASes per entry.
constexpr int kWBlock = kSampleRun;
constexpr uint32_t kWGrid = 8192;

template <bool ZR, typename T>
__global__ __launch_bounds__(kWBlock) void k_warm(const T edges, uint64_t m, uint32_t n,
                                                  uint64_t tstride, uint64_t tiles, uint32_t* P,
                                                  DevState* st, uint32_t sym, Gate gate) {
    if (gated_off(gate)) return;
    const uint32_t z = ZR ? ld_agent(&st->zroot) : 0u;
    for (uint64_t t = blockIdx.x; t < tiles; t += gridDim.x) {
        const uint64_t i = t * tstride * kWBlock + threadIdx.x;
        if (i >= m) return;
        const u32x2 e = load_entry(edges, i);
        if (e.x >= n || e.y >= n) { atomicOr(&st->status, kStatusRange); continue; }
        if (sym ? e.x >= e.y : e.x == e.y) continue;
        const uint32_t pu = P[e.x], pv = P[e.y];
        if (pu == pv || pu == e.y || pv == e.x) continue;
        (void)link<ZR, kLateSplit>(P, e.x, pu, e.y, pv, z);
    }
}

// ---- is there a giant component ----------------------------------------------------------
// One block walks kGSample sampled entries' endpoints (both ends alternating) to
// their roots. A plain solve (PICK) takes the root met most often (ties to the
// lowest ID) as the one whose component the bitmap describes; with a zero root
// it is z. At least a tenth of the endpoints in that component make it giant.
// Below that the filter would leave most entries to be hooked with one workgroup
// per CU, and the direct hook is the better one (grid of 4 M vertices, 8 M
// entries: 1.05 ms direct, 9 ms through the filter).
constexpr int kGBlock = 1024;
constexpr uint32_t kGSample = kGBlock;        // one sampled entry per thread
constexpr uint32_t kGTable = 2 * kGSample;
static_assert(kGTable == 1u << 11, "the sample's hash yields 11 bits");

// The root that kGSample sampled endpoints have most often, by one block of
// kGBlock threads; *count receives how many of *total have it (without pick, how
// many have the root g).
// root_of(x) gives a vertex's root.
template <typename T, class Root>
__device__ __forceinline__ uint32_t sample_root(const T& edges, uint64_t m, uint64_t n, bool pick,
                                                uint32_t g, uint32_t* count, uint32_t* total,
                                                const Root& root_of) {
    __shared__ uint32_t s_key[kGTable], s_cnt[kGTable];
    __shared__ uint64_t s_best[kGBlock / 64];
    __shared__ uint32_t s_tot, s_in;
    if (threadIdx.x == 0) { s_tot = 0; s_in = 0; }
    for (uint32_t i = threadIdx.x; i < kGTable; i += kGBlock) { s_key[i] = kEmpty; s_cnt[i] = 0; }
    __syncthreads();
    const uint64_t cnt = m < kGSample ? m : kGSample;
    uint32_t root = kEmpty;
    if (threadIdx.x < cnt) {
        const uint64_t q = m / cnt, r = m % cnt;
        const u32x2 e = load_entry(edges, threadIdx.x * q + threadIdx.x * r / cnt);
        const uint32_t x = threadIdx.x & 1 ? e.y : e.x;
        if (x < n) root = root_of(x);
    }
    if (root != kEmpty) {
        atomicAdd(&s_tot, 1u);
        if (!pick && root == g) atomicAdd(&s_in, 1u);
        if (pick) {
            uint32_t h = (root * 0x9E3779B1u) >> (32 - 11);
            while (true) {
                const uint32_t k = atomicCAS(&s_key[h], kEmpty, root);
                if (k == kEmpty || k == root) break;
                h = (h + 1) & (kGTable - 1);
            }
            atomicAdd(&s_cnt[h], 1u);
        }
    }
    __syncthreads();
    uint32_t in = s_in;
    if (pick) {
        uint64_t best = 0;
        for (uint32_t i = threadIdx.x; i < kGTable; i += kGBlock)
            if (s_cnt[i]) best = max(best, ((uint64_t)s_cnt[i] << 32) | (0xFFFFFFFFu - s_key[i]));
        best = wave_max_u64(best);
        if ((threadIdx.x & 63) == 0) s_best[threadIdx.x >> 6] = best;
        __syncthreads();
        best = s_best[0];
        for (int w = 1; w < kGBlock / 64; ++w) best = max(best, s_best[w]);
        g = best ? 0xFFFFFFFFu - (uint32_t)best : root_of(0);
        in = (uint32_t)(best >> 32);
    }
    *count = in;
    *total = s_tot;
    return g;
}

__device__ __forceinline__ uint32_t giant_enough(uint32_t in, uint32_t total) {
    return total && 10 * in >= total;
}

template <bool PICK, typename T>
__global__ __launch_bounds__(kGBlock) void k_find_giant(const T edges, uint64_t m,
                                                        uint32_t* P, uint64_t n,
                                                        const uint32_t* zbits, DevState* st,
                                                        int stage, Gate gate) {
    if (gated_off(gate)) return;
    uint32_t in, tot;
    const uint32_t z = PICK ? 0u : ld_agent(&st->zroot);
    const uint32_t g = sample_root(edges, m, n, PICK, z, &in, &tot, [&](uint32_t x) {
        if (!PICK && (ld_agent(&zbits[x >> 5]) >> (x & 31) & 1u)) return z;
        uint32_t p = ld_agent(&P[x]);
        while (p != x) { x = p; p = ld_agent(&P[x]); }
        return x;
    });
    if (threadIdx.x == 0) {
        const uint32_t giant = giant_enough(in, tot);
        if (PICK) st_agent(&st->zroot, g);
        if (stage < 2) st_agent(&st->giant1, giant);
        st_agent(&st->giant, giant);
        st_agent(&st->rebuild, stage ? giant : 0u);
        st_agent(&st->flat, stage || !giant ? 1u : 0u);
    }
}

// ---- the bitmap of one root's component -------------------------------------------
// Runs on a flat forest (after compress). A vertex is a member when its root is
// st->zroot, or (ZR) when it or its root is marked. With PICK the root is found
// here, as k_find_giant would, by every block for itself from the same reads (one
// launch less); block 0 records it, and with `sample` whether it is a giant
// component's (st->giant; after the first sample, 1, st->giant1 too). Each wave
// writes the two words of 64 consecutive vertices from a ballot.
template <int MODE, typename T>
__global__ __launch_bounds__(kGBlock) void k_giant_bits(const T edges, uint64_t m,
                                                        const uint32_t* P, uint64_t n,
                                                        uint32_t* zbits, DevState* st, int sample,
                                                        Gate gate) {
    if (gated_off(gate)) return;
    constexpr bool ZR = MODE == kBitsZr;
    uint32_t g;
    if (MODE == kBitsPick || (sample && blockIdx.x == 0)) {
        uint32_t in, tot;
        const uint32_t z = ZR ? ld_agent(&st->zroot) : 0u;
        g = sample_root(edges, m, n, MODE == kBitsPick, z, &in, &tot,
                        [&](uint32_t x) { return ld_agent(&P[x]); });
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            if (MODE == kBitsPick) st_agent(&st->zroot, g);
            if (sample == 1) st_agent(&st->giant1, giant_enough(in, tot));
            if (sample) st_agent(&st->giant, giant_enough(in, tot));
        }
    } else {
        g = ld_agent(&st->zroot);
    }
    // Each wave takes kR * 64 consecutive vertices and writes their 2 kR words with
    // one store (word by word, 4-byte stores to memory bound the pass: n = 2^28,
    // 1.11 ms against 0.60).
    const uint64_t words = (n + 31) / 32;
    const int lane = threadIdx.x & 63;
    constexpr int kR = 4;
    const uint64_t wave = ((uint64_t)blockIdx.x * kGBlock + threadIdx.x) >> 6;
    const uint64_t stride = ((uint64_t)gridDim.x * kGBlock) * kR;
    for (uint64_t base = wave * 64 * kR; base < n; base += stride) {
        uint32_t p[kR], b[kR];
#pragma unroll
        for (int k = 0; k < kR; ++k) {
            const uint64_t v = base + k * 64 + lane;
            p[k] = v < n ? ld_agent(&P[v]) : kEmpty;
            b[k] = (ZR && v < n) ? ld_agent(&zbits[v >> 5]) >> (v & 31) & 1u : 0u;
        }
        uint32_t mine = 0;                       // lane i's word
#pragma unroll
        for (int k = 0; k < kR; ++k) {
            const uint64_t v = base + k * 64 + lane;
            bool in = v < n && (p[k] == g || b[k]);
            if (ZR && v < n && !in && p[k] != (uint32_t)v)
                in = ld_agent(&zbits[p[k] >> 5]) >> (p[k] & 31) & 1u;
            const uint64_t ball = __ballot(in);
            if (lane == 2 * k) mine = (uint32_t)ball;
            if (lane == 2 * k + 1) mine = (uint32_t)(ball >> 32);
        }
        const uint64_t w = (base >> 5) + lane;
        if (lane < 2 * kR && w < words) st_agent(&zbits[w], mine);
    }
}

// ---- the whole bitmap in LDS ----------------------------------------------------------
// A bitmap of up to kLdsBitsWords words fits in a workgroup's LDS beside the
// waves' queues, so the entries need no regrouping: persistent workgroups stream
// them once, each thread keeping kLEPT loads in flight (an entry's register is
// reloaded with the next round's as soon as it is tested).
//  - both endpoints marked: dropped;
//  - otherwise the entry goes to its wave's queues (cc_link.h): one endpoint
//    marked, the other is marked too (LDS, and the global word when this set the
//    bit); neither, the entry is hooked in P as in the direct hook.
// The bits set since by other workgroups are not seen; a clear bit only sends an
// entry to P. Where the samples show no giant component the marking pass of a list of
// few entries per vertex leaves at once (n = 1 M, 12 parts, 4 M entries: 321 us with it,
// 306 without; 20 parts of 5,000 vertices, 16 per vertex: 132 and 143), and rows are
// left to the caller, whose hook finds them without a search per entry; a list's entries
// still come here: hooked 64 at a time, they cost what the direct hook takes.
constexpr int kLBlock = 1024;
constexpr int kLWaves = kLBlock / 64;
constexpr uint32_t kMarkGrid = 128;            // workgroups of the marking pass
constexpr uint32_t kLdsBitsWords = 36864;      // 144 KB; the queues take the rest of the 160

template <int SPLIT, int kLEPT, bool MARK, typename T>
__global__ __launch_bounds__(kLBlock) void k_hook_lds(const T edges, uint64_t m,
                                                      uint32_t n, uint32_t* P, uint32_t* zbits,
                                                      DevState* st, uint32_t sym, uint32_t tstride) {
    extern __shared__ uint32_t bits[];
    __shared__ u32x2 s_queue[kLWaves * 2 * kQueueCap];
    const uint32_t z = ld_agent(&st->zroot);
    if (((MARK && m < 8ull * n) || std::is_same<T, CsrList>::value) && !ld_agent(&st->giant)) return;
    const uint32_t words = (n + 31) / 32;
    // Plain loads: the copies of an XCD's workgroups come out of its L2 (run_hook_lds
    // sees to it that no older line is there). Each workgroup starts elsewhere, so
    // that they do not all want the same channel at once.
    constexpr int kW = 8;                              // words in flight per thread
    const uint32_t rot = (uint32_t)((uint64_t)words * (blockIdx.x & 31) / 32);
    auto turn = [&](uint32_t i) { return i + rot < words ? i + rot : i + rot - words; };
    for (uint32_t i0 = threadIdx.x; i0 < words; i0 += kW * kLBlock) {
        uint32_t w[kW];
#pragma unroll
        for (int k = 0; k < kW; ++k) w[k] = i0 + k * kLBlock < words ? zbits[turn(i0 + k * kLBlock)] : 0u;
#pragma unroll
        for (int k = 0; k < kW; ++k)
            if (i0 + k * kLBlock < words) bits[turn(i0 + k * kLBlock)] = w[k];
    }
    const int lane = threadIdx.x & 63;
    WaveQueues q;
    q.pq = s_queue + (threadIdx.x >> 6) * 2 * kQueueCap;
    q.lq = q.pq + kQueueCap;
    constexpr uint64_t kTile = (uint64_t)kLBlock * kLEPT;
    const uint64_t step = (uint64_t)gridDim.x * kTile * tstride;
    auto bit = [&](uint32_t x) { return (bits[x >> 5] >> (x & 31)) & 1u; };
    auto mark = [&](uint32_t x) {
        const uint32_t b = 1u << (x & 31);
        const uint32_t old = atomicOr(&bits[x >> 5], b);
        if (!MARK && !(old & b)) atomicOr(&zbits[x >> 5], b);
    };
    auto settle = [&](u32x2 e) {
        const uint32_t mu = bit(e.x), mv = bit(e.y);
        if (mu != mv) mark(mu ? e.y : e.x);
        return !mu && !mv;
    };
    auto hook = [&](u32x2 e) {
        const uint32_t pu = P[e.x], pv = P[e.y];
        if (pu == pv || pu == e.y || pv == e.x) return;
        (void)link<true, SPLIT>(P, e.x, pu, e.y, pv, z);
    };
    u32x2 e[kLEPT];
    const uint64_t t0 = (uint64_t)blockIdx.x * tstride * kTile + threadIdx.x;
#pragma unroll
    for (int k = 0; k < kLEPT; ++k) {
        const uint64_t i = t0 + (uint64_t)k * kLBlock;
        e[k] = load_entry(edges, i < m ? i : m - 1);
    }
    __syncthreads();
    bool bad = false;
    for (uint64_t t = t0; t - threadIdx.x < m; t += step) {
        // the last round reloads the last entry: an in-bounds address, never tested
        const bool full = t - threadIdx.x + step + kTile <= m;
#pragma unroll
        for (int k = 0; k < kLEPT; ++k) {
            const u32x2 x = e[k];
            const uint64_t i = t + (uint64_t)k * kLBlock;
            const uint64_t j = i + step;
            e[k] = load_entry(edges, full || j < m ? j : m - 1);
            const bool ok = (x.x < n) & (x.y < n), in = i < m;
            bad |= in & !ok;
            const uint32_t u = ok ? x.x : 0u, v = ok ? x.y : 0u;
            const bool live = in & (sym ? u < v : u != v);
            const bool pend = live & !(bit(u) & bit(v));
            if (MARK) {
                if (pend) (void)settle(x);
            } else {
                queue_push(q, lane, pend, x, settle, hook);
            }
        }
    }
    if (!MARK) queue_finish(q, lane, settle, hook);
    if (MARK) {
        // the new marks, one atomic per word that gained any
        __syncthreads();
        for (uint32_t i0 = threadIdx.x; i0 < words; i0 += kW * kLBlock) {
            uint32_t w[kW];
#pragma unroll
            for (int k = 0; k < kW; ++k)
                w[k] = i0 + k * kLBlock < words ? ld_agent(&zbits[turn(i0 + k * kLBlock)]) : 0u;
#pragma unroll
            for (int k = 0; k < kW; ++k) {
                if (i0 + k * kLBlock >= words) continue;
                const uint32_t i = turn(i0 + k * kLBlock);
                if (bits[i] & ~w[k]) atomicOr(&zbits[i], bits[i] & ~w[k]);
            }
        }
    }
    if (bad) atomicOr(&st->status, kStatusRange);
}

// ---- host side --------------------------------------------------------------------

uint64_t lds_bits_max_n() { return (uint64_t)kLdsBitsWords * 32; }

uint64_t warm_stride(uint64_t m, uint64_t want) {
    want = std::max<uint64_t>(want, 1);
    return std::max<uint64_t>((m + want / 2) / want, 1);
}

int run_warm(uint64_t n, uint64_t m, EdgeList E, uint32_t* P, DevState* st, bool zr, bool sym,
             uint64_t want, Gate gate, hipStream_t stream) {
    const uint64_t ts = warm_stride(m, want);
    const uint64_t tiles = ((m + kWBlock - 1) / kWBlock + ts - 1) / ts;
    const uint32_t n32 = (uint32_t)n, sy = sym ? 1u : 0u;
    const uint32_t g = (uint32_t)std::min<uint64_t>(tiles, kWGrid);
    if (zr)
        with_entries(E, [&](auto e) {
            k_warm<true><<<g, kWBlock, 0, stream>>>(e, m, n32, ts, tiles, P, st, sy, gate);
        });
    else
        with_coo(E, [&](auto e) {
            k_warm<false><<<g, kWBlock, 0, stream>>>(e, m, n32, ts, tiles, P, st, sy, gate);
        });
    CCM_HIP(hipGetLastError());
    return CC_OK;
}

int run_find_giant(uint64_t n, uint64_t m, EdgeList E, uint32_t* P, const uint32_t* zbits, DevState* st,
                   bool zr, int stage, hipStream_t stream) {
    const Gate gate = stage ? Gate{&st->giant1, 0u} : Gate{};
    if (zr)
        with_entries(E, [&](auto e) {
            k_find_giant<false><<<1, kGBlock, 0, stream>>>(e, m, P, n, zbits, st, stage, gate);
        });
    else
        with_coo(E, [&](auto e) {
            k_find_giant<true><<<1, kGBlock, 0, stream>>>(e, m, P, n, zbits, st, stage, gate);
        });
    CCM_HIP(hipGetLastError());
    return CC_OK;
}

int run_giant_bits(uint64_t n, uint64_t m, EdgeList E, const uint32_t* P, uint32_t* zbits,
                   DevState* st, int mode, int sample, Gate gate, hipStream_t stream) {
    const uint64_t blocks = (n + 4 * kGBlock - 1) / (4 * kGBlock);
    const uint32_t g = (uint32_t)std::min<uint64_t>(blocks, 2048);
    const uint32_t* none = nullptr;
    auto launch = [&](auto e) {
        k_giant_bits<kBitsPick><<<g, kGBlock, 0, stream>>>(e, m, P, n, zbits, st, sample, gate);
    };
    if (mode == kBitsZr && sample) {
        with_entries(E, [&](auto e) {
            k_giant_bits<kBitsZr><<<g, kGBlock, 0, stream>>>(e, m, P, n, zbits, st, sample, gate);
        });
    } else if (mode == kBitsZr) {
        k_giant_bits<kBitsZr><<<g, kGBlock, 0, stream>>>(none, m, P, n, zbits, st, sample, gate);
    } else if (mode == kBitsPlain) {
        k_giant_bits<kBitsPlain><<<g, kGBlock, 0, stream>>>(none, m, P, n, zbits, st, sample, gate);
    } else {
        with_coo(E, launch);
    }
    CCM_HIP(hipGetLastError());
    return CC_OK;
}

int run_hook_lds(uint64_t n, uint64_t m, EdgeList E, uint32_t* P, uint32_t* zbits, DevState* st,
                 bool split, bool sym, int device, hipStream_t stream) {
    const size_t lds = 4 * ((n + 31) / 32);
    const uint64_t cus = device_cu_count(device);
    // two workgroups per CU where two bitmaps fit; on short lists fewer entries
    // per thread, so that every CU has a tile
    const uint64_t wgs = (lds <= (60u << 10) ? 2 : 1) * cus;
    const bool wide = m >= wgs * kLBlock * 8;
    const uint64_t tile = (uint64_t)kLBlock * (wide ? 8 : 2);
    const uint32_t g = (uint32_t)std::min<uint64_t>((m + tile - 1) / tile, wgs);
    const uint32_t n32 = (uint32_t)n, sy = sym ? 1u : 0u;
    auto launch = [&](auto kernel, auto e, uint32_t ts, uint32_t blocks) -> int {
        // the largest size, whatever this call needs: the attribute belongs to the
        // kernel, and another thread's call may need more than this one
        CCM_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                    hipFuncAttributeMaxDynamicSharedMemorySize,
                                    4 * (int)kLdsBitsWords));
        kernel<<<blocks, kLBlock, lds, stream>>>(e, m, n32, P, zbits, st, sy, ts);
        CCM_HIP(hipGetLastError());
        return CC_OK;
    };
    auto pick = [&](auto e) -> int {
        using T = decltype(e);
        // Every fourth round by few workgroups, marks only: what each learns about
        // its copy, all know in the full pass, instead of hooking in P what the
        // others have marked (R-MAT n = 1,000,003, 15 M entries, whole solve: 332 us
        // without, 185 with 128 workgroups, 201 with 32, 204 with 256).
        int rc = launch(wide ? &k_hook_lds<0, 8, true, T> : &k_hook_lds<0, 2, true, T>, e, 4u,
                        std::min<uint32_t>(g, kMarkGrid));
        if (rc) return rc;
        // the copies above left lines of the bitmap in the XCDs' L2s
        if ((rc = cohere(stream))) return rc;
        if (split)
            return launch(wide ? &k_hook_lds<1, 8, false, T> : &k_hook_lds<1, 2, false, T>, e, 1u, g);
        return launch(wide ? &k_hook_lds<0, 8, false, T> : &k_hook_lds<0, 2, false, T>, e, 1u, g);
    };
    return with_entries(E, pick);
}

}  // namespace ccm

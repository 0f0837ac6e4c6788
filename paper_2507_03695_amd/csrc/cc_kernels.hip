// cc_kernels.hip — the single-graph path on gfx950: init, zero root, Initial
// Push, hook, compress (pointer jumping) and the zero-component relabelling.
//
// Memory model. P is one uint32 array shared by every wave of the device
// (Sec. I: one shared array per machine instead of per-core copies). Links
// are made only by device-scope compare-and-swap on a root's own entry, so
// two workers can never both hook the same root. Parent reads are ordinary
// L2-cached loads: on a multi-XCD device another XCD's L2 may hold an older
// value, but every value an entry ever holds is an ancestor of that vertex
// (an entry changes from itself to a root of smaller key when hooked, and
// afterwards only to further ancestors by path splitting), so a stale read
// walks a shorter prefix of the true path. A stale "root" is caught by the
// CAS, which fails and returns the current parent; the walk resumes there
// (Sec. II: a failed CAS repeats the root search). Splitting stores go only
// to non-roots, which no CAS can succeed on, so they never race with links.
// Every store to P is an agent-scope atomic store: plain stores have been
// observed to leave copies in the writing XCD's L2 that outlive later kernels'
// writes from other XCDs, so that a later reader on that XCD sees an old value.
#include <algorithm>

#include "cc_internal.h"
#include "cc_link.h"

namespace ccm {

constexpr int kBlock = 256;

// ---- init --------------------------------------------------------------------
// P_v = v (Algorithm 1 / 3 initialisation; with R the stored values stay vertex
// IDs and only the order changes). Like every store to P, a device-coherent one
// (see find_root); lanes write consecutive words, so each wave writes whole lines.
__global__ __launch_bounds__(kBlock) void k_init(uint32_t* __restrict__ P, uint64_t n,
                                                 DevState* st) {
    const uint64_t tid = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
    const uint64_t stride = (uint64_t)gridDim.x * kBlock;
    if (tid == 0) st_agent(&st->mpub, kEmpty);
    for (uint64_t v = tid; v < n; v += stride) st_agent(&P[v], (uint32_t)v);
}

// ---- zero root: sampled endpoint counts in an open-addressing table ----------

__device__ __forceinline__ uint64_t sample_index(uint64_t j, uint64_t m, uint64_t K) {
    // floor(j*m/K) without 128-bit arithmetic: m = q*K + r
    const uint64_t q = m / K, r = m % K;
    return j * q + (j * r) / K;
}

__global__ __launch_bounds__(kBlock) void k_zfill(uint32_t* keys, uint32_t* counts, uint32_t T,
                                                  DevState* st) {
    uint32_t i = blockIdx.x * kBlock + threadIdx.x;
    if (i == 0) st_agent64(&st->zsel, 0);
    for (; i < T; i += gridDim.x * kBlock) {
        st_agent(&keys[i], kEmpty);
        st_agent(&counts[i], 0u);
    }
}

__device__ __forceinline__ void table_add(uint32_t* keys, uint32_t* counts, uint32_t mask,
                                          uint32_t x) {
    uint32_t h = (x * 0x9E3779B1u) & mask;
    while (true) {
        uint32_t k = ld_agent(&keys[h]);
        if (k == kEmpty) {
            k = atomicCAS(&keys[h], kEmpty, x);
            if (k == kEmpty) k = x;
        }
        if (k == x) { atomicAdd(&counts[h], 1u); return; }
        h = (h + 1) & mask;
    }
}

__global__ __launch_bounds__(kBlock) void k_zcount(const uint32_t* __restrict__ edges, uint64_t m,
                                                   uint64_t K, uint64_t cnt, uint64_t n,
                                                   uint32_t* keys, uint32_t* counts, uint32_t mask,
                                                   DevState* st) {
    for (uint64_t j = (uint64_t)blockIdx.x * kBlock + threadIdx.x; j < cnt;
         j += (uint64_t)gridDim.x * kBlock) {
        const uint64_t i = (cnt == m) ? j : sample_index(j, m, K);
        const uint32_t u = edges[2 * i], v = edges[2 * i + 1];
        if (u >= n || v >= n) { atomicOr(&st->status, kStatusRange); continue; }
        if (u == v) continue;
        table_add(keys, counts, mask, u);
        table_add(keys, counts, mask, v);
    }
}

// Exact degree: dense counts over all entries.
__global__ __launch_bounds__(kBlock) void k_degfill(uint32_t* deg, uint64_t n, DevState* st) {
    uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i == 0) st_agent64(&st->zsel, 0);
    for (; i < n; i += (uint64_t)gridDim.x * kBlock) st_agent(&deg[i], 0u);
}

__global__ __launch_bounds__(kBlock) void k_degcount(const uint32_t* __restrict__ edges, uint64_t m,
                                                     uint64_t n, uint32_t* deg, DevState* st) {
    for (uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x; i < m;
         i += (uint64_t)gridDim.x * kBlock) {
        const uint32_t u = edges[2 * i], v = edges[2 * i + 1];
        if (u >= n || v >= n) { atomicOr(&st->status, kStatusRange); continue; }
        if (u == v) continue;
        atomicAdd(&deg[u], 1u);
        atomicAdd(&deg[v], 1u);
    }
}

__device__ __forceinline__ uint64_t pack_sel(uint32_t count, uint32_t id) {
    return count ? ((uint64_t)count << 32) | (uint64_t)(0xFFFFFFFFu - id) : 0;
}

// argmax over (count desc, id asc); ids come from a table (keys != nullptr) or
// are the indices of a dense count array.
// One atomic per workgroup on the packed key (atomics on one word serialise).
__global__ __launch_bounds__(kBlock) void k_zargmax(const uint32_t* keys, const uint32_t* counts,
                                                    uint64_t T, DevState* st) {
    __shared__ uint64_t s_best[kBlock / 64];
    uint64_t best = 0;
    // kR slots in flight per thread and few blocks: each block ends in an atomic on
    // the one word (1,024 blocks of one slot per thread: 14 us, 128 of eight: 5)
    constexpr int kR = 8;
    const uint64_t stride = (uint64_t)gridDim.x * kBlock;
    for (uint64_t i0 = (uint64_t)blockIdx.x * kBlock + threadIdx.x; i0 < T; i0 += kR * stride) {
        uint32_t id[kR], c[kR];
#pragma unroll
        for (int r = 0; r < kR; ++r) {
            const uint64_t i = i0 + r * stride;
            id[r] = !keys ? (uint32_t)i : i < T ? ld_agent(&keys[i]) : kEmpty;
            c[r] = i < T ? ld_agent(&counts[i]) : 0u;
        }
#pragma unroll
        for (int r = 0; r < kR; ++r) {
            if (id[r] == kEmpty && keys) continue;
            const uint64_t s = pack_sel(c[r], id[r]);
            best = s > best ? s : best;
        }
    }
    best = wave_max_u64(best);
    if ((threadIdx.x & 63) == 0) s_best[threadIdx.x >> 6] = best;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kBlock / 64; ++w) best = s_best[w] > best ? s_best[w] : best;
        if (best) atomicMax((unsigned long long*)&st->zsel, (unsigned long long)best);
    }
}

__global__ void k_zfinish(DevState* st, int use_hint, uint32_t hint) {
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        uint32_t z;
        if (use_hint) z = hint;
        else {
            uint64_t s = ld_agent64(&st->zsel);
            z = s ? 0xFFFFFFFFu - (uint32_t)(s & 0xFFFFFFFFu) : 0u;
        }
        st_agent(&st->zroot, z);
        st_agent(&st->zpub, z);
    }
}

// ---- Initial Push -------------------------------------------------------------
// For sampled entries (x, z) / (z, x) with x != z: P_x = z. Every x is still a
// root (run right after init), z has the smallest key, and all writers store
// the same value, so plain stores suffice.
__global__ __launch_bounds__(kBlock) void k_push(const uint32_t* __restrict__ edges, uint64_t m,
                                                 uint64_t K, uint64_t cnt, uint64_t n,
                                                 uint32_t* P, uint32_t* zbits, DevState* st) {
    const uint32_t z = ld_agent(&st->zroot);
    for (uint64_t j = (uint64_t)blockIdx.x * kBlock + threadIdx.x; j < cnt;
         j += (uint64_t)gridDim.x * kBlock) {
        const uint64_t i = (cnt == m) ? j : sample_index(j, m, K);
        const uint32_t u = edges[2 * i], v = edges[2 * i + 1];
        if (u >= n || v >= n || u == v) continue;
        uint32_t x = kEmpty;
        if (u == z) x = v;
        else if (v == z) x = u;
        if (x != kEmpty) {
            st_agent(&P[x], z);
            atomicOr(&zbits[x >> 5], 1u << (x & 31));
        }
    }
}

// Membership bitmap of the vertices connected to the zero root: cleared, with
// only z itself set.
__global__ __launch_bounds__(kBlock) void k_zbits_clear(uint32_t* zbits, uint64_t words,
                                                        const DevState* st) {
    const uint32_t z = ld_agent(&st->zroot);
    const uint64_t zw = z >> 5;
    for (uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x; i < words;
         i += (uint64_t)gridDim.x * kBlock)
        st_agent(&zbits[i], (i == zw) ? (1u << (z & 31)) : 0u);
}

// ---- hook ---------------------------------------------------------------------

constexpr int kEPT = 4;  // entries per thread per tile

// SiskinCC's messages (Sec. III, Algorithm 2): every successful link appends
// (linked root, new parent) to the log. One counter update per workgroup: the
// waves' counts are summed in LDS, thread 0 reserves the block's range, and
// each lane writes its records at its rank among the block's. Records past
// cap are counted but not written (the status word reports it). Must be
// reached by every thread of the block.
__device__ __forceinline__ void log_append(const uint32_t (&child)[kEPT],
                                           const uint32_t (&parent)[kEPT], uint32_t* log,
                                           uint64_t cap, unsigned long long* count,
                                           DevState* st) {
    __shared__ uint32_t s_w[kBlock / 64];
    __shared__ unsigned long long s_base;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint64_t mk[kEPT];
    uint32_t tot = 0;
#pragma unroll
    for (int k = 0; k < kEPT; ++k) {
        mk[k] = __ballot(child[k] != kEmpty);
        tot += (uint32_t)__popcll(mk[k]);
    }
    if (lane == 0) s_w[wave] = tot;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t t = 0;
        for (int w = 0; w < kBlock / 64; ++w) {
            const uint32_t x = s_w[w];
            s_w[w] = t;
            t += x;
        }
        s_base = t ? atomicAdd(count, (unsigned long long)t) : 0ull;
    }
    __syncthreads();
    uint64_t at = s_base + s_w[wave];
    const uint64_t below = (1ull << lane) - 1ull;
    bool full = false;
#pragma unroll
    for (int k = 0; k < kEPT; ++k) {
        if (child[k] != kEmpty) {
            const uint64_t i = at + (uint32_t)__popcll(mk[k] & below);
            if (i < cap) {
                u32x2 rec = {child[k], parent[k]};
                *reinterpret_cast<u32x2*>(log + 2 * i) = rec;
            } else {
                full = true;
            }
        }
        at += (uint32_t)__popcll(mk[k]);
    }
    if (full) atomicOr(&st->status, kStatusLogFull);
}

// Hooking of the kEPT entries (u[k], v[k]) a thread holds (entries beyond the
// input are passed as (0, 0): a self-loop, skipped); z is the zero root (ZR). Shared by the COO and the
// CSR launches. LOG (plain path only): the links made are appended to `log`
// (see log_append); every thread of the block must then call it. sym: the
// list holds every pair in both orders, so only the entries with u < v are
// hooked (each edge once; Sec. II: processing (u,v) makes (v,u) a no-op).
template <bool ZR, int SPLIT, bool LOG, bool LINKZ = false>
__device__ __forceinline__ void hook_entries(uint32_t (&u)[kEPT], uint32_t (&v)[kEPT], uint32_t n,
                                             uint32_t z, uint32_t* P, uint32_t* zbits,
                                             DevState* st, uint32_t* log, uint64_t log_cap,
                                             unsigned long long* log_count, bool sym) {
    static_assert(!(ZR && LOG), "the update log belongs to the plain path");
    bool bad = false;
#pragma unroll
    for (int k = 0; k < kEPT; ++k) {
        if (u[k] >= n || v[k] >= n) { bad = true; u[k] = v[k] = 0; }
    }
    if (bad) atomicOr(&st->status, kStatusRange);
    bool live[kEPT];
#pragma unroll
    for (int k = 0; k < kEPT; ++k) live[k] = sym ? u[k] < v[k] : u[k] != v[k];
    // A set bit means "connected to z". Both endpoints set: the entry is
    // redundant. Exactly one set: by default the entry's whole effect is to
    // connect the other endpoint to z, which its bit records (compress passes a
    // mark on to the root of its tree), so it is set and P is not touched; only
    // entries with neither endpoint marked go on to the walks. LINKZ instead
    // walks the unmarked endpoint's tree and links it under z, marking both:
    // dearer per entry, but every vertex of that tree then walks to z and is
    // marked when an entry reaches it, so the bitmap grows faster (the
    // regrouped hook's short warm-up, which seeds its filter, wants that).
    bool inu[kEPT] = {}, inv[kEPT] = {};
    if (ZR) {
        // Marking: the second endpoint's word is read coherently, so that the
        // commonest mark (first endpoint marked, second not) needs only the atomic.
        uint32_t bu[kEPT], bv[kEPT];
#pragma unroll
        for (int k = 0; k < kEPT; ++k) {
            bu[k] = live[k] ? zbits[u[k] >> 5] : 0u;
            bv[k] = !live[k] ? 0u : (LINKZ ? zbits[v[k] >> 5] : ld_agent(&zbits[v[k] >> 5]));
        }
#pragma unroll
        for (int k = 0; k < kEPT; ++k) {
            inu[k] = (bu[k] >> (u[k] & 31)) & 1u;
            inv[k] = (bv[k] >> (v[k] & 31)) & 1u;
            if (!LINKZ && live[k] && inu[k] != inv[k]) {
                if (inu[k]) atomicOr(&zbits[v[k] >> 5], 1u << (v[k] & 31));
                else zbit_set(zbits, u[k]);
            }
            live[k] = live[k] && !(inu[k] && inv[k]) && (LINKZ || (!inu[k] && !inv[k]));
        }
    }
    // LINKZ: a marked endpoint has root z (walk from z, no read of P)
    uint32_t wu[kEPT], wv[kEPT];
#pragma unroll
    for (int k = 0; k < kEPT; ++k) {
        wu[k] = (LINKZ && inu[k]) ? z : u[k];
        wv[k] = (LINKZ && inv[k]) ? z : v[k];
    }
    uint32_t pu[kEPT], pv[kEPT];
#pragma unroll
    for (int k = 0; k < kEPT; ++k) {
        pu[k] = !live[k] ? 0u : ((LINKZ && inu[k]) ? z : P[wu[k]]);
        pv[k] = !live[k] ? 0u : ((LINKZ && inv[k]) ? z : P[wv[k]]);
    }
    uint32_t child[kEPT], parent[kEPT];
#pragma unroll
    for (int k = 0; k < kEPT; ++k) {
        child[k] = kEmpty;
        parent[k] = kEmpty;
        if (!live[k]) continue;
        // a common parent, or one endpoint the parent of the other: same tree
        uint32_t r;
        if (pu[k] == pv[k]) r = pu[k];
        else if (pu[k] == wv[k]) r = wv[k];
        else if (pv[k] == wu[k]) r = wu[k];
        else r = link<ZR, SPLIT>(P, wu[k], pu[k], wv[k], pv[k], z, LOG ? &child[k] : nullptr);
        if (LOG) parent[k] = r;
        if (ZR && r == z) {
            if (!inu[k]) zbit_set(zbits, u[k]);
            if (!inv[k]) zbit_set(zbits, v[k]);
        }
    }
    if (LOG) log_append(child, parent, log, log_cap, log_count, st);
}

// One tile of kBlock*kEPT entries per workgroup; each thread loads its kEPT
// entries (coalesced, non-temporal: the edge stream must not evict P) and
// issues all their parent reads before walking any of them.
// With a zero root (ZR) the membership bitmap is consulted first: an entry
// with an endpoint known to be connected to z is settled by its bits without
// reading P (the single-GPU form of treating zero-converged vertices
// specially, Sec. IV). Bits only go from 0 to 1 and only for vertices
// connected to z, so a stale or missing bit just sends the entry down the
// ordinary path.
template <bool ZR, int SPLIT, bool LOG = false, bool LINKZ = false>
__global__ __launch_bounds__(kBlock) void k_hook(const uint32_t* __restrict__ edges, uint64_t m,
                                                 uint32_t n, uint32_t* P, uint32_t* zbits,
                                                 DevState* st, uint32_t sym,
                                                 uint32_t* log = nullptr, uint64_t log_cap = 0,
                                                 unsigned long long* log_count = nullptr) {
    const uint32_t z = ZR ? ld_agent(&st->zroot) : 0u;
    const uint64_t tile = (uint64_t)blockIdx.x * (kBlock * kEPT);
    const u32x2* E = reinterpret_cast<const u32x2*>(edges);
    uint32_t u[kEPT], v[kEPT];
#pragma unroll
    for (int k = 0; k < kEPT; ++k) {
        const uint64_t e = tile + (uint64_t)k * kBlock + threadIdx.x;
        u32x2 uv = {0u, 0u};
        if (e < m) uv = __builtin_nontemporal_load(E + e);
        u[k] = uv.x;
        v[k] = uv.y;
    }
    hook_entries<ZR, SPLIT, LOG, LINKZ>(u, v, n, z, P, zbits, st, log, log_cap, log_count,
                                        sym != 0);
}

// The direct hook of a solve whose sample showed no giant component: k_hook's
// tiles, left at once where the filter runs instead. The entries of the second
// sample (every skip-th run of kSampleRun) are hooked already.
static_assert(kBlock == kSampleRun, "a block's k-th entries are one run of the sample");
template <bool ZR, int SPLIT, bool LINKZ, typename T>
__global__ __launch_bounds__(kBlock) void k_hook_gated(const T edges, uint64_t m,
                                                       uint32_t n, uint32_t* P, uint32_t* zbits,
                                                       DevState* st, uint32_t sym, uint32_t skip,
                                                       Gate gate) {
    if (gated_off(gate)) return;
    const uint32_t z = ZR ? ld_agent(&st->zroot) : 0u;
    for (uint64_t tile = (uint64_t)blockIdx.x * (kBlock * kEPT); tile < m;
         tile += (uint64_t)gridDim.x * (kBlock * kEPT)) {
        uint32_t u[kEPT], v[kEPT];
#pragma unroll
        for (int k = 0; k < kEPT; ++k) {
            const uint64_t e = tile + (uint64_t)k * kBlock + threadIdx.x;
            u32x2 uv = {0u, 0u};
            if (e < m && (tile / kBlock + k) % skip) uv = load_entry(edges, e);
            u[k] = uv.x;
            v[k] = uv.y;
        }
        hook_entries<ZR, SPLIT, false, LINKZ>(u, v, n, z, P, zbits, st, nullptr, 0, nullptr, sym != 0);
    }
}

// ---- CSR input -------------------------------------------------------------------
// Row u of a CSR graph holds the entries (u, adj[j]) for j in [off[u], off[u+1]);
// these are the same unordered pairs as a COO list, sorted by first endpoint,
// so every consecutive run of a tile shares u (and its parent reads).
// A workgroup takes kCsrTile consecutive positions and needs the row of each:
// tstart[t] is the row that holds position t*kCsrTile (written by k_csr_tiles,
// one thread per row), and the rows that start inside the tile are found by a
// sweep of the rows between the tile's first and next tile's first row plus a
// max-scan in LDS. A tile that spans more than kSweepMax rows (long runs of
// empty rows) searches each position's row instead, so no workgroup's work
// grows with the length of such runs beyond a logarithm.
static_assert(kCsrTile == kBlock * kEPT, "a workgroup's tile");
constexpr uint32_t kSweepMax = 4 * kCsrTile;

// Checks the offsets (non-decreasing, off[0] = 0, off[n] = m) and writes the
// first row of every tile. Indices are clamped so that invalid offsets never
// make an access leave its array; the result is then only reported.
__global__ __launch_bounds__(kBlock) void k_csr_tiles(const uint64_t* __restrict__ off, uint64_t n,
                                                      uint64_t m, uint32_t* __restrict__ tstart,
                                                      uint64_t ntiles, DevState* st) {
    bool bad = false;
    for (uint64_t v = (uint64_t)blockIdx.x * kBlock + threadIdx.x; v < n;
         v += (uint64_t)gridDim.x * kBlock) {
        const uint64_t lo = off[v], hi = off[v + 1];
        if (hi < lo || hi > m || (v == 0 && lo != 0)) { bad = true; continue; }
        if (hi == lo) continue;
        for (uint64_t t = (lo + kCsrTile - 1) / kCsrTile; t * kCsrTile < hi && t < ntiles; ++t)
            tstart[t] = (uint32_t)v;
    }
    if (bad) atomicOr(&st->status, kStatusBadOffsets);
}

// Exact maximum degree from the row lengths (Algorithm 4 reads it from CSR),
// ties to the lowest ID: the packed (count, ~ID) key is reduced over the
// workgroup first and takes one atomic per workgroup (atomics on one word
// serialise), four rows in flight per thread.
__global__ __launch_bounds__(kBlock) void k_csr_zmax(const uint64_t* __restrict__ off, uint64_t n,
                                                     DevState* st) {
    __shared__ uint64_t s_best[kBlock / 64];
    uint64_t best = 0;
    const uint64_t stride = (uint64_t)gridDim.x * kBlock;
    for (uint64_t v0 = (uint64_t)blockIdx.x * kBlock + threadIdx.x; v0 < n; v0 += 4 * stride) {
        uint64_t lo[4], hi[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const uint64_t v = v0 + r * stride;
            const uint64_t vs = v < n ? v : n - 1;
            lo[r] = off[vs];
            hi[r] = off[vs + 1];
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const uint64_t v = v0 + r * stride;
            const uint64_t d = (v < n && hi[r] > lo[r]) ? hi[r] - lo[r] : 0;
            const uint64_t sel = pack_sel(d > 0xFFFFFFFFull ? 0xFFFFFFFFu : (uint32_t)d, (uint32_t)v);
            best = sel > best ? sel : best;
        }
    }
    best = wave_max_u64(best);
    if ((threadIdx.x & 63) == 0) s_best[threadIdx.x >> 6] = best;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kBlock / 64; ++w) best = s_best[w] > best ? s_best[w] : best;
        if (best) atomicMax((unsigned long long*)&st->zsel, (unsigned long long)best);
    }
}

__global__ void k_zsel_reset(DevState* st) {
    if (threadIdx.x == 0 && blockIdx.x == 0) st_agent64(&st->zsel, 0);
}

// What the host needs before it can launch: the entry count and (with the maximum
// degree found) zsel, to pinned host memory.
__global__ void k_csr_head(const uint64_t* end, const DevState* st, int zr, uint64_t* host) {
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        __hip_atomic_store(host, ld_agent64(end), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        __hip_atomic_store(host + 1, zr ? ld_agent64(&st->zsel) : 0ull, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

// Initial Push over the zero root's whole row (Algorithm 4 initial-push loop).
__global__ __launch_bounds__(kBlock) void k_csr_push(const uint64_t* __restrict__ off,
                                                     const uint32_t* __restrict__ adj, uint64_t n,
                                                     uint64_t m, uint32_t* P, uint32_t* zbits,
                                                     DevState* st) {
    const uint32_t z = ld_agent(&st->zroot);
    uint64_t lo = off[z], hi = off[z + 1];
    if (hi > m) hi = m;
    bool bad = false;
    for (uint64_t j = lo + (uint64_t)blockIdx.x * kBlock + threadIdx.x; j < hi;
         j += (uint64_t)gridDim.x * kBlock) {
        const uint32_t x = adj[j];
        if (x >= n) { bad = true; continue; }
        if (x == z) continue;
        st_agent(&P[x], z);
        zbit_set(zbits, x);
    }
    if (bad) atomicOr(&st->status, kStatusRange);
}

// Workgroup t takes tile t (a launch may cover a prefix of the tiles, as the
// warm-up does).
template <bool ZR, int SPLIT, bool LINKZ = false>
__global__ __launch_bounds__(kBlock) void k_csr_hook(const uint64_t* __restrict__ off,
                                                     const uint32_t* __restrict__ adj, uint32_t n,
                                                     uint64_t m, const uint32_t* __restrict__ tstart,
                                                     uint64_t ntiles, uint32_t* P, uint32_t* zbits,
                                                     DevState* st, uint32_t sym,
                                                     Gate gate = Gate{nullptr, 0u}) {
    __shared__ uint32_t head[kCsrTile];
    __shared__ uint32_t s_wmax[kBlock / 64];
    if (gated_off(gate)) return;
    const uint32_t z = ZR ? ld_agent(&st->zroot) : 0u;
    if (blockIdx.x >= ntiles) return;
    {
    const uint64_t t = blockIdx.x;
    const uint64_t p0 = t * kCsrTile;
    uint32_t ua = tstart[t];
    uint32_t ub = (t + 1 < ntiles) ? tstart[t + 1] : n - 1;
    if (ua >= n) ua = n - 1;                            // only with invalid offsets
    if (ub >= n || ub < ua) ub = ua;
    uint32_t v[kEPT];
#pragma unroll
    for (int k = 0; k < kEPT; ++k) {
        const uint64_t p = p0 + (uint64_t)k * kBlock + threadIdx.x;
        v[k] = p < m ? __builtin_nontemporal_load(adj + p) : 0u;
    }
    uint32_t u[kEPT];
    if (ub - ua <= kSweepMax) {
        for (int i = threadIdx.x; i < kCsrTile; i += kBlock) head[i] = 0;
        __syncthreads();
        if (threadIdx.x == 0) head[0] = ua;
        for (uint64_t x0 = (uint64_t)ua + 1; x0 <= ub; x0 += 4 * kBlock) {
            uint64_t lo[4], hi[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const uint64_t x = x0 + r * kBlock + threadIdx.x;
                const uint64_t xs = x <= ub ? x : ub;
                lo[r] = off[xs];
                hi[r] = off[xs + 1];
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const uint64_t x = x0 + r * kBlock + threadIdx.x;
                if (x <= ub && lo[r] < hi[r] && lo[r] >= p0 && lo[r] < p0 + kCsrTile)
                    head[lo[r] - p0] = (uint32_t)x;
            }
        }
        __syncthreads();
        // inclusive max-scan of head: thread i owns head[4i .. 4i + 3]
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
        uint32_t h[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) h[r] = head[4 * threadIdx.x + r];
#pragma unroll
        for (int r = 1; r < 4; ++r) h[r] = max(h[r], h[r - 1]);
        uint32_t incl = h[3];
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t y = __shfl_up(incl, o, 64);
            if (lane >= o) incl = max(incl, y);
        }
        if (lane == 63) s_wmax[wave] = incl;
        uint32_t before = __shfl_up(incl, 1, 64);
        if (lane == 0) before = 0;
        __syncthreads();
        for (int w = 0; w < wave; ++w) before = max(before, s_wmax[w]);
#pragma unroll
        for (int r = 0; r < 4; ++r) head[4 * threadIdx.x + r] = max(h[r], before);
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kEPT; ++k) u[k] = head[k * kBlock + threadIdx.x];
    } else {
        // the last row x in [ua, ub] with off[x] <= p owns p
#pragma unroll
        for (int k = 0; k < kEPT; ++k) {
            const uint64_t p = p0 + (uint64_t)k * kBlock + threadIdx.x;
            uint32_t lo = ua, hi = ub;
            while (lo < hi) {
                const uint32_t mid = lo + (hi - lo + 1) / 2;
                if (off[mid] <= p) lo = mid;
                else hi = mid - 1;
            }
            u[k] = lo;
        }
    }
#pragma unroll
    for (int k = 0; k < kEPT; ++k) {
        const uint64_t p = p0 + (uint64_t)k * kBlock + threadIdx.x;
        if (p >= m) u[k] = v[k] = 0;
    }
    hook_entries<ZR, SPLIT, false, LINKZ>(u, v, n, z, P, zbits, st, nullptr, 0, nullptr,
                                          sym != 0);
    __syncthreads();                                    // head of this tile fully used
    }
}

// ---- compress (pointer jumping) ----------------------------------------------------
// P_v <- root(v). No entry is linked any more, but another XCD's L2 can still
// hold a copy of an entry read while its vertex was a root, and that copy has
// been observed to survive into this kernel. A walk may follow such stale
// (still ancestor) values freely, but the two facts the label rests on are read
// coherently: the vertex's own entry, and the root the walk stops at (a stale
// "root" would end the walk early); if the coherent value differs, the walk
// continues from it.
// With a zero root the membership bitmap is part of the result: a set bit means
// "connected to z" (the tiled hook records such links only as bits, see
// cc_tiled.hip), so a tree that holds a marked vertex belongs to z's component.
// Here every marked vertex passes its mark on to its root; k_resolve then
// relabels the members of marked trees.
// The same pass finds the smallest member of z's component (per block;
// k_resolve reduces the blocks' minima). Outside z's tree every tree is rooted at its smallest
// ID (its keys are the IDs), so the candidates are: each member of z's tree
// (z included), each root whose own bit is set, and the root of each marked
// vertex. A root whose bit is set during this pass is the root of a marked
// vertex, so it is counted through that vertex.
// Each thread takes kVPT vertices per step of its grid-stride loop and issues
// their first reads together (one read in flight per thread would leave these
// whole-array passes latency-bound).
constexpr int kVPT = 4;

template <bool ZR>
__global__ __launch_bounds__(kBlock) void k_compress(uint32_t* P, uint64_t n, DevState* st,
                                                     uint32_t* zbits, uint32_t* bmin,
                                                     Gate gate = Gate{nullptr, 0u}) {
    if (gated_off(gate)) return;
    const uint32_t z = ZR ? ld_agent(&st->zroot) : 0u;
    const uint64_t stride = (uint64_t)gridDim.x * kBlock;
    uint32_t local_min = kEmpty;
    uint32_t passed = kEmpty;                 // root this thread last passed a mark to
    for (uint64_t v0 = (uint64_t)blockIdx.x * kBlock + threadIdx.x; v0 < n; v0 += kVPT * stride) {
        uint32_t pv[kVPT], bw[kVPT];
#pragma unroll
        for (int i = 0; i < kVPT; ++i) {
            const uint64_t v = v0 + i * stride;
            pv[i] = v < n ? ld_agent(&P[v]) : (uint32_t)v;
            if (ZR) bw[i] = v < n ? ld_agent(&zbits[v >> 5]) : 0u;
        }
#pragma unroll
        for (int i = 0; i < kVPT; ++i) {
        const uint64_t v = v0 + i * stride;
        const uint32_t p = pv[i];
        uint32_t r = (uint32_t)v;
        const bool marked = ZR && ((bw[i] >> (v & 31)) & 1u);
        uint32_t pass = kEmpty;               // root to pass v's mark to
        if (ZR && v < n && p == (uint32_t)v && ((uint32_t)v == z || marked))
            local_min = min(local_min, (uint32_t)v);
        if (v < n && p != (uint32_t)v) {
            r = p;
            while (true) {
                uint32_t q = P[r];
                while (q != r) { r = q; q = P[r]; }
                if (ZR && r == z) break;          // the zero root is never linked
                q = ld_agent(&P[r]);
                if (q == r) break;
                r = q;
            }
            if (r != p) st_agent(&P[v], r);
            if (ZR && r == z) {
                local_min = min(local_min, (uint32_t)v);
            } else if (marked) {
                pass = r;
                local_min = min(local_min, r);
            }
        }
        if (ZR) {
            // one lane per distinct root passes the mark: the members of a marked
            // tree share it, and a coherent read of its word by every one of them
            // serialises (ER n = 1.1 M, 2.5 M entries: pass 210 -> 60 us)
            uint64_t left = __ballot(pass != kEmpty && pass != passed);
            while (left) {
                const int l = __ffsll((unsigned long long)left) - 1;
                const uint32_t first = __shfl(pass, l, 64);
                if ((int)(threadIdx.x & 63) == l) zbit_set(zbits, first);
                if (pass == first) passed = first;
                left &= ~__ballot(pass == first);
            }
        }
        }
    }
    if (ZR) {
        // one value per block; k_resolve reduces them (one atomic per block on a
        // single word would serialise)
        __shared__ uint32_t s_min[kBlock / 64];
        local_min = wave_min_u32(local_min);
        if ((threadIdx.x & 63) == 0) s_min[threadIdx.x >> 6] = local_min;
        __syncthreads();
        if (threadIdx.x == 0) {
            uint32_t b = s_min[0];
            for (int w = 1; w < kBlock / 64; ++w) b = min(b, s_min[w]);
            st_agent(&bmin[blockIdx.x], b);
        }
    }
}

// Zero root only, after k_compress: every member of z's component (its root is
// z, or v or its root is marked) gets the label z, or with FINAL the component's
// smallest ID at once (no k_canon pass needed). Every block reduces compress's
// nb <= kZrGrid per-block minima for itself (8 KB; a launch of its own for that
// cost 5 us); block 0 records the result. Marks are read coherently: they were
// set by atomics.
template <bool FINAL>
__global__ __launch_bounds__(kBlock) void k_resolve(uint32_t* P, uint64_t n, DevState* st,
                                                    const uint32_t* zbits, const uint32_t* bmin,
                                                    uint32_t nb, int pub, Gate gate) {
    if (gated_off(gate)) return;
    __shared__ uint32_t s_min[kBlock / 64];
    const uint32_t z = ld_agent(&st->zroot);
    uint32_t lab = z;
    if (FINAL || blockIdx.x == 0) {
        uint32_t x = kEmpty;
        for (uint32_t i = threadIdx.x; i < nb; i += kBlock) x = min(x, ld_agent(&bmin[i]));
        x = wave_min_u32(x);
        if ((threadIdx.x & 63) == 0) s_min[threadIdx.x >> 6] = x;
        __syncthreads();
        for (int w = 0; w < kBlock / 64; ++w) x = min(x, s_min[w]);
        if (FINAL) lab = x;
        if (pub && blockIdx.x == 0 && threadIdx.x == 0) st_agent(&st->mpub, x);
    }
    const uint64_t stride = (uint64_t)gridDim.x * kBlock;
    for (uint64_t v0 = (uint64_t)blockIdx.x * kBlock + threadIdx.x; v0 < n; v0 += kVPT * stride) {
        uint32_t rr[kVPT], bv[kVPT];
#pragma unroll
        for (int i = 0; i < kVPT; ++i) {
            const uint64_t v = v0 + i * stride;
            const uint64_t vs = v < n ? v : v0;          // v0 < n
            rr[i] = ld_agent(&P[vs]);
            bv[i] = ld_agent(&zbits[vs >> 5]);
        }
#pragma unroll
        for (int i = 0; i < kVPT; ++i) {
            const uint64_t v = v0 + i * stride;
            if (v >= n) continue;
            const uint32_t r = rr[i];
            const bool inz = r == z || ((bv[i] >> (v & 31)) & 1u) ||
                             (r != (uint32_t)v && ((ld_agent(&zbits[r >> 5]) >> (r & 31)) & 1u));
            if (inz && r != lab) st_agent(&P[v], lab);
        }
    }
}

// ---- relabel the zero root's component to its smallest ID ---------------------------
__global__ __launch_bounds__(kBlock) void k_canon(uint32_t* L, uint64_t n, const DevState* st) {
    const uint32_t z = ld_agent(&st->zpub), mz = ld_agent(&st->mpub);
    if (mz == z || mz == kEmpty) return;
    const uint64_t stride = (uint64_t)gridDim.x * kBlock;
    for (uint64_t v0 = (uint64_t)blockIdx.x * kBlock + threadIdx.x; v0 < n; v0 += kVPT * stride) {
        uint32_t l[kVPT];
#pragma unroll
        for (int i = 0; i < kVPT; ++i) {
            const uint64_t v = v0 + i * stride;
            l[i] = v < n ? ld_agent(&L[v]) : kEmpty;
        }
#pragma unroll
        for (int i = 0; i < kVPT; ++i)
            if (l[i] == z) st_agent(&L[v0 + i * stride], mz);
    }
}

// ---- coherence point ----------------------------------------------------------------------
__global__ void k_cohere() {
    if (threadIdx.x == 0) {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "agent");
        __builtin_amdgcn_s_waitcnt(0);           // the write-back and invalidate complete here
    }
}

int cohere(hipStream_t stream) {
    // 64 single-wave workgroups: consecutive workgroups are dealt to the XCDs in
    // turn, so every XCD runs several of them.
    k_cohere<<<64, 64, 0, stream>>>();
    CCM_HIP(hipGetLastError());
    return CC_OK;
}

// ---- host-side launchers ---------------------------------------------------------------


static uint32_t grid_for(uint64_t work, uint64_t per_block, uint32_t cap) {
    uint64_t g = (work + per_block - 1) / per_block;
    if (g < 1) g = 1;
    return (uint32_t)(g < cap ? g : cap);
}


int run_init(Slot* s, uint64_t n, uint32_t* P, hipStream_t stream) {
    s->cur_n = n;
    s->zr_ready = false;
    k_init<<<grid_for(n, kBlock * 4, kGridCap), kBlock, 0, stream>>>(P, n, s->st);
    CCM_HIP(hipGetLastError());
    return CC_OK;
}

// Whether the hook tests every entry against the whole bitmap in LDS
// (cc_filter.hip) instead of hooking each in P. It needs a sample, two more
// passes over P and the bitmap, about 40 us in all, and drops little where the
// sample (n entries at most) leaves no giant component. Whole solves, direct
// against LDS (us): R-MAT n = 2^16, 2^20 entries 128 against 94 (plain); n =
// 1,000,003, 15 M entries 924 against 193 (zero root); ER n = 1 M, 4 M entries
// 277 against 271 (plain), 691 against 323 (zero root).
bool lds_eligible(uint64_t n, uint64_t m) {
    return n <= lds_bits_max_n() && m >= (1ull << 18) && m >= 2 * n;
}
// Blocks of the zero root's compress and resolve (8 per CU).
constexpr uint32_t kZrGrid = 2048;

static uint64_t sample_count(uint64_t m, uint64_t K) { return m <= K ? m : K; }

// Size the membership bitmap for n vertices and clear it (only z set). Marks the
// slot ready for a zero-root hook when n is the current solve's.
static int zbits_grow(Slot* s, uint64_t n, hipStream_t stream) {
    const uint64_t words = (n + 31) / 32;
    if (s->zbits_cap < words) {
        if (s->no_grow) return fail(CC_ENOMEM, "zero-root bitmap exceeds the fixed scratch");
        if (stream_capturing(stream)) return fail(CC_ENOMEM, "zero-root bitmap cannot grow under capture");
        CCM_HIP(hipStreamSynchronize(stream));
        int rc = slot_outgrow(s, s->zbits, &s->zbits_captured);
        if (rc) return rc;
        s->zbits = nullptr;
        s->zbits_cap = 0;
        if (hipMalloc(&s->zbits, words * sizeof(uint32_t)) != hipSuccess) {
            (void)hipGetLastError();
            s->zbits = nullptr;
            return fail(CC_ENOMEM, "zero-root bitmap allocation failed");
        }
        s->zbits_cap = words;
    } else if (!s->no_grow) {
        note_capture(&s->zbits_captured, stream);
    }
    return CC_OK;
}

int zbits_reset(Slot* s, uint64_t n, hipStream_t stream) {
    const uint64_t words = (n + 31) / 32;
    int rc = zbits_grow(s, n, stream);
    if (rc) return rc;
    k_zbits_clear<<<grid_for(words, kBlock, kGridCap), kBlock, 0, stream>>>(s->zbits, words, s->st);
    CCM_HIP(hipGetLastError());
    s->zr_ready = (n == s->cur_n);
    return CC_OK;
}

int run_zroot(Slot* s, uint64_t n, uint64_t m, const uint32_t* edges, uint32_t flags,
              uint32_t hint, hipStream_t stream) {
    if (flags & CC_F_ZROOT_HINT) {
        k_zfinish<<<1, 64, 0, stream>>>(s->st, 1, hint);
        CCM_HIP(hipGetLastError());
        return zbits_reset(s, n, stream);
    }
    if (flags & CC_F_ZROOT_EXACT) {
        if (s->deg_cap < n && s->no_grow)
            return fail(CC_ENOMEM, "exact-degree counts need memory beyond the fixed scratch");
        if (s->deg_cap < n) {
            if (stream_capturing(stream))
                return fail(CC_ENOMEM, "exact-degree counts cannot grow under capture");
            int rc = slot_outgrow(s, s->deg, &s->deg_captured);
            if (rc) return rc;
            s->deg = nullptr;
            s->deg_cap = 0;
            if (hipMalloc(&s->deg, n * sizeof(uint32_t)) != hipSuccess) {
                (void)hipGetLastError();
                s->deg = nullptr;
                return fail(CC_ENOMEM, "exact-degree scratch allocation failed");
            }
            s->deg_cap = n;
        } else if (!s->no_grow) {
            note_capture(&s->deg_captured, stream);
        }
        k_degfill<<<grid_for(n, kBlock, kGridCap), kBlock, 0, stream>>>(s->deg, n, s->st);
        if (m) k_degcount<<<grid_for(m, kBlock, kGridCap), kBlock, 0, stream>>>(edges, m, n, s->deg, s->st);
        k_zargmax<<<grid_for(n, 8 * kBlock, kZrGrid), kBlock, 0, stream>>>(nullptr, s->deg, n, s->st);
    } else {
        const uint64_t K = s->samples;
        const uint64_t cnt = sample_count(m, K);
        k_zfill<<<grid_for(s->table, kBlock, 1024), kBlock, 0, stream>>>(s->hkeys, s->hcounts,
                                                                          s->table, s->st);
        if (cnt)
            k_zcount<<<grid_for(cnt, kBlock, 1024), kBlock, 0, stream>>>(
                edges, m, K, cnt, n, s->hkeys, s->hcounts, s->table - 1, s->st);
        k_zargmax<<<grid_for(s->table, 8 * kBlock, 1024), kBlock, 0, stream>>>(s->hkeys, s->hcounts,
                                                                                s->table, s->st);
    }
    k_zfinish<<<1, 64, 0, stream>>>(s->st, 0, 0);
    CCM_HIP(hipGetLastError());
    return zbits_reset(s, n, stream);
}

int run_push(Slot* s, uint64_t n, uint64_t m, const uint32_t* edges, uint32_t* P,
             hipStream_t stream) {
    if (!s->zr_ready || s->cur_n != n)
        return fail(CC_EINVAL, "cc_push needs cc_init then cc_zroot on the same n");
    const uint64_t K = s->samples;
    const uint64_t cnt = sample_count(m, K);
    if (!cnt) return CC_OK;
    k_push<<<grid_for(cnt, kBlock, 1024), kBlock, 0, stream>>>(edges, m, K, cnt, n, P, s->zbits,
                                                               s->st);
    CCM_HIP(hipGetLastError());
    return CC_OK;
}

// The hook against the bitmap of one root's component (cc_filter.hip,
// cc_tiled.hip), in P after init, or with zr after zroot and push too: a sample
// hooked by Algorithm 1 / 3, pointer jumping, the bitmap, every entry against it.
// On a plain solve the most frequent root plays the zero root's part from there
// on (it is a root, so its key can become the smallest one).
//
// A skewed graph's giant component shows in a small sample; a uniform one's needs
// about n / 2 entries, so where the device finds none in the small sample, one of
// up to n entries, half the list at most, is tried. If that shows none either, the
// whole-bitmap pass (passes 0) hooks what it must in P, which costs it little; the
// sizes that were regrouped before there was a sample (tiled_eligible) hook their
// regrouped entries over the flat forest that the sample leaves, by tiles or by
// first-endpoint buckets; rows take the CSR hook, and the rest the direct hook, without
// building the tiles. Whole solves, always filtering / direct / as decided here (us):
// R-MAT n = 3 M, 12 M entries 301 / 1412 / 285; ER n = 16 M, 60 M entries 4872 / 3970 /
// 2353; grid n = 4 M, 8 M entries 9024 / 1050 / 1080. Without a giant component, buckets
// from the start / direct / regrouped after the sample: 12 parts dealt over n = 4 M, 64 M
// entries 2003 / 2766 / 1577; 20 parts dealt over n = 11 M, 128 M entries 3926 / 5768 /
// 3938; 20 parts side by side, n = 64 M, 512 M entries 20859 / 24051 / 19068; 12 parts
// dealt over n = 24 M, 256 M entries 8032 / 10849 / 9567 (2,021 of it the sample).
//
// The regrouped zero-root hook of two partition passes takes its small sample by
// the linking form instead, the first 1/1024 of the entries, which sets the bits
// itself: rewriting a bitmap of that size would cost more than it saves (0.5 ms
// of R-MAT-26's 10.2).
constexpr uint64_t kSampleSmall = 1ull << 20;

static int hook_by_bits(Slot* s, uint64_t n, uint64_t m, EdgeList E, uint32_t* P, uint32_t* bits,
                        int passes, bool zr, bool own_bits, bool p32, uint32_t flags,
                        hipStream_t stream) {
    const bool split = split_walks(flags, n);
    const bool sym = flags & CC_F_SYMMETRIC;
    DevState* st = s->st;
    const Gate always{}, again{&st->giant1, 0u}, on{passes ? &st->giant : nullptr, 1u};
    // sizes in entries that are hooked: one of two on a symmetric list
    const uint64_t live = sym ? m / 2 : m, per = sym ? 2 : 1;
    const uint64_t full = (passes ? std::min(live / 2, n - n / 16) : std::min(live / 4, n)) * per;
    const uint64_t small = std::min(full, std::min<uint64_t>(n / 16, kSampleSmall) * per);
    int rc;
    auto compress = [&](Gate g) -> int {
        if (zr)
            k_compress<true><<<grid_for(n, kBlock, kZrGrid), kBlock, 0, stream>>>(P, n, st, bits, s->bmin, g);
        else
            k_compress<false><<<grid_for(n, kBlock, kGridCap), kBlock, 0, stream>>>(P, n, st, nullptr,
                                                                                 nullptr, g);
        CCM_HIP(hipGetLastError());
        return CC_OK;
    };
    // Rows without a giant component: the CSR hook over the flat forest. Its lanes share
    // their first endpoint's reads, and it needs no search per entry (paths n = 1 M, 3 M
    // entries: hook 345 us by positions in k_hook_lds, 218 so).
    auto hook_rows = [&]() -> int {
        const CsrList& r = *E.csr;
        const Gate off{&st->giant, 0u};
        auto hook = split ? &k_csr_hook<true, 1, true> : &k_csr_hook<true, kLateSplit, true>;
        hook<<<(uint32_t)r.ntiles, kBlock, 0, stream>>>(r.off, r.adj, r.n, m, r.tstart, r.ntiles, P, bits, st,
                                                        sym ? 1u : 0u, off);
        CCM_HIP(hipGetLastError());
        return CC_OK;
    };
    if (!passes) {
        const int mode = zr ? kBitsZr : kBitsPick;
        if ((rc = run_warm(n, m, E, P, st, zr, sym, small, always, stream))) return rc;
        if ((rc = compress(always))) return rc;
        if ((rc = run_giant_bits(n, m, E, P, bits, st, mode, 1, always, stream))) return rc;
        if ((rc = run_warm(n, m, E, P, st, zr, sym, full, again, stream))) return rc;
        if ((rc = compress(again))) return rc;
        if ((rc = run_giant_bits(n, m, E, P, bits, st, mode, 2, again, stream))) return rc;
        if ((rc = run_hook_lds(n, m, E, P, bits, st, split, sym, s->device, stream))) return rc;
        return E.csr ? hook_rows() : CC_OK;
    }
    const bool link_first = zr && passes == 2;
    if (link_first) {
        const uint64_t m0 = m >> 10;
        if (m0 && (rc = run_hook(s, n, m0, (const uint32_t*)E.p, P,
                                 CC_F_ZROOT | CC_F_NO_TILE | kHookLinkZ | (flags & CC_F_SYMMETRIC), stream)))
            return rc;
        // Below 5/4 entries per vertex half of a uniform list shows no giant
        // component even where the whole has one, so the filter takes every list
        // (ER n = 67 M, 60 M entries: 7.1 ms filtered, 8.6 direct, 9.2 sampled and
        // then direct; a twentieth of R-MAT-26, n = 71 M, 52 M entries: 1.4, 2.7). The
        // sample only decides whether the survivors' bits are tested again. Beyond
        // 256 slices a larger sample's marks are worth more (a sixteenth of R-MAT-28:
        // 7.07 ms sampled, 7.47 so).
        if (4 * live < 5 * n && tiled_eligible(n, m, true)) {
            if ((rc = run_find_giant(n, m, E, P, bits, st, zr, 0, stream))) return rc;
            return run_filter(s, n, m, E, P, bits, passes, own_bits, p32, sym, always, kNoOther, stream);
        }
    } else if ((rc = run_warm(n, m, E, P, st, zr, sym, small, always, stream))) {
        return rc;
    }
    if ((rc = run_find_giant(n, m, E, P, bits, st, zr, 0, stream))) return rc;
    if (link_first) {
        if ((rc = run_warm(n, m, E, P, st, zr, sym, small, again, stream))) return rc;
        if ((rc = run_find_giant(n, m, E, P, bits, st, zr, 1, stream))) return rc;
    }
    if ((rc = run_warm(n, m, E, P, st, zr, sym, full, again, stream))) return rc;
    if ((rc = run_find_giant(n, m, E, P, bits, st, zr, 2, stream))) return rc;
    // Without a giant component, the sizes that were always regrouped hook their
    // regrouped entries, over the flat forest that the samples leave.
    const bool regroup = !E.csr && tiled_eligible(n, m, zr);
    const Gate write = link_first ? Gate{&st->rebuild, 1u} : on;
    if ((rc = compress(!regroup && !E.csr ? write : link_first ? Gate{&st->flat, 1u} : always))) return rc;
    if ((rc = run_giant_bits(n, m, E, P, bits, st, zr ? kBitsZr : kBitsPlain, 0, write, stream))) return rc;
    if ((rc = run_filter(s, n, m, E, P, bits, passes, own_bits, p32, sym, on,
                         !regroup ? kNoOther : zr ? kOtherZr : kOther, stream)))
        return rc;
    if (regroup) return CC_OK;
    if (E.csr) return hook_rows();
    const Gate off{&st->giant, 0u};
    // Longer lists on a resident grid (ER n = 200 M, 400 M entries: 31.6 ms, one
    // workgroup per tile 32.1; grid n = 33 M: 5.7 and 6.0), shorter ones without the
    // loop (ER n = 2 M, 4.2 M entries: 1.79 ms resident, 1.49 so).
    const uint64_t dt = (m + kBlock * kEPT - 1) / (kBlock * kEPT);
    const uint32_t g = (uint32_t)std::min<uint64_t>(dt, dt <= 16384 ? dt : kZrGrid);
    const uint32_t n32 = (uint32_t)n, sy = sym ? 1u : 0u;
    const uint32_t skip = (uint32_t)std::min<uint64_t>(warm_stride(m, full), 0xFFFFFFFFull);
    if (!zr)
        with_coo(E, [&](auto e) {
            k_hook_gated<false, 1, false><<<g, kBlock, 0, stream>>>(e, m, n32, P, bits, st, sy, skip, off);
        });
    else if (hook_links_z(flags, n))
        with_coo(E, [&](auto e) {
            k_hook_gated<true, 1, true><<<g, kBlock, 0, stream>>>(e, m, n32, P, bits, st, sy, skip, off);
        });
    else
        with_coo(E, [&](auto e) {
            k_hook_gated<true, 1, false><<<g, kBlock, 0, stream>>>(e, m, n32, P, bits, st, sy, skip, off);
        });
    CCM_HIP(hipGetLastError());
    return CC_OK;
}

int run_hook(Slot* s, uint64_t n, uint64_t m, const uint32_t* edges, uint32_t* P,
             uint32_t flags, hipStream_t stream) {
    if (!m) return CC_OK;
    const uint64_t per = (uint64_t)kBlock * kEPT;
    const uint64_t blocks = (m + per - 1) / per;
    if (blocks > 0x7FFFFFFFull) return fail(CC_EINVAL, "edge count too large for one launch");
    const bool zr = flags & CC_F_ZROOT;
    const uint32_t sym = (flags & CC_F_SYMMETRIC) ? 1u : 0u;
    if (zr && (!s->zr_ready || s->cur_n != n))
        return fail(CC_EINVAL, "a CC_F_ZROOT hook needs cc_init then cc_zroot on the same n");
    const bool regroup = !(flags & (CC_F_NO_SPLIT | CC_F_NO_TILE)) && !s->no_tiled;
    if (!zr && regroup && tiled_eligible(n, m, false)) {
        const int rc = run_hook_buckets(s, n, m, edges, P, sym != 0, stream);
        if (rc != kScratchCapture) return rc;
    }
    const bool split = split_walks(flags, n);
    const uint32_t n32 = (uint32_t)n;
    uint32_t* zb = s->zbits;
    const uint32_t g = (uint32_t)blocks;
    const bool linkz = hook_links_z(flags, n);
    const bool lds = !(flags & CC_F_NO_SPLIT) && lds_eligible(n, m);
    int passes = regroup ? filter_passes(n, m, zr) : 0;
    if (zr && (lds || passes)) {
        const EdgeList E{edges, false};
        FilterScratch fs{};
        int rc = passes ? filter_scratch(s, n, m, passes, false, false, stream, &fs) : CC_OK;
        if (!rc) return hook_by_bits(s, n, m, E, P, zb, passes, true, false, false, flags, stream);
        if (rc == CC_ENOMEM && tiled_eligible(n, m, true)) return fail(rc, fs.why);
        if (rc < 0 && rc != CC_ENOMEM) return rc;
    }
    if (!zr && !(flags & CC_F_NO_SPLIT) && hook_in_two_parts(n, m, split)) {
        // in two parts (ER n = 2^16 with 2^20 entries, whole solve: 0.150 -> 0.115 ms)
        const uint64_t m1 = m / 4;
        const uint32_t g1 = (uint32_t)((m1 + per - 1) / per);
        const uint32_t g2 = (uint32_t)((m - m1 + per - 1) / per);
        k_hook<false, 0><<<g1, kBlock, 0, stream>>>(edges, m1, n32, P, zb, s->st, sym);
        CCM_HIP(hipGetLastError());
        int rc = cohere(stream);
        if (rc) return rc;
        k_compress<false><<<grid_for(n, kBlock, kGridCap), kBlock, 0, stream>>>(P, n, s->st, nullptr,
                                                                             nullptr);
        CCM_HIP(hipGetLastError());
        if ((rc = cohere(stream))) return rc;
        k_hook<false, 0><<<g2, kBlock, 0, stream>>>(edges + 2 * m1, m - m1, n32, P, zb, s->st, sym);
        CCM_HIP(hipGetLastError());
        return CC_OK;
    }
    if (zr && linkz && split)
        k_hook<true, 1, false, true><<<g, kBlock, 0, stream>>>(edges, m, n32, P, zb, s->st, sym);
    else if (zr && linkz)
        k_hook<true, 0, false, true><<<g, kBlock, 0, stream>>>(edges, m, n32, P, zb, s->st, sym);
    else if (zr && split) k_hook<true, 1><<<g, kBlock, 0, stream>>>(edges, m, n32, P, zb, s->st, sym);
    else if (zr) k_hook<true, 0><<<g, kBlock, 0, stream>>>(edges, m, n32, P, zb, s->st, sym);
    else if (split) k_hook<false, 1><<<g, kBlock, 0, stream>>>(edges, m, n32, P, zb, s->st, sym);
    else k_hook<false, 0><<<g, kBlock, 0, stream>>>(edges, m, n32, P, zb, s->st, sym);
    CCM_HIP(hipGetLastError());
    return CC_OK;
}

int run_hook_log(Slot* s, uint64_t n, uint64_t m, const uint32_t* edges, uint32_t* P,
                 uint32_t flags, uint32_t* log, uint64_t log_cap, uint64_t* log_count,
                 hipStream_t stream) {
    if (flags & CC_F_ZROOT)
        return fail(CC_EINVAL, "the update log is defined for the plain path (no CC_F_ZROOT)");
    if (!m) return CC_OK;
    const uint64_t per = (uint64_t)kBlock * kEPT;
    const uint64_t blocks = (m + per - 1) / per;
    if (blocks > 0x7FFFFFFFull) return fail(CC_EINVAL, "edge count too large for one launch");
    const uint32_t g = (uint32_t)blocks;
    auto* cnt = reinterpret_cast<unsigned long long*>(log_count);
    const uint32_t sym = (flags & CC_F_SYMMETRIC) ? 1u : 0u;
    if (!split_walks(flags, n))
        k_hook<false, 0, true><<<g, kBlock, 0, stream>>>(edges, m, (uint32_t)n, P, nullptr, s->st,
                                                         sym, log, log_cap, cnt);
    else
        k_hook<false, 1, true><<<g, kBlock, 0, stream>>>(edges, m, (uint32_t)n, P, nullptr, s->st,
                                                         sym, log, log_cap, cnt);
    CCM_HIP(hipGetLastError());
    return CC_OK;
}

__global__ void k_log_count_reset(DevState* st) {
    if (threadIdx.x == 0 && blockIdx.x == 0) st_agent64(&st->log_count, 0ull);
}

__global__ void k_log_count_snap(DevState* st, uint64_t* host_word) {
    if (threadIdx.x == 0 && blockIdx.x == 0)
        __hip_atomic_store(host_word, ld_agent64(&st->log_count), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_SYSTEM);
}

int log_count_reset(Slot* s, hipStream_t stream) {
    k_log_count_reset<<<1, 64, 0, stream>>>(s->st);
    CCM_HIP(hipGetLastError());
    return CC_OK;
}

int log_count_snap(Slot* s, uint64_t* host_word, hipStream_t stream) {
    k_log_count_snap<<<1, 64, 0, stream>>>(s->st, host_word);
    CCM_HIP(hipGetLastError());
    return CC_OK;
}

// Compress and resolve against the bitmap of st->zroot's component. pub: it is the
// caller's zero root (cc_canon reads what is recorded).
static int zr_labels(Slot* s, uint64_t n, uint32_t* P, uint32_t* bits, bool final_labels, int pub,
                     Gate gate, hipStream_t stream) {
    const uint32_t g = grid_for(n, kBlock, kZrGrid);
    k_compress<true><<<g, kBlock, 0, stream>>>(P, n, s->st, bits, s->bmin, gate);
    CCM_HIP(hipGetLastError());
    if (final_labels)
        k_resolve<true><<<g, kBlock, 0, stream>>>(P, n, s->st, bits, s->bmin, g, pub, gate);
    else
        k_resolve<false><<<g, kBlock, 0, stream>>>(P, n, s->st, bits, s->bmin, g, pub, gate);
    CCM_HIP(hipGetLastError());
    return CC_OK;
}

int run_compress(Slot* s, uint64_t n, uint32_t* P, uint32_t flags, hipStream_t stream,
                 bool final_labels) {
    if (flags & CC_F_ZROOT) {
        if (!s->zr_ready || s->cur_n != n)
            return fail(CC_EINVAL, "a CC_F_ZROOT compress needs cc_init then cc_zroot on the same n");
        return zr_labels(s, n, P, s->zbits, final_labels || (flags & CC_F_CANON), 1, Gate{}, stream);
    }
    k_compress<false><<<grid_for(n, kBlock, kGridCap), kBlock, 0, stream>>>(P, n, s->st, nullptr, nullptr);
    CCM_HIP(hipGetLastError());
    return CC_OK;
}

// Every ids[i] is connected to target (the Reducer's zero-converged messages).
// With a zero root equal to target the link is the bitmap mark itself.
template <bool ZR, int SPLIT>
__global__ __launch_bounds__(kBlock) void k_hook_ids(const uint32_t* __restrict__ ids,
                                                     uint64_t count, uint32_t target, uint32_t n,
                                                     uint32_t* P, uint32_t* zbits, DevState* st) {
    const uint32_t z = ZR ? ld_agent(&st->zroot) : 0u;
    const bool mark = ZR && target == z;
    bool bad = false;
    for (uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x; i < count;
         i += (uint64_t)gridDim.x * kBlock) {
        const uint32_t x = ids[i];
        if (x >= n) { bad = true; continue; }
        if (x == target) continue;
        if (mark) {
            zbit_set(zbits, x);
            continue;
        }
        const uint32_t px = P[x], pt = P[target];
        if (px == pt || px == target || pt == x) continue;
        (void)link<ZR, SPLIT>(P, x, px, target, pt, z);
    }
    if (bad) atomicOr(&st->status, kStatusRange);
}

int run_hook_ids(Slot* s, uint64_t n, uint64_t count, const uint32_t* ids, uint32_t target,
                 uint32_t* P, uint32_t flags, hipStream_t stream) {
    const bool zr = flags & CC_F_ZROOT;
    const bool split = split_walks(flags, n);
    if (zr && (!s->zr_ready || s->cur_n != n))
        return fail(CC_EINVAL, "a CC_F_ZROOT id hook needs cc_init then cc_zroot on the same n");
    const uint32_t g = grid_for(count, kBlock, kGridCap);
    const uint32_t n32 = (uint32_t)n;
    if (zr && split) k_hook_ids<true, 1><<<g, kBlock, 0, stream>>>(ids, count, target, n32, P, s->zbits, s->st);
    else if (zr) k_hook_ids<true, 0><<<g, kBlock, 0, stream>>>(ids, count, target, n32, P, s->zbits, s->st);
    else if (split) k_hook_ids<false, 1><<<g, kBlock, 0, stream>>>(ids, count, target, n32, P, s->zbits, s->st);
    else k_hook_ids<false, 0><<<g, kBlock, 0, stream>>>(ids, count, target, n32, P, s->zbits, s->st);
    CCM_HIP(hipGetLastError());
    return CC_OK;
}

int run_canon(Slot* s, uint64_t n, uint32_t* L, hipStream_t stream) {
    k_canon<<<grid_for(n, kBlock, kGridCap), kBlock, 0, stream>>>(L, n, s->st);
    CCM_HIP(hipGetLastError());
    return CC_OK;
}

int run_csr_head(Slot* s, uint64_t n, const uint64_t* off, uint32_t flags, hipStream_t stream, uint64_t* m,
                 uint32_t* maxdeg) {
    const bool zmax = (flags & CC_F_ZROOT) && !(flags & CC_F_ZROOT_HINT);
    if (zmax) k_zsel_reset<<<1, 64, 0, stream>>>(s->st);
    int rc = cohere(stream);
    if (rc) return rc;
    if (zmax) k_csr_zmax<<<grid_for(n, 4 * kBlock, 2048), kBlock, 0, stream>>>(off, n, s->st);
    uint64_t* host = reinterpret_cast<uint64_t*>(s->host_status);
    k_csr_head<<<1, 64, 0, stream>>>(off + n, s->st, zmax, host);
    CCM_HIP(hipGetLastError());
    CCM_HIP(hipStreamSynchronize(stream));
    *m = __atomic_load_n(host, __ATOMIC_ACQUIRE);
    *maxdeg = (uint32_t)(__atomic_load_n(host + 1, __ATOMIC_RELAXED) >> 32);
    host[0] = host[1] = 0;
    return CC_OK;
}

int run_solve_csr(Slot* s, uint64_t n, uint64_t m, const uint64_t* off, const uint32_t* adj,
                  uint32_t* L, uint32_t flags, uint32_t hint, uint32_t maxdeg, hipStream_t stream) {
    if (n == 0) return CC_OK;
    int rc;
    const bool zr = flags & CC_F_ZROOT;
    const bool split = split_walks(flags, n);
    const uint32_t sym = (flags & CC_F_SYMMETRIC) ? 1u : 0u;
    const uint64_t ntiles = (m + kCsrTile - 1) / kCsrTile;
    if (ntiles > 0x7FFFFFFFull) return fail(CC_EINVAL, "entry count too large for one launch");
    if (s->csr_tiles_cap < ntiles + 1) {
        CCM_HIP(hipStreamSynchronize(stream));
        if (s->csr_tiles) CCM_HIP(hipFree(s->csr_tiles));
        s->csr_tiles = nullptr;
        s->csr_tiles_cap = 0;
        if (hipMalloc(&s->csr_tiles, (ntiles + 1) * sizeof(uint32_t)) != hipSuccess) {
            (void)hipGetLastError();
            s->csr_tiles = nullptr;
            return fail(CC_ENOMEM, "CSR tile table allocation failed");
        }
        s->csr_tiles_cap = ntiles + 1;
    }
    if ((rc = run_init(s, n, L, stream))) return rc;
    const uint32_t gn = grid_for(n, kBlock, kGridCap);
    k_csr_tiles<<<gn, kBlock, 0, stream>>>(off, n, m, s->csr_tiles, ntiles, s->st);
    CCM_HIP(hipGetLastError());
    if (zr) {
        k_zfinish<<<1, 64, 0, stream>>>(s->st, flags & CC_F_ZROOT_HINT ? 1 : 0, hint);
        CCM_HIP(hipGetLastError());
        if ((rc = zbits_reset(s, n, stream))) return rc;
        k_csr_push<<<64, kBlock, 0, stream>>>(off, adj, n, m, L, s->zbits, s->st);
        CCM_HIP(hipGetLastError());
    }
    if ((rc = cohere(stream))) return rc;
    const bool skewed = maxdeg >= 64 * (m / n + 1);      // the longest row against the mean
    if (zr && !(flags & CC_F_NO_SPLIT)) {
        // The whole-bitmap and one-pass tile filters read the rows as entries (ms:
        // extras n = 1.7 M, 10.4 M entries 0.58 direct, 0.40 so; ER n = 400,000, 1.5 M
        // entries 0.40 and 0.24; grid n = 3 M, 4 M entries 0.51 and 0.56, hence three
        // entries per two vertices at least). The regrouped hook of two passes has
        // its own CSR form below, and keeps the skewed graphs of 12 ranges and more (one
        // pass, two, us: R-MAT n = 2^23, 17 M entries 887 and 474, 69 M 1406 and 818; n =
        // 2^22, 35 M 825 and 918; ER n = 10 M, 50 M 2166 and 2324; 16 parts n = 8 M,
        // 60 M 2937 and 16004). The plain direct hook, whose lanes share their first
        // endpoint's reads, is hard to beat here: ER n = 12 M, 60 M entries 1.98 ms
        // direct, 2.54 filtered.
        const CsrList rows{off, adj, s->csr_tiles, ntiles, (uint32_t)n};
        const EdgeList E{nullptr, false, &rows};
        const bool lds = lds_eligible(n, m);
        const bool two = skewed && n > (11ull << 19) && tiled_eligible(n, m, true);
        const int passes =
            (flags & CC_F_NO_TILE) || s->no_tiled || 2 * m < 3 * n || two ? 0 : filter_passes(n, m, true);
        FilterScratch fs{};
        if (lds || (passes == 1 && !filter_scratch(s, n, m, passes, false, false, stream, &fs))) {
            if ((rc = hook_by_bits(s, n, m, E, L, s->zbits, passes, true, false, false, flags, stream)))
                return rc;
            if ((rc = run_compress(s, n, L, flags, stream, true))) return rc;
            return cohere(stream);
        }
    }
    if (zr && !(flags & (CC_F_NO_SPLIT | CC_F_NO_TILE)) && tiled_eligible(n, m, true)) {
        // as on COO input: a warm-up over the first 1/1024 of the tiles seeds the
        // bitmap, then the regrouped hook covers every position (the warm-up's
        // entries again too, which finds them joined)
        const uint64_t w = ntiles >> 10;
        if (w) {
            k_csr_hook<true, 1, true><<<(uint32_t)w, kBlock, 0, stream>>>(
                off, adj, (uint32_t)n, m, s->csr_tiles, ntiles, L, s->zbits, s->st, sym);
            CCM_HIP(hipGetLastError());
        }
        // A skewed graph's giant component is in the bitmap by the time the survivors are
        // hooked: their bits are worth a second look (ER n = 16 M, 60 M entries: 4.0 ms
        // with it, 3.0 without; R-MAT-24, 2^28 entries: 2.2 without the look, 1.8 with it).
        if ((rc = run_hook_tiled_csr(s, n, m, off, adj, L, skewed, stream, sym != 0))) return rc;
    } else if (ntiles) {
        const uint32_t g = (uint32_t)ntiles;
        const uint32_t n32 = (uint32_t)n;
        uint32_t* zb = s->zbits;
        const uint32_t* ts = s->csr_tiles;
        const bool linkz = hook_links_z(flags, n);
        if (zr && linkz && split)
            k_csr_hook<true, 1, true><<<g, kBlock, 0, stream>>>(off, adj, n32, m, ts, ntiles, L, zb, s->st, sym);
        else if (zr && linkz)
            k_csr_hook<true, 0, true><<<g, kBlock, 0, stream>>>(off, adj, n32, m, ts, ntiles, L, zb, s->st, sym);
        else if (zr && split) k_csr_hook<true, 1><<<g, kBlock, 0, stream>>>(off, adj, n32, m, s->csr_tiles, ntiles, L, zb, s->st, sym);
        else if (zr) k_csr_hook<true, 0><<<g, kBlock, 0, stream>>>(off, adj, n32, m, s->csr_tiles, ntiles, L, zb, s->st, sym);
        else if (split) k_csr_hook<false, 1><<<g, kBlock, 0, stream>>>(off, adj, n32, m, s->csr_tiles, ntiles, L, zb, s->st, sym);
        else k_csr_hook<false, 0><<<g, kBlock, 0, stream>>>(off, adj, n32, m, s->csr_tiles, ntiles, L, zb, s->st, sym);
        CCM_HIP(hipGetLastError());
    }
    if ((rc = run_compress(s, n, L, flags, stream, true))) return rc;
    return cohere(stream);
}

static uint64_t al256(uint64_t x) { return (x + 255) & ~255ull; }

uint64_t solve_scratch_bytes(uint64_t n, uint64_t m, uint32_t flags, bool lean) {
    const bool zr = flags & CC_F_ZROOT;
    uint64_t b = 0;
    if (zr) b += al256(4 * ((n + 31) / 32));
    if (zr && (flags & CC_F_ZROOT_EXACT)) b += al256(4 * n);
    if (m && !(flags & (CC_F_NO_SPLIT | CC_F_NO_TILE))) {
        const int passes = filter_passes(n, m, zr);
        if (passes && (!lean || (zr && tiled_eligible(n, m, true))))
            b += filter_scratch_bytes(n, m, passes, !zr, false);
        else if (!zr && tiled_eligible(n, m, false))
            b += bucket_scratch_bytes(n, m);
    }
    return b;
}

void slot_lend_scratch(Slot* s, char* block, uint64_t bytes, uint64_t n, uint32_t flags,
                       LentScratch* saved) {
    saved->zbits = s->zbits;
    saved->zbits_cap = s->zbits_cap;
    saved->deg = s->deg;
    saved->deg_cap = s->deg_cap;
    saved->tiled = s->tiled;
    const bool zr = flags & CC_F_ZROOT;
    char* q = block;
    s->zbits = nullptr;
    s->zbits_cap = 0;
    s->deg = nullptr;
    s->deg_cap = 0;
    s->tiled = TiledScratch{};
    if (zr) {
        const uint64_t words = (n + 31) / 32;
        s->zbits = reinterpret_cast<uint32_t*>(q);
        s->zbits_cap = words;
        q += al256(4 * words);
    }
    if (zr && (flags & CC_F_ZROOT_EXACT)) {
        s->deg = reinterpret_cast<uint32_t*>(q);
        s->deg_cap = n;
        q += al256(4 * n);
    }
    s->tiled.buf = q;
    s->tiled.cap = bytes - (uint64_t)(q - block);
    s->no_grow = true;
}

void slot_return_scratch(Slot* s, const LentScratch* saved) {
    s->zbits = saved->zbits;
    s->zbits_cap = saved->zbits_cap;
    s->deg = saved->deg;
    s->deg_cap = saved->deg_cap;
    s->tiled = saved->tiled;
    s->no_grow = false;
    s->zr_ready = false;
}

// A plain whole solve after init by the giant component.
int run_giant(Slot* s, uint64_t n, uint64_t m, EdgeList E, uint32_t* P, uint32_t* bits, int passes,
              bool p32, uint32_t flags, hipStream_t stream) {
    int rc = hook_by_bits(s, n, m, E, P, bits, passes, false, true, p32, flags, stream);
    if (rc) return rc;
    const Gate on{passes ? &s->st->giant : nullptr, 1u};
    if ((rc = zr_labels(s, n, P, bits, true, 0, on, stream))) return rc;
    if (passes) {
        // hooked direct: no root plays the zero root's part, the bitmap is unset
        k_compress<false><<<grid_for(n, kBlock, kGridCap), kBlock, 0, stream>>>(
            P, n, s->st, nullptr, nullptr, Gate{&s->st->giant, 0u});
        CCM_HIP(hipGetLastError());
    }
    return CC_OK;
}

int run_solve(Slot* s, uint64_t n, uint64_t m, const uint32_t* edges, uint32_t* L,
              uint32_t flags, uint32_t hint, hipStream_t stream) {
    if (n == 0) return CC_OK;
    int rc;
    if (!(flags & CC_F_NO_SPLIT) && small_eligible(n, m, flags, s->samples)) {
        s->cur_n = n;
        s->zr_ready = flags & CC_F_ZROOT;
        if (s->zr_ready && (rc = zbits_grow(s, n, stream))) return rc;
        if ((rc = cohere(stream))) return rc;        // before the entries are read
        if ((rc = run_solve_small(s, n, m, edges, L, flags, hint, stream))) return rc;
        return cohere(stream);
    }
    if ((rc = run_init(s, n, L, stream))) return rc;
    // One coherence point before anything reads the entries (the zero root's sample
    // and push read them too) or P. What those two steps write of P and the bitmap
    // goes to memory, and a hook may read either as it was before them: an older
    // parent is an ancestor, a clear bit only sends an entry to P.
    if ((rc = cohere(stream))) return rc;
    if (flags & CC_F_ZROOT) {
        if ((rc = run_zroot(s, n, m, edges, flags, hint, stream))) return rc;
        if ((rc = run_push(s, n, m, edges, L, stream))) return rc;
    }
    if (!(flags & (CC_F_ZROOT | CC_F_NO_SPLIT))) {
        const EdgeList E{edges, false};
        FilterScratch fs;
        const int passes = (flags & CC_F_NO_TILE) || s->no_tiled ? 0 : filter_passes(n, m, false);
        uint32_t* bits = nullptr;
        if (lds_eligible(n, m)) bits = s->gbits;
        else if (passes && !filter_scratch(s, n, m, passes, true, false, stream, &fs)) bits = fs.bits;
        if (bits) {
            if ((rc = run_giant(s, n, m, E, L, bits, passes, false, flags, stream))) return rc;
            return cohere(stream);
        }
    }
    if ((rc = run_hook(s, n, m, edges, L, flags, stream))) return rc;
    if ((rc = run_compress(s, n, L, flags, stream, true))) return rc;
    return cohere(stream);
}

}  // namespace ccm

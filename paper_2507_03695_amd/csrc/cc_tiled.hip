// cc_tiled.hip — the regrouped hooks: the filter with both membership tests in LDS,
// against the bitmap of the zero root's component or, on a plain whole solve, of the
// giant component's; and hooks of the regrouped entries without a bitmap.
//
// The plain bitmap hook pays two random L2/MALL line reads per entry (the
// bitmap is n/8 bytes, 8.5 MB at RMAT-26, twice one XCD's L2). Here the
// entries are first regrouped so that each workgroup sees only entries whose
// endpoints fall in two fixed vertex ranges ("slices" of 2^kSliceBits
// vertices), and it holds the bitmap words of both slices in LDS. Up to 22 slices
// one pass makes the (a, b) tiles (k_tile_part, below); beyond:
//
//  1. k_t1_part   — every chunk of kC1 entries is sorted in LDS by the slice
//                   of its first endpoint (a) and written back in place order;
//                   per chunk, the start of each a-segment; per a, the counts.
//  2. k_t1_scan   — per a, exclusive prefix of the segment counts over chunks
//                   (each a-bucket becomes one virtual array).
//  3. k_t1_bases  — where each a-bucket starts in the second buffer and how
//                   many level-2 chunks it has.
//  4. k_t2_part   — every kC2-entry piece of an a-bucket is gathered from its
//                   segments, sorted in LDS by the slice of the second
//                   endpoint (b) and written contiguously, with its b-runs.
//  5. k_t3_filter — one workgroup per (a, few b): both slices' bitmap words in
//                   LDS; an entry with both endpoints marked is dropped, one
//                   with a single marked endpoint marks the other (LDS and
//                   global) and is dropped, the rest go to a survivor list.
//  6. k_t4_hook   — the ordinary hook over the survivor list.
// Without a giant component: k_t2_hookplain hooks the buckets of 1-3, k_tile_hook the
// one-pass tiles.
//
// After this step the components are given by P and the bitmap together
// (k_compress / k_resolve in cc_kernels.hip read both).
//
// The regrouping only reorders entries (and drops self-loops, which are
// no-ops), hooking is order-independent (Sec. II), and every dropped entry is
// either redundant or recorded as a mark, so the labels are those of the plain
// pass. Entries whose endpoints are out of range are dropped with
// the status bit set, as in the plain hook.
#include <algorithm>

#include "cc_internal.h"
#include "cc_link.h"

namespace ccm {

constexpr int kSliceBits = 19;                       // 2^19 vertices per slice
constexpr uint32_t kSliceWords = (1u << kSliceBits) / 32;   // 16384 words = 64 KB
constexpr uint32_t kLoMask = (1u << kSliceBits) - 1;

// Packed entries. With at most 512 slices every ID is below 2^28, and inside a
// bucket the slice bits of an endpoint are known, so the buffers between the
// passes hold fewer than 8 bytes per entry:
//  level 1 (bucket a known): w = u_lo | v << 19, h = v >> 13 (4 + 2 bytes)
// (u_lo: the low 19 bits of u; the top 13 bits of w carry the low 13 bits of v).
// The survivor regions reuse this format.
//  level 2 (both slices known from the run): w = u_lo | v_lo << 19,
//  h = v_lo >> 13 (4 + 1 bytes), two arrays.
__device__ __forceinline__ uint32_t pk_w(uint32_t ulo, uint32_t v) { return ulo | (v << kSliceBits); }
__device__ __forceinline__ uint32_t pk_v1(uint32_t w, uint16_t h) {
    return (w >> kSliceBits) | ((uint32_t)h << (32 - kSliceBits));
}

// The level-2 buffer: the two arrays of the 5-byte relative form.
struct L2Buf {
    uint32_t* w;
    uint8_t* h;
};

constexpr int kMaxSlices = 512;
constexpr int kMaxSlicesOther = 256;                 // the plain bucketed hook, CSR input
constexpr int kC1 = 8192;                            // level-1 chunk (entries)
constexpr int kC2 = 8192;                            // level-2 chunk (entries)
constexpr int kPartBlock = 1024;
constexpr int kPartEPT = kC1 / kPartBlock;           // 8

// Exclusive scan of cnt[0..R) into start[0..R] by the first wave (R <= 64 * PER);
// start[R] is the total.
template <int PER>
__device__ __forceinline__ void wave_scan(const uint32_t* cnt, uint32_t* start, int R) {
    const int lane = threadIdx.x & 63;
    if (threadIdx.x < 64) {
        uint32_t c[PER], s = 0;
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const int d = lane * PER + j;
            c[j] = d < R ? cnt[d] : 0u;
            s += c[j];
        }
        uint32_t incl = s;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t y = __shfl_up(incl, off, 64);
            if (lane >= off) incl += y;
        }
        uint32_t run = incl - s;
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const int d = lane * PER + j;
            if (d < R) start[d] = run;
            run += c[j];
        }
        if (lane == 63) start[R] = incl;
    }
}

// ---- 1. level-1 partition by the first endpoint's slice -----------------------------
template <int MAXS, typename T>
__global__ __launch_bounds__(kPartBlock) void k_t1_part(const T edges,
                                                        uint64_t m, uint32_t n, int R,
                                                        uint64_t nch1, uint32_t* __restrict__ t1w,
                                                        uint16_t* __restrict__ t1h,
                                                        uint16_t* __restrict__ segT,
                                                        uint32_t* __restrict__ cnt1,
                                                        DevState* st, uint32_t sym, Gate gate) {
    if (gated_off(gate)) return;
    __shared__ u32x2 stage[kC1];
    __shared__ uint32_t hist[MAXS + 1];
    __shared__ uint32_t start[MAXS + 1];
    const uint64_t c = blockIdx.x;
    for (int i = threadIdx.x; i <= MAXS; i += kPartBlock) hist[i] = 0;
    __syncthreads();
    u32x2 e[kPartEPT];
    uint16_t rank[kPartEPT];
    bool bad = false;
#pragma unroll
    for (int k = 0; k < kPartEPT; ++k) {
        // unconditional load (clamped index): keeps all loads of the thread in flight
        const uint64_t i = c * kC1 + (uint64_t)k * kPartBlock + threadIdx.x;
        e[k] = load_entry(edges, i < m ? i : m - 1);
    }
#pragma unroll
    for (int k = 0; k < kPartEPT; ++k) {
        const uint64_t i = c * kC1 + (uint64_t)k * kPartBlock + threadIdx.x;
        if (i >= m) e[k].x = e[k].y = 0u;
        else if (e[k].x >= n || e[k].y >= n) { bad = true; e[k].x = e[k].y = 0u; }
    }
    if (bad) atomicOr(&st->status, kStatusRange);
#pragma unroll
    for (int k = 0; k < kPartEPT; ++k) {
        rank[k] = 0xFFFF;
        // self-loops are dropped; with sym (every pair listed in both orders) so
        // are the entries with u > v
        const bool live = sym ? e[k].x < e[k].y : e[k].x != e[k].y;
        if (live) rank[k] = (uint16_t)atomicAdd(&hist[e[k].x >> kSliceBits], 1u);
    }
    __syncthreads();
    wave_scan<MAXS / 64>(hist, start, R);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kPartEPT; ++k)
        if (rank[k] != 0xFFFF) stage[start[e[k].x >> kSliceBits] + rank[k]] = e[k];
    __syncthreads();
    const uint32_t kept = start[R];
    for (uint32_t i = threadIdx.x; i < kept; i += kPartBlock) {
        const u32x2 x = stage[i];
        t1w[c * kC1 + i] = pk_w(x.x & kLoMask, x.y);
        t1h[c * kC1 + i] = (uint16_t)(x.y >> (32 - kSliceBits));
    }
    for (int d = threadIdx.x; d < R; d += kPartBlock) {
        segT[(uint64_t)d * nch1 + c] = (uint16_t)start[d];
        cnt1[(uint64_t)d * nch1 + c] = hist[d];
    }
}

// ---- 2. per slice a: exclusive prefix of segment counts over chunks ------------------
// pre1 has nch1 + 1 entries per row (the last is the total). Two launches over
// (a, tile of kScanTile chunks): tile sums, then the scan of each tile offset by
// the sum of the tiles before it.
constexpr int kScanTile = 1024;
constexpr int kScanBlock = 256;

__global__ __launch_bounds__(kScanBlock) void k_t1_tsum(const uint32_t* __restrict__ cnt1,
                                                        uint64_t nch1, uint32_t ntile,
                                                        uint32_t* __restrict__ tsum, Gate gate) {
    if (gated_off(gate)) return;
    __shared__ uint32_t ws[kScanBlock / 64];
    const uint64_t a = blockIdx.x / ntile, tile = blockIdx.x % ntile;
    const uint32_t* row = cnt1 + a * nch1;
    uint32_t s = 0;
    for (int k = 0; k < kScanTile / kScanBlock; ++k) {
        const uint64_t c = tile * kScanTile + (uint64_t)k * kScanBlock + threadIdx.x;
        if (c < nch1) s += row[c];
    }
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
    if ((threadIdx.x & 63) == 0) ws[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t t = 0;
        for (int w = 0; w < kScanBlock / 64; ++w) t += ws[w];
        tsum[blockIdx.x] = t;
    }
}

__global__ __launch_bounds__(kScanBlock) void k_t1_scan(const uint32_t* __restrict__ cnt1,
                                                        uint64_t nch1, uint32_t ntile,
                                                        const uint32_t* __restrict__ tsum,
                                                        uint32_t* __restrict__ pre1, Gate gate) {
    if (gated_off(gate)) return;
    __shared__ uint32_t ws[kScanBlock / 64];
    __shared__ uint32_t s_off;
    const uint64_t a = blockIdx.x / ntile, tile = blockIdx.x % ntile;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (wave == 0) {
        // sum of the tiles before this one (ntile may exceed 64: strided lanes)
        uint32_t s = 0;
        for (uint64_t i = lane; i < tile; i += 64) s += tsum[a * ntile + i];
        for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
        if (lane == 0) s_off = s;
    }
    const uint32_t* row = cnt1 + a * nch1;
    uint32_t* out = pre1 + a * (nch1 + 1);
    // each thread scans 4 consecutive chunks of the tile
    constexpr int PER = kScanTile / kScanBlock;
    const uint64_t c0 = tile * kScanTile + (uint64_t)threadIdx.x * PER;
    uint32_t v[PER], s = 0;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        v[k] = c0 + k < nch1 ? row[c0 + k] : 0u;
        s += v[k];
    }
    uint32_t incl = s;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t y = __shfl_up(incl, off, 64);
        if (lane >= off) incl += y;
    }
    if (lane == 63) ws[wave] = incl;
    __syncthreads();
    uint32_t run = s_off + incl - s;
    for (int w = 0; w < wave; ++w) run += ws[w];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        if (c0 + k < nch1) out[c0 + k] = run;
        run += v[k];
    }
    // the thread holding the last chunk writes the row total
    if (c0 < nch1 && nch1 <= c0 + PER) out[nch1] = run;
}

// ---- 3. bucket bases and level-2 chunk counts ---------------------------------------------
// base2[a]: first entry of bucket a in the second buffer; cbase[a]: first level-2
// chunk of bucket a; cbase[R] is the total.
__global__ __launch_bounds__(kMaxSlices) void k_t1_bases(const uint32_t* __restrict__ pre1, uint64_t nch1,
                                                  int R, uint64_t* __restrict__ base2,
                                                  uint32_t* __restrict__ cbase, Gate gate) {
    if (gated_off(gate)) return;
    // one thread per slice (R <= kMaxSlices): sizes, then block-wide exclusive prefixes
    __shared__ uint64_t s_b[kMaxSlices];
    __shared__ uint32_t s_c[kMaxSlices];
    const int a = threadIdx.x;
    const uint32_t size = a < R ? pre1[(uint64_t)a * (nch1 + 1) + nch1] : 0u;
    s_b[a] = size;
    s_c[a] = (size + kC2 - 1) / kC2;
    __syncthreads();
    for (int off = 1; off < kMaxSlices; off <<= 1) {          // inclusive Hillis-Steele scan
        const uint64_t xb = a >= off ? s_b[a - off] : 0ull;
        const uint32_t xc = a >= off ? s_c[a - off] : 0u;
        __syncthreads();
        s_b[a] += xb;
        s_c[a] += xc;
        __syncthreads();
    }
    if (a < R) {
        base2[a] = s_b[a] - size;
        cbase[a] = s_c[a] - (size + kC2 - 1) / kC2;
    }
    if (a == R - 1) {
        base2[R] = s_b[a];
        cbase[R] = s_c[a];
    }
}

// ---- 4a. level-2 chunk descriptors ----------------------------------------------------------
// Level-2 chunk t of bucket a covers virtual positions [t*kC2, min((t+1)*kC2, size_a)).
// Its descriptor (8 words at desc[8 g], g = cbase[a] + t) holds what k_t2_part
// needs in one read: the first (c0) and last (c1) level-1 chunk it gathers
// from, a | count << 9, t, and the 64-bit output offset base2[a] + t*kC2. One
// thread per (a, c): it writes the fields of the chunks that start or end in
// its segment [pre[c], pre[c+1]).
__global__ __launch_bounds__(256) void k_t2_bounds(const uint32_t* __restrict__ pre1, uint64_t nch1,
                                                   int R, const uint32_t* __restrict__ cbase,
                                                   const uint64_t* __restrict__ base2,
                                                   uint32_t* __restrict__ desc, Gate gate) {
    if (gated_off(gate)) return;
    const uint64_t id = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    if (id >= (uint64_t)R * nch1) return;
    const uint64_t a = id / nch1, c = id % nch1;
    const uint32_t* pre = pre1 + a * (nch1 + 1);
    const uint32_t p0 = pre[c], p1 = pre[c + 1], size = pre[nch1];
    if (p1 <= p0) return;
    for (uint32_t t = p0 / kC2; t <= (p1 - 1) / kC2; ++t) {
        const uint32_t first = t * kC2;
        const uint32_t last = min(first + (uint32_t)kC2, size) - 1;
        uint32_t* d = desc + (uint64_t)(cbase[a] + t) * 8;
        if (first >= p0 && first < p1) {
            const uint64_t o = base2[a] + first;
            d[0] = (uint32_t)c;
            d[2] = (uint32_t)a | ((last + 1 - first) << 9);
            d[3] = t;
            d[4] = (uint32_t)o;
            d[5] = (uint32_t)(o >> 32);
        }
        if (last >= p0 && last < p1) d[1] = (uint32_t)c;
    }
}

// ---- 4b. level-2 partition by the second endpoint's slice ----------------------------------
constexpr int kWin2 = 256;   // level-1 chunks per gather window (owner index fits a byte)

// The chunk's cnt entries (entry i in e[i / kPartBlock] of thread i % kPartBlock,
// hist zeroed beforehand) sorted by the second endpoint's slice through LDS and
// written contiguously to out in the level-2 form, with the start of every
// slice's run in run2T.
template <int MAXS>
__device__ __forceinline__ void t2_sort_write(const u32x2 (&e)[kPartEPT], uint32_t cnt, int R,
                                              uint32_t* hist, uint32_t* start, u32x2* stage,
                                              L2Buf out, uint16_t* __restrict__ run2T,
                                              uint64_t nch2, uint32_t g) {
    uint16_t rank[kPartEPT];
#pragma unroll
    for (int k = 0; k < kPartEPT; ++k) {
        const uint32_t i = (uint32_t)k * kPartBlock + threadIdx.x;
        rank[k] = 0xFFFF;
        if (i < cnt) rank[k] = (uint16_t)atomicAdd(&hist[e[k].y >> kSliceBits], 1u);
    }
    __syncthreads();
    wave_scan<MAXS / 64>(hist, start, R);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kPartEPT; ++k)
        if (rank[k] != 0xFFFF) stage[start[e[k].y >> kSliceBits] + rank[k]] = e[k];
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < cnt; i += kPartBlock) {
        const u32x2 x = stage[i];
        const uint32_t vlo = x.y & kLoMask;
        out.w[i] = (x.x & kLoMask) | (vlo << kSliceBits);
        out.h[i] = (uint8_t)(vlo >> (32 - kSliceBits));
    }
    for (int d = threadIdx.x; d <= R; d += kPartBlock) run2T[(uint64_t)d * nch2 + g] = (uint16_t)start[d];
}

// Gathers level-2 chunk g of slice a from the slice's level-1 segments: entry i
// of the chunk lands in e[i / kPartBlock] of thread i % kPartBlock as (u, v).
// Returns the entry count; a and the output offset come back through a_out and
// obase. Every thread of the block calls it (it uses barriers).
__device__ __forceinline__ uint32_t t2_gather(uint32_t g, const uint32_t* __restrict__ t1w,
                                              const uint16_t* __restrict__ t1h,
                                              const uint16_t* __restrict__ segT,
                                              const uint32_t* __restrict__ pre1, uint64_t nch1,
                                              const uint32_t* __restrict__ desc, uint8_t* owner,
                                              uint32_t* s_pre, uint32_t* s_seg,
                                              u32x2 (&e)[kPartEPT], int& a_out, uint64_t& obase) {
    const uint4 d0 = reinterpret_cast<const uint4*>(desc)[2 * (uint64_t)g];
    const uint4 d1 = reinterpret_cast<const uint4*>(desc)[2 * (uint64_t)g + 1];
    const uint64_t c0 = d0.x, c1 = d0.y;
    const int a = (int)(d0.z & 0x1FFu);
    const uint32_t cnt = d0.z >> 9;
    const uint32_t t = d0.w;
    obase = (uint64_t)d1.x | ((uint64_t)d1.y << 32);
    a_out = a;
    const uint32_t* pre = pre1 + (uint64_t)a * (nch1 + 1);
    const uint32_t vlo = t * (uint32_t)kC2;
    const uint32_t vhi = vlo + cnt;
    for (uint64_t cw = c0; cw <= c1; cw += kWin2) {
        const uint32_t nw = (uint32_t)min<uint64_t>((uint64_t)kWin2, c1 - cw + 1);
        for (uint32_t i = threadIdx.x; i <= nw; i += kPartBlock) s_pre[i] = pre[cw + i];
        for (uint32_t i = threadIdx.x; i < nw; i += kPartBlock)
            s_seg[i] = segT[(uint64_t)a * nch1 + cw + i];
        __syncthreads();
        for (uint32_t i = threadIdx.x; i < nw; i += kPartBlock) {
            const uint32_t lo = max(s_pre[i], vlo), hi = min(s_pre[i + 1], vhi);
            for (uint32_t p = lo; p < hi; ++p) owner[p - vlo] = (uint8_t)i;
        }
        __syncthreads();
        const uint32_t wlo = max(s_pre[0], vlo), whi = min(s_pre[nw], vhi);
        uint32_t xw[kPartEPT];
        uint16_t xh[kPartEPT];
        bool in[kPartEPT];
#pragma unroll
        for (int k = 0; k < kPartEPT; ++k) {
            // unconditional loads (a safe in-bounds address when the position is
            // not in this window) so that all loads of the thread are in flight
            const uint32_t p = vlo + (uint32_t)k * kPartBlock + threadIdx.x;
            in[k] = p >= wlo && p < whi;
            const uint32_t i = in[k] ? owner[p - vlo] : 0u;
            const uint64_t at = in[k] ? (cw + i) * kC1 + s_seg[i] + (p - s_pre[i]) : 0ull;
            xw[k] = t1w[at];
            xh[k] = t1h[at];
        }
#pragma unroll
        for (int k = 0; k < kPartEPT; ++k)
            if (in[k]) {
                e[k].x = ((uint32_t)a << kSliceBits) | (xw[k] & kLoMask);
                e[k].y = pk_v1(xw[k], xh[k]);
            }
        __syncthreads();
    }
    return cnt;
}

// MAXS: the slices its tables hold, 256 or 512 (R-MAT-26, 130 slices: 3.68 ms with
// tables for 512, 3.63 with 256).
template <int MAXS>
__global__ __launch_bounds__(kPartBlock) void k_t2_part(const uint32_t* __restrict__ t1w,
                                                        const uint16_t* __restrict__ t1h,
                                                        const uint16_t* __restrict__ segT,
                                                        const uint32_t* __restrict__ pre1,
                                                        uint64_t nch1, int R,
                                                        const uint32_t* __restrict__ cbase,
                                                        const uint32_t* __restrict__ desc,
                                                        L2Buf tmp2, uint16_t* __restrict__ run2T,
                                                        uint64_t nch2, Gate gate) {
    if (gated_off(gate)) return;
    __shared__ u32x2 stage[kC2];
    __shared__ uint8_t owner[kC2];
    __shared__ uint32_t s_pre[kWin2 + 1];
    __shared__ uint32_t s_seg[kWin2];
    __shared__ uint32_t hist[MAXS + 1];
    __shared__ uint32_t start[MAXS + 1];
    const uint32_t g = blockIdx.x;
    if (g >= cbase[R]) return;                  // the grid is an upper bound
    for (int i = threadIdx.x; i <= MAXS; i += kPartBlock) hist[i] = 0;
    u32x2 e[kPartEPT];
    int a;
    uint64_t obase;
    const uint32_t cnt = t2_gather(g, t1w, t1h, segT, pre1, nch1, desc, owner, s_pre, s_seg, e, a,
                                   obase);
    t2_sort_write<MAXS>(e, cnt, R, hist, start, stage, L2Buf{tmp2.w + obase, tmp2.h + obase}, run2T,
                  nch2, g);
}

// Direct hook on the level-1 buckets (no bitmap): each workgroup gathers one
// level-2 chunk, whose first endpoints all lie in one slice of 2^19 vertices,
// and hooks it. The workgroups running at one time mostly take consecutive
// chunks of one slice, so their first endpoints' parent entries (2 MB) stay in
// L2; only the second endpoints' reads are random over the whole array.
// LOOP: for a launch over many chunks that may be shut by its gate (65,000 workgroups
// that leave at once take 36 us, kShutGrid of them 9). The loop costs up to a tenth of
// the pass (grid n = 33 M, 83 M entries 9.0 ms, 9.9 with it), so the others go without.
constexpr uint32_t kShutGrid = 16384;

template <bool ZR, bool LOOP>
__global__ __launch_bounds__(kPartBlock) void k_t2_hookplain(const uint32_t* __restrict__ t1w,
                                                             const uint16_t* __restrict__ t1h,
                                                             const uint16_t* __restrict__ segT,
                                                             const uint32_t* __restrict__ pre1,
                                                             uint64_t nch1, int R,
                                                             const uint32_t* __restrict__ cbase,
                                                             const uint32_t* __restrict__ desc,
                                                             uint32_t* P, DevState* st, Gate gate) {
    if (gated_off(gate)) return;
    const uint32_t z = ZR ? ld_agent(&st->zroot) : 0u;
    __shared__ uint8_t owner[kC2];
    __shared__ uint32_t s_pre[kWin2 + 1];
    __shared__ uint32_t s_seg[kWin2];
    uint32_t g = blockIdx.x;
    do {
    if (g >= cbase[R]) return;                  // the grid is an upper bound
    u32x2 e[kPartEPT];
    int a;
    uint64_t obase;
    const uint32_t cnt = t2_gather(g, t1w, t1h, segT, pre1, nch1, desc, owner, s_pre, s_seg, e, a,
                                   obase);
    bool h[kPartEPT];
    uint32_t pu[kPartEPT], pv[kPartEPT];
#pragma unroll
    for (int k = 0; k < kPartEPT; ++k) {
        h[k] = (uint32_t)k * kPartBlock + threadIdx.x < cnt;
        if (!h[k]) e[k].x = e[k].y = 0u;
    }
#pragma unroll
    for (int k = 0; k < kPartEPT; ++k) {
        pu[k] = P[e[k].x];
        pv[k] = P[e[k].y];
    }
#pragma unroll
    for (int k = 0; k < kPartEPT; ++k) {
        const uint32_t u = e[k].x, v = e[k].y;
        if (!h[k] || u == v) continue;
        if (pu[k] == pv[k] || pu[k] == v || pv[k] == u) continue;   // same tree already
        (void)link<ZR, 1>(P, u, pu[k], v, pv[k], z);
    }
    g += gridDim.x;
    } while (LOOP);
}

// ---- CSR input: the rows are the level-1 buckets ---------------------------------
// On CSR input the entries are already grouped by first endpoint: bucket a is
// the contiguous range of adj that holds the rows of slice a, so steps 1-3 are
// replaced by reading the offsets, and the level-2 pass reads adj directly and
// recovers each position's row (as the CSR hook does). The level-2 buffer uses
// adj's positions (base2[a] = start of slice a's rows), so steps 5-6 run
// unchanged. Every bound below is clamped to a monotone sequence inside
// [0, m], so offsets that are not a valid row index (reported separately) can
// change the result but never make an access leave its array.

// base2[a] = running maximum of off[a * 2^19] clamped to m (base2[R] = m);
// cbase = prefix of the chunk counts. One block, R <= 256.
__global__ __launch_bounds__(256) void k_c_bases(const uint64_t* __restrict__ off, uint64_t n,
                                                 uint64_t m, int R, uint64_t* __restrict__ base2,
                                                 uint32_t* __restrict__ cbase) {
    __shared__ uint64_t s_b[257];
    __shared__ uint32_t s_c[256];
    const int a = threadIdx.x;
    uint64_t lo = 0;
    if (a < R) {
        lo = off[(uint64_t)a << kSliceBits];
        lo = lo < m ? lo : m;
    }
    s_b[a] = lo;
    __syncthreads();
    for (int o = 1; o < 256; o <<= 1) {                 // inclusive running maximum
        const uint64_t x = a >= o ? s_b[a - o] : 0ull;
        __syncthreads();
        s_b[a] = s_b[a] > x ? s_b[a] : x;
        __syncthreads();
    }
    if (a == 0) s_b[256] = m;
    __syncthreads();
    const uint64_t hi = a + 1 < R ? s_b[a + 1] : m;
    const uint32_t chunks = a < R ? (uint32_t)((hi - s_b[a] + kC2 - 1) / kC2) : 0u;
    s_c[a] = chunks;
    __syncthreads();
    for (int o = 1; o < 256; o <<= 1) {
        const uint32_t x = a >= o ? s_c[a - o] : 0u;
        __syncthreads();
        s_c[a] += x;
        __syncthreads();
    }
    if (a < R) {
        base2[a] = s_b[a];
        cbase[a] = s_c[a] - chunks;
    }
    if (a == R - 1) {
        base2[R] = m;
        cbase[R] = s_c[a];
    }
}

// cfirst[g]: the row holding the first position of level-2 chunk g. One thread
// per row: it writes the chunks of its slice that start inside it.
__global__ __launch_bounds__(256) void k_c_first(const uint64_t* __restrict__ off, uint64_t n,
                                                 const uint64_t* __restrict__ base2,
                                                 const uint32_t* __restrict__ cbase,
                                                 uint32_t* __restrict__ cfirst) {
    for (uint64_t v = (uint64_t)blockIdx.x * 256 + threadIdx.x; v < n;
         v += (uint64_t)gridDim.x * 256) {
        const uint64_t a = v >> kSliceBits;
        const uint64_t B0 = base2[a], B1 = base2[a + 1];
        uint64_t lo = off[v], hi = off[v + 1];
        lo = lo > B0 ? lo : B0;
        hi = hi < B1 ? hi : B1;
        if (hi <= lo) continue;
        const uint32_t cb = cbase[a];
        for (uint64_t t = (lo - B0 + kC2 - 1) / kC2; B0 + t * kC2 < hi; ++t)
            cfirst[cb + t] = (uint32_t)v;
    }
}

constexpr uint32_t kSweepMax2 = 4 * kC2;   // rows a chunk sweeps before it searches instead

__global__ __launch_bounds__(kPartBlock) void k_t2_csr(const uint64_t* __restrict__ off,
                                                       const uint32_t* __restrict__ adj,
                                                       uint64_t n, int R,
                                                       const uint64_t* __restrict__ base2,
                                                       const uint32_t* __restrict__ cbase,
                                                       const uint32_t* __restrict__ cfirst,
                                                       L2Buf tmp2,
                                                       uint16_t* __restrict__ run2T,
                                                       uint64_t nch2, DevState* st, uint32_t sym) {
    __shared__ u32x2 stage[kC2];
    // the rows of the positions live in the first half of the sort's staging
    // area: they are read into registers before t2_sort_write first writes it
    // (after two barriers), so both fit with two workgroups per CU
    uint32_t* head = reinterpret_cast<uint32_t*>(stage);
    __shared__ uint32_t hist[kMaxSlicesOther + 1];
    __shared__ uint32_t start[kMaxSlicesOther + 1];
    __shared__ uint32_t s_w[kPartBlock / 64];
    __shared__ int s_a;
    const uint32_t g = blockIdx.x;
    if (g >= cbase[R]) return;                  // the grid is an upper bound
    if (threadIdx.x == 0) {                     // the slice whose chunks hold g
        int lo = 0, hi = R - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) / 2;
            if (cbase[mid] <= g) lo = mid;
            else hi = mid - 1;
        }
        s_a = lo;
    }
    for (int i = threadIdx.x; i <= kMaxSlicesOther; i += kPartBlock) hist[i] = 0;
    for (int i = threadIdx.x; i < kC2; i += kPartBlock) head[i] = 0;
    __syncthreads();
    const int a = s_a;
    const uint64_t pos0 = base2[a] + (uint64_t)(g - cbase[a]) * kC2;
    const uint64_t pend = base2[a + 1];
    const uint32_t cnt = (uint32_t)min<uint64_t>((uint64_t)kC2, pend - pos0);
    const uint32_t vlo = (uint32_t)a << kSliceBits;
    const uint32_t vhi = (uint32_t)min<uint64_t>(((uint64_t)a + 1) << kSliceBits, n) - 1;
    auto clampv = [&](uint32_t x) { return x < vlo ? vlo : (x > vhi ? vhi : x); };
    const uint32_t ua = clampv(cfirst[g]);
    uint32_t ub = (g + 1 < cbase[a + 1]) ? clampv(cfirst[g + 1]) : vhi;
    if (ub < ua) ub = ua;
    uint32_t v[kPartEPT];
#pragma unroll
    for (int k = 0; k < kPartEPT; ++k) {
        const uint32_t i = (uint32_t)k * kPartBlock + threadIdx.x;
        v[k] = i < cnt ? __builtin_nontemporal_load(adj + pos0 + i) : 0u;
    }
    uint32_t u[kPartEPT];
    if (ub - ua <= kSweepMax2) {
        if (threadIdx.x == 0) head[0] = ua;
        for (uint64_t x0 = (uint64_t)ua + 1; x0 <= ub; x0 += 4 * kPartBlock) {
            uint64_t lo[4], hi[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const uint64_t x = x0 + r * kPartBlock + threadIdx.x;
                const uint64_t xs = x <= ub ? x : ub;
                lo[r] = off[xs];
                hi[r] = off[xs + 1];
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const uint64_t x = x0 + r * kPartBlock + threadIdx.x;
                if (x <= ub && lo[r] < hi[r] && lo[r] >= pos0 && lo[r] < pos0 + cnt)
                    head[lo[r] - pos0] = (uint32_t)x;
            }
        }
        __syncthreads();
        // inclusive max-scan of head: thread i owns head[8i .. 8i + 7]
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
        uint32_t h[kPartEPT];
#pragma unroll
        for (int r = 0; r < kPartEPT; ++r) h[r] = head[kPartEPT * threadIdx.x + r];
#pragma unroll
        for (int r = 1; r < kPartEPT; ++r) h[r] = max(h[r], h[r - 1]);
        uint32_t incl = h[kPartEPT - 1];
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t y = __shfl_up(incl, o, 64);
            if (lane >= o) incl = max(incl, y);
        }
        if (lane == 63) s_w[wave] = incl;
        uint32_t before = __shfl_up(incl, 1, 64);
        if (lane == 0) before = 0;
        __syncthreads();
        for (int w = 0; w < wave; ++w) before = max(before, s_w[w]);
#pragma unroll
        for (int r = 0; r < kPartEPT; ++r) head[kPartEPT * threadIdx.x + r] = max(h[r], before);
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kPartEPT; ++k) u[k] = head[k * kPartBlock + threadIdx.x];
    } else {
        // the last row x in [ua, ub] with off[x] <= p owns position p
#pragma unroll
        for (int k = 0; k < kPartEPT; ++k) {
            const uint64_t p = pos0 + (uint64_t)k * kPartBlock + threadIdx.x;
            uint32_t lo = ua, hi = ub;
            while (lo < hi) {
                const uint32_t mid = lo + (hi - lo + 1) / 2;
                if (off[mid] <= p) lo = mid;
                else hi = mid - 1;
            }
            u[k] = lo;
        }
    }
    bool bad = false;
    u32x2 e[kPartEPT];
#pragma unroll
    for (int k = 0; k < kPartEPT; ++k) {
        const uint32_t uu = clampv(u[k]);
        uint32_t vv = v[k];
        if ((uint32_t)k * kPartBlock + threadIdx.x < cnt && vv >= n) {
            bad = true;
            vv = uu;                              // skipped as a self-loop
        }
        if (sym && vv < uu) vv = uu;              // the reverse entry covers it
        e[k].x = uu;
        e[k].y = vv;
    }
    if (bad) atomicOr(&st->status, kStatusRange);
    t2_sort_write<kMaxSlicesOther>(e, cnt, R, hist, start, stage, L2Buf{tmp2.w + pos0, tmp2.h + pos0}, run2T, nch2,
                  g);
}

// ---- 5. the filter over bucket (a, b) with both slices' bitmap words in LDS ---------------
//
// A set bit means "connected to the zero root" (the Initial Push's bits are
// stronger: in z's tree already), as in the direct hook. An entry with
// both endpoints marked is dropped: the two are connected anyway. An entry with
// exactly one marked endpoint is dropped too, after marking the other endpoint:
// that mark is the entry's link to z, and compress later puts every tree that
// holds a marked vertex into z's component. Each mark rests on an entry and an
// earlier mark, so the marks never claim a connection the graph lacks. Only
// entries with neither endpoint marked are kept, for the survivor hook, which
// does not consult the bitmap.
constexpr int kHook3Block = 1024;
constexpr int kWaves3 = kHook3Block / 64;
constexpr int kWin3 = 1900;      // level-2 chunks per window
constexpr int kRunsInFlight = 12; // entries a lane loads at once (a wave: 12 x 64 consecutive)

// Exclusive scan in place of n <= 2 * kHook3Block values (x[n] receives the
// total); every thread of the workgroup calls it.
__device__ __forceinline__ void block_scan_2048(uint32_t* x, uint32_t n, uint32_t* wsum) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t i0 = 2 * tid, i1 = 2 * tid + 1;
    const uint32_t a0 = i0 < n ? x[i0] : 0u, a1 = i1 < n ? x[i1] : 0u;
    const uint32_t s = a0 + a1;
    uint32_t incl = s;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t y = __shfl_up(incl, off, 64);
        if (lane >= off) incl += y;
    }
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    if (tid == 0) {
        uint32_t run = 0;
        for (int w = 0; w < kHook3Block / 64; ++w) { const uint32_t t = wsum[w]; wsum[w] = run; run += t; }
        wsum[kHook3Block / 64] = run;
    }
    __syncthreads();
    const uint32_t excl = wsum[wave] + incl - s;
    if (i0 < n) x[i0] = excl;
    if (i1 < n) x[i1] = excl + a0;
    if (tid == 0) x[n] = wsum[kHook3Block / 64];
    __syncthreads();
}

// Second-endpoint slices handled by one workgroup of the two-pass filter: two up to
// 256 slices (four and eight measured 0.3 ms worse on R-MAT-26); beyond, where a
// (slice, slice) tile is mostly small against the 64 KB of bitmap it needs, eight
// share one copy of the first slice.
constexpr int kFewSlices = 256;
__host__ __device__ inline int b_per_block(int R) { return R <= kFewSlices ? 2 : 8; }

// Survivor regions: workgroup (a, bg) of the filter reads exactly the entries of
// tiles (a, b), b in group bg; its kept entries go to a region of that
// size inside [base2[a], base2[a+1]) of the survivor buffer; regions are
// consecutive, so wgoff[w + 1] ends region w (wgoff has R * nbg + 1 entries).
// One block per a.
__global__ __launch_bounds__(256) void k_t3_regions(const uint16_t* __restrict__ run2T,
                                                    uint64_t nch2, int R,
                                                    const uint32_t* __restrict__ cbase,
                                                    uint32_t* __restrict__ wgsize, Gate gate) {
    if (gated_off(gate)) return;
    // one block per (a, bg): the group's entries summed over bucket a's chunks
    __shared__ uint32_t ws[4];
    const int kb = b_per_block(R), nbg = (R + kb - 1) / kb;
    const int a = blockIdx.x / nbg, bg = blockIdx.x % nbg;
    const int blo = bg * kb, bhi = min(R, blo + kb);
    const uint32_t g0 = cbase[a], g1 = cbase[a + 1];
    uint32_t t = 0;
    for (uint32_t g = g0 + threadIdx.x; g < g1; g += 256)
        t += (uint32_t)run2T[(uint64_t)bhi * nch2 + g] - (uint32_t)run2T[(uint64_t)blo * nch2 + g];
    for (int off = 32; off > 0; off >>= 1) t += __shfl_xor(t, off, 64);
    if ((threadIdx.x & 63) == 0) ws[threadIdx.x >> 6] = t;
    __syncthreads();
    if (threadIdx.x == 0) wgsize[blockIdx.x] = ws[0] + ws[1] + ws[2] + ws[3];
}

// Per slice a, the regions' offsets: base2[a] plus the sizes of the groups
// before bg (at most 128 groups). One wave per a.
__global__ __launch_bounds__(64) void k_t3_offsets(const uint32_t* __restrict__ wgsize, int R,
                                                   const uint64_t* __restrict__ base2,
                                                   uint64_t* __restrict__ wgoff, Gate gate) {
    if (gated_off(gate)) return;
    static_assert(kFewSlices / 2 <= 128 && kMaxSlices / 8 <= 128, "two groups per lane");
    const int a = blockIdx.x, lane = threadIdx.x;
    const int kb = b_per_block(R), nbg = (R + kb - 1) / kb;
    const uint32_t* size = wgsize + (uint64_t)a * nbg;
    const uint32_t x0 = 2 * lane < nbg ? size[2 * lane] : 0u;
    const uint32_t x1 = 2 * lane + 1 < nbg ? size[2 * lane + 1] : 0u;
    uint32_t incl = x0 + x1;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t y = __shfl_up(incl, off, 64);
        if (lane >= off) incl += y;
    }
    const uint64_t run = base2[a] + (incl - x0 - x1);
    uint64_t* out = wgoff + (uint64_t)a * nbg;
    if (2 * lane < nbg) out[2 * lane] = run;
    if (2 * lane + 1 < nbg) out[2 * lane + 1] = run + x0;
    if (a == R - 1 && lane == 63) out[nbg] = run + x0 + x1;   // end of the last region
}

// Run holding index j0 of the window (last t < nw with s_pre[t] <= j0), found
// by the whole wave in two 64-way ballot steps (nw <= 64 * 64).
__device__ __forceinline__ uint32_t t3_find_run(const uint32_t* s_pre, uint32_t nw, uint32_t j0,
                                                int lane) {
    const uint32_t stride = (nw + 63) / 64;
    const uint32_t i1 = (uint32_t)lane * stride;
    const bool c1 = i1 < nw && s_pre[i1] <= j0;
    const uint64_t b1 = __ballot(c1);
    const uint32_t base = (63u - (uint32_t)__clzll((long long)b1)) * stride;
    const uint32_t i2 = base + (uint32_t)lane;
    const bool c2 = (uint32_t)lane < stride && i2 < nw && s_pre[i2] <= j0;
    const uint64_t b2 = __ballot(c2);
    return base + (63u - (uint32_t)__clzll((long long)b2));
}

// Offset of index j of the window (j in [jb, jb + 64), the indices one wave
// handles together): t is the run holding index jb, kept wave-uniform and
// advanced here to the run holding jb + 63. Runs are about as long as a wave,
// so this is usually one step; lanes past a run's end take the next run's
// offset. Every branch depends on wave-uniform values only.
__device__ __forceinline__ uint32_t t3_offset(const uint32_t* s_pre, const uint32_t* s_off,
                                              uint32_t nw, uint32_t& t, uint32_t jb, uint32_t j) {
    // the table reads have one address for the whole wave: keep them scalar
    uint32_t off = __builtin_amdgcn_readfirstlane(s_off[t]);
    uint32_t nxt = __builtin_amdgcn_readfirstlane(s_pre[t + 1]);
    while (t + 1 < nw && nxt < jb + 64) {
        ++t;
        const uint32_t o = __builtin_amdgcn_readfirstlane(s_off[t]);
        off = j >= nxt ? o : off;
        nxt = __builtin_amdgcn_readfirstlane(s_pre[t + 1]);
    }
    return off;
}

// The marks a workgroup added to its copy of a slice go to the global bitmap in
// one pass over the words, with one atomic per word that gained bits there (an
// atomic per mark would repeat every mark in each of the slice's workgroups:
// R-MAT n = 2^22, 2^26 entries: filter 782 -> 472 us).
__device__ __forceinline__ void t3_flush(const uint32_t* w, uint32_t* zbits, uint64_t w0,
                                         uint64_t words) {
    constexpr int PER = 4;
    for (uint32_t at = threadIdx.x; at < kSliceWords; at += PER * kHook3Block) {
        uint32_t g[PER];
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const uint64_t i = w0 + at + (uint32_t)k * kHook3Block;
            g[k] = i < words ? ld_agent(&zbits[i]) : kEmpty;
        }
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const uint32_t i = at + (uint32_t)k * kHook3Block;
            const uint32_t add = w[i] & ~g[k];
            if (add) atomicOr(&zbits[w0 + i], add);
        }
    }
}

// What a launch of the filter does with the entries that neither bit settles.
//  kMarkTiles  only marks (the first eighth of each workgroup's entries of the
//              one-pass tiles): the entries all come again in the full pass. Each
//              workgroup knows only the marks its copies held at the start and
//              those of its own entries; this launch's flush shows every workgroup
//              the others' marks before any entry is hooked (R-MAT n = 2^22, 2^26
//              entries: both passes 335 us, the full one alone 472).
//  kFullTiles  the one-pass tiles: hooked in P from the wave's queue. Its walks are
//              short where the giant component was sampled, so they split late: on
//              R-MAT n = 2^22 late, full and no splitting take 513, 511 and 516 us
//              whole, but a path of 2 M vertices beside 2 M vertices of a uniform
//              graph (entries in order) 4.0 ms split late, 4.5 split fully; without
//              any, each walk would be as long as the path hooked so far.
//  The one-pass tiles are one index space, tile after tile, cut into equal parts,
//  one per workgroup: lists whose first endpoints lie in few slices (a share of a
//  larger graph, sorted rows) fill few tiles.
//  kFullRuns   the two-pass tiles: kept for the survivor hook (a tile is short,
//              2^16 entries on R-MAT-26, and hooking its rest at its end
//              would leave the CU waiting: filter 4.2 ms against 2.9 + 0.4)
//  kManyRuns   the same beyond kFewSlices slices, where a tile is small: marks go
//              to the global bitmap one by one, where the others see them at once
//              (t3_flush's pass over a slice costs as much as some ten thousand)
//  kMixedRuns  the same on lists whose workgroups may be small: those of fewer than
//              kFlushEntries entries mark one by one (zero root, ER n = 67 M, 60 M
//              entries 7.6 ms with flushes, 7.1 so; a twentieth of R-MAT-26 2.4 and
//              1.9), the others flush: a share of a larger graph fills few first slices
//              (16 shares of R-MAT-26: 21.3 ms with flushes, 27.4 one by one). The small
//              ones also write the entries that are kept, which are most, when they are
//              first settled; where marks settle most, a second look when the second
//              queue is full saves more (R-MAT-24 rows, 60 M entries, 121,000 to a
//              workgroup: survivor hook 65 us with it, 118 without). The choice in the
//              kernel spills three registers, so long lists take kFullRuns.
enum FilterMode { kMarkTiles, kFullTiles, kFullRuns, kManyRuns, kMixedRuns };
constexpr uint32_t kFlushEntries = 32768;
constexpr uint32_t kMarkPart = 8;
constexpr uint32_t kTileCost = 8192;  // entries' worth of a tile's fixed time (8 us)

template <int MODE>
__global__ __launch_bounds__(kHook3Block) void k_t3_filter(L2Buf tmp2,
                                                           const uint16_t* __restrict__ run2T,
                                                           uint64_t nch2, int R,
                                                           const uint32_t* __restrict__ wcnt,
                                                           const uint64_t* __restrict__ base2,
                                                           const uint32_t* __restrict__ cbase,
                                                           uint32_t* zbits, uint64_t words,
                                                           uint32_t* P, uint32_t* __restrict__ sw,
                                                           uint16_t* __restrict__ sh,
                                                           const uint64_t* __restrict__ wgoff,
                                                           uint32_t* __restrict__ wgcnt,
                                                           DevState* st, Gate gate) {
    if (gated_off(gate)) return;
    constexpr bool RUNS = MODE >= kFullRuns, TILES = !RUNS;
    __shared__ uint32_t sa[kSliceWords];
    __shared__ uint32_t sb[kSliceWords];
    __shared__ uint32_t s_off[kWin3];
    __shared__ uint32_t s_pre[kWin3 + 1];
    __shared__ u32x2 s_queue[kWaves3 * 2 * kQueueCap];
    __shared__ uint32_t wsum[kWaves3 + 1];
    const uint32_t z = ld_agent(&st->zroot);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    // Launch order: consecutive workgroups take different a (and spread over
    // the b groups), so the workgroups running at the same time hold few
    // copies of any one slice and see each other's marks through the global
    // bitmap sooner. (a, bg) = (i mod R, (i div R + a) mod nbg) is a bijection.
    const int kB = TILES ? 1 : b_per_block(R);
    const uint32_t nbg = ((uint32_t)R + kB - 1) / kB;
    int a = (int)(blockIdx.x % (uint32_t)R);
    const int bg = (int)((blockIdx.x / (uint32_t)R + (uint32_t)a) % nbg);
    uint32_t cb = 0, nch = (uint32_t)nch2;               // first chunk, chunks
    const uint32_t* srcw = tmp2.w;
    const uint8_t* srch = tmp2.h;
    // one-pass tiles: this workgroup's entries [lo, hi) of the tiles' index space;
    // d is the tile they are in now, at its index td, nd wide; a tile's width is its
    // entries and kTileCost more, the time its slices take to load and write back
    const uint32_t nwin = ((uint32_t)nch2 + kWin3 - 1) / kWin3;
    uint32_t lo = 0, hi = 0, d = 0, td = 0, nd = 0;
    if (TILES) {
        const uint32_t tiles = (uint32_t)(R * R);
        for (uint32_t i = threadIdx.x; i < tiles; i += kHook3Block) {
            uint32_t t = 0;
            for (uint32_t w = 0; w < nwin; ++w) t += wcnt[(uint64_t)i * nwin + w];
            s_off[i] = t ? t + kTileCost : 0u;
        }
        __syncthreads();
        wave_scan<8>(s_off, s_pre, (int)tiles);
        __syncthreads();
        const uint64_t all = s_pre[tiles];
        lo = (uint32_t)(all * blockIdx.x / gridDim.x);
        hi = (uint32_t)(all * (blockIdx.x + 1ull) / gridDim.x);
        if (lo >= hi) return;
        if (MODE == kMarkTiles) hi = lo + (hi - lo + kMarkPart - 1) / kMarkPart;
        for (uint32_t i = threadIdx.x; i < tiles; i += kHook3Block)
            if (s_pre[i] <= lo && lo < s_pre[i + 1]) { wsum[0] = i; wsum[1] = s_pre[i]; wsum[2] = s_off[i]; }
        __syncthreads();
        d = __builtin_amdgcn_readfirstlane(wsum[0]);
        td = __builtin_amdgcn_readfirstlane(wsum[1]);
        nd = __builtin_amdgcn_readfirstlane(wsum[2]);
        a = (int)(d / (uint32_t)R);
        __syncthreads();
    } else {
        cb = cbase[a];
        nch = cbase[a + 1] - cb;
        srcw = tmp2.w + base2[a];
        srch = tmp2.h + base2[a];
    }
    const uint32_t wi = (uint32_t)a * nbg + (uint32_t)bg;   // region index (kFullRuns)
    __shared__ uint32_t s_used;
    if (RUNS && threadIdx.x == 0) {
        s_used = 0;
        if (nch == 0) wgcnt[wi] = 0;
    }
    if (nch == 0) return;
    uint32_t* ow = nullptr;
    uint16_t* oh = nullptr;
    uint32_t cap = 0;
    if (RUNS) {
        ow = sw + wgoff[wi];
        oh = sh + wgoff[wi];
        cap = (uint32_t)(wgoff[wi + 1] - wgoff[wi]);
    }
    const bool direct = MODE == kMixedRuns && cap < kFlushEntries;
    const bool one_by_one = MODE == kManyRuns || direct;
    constexpr int PER = kSliceWords / kHook3Block;       // 16 words per thread per slice
    auto load_slice = [&](uint32_t* dst, int slice) {
        const uint64_t w0 = (uint64_t)slice * kSliceWords;
        uint32_t x[PER];
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const uint64_t i = (uint64_t)k * kHook3Block + threadIdx.x;
            x[k] = w0 + i < words ? zbits[w0 + i] : 0u;
        }
#pragma unroll
        for (int k = 0; k < PER; ++k) dst[(uint32_t)k * kHook3Block + threadIdx.x] = x[k];
    };
    load_slice(sa, a);
    WaveQueues q;
    q.pq = s_queue + wave * 2 * kQueueCap;
    q.lq = q.pq + kQueueCap;
    constexpr uint32_t kRange = 64 * kRunsInFlight;      // entries per wave per range
    constexpr uint32_t kStep = kWaves3 * kRange;
    for (int bi = 0; TILES || bi < kB; ++bi) {
        if (TILES && bi) {
            // the next tile that holds entries (there is one: td + nd < hi)
            if (td + nd >= hi) break;
            do {
                td += nd;
                ++d;
                nd = 0;
                for (uint32_t w = 0; w < nwin; ++w) nd += wcnt[(uint64_t)d * nwin + w];
                nd = nd ? nd + kTileCost : 0u;
            } while (nd == 0);
            const int na = (int)(d / (uint32_t)R);
            if (na != a) {
                __syncthreads();
                t3_flush(sa, zbits, (uint64_t)a * kSliceWords, words);
                __syncthreads();
                a = na;
                load_slice(sa, a);
            }
        }
        const int b = TILES ? (int)(d % (uint32_t)R) : bg * kB + bi;
        if (b >= R) break;
        // the entries [jlo, jhi) of the tile are this workgroup's
        const uint32_t jlo = TILES && lo > td ? lo - td : 0u;
        const uint32_t jhi = TILES ? min(hi - td, nd - kTileCost) : 0xFFFFFFFFu;
        if (TILES && jlo >= jhi) continue;                // only the cost's end of the tile
        __syncthreads();                                  // previous slice b fully used
        if (b != a) load_slice(sb, b);
        uint32_t* lb = (a == b) ? sa : sb;
        const uint32_t abase = (uint32_t)a << kSliceBits;
        const uint32_t bbase = (uint32_t)b << kSliceBits;
        const uint64_t row = TILES ? d : (uint32_t)b;
        uint32_t jw = 0;                                  // tile index of the window's first
        // Second looks (endpoints relative to the slices' first IDs), with the bits as
        // they are then: both marked, dropped; one marked, the other is marked (in
        // LDS; t3_flush takes the slice's new marks to the global bitmap); neither,
        // hooked in P (Algorithm 3, walks split from their sixteenth step on).
        auto settle = [&](u32x2 x) {
            const bool mu = (sa[x.x >> 5] >> (x.x & 31)) & 1u, mv = (lb[x.y >> 5] >> (x.y & 31)) & 1u;
            if (mu != mv) {
                const uint32_t lo = mu ? x.y : x.x, bit = 1u << (lo & 31);
                const uint32_t old = atomicOr(mu ? &lb[lo >> 5] : &sa[lo >> 5], bit);
                if (one_by_one && !(old & bit)) {
                    const uint32_t y = (mu ? bbase : abase) + lo;
                    atomicOr(&zbits[y >> 5], bit);
                }
            }
            return !mu && !mv;
        };
        auto hook = [&](u32x2 x) {
            const uint32_t u = abase + x.x, v = bbase + x.y;
            if (MODE == kMarkTiles) return;
            if (RUNS) {
                // one lane reserves room for all that are here
                const uint64_t here = __ballot(true);
                const int first = __ffsll((unsigned long long)here) - 1;
                uint32_t at = 0;
                if (lane == first) at = atomicAdd(&s_used, (uint32_t)__popcll(here));
                at = __shfl(at, first, 64) + (uint32_t)__popcll(here & ((1ull << lane) - 1ull));
                if (at < cap) {
                    ow[at] = pk_w(x.x, v);
                    oh[at] = (uint16_t)(v >> (32 - kSliceBits));
                } else {
                    // cannot happen (the region holds all of the workgroup's entries)
                    atomicOr(&st->status, kStatusInternal);
                }
                return;
            }
            const uint32_t pu = P[u], pv = P[v];
            if (u == v || pu == pv || pu == v || pv == u) return;
            (void)link<true, kLateSplit>(P, u, pu, v, pv, z);
        };
        for (uint32_t w0 = 0; w0 < nch; w0 += kWin3) {
            const uint32_t nw = min((uint32_t)kWin3, nch - w0);
            if (TILES) {
                if (jw >= jhi) break;
                const uint32_t wn = wcnt[row * nwin + w0 / kWin3];
                if (jw + wn <= jlo) { jw += wn; continue; }
            }
            __syncthreads();
            for (uint32_t t = threadIdx.x; t < nw; t += kHook3Block) {
                const uint64_t g = (uint64_t)cb + w0 + t;
                const uint32_t r0 = run2T[row * nch2 + g];
                const uint32_t r1 = run2T[(row + 1) * nch2 + g];
                s_off[t] = r0;
                s_pre[t] = r1 - r0;
            }
            __syncthreads();
            block_scan_2048(s_pre, nw, wsum);        // run lengths -> starts; s_pre[nw] = total
            // index of the window's j-th entry in run t: j + s_off[t] (mod 2^32;
            // every index of a bucket is below 2^32)
            for (uint32_t t = threadIdx.x; t < nw; t += kHook3Block)
                s_off[t] = (w0 + t) * (uint32_t)kC2 + s_off[t] - s_pre[t];
            __syncthreads();
            const uint32_t total = TILES ? min(s_pre[nw], jhi - jw) : s_pre[nw];
            const uint32_t first = TILES && jlo > jw ? jlo - jw : 0u;
            if (TILES) jw += s_pre[nw];
            if (s_pre[nw] < 8 * nw) {
                // Short runs (a slice of few vertices): following them one by one
                // would take a step per run, empty ones too; each lane searches its own.
                // (R-MAT n = 2^23 + 4099, 15 M entries: filter 2340 us following, 246 searching)
                for (uint32_t jb = first + (uint32_t)wave * 64; jb < total; jb += kHook3Block) {
                    const uint32_t j = jb + (uint32_t)lane;
                    const bool h = j < total;
                    uint32_t at = 0;
                    if (h) {
                        uint32_t t0 = 0, t1 = nw;            // s_pre[t0] <= j < s_pre[t1]
                        while (t1 - t0 > 1) {
                            const uint32_t tm = (t0 + t1) / 2;
                            if (s_pre[tm] <= j) t0 = tm;
                            else t1 = tm;
                        }
                        at = j + s_off[t0];
                    }
                    at = h ? at : __builtin_amdgcn_readfirstlane(at);   // lane 0 has an entry
                    const uint32_t w = srcw[at], h8 = srch[at];
                    const u32x2 x = {w & kLoMask, (w >> kSliceBits) | (h8 << (32 - kSliceBits))};
                    const uint32_t both =
                        (sa[x.x >> 5] >> (x.x & 31)) & (lb[x.y >> 5] >> (x.y & 31)) & 1u;
                    if (MODE == kMarkTiles) {
                        if (h && !both) (void)settle(x);
                    } else {
                        queue_push(q, lane, h && !both, x, settle, hook, direct);
                    }
                }
                continue;
            }
            // The window's entries form one index space [0, total); each wave
            // takes ranges of kRange consecutive indices. Register k holds index
            // j0 + 64k + lane; right after it is tested it is reloaded with index
            // jn + 64k + lane of the next range, so the next range's loads are in
            // flight meanwhile. Past the end a lane reads the wave's first entry: a
            // slot that no entry was written to (a chunk's first one may be such, when
            // all of its entries were dropped) can hold endpoints beyond a slice, whose
            // bit test would read past the slice's words.
            uint32_t j0 = first + (uint32_t)wave * kRange;
            if (j0 >= total) continue;
            uint32_t ew[kRunsInFlight], eh[kRunsInFlight];
            uint32_t t = __builtin_amdgcn_readfirstlane(t3_find_run(s_pre, nw, j0, lane));
            uint32_t safe = 0;                               // the entry j0 (j0 < total)
#pragma unroll
            for (int k = 0; k < kRunsInFlight; ++k) {
                const uint32_t jb = j0 + (uint32_t)k * 64, j = jb + (uint32_t)lane;
                const uint32_t off = t3_offset(s_pre, s_off, nw, t, jb, j);
                if (k == 0) safe = __builtin_amdgcn_readfirstlane(j + off);
                const uint32_t at = j < total ? j + off : safe;
                ew[k] = __builtin_nontemporal_load(srcw + at);
                eh[k] = __builtin_nontemporal_load(srch + at);
            }
            while (true) {
                const uint32_t jn = j0 + kStep;
                const bool more = jn < total;
                uint32_t tn = more ? __builtin_amdgcn_readfirstlane(t3_find_run(s_pre, nw, jn, lane)) : 0u;
#pragma unroll
                for (int k = 0; k < kRunsInFlight; ++k) {
                    const u32x2 x = {ew[k] & kLoMask, (ew[k] >> kSliceBits) | (eh[k] << (32 - kSliceBits))};
                    {
                        const uint32_t jb = jn + (uint32_t)k * 64, j = jb + (uint32_t)lane;
                        const uint32_t off = more ? t3_offset(s_pre, s_off, nw, tn, jb, j) : 0u;
                        const uint32_t at = more && j < total ? j + off : safe;
                        ew[k] = __builtin_nontemporal_load(srcw + at);
                        eh[k] = __builtin_nontemporal_load(srch + at);
                    }
                    const bool h = j0 + (uint32_t)k * 64 + (uint32_t)lane < total;
                    const uint32_t both =
                        (sa[x.x >> 5] >> (x.x & 31)) & (lb[x.y >> 5] >> (x.y & 31)) & 1u;
                    const bool pend = h && !both;
                    if (MODE == kMarkTiles) {
                        if (pend) (void)settle(x);
                    } else {
                        queue_push(q, lane, pend, x, settle, hook, direct);
                    }
                }
                if (!more) break;
                j0 = jn;
            }
        }
        // this slice's pending entries are settled before the next slice's
        // bitmap replaces it
        if (MODE != kMarkTiles) queue_finish(q, lane, settle, hook, direct);
        if (b != a && !one_by_one) {
            __syncthreads();
            t3_flush(sb, zbits, (uint64_t)b * kSliceWords, words);
        }
    }
    __syncthreads();
    if (!one_by_one) t3_flush(sa, zbits, (uint64_t)a * kSliceWords, words);
    if (RUNS && threadIdx.x == 0) wgcnt[wi] = min(s_used, cap);
}

// ---- 6. the survivor hook -------------------------------------------------------------------
// Work items of kItem consecutive entries of one region: an exclusive prefix of
// the regions' item counts, then a grid-stride loop over items, each mapped to
// its region by a binary search of that prefix (regions are of very different
// sizes: R-MAT-26's 320,000 path entries survive in two).
constexpr int kPackBlock = 1024;
constexpr uint32_t kItem = 1024;     // entries per work item (4 per thread)

// ipref[w] = sum over v < w of ceil(cnt[v] / kItem); ipref[nw] = total; one block.
__global__ __launch_bounds__(kPackBlock) void k_t4_scan(const uint32_t* __restrict__ cnt,
                                                        uint32_t nw, uint32_t* __restrict__ ipref, Gate gate) {
    if (gated_off(gate)) return;
    __shared__ uint32_t ws[kPackBlock / 64 + 1];
    __shared__ uint32_t s_carry;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (threadIdx.x == 0) s_carry = 0;
    for (uint32_t base = 0; base < nw; base += kPackBlock) {
        const uint32_t i = base + threadIdx.x;
        const uint32_t x = i < nw ? (cnt[i] + kItem - 1) / kItem : 0u;
        uint32_t incl = x;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t y = __shfl_up(incl, off, 64);
            if (lane >= off) incl += y;
        }
        if (lane == 63) ws[wave] = incl;
        __syncthreads();
        if (threadIdx.x == 0) {
            uint32_t run = s_carry;
            for (int w = 0; w < kPackBlock / 64; ++w) { const uint32_t t = ws[w]; ws[w] = run; run += t; }
            ws[kPackBlock / 64] = run;
        }
        __syncthreads();
        if (i < nw) ipref[i] = ws[wave] + incl - x;
        __syncthreads();
        if (threadIdx.x == 0) s_carry = ws[kPackBlock / 64];
        __syncthreads();
    }
    if (threadIdx.x == 0) ipref[nw] = s_carry;
}

// Algorithm 3's hooking loop (keys of Formula 1 as an order, path splitting)
// over the kept entries. Their bits are tested once more first: every
// workgroup's marks are in the bitmap by now, and most entries were kept only
// because their own workgroup had not seen them. Where no giant component was seen
// the test drops little and is left out (zero root, ER n = 67 M, 60 M entries:
// 6.1 ms with it, 5.5 without).
constexpr int kHook4Block = 256;
constexpr int kHook4EPT = (int)kItem / kHook4Block;
constexpr int kHook4Grid = 2048;     // 8 workgroups per CU

__global__ __launch_bounds__(kHook4Block) void k_t4_hook(const uint32_t* __restrict__ sw,
                                                         const uint16_t* __restrict__ sh,
                                                         const uint64_t* __restrict__ wgoff,
                                                         const uint32_t* __restrict__ cnt,
                                                         const uint32_t* __restrict__ ipref,
                                                         uint32_t nw, int nbg, uint32_t* P,
                                                         uint32_t* zbits, DevState* st, Gate again,
                                                         Gate gate) {
    if (gated_off(gate)) return;
    __shared__ uint32_t s_w;
    const uint32_t z = ld_agent(&st->zroot);
    const uint32_t items = ld_agent(&ipref[nw]);
    const bool test = !gated_off(again);
    for (uint32_t it = blockIdx.x; it < items; it += gridDim.x) {
        __syncthreads();                       // s_w of the previous item consumed
        if (threadIdx.x == 0) {
            uint32_t lo = 0, hi = nw - 1;      // last w with ipref[w] <= it
            while (lo < hi) {
                const uint32_t mid = (lo + hi + 1) / 2;
                if (ipref[mid] <= it) lo = mid; else hi = mid - 1;
            }
            s_w = lo;
        }
        __syncthreads();
        const uint32_t w = s_w;
        const uint32_t abase = (uint32_t)(w / (uint32_t)nbg) << kSliceBits;
        const uint32_t k0 = (it - ipref[w]) * kItem;
        const uint32_t c = min(cnt[w] - k0, kItem);
        const uint64_t base = wgoff[w] + k0;
        uint32_t u[kHook4EPT], v[kHook4EPT];
        bool h[kHook4EPT];
#pragma unroll
        for (int k = 0; k < kHook4EPT; ++k) {
            const uint32_t i = (uint32_t)k * kHook4Block + threadIdx.x;
            h[k] = i < c;
            const uint64_t at = base + (h[k] ? i : 0u);
            const uint32_t x = sw[at];
            u[k] = abase | (x & kLoMask);
            v[k] = pk_v1(x, sh[at]);
        }
        uint32_t bu[kHook4EPT], bv[kHook4EPT];
#pragma unroll
        for (int k = 0; k < kHook4EPT; ++k) {
            bu[k] = test ? ld_agent(&zbits[u[k] >> 5]) : 0u;
            bv[k] = test ? ld_agent(&zbits[v[k] >> 5]) : 0u;
        }
#pragma unroll
        for (int k = 0; k < kHook4EPT; ++k) {
            const bool mu = (bu[k] >> (u[k] & 31)) & 1u, mv = (bv[k] >> (v[k] & 31)) & 1u;
            if (h[k] && mu != mv) {
                if (mu) atomicOr(&zbits[v[k] >> 5], 1u << (v[k] & 31));
                else atomicOr(&zbits[u[k] >> 5], 1u << (u[k] & 31));
            }
            h[k] = h[k] && !mu && !mv;
        }
        uint32_t pu[kHook4EPT], pv[kHook4EPT];
#pragma unroll
        for (int k = 0; k < kHook4EPT; ++k) {
            pu[k] = P[h[k] ? u[k] : 0u];
            pv[k] = P[h[k] ? v[k] : 0u];
        }
#pragma unroll
        for (int k = 0; k < kHook4EPT; ++k) {
            if (!h[k]) continue;
            if (pu[k] == pv[k] || pu[k] == v[k] || pv[k] == u[k]) continue;
            (void)link<true, 1>(P, u[k], pu[k], v[k], pv[k], z);
        }
    }
}

// ---- few slices: one pass over (a, b) ------------------------------------------------------
// With at most kMaxOnePass slices the (a, b) tiles are few enough (R * R <= 484)
// that one LDS sort of an 8192-entry chunk leaves runs of 17 entries per tile, on
// average and on uniform lists (others leave shorter and empty ones), so the second
// partition pass (11 B per entry read and written, and its tables) is not needed: 8 B
// read, 5 written, 5 read per entry in all. The tiles take the filter's form at once:
// chunk c's entries at [c * kC2, ...) sorted by tile, run2T[d * nch + c] the start of
// tile d's run.
constexpr int kMaxOnePass = 22;
constexpr int kMaxTiles = kMaxOnePass * kMaxOnePass;

template <typename T>
__global__ __launch_bounds__(kPartBlock) void k_tile_part(const T edges, uint64_t m,
                                                          uint32_t n, int R, uint64_t nch,
                                                          L2Buf out, uint16_t* __restrict__ run2T,
                                                          DevState* st, uint32_t sym, Gate gate) {
    if (gated_off(gate)) return;
    __shared__ u32x2 stage[kC2];
    __shared__ uint32_t hist[kMaxTiles + 1];
    __shared__ uint32_t start[kMaxTiles + 1];
    const uint64_t c = blockIdx.x;
    const int tiles = R * R;
    for (int i = threadIdx.x; i <= tiles; i += kPartBlock) hist[i] = 0;
    __syncthreads();
    u32x2 e[kPartEPT];
    uint16_t rank[kPartEPT];
    bool bad = false;
#pragma unroll
    for (int k = 0; k < kPartEPT; ++k) {
        const uint64_t i = c * kC2 + (uint64_t)k * kPartBlock + threadIdx.x;
        e[k] = load_entry(edges, i < m ? i : m - 1);
    }
    auto tile = [&](u32x2 x) { return (x.x >> kSliceBits) * (uint32_t)R + (x.y >> kSliceBits); };
#pragma unroll
    for (int k = 0; k < kPartEPT; ++k) {
        const uint64_t i = c * kC2 + (uint64_t)k * kPartBlock + threadIdx.x;
        bool live = i < m;
        if (live && (e[k].x >= n || e[k].y >= n)) { bad = true; live = false; }
        live = live && (sym ? e[k].x < e[k].y : e[k].x != e[k].y);
        rank[k] = 0xFFFF;
        if (live) rank[k] = (uint16_t)atomicAdd(&hist[tile(e[k])], 1u);
    }
    if (bad) atomicOr(&st->status, kStatusRange);
    __syncthreads();
    wave_scan<8>(hist, start, tiles);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kPartEPT; ++k)
        if (rank[k] != 0xFFFF) stage[start[tile(e[k])] + rank[k]] = e[k];
    __syncthreads();
    const uint32_t kept = start[tiles];
    for (uint32_t i = threadIdx.x; i < kept; i += kPartBlock) {
        const u32x2 x = stage[i];
        const uint32_t vlo = x.y & kLoMask;
        out.w[c * kC2 + i] = (x.x & kLoMask) | (vlo << kSliceBits);
        out.h[c * kC2 + i] = (uint8_t)(vlo >> (32 - kSliceBits));
    }
    for (int d = threadIdx.x; d <= tiles; d += kPartBlock)
        run2T[(uint64_t)d * nch + c] = (uint16_t)start[d];
}

// wcnt[d * nwin + w]: entries of tile d in the w-th window of kWin3 chunks. One
// block per (d, w).
__global__ __launch_bounds__(256) void k_tile_count(const uint16_t* __restrict__ run2T, uint64_t nch,
                                                    uint32_t nwin, uint32_t* __restrict__ wcnt,
                                                    Gate gate) {
    if (gated_off(gate)) return;
    __shared__ uint32_t ws[4];
    const uint64_t d = blockIdx.x / nwin, w = blockIdx.x % nwin;
    const uint64_t c1 = min((w + 1) * kWin3, nch);
    uint32_t t = 0;
    for (uint64_t c = w * kWin3 + threadIdx.x; c < c1; c += 256)
        t += (uint32_t)run2T[(d + 1) * nch + c] - (uint32_t)run2T[d * nch + c];
    for (int off = 32; off > 0; off >>= 1) t += __shfl_xor(t, off, 64);
    if ((threadIdx.x & 63) == 0) ws[threadIdx.x >> 6] = t;
    __syncthreads();
    if (threadIdx.x == 0) wcnt[blockIdx.x] = ws[0] + ws[1] + ws[2] + ws[3];
}

// The tiles' entries hooked in P, without a bitmap, tile after tile: for lists whose
// sample shows no giant component. Both endpoints' parent entries of a tile are 2 MB
// each. The tiles are one index space (a tile kVisit wider than its entries, the time
// its run table takes to read) cut into parts, one per workgroup: kHookPart, or wider
// on long lists (kHookParts of them; 16,000 workgroups that leave at a shut gate take 9
// us, these 5). Consecutive workgroups go to the XCDs in turn, so part numbers are dealt
// so that an XCD's workgroups take neighbouring parts and share the slices in its L2.
// Bound by the reads of the parents: 12 parts dealt over n = 4 M, 64 M entries, whole
// solve 1.59 ms; by first-endpoint buckets, without the sample, 2.00.
constexpr uint32_t kHookPart = 8192, kHookParts = 8192;
constexpr uint32_t kVisit = 1024;
constexpr int kXcds = 8;
constexpr int kTileEPT = 4;

template <bool ZR>
__global__ __launch_bounds__(kHook3Block) void k_tile_hook(L2Buf tmp2,
                                                           const uint16_t* __restrict__ run2T,
                                                           uint64_t nch, int R,
                                                           const uint32_t* __restrict__ wcnt,
                                                           uint32_t* P, DevState* st,
                                                           uint32_t wide_part, Gate gate) {
    if (gated_off(gate)) return;
    __shared__ uint32_t s_off[kWin3];
    __shared__ uint32_t s_pre[kWin3 + 1];
    __shared__ uint32_t s_tile[kMaxTiles + 1];
    __shared__ uint32_t wsum[kWaves3 + 1];
    const uint32_t z = ZR ? ld_agent(&st->zroot) : 0u;
    const uint32_t tiles = (uint32_t)(R * R);
    const uint32_t nwin = ((uint32_t)nch + kWin3 - 1) / kWin3;
    for (uint32_t i = threadIdx.x; i < tiles; i += kHook3Block) {
        uint32_t t = 0;
        for (uint32_t w = 0; w < nwin; ++w) t += wcnt[(uint64_t)i * nwin + w];
        s_off[i] = t ? t + kVisit : 0u;
    }
    __syncthreads();
    wave_scan<8>(s_off, s_tile, (int)tiles);
    __syncthreads();
    const uint32_t all = s_tile[tiles];
    const uint32_t parts = (all + wide_part - 1) / wide_part, per = (parts + kXcds - 1) / kXcds;
    const uint32_t part = blockIdx.x % kXcds * per + blockIdx.x / kXcds;
    if (blockIdx.x / kXcds >= per || part >= parts) return;
    const uint32_t lo = part * wide_part, hi = min(all, lo + wide_part);
    uint32_t d = 0;
    for (uint32_t top = tiles; top - d > 1;) {              // last d with s_tile[d] <= lo
        const uint32_t mid = (d + top) / 2;
        if (s_tile[mid] <= lo) d = mid;
        else top = mid;
    }
    for (; d < tiles && s_tile[d] < hi; ++d) {
        const uint32_t wide = s_tile[d + 1] - s_tile[d];
        if (!wide) continue;
        const uint32_t jlo = lo > s_tile[d] ? lo - s_tile[d] : 0u;
        const uint32_t jhi = min(hi - s_tile[d], wide - kVisit);
        if (jlo >= jhi) continue;                           // only the visit's end
        const uint32_t abase = d / (uint32_t)R << kSliceBits, bbase = d % (uint32_t)R << kSliceBits;
        uint32_t jw = 0;                                    // tile index of the window's first
        for (uint32_t w0 = 0; w0 < (uint32_t)nch && jw < jhi; w0 += kWin3) {
            const uint32_t wn = wcnt[(uint64_t)d * nwin + w0 / kWin3];
            if (jw + wn <= jlo) { jw += wn; continue; }
            const uint32_t nw = min((uint32_t)kWin3, (uint32_t)nch - w0);
            __syncthreads();
            for (uint32_t t = threadIdx.x; t < nw; t += kHook3Block) {
                const uint64_t g = (uint64_t)w0 + t;
                const uint32_t r0 = run2T[(uint64_t)d * nch + g];
                s_off[t] = r0;
                s_pre[t] = run2T[(uint64_t)(d + 1) * nch + g] - r0;
            }
            __syncthreads();
            block_scan_2048(s_pre, nw, wsum);
            for (uint32_t t = threadIdx.x; t < nw; t += kHook3Block)
                s_off[t] = (w0 + t) * (uint32_t)kC2 + s_off[t] - s_pre[t];
            __syncthreads();
            const uint32_t total = min(wn, jhi - jw), first = jlo > jw ? jlo - jw : 0u;
            jw += wn;
            for (uint32_t jb = first + threadIdx.x; jb < total; jb += kTileEPT * kHook3Block) {
                uint32_t u[kTileEPT], v[kTileEPT], pu[kTileEPT], pv[kTileEPT];
#pragma unroll
                for (int k = 0; k < kTileEPT; ++k) {
                    const uint32_t j = min(jb + (uint32_t)k * kHook3Block, total - 1);
                    uint32_t t0 = 0, t1 = nw;               // s_pre[t0] <= j < s_pre[t1]
                    while (t1 - t0 > 1) {
                        const uint32_t tm = (t0 + t1) / 2;
                        if (s_pre[tm] <= j) t0 = tm;
                        else t1 = tm;
                    }
                    const uint32_t at = j + s_off[t0], w = tmp2.w[at], h8 = tmp2.h[at];
                    u[k] = abase | (w & kLoMask);
                    v[k] = bbase | (w >> kSliceBits) | (h8 << (32 - kSliceBits));
                }
#pragma unroll
                for (int k = 0; k < kTileEPT; ++k) { pu[k] = P[u[k]]; pv[k] = P[v[k]]; }
#pragma unroll
                for (int k = 0; k < kTileEPT; ++k) {
                    if (jb + (uint32_t)k * kHook3Block >= total) continue;
                    if (pu[k] == pv[k] || pu[k] == v[k] || pv[k] == u[k]) continue;
                    (void)link<ZR, 1>(P, u[k], pu[k], v[k], pv[k], z);
                }
            }
        }
    }
}

// ---- host side --------------------------------------------------------------------

static int slices(uint64_t n) { return (int)((n + (1ull << kSliceBits) - 1) >> kSliceBits); }

// The plain hook of a step call takes the first-endpoint buckets from 4 slices
// (ER n = 2^21, 16 entries per vertex: 1.04 ms regrouped against 1.79 ms direct).
bool tiled_eligible(uint64_t n, uint64_t m, bool zr) {
    const uint64_t R = (n + (1ull << kSliceBits) - 1) >> kSliceBits;
    return R >= (zr ? 8u : 4u) && R <= (uint64_t)kMaxSlicesOther && m >= (1ull << 24) &&
           m < (1ull << 32);
}

// The filter over tiles: 0 = not taken, 1 = one partition pass, 2 = two. Below one
// entry per vertex a plain solve's component is seldom worth it; with a zero root
// two passes take such lists too, since a share of a skewed graph is one (a
// twentieth of R-MAT-26, n = 71 M, 52 M entries: 1.4 ms against 2.7 direct; ER
// n = 67 M, 60 M entries 7.1 and 8.6, pieces of a path 5.8 and 3.4). A plain solve
// takes two passes from 5/2 entries per vertex where it has the buckets too (ER
// n = 67 M, 134 M entries 10.1 ms against 9.3 by buckets, 200 M 10.5 and 11.9).
// Two passes start at the size their fixed costs (16 launches) are worth; one pass was faster from 2^20 entries on
// (R-MAT n = 3 M, 12 M entries: 918 us direct, 314 here). Up to 512 slices: a
// sixteenth of R-MAT-28 (n = 2^28, 2^28 entries), 10.0 ms direct, 7.1 here (plain
// 13.5 and 6.6); beyond, a tile holds fewer entries than its bitmaps words.
int filter_passes(uint64_t n, uint64_t m, bool zr) {
    const uint64_t R = (n + (1ull << kSliceBits) - 1) >> kSliceBits;
    if (n <= lds_bits_max_n() || R > (uint64_t)kMaxSlices || m >= (1ull << 32)) return 0;
    if (m < n && (!zr || R <= (uint64_t)kMaxOnePass || R > (uint64_t)kMaxSlicesOther)) return 0;
    // (below 2^31: a tile's width in the filter's index space exceeds its entries)
    if (R <= (uint64_t)kMaxOnePass && m < (1ull << 31)) return m >= (1ull << 20) ? 1 : 0;
    if (!zr && R <= (uint64_t)kMaxSlicesOther && 2 * m < 5 * n) return 0;
    return m >= (1ull << 24) ? 2 : 0;
}

// Where everything lies in the regrouped hooks' scratch block (byte offsets).
struct TiledLayout {
    int R;
    uint64_t nch1, nch2;
    uint64_t t1w, t1h, seg, cnt1, tsum, pre1, base2, cbase, desc;   // level 1 (two passes, buckets)
    uint64_t w, h, run2, wcnt;                                      // the filter's tiles
    uint64_t wgoff, wgcnt, ipref;                                   // the survivors' regions
    uint64_t bits, p32;                                             // plain whole solves
    uint64_t total;
};

// passes: 0 = no tiles; 1, 2 = the filter's; 3 = the plain bucketed hook.
static TiledLayout tiled_layout(uint64_t n, uint64_t m, int passes, bool bits, bool p32) {
    TiledLayout l{};
    l.R = slices(n);
    const uint64_t R = (uint64_t)l.R;
    l.nch1 = (m + kC1 - 1) / kC1;
    l.nch2 = passes == 1 ? l.nch1 : m / kC2 + R + 1;
    const uint64_t cap = l.nch1 * kC1;
    const uint64_t ntile = (l.nch1 + kScanTile - 1) / kScanTile;
    uint64_t at = 0;
    auto take = [&](uint64_t bytes) {
        const uint64_t o = at;
        at += (bytes + 255) & ~255ull;
        return o;
    };
    if (passes >= 2) {
        l.t1w = take(4 * cap);
        l.t1h = take(2 * cap);
        l.seg = take(2 * l.nch1 * R);
        l.cnt1 = take(4 * l.nch1 * R);
        l.tsum = take(4 * ntile * R);
        l.pre1 = take(4 * (l.nch1 + 1) * R);
        l.base2 = take(8 * (R + 1));
        l.cbase = take(4 * (R + 1));
        l.desc = take(32 * l.nch2);
    }
    if (passes == 1 || passes == 2) {
        l.w = take(4 * cap);
        l.h = take(cap);
        l.run2 = take(2 * l.nch2 * ((passes == 1 ? R * R : R) + 1));
    }
    if (passes == 1) l.wcnt = take(4 * R * R * ((l.nch1 + kWin3 - 1) / kWin3));
    if (passes == 2) {
        const uint64_t kb = (uint64_t)b_per_block(l.R), nwg = R * ((R + kb - 1) / kb);
        l.wgoff = take(8 * (nwg + 1));
        l.wgcnt = take(4 * nwg);
        l.ipref = take(4 * (nwg + 1));
    }
    if (bits) l.bits = take(4 * ((n + 31) / 32));
    if (p32) l.p32 = take(4 * n);
    l.total = at;
    return l;
}

uint64_t filter_scratch_bytes(uint64_t n, uint64_t m, int passes, bool bits, bool p32) {
    return tiled_layout(n, m, passes, bits, p32).total;
}
uint64_t bucket_scratch_bytes(uint64_t n, uint64_t m) {
    return tiled_layout(n, m, 3, false, false).total;
}

static int grow(Slot* s, uint64_t bytes, hipStream_t stream, const char** why) {
    if (s->tiled.cap < bytes) {
        if (s->no_grow) {
            *why = "regrouped-hook scratch exceeds the fixed scratch";
            return CC_ENOMEM;
        }
        if (stream_capturing(stream)) {          // growing waits for the stream
            *why = "regrouped-hook scratch cannot grow under capture";
            return kScratchCapture;
        }
        *why = "tiled hook scratch allocation failed";
        CCM_HIP(hipStreamSynchronize(stream));
        int rc = slot_outgrow(s, s->tiled.buf, &s->tiled.captured);
        if (rc) return rc;
        s->tiled.buf = nullptr;
        s->tiled.cap = 0;
        if (hipMalloc(&s->tiled.buf, bytes) != hipSuccess) {
            (void)hipGetLastError();
            s->tiled.buf = nullptr;
            return CC_ENOMEM;
        }
        s->tiled.cap = bytes;
    } else if (!s->no_grow) {
        note_capture(&s->tiled.captured, stream);
    }
    return CC_OK;
}

int filter_scratch(Slot* s, uint64_t n, uint64_t m, int passes, bool bits, bool p32,
                   hipStream_t stream, FilterScratch* out) {
    const TiledLayout l = tiled_layout(n, m, passes, bits, p32);
    int rc = grow(s, l.total, stream, &out->why);
    if (rc) return rc;
    out->buf = s->tiled.buf;
    out->bits = bits ? reinterpret_cast<uint32_t*>(s->tiled.buf + l.bits) : nullptr;
    out->p32 = p32 ? reinterpret_cast<uint32_t*>(s->tiled.buf + l.p32) : nullptr;
    return CC_OK;
}

void tiled_free(TiledScratch* t) {
    if (t->buf) (void)hipFree(t->buf);
    *t = TiledScratch{};
}

// Steps 1-3 and the level-2 chunk descriptors on a COO list.
static int level1(const TiledLayout& l, char* q, uint64_t n, uint64_t m, EdgeList E, DevState* st,
                  bool sym, Gate gate, hipStream_t stream) {
    auto* t1w = reinterpret_cast<uint32_t*>(q + l.t1w);
    auto* t1h = reinterpret_cast<uint16_t*>(q + l.t1h);
    auto* seg = reinterpret_cast<uint16_t*>(q + l.seg);
    auto* cnt1 = reinterpret_cast<uint32_t*>(q + l.cnt1);
    auto* tsum = reinterpret_cast<uint32_t*>(q + l.tsum);
    auto* pre1 = reinterpret_cast<uint32_t*>(q + l.pre1);
    auto* base2 = reinterpret_cast<uint64_t*>(q + l.base2);
    auto* cbase = reinterpret_cast<uint32_t*>(q + l.cbase);
    auto* desc = reinterpret_cast<uint32_t*>(q + l.desc);
    const uint32_t ntile = (uint32_t)((l.nch1 + kScanTile - 1) / kScanTile);
    const uint32_t R = (uint32_t)l.R;
    const uint32_t g1 = (uint32_t)l.nch1;
    int rc;
    // every kernel below reads tables the previous one wrote: coherence points between
    if ((rc = cohere(stream))) return rc;
    with_coo(E, [&](auto e) {
        auto part = l.R <= kFewSlices ? &k_t1_part<kFewSlices, decltype(e)> : &k_t1_part<kMaxSlices, decltype(e)>;
        part<<<g1, kPartBlock, 0, stream>>>(e, m, (uint32_t)n, l.R, l.nch1, t1w, t1h, seg, cnt1, st,
                                            sym ? 1u : 0u, gate);
    });
    if ((rc = cohere(stream))) return rc;
    k_t1_tsum<<<R * ntile, kScanBlock, 0, stream>>>(cnt1, l.nch1, ntile, tsum, gate);
    if ((rc = cohere(stream))) return rc;
    k_t1_scan<<<R * ntile, kScanBlock, 0, stream>>>(cnt1, l.nch1, ntile, tsum, pre1, gate);
    if ((rc = cohere(stream))) return rc;
    k_t1_bases<<<1, kMaxSlices, 0, stream>>>(pre1, l.nch1, l.R, base2, cbase, gate);
    if ((rc = cohere(stream))) return rc;
    const uint64_t pairs = (uint64_t)R * l.nch1;
    k_t2_bounds<<<(uint32_t)((pairs + 255) / 256), 256, 0, stream>>>(pre1, l.nch1, l.R, cbase, base2,
                                                                    desc, gate);
    return cohere(stream);
}

template <bool ZR>
static void hook_level1(const TiledLayout& l, char* q, uint32_t* P, DevState* st, Gate gate,
                        hipStream_t stream) {
    const bool loop = gate.word && l.nch2 > 2 * kShutGrid;
    auto hook = loop ? &k_t2_hookplain<ZR, true> : &k_t2_hookplain<ZR, false>;
    hook<<<loop ? kShutGrid : (uint32_t)l.nch2, kPartBlock, 0, stream>>>(
        reinterpret_cast<uint32_t*>(q + l.t1w), reinterpret_cast<uint16_t*>(q + l.t1h),
        reinterpret_cast<uint16_t*>(q + l.seg), reinterpret_cast<uint32_t*>(q + l.pre1), l.nch1, l.R,
        reinterpret_cast<uint32_t*>(q + l.cbase), reinterpret_cast<uint32_t*>(q + l.desc), P, st, gate);
}

int run_hook_buckets(Slot* s, uint64_t n, uint64_t m, const uint32_t* edges, uint32_t* P, bool sym,
                     hipStream_t stream) {
    const TiledLayout l = tiled_layout(n, m, 3, false, false);
    const char* why = "";
    int rc = grow(s, l.total, stream, &why);
    if (rc == CC_ENOMEM) return fail(rc, why);
    if (rc) return rc;
    char* q = s->tiled.buf;
    if ((rc = level1(l, q, n, m, EdgeList{edges, false}, s->st, sym, Gate{}, stream))) return rc;
    // the plain path hooks the level-2 chunks as they are gathered
    hook_level1<false>(l, q, P, s->st, Gate{}, stream);
    CCM_HIP(hipGetLastError());
    return CC_OK;
}

// Steps 5-6 on the level-2 buffers: survivors to (sw, sh), then hooked.
static int filter_runs(int R, uint64_t m, uint64_t nch2, L2Buf tmp2, uint16_t* run2, uint64_t* base2,
                       uint32_t* cbase, uint32_t* sw, uint16_t* sh, uint64_t* wgoff,
                       uint32_t* wgcnt, uint32_t* ipref, uint32_t* P, uint32_t* zbits,
                       uint64_t words, DevState* st, Gate again, Gate gate, hipStream_t stream) {
    const uint32_t nbg = (uint32_t)((R + b_per_block(R) - 1) / b_per_block(R));
    const uint32_t nwg = (uint32_t)R * nbg;
    int rc;
    k_t3_regions<<<nwg, 256, 0, stream>>>(run2, nch2, R, cbase, wgcnt, gate);
    if ((rc = cohere(stream))) return rc;
    k_t3_offsets<<<(uint32_t)R, 64, 0, stream>>>(wgcnt, R, base2, wgoff, gate);
    if ((rc = cohere(stream))) return rc;
    auto filter = R > kFewSlices                    ? &k_t3_filter<kManyRuns>
                  : m < 2ull * kFlushEntries * nwg ? &k_t3_filter<kMixedRuns>
                                                   : &k_t3_filter<kFullRuns>;
    filter<<<nwg, kHook3Block, 0, stream>>>(tmp2, run2, nch2, R, nullptr, base2, cbase, zbits, words, P,
                                            sw, sh, wgoff, wgcnt, st, gate);
    if ((rc = cohere(stream))) return rc;
    k_t4_scan<<<1, kPackBlock, 0, stream>>>(wgcnt, nwg, ipref, gate);
    if ((rc = cohere(stream))) return rc;
    k_t4_hook<<<kHook4Grid, kHook4Block, 0, stream>>>(sw, sh, wgoff, wgcnt, ipref, nwg, (int)nbg, P,
                                                      zbits, st, again, gate);
    CCM_HIP(hipGetLastError());
    return CC_OK;
}

int run_filter(Slot* s, uint64_t n, uint64_t m, EdgeList E, uint32_t* P, uint32_t* zbits, int passes,
               bool bits, bool p32, bool sym, Gate gate, int other, hipStream_t stream) {
    const TiledLayout l = tiled_layout(n, m, passes, bits, p32);
    const Gate part = other != kNoOther ? Gate{} : gate, off{gate.word, !gate.want};
    if (s->tiled.cap < l.total) return fail(CC_EDEVICE, "regrouped-hook scratch too small (a bug)");
    char* q = s->tiled.buf;
    const L2Buf tmp2{reinterpret_cast<uint32_t*>(q + l.w), reinterpret_cast<uint8_t*>(q + l.h)};
    auto* run2 = reinterpret_cast<uint16_t*>(q + l.run2);
    const uint64_t words = (n + 31) / 32;
    int rc;
    if (passes == 1) {
        const uint32_t g = (uint32_t)l.nch1;
        with_entries(E, [&](auto e) {
            k_tile_part<<<g, kPartBlock, 0, stream>>>(e, m, (uint32_t)n, l.R, l.nch1, tmp2, run2, s->st,
                                                      sym ? 1u : 0u, part);
        });
        if ((rc = cohere(stream))) return rc;
        const uint32_t nwin = (uint32_t)((l.nch1 + kWin3 - 1) / kWin3);
        auto* wcnt = reinterpret_cast<uint32_t*>(q + l.wcnt);
        k_tile_count<<<(uint32_t)(l.R * l.R) * nwin, 256, 0, stream>>>(run2, l.nch1, nwin, wcnt, part);
        if ((rc = cohere(stream))) return rc;
        // one workgroup per CU is resident; no more than its copies are worth
        const uint32_t wgs = (uint32_t)std::max<uint64_t>(
            1, std::min<uint64_t>(m >> 13, (uint64_t)device_cu_count(s->device)));
        k_t3_filter<kMarkTiles><<<wgs, kHook3Block, 0, stream>>>(
            tmp2, run2, l.nch1, l.R, wcnt, nullptr, nullptr, zbits, words, P, nullptr, nullptr, nullptr,
            nullptr, s->st, gate);
        if ((rc = cohere(stream))) return rc;
        k_t3_filter<kFullTiles><<<wgs, kHook3Block, 0, stream>>>(
            tmp2, run2, l.nch1, l.R, wcnt, nullptr, nullptr, zbits, words, P, nullptr, nullptr, nullptr,
            nullptr, s->st, gate);
        if (other != kNoOther) {
            const uint64_t all = m + (uint64_t)(l.R * l.R) * kVisit;
            const uint64_t part = std::max<uint64_t>(kHookPart, all / kHookParts);
            const uint32_t gh = (uint32_t)((all / part + kXcds) / kXcds * kXcds);
            auto hook = other == kOtherZr ? &k_tile_hook<true> : &k_tile_hook<false>;
            hook<<<gh, kHook3Block, 0, stream>>>(tmp2, run2, l.nch1, l.R, wcnt, P, s->st, (uint32_t)part, off);
        }
        CCM_HIP(hipGetLastError());
        return CC_OK;
    }
    if ((rc = level1(l, q, n, m, E, s->st, sym, part, stream))) return rc;
    // the other hook reads the level-1 buckets, whose room the filter's survivors take
    // (only one of the two runs)
    if (other == kOtherZr) hook_level1<true>(l, q, P, s->st, off, stream);
    else if (other == kOther) hook_level1<false>(l, q, P, s->st, off, stream);
    auto* cbase = reinterpret_cast<uint32_t*>(q + l.cbase);
    auto* base2 = reinterpret_cast<uint64_t*>(q + l.base2);
    auto part2 = l.R <= kFewSlices ? &k_t2_part<kFewSlices> : &k_t2_part<kMaxSlices>;
    part2<<<(uint32_t)l.nch2, kPartBlock, 0, stream>>>(
        reinterpret_cast<uint32_t*>(q + l.t1w), reinterpret_cast<uint16_t*>(q + l.t1h),
        reinterpret_cast<uint16_t*>(q + l.seg), reinterpret_cast<uint32_t*>(q + l.pre1), l.nch1, l.R,
        cbase, reinterpret_cast<uint32_t*>(q + l.desc), tmp2, run2, l.nch2, gate);
    if ((rc = cohere(stream))) return rc;
    // the survivor regions live in the level-1 buffers, free once the level-2
    // partition has read them (positions [base2[a], base2[a+1]) for slice a)
    return filter_runs(l.R, m, l.nch2, tmp2, run2, base2, cbase, reinterpret_cast<uint32_t*>(q + l.t1w),
                       reinterpret_cast<uint16_t*>(q + l.t1h), reinterpret_cast<uint64_t*>(q + l.wgoff),
                       reinterpret_cast<uint32_t*>(q + l.wgcnt), reinterpret_cast<uint32_t*>(q + l.ipref),
                       P, zbits, words, s->st, Gate{&s->st->giant, 1u}, gate, stream);
}

// The regrouped zero-root hook on CSR input (steps 4-5 on adj's own buckets).
int run_hook_tiled_csr(Slot* s, uint64_t n, uint64_t m, const uint64_t* off, const uint32_t* adj,
                       uint32_t* P, bool retest, hipStream_t stream, bool sym) {
    const int R = slices(n);
    const uint64_t nch2 = m / kC2 + (uint64_t)R + 1;
    auto al = [](uint64_t x) { return (x + 255) & ~255ull; };
    const uint64_t b_tmp2 = al(4 * m) + al(m);
    const uint64_t b_base2 = al(8 * (R + 1)), b_cbase = al(4 * (R + 1));
    const uint64_t b_cfirst = al(4 * nch2), b_run2 = al(2 * nch2 * (R + 1));
    const uint64_t b_sw = al(4 * m), b_sh = al(2 * m);
    const uint64_t kb = (uint64_t)b_per_block(R), nwg = (uint64_t)R * ((R + kb - 1) / kb);
    const uint64_t b_wgoff = al(8 * (nwg + 1)), b_wgcnt = al(4 * nwg), b_ipref = al(4 * (nwg + 1));
    const char* why = "";
    int rc = grow(s, b_sw + b_sh + b_tmp2 + b_base2 + b_cbase + b_cfirst + b_run2 + b_wgoff + b_wgcnt +
                         b_ipref, stream, &why);
    if (rc == CC_ENOMEM || rc == kScratchCapture) return fail(CC_ENOMEM, why);
    if (rc) return rc;
    char* q = s->tiled.buf;
    uint32_t* sw = reinterpret_cast<uint32_t*>(q); q += b_sw;
    uint16_t* sh = reinterpret_cast<uint16_t*>(q); q += b_sh;
    const L2Buf tmp2{reinterpret_cast<uint32_t*>(q), reinterpret_cast<uint8_t*>(q + al(4 * m))};
    q += b_tmp2;
    uint64_t* base2 = reinterpret_cast<uint64_t*>(q); q += b_base2;
    uint32_t* cbase = reinterpret_cast<uint32_t*>(q); q += b_cbase;
    uint32_t* cfirst = reinterpret_cast<uint32_t*>(q); q += b_cfirst;
    uint16_t* run2 = reinterpret_cast<uint16_t*>(q); q += b_run2;
    uint64_t* wgoff = reinterpret_cast<uint64_t*>(q); q += b_wgoff;
    uint32_t* wgcnt = reinterpret_cast<uint32_t*>(q); q += b_wgcnt;
    uint32_t* ipref = reinterpret_cast<uint32_t*>(q);
    if ((rc = cohere(stream))) return rc;
    k_c_bases<<<1, 256, 0, stream>>>(off, n, m, R, base2, cbase);
    if ((rc = cohere(stream))) return rc;
    const uint64_t gv = std::min<uint64_t>((n + 255) / 256, 8192);
    k_c_first<<<(uint32_t)gv, 256, 0, stream>>>(off, n, base2, cbase, cfirst);
    if ((rc = cohere(stream))) return rc;
    k_t2_csr<<<(uint32_t)nch2, kPartBlock, 0, stream>>>(off, adj, n, R, base2, cbase, cfirst, tmp2,
                                                       run2, nch2, s->st, sym ? 1u : 0u);
    if ((rc = cohere(stream))) return rc;
    return filter_runs(R, m, nch2, tmp2, run2, base2, cbase, sw, sh, wgoff, wgcnt, ipref, P, s->zbits,
                       (n + 31) / 32, s->st, retest ? Gate{} : Gate{&s->st->zroot, kEmpty}, Gate{}, stream);
}

}  // namespace ccm

// cc_internal.h — declarations shared by the library's own translation units.
// Not installed; the public interface is include/cc.h.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>

#include <map>
#include <mutex>
#include <string>
#include <vector>

#include "cc.h"

namespace ccm {

// Device-resident state of one solve slot (a context has one; the server one per
// slot). Lives in device memory; kernels read and update it, the host reads it
// only through explicit copies.
struct DevState {
    uint32_t status;    // kStatus* bits, reported and cleared by slot_sync
    uint32_t zroot;     // the root whose component the bitmap describes: the zero root,
                        // or the giant component's root of a plain whole solve
    uint32_t zpub;      // the zero root chosen by the latest cc_zroot (cc_get_zroot, cc_canon)
    uint32_t mpub;      // smallest member of zpub's component (zero-root compress; cc_canon)
    uint64_t zsel;      // packed argmax (count << 32) | (0xFFFFFFFF - id); 0 = none
    uint64_t log_count; // messages of a drained update log (cc_hook_log_drain)
    uint32_t giant1;    // a small sample shows a giant component
    uint32_t giant;     // the filter's kernels run (else the direct hook's)
    uint32_t rebuild;   // the bitmap is to be written after a sample without it
    uint32_t flat;      // the forest is to be flattened after the samples
    uint64_t pad2[2];
};
static_assert(sizeof(DevState) == 64, "DevState is one 64-byte block");

constexpr uint32_t kStatusRange = 1u;
constexpr uint32_t kStatusInternal = 2u;   // a scratch bound check failed (a bug)
constexpr uint32_t kStatusLogFull = 4u;    // an update log ran out of capacity
constexpr uint32_t kStatusBadOffsets = 8u; // CSR offsets not a valid row index
constexpr uint32_t kEmpty = 0xFFFFFFFFu;

// Path splitting in the direct hooks' walks pays only where the parent array
// outgrows one XCD's L2 (4 MB): below that every walk step is an L2 hit and the
// splitting stores, which go to memory, cost more than the steps they save
// (ER n = 2^16, 2^20 entries: 0.82 ms with splitting, 0.14 ms without; R-MAT
// n = 2^22 direct hook: 4.9 ms with, 7.2 ms without). CC_F_NO_SPLIT turns it
// off everywhere.
constexpr uint64_t kSplitMinBytes = 4ull << 20;
__host__ __device__ inline bool split_walks(uint32_t flags, uint64_t n, uint64_t entry_bytes = 4) {
    return !(flags & CC_F_NO_SPLIT) && n * entry_bytes > kSplitMinBytes;
}
// Hooking in two parts: without path splitting the walks of one pass grow long
// while the forest forms (link by index makes chains that nothing shortens),
// and every later entry walks them. Where that applies to enough entries per
// vertex, the first quarter of the entries is hooked, the forest pointer-jumped
// (a flat forest with the same components, from which Algorithm 1 continues)
// and the rest hooked over it.
__host__ __device__ inline bool hook_in_two_parts(uint64_t n, uint64_t m, bool split) {
    return !split && m >= (1ull << 18) && m >= 4 * n;
}
constexpr uint32_t kGridCap = 256 * 32;   // blocks of a grid-stride launch over n

// One graph of a batched launch: where its entries and labels live.
struct GraphDesc {
    const int32_t* edges;   // 2*m int32, local IDs
    int32_t* L;             // n int32 labels (also the parent array when it is not in LDS)
    int32_t* status;        // where the graph's status code goes
    uint32_t n;
    uint32_t pad;
    int64_t m;
};
static_assert(sizeof(GraphDesc) == 40, "GraphDesc layout");

// Scratch of the batched path: the work tickets, the work lists, the chunk
// tables of the whole-device graphs and the descriptors, uploaded in one copy
// per launch (layout in cc_batch.hip).
struct BatchScratch {
    char* dev = nullptr;       // device
    char* host = nullptr;      // pinned host staging of the same layout
    uint64_t cap = 0;          // graphs
};

// A batch schedule (cc_batch_sched): which graphs run on the whole device, which
// on one wavefront, the rest on one workgroup each.
typedef cc_batch_sched BatchSched;

// Scratch of the regrouped hooks (one block, grown on demand).
struct TiledScratch {
    char* buf = nullptr;
    uint64_t cap = 0;
    bool captured = false;     // see Slot::kept
};

// Scratch owned by one slot.
struct Slot {
    int device = 0;
    DevState* st = nullptr;        // device
    uint32_t* hkeys = nullptr;     // device, zroot hash table keys   [table]
    uint32_t* hcounts = nullptr;   // device, zroot hash table counts [table]
    uint32_t* bmin = nullptr;      // device, per-block minima of compress [kGridCap]
    uint32_t* xs = nullptr;        // device, export counts and offsets [4 * kGridCap + 2]
    uint32_t table = 0;            // power of two >= 4 * samples
    uint32_t samples = 0;          // K
    uint32_t* deg = nullptr;       // device, exact-degree counts (grown on demand)
    uint64_t deg_cap = 0;
    bool deg_captured = false;
    uint32_t* host_status = nullptr;  // pinned host block of 64 bytes (status word, read-backs)
    BatchScratch batch;
    // Zero-root membership bitmap: bit x set => x is in the zero root's tree.
    uint32_t* zbits = nullptr;     // device, ceil(n/32) words (grown on demand)
    uint64_t zbits_cap = 0;        // words
    bool zbits_captured = false;
    // Buffers that a larger solve outgrew after work captured into a graph had used
    // them: a replay still reads and writes them, so they are freed with the slot.
    // (A buffer that no capture has used is freed when it is outgrown.)
    std::vector<void*> kept;
    // Bitmap of a plain whole solve's giant component (cc_filter.hip), for arrays
    // of at most lds_bits_max_n() vertices.
    uint32_t* gbits = nullptr;
    // Host-side order of the steps: a CC_F_ZROOT hook needs cc_zroot after the
    // latest cc_init on the same n (the bitmap describes that solve).
    uint64_t cur_n = 0;
    bool zr_ready = false;
    TiledScratch tiled;
    uint32_t* csr_tiles = nullptr; // device, first row of every CSR tile (grown on demand)
    uint64_t csr_tiles_cap = 0;
    // Nothing is grown: a solve that would need a larger buffer than the slot
    // holds fails with CC_ENOMEM (a server's lent block, the allocation-free
    // entry point).
    bool no_grow = false;
    // The regrouped hooks (buffers per entry) are not taken (the allocation-free
    // entry point, whose fixed scratch cannot hold them).
    bool no_tiled = false;
};

int slot_create(Slot* s, int device, uint32_t samples);
void slot_destroy(Slot* s);
// Whether work queued on `stream` is being captured (also where that cannot be told).
bool stream_capturing(hipStream_t stream);
// A grown buffer is about to be used on `stream`.
inline void note_capture(bool* captured, hipStream_t stream) {
    if (!*captured) *captured = stream_capturing(stream);
}
// A buffer of the slot makes room for a larger one: freed, or kept (Slot::kept).
int slot_outgrow(Slot* s, void* buf, bool* captured);

// A graph's rows as entries (u, adj[i]), off[u] <= i < off[u + 1]; tstart[t] is the
// row of position t * kCsrTile.
constexpr int kCsrTile = 1024;
struct CsrList {
    const uint64_t* off;
    const uint32_t* adj;
    const uint32_t* tstart;
    uint64_t ntiles;
    uint32_t n;
};
// The entries of a solve: a COO list of 2m IDs of 32 bits, or of 64 (wide), or a CSR
// graph (csr not NULL).
struct EdgeList {
    const void* p;
    bool wide;
    const CsrList* csr = nullptr;
};
// f(entries) with the type that load_entry takes. Only the zero-root filters come
// with CSR graphs (with_entries), the others with COO lists.
template <class F>
auto with_coo(const EdgeList& E, const F& f) {
    return E.wide ? f((const uint64_t*)E.p) : f((const uint32_t*)E.p);
}
template <class F>
auto with_entries(const EdgeList& E, const F& f) {
    return E.csr ? f(*E.csr) : with_coo(E, f);
}

// Which launches of a solve run is in part decided on the device: a kernel given
// a gate leaves at once unless *word == want (word NULL: always runs).
struct Gate {
    const uint32_t* word;
    uint32_t want;
};

// Enqueue steps (arguments already validated by the caller).
int run_init(Slot* s, uint64_t n, uint32_t* P, hipStream_t stream);
int run_zroot(Slot* s, uint64_t n, uint64_t m, const uint32_t* edges, uint32_t flags,
              uint32_t hint, hipStream_t stream);
int run_push(Slot* s, uint64_t n, uint64_t m, const uint32_t* edges, uint32_t* P,
             hipStream_t stream);
// How the direct zero-root hooks settle an entry with exactly one endpoint in
// the membership bitmap. Linking the other endpoint's tree under z costs a walk,
// a coherent read and a CAS on P, but every vertex of that tree then walks to z
// and is marked when an entry reaches it, so the bitmap grows faster; marking
// the endpoint alone (compress passes the mark on to its tree) touches no P.
// Once P outgrows the MALL (256 MB) each of those P accesses goes to HBM and
// marking wins: R-MAT-30 1/16 share (4 GiB P), 46.9 -> 40.8 ms (37.6 with the
// second endpoint's word read coherently, so that its mark is one atomic);
// R-MAT-26 + extras direct, 21.7 -> 21.1 ms. Below it linking wins: R-MAT-22 direct 2.2
// against 2.8 ms, R-MAT-24 5.5 against 5.8, R-MAT-26 1/16 share 2.8 against
// 3.2. kHookLinkZ, an internal flag of run_hook (beside the public CC_F_*,
// never accepted from a caller), asks for linking at any size: the regrouped
// hook's warm-up seeds its filter's bitmap (10.1 against 10.4 ms on R-MAT-26 +
// extras).
constexpr uint32_t kHookLinkZ = 0x80000000u;
constexpr uint64_t kMallBytes = 256ull << 20;
inline bool hook_links_z(uint32_t flags, uint64_t n) {
    return (flags & kHookLinkZ) || n * 4 <= kMallBytes;
}
int run_hook(Slot* s, uint64_t n, uint64_t m, const uint32_t* edges, uint32_t* P,
             uint32_t flags, hipStream_t stream);
// final_labels (zero root): z's component ends labelled with its smallest ID
// directly, as run_canon would make it; otherwise it keeps the label z.
int run_compress(Slot* s, uint64_t n, uint32_t* P, uint32_t flags, hipStream_t stream,
                 bool final_labels = false);
// Plain-path hook that appends its links to a caller-owned log (cc_hook_log).
int run_hook_log(Slot* s, uint64_t n, uint64_t m, const uint32_t* edges, uint32_t* P,
                 uint32_t flags, uint32_t* log, uint64_t log_cap, uint64_t* log_count,
                 hipStream_t stream);
// The log counter of the slot's DevState set to 0 (a kernel: capturable).
int log_count_reset(Slot* s, hipStream_t stream);
// The counter's value written to a pinned host word (a kernel, ordered on stream).
int log_count_snap(Slot* s, uint64_t* host_word, hipStream_t stream);
int run_canon(Slot* s, uint64_t n, uint32_t* L, hipStream_t stream);
int run_hook_ids(Slot* s, uint64_t n, uint64_t count, const uint32_t* ids, uint32_t target,
                 uint32_t* P, uint32_t flags, hipStream_t stream);

// Exchange (cc_exchange.hip): synchronous export of a share's parent array.
int run_export(Slot* s, uint64_t n, const uint32_t* P, uint32_t zroot, uint32_t* pairs,
               uint64_t pairs_cap, uint32_t* zero_ids, uint64_t zero_cap, uint64_t* n_pairs,
               uint64_t* n_zero, hipStream_t stream);
// Compact IDs of the exchange (cc_exchange.hip); k in 1..4, buffers 4-byte aligned.
int run_pack_ids(Slot* s, uint64_t count, const uint32_t* ids, uint32_t k, uint8_t* out,
                 hipStream_t stream);
int run_unpack_ids(Slot* s, uint64_t count, const uint8_t* in, uint32_t k, uint32_t* ids,
                   hipStream_t stream);
int run_giant(Slot* s, uint64_t n, uint64_t m, EdgeList E, uint32_t* P, uint32_t* bits, int passes,
              bool p32, uint32_t flags, hipStream_t stream);
bool lds_eligible(uint64_t n, uint64_t m);
int run_solve(Slot* s, uint64_t n, uint64_t m, const uint32_t* edges, uint32_t* L,
              uint32_t flags, uint32_t hint, hipStream_t stream);
// Whole path on CSR input (m = off[n], read by the caller).
int run_solve_csr(Slot* s, uint64_t n, uint64_t m, const uint64_t* off, const uint32_t* adj,
                  uint32_t* L, uint32_t flags, uint32_t hint, uint32_t maxdeg, hipStream_t stream);
// What run_solve_csr needs of the offsets, waited for: m = off[n], and with CC_F_ZROOT
// (no hint) the longest row, whose vertex is left in DevState::zsel; else maxdeg 0.
int run_csr_head(Slot* s, uint64_t n, const uint64_t* off, uint32_t flags, hipStream_t stream, uint64_t* m,
                 uint32_t* maxdeg);
// Plain path with 64-bit IDs (cc_wide.hip).
int run_solve_w(Slot* s, uint64_t n, uint64_t m, const uint64_t* edges, uint64_t* L,
                uint32_t flags, hipStream_t stream);
// Size the zero-root membership bitmap for n and clear it (only z set).
int zbits_reset(Slot* s, uint64_t n, hipStream_t stream);
// Copy the status word to the host, clear it, wait for the stream; CC_OK,
// CC_ERANGE, CC_ENOMEM (a full update log) or CC_EINVAL (bad CSR offsets).
int slot_sync(Slot* s, hipStream_t stream);

// Regrouped hooks (cc_tiled.hip). The plain hook of first-endpoint buckets
// applies to (n, m); with zr, the sizes at which the zero-root hook has always
// been regrouped (it fails rather than run direct when its scratch cannot grow).
bool tiled_eligible(uint64_t n, uint64_t m, bool zr);
// The filter over (first slice, second slice) tiles, both membership tests in
// LDS: 0 = not for these sizes, else its partition passes (1 or 2).
int filter_passes(uint64_t n, uint64_t m, bool zr);
uint64_t filter_scratch_bytes(uint64_t n, uint64_t m, int passes, bool bits, bool p32);
uint64_t bucket_scratch_bytes(uint64_t n, uint64_t m);
// Size the slot's scratch for the filter (passes 0: only the arrays asked for):
// with a bitmap of its own (bits), with a 32-bit parent array (p32). Not CC_OK
// where it cannot grow now: kScratchCapture under capture, else CC_ENOMEM. Most
// callers go on by another hook then, so the failure's text is left to the one that
// does not: `why`.
constexpr int kScratchCapture = 1;
struct FilterScratch {
    char* buf;
    uint32_t* bits;
    uint32_t* p32;
    const char* why;
};
int filter_scratch(Slot* s, uint64_t n, uint64_t m, int passes, bool bits, bool p32,
                   hipStream_t stream, FilterScratch* out);
// The filter on scratch sized by filter_scratch with the same arguments: every
// entry tested against zbits, the rest hooked in P (key order of DevState::zroot).
// other: what is to happen where the gate is shut, without a bitmap. kOther, kOtherZr:
// the regrouped entries are hooked in P (key = ID, or with the zero root's keys).
enum OtherHook { kNoOther, kOther, kOtherZr };
int run_filter(Slot* s, uint64_t n, uint64_t m, EdgeList E, uint32_t* P, uint32_t* zbits, int passes,
               bool bits, bool p32, bool sym, Gate gate, int other, hipStream_t stream);
// The plain hook (key = ID) over first-endpoint buckets. kScratchCapture (nothing
// queued) where its scratch would have to grow under capture.
int run_hook_buckets(Slot* s, uint64_t n, uint64_t m, const uint32_t* edges, uint32_t* P, bool sym,
                     hipStream_t stream);
// Device bytes a whole-path solve (run_solve) grows in its slot for these
// arguments: the bitmap, exact degrees, the regrouped hooks' buffers. lean: the
// least it can do with (the filter on a plain solve, and below the sizes of
// tiled_eligible, is left out).
uint64_t solve_scratch_bytes(uint64_t n, uint64_t m, uint32_t flags, bool lean);
// Lend a block of device memory of `bytes` (solve_scratch_bytes of the same
// arguments, lean or not) to a slot for one run_solve: its grown buffers point
// into the block and nothing is allocated; slot_return_scratch gives the slot
// its own buffers back.
struct LentScratch {
    uint32_t* zbits; uint64_t zbits_cap;
    uint32_t* deg; uint64_t deg_cap;
    TiledScratch tiled;
};
void slot_lend_scratch(Slot* s, char* block, uint64_t bytes, uint64_t n, uint32_t flags,
                       LentScratch* saved);
void slot_return_scratch(Slot* s, const LentScratch* saved);
void tiled_free(TiledScratch* t);
// The same on CSR input, where the rows already are the first-endpoint buckets. retest:
// the survivors' bits are tested once more before they are hooked.
int run_hook_tiled_csr(Slot* s, uint64_t n, uint64_t m, const uint64_t* off, const uint32_t* adj,
                       uint32_t* P, bool retest, hipStream_t stream, bool sym = false);

// Hooks that test a bitmap in LDS (cc_filter.hip).
// Largest n whose whole bitmap fits a workgroup's LDS.
uint64_t lds_bits_max_n();
// The bitmap of st->zroot's component, from a flat forest; kBitsPick finds the
// root first (the one most often seen above sampled endpoints). sample: 1 records
// st->giant1 and st->giant (after the first sample), 2 st->giant, 0 neither.
enum BitsMode { kBitsPick, kBitsPlain, kBitsZr };
int run_giant_bits(uint64_t n, uint64_t m, EdgeList E, const uint32_t* P, uint32_t* zbits,
                   DevState* st, int mode, int sample, Gate gate, hipStream_t stream);
// Whether the forest shows a giant component (the zero root's, by P and zbits,
// with zr): st->giant. Stages 1 and 2 run where st->giant1 is 0; 0 and 1 set it too,
// 1 and 2 set st->rebuild. A plain solve's root: st->zroot.
int run_find_giant(uint64_t n, uint64_t m, EdgeList E, uint32_t* P, const uint32_t* zbits, DevState* st,
                   bool zr, int stage, hipStream_t stream);
// run_warm hooks every warm_stride-th run of kSampleRun entries.
constexpr int kSampleRun = 256;
uint64_t warm_stride(uint64_t m, uint64_t want);
// About `want` entries hooked in P (no bitmap), spread evenly over the list.
int run_warm(uint64_t n, uint64_t m, EdgeList E, uint32_t* P, DevState* st, bool zr, bool sym,
             uint64_t want, Gate gate, hipStream_t stream);
// Every entry tested against the whole bitmap in LDS, the rest hooked in P. Rows without
// a giant component (st->giant) are left alone.
int run_hook_lds(uint64_t n, uint64_t m, EdgeList E, uint32_t* P, uint32_t* zbits, DevState* st,
                 bool split, bool sym, int device, hipStream_t stream);

// A whole solve of a small graph in one launch (cc_batch.hip). With CC_F_ZROOT the
// slot's bitmap holds n bits and its sample covers every entry.
bool small_eligible(uint64_t n, uint64_t m, uint32_t flags, uint32_t samples);
int run_solve_small(Slot* s, uint64_t n, uint64_t m, const uint32_t* edges, uint32_t* L,
                    uint32_t flags, uint32_t hint, hipStream_t stream);

// Batched path (cc_batch.hip).
// The schedule taken when nothing else is known about a batch.
BatchSched batch_default_sched();
// Largest n of a wave-role graph on this device (its LDS per wavefront).
int batch_wave_cap(int device, uint32_t* cap);
// Role of one graph under a schedule: kRoleTile, kRoleWave or kRoleMulti.
constexpr int kRoleTile = 0, kRoleWave = 1, kRoleMulti = 2;
int batch_role(const GraphDesc& d, const BatchSched& sc, uint32_t wave_cap);
// Enqueue one batch (the whole-device launches of its multi graphs, then the
// persistent launch) over G graphs described on the host.
int launch_batch(Slot* s, uint32_t G, const GraphDesc* descs, const BatchSched& sc,
                 hipStream_t stream);
// Size the slot's batch scratch for G graphs now (so later launches of at most
// G graphs allocate nothing).
int batch_reserve(Slot* s, uint32_t G);
// Offsets read back and checked, descriptors built (cc_batch's arguments).
int batch_descs(uint32_t G, const int64_t* vtx_off, const int64_t* edge_off, const int32_t* edges,
                int32_t* L, int32_t* status, hipStream_t stream, std::vector<GraphDesc>* out);
void batch_scratch_free(BatchScratch* b);
// A captured cc_batch (opaque handle): creation takes descriptors built by
// batch_descs and captures the upload and the launches into a graph.
int batch_graph_create(Slot* s, uint32_t G, const GraphDesc* descs, const BatchSched& sc,
                       void** out);
int batch_graph_launch(void* g, hipStream_t stream);
void batch_graph_destroy(void* g);

// Error reporting.
int fail(int code, const std::string& detail);
int hip_fail(hipError_t e, const char* what);
#define CCM_HIP(call)                                             \
    do {                                                          \
        hipError_t e_ = (call);                                   \
        if (e_ != hipSuccess) return ::ccm::hip_fail(e_, #call);  \
    } while (0)

int device_cu_count(int device);

// Coherence point between dependent kernels on one stream. Each XCD of the
// device has its own L2; a clean line cached on one XCD is not invalidated when
// another XCD (or an atomic performed beyond the L2) changes the data, and the
// kernel boundary alone has been observed not to drop such lines. This launch
// runs workgroups on every XCD, each writing back and invalidating its L2
// (agent-scope acquire-release fence), so the next kernel on the stream reads
// what the previous ones wrote.
int cohere(hipStream_t stream);

// Coherent (agent-scope) accesses to the small shared words of DevState.

__device__ __forceinline__ uint32_t ld_agent(const uint32_t* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t ld_agent64(const uint64_t* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_agent(uint32_t* p, uint32_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_agent64(uint64_t* p, uint64_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Race-testing builds (compiled with CCM_STRESS_DELAYS, a separate library):
// before each link CAS and each path-splitting store a wave pauses for 0 to 7
// short sleeps, drawn from the clock, the lane and `salt`. The pause widens the
// windows in which other waves change the same entries. The ordinary build
// compiles this to nothing.
__device__ __forceinline__ void stress_delay(uint32_t salt) {
#ifdef CCM_STRESS_DELAYS
    uint32_t h = (salt ^ (threadIdx.x * 0x9E3779B9u) ^ (uint32_t)clock64()) * 0x85EBCA6Bu;
    h ^= h >> 13;
    for (uint32_t i = 0; i < (h & 7u); ++i) __builtin_amdgcn_s_sleep(2);
#else
    (void)salt;
#endif
}

// Device, memory budget and zero-root sample count of a context.
int ctx_info(cc_ctx* ctx, int* device, uint64_t* budget, uint32_t* samples);

// Batch schedule tuner (cc_tune.hip): picks stored per device and shape, in
// memory and optionally in a file.
struct Tuner {
    std::mutex mu;
    std::string path;                          // the cache file ("" = none)
    std::map<std::string, BatchSched> picks;   // key: device | signature
    bool forced = false;
    BatchSched force{};
    bool autotune = false;
};
// Read the cache file (if any) into the tuner.
void tuner_open(Tuner* t, const char* path_opt, bool autotune);
// The schedule cc_batch takes for these graphs, and its source (CC_SCHED_*).
// With autotune and no stored pick, tunes first (runs the batch).
int tuner_choose(Tuner* t, Slot* s, uint32_t G, const GraphDesc* descs, hipStream_t stream,
                 BatchSched* out, uint32_t* source);
int tuner_tune(Tuner* t, Slot* s, uint32_t G, const GraphDesc* descs, uint32_t reps,
               hipStream_t stream, cc_batch_tune_result* out);
// Stored pick or default for these graphs (no forcing, no tuning): the server's.
BatchSched tuner_lookup(Tuner* t, int device, uint32_t G, const GraphDesc* descs);
Tuner* ctx_tuner(cc_ctx* ctx);

}  // namespace ccm

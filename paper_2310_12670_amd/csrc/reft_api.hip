// C-ABI host logic of libreft (see include/reft.h): the plan (host integer arithmetic and device
// tables), the bucket pipelines that pair the gather / scatter kernels with chunked
// hipMemcpyAsync transfers, and the XOR encode / decode entry points.
#include "../../include/reft.h"
#include "reft_rules.hpp"
#include "reft_internal.hpp"

#include <atomic>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <algorithm>
#include <exception>
#include <map>
#include <memory>
#include <mutex>
#include <new>
#include <vector>

using namespace reft;

// ------------------------------------------------------------------------------------------------
// errors and tunables
// ------------------------------------------------------------------------------------------------
static thread_local char g_err[512] = "";

static int fail(int code, const char *fmt, ...)
{
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof g_err, fmt, ap);
    va_end(ap);
    return code;
}

// Entry points that build host-side tables must not let an allocation failure escape the C ABI.
#define REFT_GUARD_BEGIN try {
#define REFT_GUARD_END(who)                                                                       \
    }                                                                                             \
    catch (const std::exception &e)                                                               \
    {                                                                                             \
        return fail(REFT_EINVAL, "%s: host allocation failed (%s)", who, e.what());               \
    }

#define HIPCHK(expr)                                                                              \
    do {                                                                                          \
        hipError_t e_ = (expr);                                                                   \
        if (e_ != hipSuccess)                                                                     \
            return fail(REFT_EHIP, "%s failed: %s (%s:%d)", #expr, hipGetErrorString(e_),         \
                        __FILE__, __LINE__);                                                      \
    } while (0)

static std::atomic<uint64_t> g_max_wgs{0};       // 0 = stream kernel: a wave per unit, others: 16 per compute unit
static std::atomic<uint64_t> g_nontemporal{1};
static std::atomic<uint64_t> g_unroll{4};
static std::atomic<uint64_t> g_tile_shift{18};   // read at plan creation
static std::atomic<uint64_t> g_host_only{0};     // read at plan creation: no device tables
static std::atomic<uint64_t> g_link_wgs{32};     // grid cap of kernels bound by the host link
static std::atomic<uint64_t> g_small_pieces{1}; // spans starting in a tile that make it count as dense
static std::atomic<uint64_t> g_dma_min{4 << 20}; // spans of at least this many bytes are copied by DMA
static std::atomic<uint64_t> g_gather_min{8};    // shortest run of smaller pieces worth a gather kernel
static std::atomic<uint64_t> g_dma_streams{1};   // 2 = piece copies alternate with a helper stream
static std::atomic<uint64_t> g_graph_copies{0};  // piece copies as a hipGraph: 0 off, 1 independent nodes, 2 chain
static std::atomic<uint64_t> g_burst{1};         // parity encode may use the write-burst kernel
static std::atomic<uint64_t> g_burst_min_rows{kBurstMinRows};    // ... from this many sources on
static std::atomic<uint64_t> g_burst_min_bytes{kBurstMinBytes};  // ... and from this stream length on
static std::atomic<uint64_t> g_burst_stage{32768};   // stream bytes per workgroup and round
static std::atomic<uint64_t> g_burst_wgs{2};         // resident workgroups per compute unit
static std::atomic<uint64_t> g_burst_polls{6};       // bound on a writer wave's wait per round (0 = no waiting)
static std::atomic<uint64_t> g_burst_nap{16};        // pause between polls, units of 1024 cycles

extern "C" int reft_set_tunable(const char *name, uint64_t value)
{
    if (!name) return fail(REFT_EINVAL, "reft_set_tunable: null name");
    if (!strcmp(name, "max_wgs")) {
        if (value > (1u << 20)) return fail(REFT_EINVAL, "max_wgs out of range");
        g_max_wgs = value;
    } else if (!strcmp(name, "nontemporal")) {
        if (value > 1) return fail(REFT_EINVAL, "nontemporal must be 0 or 1");
        g_nontemporal = value;
    } else if (!strcmp(name, "unroll")) {
        if (value != 1 && value != 2 && value != 4)
            return fail(REFT_EINVAL, "unroll must be 1, 2 or 4");
        g_unroll = value;
    } else if (!strcmp(name, "tile_shift")) {
        if (value < 12 || value > 24) return fail(REFT_EINVAL, "tile_shift must be in [12, 24]");
        g_tile_shift = value;
    } else if (!strcmp(name, "link_wgs")) {
        if (value < 1 || value > (1u << 20)) return fail(REFT_EINVAL, "link_wgs out of range");
        g_link_wgs = value;
    } else if (!strcmp(name, "dma_min_bytes")) {
        g_dma_min = value;
    } else if (!strcmp(name, "dma_streams")) {
        if (value < 1 || value > 2) return fail(REFT_EINVAL, "dma_streams must be 1 or 2");
        g_dma_streams = value;
    } else if (!strcmp(name, "graph_copies")) {
        if (value > 2) return fail(REFT_EINVAL, "graph_copies must be 0, 1 or 2");
        g_graph_copies = value;
    } else if (!strcmp(name, "gather_min_pieces")) {
        if (value < 1) return fail(REFT_EINVAL, "gather_min_pieces must be at least 1");
        g_gather_min = value;
    } else if (!strcmp(name, "small_pieces")) {
        if (value > 0xffffffffull) return fail(REFT_EINVAL, "small_pieces out of range");
        g_small_pieces = value;
    } else if (!strcmp(name, "host_only_plans")) {
        if (value > 1) return fail(REFT_EINVAL, "host_only_plans must be 0 or 1");
        g_host_only = value;
    } else if (!strcmp(name, "burst")) {
        if (value > 1) return fail(REFT_EINVAL, "burst must be 0 or 1");
        g_burst = value;
    } else if (!strcmp(name, "burst_min_rows")) {
        if (value < 1) return fail(REFT_EINVAL, "burst_min_rows must be at least 1");
        g_burst_min_rows = value;
    } else if (!strcmp(name, "burst_min_bytes")) {
        g_burst_min_bytes = value;
    } else if (!strcmp(name, "burst_stage_bytes")) {
        if (value < 4096 || value > 65536 || value % 4096)
            return fail(REFT_EINVAL, "burst_stage_bytes must be a multiple of 4096 in [4096, 65536]");
        g_burst_stage = value;
    } else if (!strcmp(name, "burst_wgs_per_cu")) {
        if (value < 1 || value > 8) return fail(REFT_EINVAL, "burst_wgs_per_cu must be in [1, 8]");
        g_burst_wgs = value;
    } else if (!strcmp(name, "burst_max_polls")) {
        if (value > 100000) return fail(REFT_EINVAL, "burst_max_polls must be at most 100000");
        g_burst_polls = value;
    } else if (!strcmp(name, "burst_nap")) {
        if (value > 1024) return fail(REFT_EINVAL, "burst_nap must be at most 1024");
        g_burst_nap = value;

    } else {
        return fail(REFT_EINVAL, "unknown tunable '%s'", name);
    }
    return REFT_OK;
}

extern "C" int reft_get_tunable(const char *name, uint64_t *value)
{
    if (!name || !value) return fail(REFT_EINVAL, "reft_get_tunable: null argument");
    if (!strcmp(name, "max_wgs")) *value = g_max_wgs;
    else if (!strcmp(name, "nontemporal")) *value = g_nontemporal;
    else if (!strcmp(name, "unroll")) *value = g_unroll;
    else if (!strcmp(name, "tile_shift")) *value = g_tile_shift;
    else if (!strcmp(name, "host_only_plans")) *value = g_host_only;
    else if (!strcmp(name, "link_wgs")) *value = g_link_wgs;
    else if (!strcmp(name, "small_pieces")) *value = g_small_pieces;
    else if (!strcmp(name, "dma_min_bytes")) *value = g_dma_min;
    else if (!strcmp(name, "gather_min_pieces")) *value = g_gather_min;
    else if (!strcmp(name, "dma_streams")) *value = g_dma_streams;
    else if (!strcmp(name, "graph_copies")) *value = g_graph_copies;
    else if (!strcmp(name, "burst")) *value = g_burst;
    else if (!strcmp(name, "burst_min_rows")) *value = g_burst_min_rows;
    else if (!strcmp(name, "burst_min_bytes")) *value = g_burst_min_bytes;
    else if (!strcmp(name, "burst_stage_bytes")) *value = g_burst_stage;
    else if (!strcmp(name, "burst_wgs_per_cu")) *value = g_burst_wgs;
    else if (!strcmp(name, "burst_max_polls")) *value = g_burst_polls;
    else if (!strcmp(name, "burst_nap")) *value = g_burst_nap;
    else return fail(REFT_EINVAL, "unknown tunable '%s'", name);
    return REFT_OK;
}

extern "C" const char *reft_last_error(void) { return g_err; }
extern "C" const char *reft_version(void) { return "libreft 0.1 (gfx950)"; }

// ------------------------------------------------------------------------------------------------
// plan
// ------------------------------------------------------------------------------------------------
namespace {
constexpr int kRing = 32;       // pointer tables the plan's cache holds at once
constexpr int kUsers = 4;       // streams per cached table whose most recent use is tracked
// Capacity of the cache, in rows of T pointers: kCacheRows for the null stream's tables and kSideRows, enough for the widest
// table, that these leave to other streams (see null_end).  Of many spans there are kCacheRows in all, those for the null
// stream among them, and its tables may lie in the others as well (where a call on 65,536 spans leaves an event, 2 us,
// it has spent more than ten times that on comparing pointers).
constexpr uint32_t kCacheRows = 72, kSideRows = REFT_MAX_K + 1;
constexpr uint64_t kManySpans = 65536;
static_assert(kCacheRows >= 2 * kSideRows, "the widest table must fit on either side");
constexpr int kMaxSlots = 64;   // staging slots used by the staged bucket pipelines
constexpr int kGroups = 2;      // the slots form two groups that alternate (double buffering)
constexpr uint32_t kCtrBlocks = 8;  // burst launches that may be in flight on one ring of counters
constexpr size_t kPieceLists = 8;   // classified bucket ranges a plan remembers

struct Event {
    hipEvent_t ev = nullptr;
    bool recorded = false;
};

struct Run {            // stream range [a, b) of consecutive small pieces: gather kernel + one copy
    uint64_t a, b;
};
struct Dma {            // a span, or a bucket's piece of one, copied by the DMA path straight from its tensor
    uint64_t o, n, span;
};
// How the bytes of a bucket range travel in the staged transport (see classify_pieces); depends
// on the plan and two tunables only, so it is computed once and kept.
struct PieceLists {
    uint64_t b0 = 0, b1 = 0, dma_min = 0, gather_min = 0, tick = 0;
    std::vector<Run> runs;
    std::vector<Dma> dmas;
};

// One cached pointer table: `len` pointers at position `pos` of the plan's pool (pinned host
// mirror and device copy).  `uploaded` is recorded behind the host-to-device copy; used[i] behind
// the last kernel that read the table on stream user[i], but for readers on the null stream in the
// pool's first rows (see null_end).
struct PtrEntry {
    bool live = false;
    uint64_t pos = 0, len = 0, hash = 0, tick = 0;
    uint64_t upload = 0;    // number of the upload that brought it, of all of the plan's
    int in_place = -1;      // whether a source lies where the result for in_place_vb goes (see in_place());
    uint64_t in_place_vb = 0;   // -1: not looked at
    hipStream_t up_stream = nullptr;
    Event uploaded;
    hipStream_t user[kUsers] = {};
    Event used[kUsers];
};

// A plan derived from a base plan for the rotated placement, with the recipe that turns the
// caller's pointers into its rows: entry (q * T' + t) says where piece t of row q starts.
struct RowRecipe {
    uint32_t span;      // span of the base plan, or kContig / kZeros
    uint32_t of;        // the member whose shard (or, with kContig, parity unit) it lies in, or kOut
    uint64_t add;       // byte offset inside that span (or inside the unit)
};
constexpr uint32_t kContig = 0xffffffffu, kZeros = 0xfffffffeu;
constexpr uint32_t kOut = 0xffffffffu;   // the tensors that receive a decoded shard
}  // namespace

// What a plan knows of the rings of slots that staged calls were given.
struct SlotRing {
    bool alone = false;               // the last call had one stream for everything and left no events behind its slots: its
                                      // completion event says when they are free
    int known = 0;
    struct Layout {                   // where groups lay: group g at `at` + g * `bytes`
        uint64_t at, bytes;
    } layout[4];                      // no two in the same memory
};

// Pointers that a caller passed, and where in the derived plan's cache the rows made of them went.
struct SeenPointers {
    std::vector<const void *> ptrs;
    int entry = 0;
    uint64_t upload = 0;              // 0: none
};

// The spans whose pointers a recipe may ask for: of member `of`'s shard or, with kOut, of the tensors.
struct PointerRange {
    uint32_t of;
    uint64_t first, end;
};

struct DerivedPlan {
    reft_plan *plan = nullptr;
    uint32_t nwin = 0;
    std::vector<RowRecipe> recipe;
    std::vector<PointerRange> uses;   // one for each member
    std::vector<uint32_t> units;      // members whose parity units it asks for
    SeenPointers seen[2];             // of the two most recent sets, seen[last] the newer one's
    int last = 0;
};

struct reft_plan {
    bool host_only = false;           // sizing only: no device tables, data calls are refused
    int device = 0;
    int num_cus = 256;
    uint64_t T = 0, NB = 0, L = 0, max_bucket = 0;
    uint32_t tile_shift = 16;
    uint32_t unit_shift = 0;          // blocks of the device's look-up table of units
    uint32_t grid = 0;                // see head_of
    uint32_t unit = 1024;             // see unit_bytes
    bool odd = false, windows = false;   // see PlanTables
    uint32_t burst_shift = 16;        // tiles of the burst kernel's look-up table
    uint64_t ntiles = 0;
    std::vector<uint64_t> off;        // [T+1]
    std::vector<uint64_t> unit_off;   // [T+1] (of plans with device tables)
    std::vector<uint64_t> bstart;     // [NB+1]
    std::vector<uint32_t> first;      // [ntiles] host copy of the tile table
    uint8_t *d_tables = nullptr;      // device memory of the plan; the pointers below point into it
    uint64_t *d_off = nullptr, *d_unit_off = nullptr;
    uint32_t *d_unit_span = nullptr, *d_tile_span = nullptr;
    // cache of pointer tables: a pool of ring_cap pointers (pinned host mirror and device copy)
    // handed out front to back, and the tables that currently live in it
    uint64_t ring_cap = 0, ring_head = 0, ring_tick = 0, uploads = 0;
    // Room below null_end is left to the null stream: kernels on it may have read tables there without an event
    // behind them, so that only what comes behind them on that stream may overwrite that room.  The null stream's tables
    // lie in the first null_cap pointers' room as far as null_most allows; the rest is other streams' in any case, and
    // there each reader leaves its event.  (4 x 0.9 MB encoded call after call 6.6 us with an event behind each, 4.4
    // without; 4 x 14.7 MB 13.9, 12.85.)
    uint64_t null_end = 0, null_cap = 0, null_most = 0;
    uint64_t *h_ptr = nullptr;
    uint64_t *d_ptr = nullptr;
    PtrEntry ring[kRing];
    // host scratch for the row tables of the XOR entry points ((REFT_MAX_K + 1) * T pointers)
    std::vector<const void *> row_buf;
    // classified piece lists of recent bucket ranges (the whole stream's is made at creation)
    std::vector<PieceLists> pieces;
    uint64_t pieces_tick = 0;
    // stream on which the most recent snapshot's completion event was recorded
    hipStream_t last_pack_stream = nullptr;
    SlotRing pack_ring, rest_ring;                            // of snapshots, and of restores
    hipStream_t rest_stream = nullptr;                        // on which rest_done was recorded
    // device address of the library's static scratch on this plan's GPU (see reft_parity_encode_noalloc)
    unsigned char *scratch = nullptr;
    // bucket pipelines
    Event pack_filled[kGroups], pack_free[kGroups], pack_done, pack_begin, rest_begin;
    Event rest_filled[kGroups], rest_free[kGroups], rest_done, rest_copied;
    // helper stream for the staged transport's piece copies (tunable "dma_streams" = 2), default
    // priority, and the events that fork it from / join it to copy_stream
    hipStream_t aux = nullptr;
    Event aux_fork, aux_join;
    // rotated parity placement: plans derived from this one (merged piece lists of shifted
    // windows), keyed by (kind, k, member, segment), and a small all-zero device buffer that
    // stands in for the zero extension of the last segment
    std::map<uint64_t, DerivedPlan> derived;
    void *zeros = nullptr;
    // the piece copies of recent snapshot / restore calls as instantiated graphs (see copy_graph)
    struct CopyGraph {
        std::vector<uint64_t> key;
        hipGraphExec_t exec = nullptr;
        uint64_t used = 0;
        hipEvent_t done = nullptr;    // recorded behind the most recent launch
    };
    std::vector<CopyGraph> graphs;
    uint64_t graph_tick = 0;
    // write-burst kernel: spans that start in each tile where any do, sorted (plans with many span boundaries keep
    // the stream kernel), and a ring of counter blocks, one per launch in flight
    std::vector<uint32_t> tile_spans_sorted;
    uint32_t *burst_ctr = nullptr;
    uint32_t burst_next = 0;

    PlanTables tables() const
    {
        return PlanTables{d_off, d_unit_off, d_unit_span, d_tile_span, T, L, unit_shift, burst_shift, grid, unit, odd, windows};
    }

    // lo < hi <= L.  All numbers of a span whose bytes are all in the range are dealt, also those behind its units that have
    // no bytes (see align_of): a span that is turned has units under every one of them.  (Without them a launch that ended
    // with such a span in front of the stream's end left up to 31 KiB of it unmoved.)
    StreamRange range(uint64_t lo, uint64_t hi) const
    {
        StreamRange r{lo, hi, 0, unit_off[T] - 1};
        if (lo > 0) {
            const uint64_t i = (uint64_t)(std::upper_bound(off.begin(), off.end() - 1, lo) - off.begin()) - 1;
            r.first = unit_off[i] + first_unit_at(lo - off[i], head_of(off[i], grid, unit), unit);
        }
        if (hi < L) {
            const uint64_t i = (uint64_t)(std::upper_bound(off.begin(), off.end() - 1, hi - 1) - off.begin()) - 1;
            r.last = hi == off[i + 1] ? unit_off[i + 1] - 1
                                      : unit_off[i] + last_unit_at(hi - 1 - off[i], head_of(off[i], grid, unit), unit);
        }
        return r;
    }
    StreamRange all() const { return range(0, L); }
};

static LaunchCfg launch_cfg(const reft_plan *p)
{
    const uint64_t cap = g_max_wgs;
    const uint64_t w = cap ? cap : 16ull * (uint64_t)(p ? p->num_cus : 256);
    return LaunchCfg{(uint32_t)w, cap != 0, cap != 0, (uint32_t)g_unroll.load(), g_nontemporal.load() != 0};
}

// Kernels whose rate is set by the host link need only a few workgroups to saturate it.
static LaunchCfg link_cfg(const reft_plan *p, uint32_t halves)
{
    LaunchCfg c = launch_cfg(p);
    c.max_wgs = link_cap(g_link_wgs.load(), halves, c.max_wgs);
    c.capped = true;
    c.runs = false;
    return c;
}

// The address at which the GPU sees a host buffer, or 0 if it is not mapped for device access
// (pageable memory).  Clears the sticky error a failed lookup leaves behind.
static uint64_t device_view_of_host(const void *host)
{
    void *d = nullptr;
    if (hipHostGetDevicePointer(&d, const_cast<void *>(host), 0) != hipSuccess) {
        (void)hipGetLastError();
        return 0;
    }
    return (uint64_t)(uintptr_t)d;
}

// The same for the `bytes` bytes from there on, or 0 unless one allocation holds all of them (between two that both ends
// lie in there may be memory that the GPU does not see).
static uint64_t device_view_of_host(const void *host, uint64_t bytes)
{
    const uint64_t a = device_view_of_host(host);
    hipDeviceptr_t base = nullptr;
    size_t n = 0;
    if (!a) return 0;
    if (hipMemGetAddressRange(&base, &n, (hipDeviceptr_t)(uintptr_t)a) != hipSuccess) {
        (void)hipGetLastError();
        return 0;
    }
    return a - (uint64_t)(uintptr_t)base + bytes <= n ? a : 0;
}

static int make_event(Event &e, unsigned flags = hipEventDisableTiming)
{
    HIPCHK(hipEventCreateWithFlags(&e.ev, flags));
    e.recorded = false;
    return REFT_OK;
}

static int record(Event &e, hipStream_t s)
{
    HIPCHK(hipEventRecord(e.ev, s));
    e.recorded = true;
    return REFT_OK;
}

static int wait_on(hipStream_t s, const Event &e)
{
    if (e.recorded) HIPCHK(hipStreamWaitEvent(s, e.ev, 0));
    return REFT_OK;
}

// Whether work given to `a` and to `b`, maybe by two threads in turn, runs in order by itself: hipStreamPerThread is one
// handle for a stream of every thread's own.
static bool same_stream(hipStream_t a, hipStream_t b) { return a == b && a != hipStreamPerThread; }

// ------------------------------------------------------------------------------------------------
// static device memory of the library
// ------------------------------------------------------------------------------------------------
// `scratch` serves reft_parity_encode_noalloc, the entry point for callers that cannot allocate:
// a table of up to kScratchPtrs span pointers, then one block of burst counters.  Every GPU the
// library runs on holds its own copy until the process ends.  `static_ctr` is the ring of counter
// blocks of reft_reconstruct, which has no plan to keep them in.  In host code these names are
// stand-ins, not device addresses: the addresses come from hipGetSymbolAddress, once per device.
constexpr uint32_t kScratchPtrs = 32768;
constexpr size_t kScratchPtrBytes = (size_t)kScratchPtrs * sizeof(uint64_t);
constexpr size_t kScratchBytes = kScratchPtrBytes + 2560;            // 256 KiB + counters
static_assert(kBurstCtrBytes <= 2560, "the counter block must fit behind the pointer table");
static __device__ __align__(256) unsigned char scratch[kScratchBytes];
static __device__ __align__(256) uint32_t static_ctr[kCtrBlocks * (kBurstCtrBytes / sizeof(uint32_t))];

namespace {
constexpr int kMaxDevices = 64;
struct DeviceStatics {
    bool known = false;
    unsigned char *scratch = nullptr;
    uint32_t *ctr = nullptr;
    int num_cus = 256;
};
std::mutex g_statics_mu;
DeviceStatics g_statics[kMaxDevices];
}  // namespace

// The addresses of the static arrays on the current device (resolved on first use per device).
static int device_statics(const DeviceStatics **out)
{
    int dev = -1;
    HIPCHK(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return fail(REFT_EINVAL, "GPU %d: unsupported device index", dev);
    std::lock_guard<std::mutex> lock(g_statics_mu);
    DeviceStatics &d = g_statics[dev];
    if (!d.known) {
        void *a = nullptr, *b = nullptr;
        HIPCHK(hipGetSymbolAddress(&a, HIP_SYMBOL(scratch)));
        HIPCHK(hipGetSymbolAddress(&b, HIP_SYMBOL(static_ctr)));
        if (!a || !b) return fail(REFT_EHIP, "hipGetSymbolAddress returned a null address");
        hipDeviceProp_t prop;
        HIPCHK(hipGetDeviceProperties(&prop, dev));
        d.scratch = (unsigned char *)a;
        d.ctr = (uint32_t *)b;
        d.num_cus = prop.multiProcessorCount > 0 ? prop.multiProcessorCount : 256;
        d.known = true;
    }
    *out = &d;
    return REFT_OK;
}

// ------------------------------------------------------------------------------------------------
// cache of pointer tables
// ------------------------------------------------------------------------------------------------
static void free_ring(reft_plan *p)
{
    if (p->h_ptr) (void)hipHostFree(p->h_ptr);
    p->h_ptr = nullptr;
    p->ring_cap = 0;
}

// A filter in front of the comparison of all pointers, which decides: about 64 of them will do.  (All
// of them, one multiply behind the other: the first call of an encode with 98,304 took 415 us, this way 299.)
static uint64_t hash_ptrs(const void *const *ptrs, size_t n)
{
    const size_t step = n / 64 + 1;
    uint64_t h = 0x9e3779b97f4a7c15ull ^ n;
    for (size_t i = 0; i < n; i += step) {
        h ^= (uint64_t)(uintptr_t)ptrs[i];
        h *= 0x100000001b3ull;
        h ^= h >> 29;
    }
    return h;
}

// The host waits for exactly the work behind which an event was recorded that may still read the entry's table (its
// upload and kernels): never for the whole device.
static int retire_entry(PtrEntry &e)
{
    if (e.uploaded.recorded) HIPCHK(hipEventSynchronize(e.uploaded.ev));
    e.uploaded.recorded = false;
    for (int i = 0; i < kUsers; ++i) {
        if (e.used[i].recorded) HIPCHK(hipEventSynchronize(e.used[i].ev));
        e.used[i].recorded = false;
        e.user[i] = nullptr;
    }
    e.live = false;
    return REFT_OK;
}

// A live entry's table for work on stream s.
static int use_entry(reft_plan *p, int entry, hipStream_t s, const uint64_t **dev_tab)
{
    PtrEntry &e = p->ring[entry];
    if (!same_stream(e.up_stream, s) && e.uploaded.recorded) HIPCHK(hipStreamWaitEvent(s, e.uploaded.ev, 0));
    e.tick = ++p->ring_tick;
    *dev_tab = p->d_ptr + e.pos;
    return REFT_OK;
}

// Make `rows` x T pointers available on the device: reuse the cached table that already holds
// exactly these pointers (a trainer passes the same tensors every iteration; a stream other than
// the one that uploaded it waits for the upload only), else take the next room in the pool,
// retiring the tables that lie there, and start the upload on `s`.  On success *dev_tab is the
// device table and *entry the cache index to pass to release_ptrs after the last kernel that
// reads the table.
static int upload_ptrs(reft_plan *p, const void *const *ptrs, uint32_t rows, hipStream_t s,
                       const uint64_t **dev_tab, int *entry)
{
    static_assert(sizeof(void *) == sizeof(uint64_t), "pointers are 64-bit");
    const uint64_t n = (uint64_t)rows * p->T;
    const uint64_t least = s == nullptr ? 0 : p->null_end, most = s == nullptr ? p->null_most : p->ring_cap;
    if (n > most - least)
        return fail(REFT_ESIZE, "pointer table of %u rows exceeds the plan's cache (%llu pointers)",
                    rows, (unsigned long long)p->ring_cap);
    const uint64_t h = hash_ptrs(ptrs, n);
    int rc;
    for (int i = 0; i < kRing; ++i) {
        PtrEntry &e = p->ring[i];
        if (e.live && e.len == n && e.hash == h &&
            !memcmp(p->h_ptr + e.pos, ptrs, n * sizeof(uint64_t))) {
            *entry = i;
            return use_entry(p, i, s, dev_tab);
        }
    }
    const uint64_t pos = p->ring_head + n > most || p->ring_head < least ? least : p->ring_head;
    int slot = -1;
    for (int i = 0; i < kRing; ++i) {
        PtrEntry &e = p->ring[i];
        if (e.live && e.pos < pos + n && pos < e.pos + e.len && (rc = retire_entry(e))) return rc;
        if (!e.live && slot < 0) slot = i;
    }
    if (slot < 0) {                                    // every slot is live: the oldest goes
        slot = 0;
        for (int i = 1; i < kRing; ++i)
            if (p->ring[i].tick < p->ring[slot].tick) slot = i;
        if ((rc = retire_entry(p->ring[slot]))) return rc;
    }
    PtrEntry &e = p->ring[slot];
    memcpy(p->h_ptr + pos, ptrs, n * sizeof(uint64_t));
    HIPCHK(hipMemcpyAsync(p->d_ptr + pos, p->h_ptr + pos, n * sizeof(uint64_t),
                          hipMemcpyHostToDevice, s));
    HIPCHK(hipEventRecord(e.uploaded.ev, s));
    e.uploaded.recorded = true;
    e.up_stream = s;
    e.live = true;
    e.pos = pos;
    e.len = n;
    e.hash = h;
    e.in_place = -1;
    e.tick = ++p->ring_tick;
    e.upload = ++p->uploads;
    p->ring_head = pos + n;
    *dev_tab = p->d_ptr + pos;
    *entry = slot;
    return REFT_OK;
}

// Record, on stream s, that the kernels queued so far were the last ones to read entry's table (or
// leave its room to the null stream).
static int release_ptrs(reft_plan *p, int entry, hipStream_t s)
{
    PtrEntry &e = p->ring[entry];
    if (s == nullptr && e.pos + e.len <= p->null_cap) {
        if (p->null_end < e.pos + e.len) p->null_end = e.pos + e.len;
        return REFT_OK;
    }
    int i = -1;
    for (int u = 0; u < kUsers && i < 0; ++u)
        if (e.used[u].recorded && same_stream(e.user[u], s)) i = u;
    for (int u = 0; u < kUsers && i < 0; ++u)
        if (!e.used[u].recorded) i = u;
    for (int u = 0; u < kUsers && i < 0; ++u)
        if (hipEventQuery(e.used[u].ev) == hipSuccess) i = u;
    if (i < 0) {                                       // more streams than tracked: wait for one
        i = 0;
        HIPCHK(hipEventSynchronize(e.used[0].ev));
    }
    (void)hipGetLastError();                           // hipEventQuery's "not ready" is no error
    e.user[i] = s;
    HIPCHK(hipEventRecord(e.used[i].ev, s));
    e.used[i].recorded = true;
    return REFT_OK;
}

static int check_plan(const reft_plan *p, const char *who)
{
    if (!p) return fail(REFT_EINVAL, "%s: null plan", who);
    if (p->host_only)
        return fail(REFT_EINVAL, "%s: the plan was created host-only (no device tables)", who);
    int dev = -1;
    HIPCHK(hipGetDevice(&dev));
    if (dev != p->device)
        return fail(REFT_EINVAL, "%s: plan belongs to GPU %d but GPU %d is current", who,
                    p->device, dev);
    return REFT_OK;
}

static int check_span_ptrs(const reft_plan *p, const void *const *ptrs, uint32_t rows,
                           const char *who)
{
    if (!ptrs) return fail(REFT_EINVAL, "%s: null pointer array", who);
    for (uint32_t r = 0; r < rows; ++r)
        for (uint64_t t = 0; t < p->T; ++t)
            if (!ptrs[r * p->T + t] && p->off[t + 1] != p->off[t])
                return fail(REFT_EINVAL, "%s: span %llu of shard %u is null but has %llu bytes",
                            who, (unsigned long long)t, r,
                            (unsigned long long)(p->off[t + 1] - p->off[t]));
    return REFT_OK;
}

static const PieceLists &pieces_of(reft_plan *p, uint64_t b0, uint64_t b1);

extern "C" int reft_plan_create(const uint64_t *span_nbytes, uint64_t T,
                                const uint64_t *bucket_nbytes, uint64_t NB,
                                uint64_t uniform_bucket, reft_plan **out)
{
    REFT_GUARD_BEGIN
    if (!out) return fail(REFT_EINVAL, "reft_plan_create: null out");
    *out = nullptr;
    if (!span_nbytes || T == 0) return fail(REFT_EINVAL, "reft_plan_create: no spans");
    if (T >= 0xffffffffull) return fail(REFT_EINVAL, "reft_plan_create: too many spans");

    reft_plan *p = new (std::nothrow) reft_plan;
    if (!p) return fail(REFT_EINVAL, "reft_plan_create: out of host memory");
    struct Guard {
        reft_plan *p;
        ~Guard() { if (p) reft_plan_destroy(p); }
    } guard{p};

    p->T = T;
    p->off.resize(T + 1);
    p->off[0] = 0;
    for (uint64_t t = 0; t < T; ++t)
        if (__builtin_add_overflow(p->off[t], span_nbytes[t], &p->off[t + 1]))
            return fail(REFT_ESIZE, "reft_plan_create: stream length overflows 64 bits");
    p->L = p->off[T];

    // buckets
    p->bstart.push_back(0);
    if (uniform_bucket) {
        for (uint64_t b = 0; b < p->L; b += uniform_bucket)
            p->bstart.push_back(b + uniform_bucket < p->L ? b + uniform_bucket : p->L);
    } else if (!bucket_nbytes && NB == 0) {
        if (p->L) p->bstart.push_back(p->L);              // no bucketing asked: one bucket
    } else {
        if (NB && !bucket_nbytes) return fail(REFT_EINVAL, "reft_plan_create: null bucket list");
        uint64_t acc = 0;
        for (uint64_t b = 0; b < NB; ++b) {
            if (bucket_nbytes[b] == 0)
                return fail(REFT_EINVAL, "reft_plan_create: bucket %llu has zero length",
                            (unsigned long long)b);
            if (__builtin_add_overflow(acc, bucket_nbytes[b], &acc) || acc > p->L)
                return fail(REFT_ESIZE, "reft_plan_create: buckets exceed the stream length");
            p->bstart.push_back(acc);
        }
        if (acc != p->L)
            return fail(REFT_ESIZE, "reft_plan_create: buckets cover %llu of %llu stream bytes",
                        (unsigned long long)acc, (unsigned long long)p->L);
    }
    p->NB = p->bstart.size() - 1;
    for (uint64_t b = 0; b < p->NB; ++b)
        if (p->bstart[b + 1] - p->bstart[b] > p->max_bucket)
            p->max_bucket = p->bstart[b + 1] - p->bstart[b];

    // tile table: first span that owns a byte of tile t (zero-length spans never qualify)
    p->tile_shift = (uint32_t)g_tile_shift.load();
    const uint64_t tile = 1ull << p->tile_shift;
    p->ntiles = (p->L + tile - 1) >> p->tile_shift;
    std::vector<uint32_t> &first = p->first;
    first.assign(p->ntiles ? p->ntiles : 1, 0);
    {
        uint64_t i = 0;
        for (uint64_t t = 0; t < p->ntiles; ++t) {
            const uint64_t o = t << p->tile_shift;
            while (p->off[i + 1] <= o) ++i;      // o < L = off[T] keeps i < T
            first[t] = (uint32_t)i;
        }
        for (uint64_t t = 0; t < p->ntiles; ++t) {
            const uint64_t nxt = t + 1 < p->ntiles ? first[t + 1] : T - 1;
            if (nxt > first[t]) p->tile_spans_sorted.push_back((uint32_t)(nxt - first[t]));
        }
        std::sort(p->tile_spans_sorted.begin(), p->tile_spans_sorted.end());
    }

    if (g_host_only.load()) {
        p->host_only = true;
        guard.p = nullptr;
        *out = p;
        return REFT_OK;
    }
    // (beyond this the pointer pool alone is 1.2 TB)
    if (T >= kWholeBlock) return fail(REFT_EINVAL, "reft_plan_create: too many spans for a GPU");
    HIPCHK(hipGetDevice(&p->device));
    hipDeviceProp_t prop;
    HIPCHK(hipGetDeviceProperties(&prop, p->device));
    p->num_cus = prop.multiProcessorCount > 0 ? prop.multiProcessorCount : 256;
    // The stream kernel's look-up table: an entry per unit (a look-up then needs no search) as long as that is
    // no more than 16,384 entries or 4 per span, else blocks of units (with 8 per span 0.3 % faster at 10 KB a span,
    // but plans of 49,152 spans take 1.9 ms to make instead of 1.0).  (Made here and not by a kernel: that would wait
    // behind whatever the null stream still has to do, and plan creation with it.)
    p->grid = grid_of(p->L, T);
    p->unit = (uint32_t)unit_bytes(p->L, T);
    p->unit_off.resize(T + 1);
    uint64_t number = 0, apart = 0;
    const uint64_t align = align_of(p->L, T);
    for (uint64_t t = 0; t < T; ++t) {
        const uint64_t b = p->off[t], n = p->off[t + 1] - b;
        if (b % 64) apart += n;
        if (n) number = first_number(number, b, align);
        p->unit_off[t] = number;
        number += p->unit == kUnit ? units_of(n, head_of(b, p->grid)) : units_of(n, kSmallUnit, kSmallUnit);
    }
    p->unit_off[T] = number;
    p->odd = odd_stream(apart, p->L);
    const uint64_t units = p->unit_off[T], most = std::min<uint64_t>(std::max<uint64_t>(16384, 4 * T), 1ull << 31);
    p->unit_shift = 0;
    while ((units >> p->unit_shift) > most) ++p->unit_shift;
    const uint64_t nblocks = (units >> p->unit_shift) + 1;
    // One allocation and one copy for the tables: span offsets, unit offsets, the burst kernel's spans of tiles (4096 of
    // them at most, it walks on from there) and the units' spans; behind them the burst counters and the device half
    // of the pointer pool.
    p->burst_shift = p->tile_shift;
    while ((p->L >> p->burst_shift) >= 4096) ++p->burst_shift;
    const size_t burst_tiles = (size_t)(p->L >> p->burst_shift) + 1;
    auto behind = [](size_t at, size_t bytes) { return (at + bytes + 255) & ~(size_t)255; };
    const size_t at_unit_off = behind(0, (T + 1) * sizeof(uint64_t));
    const size_t at_tile_span = behind(at_unit_off, (T + 1) * sizeof(uint64_t));
    const size_t at_unit_span = behind(at_tile_span, burst_tiles * sizeof(uint32_t));
    const size_t at_ctr = behind(at_unit_span, (nblocks + 3) * sizeof(uint32_t));
    const size_t at_ptr = behind(at_ctr, kCtrBlocks * kBurstCtrBytes);
    p->ring_cap = (T < kManySpans ? kCacheRows + kSideRows : kCacheRows) * T;
    p->null_cap = p->ring_cap - kSideRows * T;
    p->null_most = T < kManySpans ? p->null_cap : p->ring_cap;
    HIPCHK(hipHostMalloc((void **)&p->h_ptr, p->ring_cap * sizeof(uint64_t), hipHostMallocDefault));
    // Made in the pinned mirror of the pool, which is not in use yet, where they fit (256 spans of 60 KB: 91 us for all of
    // this function from other memory, 66 so).  Gaps are not read.
    std::unique_ptr<uint64_t[]> heap;
    if (at_ctr > p->ring_cap * sizeof(uint64_t)) heap.reset(new uint64_t[at_ctr / sizeof(uint64_t)]);
    uint64_t *const tables = heap ? heap.get() : p->h_ptr;
    std::copy(p->off.begin(), p->off.end(), tables);
    std::copy(p->unit_off.begin(), p->unit_off.end(), tables + at_unit_off / sizeof(uint64_t));
    uint32_t *const tile_span = (uint32_t *)((uint8_t *)tables + at_tile_span);
    for (size_t t = 0; t < burst_tiles; ++t) {
        const size_t at = t << (p->burst_shift - p->tile_shift);
        tile_span[t] = at < p->ntiles ? first[at] : 0;
    }
    uint32_t *const lookup = (uint32_t *)((uint8_t *)tables + at_unit_span);
    for (uint64_t t = 0, i = 0; i < T; ++i) {                        // t: the first block without an entry
        const uint64_t end = p->unit_off[i + 1], whole = end >> p->unit_shift;
        if (whole > t) {                       // (four at a time: up to three too many, for the spans behind)
            for (; t < whole; t += 4) std::fill_n(lookup + t, 4, (uint32_t)i | kWholeBlock);
            t = whole;
        }
        if (t << p->unit_shift < end) lookup[t++] = (uint32_t)i;
    }
    HIPCHK(hipMalloc((void **)&p->d_tables, at_ptr + p->ring_cap * sizeof(uint64_t)));
    HIPCHK(hipMemcpy(p->d_tables, tables, at_ctr, hipMemcpyHostToDevice));
    p->d_off = (uint64_t *)p->d_tables;
    p->d_unit_off = (uint64_t *)(p->d_tables + at_unit_off);
    p->d_tile_span = (uint32_t *)(p->d_tables + at_tile_span);
    p->d_unit_span = (uint32_t *)(p->d_tables + at_unit_span);
    p->burst_ctr = (uint32_t *)(p->d_tables + at_ctr);
    p->d_ptr = (uint64_t *)(p->d_tables + at_ptr);
    int rc;
    const DeviceStatics *ds = nullptr;
    if ((rc = device_statics(&ds))) return rc;
    p->scratch = ds->scratch;
    for (int i = 0; i < kRing; ++i) {
        if ((rc = make_event(p->ring[i].uploaded))) return rc;
        // A use of a table is only ever waited for (by the host, so that the table may be overwritten);
        // nothing is read that the kernels in front of the event wrote.  So the event needs no
        // system fence, which would write the caches back behind every call: 4 x 14.7 MB encoded
        // call after call 16.2 us with it, 14.2 without.
        for (int u = 0; u < kUsers; ++u)
            if ((rc = make_event(p->ring[i].used[u], hipEventDisableTiming | hipEventDisableSystemFence)))
                return rc;
    }
    for (int i = 0; i < kGroups; ++i) {
        if ((rc = make_event(p->pack_filled[i])) || (rc = make_event(p->pack_free[i])) ||
            (rc = make_event(p->rest_filled[i])) || (rc = make_event(p->rest_free[i])))
            return rc;
    }
    if ((rc = make_event(p->pack_done)) || (rc = make_event(p->rest_done)) ||
        (rc = make_event(p->rest_copied)) || (rc = make_event(p->pack_begin)) ||
        (rc = make_event(p->rest_begin)) || (rc = make_event(p->aux_fork)) ||
        (rc = make_event(p->aux_join)))
        return rc;
    // The helper stream exists only where it is asked for: a stream takes its place among the
    // process's few hardware queues when it is created, whether it ever gets work or not (two
    // idle helper streams made here were enough to push a snapshot and a restore, on streams
    // created after them, onto one queue, where they took turns on the link).
    if (g_dma_streams.load() == 2) HIPCHK(hipStreamCreateWithFlags(&p->aux, hipStreamNonBlocking));
    // everything else a data-moving call needs is made here too: the host scratch for row tables, and
    // the whole stream's piece lists for the staged transport
    p->row_buf.resize((size_t)(REFT_MAX_K + 1) * T);
    p->pieces.reserve(kPieceLists);
    (void)pieces_of(p, 0, p->NB);

    guard.p = nullptr;
    *out = p;
    return REFT_OK;
    REFT_GUARD_END("reft_plan_create")
}

extern "C" void reft_plan_destroy(reft_plan *p)
{
    if (!p) return;
    // let everything that still reads the plan's tables finish
    auto drain = [](Event &e) {
        if (e.ev) {
            if (e.recorded) (void)hipEventSynchronize(e.ev);
            (void)hipEventDestroy(e.ev);
            e.ev = nullptr;
        }
    };
    for (int i = 0; i < kRing; ++i) {
        drain(p->ring[i].uploaded);
        for (int u = 0; u < kUsers; ++u) drain(p->ring[i].used[u]);
    }
    if (p->null_end) {                                 // the plan's GPU need not be the current one
        int dev = p->device;
        (void)hipGetDevice(&dev);
        if (dev != p->device) (void)hipSetDevice(p->device);
        (void)hipStreamSynchronize(nullptr);
        if (dev != p->device) (void)hipSetDevice(dev);
    }
    for (int i = 0; i < kGroups; ++i) {
        drain(p->pack_filled[i]);
        drain(p->pack_free[i]);
        drain(p->rest_filled[i]);
        drain(p->rest_free[i]);
    }
    drain(p->pack_done);
    drain(p->rest_done);
    drain(p->rest_copied);
    drain(p->aux_fork);
    drain(p->aux_join);
    if (p->aux) (void)hipStreamDestroy(p->aux);
    drain(p->pack_begin);
    drain(p->rest_begin);
    free_ring(p);
    for (auto &g : p->graphs) {
        if (g.done) {
            (void)hipEventSynchronize(g.done);
            (void)hipEventDestroy(g.done);
        }
        if (g.exec) (void)hipGraphExecDestroy(g.exec);
    }
    for (auto &kv : p->derived) reft_plan_destroy(kv.second.plan);
    p->derived.clear();
    if (p->zeros) (void)hipFree(p->zeros);
    if (p->d_tables) (void)hipFree(p->d_tables);
    delete p;
}

extern "C" uint64_t reft_plan_stream_bytes(const reft_plan *p) { return p ? p->L : 0; }
extern "C" uint64_t reft_plan_num_spans(const reft_plan *p) { return p ? p->T : 0; }
extern "C" uint64_t reft_plan_num_buckets(const reft_plan *p) { return p ? p->NB : 0; }
extern "C" uint64_t reft_plan_max_bucket_bytes(const reft_plan *p) { return p ? p->max_bucket : 0; }

static uint64_t slot_stride(const reft_plan *p)
{
    // room for the bucket plus the sub-256-byte phase that keeps slot addresses congruent to
    // stream offsets (so 16-byte-aligned spans stay aligned in the slot)
    return (p->max_bucket + 256 + 255) & ~255ull;
}

extern "C" uint64_t reft_plan_staging_slot_bytes(const reft_plan *p)
{
    return p ? slot_stride(p) : 0;
}

extern "C" int reft_plan_bucket_range(const reft_plan *p, uint64_t b, uint64_t *begin,
                                      uint64_t *end)
{
    if (!p || !begin || !end) return fail(REFT_EINVAL, "reft_plan_bucket_range: null argument");
    if (b >= p->NB) return fail(REFT_EINVAL, "reft_plan_bucket_range: bucket %llu of %llu",
                                (unsigned long long)b, (unsigned long long)p->NB);
    *begin = p->bstart[b];
    *end = p->bstart[b + 1];
    return REFT_OK;
}

extern "C" int reft_plan_tile_info(const reft_plan *p, uint64_t *tile_bytes, uint64_t *ntiles)
{
    if (!p || !tile_bytes || !ntiles) return fail(REFT_EINVAL, "reft_plan_tile_info: null argument");
    *tile_bytes = 1ull << p->tile_shift;
    *ntiles = p->ntiles;
    return REFT_OK;
}

extern "C" int reft_plan_tile_first_span(const reft_plan *p, uint64_t t, uint64_t *span)
{
    if (!p || !span) return fail(REFT_EINVAL, "reft_plan_tile_first_span: null argument");
    if (t >= p->ntiles) return fail(REFT_EINVAL, "reft_plan_tile_first_span: tile out of range");
    *span = p->first[t];
    return REFT_OK;
}

extern "C" int reft_plan_span_offset(const reft_plan *p, uint64_t t, uint64_t *offset)
{
    if (!p || !offset) return fail(REFT_EINVAL, "reft_plan_span_offset: null argument");
    if (t > p->T) return fail(REFT_EINVAL, "reft_plan_span_offset: span out of range");
    *offset = p->off[t];
    return REFT_OK;
}

extern "C" int reft_plan_split(const reft_plan *p, double t_bubble, double t_ss, uint64_t *cut)
{
    if (!p || !cut) return fail(REFT_EINVAL, "reft_plan_split: null argument");
    if (!(t_ss > 0.0) || !(t_bubble >= 0.0))
        return fail(REFT_EINVAL, "reft_plan_split: need t_ss > 0 and t_bubble >= 0");
    const long double x = (long double)p->L * ((long double)t_bubble / (long double)t_ss);
    *cut = x >= (long double)p->L ? p->L : (uint64_t)x;   // floor, clamped to L
    return REFT_OK;
}

extern "C" int reft_plan_staged_work(reft_plan *p, uint64_t *gather_launches, uint64_t *copies)
{
    REFT_GUARD_BEGIN
    if (!p || !gather_launches || !copies)
        return fail(REFT_EINVAL, "reft_plan_staged_work: null argument");
    const PieceLists &pl = pieces_of(p, 0, p->NB);
    *gather_launches = pl.runs.size();
    *copies = pl.runs.size() + pl.dmas.size();
    return REFT_OK;
    REFT_GUARD_END("reft_plan_staged_work")
}

extern "C" int reft_plan_burst_stats(reft_plan *p, uint64_t stats[4])
{
    int rc = check_plan(p, "reft_plan_burst_stats");
    if (rc) return rc;
    if (!stats) return fail(REFT_EINVAL, "reft_plan_burst_stats: null argument");
    stats[0] = stats[1] = stats[2] = stats[3] = 0;
    if (p->burst_next == 0) return REFT_OK;              // no burst launch on this plan yet
    const uint32_t slot = (p->burst_next - 1) % kCtrBlocks;
    const uint32_t *blk = p->burst_ctr + (size_t)slot * (kBurstCtrBytes / sizeof(uint32_t));
    uint32_t w[4] = {0, 0, 0, 0};
    HIPCHK(hipDeviceSynchronize());                      // a diagnostic: the launch must have ended
    HIPCHK(hipMemcpy(w, blk + kBurstDiagWord, 3 * sizeof(uint32_t), hipMemcpyDeviceToHost));
    HIPCHK(hipMemcpy(w + 3, blk + 8 * 64, sizeof(uint32_t), hipMemcpyDeviceToHost));
    for (int i = 0; i < 4; ++i) stats[i] = w[i];
    return REFT_OK;
}

// ------------------------------------------------------------------------------------------------
// how the bytes of a bucket range travel between the tensors and the host (staged transport)
// ------------------------------------------------------------------------------------------------
// A span of at least dma_min bytes (in the range) needs no kernel: the runtime's copy engines move it
// between the tensor and the host buffer in one copy, wherever bucket boundaries fall, which costs
// kernels running beside it next to nothing.  Smaller spans are worth copies of their own only when
// few of them lie together; a run of at least gather_min consecutive pieces of them inside one
// bucket is gathered into a staging slot by one kernel launch and leaves as one copy.  What is not
// gathered needs no slot, so a copy goes on over a bucket's end (spans of 0.9 MB in buckets of 64 KiB,
// 270 MB: 7.6 ms, a copy per bucket and span 45 ms).
//
// Where the line lies: a copy costs 9.3 us on the link beside its bytes, as much as 530 KB (spans of
// 64 KiB, 256 KiB, 1 MiB, 4 MiB one by one: 6.3, 18.6, 37.5, 50.1 GB/s; gathered: 54.8 at all sizes), and a span that is
// copied between smaller ones ends their run, whose next part has a kernel and a copy of its own.  Gathering a span of 1 MiB
// costs the device 0.4 us and kernels beside it up to 2.  us, spans copied from 1 / 2 / 4 / 8 MiB on, alone, and beside a
// loop of GEMMs (and what that loses): 128 MB in 256 spans (log-uniform 64 : 65536) 3941 / 2710 / 2319 / 2319, 13368 /
// 6290 / 3208 / 3209 (639 / 91 / 79 / 86); 460 MB in 2424 10327 / 8343 / 8344 / 8345, 49885 / 12633 / 13369 / 13304 (1772
// / 244 / 328 / 362); but 400 MB in 200 of 1 to 4 MiB 8859 / 8442 / 7244 / 7242, 8876 / 8765 / 11019 / 11283 (220 / 214 /
// 398 / 268).  That is one stream for kernels and copies, beside long GEMMs.  Such states saved and loaded again, copied from 1 / 4
// MiB on, alone, beside GEMMs of 0.13 ms, and of 0.8 ms: 423 MB in 160 on one stream 17767 / 15354, 17912 / 16457, 17934 / 22964;
// on two, as calls beside compute should have, 17896 / 15245, 17980 / 15559, 17946 / 18386 (the GEMMs lose 0.2 to 0.6 ms / 0.3 to
// 0.4 ms).  And seven of them and two smaller ones in turn, 681 MB in 436, on two 31401 / 24735, 37910 / 25408, 76010 / 28372.
// So the line does not depend on a span's neighbours: of copies one stream beside long GEMMs alone would gain.
static void classify_pieces(const reft_plan *p, uint64_t bucket_begin, uint64_t bucket_end,
                            uint64_t dma_min, uint64_t gather_min, std::vector<Run> &runs,
                            std::vector<Dma> &dmas)
{
    if (bucket_begin >= bucket_end) return;
    const uint64_t lo = p->bstart[bucket_begin], hi = p->bstart[bucket_end];
    std::vector<Dma> pending;                            // pieces of small spans, all in bucket b
    auto copy = [&](const Dma &d) {
        if (!dmas.empty() && dmas.back().span == d.span && dmas.back().o + dmas.back().n == d.o)
            dmas.back().n += d.n;
        else
            dmas.push_back(d);
    };
    auto flush = [&]() {
        if (pending.empty()) return;
        if (pending.size() >= gather_min)
            runs.push_back(Run{pending.front().o, pending.back().o + pending.back().n});
        else
            for (const Dma &d : pending) copy(d);
        pending.clear();
    };
    uint64_t b = bucket_begin;
    // the span that owns byte lo: the last one that starts at or before it
    uint64_t i = (uint64_t)(std::upper_bound(p->off.begin(), p->off.end() - 1, lo) - p->off.begin()) - 1;
    for (; i < p->T && p->off[i] < hi; ++i) {
        uint64_t o = p->off[i] < lo ? lo : p->off[i];
        const uint64_t e = p->off[i + 1] < hi ? p->off[i + 1] : hi;
        if (o >= e) continue;                            // no bytes
        if (e - o >= dma_min) {
            flush();
            dmas.push_back(Dma{o, e - o, i});
            continue;
        }
        while (o < e) {
            if (o >= p->bstart[b + 1]) {                 // a run never crosses a bucket
                flush();
                while (o >= p->bstart[b + 1]) ++b;       // o < hi = bstart[bucket_end]
            }
            const uint64_t pe = p->bstart[b + 1] < e ? p->bstart[b + 1] : e;
            pending.push_back(Dma{o, pe - o, i});
            o = pe;
        }
    }
    flush();
}

// The piece lists of buckets [b0, b1) under the current tunables: made once per range and kept
// (the least recently used of kPieceLists ranges goes when another one is asked for).
static const PieceLists &pieces_of(reft_plan *p, uint64_t b0, uint64_t b1)
{
    const uint64_t dma_min = g_dma_min.load(), gather_min = g_gather_min.load();
    for (auto &pl : p->pieces)
        if (pl.b0 == b0 && pl.b1 == b1 && pl.dma_min == dma_min && pl.gather_min == gather_min) {
            pl.tick = ++p->pieces_tick;
            return pl;
        }
    PieceLists *pl = nullptr;
    p->pieces.reserve(kPieceLists);                     // references handed out stay valid
    if (p->pieces.size() < kPieceLists) {
        p->pieces.emplace_back();
        pl = &p->pieces.back();
    } else {
        pl = &p->pieces[0];
        for (auto &q : p->pieces)
            if (q.tick < pl->tick) pl = &q;
        pl->runs.clear();
        pl->dmas.clear();
    }
    pl->b0 = b0;
    pl->b1 = b1;
    pl->dma_min = dma_min;
    pl->gather_min = gather_min;
    pl->tick = ++p->pieces_tick;
    classify_pieces(p, b0, b1, dma_min, gather_min, pl->runs, pl->dmas);
    return *pl;
}

// The piece copies of a call as one hipGraph of memcpy nodes, launched on copy_stream.  A trainer
// snapshots the same tensors into the same host buffer every time, so the graph is built once
// (keyed by direction, host buffer, bucket range and the span pointers) and replayed: the
// runtime then issues the copies without a host call each, and independent nodes may use more
// than one copy engine (2106 copies of 8 KiB ... 11 MiB, 11.8 GB: 52.6 GB/s as stream copies,
// 54.7 as a chain of nodes, 55.6 as independent nodes; one copy of everything: 57.0).  Off by
// default: two such graphs launched on two streams do not run side by side, so a snapshot and a
// restore that should share the link in both directions take turns instead.
constexpr size_t kCopyGraphs = 8;

static int copy_graph(reft_plan *p, const std::vector<Dma> &dmas, hipStream_t cs, bool to_host,
                      const void *host_base, const void *const *span_ptrs, uint64_t mode)
{
    std::vector<uint64_t> key;
    key.reserve(4 + 3 * dmas.size());
    key.push_back(to_host ? 1 : 0);
    key.push_back((uint64_t)(uintptr_t)host_base);
    key.push_back(mode);
    key.push_back(dmas.size());
    for (const Dma &d : dmas) {
        key.push_back(d.o);
        key.push_back(d.n);
        key.push_back((uint64_t)(uintptr_t)span_ptrs[d.span]);
    }
    reft_plan::CopyGraph *hit = nullptr;
    for (auto &g : p->graphs)
        if (g.key == key) hit = &g;
    if (!hit) {
        hipGraph_t graph = nullptr;
        HIPCHK(hipGraphCreate(&graph, 0));
        struct Guard {
            hipGraph_t g;
            ~Guard() { (void)hipGraphDestroy(g); }
        } guard{graph};
        hipGraphNode_t prev = nullptr;
        for (const Dma &d : dmas) {
            uint8_t *dev = (uint8_t *)span_ptrs[d.span] + (d.o - p->off[d.span]);
            uint8_t *host = (uint8_t *)host_base + d.o;
            hipGraphNode_t node = nullptr;
            HIPCHK(hipGraphAddMemcpyNode1D(&node, graph, mode == 2 && prev ? &prev : nullptr,
                                           mode == 2 && prev ? 1 : 0, to_host ? (void *)host : (void *)dev,
                                           to_host ? (const void *)dev : (const void *)host, d.n,
                                           to_host ? hipMemcpyDeviceToHost : hipMemcpyHostToDevice));
            prev = node;
        }
        hipGraphExec_t exec = nullptr;
        HIPCHK(hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0));
        if (p->graphs.size() >= kCopyGraphs) {
            // the least recently used one goes; it may still be running
            size_t lru = 0;
            for (size_t i = 1; i < p->graphs.size(); ++i)
                if (p->graphs[i].used < p->graphs[lru].used) lru = i;
            HIPCHK(hipEventSynchronize(p->graphs[lru].done));
            (void)hipGraphExecDestroy(p->graphs[lru].exec);
            (void)hipEventDestroy(p->graphs[lru].done);
            p->graphs.erase(p->graphs.begin() + (long)lru);
        }
        hipEvent_t done = nullptr;
        HIPCHK(hipEventCreateWithFlags(&done, hipEventDisableTiming));
        p->graphs.push_back(reft_plan::CopyGraph{std::move(key), exec, 0, done});
        hit = &p->graphs.back();
    }
    hit->used = ++p->graph_tick;
    HIPCHK(hipGraphLaunch(hit->exec, cs));
    HIPCHK(hipEventRecord(hit->done, cs));
    return REFT_OK;
}

// Issue the piece copies on copy_stream, or alternately on copy_stream and the plan's helper
// stream (forked from and joined back to copy_stream, so ordering on copy_stream still covers
// every copy): two queues hide the set-up gap between consecutive small copies.
template <typename Issue>
static int issue_piece_copies(reft_plan *p, const std::vector<Dma> &dmas, hipStream_t cs, Issue issue)
{
    int rc;
    const bool two = g_dma_streams.load() == 2 && dmas.size() >= 4;
    if (two) {
        // made with the plan when "dma_streams" was 2 then, else on the first call that wants it
        if (!p->aux) HIPCHK(hipStreamCreateWithFlags(&p->aux, hipStreamNonBlocking));
        if ((rc = record(p->aux_fork, cs))) return rc;
        if ((rc = wait_on(p->aux, p->aux_fork))) return rc;
    }
    for (size_t i = 0; i < dmas.size(); ++i) HIPCHK(issue(dmas[i], (two && (i & 1)) ? p->aux : cs));
    if (two) {
        if ((rc = record(p->aux_join, p->aux))) return rc;
        if ((rc = wait_on(cs, p->aux_join))) return rc;
    }
    return REFT_OK;
}

// ------------------------------------------------------------------------------------------------
// S1 + S2 + S3: snapshot
// ------------------------------------------------------------------------------------------------
// Record the snapshot completion event behind the call's last work.  The event covers every
// snapshot call issued on the plan so far: when the previous call ended on another stream, this
// one's completion also waits (on the device) for that call's.
static int record_pack_done(reft_plan *p, hipStream_t s)
{
    int rc;
    if (p->pack_done.recorded && !same_stream(p->last_pack_stream, s) && (rc = wait_on(s, p->pack_done))) return rc;
    p->last_pack_stream = s;
    return record(p->pack_done, s);
}

static int staging_slots(const reft_plan *p, const void *staging, uint64_t staging_bytes,
                         const char *who, int *nslots)
{
    if (p->NB == 0) {
        *nslots = 1;
        return REFT_OK;
    }
    if (!staging) return fail(REFT_EINVAL, "%s: null staging buffer", who);
    if ((uintptr_t)staging & 255)
        return fail(REFT_EINVAL, "%s: staging buffer must be 256-byte aligned", who);
    const uint64_t n = staging_bytes / slot_stride(p);
    if (n < 1)
        return fail(REFT_ESIZE, "%s: staging has %llu bytes, one slot needs %llu", who,
                    (unsigned long long)staging_bytes, (unsigned long long)slot_stride(p));
    *nslots = n > (uint64_t)kMaxSlots ? kMaxSlots : (int)n;
    return REFT_OK;
}

// Before a staged call puts anything into the ring of slots, on stream s.  Its groups then wait for the events behind the same
// group of calls before, free[g], the first one first.  Before that it waits for what these do not stand for:
//
// A call that had one stream for everything left none behind its slots, but is through where its completion event `done` is.
// (Such calls need no events between their kernels and copies.  Each made the device write its caches back and what was
// behind it wait: 14.7 MB in 256 tensors saved and loaded 578 us with them, 562 without, 2 MB 127 and 111.  A wait for an
// event of the same stream costs nothing there, so none is left out: a handle does not tell whether it is the same.)
//
// Where a ring takes part of the memory of one with groups of another size or at another place, a group's memory may have
// been the other group's.
static int ring_taken(SlotRing &r, hipStream_t s, uint64_t at, uint64_t group_bytes, bool alone, const Event *free, const Event &done)
{
    int rc;
    if (r.alone && (rc = wait_on(s, done))) return rc;
    bool is_known = false, apart = true;
    for (int i = 0; i < r.known; ++i) {
        const SlotRing::Layout &l = r.layout[i];
        if (l.at == at && l.bytes == group_bytes) is_known = true;
        else if (l.at < at + kGroups * group_bytes && at < l.at + kGroups * l.bytes) apart = false;
    }
    if (!is_known) {
        if (!apart || r.known == (int)(sizeof r.layout / sizeof *r.layout)) {
            for (int g = 0; g < kGroups; ++g)
                if ((rc = wait_on(s, free[g]))) return rc;
            r.known = 0;
        }
        r.layout[r.known++] = SlotRing::Layout{at, group_bytes};
    }
    r.alone = alone;
    return REFT_OK;
}

// Where a staged call ends before its completion event is recorded: what it has queued, first work on `first`, then work on
// `second` that waits for it, still uses slots and its pointer table.
struct FailedCall {
    reft_plan *p;
    hipStream_t first, second, reader;        // reader: of the two, the one whose kernels read the table
    Event *filled, *free;
    int entry = 0;
    bool armed = false;

    int done(int rc)
    {
        if (rc == REFT_OK) armed = false;
        return rc;
    }
    ~FailedCall()
    {
        if (!armed) return;
        char text[sizeof g_err];
        memcpy(text, g_err, sizeof text);
        if (first == second || (record(filled[0], first) == REFT_OK && wait_on(second, filled[0]) == REFT_OK))
            for (int g = 0; g < kGroups; ++g)        // (a group that it has not come to may still be an earlier call's)
                if (wait_on(second, free[g]) == REFT_OK) (void)record(free[g], second);
        (void)release_ptrs(p, entry, reader);
        memcpy(g_err, text, sizeof text);
    }
};

// Record the restore completion event, which also stands for the ring of slots' last use (see ring_taken).
static int record_rest_done(reft_plan *p, hipStream_t s)
{
    int rc;
    if (p->rest_ring.alone && !same_stream(p->rest_stream, s) && (rc = wait_on(s, p->rest_done))) return rc;
    p->rest_stream = s;
    return record(p->rest_done, s);
}

// Whether a staged call on one stream moves its bytes, [lo, hi) of the stream, by a kernel across the link, as a direct one
// does.  Of up to 4 MiB that a kernel would gather or scatter in any case, it does so in less time than a copy takes to be
// set up, to wait for that kernel and to move them, and disturbs kernels beside it no more.  us, copies / across the link
// (and what a loop of GEMMs loses to either): saved, 0.5 MB 31 / 15 (6 / 5), 2 MB 57 / 41 (11 / 8), 4 MB 92 / 78 (18 /
// 17), 8 MB 164 / 157 (28 / 51); loaded, 28 / 19 (7 / 5), 54 / 47 (12 / 10), 91 / 79 (20 / 17), 162 / 150 (29 / 40).
constexpr uint64_t kLinkBytes = 4 << 20;
static bool across_link(const std::vector<Run> &runs, uint64_t lo, uint64_t hi)
{
    return !runs.empty() && hi - lo <= kLinkBytes;
}

extern "C" int reft_snapshot_pack_range(reft_plan *p, const void *const *span_ptrs, void *staging,
                                        uint64_t staging_bytes, void *host_dst, uint64_t host_cap,
                                        uint64_t bucket_begin, uint64_t bucket_end,
                                        reft_stream pack_stream, reft_stream copy_stream)
{
    REFT_GUARD_BEGIN
    int rc = check_plan(p, "reft_snapshot_pack");
    if (rc) return rc;
    if (bucket_begin > bucket_end || bucket_end > p->NB)
        return fail(REFT_EINVAL, "reft_snapshot_pack: bucket range [%llu, %llu) outside [0, %llu]",
                    (unsigned long long)bucket_begin, (unsigned long long)bucket_end,
                    (unsigned long long)p->NB);
    if ((rc = check_span_ptrs(p, span_ptrs, 1, "reft_snapshot_pack"))) return rc;
    if (host_cap < p->L)
        return fail(REFT_ESIZE, "reft_snapshot_pack: host buffer holds %llu bytes, stream has %llu",
                    (unsigned long long)host_cap, (unsigned long long)p->L);
    if (p->L && !host_dst) return fail(REFT_EINVAL, "reft_snapshot_pack: null host buffer");
    hipStream_t ps = (hipStream_t)pack_stream, cs = (hipStream_t)copy_stream;
    const PlanTables pt = p->tables();
    const uint64_t *tab = nullptr;
    int entry = 0;

    if (!staging) {
        // Direct path: the gather kernel stores straight into the pinned host buffer over the
        // host link, one launch per bucket, in order on pack_stream.  No staging, no DMA.
        const uint64_t hview = p->L ? device_view_of_host(host_dst) : 0;
        if (p->L && !hview)
            return fail(REFT_EINVAL, "reft_snapshot_pack: host buffer is not mapped for device "
                                     "access (not pinned); pass a staging ring to copy it by DMA");
        if ((rc = upload_ptrs(p, span_ptrs, 1, ps, &tab, &entry))) return rc;
        // Stores across the link: 32 / 48 / 64 workgroups move tensors of 8 MiB at 53.7 / 54.5 / 54.3
        // and of 10 KB at 51.6 / 53.5 / 53.9 GB/s.
        const LaunchCfg cfg = link_cfg(p, 3);
        for (uint64_t b = bucket_begin; b < bucket_end; ++b)
            HIPCHK(launch_gather(pt, tab, 1, false, false, nullptr, hview, p->range(p->bstart[b], p->bstart[b + 1]),
                                 cfg, ps));
        if ((rc = release_ptrs(p, entry, ps))) return rc;
        return record_pack_done(p, ps);
    }

    // Staged transport.  Large pieces go by DMA straight from their tensors; runs of small pieces
    // are gathered into staging slots and leave as one copy each (see classify_pieces).  The slots
    // form two groups that alternate between the streams; the streams meet only once per group
    // (cross-stream events are costly when thousands are in flight).
    int nslots = 1;
    if ((rc = staging_slots(p, staging, staging_bytes, "reft_snapshot_pack", &nslots))) return rc;
    const PieceLists &pl = pieces_of(p, bucket_begin, bucket_end);
    const std::vector<Run> &runs = pl.runs;
    const std::vector<Dma> &dmas = pl.dmas;
    const uint64_t lo = p->bstart[bucket_begin], hi = p->bstart[bucket_end];
    if (uint64_t hview; ps == cs && across_link(runs, lo, hi) &&
                        (hview = device_view_of_host((uint8_t *)host_dst + lo, hi - lo))) {
        if ((rc = upload_ptrs(p, span_ptrs, 1, ps, &tab, &entry))) return rc;
        HIPCHK(launch_gather(pt, tab, 1, false, false, nullptr, hview - lo, p->range(lo, hi), link_cfg(p, 3), ps));
        if ((rc = release_ptrs(p, entry, ps))) return rc;
        return record_pack_done(p, ps);
    }
    const uint64_t stride = slot_stride(p);
    // The tensors are read on both streams.  The caller orders pack_stream behind whatever
    // produced them; copy_stream joins pack_stream here so the same ordering covers its copies.
    if (ps != cs) {
        if ((rc = record(p->pack_begin, ps))) return rc;
        if ((rc = wait_on(cs, p->pack_begin))) return rc;
    }
    FailedCall failed{p, ps, cs, ps, p->pack_filled, p->pack_free};
    if (!runs.empty()) {
        if ((rc = upload_ptrs(p, span_ptrs, 1, ps, &tab, &failed.entry))) return rc;
        failed.armed = true;
        const LaunchCfg cfg = launch_cfg(p);
        const int ngroups = nslots >= kGroups ? kGroups : 1;
        const uint64_t per_group = (uint64_t)(nslots / ngroups);
        const bool alone = ps == cs;                      // one stream, in order by itself
        if ((rc = ring_taken(p->pack_ring, ps, (uint64_t)(uintptr_t)staging, per_group * stride, alone, p->pack_free, p->pack_done)))
            return rc;
        uint64_t batch = 0;
        for (uint64_t r0 = 0; r0 < runs.size(); r0 += per_group, ++batch) {
            const int g = (int)(batch % (uint64_t)ngroups);
            const uint64_t r1 = r0 + per_group < runs.size() ? r0 + per_group : runs.size();
            // the group's previous occupants must have left for the host
            if ((rc = wait_on(ps, p->pack_free[g]))) return rc;
            for (uint64_t r = r0; r < r1; ++r) {
                const uint64_t slot = (uint64_t)g * per_group + (r - r0);
                const uint64_t slot_addr =
                    (uint64_t)(uintptr_t)staging + slot * stride + (runs[r].a & 255);
                HIPCHK(launch_gather(pt, tab, 1, false, false, nullptr, slot_addr - runs[r].a,
                                     p->range(runs[r].a, runs[r].b), cfg, ps));
            }
            if (!alone && ((rc = record(p->pack_filled[g], ps)) || (rc = wait_on(cs, p->pack_filled[g])))) return rc;
            for (uint64_t r = r0; r < r1; ++r) {
                const uint64_t slot = (uint64_t)g * per_group + (r - r0);
                const uint64_t slot_addr =
                    (uint64_t)(uintptr_t)staging + slot * stride + (runs[r].a & 255);
                HIPCHK(hipMemcpyAsync((uint8_t *)host_dst + runs[r].a,
                                      (const void *)(uintptr_t)slot_addr, runs[r].b - runs[r].a,
                                      hipMemcpyDeviceToHost, cs));
            }
            if (!alone && (rc = record(p->pack_free[g], cs))) return rc;
        }
        if ((rc = release_ptrs(p, failed.entry, ps))) return rc;
    }
    const uint64_t gmode = g_graph_copies.load();
    if (gmode && g_dma_streams.load() == 1 && dmas.size() >= 8) {
        if ((rc = copy_graph(p, dmas, cs, true, host_dst, span_ptrs, gmode))) return rc;
    } else if ((rc = issue_piece_copies(p, dmas, cs, [&](const Dma &d, hipStream_t st) {
                   return hipMemcpyAsync((uint8_t *)host_dst + d.o,
                                         (const uint8_t *)span_ptrs[d.span] + (d.o - p->off[d.span]),
                                         d.n, hipMemcpyDeviceToHost, st);
               })))
        return rc;
    // completion: every copy above is on copy_stream, the gathered ones behind their kernels
    return failed.done(record_pack_done(p, cs));
    REFT_GUARD_END("reft_snapshot_pack")
}

extern "C" int reft_snapshot_pack(reft_plan *p, const void *const *span_ptrs, void *staging,
                                  uint64_t staging_bytes, void *host_dst, uint64_t host_cap,
                                  reft_stream pack_stream, reft_stream copy_stream)
{
    return reft_snapshot_pack_range(p, span_ptrs, staging, staging_bytes, host_dst, host_cap, 0,
                                    p ? p->NB : 0, pack_stream, copy_stream);
}

extern "C" int reft_plan_bucket_of(const reft_plan *p, uint64_t offset, uint64_t *bucket)
{
    if (!p || !bucket) return fail(REFT_EINVAL, "reft_plan_bucket_of: null argument");
    if (offset > p->L) return fail(REFT_EINVAL, "reft_plan_bucket_of: offset beyond the stream");
    // number of buckets that end at or before `offset` = index of the bucket holding it
    uint64_t lo = 0, hi = p->NB;
    while (lo < hi) {
        const uint64_t mid = (lo + hi) / 2;
        if (p->bstart[mid + 1] <= offset) lo = mid + 1;
        else hi = mid;
    }
    *bucket = lo;
    return REFT_OK;
}

extern "C" int reft_snapshot_wait(reft_plan *p)
{
    int rc = check_plan(p, "reft_snapshot_wait");
    if (rc) return rc;
    if (p->pack_done.recorded) HIPCHK(hipEventSynchronize(p->pack_done.ev));
    return REFT_OK;
}

extern "C" int reft_snapshot_query(reft_plan *p)
{
    int rc = check_plan(p, "reft_snapshot_query");
    if (rc) return rc;
    if (!p->pack_done.recorded) return 1;
    hipError_t e = hipEventQuery(p->pack_done.ev);
    if (e == hipSuccess) return 1;
    if (e == hipErrorNotReady) return 0;
    return fail(REFT_EHIP, "hipEventQuery failed: %s", hipGetErrorString(e));
}

// ------------------------------------------------------------------------------------------------
// completed / ongoing snapshot pair
// ------------------------------------------------------------------------------------------------
struct reft_ckpt {
    reft_plan *plan = nullptr;
    void *buf[2] = {nullptr, nullptr};
    uint64_t cap = 0;
    // pinned, device-visible: committed[i] = generation whose every byte has landed in buf[i]
    uint64_t *committed = nullptr;
    uint64_t begun[2] = {0, 0};      // generation most recently started in buf[i] (host side)
    uint64_t generation = 0;
    int ongoing = -1;                // buffer of the snapshot in progress, -1 if none
    Event committed_ev[2];           // recorded behind the commit kernel of buf[i]
};

// 1 if a commit has been queued into buffer i and has not landed yet, 0 if not, negative on error.
static int commit_pending(reft_ckpt *c, int i)
{
    if (!c->committed_ev[i].recorded) return 0;
    const hipError_t e = hipEventQuery(c->committed_ev[i].ev);
    if (e == hipSuccess) {
        c->committed_ev[i].recorded = false;
        return 0;
    }
    if (e == hipErrorNotReady) {
        (void)hipGetLastError();
        return 1;
    }
    return fail(REFT_EHIP, "hipEventQuery failed: %s", hipGetErrorString(e));
}

__global__ void k_commit(uint64_t *slot, uint64_t generation)
{
    // runs after every transfer queued before it on its stream; the store is visible to the host
    __hip_atomic_store(slot, generation, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

extern "C" int reft_ckpt_create(reft_plan *p, void *host_buf0, void *host_buf1, uint64_t cap,
                                reft_ckpt **out)
{
    if (!out) return fail(REFT_EINVAL, "reft_ckpt_create: null out");
    *out = nullptr;
    int rc = check_plan(p, "reft_ckpt_create");
    if (rc) return rc;
    if (!host_buf0 || !host_buf1 || host_buf0 == host_buf1)
        return fail(REFT_EINVAL, "reft_ckpt_create: need two distinct host buffers");
    if (cap < p->L) return fail(REFT_ESIZE, "reft_ckpt_create: buffers hold %llu bytes, stream has %llu",
                                (unsigned long long)cap, (unsigned long long)p->L);
    reft_ckpt *c = new (std::nothrow) reft_ckpt;
    if (!c) return fail(REFT_EINVAL, "reft_ckpt_create: out of host memory");
    c->plan = p;
    c->buf[0] = host_buf0;
    c->buf[1] = host_buf1;
    c->cap = cap;
    hipError_t e = hipHostMalloc((void **)&c->committed, 2 * sizeof(uint64_t), hipHostMallocDefault);
    if (e != hipSuccess) {
        delete c;
        return fail(REFT_EHIP, "hipHostMalloc failed: %s", hipGetErrorString(e));
    }
    c->committed[0] = c->committed[1] = 0;
    for (int i = 0; i < 2; ++i)
        if ((rc = make_event(c->committed_ev[i]))) {
            reft_ckpt_destroy(c);
            return rc;
        }
    *out = c;
    return REFT_OK;
}

extern "C" void reft_ckpt_destroy(reft_ckpt *c)
{
    if (!c) return;
    // a commit kernel that is still queued stores into the flags: let it finish first
    for (int i = 0; i < 2; ++i)
        if (c->committed_ev[i].ev) {
            if (c->committed_ev[i].recorded) (void)hipEventSynchronize(c->committed_ev[i].ev);
            (void)hipEventDestroy(c->committed_ev[i].ev);
        }
    if (c->committed) (void)hipHostFree(c->committed);
    delete c;
}

extern "C" int reft_ckpt_wait(reft_ckpt *c)
{
    if (!c) return fail(REFT_EINVAL, "reft_ckpt_wait: null argument");
    for (int i = 0; i < 2; ++i)
        if (c->committed_ev[i].recorded) {
            HIPCHK(hipEventSynchronize(c->committed_ev[i].ev));
            c->committed_ev[i].recorded = false;
        }
    return REFT_OK;
}

static uint64_t committed_of(const reft_ckpt *c, int i)
{
    return __atomic_load_n(&c->committed[i], __ATOMIC_ACQUIRE);
}

// Index of the newest buffer whose snapshot is complete and not being overwritten, or -1.
static int latest_complete(const reft_ckpt *c, uint64_t *gen)
{
    int best = -1;
    uint64_t best_gen = 0;
    for (int i = 0; i < 2; ++i) {
        const uint64_t g = committed_of(c, i);
        if (g != 0 && g == c->begun[i] && g > best_gen) {
            best = i;
            best_gen = g;
        }
    }
    if (gen) *gen = best_gen;
    return best;
}

extern "C" int reft_ckpt_begin(reft_ckpt *c, void **host_dst, uint64_t *generation)
{
    if (!c || !host_dst) return fail(REFT_EINVAL, "reft_ckpt_begin: null argument");
    // While a commit is in flight its buffer is neither complete nor free, and overwriting the
    // other one would leave no complete snapshot should that commit never land.
    for (int i = 0; i < 2; ++i) {
        const int pend = commit_pending(c, i);
        if (pend < 0) return pend;
        if (pend)
            return fail(REFT_EBUSY, "reft_ckpt_begin: the commit of generation %llu has not landed "
                                    "yet (reft_ckpt_wait blocks until it has)",
                        (unsigned long long)c->begun[i]);
    }
    // write into the buffer that does not hold the newest complete snapshot
    const int keep = latest_complete(c, nullptr);
    const int i = keep == 0 ? 1 : 0;
    c->generation += 1;
    c->begun[i] = c->generation;     // from here until its commit lands, buffer i counts as torn
    c->ongoing = i;
    *host_dst = c->buf[i];
    if (generation) *generation = c->generation;
    return REFT_OK;
}

extern "C" int reft_ckpt_commit(reft_ckpt *c, reft_stream stream)
{
    if (!c) return fail(REFT_EINVAL, "reft_ckpt_commit: null argument");
    if (c->ongoing < 0) return fail(REFT_EINVAL, "reft_ckpt_commit: no snapshot was begun");
    int rc = check_plan(c->plan, "reft_ckpt_commit");
    if (rc) return rc;
    hipLaunchKernelGGL(k_commit, dim3(1), dim3(1), 0, (hipStream_t)stream,
                       c->committed + c->ongoing, c->begun[c->ongoing]);
    HIPCHK(hipGetLastError());
    if ((rc = record(c->committed_ev[c->ongoing], (hipStream_t)stream))) return rc;
    c->ongoing = -1;
    return REFT_OK;
}

extern "C" int reft_ckpt_latest(reft_ckpt *c, const void **host_src, uint64_t *generation)
{
    if (!c || !host_src) return fail(REFT_EINVAL, "reft_ckpt_latest: null argument");
    uint64_t g = 0;
    const int i = latest_complete(c, &g);
    *host_src = i < 0 ? nullptr : c->buf[i];
    if (generation) *generation = g;
    return REFT_OK;
}

// ------------------------------------------------------------------------------------------------
// S1 / S7 between device buffers
// ------------------------------------------------------------------------------------------------
extern "C" int reft_pack_device(reft_plan *p, const void *const *span_ptrs, void *dst_dev,
                                uint64_t dst_cap, reft_stream stream)
{
    int rc = check_plan(p, "reft_pack_device");
    if (rc) return rc;
    if ((rc = check_span_ptrs(p, span_ptrs, 1, "reft_pack_device"))) return rc;
    if (dst_cap < p->L) return fail(REFT_ESIZE, "reft_pack_device: destination too small");
    if (p->L == 0) return REFT_OK;
    if (!dst_dev) return fail(REFT_EINVAL, "reft_pack_device: null destination");
    hipStream_t s = (hipStream_t)stream;
    const uint64_t *tab = nullptr;
    int entry = 0;
    if ((rc = upload_ptrs(p, span_ptrs, 1, s, &tab, &entry))) return rc;
    HIPCHK(launch_gather(p->tables(), tab, 1, false, false, nullptr, (uint64_t)(uintptr_t)dst_dev, p->all(),
                         launch_cfg(p), s));
    return release_ptrs(p, entry, s);
}

extern "C" int reft_unpack_device(reft_plan *p, const void *src_dev, uint64_t src_bytes,
                                  void *const *span_ptrs, reft_stream stream)
{
    int rc = check_plan(p, "reft_unpack_device");
    if (rc) return rc;
    if ((rc = check_span_ptrs(p, span_ptrs, 1, "reft_unpack_device"))) return rc;
    if (src_bytes != p->L)
        return fail(REFT_ESIZE, "reft_unpack_device: source has %llu bytes, stream has %llu",
                    (unsigned long long)src_bytes, (unsigned long long)p->L);
    if (p->L == 0) return REFT_OK;
    if (!src_dev) return fail(REFT_EINVAL, "reft_unpack_device: null source");
    hipStream_t s = (hipStream_t)stream;
    const uint64_t *tab = nullptr;
    int entry = 0;
    if ((rc = upload_ptrs(p, span_ptrs, 1, s, &tab, &entry))) return rc;
    HIPCHK(launch_scatter(p->tables(), tab, (uint64_t)(uintptr_t)src_dev, p->all(), launch_cfg(p),
                          s));
    return release_ptrs(p, entry, s);
}

// ------------------------------------------------------------------------------------------------
// S4: parity over span tables
// ------------------------------------------------------------------------------------------------
static BurstCfg burst_cfg(uint32_t *ring, uint32_t slot, int num_cus)
{
    BurstCfg bc;
    bc.ctr = ring + (size_t)slot * (kBurstCtrBytes / sizeof(uint32_t));
    bc.stage_bytes = (uint32_t)g_burst_stage.load();
    bc.wgs_per_cu = (uint32_t)g_burst_wgs.load();
    bc.num_cus = (uint32_t)num_cus;
    bc.max_polls = (uint32_t)g_burst_polls.load();
    bc.nap = (uint32_t)g_burst_nap.load();
    return bc;
}

// The burst kernel walks a stage piece by piece, the stream kernel spreads pieces over its waves: the
// former pays where at most one tile in eight holds a span boundary ("small_pieces" of them).
// Measured for 8 rows, burst / stream kernel: 0.5 GB in spans of 0.2 MB 134 / 107 us, 2 GB in spans
// of 0.9 MB 431 / 405 us.
static bool few_dense_tiles(const reft_plan *p)
{
    const auto &v = p->tile_spans_sorted;
    const uint32_t most = (uint32_t)g_small_pieces.load();
    const uint64_t dense = most ? (uint64_t)(v.end() - std::lower_bound(v.begin(), v.end(), most)) : p->ntiles;
    return dense * 8 <= p->ntiles;
}

// Whether `rows` rows go through the burst kernel: very long rows, few span boundaries.  A launch into tensors
// needs rows four times as long.
static bool burst_applies(const reft_plan *p, uint32_t rows, bool tensors)
{
    return g_burst.load() && p->L / (tensors ? 4 : 1) >= g_burst_min_bytes.load() && rows <= (uint32_t)kMaxSrc &&
           rows >= g_burst_min_rows.load() && few_dense_tiles(p);
}

// Whether some span's result goes to where a source row of the cached table has that very span.  The
// destination is contiguous at vb or, with vb = 0, the table's last row.  The answer depends on these
// addresses alone, so it is kept with the table.
static bool in_place(reft_plan *p, int entry, uint64_t vb)
{
    PtrEntry &e = p->ring[entry];
    if (e.in_place >= 0 && e.in_place_vb == vb) return e.in_place != 0;
    const uint64_t T = p->T, *row = p->h_ptr + e.pos;
    const uint64_t *const end = row + e.len - (vb ? 0 : T), *const dst = vb ? nullptr : end;
    e.in_place = 0;
    e.in_place_vb = vb;
    for (; row < end; row += T)
        for (uint64_t t = 0; t < T; ++t)
            if (row[t] == (dst ? dst[t] : vb + p->off[t]) && p->off[t + 1] != p->off[t]) e.in_place = 1;
    return e.in_place != 0;
}

// The XOR passes over a device table of `nrows` rows of span pointers (row stride T of plan p)
// into a contiguous destination or, if dtab is given, into the destination's own spans (dst_row
// is the host copy of that row, used to decide which kernel applies).  More than kMaxStreamSrc rows
// are folded in passes.  over_source: the destination is one of the first kMaxStreamSrc rows (the burst
// kernel needs no telling: a stage is read, and a round later written, by one workgroup, every byte
// once).  ctr_ring holds ctr_blocks blocks of burst counters; *ctr_next picks one.
static int xor_passes(reft_plan *p, const uint64_t *tab, uint32_t nrows, const uint64_t *dtab,
                      const void *const *dst_row, void *dst_contig, bool over_source, uint32_t *ctr_ring,
                      uint32_t ctr_blocks, uint32_t *ctr_next, hipStream_t s)
{
    const uint64_t T = p->T;
    const LaunchCfg cfg = launch_cfg(p);
    const PlanTables pt = p->tables();
    // Very long rows: reads and writes are separated in time with the burst kernel.  Destination spans that are not
    // all aligned alike relative to their stream offsets, which its staging image cannot represent, keep the stream
    // kernel, and more rows go through it in one pass, up to kMaxStreamSrc.
    bool burst = burst_applies(p, nrows, dst_row != nullptr);
    uint64_t vb = (uint64_t)(uintptr_t)dst_contig;
    if (burst && dst_row) {
        bool have = false;
        for (uint64_t t = 0; t < T && burst; ++t) {
            if (p->off[t + 1] == p->off[t]) continue;
            const uint64_t c = ((uint64_t)(uintptr_t)dst_row[t] - p->off[t]) & 15u;
            if (!have) { vb = c; have = true; }
            else burst = c == vb;
        }
    }
    if (burst) {
        const BurstCfg bc = burst_cfg(ctr_ring, (*ctr_next)++ % ctr_blocks, p->num_cus);
        HIPCHK(launch_gather_burst(pt, tab, (int)nrows, dtab, vb, 0, p->L, cfg, bc, s));
        return REFT_OK;
    }
    for (uint32_t done = 0; done < nrows;) {
        const bool acc = done > 0;
        const uint32_t cap = (uint32_t)kMaxStreamSrc - (acc ? 1u : 0u);
        const uint32_t n = nrows - done < cap ? nrows - done : cap;
        HIPCHK(launch_gather(pt, tab + (uint64_t)done * T, (int)n, acc, over_source, dtab,
                             (uint64_t)(uintptr_t)dst_contig, p->all(), cfg, s));
        done += n;
    }
    return REFT_OK;
}

// XOR of `nrows` rows of a table in the plan's cache into a contiguous destination or, with `tensors`, into the spans of
// the table's last row.  apart: a contiguous destination overlaps no source, by the entry point's rules.
static int xor_table(reft_plan *p, int entry, const uint64_t *tab, uint32_t nrows, bool tensors, void *dst_contig, bool apart,
                     hipStream_t s)
{
    int rc;
    const uint64_t at = (uint64_t)nrows * p->T;
    const void *const *dst_row = tensors ? (const void *const *)(p->h_ptr + p->ring[entry].pos + at) : nullptr;
    const bool over_source = (tensors || !apart) && in_place(p, entry, (uint64_t)(uintptr_t)dst_contig);
    if ((rc = xor_passes(p, tab, nrows, tensors ? tab + at : nullptr, dst_row, dst_contig, over_source, p->burst_ctr,
                         kCtrBlocks, &p->burst_next, s)))
        return rc;
    return release_ptrs(p, entry, s);
}

// The same of host rows, which are uploaded as one table through the plan's cache; dst_row: the tensors, or null (rows and
// dst_row may lie in the plan's row_buf).
static int xor_rows(reft_plan *p, const void *const *rows, uint32_t nrows, const void *const *dst_row,
                    void *dst_contig, bool apart, hipStream_t s, int *used = nullptr)
{
    int rc;
    const uint64_t T = p->T;
    const uint64_t *tab = nullptr;
    int entry = 0;
    if (dst_row) {
        // one table: the source rows, then the destination row
        const void **all = p->row_buf.data();
        if (rows != all) std::copy(rows, rows + (size_t)nrows * T, all);
        if (dst_row != all + (size_t)nrows * T) std::copy(dst_row, dst_row + T, all + (size_t)nrows * T);
        if ((rc = upload_ptrs(p, all, nrows + 1, s, &tab, &entry))) return rc;
    } else {
        if ((rc = upload_ptrs(p, rows, nrows, s, &tab, &entry))) return rc;
    }
    if (used) *used = entry;
    return xor_table(p, entry, tab, nrows, dst_row != nullptr, dst_contig, apart, s);
}

extern "C" int reft_parity_encode(reft_plan *p, const void *const *shard_span_ptrs, uint32_t k,
                                  void *parity_dev, reft_stream stream)
{
    REFT_GUARD_BEGIN
    int rc = check_plan(p, "reft_parity_encode");
    if (rc) return rc;
    if (k < 1 || k > REFT_MAX_K)
        return fail(REFT_EINVAL, "reft_parity_encode: k = %u outside [1, %d]", k, REFT_MAX_K);
    if ((rc = check_span_ptrs(p, shard_span_ptrs, k, "reft_parity_encode"))) return rc;
    if (p->L == 0) return REFT_OK;
    if (!parity_dev) return fail(REFT_EINVAL, "reft_parity_encode: null parity buffer");
    return xor_rows(p, shard_span_ptrs, k, nullptr, parity_dev, true, (hipStream_t)stream);
    REFT_GUARD_END("reft_parity_encode")
}

// S1 + S4 in one pass: the parity of the k shards and the packed stream of shard `own`.
extern "C" int reft_parity_encode_pack(reft_plan *p, const void *const *shard_span_ptrs, uint32_t k,
                                       uint32_t own, void *parity_dev, void *packed_dev,
                                       uint64_t packed_cap, reft_stream stream)
{
    REFT_GUARD_BEGIN
    int rc = check_plan(p, "reft_parity_encode_pack");
    if (rc) return rc;
    if (k < 1 || k > REFT_MAX_K)
        return fail(REFT_EINVAL, "reft_parity_encode_pack: k = %u outside [1, %d]", k, REFT_MAX_K);
    if (own >= k) return fail(REFT_EINVAL, "reft_parity_encode_pack: own = %u but k = %u", own, k);
    if ((rc = check_span_ptrs(p, shard_span_ptrs, k, "reft_parity_encode_pack"))) return rc;
    if (packed_cap < p->L) return fail(REFT_ESIZE, "reft_parity_encode_pack: packed buffer too small");
    if (p->L == 0) return REFT_OK;
    if (!parity_dev || !packed_dev)
        return fail(REFT_EINVAL, "reft_parity_encode_pack: null parity or packed buffer");
    hipStream_t s = (hipStream_t)stream;
    const uint64_t T = p->T;
    // the own shard's row first: the fused kernel packs the first row it reads
    const void **rows = p->row_buf.data();
    std::copy(shard_span_ptrs + (size_t)own * T, shard_span_ptrs + (size_t)(own + 1) * T, rows);
    for (uint32_t j = 0, r = 1; j < k; ++j)
        if (j != own) {
            std::copy(shard_span_ptrs + (size_t)j * T, shard_span_ptrs + (size_t)(j + 1) * T,
                      rows + (size_t)r * T);
            ++r;
        }
    const LaunchCfg cfg = launch_cfg(p);
    const uint64_t vb = (uint64_t)(uintptr_t)parity_dev, vb2 = (uint64_t)(uintptr_t)packed_dev;
    const uint64_t *tab = nullptr;
    int entry = 0;
    if ((rc = upload_ptrs(p, rows, k, s, &tab, &entry))) return rc;
    if (k <= (uint32_t)kMaxStreamSrc) {
        // TB/s over (k + 2) L bytes, this / a write-burst kernel with two images: 8 rows of 15.0 GB 6.08 / 6.02,
        // of 11.8 GB 6.37 / 6.33, of 2.4 GB 6.24 / 6.14, of 0.6 GB 6.21 / 5.93; 5 rows 6.33 / 5.66; two
        // launches 5.6
        HIPCHK(launch_gather_pack(p->tables(), tab, (int)k, vb, vb2, p->all(), cfg, s));
    } else {
        if ((rc = xor_passes(p, tab, k, nullptr, nullptr, parity_dev, false, p->burst_ctr,
                             kCtrBlocks, &p->burst_next, s)))
            return rc;
        HIPCHK(launch_gather(p->tables(), tab, 1, false, false, nullptr, vb2, p->all(), cfg, s));
    }
    return release_ptrs(p, entry, s);
    REFT_GUARD_END("reft_parity_encode_pack")
}

// ------------------------------------------------------------------------------------------------
// S4 for callers that cannot allocate
// ------------------------------------------------------------------------------------------------
namespace {
constexpr uint32_t kPtrChunk = 256;
struct PtrChunk {
    uint64_t p[kPtrChunk];
};
}  // namespace

// Pointers travel to the device as kernel arguments, 256 at a time: no pinned staging, nothing the
// call would have to keep alive, and the launch is an ordinary kernel node for a capturing caller.
__global__ void k_store_ptrs(uint64_t *dst, PtrChunk c, uint32_t n)
{
    if (threadIdx.x < n) dst[threadIdx.x] = c.p[threadIdx.x];
}

extern "C" int reft_parity_encode_noalloc(reft_plan *p, const void *const *shard_span_ptrs,
                                          uint32_t k, void *parity_dev, reft_stream stream)
{
    int rc = check_plan(p, "reft_parity_encode_noalloc");
    if (rc) return rc;
    if (k < 1 || k > REFT_MAX_K)
        return fail(REFT_EINVAL, "reft_parity_encode_noalloc: k = %u outside [1, %d]", k, REFT_MAX_K);
    const uint64_t n = (uint64_t)k * p->T;
    if (n > kScratchPtrs)
        return fail(REFT_ESIZE, "reft_parity_encode_noalloc: k * T = %llu span pointers, the static "
                                "scratch holds %u", (unsigned long long)n, kScratchPtrs);
    if ((rc = check_span_ptrs(p, shard_span_ptrs, k, "reft_parity_encode_noalloc"))) return rc;
    if (p->L == 0) return REFT_OK;
    if (!parity_dev) return fail(REFT_EINVAL, "reft_parity_encode_noalloc: null parity buffer");
    if (!p->scratch) return fail(REFT_EINVAL, "reft_parity_encode_noalloc: no static scratch on this GPU");
    hipStream_t s = (hipStream_t)stream;
    // p->scratch is the device address of `scratch` on the plan's GPU (hipGetSymbolAddress at plan
    // creation): the pointer table first, one block of burst counters behind it.  The table is
    // overwritten here and the counters are cleared by a kernel before each burst launch, so
    // nothing of an earlier call survives into this one.
    uint64_t *tab = (uint64_t *)p->scratch;
    uint32_t *ctr = (uint32_t *)(p->scratch + kScratchPtrBytes);
    for (uint64_t i = 0; i < n; i += kPtrChunk) {
        PtrChunk c;
        const uint32_t m = (uint32_t)(n - i < kPtrChunk ? n - i : kPtrChunk);
        for (uint32_t j = 0; j < m; ++j) c.p[j] = (uint64_t)(uintptr_t)shard_span_ptrs[i + j];
        for (uint32_t j = m; j < kPtrChunk; ++j) c.p[j] = 0;
        hipLaunchKernelGGL(k_store_ptrs, dim3(1), dim3(kPtrChunk), 0, s, tab + i, c, m);
        HIPCHK(hipGetLastError());
    }
    uint32_t next = 0;
    return xor_passes(p, tab, k, nullptr, nullptr, parity_dev, false, ctr, 1, &next, s);
}

// ------------------------------------------------------------------------------------------------
// rotated placement of the parity (section 4.2): every member protects one segment of every other
// ------------------------------------------------------------------------------------------------
namespace {
// One operand of a rotated XOR over len bytes: the bytes at stream offsets [w, w + len) of member
// `of`'s shard (bytes at or beyond L read as zero) or of the output, or the first len bytes of
// member `of`'s parity unit.
struct WinSpec {
    bool contig;
    uint32_t of;
    uint64_t w;
};
// One XOR: as many windows of len bytes as every other segment of the same derived plan has.
struct Segment {
    uint64_t len;
    std::vector<WinSpec> wins;
};
}  // namespace

static uint32_t rot_index(uint32_t i, uint32_t j) { return i < j ? i : i - 1; }

extern "C" uint64_t reft_segment_bytes(const reft_plan *p, uint32_t k)
{
    return (!p || k < 2) ? 0 : (p->L + (k - 2)) / (k - 1);
}

static int ensure_zeros(reft_plan *p)
{
    if (p->zeros) return REFT_OK;
    HIPCHK(hipMalloc(&p->zeros, 256));
    HIPCHK(hipMemset(p->zeros, 0, 256));
    return REFT_OK;
}

static void add_use(std::vector<PointerRange> &uses, uint32_t of, uint64_t first, uint64_t end)
{
    for (PointerRange &r : uses)
        if (r.of == of) {
            r.first = std::min(r.first, first);
            r.end = std::max(r.end, end);
            return;
        }
    uses.push_back(PointerRange{of, first, end});
}

// The plan whose stream is the segments one after the other and whose spans are the merged pieces of
// their windows (every span boundary of every window becomes a boundary), with the recipe that turns
// the caller's pointers into its rows.  Built on first use and kept in the base plan.
static int derived_plan(reft_plan *p, uint64_t key, const std::vector<Segment> &segs,
                        DerivedPlan **out)
{
    int rc = ensure_zeros(p);
    if (rc) return rc;
    DerivedPlan dp;
    std::vector<uint64_t> sizes;
    std::vector<std::pair<uint32_t, uint64_t>> piece;      // (segment, offset in it) of every piece
    for (uint32_t g = 0; g < segs.size(); ++g) {
        std::vector<uint64_t> cuts{0, segs[g].len};
        for (const WinSpec &win : segs[g].wins) {
            if (win.contig) {
                dp.units.push_back(win.of);
                continue;
            }
            add_use(dp.uses, win.of, (uint64_t)(std::upper_bound(p->off.begin(), p->off.end(), win.w) - p->off.begin()) - 1,
                    (uint64_t)(std::lower_bound(p->off.begin(), p->off.end() - 1, win.w + segs[g].len) - p->off.begin()));
            // span starts strictly inside (w, w + len); off[T] = L makes the end of the stream a
            // boundary too, so the zero extension of the last segment starts on a piece boundary
            auto lo = std::upper_bound(p->off.begin(), p->off.end(), win.w);
            for (; lo != p->off.end() && *lo < win.w + segs[g].len; ++lo) cuts.push_back(*lo - win.w);
        }
        std::sort(cuts.begin(), cuts.end());
        cuts.erase(std::unique(cuts.begin(), cuts.end()), cuts.end());
        for (size_t i = 0; i + 1 < cuts.size(); ++i) {
            sizes.push_back(cuts[i + 1] - cuts[i]);
            piece.emplace_back(g, cuts[i]);
        }
    }
    if ((rc = reft_plan_create(sizes.data(), sizes.size(), nullptr, 0, 0, &dp.plan))) return rc;
    struct Guard {
        reft_plan *d;
        ~Guard() { if (d) reft_plan_destroy(d); }
    } guard{dp.plan};
    dp.plan->windows = true;
    dp.nwin = (uint32_t)segs[0].wins.size();
    dp.recipe.resize((size_t)dp.nwin * sizes.size());
    for (uint32_t q = 0; q < dp.nwin; ++q)
        for (size_t t = 0; t < sizes.size(); ++t) {
            RowRecipe &r = dp.recipe[(size_t)q * sizes.size() + t];
            const WinSpec &win = segs[piece[t].first].wins[q];
            const uint64_t x = piece[t].second, y = win.w + x;
            if (win.contig) {
                r = RowRecipe{kContig, win.of, x};
            } else if (y >= p->L) {                    // zero extension of the last segment
                if (sizes[t] > 256) return fail(REFT_EINVAL, "internal: zero pad too long");
                r = RowRecipe{kZeros, 0, 0};
            } else {
                const uint64_t sp = (uint64_t)(std::upper_bound(p->off.begin(), p->off.end(), y) -
                                               p->off.begin()) - 1;        // off[sp] <= y < off[sp + 1]
                r = RowRecipe{(uint32_t)sp, win.of, y - p->off[sp]};
            }
        }
    guard.d = nullptr;
    auto ins = p->derived.emplace(key, std::move(dp));
    *out = &ins.first->second;
    return REFT_OK;
}

// The derived plan's rows, one after the other in its row_buf, from the caller's pointers.
static int derived_rows(const reft_plan *p, const DerivedPlan &dp, const void *const *shard_span_ptrs,
                        const void *const *parity_ptrs, const void *const *out_span_ptrs)
{
    const void **row = dp.plan->row_buf.data();
    for (const RowRecipe &r : dp.recipe) {
        if (r.span == kContig) {
            *row++ = (const uint8_t *)parity_ptrs[r.of] + r.add;
        } else if (r.span == kZeros) {
            *row++ = p->zeros;
        } else {
            const void *const s = r.of == kOut ? out_span_ptrs[r.span]
                                               : shard_span_ptrs[(size_t)r.of * p->T + r.span];
            if (!s) return fail(REFT_EINVAL, "rotated parity: span %u is null but has bytes", r.span);
            *row++ = (const uint8_t *)s + r.add;
        }
    }
    return REFT_OK;
}

// The pointers that a call was given: the shards' and, of a decode, the parity units and the tensors.
struct CallerPointers {
    const void *const *shards;
    const void *const *parity, *const *out;                // null in an encode
    uint64_t T;

    // each(pointers, count) for every piece that the plan's rows are made of, until one answers false
    template <class Each>
    bool all(const DerivedPlan &dp, Each each) const
    {
        for (const PointerRange &r : dp.uses)
            if (!each((r.of == kOut ? out : shards + r.of * T) + r.first, r.end - r.first)) return false;
        for (uint32_t i : dp.units)
            if (!each(parity + i, 1)) return false;
        return true;
    }
};

// The XOR that a derived plan stands for.  Its rows are many times the caller's pointers, to make, to compare and to keep: so
// these are compared, with those of the last two sets, and where they are the same and their rows still in the derived
// plan's cache, that table is used.  (One unit and one decode, 8 members of 34 MB in 9236 spans: 117 us of host work, 26 so.)
// Of a unit that is a window of each member's pointers.  (All of them compared, a unit of 16 members' 76 MB in 11,490 spans
// took 25 us a call, so 17, and 17 to 33 with its rows made each time.)
static int xor_derived(reft_plan *p, DerivedPlan &dp, const CallerPointers &from, void *dst_contig, hipStream_t s)
{
    int rc;
    reft_plan *d = dp.plan;
    const bool tensors = from.out != nullptr;
    const uint32_t nrows = dp.nwin - (tensors ? 1 : 0);
    for (int i = 0; i < 2; ++i) {
        const int at = dp.last ^ i;
        const SeenPointers &seen = dp.seen[at];
        if (!seen.upload || !d->ring[seen.entry].live || d->ring[seen.entry].upload != seen.upload) continue;
        const void *const *had = seen.ptrs.data();
        if (!from.all(dp, [&](const void *const *ptrs, uint64_t n) {
                const bool same = n == 0 || !memcmp(had, ptrs, n * sizeof *ptrs);
                had += n;
                return same;
            }))
            continue;
        const uint64_t *tab = nullptr;
        dp.last = at;
        if ((rc = use_entry(d, seen.entry, s, &tab))) return rc;
        return xor_table(d, seen.entry, tab, nrows, tensors, dst_contig, false, s);
    }
    if ((rc = derived_rows(p, dp, from.shards, from.parity, from.out))) return rc;
    SeenPointers &seen = dp.seen[dp.last ^= 1];
    seen.upload = 0;
    seen.ptrs.clear();
    from.all(dp, [&](const void *const *ptrs, uint64_t n) {
        seen.ptrs.insert(seen.ptrs.end(), ptrs, ptrs + n);
        return true;
    });
    const void **rows = d->row_buf.data();
    if ((rc = xor_rows(d, rows, nrows, tensors ? rows + (size_t)nrows * d->T : nullptr, dst_contig, false, s, &seen.entry)))
        return rc;
    seen.upload = d->ring[seen.entry].upload;
    return REFT_OK;
}

extern "C" int reft_parity_encode_rotated(reft_plan *p, const void *const *shard_span_ptrs,
                                          uint32_t k, uint32_t member, void *parity_dev,
                                          reft_stream stream)
{
    REFT_GUARD_BEGIN
    int rc = check_plan(p, "reft_parity_encode_rotated");
    if (rc) return rc;
    if (k < 2 || k > REFT_MAX_K)
        return fail(REFT_EINVAL, "reft_parity_encode_rotated: k = %u outside [2, %d]", k, REFT_MAX_K);
    if (member >= k)
        return fail(REFT_EINVAL, "reft_parity_encode_rotated: member = %u but k = %u", member, k);
    if (!shard_span_ptrs) return fail(REFT_EINVAL, "reft_parity_encode_rotated: null pointer array");
    const uint64_t Lseg = reft_segment_bytes(p, k);
    if (Lseg == 0) return REFT_OK;
    if (!parity_dev) return fail(REFT_EINVAL, "reft_parity_encode_rotated: null parity buffer");
    const uint64_t key = (1ull << 56) | ((uint64_t)k << 32) | member;
    DerivedPlan *dp = nullptr;
    auto it = p->derived.find(key);
    if (it != p->derived.end()) {
        dp = &it->second;
    } else {
        Segment seg{Lseg, {}};
        for (uint32_t j = 0; j < k; ++j)
            if (j != member) seg.wins.push_back(WinSpec{false, j, (uint64_t)rot_index(member, j) * Lseg});
        if ((rc = derived_plan(p, key, {seg}, &dp))) return rc;
    }
    return xor_derived(p, *dp, CallerPointers{shard_span_ptrs, nullptr, nullptr, p->T}, parity_dev,
                       (hipStream_t)stream);
    REFT_GUARD_END("reft_parity_encode_rotated")
}

extern "C" int reft_reconstruct_rotated(reft_plan *p, const void *const *shard_span_ptrs,
                                        const void *const *parity_ptrs, uint32_t k, uint32_t lost,
                                        void *const *out_span_ptrs, reft_stream stream)
{
    REFT_GUARD_BEGIN
    int rc = check_plan(p, "reft_reconstruct_rotated");
    if (rc) return rc;
    if (k < 2 || k > REFT_MAX_K)
        return fail(REFT_EINVAL, "reft_reconstruct_rotated: k = %u outside [2, %d]", k, REFT_MAX_K);
    if (lost >= k) return fail(REFT_EINVAL, "reft_reconstruct_rotated: lost = %u but k = %u", lost, k);
    if (!shard_span_ptrs || !parity_ptrs)
        return fail(REFT_EINVAL, "reft_reconstruct_rotated: null pointer array");
    if ((rc = check_span_ptrs(p, out_span_ptrs, 1, "reft_reconstruct_rotated(out)"))) return rc;
    const uint64_t Lseg = reft_segment_bytes(p, k);
    if (Lseg == 0) return REFT_OK;
    for (uint32_t r = 0; r + 1 < k && (uint64_t)r * Lseg < p->L; ++r)
        if (!parity_ptrs[r < lost ? r : r + 1])
            return fail(REFT_EINVAL, "reft_reconstruct_rotated: parity unit of member %u is null",
                        r < lost ? r : r + 1);
    // All segments at once: every one is the XOR of k - 1 operands, so the derived plan's stream is
    // the lost shard's and one launch decodes it (one unit and one decode, 16 members of 842 MB: 5.1 ms
    // with 16 launches of two passes each, 2.46 with one launch for either).
    const uint64_t key = (2ull << 56) | ((uint64_t)k << 32) | lost;
    DerivedPlan *dp = nullptr;
    auto it = p->derived.find(key);
    if (it != p->derived.end()) {
        dp = &it->second;
    } else {
        std::vector<Segment> segs;
        for (uint32_t r = 0; r + 1 < k && (uint64_t)r * Lseg < p->L; ++r) {
            const uint64_t o0 = (uint64_t)r * Lseg;
            const uint32_t i = r < lost ? r : r + 1;      // the member that protects segment r
            // the parity unit, the other segments it covers, and last the destination (its own span
            // boundaries must be piece boundaries too)
            Segment seg{p->L - o0 < Lseg ? p->L - o0 : Lseg, {WinSpec{true, i, 0}}};
            for (uint32_t j = 0; j < k; ++j)
                if (j != i && j != lost)
                    seg.wins.push_back(WinSpec{false, j, (uint64_t)rot_index(i, j) * Lseg});
            seg.wins.push_back(WinSpec{false, kOut, o0});
            segs.push_back(std::move(seg));
        }
        if ((rc = derived_plan(p, key, segs, &dp))) return rc;
    }
    return xor_derived(p, *dp, CallerPointers{shard_span_ptrs, parity_ptrs, (const void *const *)out_span_ptrs, p->T},
                       nullptr, (hipStream_t)stream);
    REFT_GUARD_END("reft_reconstruct_rotated")
}

// ------------------------------------------------------------------------------------------------
// several redundancy strategies at once (section 4.2): which lost members can be recovered, how
// ------------------------------------------------------------------------------------------------
extern "C" int reft_recovery_plan(uint32_t k, const uint32_t *copy_offsets, uint32_t n_copies,
                                  int parity_units, const uint8_t *lost, reft_recovery_step *steps,
                                  uint32_t *nsteps)
{
    if (!lost || !steps || !nsteps) return fail(REFT_EINVAL, "reft_recovery_plan: null argument");
    *nsteps = 0;
    if (k < 2 || k > REFT_MAX_K)
        return fail(REFT_EINVAL, "reft_recovery_plan: k = %u outside [2, %d]", k, REFT_MAX_K);
    if (n_copies && !copy_offsets) return fail(REFT_EINVAL, "reft_recovery_plan: null offsets");
    for (uint32_t a = 0; a < n_copies; ++a)
        if (copy_offsets[a] < 1 || copy_offsets[a] >= k)
            return fail(REFT_EINVAL, "reft_recovery_plan: copy offset %u outside [1, %u)",
                        copy_offsets[a], k);
    uint32_t nlost = 0, stuck = 0, first_stuck = 0;
    for (uint32_t x = 0; x < k; ++x) nlost += lost[x] ? 1u : 0u;
    for (uint32_t x = 0; x < k; ++x) {
        if (!lost[x]) continue;
        bool done = false;
        for (uint32_t a = 0; a < n_copies && !done; ++a) {
            const uint32_t holder = (x + k - copy_offsets[a]) % k;      // holder + d = x (mod k)
            if (lost[holder]) continue;
            steps[(*nsteps)++] = reft_recovery_step{x, REFT_RECOVER_COPY, holder, a};
            done = true;
        }
        // every segment of x is covered by the unit of another member: all of them must be there
        if (!done && parity_units && nlost == 1) {
            steps[(*nsteps)++] = reft_recovery_step{x, REFT_RECOVER_DECODE, 0, 0};
            done = true;
        }
        if (!done && stuck++ == 0) first_stuck = x;
    }
    if (stuck)
        return fail(REFT_EUNRECOVERABLE,
                    "reft_recovery_plan: %u of the %u lost members cannot be recovered (first: "
                    "member %u): no surviving duplicate%s", stuck, nlost, first_stuck,
                    parity_units ? ", and with more than one member lost a parity unit is missing too"
                                 : "");
    return REFT_OK;
}

// ------------------------------------------------------------------------------------------------
// S6: single-loss decode
// ------------------------------------------------------------------------------------------------
extern "C" int reft_reconstruct(const void *const *shards, uint32_t k, const void *parity,
                                uint64_t L, void *out_dev, uint32_t *lost_index,
                                reft_stream stream)
{
    REFT_GUARD_BEGIN
    if (!shards) return fail(REFT_EINVAL, "reft_reconstruct: null shard array");
    if (k < 1 || k > REFT_MAX_K - 1)
        return fail(REFT_EINVAL, "reft_reconstruct: k = %u outside [1, %d]", k, REFT_MAX_K - 1);
    uint32_t nlost = 0, lost = 0;
    for (uint32_t s = 0; s < k; ++s)
        if (!shards[s]) {
            if (nlost == 0) lost = s;
            ++nlost;
        }
    if (nlost >= 2)
        return fail(REFT_EUNRECOVERABLE,
                    "reft_reconstruct: %u of %u shards are lost; one parity decodes one loss",
                    nlost, k);
    if (nlost == 0) return fail(REFT_EINVAL, "reft_reconstruct: no shard is marked lost (NULL)");
    if (lost_index) *lost_index = lost;
    if (L == 0) return REFT_OK;
    if (!parity || !out_dev) return fail(REFT_EINVAL, "reft_reconstruct: null parity or output");

    uint64_t src[REFT_MAX_K];
    uint32_t n = 0;
    src[n++] = (uint64_t)(uintptr_t)parity;
    for (uint32_t s = 0; s < k; ++s)
        if (shards[s]) src[n++] = (uint64_t)(uintptr_t)shards[s];

    const LaunchCfg cfg = launch_cfg(nullptr);
    const uint32_t tile_shift = (uint32_t)g_tile_shift.load();
    hipStream_t st = (hipStream_t)stream;
    BurstCfg bc{};
    const uint64_t min_rows = contig_burst_min_rows(g_burst_min_rows.load());
    const bool burst_ok = g_burst.load() && L >= contig_burst_min_bytes(g_burst_min_bytes.load());
    uint32_t *ring = nullptr;
    int num_cus = 256;
    if (burst_ok) {
        // counter blocks from the ring in the library's static device memory (no allocation)
        const DeviceStatics *ds = nullptr;
        int rc = device_statics(&ds);
        if (rc) return rc;
        ring = ds->ctr;
        num_cus = ds->num_cus;
    }
    static std::atomic<uint32_t> next_slot{0};
    uint32_t done = 0;
    while (done < n) {
        SrcBases b{};
        int m = 0;
        if (done > 0) b.p[m++] = (uint64_t)(uintptr_t)out_dev;     // fold into the partial result
        while (m < kMaxSrc && done < n) b.p[m++] = src[done++];
        if (burst_ok && (uint32_t)m >= min_rows) {
            // reads and writes separated in time; folding in place is safe: a stage of the
            // output is read and, a round later, written by the same workgroup only
            bc = burst_cfg(ring, next_slot++ % kCtrBlocks, num_cus);
            HIPCHK(launch_xor_contig_burst(b, m, (uint64_t)(uintptr_t)out_dev, L, cfg, bc, st));
        } else {
            HIPCHK(launch_xor_contig(b, m, (uint64_t)(uintptr_t)out_dev, L, tile_shift, cfg, st));
        }
    }
    return REFT_OK;
    REFT_GUARD_END("reft_reconstruct")
}

// S6 + S7 in one pass: survivors read in place through their span tables, the parity as a
// contiguous stream, the result written straight into the lost shard's tensors.
extern "C" int reft_reconstruct_spans(reft_plan *p, const void *const *shard_span_ptrs, uint32_t k,
                                      uint32_t lost, const void *parity_dev,
                                      void *const *out_span_ptrs, reft_stream stream)
{
    REFT_GUARD_BEGIN
    int rc = check_plan(p, "reft_reconstruct_spans");
    if (rc) return rc;
    if (k < 1 || k > REFT_MAX_K - 1)
        return fail(REFT_EINVAL, "reft_reconstruct_spans: k = %u outside [1, %d]", k,
                    REFT_MAX_K - 1);
    if (lost >= k) return fail(REFT_EINVAL, "reft_reconstruct_spans: lost = %u but k = %u", lost, k);
    if (!shard_span_ptrs) return fail(REFT_EINVAL, "reft_reconstruct_spans: null pointer array");
    if ((rc = check_span_ptrs(p, out_span_ptrs, 1, "reft_reconstruct_spans(out)"))) return rc;
    // rows: the k-1 survivors, then the parity expressed as a span row
    const uint64_t T = p->T;
    const void **rows = p->row_buf.data();                     // (REFT_MAX_K + 1) * T entries
    uint32_t r = 0;
    for (uint32_t s = 0; s < k; ++s) {
        if (s == lost) continue;
        if ((rc = check_span_ptrs(p, shard_span_ptrs + (size_t)s * T, 1, "reft_reconstruct_spans")))
            return rc;
        for (uint64_t t = 0; t < T; ++t) rows[(size_t)r * T + t] = shard_span_ptrs[(size_t)s * T + t];
        ++r;
    }
    if (p->L == 0) return REFT_OK;
    if (!parity_dev) return fail(REFT_EINVAL, "reft_reconstruct_spans: null parity");
    for (uint64_t t = 0; t < T; ++t)
        rows[(size_t)r * T + t] = (const uint8_t *)parity_dev + p->off[t];
    ++r;                                                       // r == k source rows
    return xor_rows(p, rows, k, (const void *const *)out_span_ptrs, nullptr, false, (hipStream_t)stream);
    REFT_GUARD_END("reft_reconstruct_spans")
}

// ------------------------------------------------------------------------------------------------
// S5 + S7: restore
// ------------------------------------------------------------------------------------------------
extern "C" int reft_restore(reft_plan *p, const void *host_src, uint64_t host_bytes, void *staging,
                            uint64_t staging_bytes, void *const *span_ptrs,
                            reft_stream copy_stream, reft_stream unpack_stream)
{
    REFT_GUARD_BEGIN
    int rc = check_plan(p, "reft_restore");
    if (rc) return rc;
    if ((rc = check_span_ptrs(p, span_ptrs, 1, "reft_restore"))) return rc;
    if (host_bytes != p->L)
        return fail(REFT_ESIZE, "reft_restore: host snapshot has %llu bytes, stream has %llu",
                    (unsigned long long)host_bytes, (unsigned long long)p->L);
    if (p->L && !host_src) return fail(REFT_EINVAL, "reft_restore: null host buffer");
    hipStream_t cs = (hipStream_t)copy_stream, us = (hipStream_t)unpack_stream;
    const PlanTables pt = p->tables();
    const uint64_t *tab = nullptr;
    int entry = 0;

    if (!staging) {
        // Direct path: the scatter kernel loads the snapshot from pinned host memory itself.
        const uint64_t hview = p->L ? device_view_of_host(host_src) : 0;
        if (p->L && !hview)
            return fail(REFT_EINVAL, "reft_restore: host buffer is not mapped for device access "
                                     "(not pinned); pass a staging ring to copy it by DMA");
        if ((rc = upload_ptrs(p, span_ptrs, 1, us, &tab, &entry))) return rc;
        const LaunchCfg cfg = link_cfg(p, 4);   // reads across the link need about twice the waves of writes
        for (uint64_t b = 0; b < p->NB; ++b)
            HIPCHK(launch_scatter(pt, tab, hview, p->range(p->bstart[b], p->bstart[b + 1]), cfg, us));
        if ((rc = release_ptrs(p, entry, us))) return rc;
        return record_rest_done(p, us);
    }

    int nslots = 1;
    if ((rc = staging_slots(p, staging, staging_bytes, "reft_restore", &nslots))) return rc;
    const PieceLists &pl = pieces_of(p, 0, p->NB);
    const std::vector<Run> &runs = pl.runs;
    const std::vector<Dma> &dmas = pl.dmas;
    if (uint64_t hview; us == cs && across_link(runs, 0, p->L) && (hview = device_view_of_host(host_src, p->L))) {
        if ((rc = upload_ptrs(p, span_ptrs, 1, us, &tab, &entry))) return rc;
        HIPCHK(launch_scatter(pt, tab, hview, p->all(), link_cfg(p, 4), us));
        if ((rc = release_ptrs(p, entry, us))) return rc;
        return record_rest_done(p, us);
    }
    const uint64_t stride = slot_stride(p);
    const bool alone = us == cs;                          // one stream, in order by itself
    // The tensors are written on both streams.  The caller orders unpack_stream behind their last
    // use; copy_stream joins unpack_stream here so the same ordering covers its copies.
    if (!alone) {
        if ((rc = record(p->rest_begin, us))) return rc;
        if ((rc = wait_on(cs, p->rest_begin))) return rc;
    }
    // large pieces: straight from the host snapshot into their tensors
    const uint64_t gmode = g_graph_copies.load();
    if (gmode && g_dma_streams.load() == 1 && dmas.size() >= 8) {
        if ((rc = copy_graph(p, dmas, cs, false, host_src, (const void *const *)span_ptrs, gmode)))
            return rc;
    } else if ((rc = issue_piece_copies(p, dmas, cs, [&](const Dma &d, hipStream_t st) {
                   return hipMemcpyAsync((uint8_t *)span_ptrs[d.span] + (d.o - p->off[d.span]),
                                         (const uint8_t *)host_src + d.o, d.n, hipMemcpyHostToDevice,
                                         st);
               })))
        return rc;
    FailedCall failed{p, cs, us, us, p->rest_filled, p->rest_free};
    if (!runs.empty()) {
        if ((rc = upload_ptrs(p, span_ptrs, 1, us, &tab, &failed.entry))) return rc;
        failed.armed = true;
        const LaunchCfg cfg = launch_cfg(p);
        const int ngroups = nslots >= kGroups ? kGroups : 1;
        const uint64_t per_group = (uint64_t)(nslots / ngroups);
        if ((rc = ring_taken(p->rest_ring, cs, (uint64_t)(uintptr_t)staging, per_group * stride, alone, p->rest_free, p->rest_done)))
            return rc;
        uint64_t batch = 0;
        for (uint64_t r0 = 0; r0 < runs.size(); r0 += per_group, ++batch) {
            const int g = (int)(batch % (uint64_t)ngroups);
            const uint64_t r1 = r0 + per_group < runs.size() ? r0 + per_group : runs.size();
            // the group's previous occupants must have been scattered
            if ((rc = wait_on(cs, p->rest_free[g]))) return rc;
            for (uint64_t r = r0; r < r1; ++r) {
                const uint64_t slot = (uint64_t)g * per_group + (r - r0);
                const uint64_t slot_addr =
                    (uint64_t)(uintptr_t)staging + slot * stride + (runs[r].a & 255);
                HIPCHK(hipMemcpyAsync((void *)(uintptr_t)slot_addr,
                                      (const uint8_t *)host_src + runs[r].a, runs[r].b - runs[r].a,
                                      hipMemcpyHostToDevice, cs));
            }
            if (!alone && ((rc = record(p->rest_filled[g], cs)) || (rc = wait_on(us, p->rest_filled[g])))) return rc;
            for (uint64_t r = r0; r < r1; ++r) {
                const uint64_t slot = (uint64_t)g * per_group + (r - r0);
                const uint64_t slot_addr =
                    (uint64_t)(uintptr_t)staging + slot * stride + (runs[r].a & 255);
                HIPCHK(launch_scatter(pt, tab, slot_addr - runs[r].a, p->range(runs[r].a, runs[r].b), cfg, us));
            }
            if (!alone && (rc = record(p->rest_free[g], us))) return rc;
        }
        if ((rc = release_ptrs(p, failed.entry, us))) return rc;
    }
    // completion on unpack_stream: behind the scatter kernels and behind every direct copy
    if (!alone && ((rc = record(p->rest_copied, cs)) || (rc = wait_on(us, p->rest_copied)))) return rc;
    return failed.done(record_rest_done(p, us));
    REFT_GUARD_END("reft_restore")
}

extern "C" int reft_restore_wait(reft_plan *p)
{
    int rc = check_plan(p, "reft_restore_wait");
    if (rc) return rc;
    if (p->rest_done.recorded) HIPCHK(hipEventSynchronize(p->rest_done.ev));
    return REFT_OK;
}

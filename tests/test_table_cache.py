"""The plan's cache of pointer tables without a GPU: the host code of ``reft_api.hip`` as it is, on a HIP runtime that
moves nothing and completes nothing before the host waits for it.  Every call's work on a stream carries a vector
clock, so that an upload into room which a queued kernel may still read, and a kernel that may read a table before it
has arrived, are seen whatever the order in which a GPU would have run them."""
import ctypes
import os
import random
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2310_12670_amd", "csrc")

SOURCE = r"""
#include <hip/hip_runtime_api.h>
#include "reft_internal.hpp"
#include <algorithm>
#include <cstdlib>
#include <cstring>
#include <map>
#include <vector>

using Clock = std::map<uintptr_t, uint64_t>;                 // stream -> number of its last operation that is known
struct Event { Clock clock; };
struct Op { uintptr_t lo, hi, stream; uint64_t index; };

static std::map<uintptr_t, Clock> streams;
static Clock host;                                           // what the host has waited for
static std::vector<Op> reads, uploads, sources;
static uintptr_t current;                                    // the stream of the call under way
static uint64_t races, foreign, events, unpinned;
static const uint64_t *last_tab;                             // the last kernel's rows of pointers, and how many pointers
static uint64_t last_words;
struct Launch { reft::PlanTables pt; reft::StreamRange range; };
static std::vector<Launch> launches;                         // of the stream kernel
static uintptr_t thread;                                     // the calling thread, which hipStreamPerThread's stream is of
static std::map<uintptr_t, size_t> mapped;                   // host memory that kernels see, at its own addresses
struct Access { Op op; bool write; };
static std::vector<Access> accesses;                         // of kernels to contiguous memory, and of copies
static uint64_t clashes, copies;
static int64_t copies_left = -1;                             // copies up to one that fails
static std::map<uintptr_t, size_t> pinned;

static void join(Clock &a, const Clock &b)
{
    for (auto &x : b) a[x.first] = a[x.first] < x.second ? x.second : a[x.first];
}
static uintptr_t id(hipStream_t s) { return s == hipStreamPerThread ? 1000 + thread : (uintptr_t)s; }
static Clock &on(hipStream_t s)
{
    if ((uintptr_t)s != current) ++foreign;
    Clock &c = streams[id(s)];
    join(c, host);
    ++c[id(s)];
    return c;
}
static bool known(Clock &c, const Op &o) { return c[o.stream] >= o.index; }
static void check(const std::vector<Op> &ops, uintptr_t lo, uintptr_t hi, Clock &c)
{
    for (const Op &o : ops)
        if (o.lo < hi && lo < o.hi && !known(c, o)) ++races;
}
static Op op(const void *p, size_t n, hipStream_t s, Clock &c)
{
    return Op{(uintptr_t)p, (uintptr_t)p + n, id(s), c[id(s)]};
}
static void access(uint64_t p, uint64_t n, bool write, hipStream_t s, Clock &c)
{
    const Op o = op((const void *)p, n, s, c);
    for (const Access &a : accesses)
        if (a.op.lo < o.hi && o.lo < a.op.hi && (a.write || write) && !known(c, a.op)) ++clashes;
    accesses.push_back(Access{o, write});
}
// Every unit's span by the look-up table, as a wave finds it, against the unit numbers.
static void look_up_all(const reft::PlanTables &pt)
{
    uint64_t i = 0;
    for (uint64_t u = 0; u < pt.unit_off[pt.T]; ++u) {
        while (pt.unit_off[i + 1] <= u) ++i;
        const uint32_t first = pt.unit_span[u >> pt.unit_shift], at = first & ~reft::kWholeBlock;
        if (first & reft::kWholeBlock ? at != i : at > i || pt.unit_off[at] > u) ++races;
    }
}
static hipError_t kernel(const uint64_t *tab, uint64_t n, const uint64_t *row, uint64_t m, hipStream_t s)
{
    last_tab = tab;
    last_words = n + (row ? m : 0);
    Clock &c = on(s);
    for (auto part : {std::pair<const uint64_t *, uint64_t>{tab, n}, {row, row ? m : 0}}) {
        if (!part.second) continue;
        const Op o = op(part.first, part.second * 8, s, c);
        check(uploads, o.lo, o.hi, c);
        reads.push_back(o);
    }
    return hipSuccess;
}

extern "C" {
void sim_call(uintptr_t s) { current = s; }
void sim_thread(uintptr_t t) { thread = t; }
void sim_map(uintptr_t p, size_t n) { mapped[p] = n; }
void sim_fail(int64_t copies) { copies_left = copies; }
uint64_t sim_clashes() { return clashes; }                   // accesses to the same memory that nothing keeps in order
uint64_t sim_races() { return races; }
uint64_t sim_uploads() { return uploads.size(); }
uint64_t sim_copies() { return copies; }
uint64_t sim_table(uint64_t *out)                            // what the last kernel's table was uploaded from
{
    for (size_t i = uploads.size(); i-- > 0;)
        if (uploads[i].lo <= (uintptr_t)last_tab && (uintptr_t)last_tab < uploads[i].hi) {
            memcpy(out, (const void *)(sources[i].lo + ((uintptr_t)last_tab - uploads[i].lo)), last_words * 8);
            return last_words;
        }
    return 0;
}
uint64_t sim_foreign() { return foreign; }
uint64_t sim_events() { return events; }

hipError_t hipMemcpyAsync(void *d, const void *h, size_t n, hipMemcpyKind, hipStream_t s)
{
    ++copies;
    if (copies_left >= 0 && copies_left-- == 0) return hipErrorNotSupported;
    Clock &c = on(s);
    access((uint64_t)h, n, false, s, c);
    access((uint64_t)d, n, true, s, c);
    const Op to = op(d, n, s, c), from = op(h, n, s, c);
    check(reads, to.lo, to.hi, c);
    check(uploads, to.lo, to.hi, c);
    auto it = pinned.upper_bound(from.lo);                   // the host has just written there
    if (it != pinned.begin() && from.lo < (--it)->first + it->second) check(sources, from.lo, from.hi, host);
    uploads.push_back(to);
    sources.push_back(from);
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { *e = (hipEvent_t) new Event; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t e) { delete (Event *)e; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) { ++events; ((Event *)e)->clock = on(s); return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t e) { join(host, ((Event *)e)->clock); return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t e)
{
    for (auto &x : ((Event *)e)->clock)
        if (host[x.first] < x.second) return hipErrorNotReady;
    return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) { join(on(s), ((Event *)e)->clock); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) { join(host, streams[id(s)]); return hipSuccess; }
hipError_t hipDeviceSynchronize() { for (auto &x : streams) join(host, x.second); return hipSuccess; }
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode *) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *, unsigned) { return hipErrorNotSupported; }
hipError_t hipStreamDestroy(hipStream_t) { return hipErrorNotSupported; }
hipError_t hipMalloc(void **p, size_t n) { *p = malloc(n); return hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { pinned[(uintptr_t)(*p = malloc(n))] = n; return hipSuccess; }
// the tables of a freed plan are gone: what reads or fills them has to be known by then
static hipError_t release(void *p) { free(p); return hipSuccess; }
hipError_t hipFree(void *p) { return release(p); }
hipError_t hipHostFree(void *p) { pinned.erase((uintptr_t)p); return release(p); }
uint64_t sim_unpinned() { return unpinned; }
uint64_t sim_unfinished()                                    // accesses that the host does not know to have ended
{
    uint64_t n = 0;
    for (const Access &a : accesses) n += !known(host, a.op);
    return n;
}
uint64_t sim_end()                                           // operations that the host does not know to have ended
{
    uint64_t n = 0;
    for (auto *ops : {&reads, &uploads})
        for (const Op &o : *ops) n += !known(host, o);
    streams.clear(), host.clear(), reads.clear(), uploads.clear(), sources.clear(), launches.clear(), accesses.clear(), mapped.clear();
    races = foreign = events = unpinned = clashes = thread = 0;
    copies_left = -1;
    return n;
}
hipError_t hipMemcpy(void *d, const void *h, size_t n, hipMemcpyKind)
{
    auto it = pinned.upper_bound((uintptr_t)h);
    if (it == pinned.begin() || (uintptr_t)h + n > (--it)->first + it->second) ++unpinned;
    memcpy(d, h, n);
    return hipSuccess;
}
hipError_t hipMemset(void *, int, size_t) { return hipSuccess; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *p, int) { memset(p, 0, sizeof *p); return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "no GPU"; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipGetSymbolAddress(void **p, const void *) { static char x[1 << 20]; *p = x; return hipSuccess; }
hipError_t hipMemGetAddressRange(hipDeviceptr_t *base, size_t *n, hipDeviceptr_t p)
{
    auto it = mapped.upper_bound((uintptr_t)p);
    if (it == mapped.begin() || (uintptr_t)p >= (--it)->first + it->second) return hipErrorInvalidValue;
    *base = (hipDeviceptr_t)it->first;
    *n = it->second;
    return hipSuccess;
}
hipError_t hipHostGetDevicePointer(void **d, void *h, unsigned)
{
    size_t n;
    *d = h;
    return hipMemGetAddressRange(&h, &n, h);
}
hipError_t hipGraphAddMemcpyNode1D(hipGraphNode_t *, hipGraph_t, const hipGraphNode_t *, size_t, void *, const void *, size_t,
                                   hipMemcpyKind) { return hipErrorNotSupported; }
hipError_t hipGraphCreate(hipGraph_t *, unsigned) { return hipErrorNotSupported; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipErrorNotSupported; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipErrorNotSupported; }
hipError_t hipGraphInstantiate(hipGraphExec_t *, hipGraph_t, hipGraphNode_t *, char *, size_t) { return hipErrorNotSupported; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipErrorNotSupported; }
hipError_t hipLaunchKernel(const void *, dim3, dim3, void **, size_t, hipStream_t) { return hipErrorNotSupported; }
hipError_t __hipPopCallConfiguration(dim3 *, dim3 *, size_t *, hipStream_t *) { return hipErrorNotSupported; }
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipErrorNotSupported; }
void **__hipRegisterFatBinary(const void *) { return nullptr; }
void __hipRegisterFunction(void **, const void *, char *, const char *, unsigned, void *, void *, void *, void *, int *) {}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
void __hipUnregisterFatBinary(void **) {}
char __hip_fatbin[1];
}

namespace reft {
hipError_t launch_gather(const PlanTables &pt, const uint64_t *tab, int nrows, bool, bool, const uint64_t *dtab, uint64_t vb,
                         const StreamRange &r, const LaunchCfg &, hipStream_t s)
{
    launches.push_back(Launch{pt, r});
    look_up_all(pt);
    kernel(tab, nrows * pt.T, dtab, pt.T, s);
    if (!dtab) access(vb + r.lo, r.hi - r.lo, true, s, on(s));
    return hipSuccess;
}
hipError_t launch_gather_pack(const PlanTables &pt, const uint64_t *tab, int nrows, uint64_t, uint64_t, const StreamRange &,
                              const LaunchCfg &, hipStream_t s) { return kernel(tab, nrows * pt.T, nullptr, 0, s); }
hipError_t launch_gather_burst(const PlanTables &pt, const uint64_t *tab, int nrows, const uint64_t *dtab, uint64_t, uint64_t,
                               uint64_t, const LaunchCfg &, const BurstCfg &, hipStream_t s) { return kernel(tab, nrows * pt.T, dtab, pt.T, s); }
hipError_t launch_scatter(const PlanTables &pt, const uint64_t *tab, uint64_t vb, const StreamRange &r, const LaunchCfg &, hipStream_t s)
{
    launches.push_back(Launch{pt, r});
    kernel(tab, pt.T, nullptr, 0, s);
    access(vb + r.lo, r.hi - r.lo, false, s, on(s));
    return hipSuccess;
}
hipError_t launch_xor_contig(const SrcBases &, int, uint64_t, uint64_t, uint32_t, const LaunchCfg &, hipStream_t) { return hipSuccess; }
hipError_t launch_xor_contig_burst(const SrcBases &, int, uint64_t, uint64_t, const LaunchCfg &, const BurstCfg &, hipStream_t) { return hipSuccess; }
}
"""

SIZES = [4096, 17, 0, 70_000, 1 << 20]
T, L = len(SIZES), sum(SIZES)
BUF = 1 << 40


def compile_with(runtime_source, d):
    (d / "runtime.cpp").write_text(runtime_source)
    api, runtime, so = str(d / "api.o"), str(d / "runtime.o"), str(d / "lib.so")
    subprocess.run(["hipcc", "--offload-host-only", "--offload-arch=gfx950", "-fuse-cuid=none", "-O1", "-std=c++17", "-fPIC",
                    "-c", "-o", api, os.path.join(CSRC, "reft_api.hip")], check=True)
    subprocess.run(["g++", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + CSRC, "-O1", "-std=c++17", "-fPIC", "-w",
                    "-c", "-o", runtime, str(d / "runtime.cpp")], check=True)
    subprocess.run(["g++", "-shared", "-Wl,-Bsymbolic", "-o", so, api, runtime], check=True)
    lib = ctypes.CDLL(so)
    p, u32, u64 = ctypes.c_void_p, ctypes.c_uint32, ctypes.c_uint64
    lib.reft_plan_create.argtypes = [p, u64, p, u64, u64, p]
    lib.reft_plan_destroy.argtypes = [p]
    lib.reft_pack_device.argtypes = [p, p, p, u64, p]
    lib.reft_parity_encode.argtypes = [p, p, u32, p, p]
    lib.reft_reconstruct_spans.argtypes = [p, p, u32, u32, p, p, p]
    lib.reft_last_error.restype = ctypes.c_char_p
    lib.sim_call.argtypes = [p]
    for f in (lib.sim_races, lib.sim_foreign, lib.sim_events, lib.sim_end, lib.sim_unpinned):
        f.restype = u64
    return lib


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return compile_with(SOURCE, tmp_path_factory.mktemp("table_cache"))


class Calls:
    """A plan and calls on it; set `i` of pointers differs from every other set."""

    def __init__(self, lib, sizes=SIZES):
        self.lib, self.plan, self.spans = lib, ctypes.c_void_p(), len(sizes)
        lib.sim_end()
        sizes = (ctypes.c_uint64 * len(sizes))(*sizes)
        assert lib.reft_plan_create(sizes, len(sizes), None, 0, 0, ctypes.byref(self.plan)) == 0, lib.reft_last_error()

    def pointers(self, rows, i):
        row = np.zeros((rows, self.spans), np.uint64)      # (empty spans have null pointers)
        row[:, :T] = (1 << 44) + (i << 32) + (np.arange(rows)[:, None] << 24) + (np.arange(T) << 21)
        return (ctypes.c_void_p * row.size).from_buffer(row)

    def rows(self, n, i, stream):
        """A call whose table has n rows: a pack, an encode of n shards or, from 34 on, a decode of n - 33 into tensors."""
        self.lib.sim_call(stream)
        if n == 1:
            rc = self.lib.reft_pack_device(self.plan, self.pointers(1, i), BUF, L, stream)
        elif n < 34:
            rc = self.lib.reft_parity_encode(self.plan, self.pointers(n, i), n, BUF, stream)
        else:
            k = n - 33
            rc = self.lib.reft_reconstruct_spans(self.plan, self.pointers(k, i), k, 0, BUF, self.pointers(1, i + 100), stream)
        assert rc == 0, self.lib.reft_last_error()
        assert self.lib.sim_races() == 0
        assert self.lib.sim_foreign() == 0          # nothing is recorded on a stream that the call was not given

    def end(self):
        self.lib.reft_plan_destroy(self.plan)
        assert self.lib.sim_end() == 0


def test_a_shorter_table_takes_part_of_the_room(lib):
    """Nine tables of eight rows fill the pool; one row on the null stream and one on another one take the room of two of
    the first table's rows, while its kernel may still wait for its turn."""
    c = Calls(lib)
    for i in range(9):
        c.rows(8, i, None)
    c.rows(1, 20, None)
    c.rows(1, 21, 1)
    c.end()


def test_the_oldest_of_many_tables_gives_up_its_slot(lib):
    """33 tables of a row: the first one's slot is needed, not its room, which other streams come to later."""
    c = Calls(lib)
    for i in range(33):
        c.rows(1, i, None)
    for i in range(60):
        c.rows(2, 40 + i, 1)
    c.end()


def test_a_known_table_on_the_null_stream_records_nothing(lib):
    """However many tables there are room for (72 rows), and whatever other streams do in between."""
    c = Calls(lib)
    mine = (1, 8, 33 + 8, 16, 32, 33 + 4)
    for n in mine:
        c.rows(n, n, None)
    before = lib.sim_events()
    for _ in range(5):
        for n in mine:
            c.rows(n, n, None)
    assert lib.sim_events() == before
    for i in range(20):
        c.rows(16, 50 + i, 1)
    before = lib.sim_events()
    for n in mine:
        c.rows(n, n, None)
    assert lib.sim_events() == before
    c.end()


@pytest.mark.parametrize("spans", [T, 65_536])
@pytest.mark.parametrize("null", [0.0, 0.2, 0.5, 0.9, 1.0])
@pytest.mark.parametrize("seed", [1, 2, 3])
def test_calls_of_all_sizes_on_three_streams(lib, seed, null, spans):
    """The widest tables (32 rows) among them, old and new pointers, a second phase on side streams alone."""
    rng = random.Random(seed)
    c = Calls(lib, SIZES + [0] * (spans - T))
    for step in range(600 if spans == T else 60):
        n = rng.choice((1, 1, 1, 2, 4, 8, 8, 16, 32, 33 + 4, 33 + 8, 33 + 31))
        stream = None if step < (500 if spans == T else 50) and rng.random() < null else rng.choice((1, 2))
        c.rows(n, rng.choice((n, n, rng.randrange(50), 1000 + step)), stream)
    c.end()


@pytest.mark.parametrize("sizes", [[60_000] * 256, [40] * 20_000, [300, 1, 0, 511] * 3000, [10_752] * 5000, [3 << 20] * 150,
                                   [70_001, 0, 131_072] * 200, [1 << 30] * 8 + [4] * 300 + [0] * 40 + [5 << 20] * 4])
def test_tables_of_a_plan(lib, sizes):
    """Every unit finds its span; and the tables are copied from pinned memory, as the pool's mirror holds all of these (from
    fresh pages the copy took a fifth of all plan creation)."""
    c = Calls(lib, sizes)
    p = (ctypes.c_void_p * len(sizes))(*range(1 << 44, (1 << 44) + len(sizes)))
    assert lib.reft_pack_device(c.plan, p, BUF, sum(sizes), None) == 0, lib.reft_last_error()
    assert lib.sim_races() == 0
    assert lib.sim_unpinned() == 0
    c.end()

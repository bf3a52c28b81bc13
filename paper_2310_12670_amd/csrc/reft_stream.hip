// The ragged stream kernel of libreft: gather (snapshot pack, XOR parity over span tables), fused
// decode into tensors, and scatter (restore), for spans of any size, alignment and number.
//
//   place of stream byte o  <-  XOR over K sources of their byte o,    o in [lo, hi)
//
// A source is a row of span pointers or a contiguous buffer; the destination is a contiguous buffer
// or a row of span pointers, and may itself be the last source.  With kPacked, the bytes of the first
// source alone go to a second contiguous buffer as well (the packed stream of one shard beside the
// parity of all), so that it is read once for both.
//
// The unit of work is one wavefront's: S = 1024 U consecutive stream bytes, U chunks of 16 bytes per
// lane and source, all in flight at once.  A wave finds the span that owns its unit's first byte with
// one look-up in the plan's table and one coalesced load of 64 span ends (locate), and from there
//   - a unit inside one span, the usual case, needs K span pointers and then only vector accesses at
//     uniform bases;
//   - a unit that spans share is done 1 KiB at a time, and where a boundary falls into that KiB
//     every lane finds its own span by comparing with the boundaries, which the wave broadcasts one
//     by one.
// Waves do not meet: no LDS, no barrier, so the chain of dependent loads (table, span ends,
// pointers, data: 2 - 4 us) of one wave hides behind the others, and short streams, which have few
// units, spread over the whole chip.
#include "reft_device.hpp"
#include "reft_rules.hpp"

#include <algorithm>

namespace reft {

// The last of a launch's K sources.
enum LastRow : uint32_t {
    kLastTable = 0,      // an ordinary row of the table
    kLastDest = 1,       // the destination's current bytes (accumulate)
    kLastContig = 2,     // the contiguous buffer whose virtual base is cbase
};

// Forms of the kernel.
enum Form {
    kPlain,
    kPacked,             // with the packed stream of the first source
    kRuns,               // a wave takes several units together (see k_stream)
    kInPlace,            // a row of the table is the destination: as with kLastDest, every byte is read and
                         // written once only.  (As an argument of the plain form it costs that 1 to 5 %.)
};

struct StreamArgs {
    PlanTables pt;
    const uint64_t *tab;     // rows of span pointers, row stride T
    const uint64_t *dtab;    // the destination's row, or null: contiguous
    uint64_t vb;             // contiguous destination: byte o lies at vb + o
    uint64_t vb2;            // kPacked: byte o of the first source goes to vb2 + o
    uint64_t cbase;          // kLastContig: byte o lies at cbase + o
    uint64_t lo, hi;         // stream range, lo < hi <= L
    uint64_t first_unit, nunits;
    uint32_t phase;          // unit u starts at stream byte u * S - phase
    uint32_t last;           // LastRow
    uint32_t spread;         // units in the order of unit_of_wave
    uint32_t run;            // kRuns: consecutive units that one wave takes together
};

// The tables do not change while the kernel runs; read through the constant address space, entries at
// a uniform index are scalar loads (through ordinary pointers the compiler takes vector loads, since
// the kernel's stores might alias, and then waits for them one by one).
#define REFT_CONST __attribute__((address_space(4)))
__device__ __forceinline__ uint64_t entry(const uint64_t *tab, uint64_t i)
{
    return ((const REFT_CONST uint64_t *)(uint64_t)tab)[i];
}
__device__ __forceinline__ uint32_t entry(const uint32_t *tab, uint64_t i)
{
    return ((const REFT_CONST uint32_t *)(uint64_t)tab)[i];
}

__device__ __forceinline__ uint64_t readlane64(uint64_t v, uint32_t l)
{
    const uint32_t a = __builtin_amdgcn_readlane((uint32_t)v, l);
    const uint32_t b = __builtin_amdgcn_readlane((uint32_t)(v >> 32), l);
    return (uint64_t)b << 32 | a;
}

// Span i owns stream bytes [b, e), and lane l holds the end of span base + l, where i = base + c.
// All but `ends` are the same in every lane.
struct Owner {
    uint64_t i, b, e, base, ends;
    uint32_t c;
};

// The span that owns byte x < L; span i is that one or an earlier one.  64 span ends per step: the
// number of them at or below x says how far to go on.
__device__ __forceinline__ void locate(const PlanTables &pt, Owner &o, uint64_t i, uint64_t x, uint32_t lane)
{
    o.b = entry(pt.off, i);
    for (;; i += 64) {
        const uint64_t at = i + 1 + lane < pt.T ? i + 1 + lane : pt.T;
        o.ends = entry(pt.off, at);                                   // off[T] = L > x ends the search
        o.c = (uint32_t)__popcll(__ballot(o.ends <= x));
        if (o.c) o.b = readlane64(o.ends, o.c - 1);
        if (o.c < 64) break;
    }
    o.base = i;
    o.i = i + o.c;
    o.e = readlane64(o.ends, o.c);
}

// The address of the first byte of span q (which starts at stream byte b) in source row j.
template <int K>
__device__ __forceinline__ uint64_t source_of(const StreamArgs &a, int j, uint64_t q, uint64_t b)
{
    if (j == K - 1 && a.last != kLastTable) {
        if (a.last == kLastContig) return a.cbase + b;
        return a.dtab ? entry(a.dtab, q) : a.vb + b;
    }
    return entry(a.tab, (uint64_t)j * a.pt.T + q);
}

template <bool NT>
__device__ __forceinline__ void st16_any(uint64_t p, u32x4 v)
{
    if constexpr (NT) __builtin_nontemporal_store(v, (REFT_GLOBAL u32x4_any *)p);
    else *(REFT_GLOBAL u32x4_any *)p = v;
}

// The XOR of the 16 bytes at address(j), j < K; all loads before the first use.  With PACK the first
// 16 go to pack.
template <int K, bool NT, bool PACK, class Address>
__device__ __forceinline__ u32x4 xor_16(Address address, uint64_t pack)
{
    gcptr16 s[K];
#pragma unroll
    for (int j = 0; j < K; ++j) s[j] = as_gc16(address(j));
    u32x4 t[K];
#pragma unroll
    for (int j = 0; j < K; ++j) t[j] = ld16<NT>(s[j]);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (PACK) st16_any<NT>(pack, t[0]);
    u32x4 v = t[0];
#pragma unroll
    for (int j = 1; j < K; ++j) v ^= t[j];
    return v;
}

// 1 KiB of span o.i from stream byte x on, wholly inside the span and the range.
template <int K, bool NT, bool PACK>
__device__ __forceinline__ void move_kib(const StreamArgs &a, const Owner &o, uint64_t x, uint32_t lane)
{
    const uint64_t r = x - o.b + lane * 16;
    const u32x4 v = xor_16<K, NT, PACK>([&](int j) { return source_of<K>(a, j, o.i, o.b) + r; },
                                        a.vb2 + x + lane * 16);
    st16_any<NT>(a.dtab ? entry(a.dtab, o.i) + r : a.vb + x + lane * 16, v);
}

// The unit of V KiB at stream byte x, wholly inside span i and the range.  Inside a span the units
// move together by up to 127 bytes so that the first source, and with it those that are aligned like
// it, is read in whole cache lines, or, where it stands (nearly) alone, the destination is written in
// such: a unit then starts where the one before it in the span ends, the span's first such unit moves
// the bytes in front of it as well, and the last one, behind which there is no room, stays where it
// is; the few bytes that come twice get the same value.  Where the destination is a source
// nothing may come twice, and nothing is moved.  (Shards of tensors at odd stream offsets are aligned alike:
// 8 x 56 MB encoded in 87 instead of 108 us, 8 x 132 MB of small tensors in 221 instead of 262.)
//
// kRuns: the units behind it as well, up to `most` in all, as far as they lie wholly inside the span and the
// range; returns how many.
template <int K, int V, bool NT, Form F>
__device__ __forceinline__ uint32_t move_units(const StreamArgs &a, uint64_t i, uint64_t x, uint32_t lane,
                                               uint32_t most)
{
    constexpr bool PACK = F == kPacked;
    constexpr uint32_t S = 1024 * V;
    // everything that is known of span i in one go, without branches between the loads (where there
    // is no such table, an entry of another one is loaded and not used)
    const uint64_t b = entry(a.pt.off, i), e = entry(a.pt.off, i + 1);
    const uint64_t dt = entry(a.dtab ? a.dtab : a.pt.off, i);
    uint64_t p[K];
#pragma unroll
    for (int j = 0; j < K - 1; ++j) p[j] = entry(a.tab, (uint64_t)j * a.pt.T + i);
    p[K - 1] = entry(a.last == kLastTable ? a.tab + (uint64_t)(K - 1) * a.pt.T : a.pt.off, i);
    const uint64_t r = x - b;
    uint64_t d = (a.dtab ? dt : a.vb + b) + r;
    if (a.last == kLastContig) p[K - 1] = a.cbase + b;
    if (a.last == kLastDest) p[K - 1] = d - r;
    gcptr16 s[K];
#pragma unroll
    for (int j = 0; j < K; ++j) s[j] = as_gc16(p[j] + r);
    uint32_t alike = 0;
#pragma unroll
    for (int j = 1; j < K; ++j) alike += (((uint32_t)(uint64_t)s[j] ^ (uint32_t)(uint64_t)s[0]) & 15u) == 0;
    const uint32_t to_line = (uint32_t)(0 - (2 * alike >= K ? (uint64_t)s[0] : d)) & 127u;
    // vmcnt(0), once in front of a run: the compiler may otherwise take registers for still in flight from
    // before and wait for them in every round, and with them for the stores of the round before (2 sources,
    // 126 MB by 4 workgroups: 2217 us so, 1583 with this)
    if constexpr (F == kRuns) __builtin_amdgcn_s_waitcnt(0x0f70);
    for (uint32_t done = 1;; ++done) {
        uint32_t lead = F == kInPlace ? 0 : to_line;
        if (lead) {
            if (a.last == kLastDest || x + S + 128 > (e < a.hi ? e : a.hi)) lead = 0;
        }
        if (lead) {
            const int64_t first = (int64_t)(b > a.lo ? b : a.lo);
            if ((int64_t)x - (int64_t)S < first && lane * 16 < lead) {
                st16_any<NT>(d + lane * 16, xor_16<K, NT, PACK>([&](int j) { return (uint64_t)s[j] + lane * 16; },
                                                                a.vb2 + x + lane * 16));
            }
            d += lead;
#pragma unroll
            for (int j = 0; j < K; ++j) s[j] = as_gc16((uint64_t)s[j] + lead);
        }
        // all loads of up to 16 chunks before the first use (left alone, the compiler alternates them)
        constexpr int R = K * V <= 16 ? K : 16 / V;
        u32x4 v[V] = {};
#pragma unroll
        for (int j = 0; j < K; j += R) {
            u32x4 t[R][V];
#pragma unroll
            for (int q = 0; q < R && j + q < K; ++q) {
#pragma unroll
                for (int u = 0; u < V; ++u) t[q][u] = ld16<NT>(s[j + q] + lane + u * 64);
            }
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (PACK) {
                if (j == 0) {
#pragma unroll
                    for (int u = 0; u < V; ++u) st16_any<NT>(a.vb2 + x + lead + (lane + u * 64) * 16, t[0][u]);
                }
            }
#pragma unroll
            for (int q = 0; q < R && j + q < K; ++q) {
#pragma unroll
                for (int u = 0; u < V; ++u) v[u] ^= t[q][u];
            }
        }
#pragma unroll
        for (int u = 0; u < V; ++u) st16_any<NT>(d + (uint64_t)(lane + u * 64) * 16, v[u]);
        if constexpr (F != kRuns) return 1;
        x += S;
        if (done == most || x + S > (e < a.hi ? e : a.hi)) return done;
        d += S - lead;
#pragma unroll
        for (int j = 0; j < K; ++j) s[j] = as_gc16((uint64_t)s[j] + S - lead);
    }
}

// n bytes from stream byte p on, all inside span q (which starts at b), one by one.
template <int K, bool PACK>
__device__ __forceinline__ void move_bytes(const StreamArgs &a, uint64_t q, uint64_t b, uint64_t p, uint32_t n)
{
    const uint64_t d = (a.dtab ? entry(a.dtab, q) - b : a.vb) + p;
    uint64_t s[K];
#pragma unroll
    for (int j = 0; j < K; ++j) s[j] = source_of<K>(a, j, q, b) + (p - b);
    for (uint32_t t = 0; t < n; t += 4) {                      // 4 K bytes in flight
        uint32_t v[4] = {0, 0, 0, 0};
#pragma unroll
        for (int j = 0; j < K; ++j) {
#pragma unroll
            for (uint32_t c = 0; c < 4; ++c) {
                const uint8_t x = ld8(s[j] + (t + c < n ? t + c : n - 1));
                if (PACK && j == 0 && t + c < n) st8(a.vb2 + p + t + c, x);
                v[c] ^= x;
            }
        }
#pragma unroll
        for (uint32_t c = 0; c < 4; ++c)
            if (t + c < n) st8(d + t + c, (uint8_t)v[c]);
    }
}

// 1 KiB from stream byte x on that several spans share or that reaches out of the range.  o owns the
// first of its bytes that lies in the range, y1 is the end of them; lane l holds the end of span
// base + l (ends), span o.i is base + c.
//
// A lane whose 16 bytes reach over the end of its span moves the span's last 16 bytes instead, and
// then the next span's first 16: bytes that its neighbours move too are written twice, with the same
// value.  Bytes are moved one by one only in spans that have fewer than 16 in the range, and, where
// the destination is a source (a byte must then be read and written once), in every straddling lane.
template <int K, bool NT, Form F>
__device__ __forceinline__ void move_shared(const StreamArgs &a, const Owner &o, uint64_t x, uint64_t y1,
                                            uint32_t lane)
{
    constexpr bool PACK = F == kPacked;
    constexpr uint32_t kNone = 0xffffffffu;
    const uint32_t at = lane * 16;
    // my span: `skip` spans behind o's, from byte `from` of this KiB on (if skip), up to byte `to`;
    // the next one with bytes: `skip2` spans behind o's, up to byte `to2`
    uint32_t skip = 0, from = 0, to = kNone, skip2 = 0, to2 = kNone;
    uint64_t base = o.base, ends = o.ends;
    uint32_t j = o.c;
    for (;;) {
        const uint32_t rel = (uint32_t)(ends - x);
        const uint32_t n = (uint32_t)__popcll(__ballot(ends < y1));   // ends ascend: lanes 0 .. n - 1
        for (; j < n; ++j) {
            const uint32_t bnd = __builtin_amdgcn_readlane(rel, j);
            const uint32_t s = (uint32_t)(base - o.i) + j + 1;
            if (at >= bnd) {
                skip = s;
                from = bnd;
            } else if (to == kNone || bnd == to) {
                to = bnd;
                skip2 = s;
            } else if (to2 == kNone) {
                to2 = bnd;
            }
        }
        if (n < 64) break;
        base += 64;
        const uint64_t idx = base + 1 + lane < a.pt.T ? base + 1 + lane : a.pt.T;
        ends = entry(a.pt.off, idx);
        j = 0;
    }
    // the end of span o.i + skip2, where no boundary in this KiB gave it
    const uint64_t end2 = __shfl(ends, (int)((uint32_t)(o.i - base) + skip2) & 63);
    const uint64_t me = x + at;                                // may wrap below 0 in the first unit
    const uint64_t lo = (int64_t)me < (int64_t)a.lo ? a.lo : me;
    const uint64_t hi = (int64_t)(me + 16) > (int64_t)y1 ? y1 : me + 16;
    if ((int64_t)lo >= (int64_t)hi) return;
    // the parts of the two spans that lie in the range (of the first, as far as it is known): [w0, w1), [w1, w2)
    const uint64_t q = o.i + skip, b = skip ? x + from : o.b, q2 = o.i + skip2;
    const uint64_t w0 = b < a.lo ? a.lo : b, w1 = to == kNone ? y1 : x + to;
    const uint64_t w2 = to2 != kNone ? x + to2 : end2 < a.hi ? end2 : a.hi;
    const bool one = w1 >= hi;                                 // all my bytes belong to span q
    bool can = a.last != kLastDest || (one && hi - lo == 16);
    if constexpr (F == kInPlace) can = one && hi - lo == 16;
    if (can && w1 - w0 >= 16 && (one || (w2 - w1 >= 16 && w2 >= hi))) {
        const uint64_t p = lo < w1 - 16 ? lo : w1 - 16;
        const uint64_t d = (a.dtab ? entry(a.dtab, q) - b : a.vb) + p;
        if constexpr (K <= 4) {                                // both at once, where registers allow
            gcptr16 s[K], s2[K];
            uint64_t d2 = 0;
            u32x4 t[K], t2[K];
#pragma unroll
            for (int j = 0; j < K; ++j) s[j] = as_gc16(source_of<K>(a, j, q, b) + (p - b));
            if (!one) {
                d2 = a.dtab ? entry(a.dtab, q2) : a.vb + w1;
#pragma unroll
                for (int j = 0; j < K; ++j) s2[j] = as_gc16(source_of<K>(a, j, q2, w1));
            }
#pragma unroll
            for (int j = 0; j < K; ++j) t[j] = ld16<NT>(s[j]);
            if (!one) {
#pragma unroll
                for (int j = 0; j < K; ++j) t2[j] = ld16<NT>(s2[j]);
            }
            if constexpr (PACK) {
                st16_any<NT>(a.vb2 + p, t[0]);
                if (!one) st16_any<NT>(a.vb2 + w1, t2[0]);
            }
#pragma unroll
            for (int j = 1; j < K; ++j) t[0] ^= t[j];
            st16_any<NT>(d, t[0]);
            if (!one) {
#pragma unroll
                for (int j = 1; j < K; ++j) t2[0] ^= t2[j];
                st16_any<NT>(d2, t2[0]);
            }
        } else {
            st16_any<NT>(d, xor_16<K, NT, PACK>([&](int j) { return source_of<K>(a, j, q, b) + (p - b); },
                                                a.vb2 + p));
            if (!one)
                st16_any<NT>(a.dtab ? entry(a.dtab, q2) : a.vb + w1,
                             xor_16<K, NT, PACK>([&](int j) { return source_of<K>(a, j, q2, w1); }, a.vb2 + w1));
        }
        return;
    }
    // spans of less than 16 bytes
    uint64_t i = q, begin = b;
    for (uint64_t p = lo;;) {
        const uint64_t e = entry(a.pt.off, i + 1);
        move_bytes<K, PACK>(a, i, begin, p, (uint32_t)((e < hi ? e : hi) - p));
        if (e >= hi) break;
        p = begin = e;
        do ++i; while (entry(a.pt.off, i + 1) <= p);                  // p < hi <= L = off[T]
    }
}

// The workgroup (1 or 4 waves) has no meaning beyond the dispatch.  Unless the caller caps the grid
// there is one wave per unit, dispatched in order, so that the chip moves through its streams in
// narrow windows; that is what HBM likes best here (copy of 2 GiB by 1 KiB units: 6.6 TB/s with
// workgroups of 64 threads, 6.5 with 256, 6.2 with 1024; 4.8 - 5.9 with a persistent grid).
//
// kRuns (a grid of few waves, each with many units): a wave takes a.run consecutive units together and
// looks up once for those that lie in one span; without, look-ups and data of its units follow one
// another.  126 MB in spans of 3 MB by 4 / 16 / 64 workgroups, us, without and with: packed 1869 / 479 / 134
// and 1186 / 315 / 102 (tiles walked by workgroups: 1620 / 432 / 145), parity of 4: 3563 / 906 / 247 and
// 2593 / 677 / 196 (3168 / 817 / 253).
template <int K, int U, bool NT, Form F = kPlain>
__global__ void __launch_bounds__(256) k_stream(const StreamArgs a)
{
    constexpr uint32_t S = 1024 * U;
    const uint32_t lane = threadIdx.x & 63;
    const uint32_t waves = blockDim.x >> 6;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint64_t stride = (uint64_t)gridDim.x * waves;
    // kRuns: units left of this run, and how many of them the last step moved
    uint32_t left = F == kRuns ? a.run : 1, done = 1;
    for (uint64_t w = ((uint64_t)blockIdx.x * waves + wave) * (F == kRuns ? a.run : 1); w < a.nunits;
         w += F != kRuns ? stride : (left -= done) ? done : done + (stride - 1) * (left = a.run)) {
        Owner o;
        // streaming launches only: the few instructions more delay a short one by 0.2 us
        const uint64_t un = NT && F != kRuns && U <= 2 && a.spread ? unit_of_wave<U>(w, a.nunits) : w;
        const uint64_t x = (a.first_unit + un) * S - a.phase;  // below 0 (wraps) in the first unit
        const uint64_t y0 = (int64_t)x < (int64_t)a.lo ? a.lo : x;
        const uint64_t y1 = (int64_t)(x + S) > (int64_t)a.hi ? a.hi : x + S;
        const uint32_t first = entry(a.pt.first_span, y0 >> a.pt.tile_shift);
        if ((first & kWholeBlock) && y1 - y0 == S && y1 <= ((y0 >> a.pt.tile_shift) + 1) << a.pt.tile_shift) {
            done = move_units<K, U, NT, F>(a, first & ~kWholeBlock, x, lane, left);
            continue;
        }
        locate(a.pt, o, first & ~kWholeBlock, y0, lane);
        if (y1 - y0 == S && y1 <= o.e) {
            done = move_units<K, U, NT, F>(a, o.i, x, lane, left);
            continue;
        }
        done = 1;
#pragma unroll 1
        for (uint32_t u = 0; u < U; ++u) {
            const uint64_t xs = x + u * 1024;
            const uint64_t z0 = (int64_t)xs < (int64_t)a.lo ? a.lo : xs;
            const uint64_t z1 = (int64_t)(xs + 1024) > (int64_t)y1 ? y1 : xs + 1024;
            if ((int64_t)z0 >= (int64_t)z1) continue;
            if (z0 >= o.e) locate(a.pt, o, o.i, z0, lane);
            if (z1 - z0 == 1024 && z1 <= o.e) move_kib<K, NT, F == kPacked>(a, o, xs, lane);
            else move_shared<K, NT, F>(a, o, xs, z1, lane);
        }
    }
}

// ------------------------------------------------------------------------------------------------
// launch
// ------------------------------------------------------------------------------------------------
// Traffic (read and written) up to which a launch may find and leave its data in the 256 MB cache: it
// then uses plain accesses (4 x 14.7 MB, 73 MB of traffic: 15.5 us, with streaming ones 16.9; from
// 8 x 14.7 MB on streaming ones are as fast or faster) and workgroups of four waves (16 against 17 us:
// fewer to dispatch; long streams prefer single waves, 4.12 against 4.23 ms for 25.8 GB of copies).
constexpr uint64_t kCachedTraffic = 96ull << 20;

// KiB per wave and source.  Small units keep the windows narrow in which the chip moves through its
// streams; one source alone needs two to cover the look-ups in front of the data.  us for 1 and 2 KiB:
// 1 source 4.00 and 3.99 ms (25.8 GB in long spans), 418 and 377 us (2.1 GB in short ones); 2 sources
// 745 and 776 (4.9 GB); 4: 1303 and 1418 (8.2 GB); 8: 2380 and 2595 (14.8 GB), 211 and 224 (1.2 GB,
// short spans); 16: 2299 and 2405 (14.3 GB).
static uint32_t long_stream_unroll(int nsrc) { return nsrc == 1 ? 2 : 1; }

// LDS to ask for, which the kernel does not use, so that no more waves share a compute unit than its streams
// want: the more there are, the wider the windows in which the chip moves through memory.  Swept from 8 to 20 waves
// on 0.5 to 14 GB (encode, decode, with packed stream, rotated): the best is 14 to 16 with 4 sources, 14 with 5 and
// 6, 13, 12 with 8, 12, 11, 11, 10 with 12, 9, 9, 8 with 15 and 16, and one more or less costs 0.2 to 1 %.  us, with 80
// KiB in flight as the rule (22 waves with 4 sources, 12 with 8, 8 from 12 on) / with this one: 4 sources 738 / 720,
// 5: 871 / 852, 9: 1392 / 1310, 10: 1482 / 1428, 12: 1779 / 1713 and, in spans of 10 KB, 309 / 302.
static uint32_t crowd_limit(int nsrc)
{
    if (nsrc < 4) return 0;
    const uint32_t waves = std::max({20 - nsrc, 17 - 5 * nsrc / 8, 8});
    return 160 * 1024 / waves / 512 * 512;
}

#define REFT_PICK_MANY(K)                                                                         \
    (cfg.nontemporal ? (cfg.unroll == 1 ? k_stream<K, 1, true> : k_stream<K, 2, true>)            \
                     : (cfg.unroll == 1 ? k_stream<K, 1, false> : k_stream<K, 2, false>))

#define REFT_PICK_PACK(K) (cfg.nontemporal ? k_stream<K, 1, true, kPacked> : k_stream<K, 1, false, kPacked>)

#define REFT_PICK_RUNS(K) (cfg.nontemporal ? k_stream<K, 4, true, kRuns> : k_stream<K, 4, false, kRuns>)

#define REFT_PICK_IN_PLACE(K) k_stream<K, 1, true, kInPlace>

#define REFT_CASES_4(PICK)                                                                        \
    case 1: fn = PICK(1); break;                                                                  \
    case 2: fn = PICK(2); break;                                                                  \
    case 3: fn = PICK(3); break;                                                                  \
    case 4: fn = PICK(4); break;

#define REFT_CASES_5_8(PICK)                                                                      \
    case 5: fn = PICK(5); break;                                                                  \
    case 6: fn = PICK(6); break;                                                                  \
    case 7: fn = PICK(7); break;                                                                  \
    case 8: fn = PICK(8); break;

#define REFT_CASES_9_16(PICK)                                                                     \
    case 9: fn = PICK(9); break;                                                                  \
    case 10: fn = PICK(10); break;                                                                \
    case 11: fn = PICK(11); break;                                                                \
    case 12: fn = PICK(12); break;                                                                \
    case 13: fn = PICK(13); break;                                                                \
    case 14: fn = PICK(14); break;                                                                \
    case 15: fn = PICK(15); break;                                                                \
    case 16: fn = PICK(16); break;

static hipError_t launch_stream(StreamArgs a, int nsrc, uint64_t contig, Form form, LaunchCfg cfg,
                                hipStream_t stream)
{
    void (*fn)(const StreamArgs) = nullptr;
    const bool cached = (uint64_t)(nsrc + (form == kPacked ? 2 : 1)) * (a.hi - a.lo) <= kCachedTraffic;
    // a capped grid (few waves, say on the host link) wants all that a wave may have in flight
    const uint32_t unroll = cfg.capped ? 4 : cached ? 1 : long_stream_unroll(nsrc);
    if (unroll < cfg.unroll) cfg.unroll = unroll;
    if (cached && !cfg.capped) cfg.nontemporal = false;
    if (nsrc > kMaxSrc && cfg.unroll > 2) cfg.unroll = 2;    // 2 KiB of 9 sources and more: 18 loads a lane
    if (form == kPacked || form == kInPlace) cfg.unroll = 1;
    // units start where the contiguous operand is 16-byte aligned
    const uint64_t S = 1024ull * cfg.unroll;
    a.phase = (uint32_t)contig & 15u;
    a.first_unit = (a.lo + a.phase) / S;
    a.nunits = (a.hi - 1 + a.phase) / S - a.first_unit + 1;
    const uint32_t waves = cached || cfg.capped ? 4 : 1;
    a.run = 1;
    // (in short spans the tensors' places have little to do with the stream's: 8 x 132 MB in spans of 10 KB 204.6
    // us in plain order, 206.2 so)
    a.spread = waves == 1 && a.first_unit % 32 == 0 && a.pt.L / a.pt.T >= 64 * 1024;
    if (form == kPlain && cfg.runs && cfg.unroll == 4) {
        a.run = run_of_units(a.nunits, waves * (uint64_t)cfg.max_wgs, nsrc, a.pt.L / a.pt.T);
        if (a.run > 1) form = kRuns;
    }
    switch (form) {
    case kPlain:
        switch (nsrc) {
            REFT_CASES_9_16(REFT_PICK_MANY)
        default: REFT_PICK_K(k_stream, fn, nsrc)
        }
        break;
    case kPacked:
        switch (nsrc) {
            REFT_CASES_4(REFT_PICK_PACK) REFT_CASES_5_8(REFT_PICK_PACK) REFT_CASES_9_16(REFT_PICK_PACK)
        default: return hipErrorInvalidValue;
        }
        break;
    case kRuns:
        switch (nsrc) {
            REFT_CASES_4(REFT_PICK_RUNS)
        default: return hipErrorInvalidValue;
        }
        break;
    case kInPlace:
        switch (nsrc) {
            REFT_CASES_4(REFT_PICK_IN_PLACE) REFT_CASES_5_8(REFT_PICK_IN_PLACE)
            REFT_CASES_9_16(REFT_PICK_IN_PLACE)
        default: return hipErrorInvalidValue;
        }
        break;
    }
    const uint32_t g = stream_grid((a.nunits + a.run - 1) / a.run, waves, cfg.capped ? cfg.max_wgs : 0);
    hipLaunchKernelGGL(fn, dim3(g), dim3(64 * waves), waves == 1 ? crowd_limit(nsrc) : 0, stream, a);
    return hipGetLastError();
}

hipError_t launch_gather(const PlanTables &pt, const uint64_t *tab, int nrows, bool acc, bool in_place,
                         const uint64_t *dtab, uint64_t dst_vbase, uint64_t lo, uint64_t hi,
                         const LaunchCfg &cfg, hipStream_t stream)
{
    if (lo >= hi) return hipSuccess;
    if (hi > pt.L) return hipErrorInvalidValue;
    StreamArgs a{};
    a.pt = pt;
    a.tab = tab;
    a.dtab = dtab;
    a.vb = dst_vbase;
    a.lo = lo;
    a.hi = hi;
    a.last = acc ? kLastDest : kLastTable;
    return launch_stream(a, nrows + (acc ? 1 : 0), dtab ? 0 : dst_vbase, in_place && !acc ? kInPlace : kPlain, cfg,
                         stream);
}

hipError_t launch_gather_pack(const PlanTables &pt, const uint64_t *tab, int nrows, uint64_t vb,
                              uint64_t vb2, uint64_t lo, uint64_t hi, const LaunchCfg &cfg,
                              hipStream_t stream)
{
    if (lo >= hi) return hipSuccess;
    if (hi > pt.L) return hipErrorInvalidValue;
    StreamArgs a{};
    a.pt = pt;
    a.tab = tab;
    a.vb = vb;
    a.vb2 = vb2;
    a.lo = lo;
    a.hi = hi;
    a.last = kLastTable;
    return launch_stream(a, nrows, vb, kPacked, cfg, stream);
}

hipError_t launch_scatter(const PlanTables &pt, const uint64_t *tab, uint64_t src_vbase,
                          uint64_t lo, uint64_t hi, const LaunchCfg &cfg, hipStream_t stream)
{
    if (lo >= hi) return hipSuccess;
    if (hi > pt.L) return hipErrorInvalidValue;
    StreamArgs a{};
    a.pt = pt;
    a.dtab = tab;
    a.cbase = src_vbase;
    a.lo = lo;
    a.hi = hi;
    a.last = kLastContig;
    return launch_stream(a, 1, src_vbase, kPlain, cfg, stream);
}

}  // namespace reft

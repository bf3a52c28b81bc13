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
// The unit of work is one wavefront's: a KiB of one span (units_of), 16 bytes per lane and source, all in flight
// at once.  A wave looks up its unit's span (a table with an entry per unit, or per block of units in long
// streams), loads what is known of the span, K span pointers among it, and then has only vector accesses at uniform
// bases; the span's last unit differs in nothing but the lanes that store.  No unit has bytes of two spans, so
// there is nothing to search and nothing for lanes to decide.  Only in streams of spans of a few hundred bytes, where most
// of a wave would stay empty, several units share one (k_stream_small).
//
// Waves do not meet: no LDS, no barrier, so the chain of dependent loads (table, span, data: 2 - 3 us) of one wave
// hides behind the others, and short streams, which have few units, spread over the whole chip.
//
// Before, the units were KiB of the stream: a wave whose KiB held a boundary broadcast the boundaries, every lane
// found its own span, and straddling lanes moved 16 bytes of either.  us, so and now: parity of 4 x 14.7 MB in 256 odd
// tensors 14.8 / 13.8, one of them decoded 15.7 / 13.85, 14.7 MB packed and unpacked 19.1 / 16.5, parity of 8 x 132 MB in
// 12,288 odd tensors 209 / 196 (5.7 / 6.1 TB/s), 528 MB in 49,152 packed and unpacked 379 / 354, parity of 4 x 0.5 GB in
// spans of 130 KB 459 / 424, of 16 x 132 MB in spans of 10 KB 400 / 366; long spans the same.
#include "reft_device.hpp"
#include "reft_rules.hpp"

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
    const uint64_t *off, *unit_off;   // of the plan's tables (PlanTables)
    const uint32_t *unit_span;
    uint64_t T;
    const uint64_t *tab;     // rows of span pointers, row stride T
    const uint64_t *last_row, *dest_row;   // of the last source and the destination, or any table (not used)
    uint64_t vb;             // contiguous destination: byte o lies at vb + o
    uint64_t vb2;            // kPacked: byte o of the first source goes to vb2 + o
    uint64_t cbase;          // kLastContig: byte o lies at cbase + o
    StreamRange range;       // lo < hi <= L
    uint64_t first_step, nsteps;   // a wave's step is U units: step x has units x U .. x U + U - 1
    uint64_t stride;         // waves of the grid
    uint32_t waves;          // waves per workgroup
    uint32_t unit_shift;
    uint32_t grid;           // see head_of
    uint32_t last;           // LastRow
    uint32_t ragged;         // the destination has a row
    uint32_t spread;         // Spread
    uint32_t run;            // kRuns: consecutive steps that one wave takes together
    uint32_t once, pack;     // k_stream_small: the destination is a source; with the packed stream
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

// The span that owns unit u; all lanes get the same answer.  Where a block of units is shared by spans, 64 ends per
// step: the number of them at or below u says how far to go on.
__device__ __forceinline__ uint64_t span_of(const StreamArgs &a, uint64_t u, uint32_t lane)
{
    const uint32_t first = entry(a.unit_span, u >> a.unit_shift);
    uint64_t i = first & ~kWholeBlock;
    if (first & kWholeBlock) return i;
    for (;; i += 64) {
        const uint64_t at = i + 1 + lane < a.T ? i + 1 + lane : a.T;
        const uint32_t c = (uint32_t)__popcll(__ballot(entry(a.unit_off, at) <= u));   // unit_off[T] > u ends the search
        if (c < 64) return i + c;
    }
}

// What a wave knows of a span.
template <int K>
struct Span {
    uint64_t u0, u1;         // its units
    int64_t lo, hi;          // its bytes in the range, from its first one on (lo may lie below 0)
    uint64_t s[K], d, d2;    // where its first byte lies in the sources, the destination and the packed stream
    uint32_t head, lead;     // see piece_of
    uint32_t turn;           // see turn_of (0 where some of the span is not in the range)
};

// What a kernel knows of the orders in which a launch may deal its steps (Spread).
enum Deal {
    kAsNumbered = 0,         // kInOrder alone
    kFarAlone = 1,           // kFarUnturned alone
    kAnyOrder = 2,           // all but kFarUnturned
};

// Span i, everything in one go (what the last source and the destination have no table for comes from another one
// and is not used: a branch there costs the wave another wait).
//
// The lead: a span's units lie so that the first source, and with it those that are aligned like it, is read in
// whole cache lines, or, where it stands (nearly) alone, the destination is written in such.  (Shards of tensors at
// odd stream offsets are aligned alike: 8 x 56 MB encoded in 87 instead of 108 us.)
template <int K, Deal D>
__device__ __forceinline__ Span<K> load_span(const StreamArgs &a, uint64_t i)
{
    Span<K> o;
    const uint64_t b = entry(a.off, i), e = entry(a.off, i + 1);
    o.u0 = entry(a.unit_off, i);
    o.u1 = entry(a.unit_off, i + 1);
    const uint64_t dt = entry(a.dest_row, i);
#pragma unroll
    for (int j = 0; j < K - 1; ++j) o.s[j] = entry(a.tab, (uint64_t)j * a.T + i);
    o.s[K - 1] = entry(a.last_row, i);
    __builtin_amdgcn_sched_barrier(0);       // (the compiler waits for the first before it asks for the last)
    o.d = a.ragged ? dt : a.vb + b;
    o.d2 = a.vb2 + b;
    if (a.last == kLastContig) o.s[K - 1] = a.cbase + b;
    if (a.last == kLastDest) o.s[K - 1] = o.d;
    o.head = (uint32_t)head_of((uint32_t)b, a.grid);
    o.lo = (int64_t)(a.range.lo - b);
    o.hi = (int64_t)((e < a.range.hi ? e : a.range.hi) - b);
    uint32_t alike = 0;
#pragma unroll
    for (int j = 1; j < K; ++j) alike += (((uint32_t)o.s[j] ^ (uint32_t)o.s[0]) & 15u) == 0;
    const uint64_t ref = (2 * alike >= K ? o.s[0] : o.d) + o.head;
    const bool wide = D == kAnyOrder && a.spread && o.u1 - o.u0 > kTurned;
    o.lead = (uint32_t)(0 - ref) & ((wide ? kMaxLead : kLineLead) - 1);
    o.turn = wide && b >= a.range.lo && e <= a.range.hi ? turn_of(o.u0, (ref + o.lead - kUnit) / kUnit) : 0;
    return o;
}

// A lane's offset from a uniform base.  (Hidden from the compiler, which otherwise widens it to 64 bits outside of the
// loop and then adds it to every base in vector registers, where a load takes base and 32-bit offset as they are.)
__device__ __forceinline__ uint32_t lane_offset(uint32_t at)
{
    asm volatile("" : "+v"(at));
    return at;
}

// Loads of the 16 bytes `at` bytes (at least 0) behind p.
template <bool NT>
__device__ __forceinline__ u32x4 ld16_at(uint64_t p, uint32_t at)
{
    return ld16<NT>((gcptr16)((const REFT_GLOBAL char *)p + at));
}

template <bool NT>
__device__ __forceinline__ void st16_at(uint64_t p, uint32_t at, u32x4 v)
{
    REFT_GLOBAL u32x4_any *const q = (REFT_GLOBAL u32x4_any *)((REFT_GLOBAL char *)p + at);
    if constexpr (NT) __builtin_nontemporal_store(v, q);
    else *q = v;
}

// The same where results are written through the L2 (writes_through).  As buffer accesses: they take the two bits of a store
// together, and the loads' bases stay in scalar registers as they are (8 x 3.1 GB 4139 us with global accesses, 4130 with
// these stores, 4103 with these loads, 4080 with both; copies with such loads 2 to 4 % more, so theirs are ordinary).
typedef unsigned int u32x4_raw __attribute__((ext_vector_type(4)));
constexpr int kNontemporal = 2, kDeviceScope = 16;            // bits nt and sc1
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_at(uint64_t p)
{
    return __builtin_amdgcn_make_buffer_rsrc((void *)p, 0, 0xffffffffu, 0x00020000);
}
__device__ __forceinline__ u32x4 ld16_through(uint64_t p, uint32_t at)
{
    return (u32x4)__builtin_amdgcn_raw_buffer_load_b128(buffer_at(p), at, 0, kNontemporal);
}
__device__ __forceinline__ void st16_through(uint64_t p, uint32_t at, u32x4 v)
{
    __builtin_amdgcn_raw_buffer_store_b128((u32x4_raw)v, buffer_at(p), at, 0, kNontemporal | kDeviceScope);
}

// The XOR of the sources' 16 bytes at byte `from` + `at` of the span, all loads before the first use (left alone,
// the compiler alternates them); stored if `store`.
template <int K, bool NT, bool PACK, bool THROUGH = false>
__device__ __forceinline__ void move_16(const Span<K> &o, int64_t from, uint32_t at, bool store)
{
    u32x4 t[K];
    at = lane_offset(at);
#pragma unroll
    for (int j = 0; j < K; ++j) {
        if constexpr (THROUGH && K > 1) t[j] = ld16_through(o.s[j] + from, at);
        else t[j] = ld16_at<NT>(o.s[j] + from, at);
    }
    __builtin_amdgcn_sched_barrier(0);
    u32x4 v = t[0];
#pragma unroll
    for (int j = 1; j < K; ++j) v ^= t[j];
    if (store) {
        at = lane_offset(at);
        if constexpr (THROUGH) {
            if constexpr (PACK) st16_through(o.d2 + from, at, t[0]);
            st16_through(o.d + from, at, v);
        } else {
            if constexpr (PACK) st16_at<NT>(o.d2 + from, at, t[0]);
            st16_at<NT>(o.d + from, at, v);
        }
    }
}

// Byte x of the span.
template <int K, bool PACK>
__device__ __forceinline__ void move_byte(const Span<K> &o, int64_t x)
{
    uint8_t t[K];
#pragma unroll
    for (int j = 0; j < K; ++j) t[j] = ld8(o.s[j] + x);
    if constexpr (PACK) st8(o.d2 + x, t[0]);
#pragma unroll
    for (int j = 1; j < K; ++j) t[0] ^= t[j];
    st8(o.d + x, t[0]);
}

// Unit u of span o.  All lanes load, those behind the piece's end its last 16 bytes, and one of them stores these: a
// few bytes come twice, with the same value.  Only where fewer than 16 bytes of the span lie in the range up to
// the piece's end, and where the destination is a source (a byte must then be read and written once), the bytes
// behind the last whole 16 go one per lane.
template <int K, bool NT, Form F, bool THROUGH = false>
__device__ __forceinline__ void move_unit(const StreamArgs &a, const Span<K> &o, uint64_t u, uint32_t lane)
{
    constexpr bool PACK = F == kPacked;
    const bool once = F == kInPlace || a.last == kLastDest;
    const int64_t lo = o.lo > 0 ? o.lo : 0;
    const Piece p = piece_of(u - o.u0, o.head, once ? 0 : o.lead, lo, o.hi);
    if (p.s >= p.t) return;
    const int32_t len = (int32_t)(p.t - p.s);                  // at most kUnit + kMaxLead - 1
    if (!once && p.t - lo >= 16) {
        const int64_t from = len < 16 ? p.t - 16 : p.s;        // a short piece takes bytes in front of it along
        const int32_t n = len < 16 ? 16 : len;
        move_16<K, NT, PACK, THROUGH>(o, from, (uint32_t)lane_place((int32_t)lane * 16, n), (int32_t)lane * 16 < n);
        if (n > (int32_t)kUnit && (int32_t)lane * 16 < n - (int32_t)kUnit)
            move_16<K, NT, PACK, THROUGH>(o, from, (uint32_t)lane_place((int32_t)(kUnit + lane * 16), n), true);
        return;
    }
    if ((int32_t)lane * 16 + 16 <= len) move_16<K, NT, PACK, THROUGH>(o, p.s, lane * 16, true);
    const int32_t whole = len & ~15;
    if ((int32_t)lane < len - whole) move_byte<K, PACK>(o, p.s + whole + lane);
}

// The first M KiB at most of the `len` bytes (at least 16) at byte `from` of the span, all loads of up to 32 chunks
// before the first use.
template <int K, int M, bool NT, bool THROUGH>
__device__ __forceinline__ void move_chunks(const Span<K> &o, int64_t from, int32_t len, bool twice, uint32_t lane)
{
    constexpr int R = K * M <= 32 ? K : 32 / M;
    u32x4 v[M] = {};
    uint32_t at[M];
#pragma unroll
    for (int c = 0; c < M; ++c) at[c] = lane_offset((uint32_t)lane_place((int32_t)(c * kUnit + lane * 16), len));
#pragma unroll
    for (int j = 0; j < K; j += R) {
        u32x4 t[R][M];
#pragma unroll
        for (int q = 0; q < R && j + q < K; ++q) {
#pragma unroll
            for (int c = 0; c < M; ++c) t[q][c] = ld16_at<NT>(o.s[j + q] + from, at[c]);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < R && j + q < K; ++q) {
#pragma unroll
            for (int c = 0; c < M; ++c) v[c] ^= t[q][c];
        }
    }
#pragma unroll
    for (int c = 0; c < M; ++c)
        if ((int32_t)(c * kUnit + lane * 16) + (twice ? 0 : 15) < len) {
            if constexpr (THROUGH) st16_through(o.d + from, at[c], v[c]);
            else st16_at<NT>(o.d + from, at[c], v[c]);
        }
}

// `n` units (at most U) of span o from u on together; as move_unit, where it says which bytes come twice.  us, one by one /
// so: decode of 2 sources in spans of 70 KB by 16 workgroups 387 / 301, packed 311 / 261; parity of 8 in spans of 10 KB by 64
// 0.64 / 0.55 of units of the stream; direct restore of 0.5 GB in spans of 10 KB 9913 / 9580; copies of 60,000 spans of
// 1500 bytes 42 / 33 (of 700 bytes, whose steps have two spans, 31 / 33).
template <int K, int U, bool NT, bool THROUGH>
__device__ __forceinline__ void move_units(const StreamArgs &a, const Span<K> &o, uint64_t u, uint32_t n, uint32_t lane)
{
    const bool once = a.last == kLastDest;
    const int64_t lo = o.lo > 0 ? o.lo : 0;
    const uint32_t lead = once ? 0 : o.lead;
    const Piece p = {piece_of(u - o.u0, o.head, lead, lo, o.hi).s, piece_of(u - o.u0 + n - 1, o.head, lead, lo, o.hi).t};
    if (p.s >= p.t) return;
    const bool twice = !once && p.t - lo >= 16;
    int32_t len = (int32_t)(p.t - p.s);                        // at most U * kUnit + kMaxLead - 1
    if (twice && len < 16) len = 16;
    const int64_t from = p.t - len;
    if (len >= 16) {
        if (U > 3 && len > 3 * (int32_t)kUnit) move_chunks<K, U, NT, THROUGH>(o, from, len, twice, lane);
        else if (U > 2 && len > 2 * (int32_t)kUnit) move_chunks<K, 3, NT, THROUGH>(o, from, len, twice, lane);
        else if (len > (int32_t)kUnit) move_chunks<K, 2, NT, THROUGH>(o, from, len, twice, lane);
        else move_chunks<K, 1, NT, THROUGH>(o, from, len, twice, lane);
        if (len > U * (int32_t)kUnit && (int32_t)lane * 16 < len - U * (int32_t)kUnit)
            move_16<K, NT, false, THROUGH>(o, from, (uint32_t)lane_place((int32_t)(U * kUnit + lane * 16), len), true);
    }
    if (!twice && (int32_t)lane < (len & 15)) move_byte<K, false>(o, p.s + (len & ~15) + lane);
}

// The U units from u on, and kRuns the steps behind them, up to `most` in all, as far as all their bytes are
// of span o and in the range; returns how many steps.
template <int K, int U, bool NT, Form F, bool THROUGH>
__device__ __forceinline__ uint32_t move_steps(const StreamArgs &a, const Span<K> &o, uint64_t u, uint32_t lane,
                                               uint32_t most)
{
    constexpr bool PACK = F == kPacked;
    constexpr int64_t S = U * (int64_t)kUnit;
    const bool once = F == kInPlace || a.last == kLastDest;
    const uint32_t lead = once ? 0 : o.lead;
    int64_t x = (int64_t)((u - o.u0) * kUnit + o.head + lead - kUnit);
    const bool whole = (u > o.u0 || x == 0) && x >= o.lo && x + S <= o.hi;
    if (!whole) return 0;
    // vmcnt(0), once in front of a run: the compiler may otherwise take registers for still in flight from
    // before and wait for them in every round, and with them for the stores of the round before (2 sources,
    // 126 MB by 4 workgroups: 2217 us so, 1583 with this; with 3 and 4 sources it takes 0.3 to 1 % itself)
    if constexpr (F == kRuns) __builtin_amdgcn_s_waitcnt(0x0f70);
    for (uint32_t done = 1;; ++done) {
        // all loads of up to 32 chunks before the first use
        constexpr int R = K * U <= 32 ? K : 32 / U;
        u32x4 v[U] = {};
        const uint32_t at = lane_offset(lane * 16);
#pragma unroll
        for (int j = 0; j < K; j += R) {
            u32x4 t[R][U];
#pragma unroll
            for (int q = 0; q < R && j + q < K; ++q) {
#pragma unroll
                for (int c = 0; c < U; ++c) t[q][c] = ld16_at<NT>(o.s[j + q] + x + c * kUnit, at);
            }
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (PACK) {
                if (j == 0) {
#pragma unroll
                    for (int c = 0; c < U; ++c) st16_at<NT>(o.d2 + x + c * kUnit, at, t[0][c]);
                }
            }
#pragma unroll
            for (int q = 0; q < R && j + q < K; ++q) {
#pragma unroll
                for (int c = 0; c < U; ++c) v[c] ^= t[q][c];
            }
        }
#pragma unroll
        for (int c = 0; c < U; ++c) {
            if constexpr (THROUGH) st16_through(o.d + x + c * kUnit, at, v[c]);
            else st16_at<NT>(o.d + x + c * kUnit, at, v[c]);
        }
        if constexpr (F != kRuns) return 1;
        x += S;
        if (done == most || x + S > o.hi) return done;
    }
}

// The workgroup (1, 2 or 4 waves) has no meaning beyond the dispatch, but that two waves share an L2 (in_pairs).
// Unless the caller caps the grid there is one wave per step, dispatched in order, so that the chip moves through its streams in
// narrow windows; that is what HBM likes best here (copy of 2 GiB by 1 KiB units: 6.6 TB/s with
// workgroups of 64 threads, 6.5 with 256, 6.2 with 1024; 4.8 - 5.9 with a persistent grid).
//
// kRuns (a grid of few waves, each with many units): a wave takes a.run consecutive steps together and
// looks up once for those that lie in one span; without, look-ups and data of its steps follow one
// another.  126 MB in spans of 3 MB by 4 / 16 / 64 workgroups, us, without and with: packed 1869 / 479 / 134
// and 1186 / 315 / 102 (tiles walked by workgroups: 1620 / 432 / 145), parity of 4: 3563 / 906 / 247 and
// 2593 / 677 / 196 (3168 / 817 / 253).
//
// D: see Deal.  (Where short spans are copied, what the kernel would have to ask and to work out for the orders costs 1 to 6 %,
// and launches of 20 to 80 us, whose waves are few, 1 to 2.)
template <int K, int U, bool NT, Form F = kPlain, Deal D = kAsNumbered, bool THROUGH = false>
__global__ void __launch_bounds__(256) k_stream(const StreamArgs a)
{
    const uint32_t lane = threadIdx.x & 63;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // all arguments at once: left alone, the compiler loads a few, looks whether there is work, and then loads the
    // others, and the first wave on a die waits for host memory twice
    asm volatile("" ::"s"(a.off), "s"(a.unit_off), "s"(a.unit_span), "s"(a.T), "s"(a.tab), "s"(a.last_row),
                 "s"(a.dest_row), "s"(a.vb), "s"(a.cbase), "s"(a.range.lo), "s"(a.range.hi), "s"(a.first_step), "s"(a.nsteps), "s"(a.waves),
                 "s"(a.unit_shift), "s"(a.grid), "s"(a.last), "s"(a.ragged), "s"(a.stride), "s"(a.spread));
    // kRuns: steps left of this run, and how many of them the last round moved
    uint32_t left = F == kRuns ? a.run : 1, done = 1;
    for (uint64_t w = ((uint64_t)blockIdx.x * a.waves + wave) * (F == kRuns ? a.run : 1); w < a.nsteps;
         w += F != kRuns ? a.stride : (left -= done) ? done : done + (a.stride - 1) * (left = a.run)) {
        // streaming launches only: the few instructions more delay a short one by 0.2 us
        uint64_t step = w;
        if (D == kFarAlone) step = unit_of_wave<U>(w, a.nsteps);
        if (D == kAnyOrder && a.spread)
            step = a.spread == kFar ? unit_of_wave<U>(w, a.nsteps)
                                    : a.spread == kNear ? near_step_of_wave(w, a.nsteps) : pair_step_of_wave(w, a.nsteps);
        uint64_t u = (a.first_step + step) * U;
        if (U > 1 && u < a.range.first) u = a.range.first;
        uint64_t end = (a.first_step + step + 1) * U;
        if (U > 1 && end > a.range.last + 1) end = a.range.last + 1;
        Span<K> o = load_span<K, D>(a, span_of(a, u, lane));
        const bool one = end - u == U && end <= o.u1;
        if (D == kAnyOrder && one) {
            u = turned<U>(u, o.u0, o.u1, o.turn);
            end = u + U;
        }
        if constexpr (U == 1 && F != kRuns) {
            move_unit<K, NT, F, THROUGH>(a, o, u, lane);
        } else {
            done = one ? move_steps<K, U, NT, F, THROUGH>(a, o, u, lane, left) : 0;
            if (done) continue;
            done = 1;
            for (;;) {
                const uint64_t part = end < o.u1 ? end : o.u1;
                if constexpr (K > kMaxSrc) {                // (as many loads as registers allow in one unit already)
                    for (; u < part; ++u) move_unit<K, NT, F, THROUGH>(a, o, u, lane);
                } else {
                    if (part - u == 1) move_unit<K, NT, F, THROUGH>(a, o, u, lane);
                    else move_units<K, U, NT, THROUGH>(a, o, u, (uint32_t)(part - u), lane);
                    u = part;
                }
                if (u == end) break;
                o = load_span<K, D>(a, span_of(a, u, lane));
            }
        }
    }
}

// Streams of tiny spans (kSmallMeanSpan): units of kSmallUnit bytes, each one's by 16 lanes, so that a wave moves four of
// them, U times over; what a wave knows of its span in k_stream, each lane loads here for its own.  Bound by the rate at
// which waves start (about 4 per ns) and by that chain of loads.  us, units of the stream (see above) / a wave per span
// / so: 100,000 spans of 40 bytes packed 8.8 / 24.4 / 7.5, parity of 8 32.3 / 40.7 / 19.9; of 300 bytes 19.9 / 26.0 / 16.7
// and 91.8 / 102 / 58; 4 MB in 300 by 16 workgroups, two units per lane in flight, 108 / 128 / 47 and 246 / 269 / 91.
template <int K, int U>
__global__ void __launch_bounds__(256) k_stream_small(const StreamArgs a)
{
    constexpr uint32_t G = kSmallUnit / 16, N = 64 / G;
    const uint32_t lane = threadIdx.x & 63, me = lane % G;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    for (uint64_t w = (uint64_t)blockIdx.x * a.waves + wave; w < a.nsteps; w += a.stride) {
        uint64_t u[U], i[U];
#pragma unroll
        for (int c = 0; c < U; ++c) {
            u[c] = a.range.first + (w * U + c) * N + lane / G;
            i[c] = entry(a.unit_span, u[c] < a.range.last ? u[c] : a.range.last) & ~kWholeBlock;
        }
        uint64_t b[U], e[U], u0[U], d[U], s[U][K];
#pragma unroll
        for (int c = 0; c < U; ++c) {
            b[c] = entry(a.off, i[c]);
            e[c] = entry(a.off, i[c] + 1);
            u0[c] = entry(a.unit_off, i[c]);
            d[c] = entry(a.dest_row, i[c]);
#pragma unroll
            for (int j = 0; j < K - 1; ++j) s[c][j] = entry(a.tab, (uint64_t)j * a.T + i[c]);
            s[c][K - 1] = entry(a.last_row, i[c]);
        }
        __builtin_amdgcn_sched_barrier(0);
        int64_t from[U], byte[U];              // where a lane's 16 bytes begin, and where its single byte lies
        bool wide[U], narrow[U];               // whether it has them
        u32x4 t[U][K];
#pragma unroll
        for (int c = 0; c < U; ++c) {
            if (!a.ragged) d[c] = a.vb + b[c];
            if (a.last == kLastContig) s[c][K - 1] = a.cbase + b[c];
            if (a.last == kLastDest) s[c][K - 1] = d[c];
            const int64_t first = (int64_t)(a.range.lo - b[c]), lo = first > 0 ? first : 0;
            const int64_t hi = (int64_t)((e[c] < a.range.hi ? e[c] : a.range.hi) - b[c]);
            const Piece p = piece_of(u[c] - u0[c], kSmallUnit, 0, lo, hi, kSmallUnit);
            const int32_t len = u[c] <= a.range.last && p.s < p.t ? (int32_t)(p.t - p.s) : 0;
            const int32_t at = (int32_t)me * 16, whole = len & ~15;
            // as in move_unit
            const bool twice = !a.once && p.t - lo >= 16;
            const int32_t n = twice && len < 16 ? 16 : len;
            from[c] = p.t - n + (twice ? lane_place(at, n) : at);
            wide[c] = len && at + (twice ? 0 : 15) < n;
            byte[c] = p.s + whole + me;
            narrow[c] = !twice && (int32_t)me < len - whole;
#pragma unroll
            for (int j = 0; j < K; ++j)        // (16 bytes that are there, where none are wanted)
                t[c][j] = ld16<false>(as_gc16(wide[c] ? s[c][j] + from[c] : (uint64_t)a.off));
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int c = 0; c < U; ++c) {
            if (wide[c]) {
                if (a.pack) st16_at<false>(a.vb2 + b[c] + from[c], 0, t[c][0]);
#pragma unroll
                for (int j = 1; j < K; ++j) t[c][0] ^= t[c][j];
                st16_at<false>(d[c] + from[c], 0, t[c][0]);
            }
            if (narrow[c]) {
                uint8_t x[K];
#pragma unroll
                for (int j = 0; j < K; ++j) x[j] = ld8(s[c][j] + byte[c]);
                if (a.pack) st8(a.vb2 + b[c] + byte[c], x[0]);
#pragma unroll
                for (int j = 1; j < K; ++j) x[0] ^= x[j];
                st8(d[c] + byte[c], x[0]);
            }
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

#define REFT_PICK_MANY(K)                                                                         \
    (cfg.nontemporal ? (cfg.unroll == 1 ? k_stream<K, 1, true> : k_stream<K, 2, true>)            \
                     : (cfg.unroll == 1 ? k_stream<K, 1, false> : k_stream<K, 2, false>))

// (only one source has two units a step in a launch that spreads them)
#define REFT_PICK_SPREAD(K)                                                                       \
    (cfg.unroll == 1 ? k_stream<K, 1, true, kPlain, kAnyOrder> : k_stream<K, K == 1 ? 2 : 1, true, kPlain, kAnyOrder>)

#define REFT_PICK_FAR(K)                                                                          \
    (cfg.unroll == 1 ? k_stream<K, 1, true, kPlain, kFarAlone> : k_stream<K, K == 1 ? 2 : 1, true, kPlain, kFarAlone>)

#define REFT_PICK_THROUGH(K)                                                                      \
    (cfg.unroll == 1 ? k_stream<K, 1, true, kPlain, kAnyOrder, true>                              \
                     : k_stream<K, K == 1 ? 2 : 1, true, kPlain, kAnyOrder, true>)

#define REFT_PICK_PACK(K)                                                                         \
    (through ? k_stream<K, 1, true, kPacked, kAnyOrder, K != 1>                                   \
     : a.spread == kFarUnturned ? k_stream<K, 1, true, kPacked, kFarAlone>                        \
     : a.spread ? k_stream<K, 1, true, kPacked, kAnyOrder>                                        \
                : cfg.nontemporal ? k_stream<K, 1, true, kPacked> : k_stream<K, 1, false, kPacked>)

#define REFT_PICK_RUNS(K) (cfg.nontemporal ? k_stream<K, 4, true, kRuns> : k_stream<K, 4, false, kRuns>)

#define REFT_PICK_IN_PLACE(K)                                                                     \
    (a.spread == kFarUnturned ? k_stream<K, 1, true, kInPlace, kFarAlone> : k_stream<K, 1, true, kInPlace, kAnyOrder>)

#define REFT_PICK_SMALL(K) (two ? k_stream_small<K, 2> : k_stream_small<K, 1>)

#define REFT_PICK_SMALL_MANY(K) k_stream_small<K, 1>

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

static hipError_t launch_small(StreamArgs a, int nsrc, Form form, const LaunchCfg &cfg, hipStream_t stream)
{
    void (*fn)(const StreamArgs) = nullptr;
    const bool two = cfg.capped && nsrc <= kMaxSrc;
    switch (nsrc) {
        REFT_CASES_4(REFT_PICK_SMALL) REFT_CASES_5_8(REFT_PICK_SMALL) REFT_CASES_9_16(REFT_PICK_SMALL_MANY)
    default: return hipErrorInvalidValue;
    }
    const uint64_t units = (two ? 2 : 1) * 64 / (kSmallUnit / 16);
    a.once = form == kInPlace || a.last == kLastDest;
    a.pack = form == kPacked;
    a.nsteps = (a.range.last - a.range.first) / units + 1;
    a.waves = 4;
    const uint32_t g = stream_grid(a.nsteps, a.waves, cfg.capped ? cfg.max_wgs : 0);
    a.stride = (uint64_t)g * a.waves;
    hipLaunchKernelGGL(fn, dim3(g), dim3(64 * a.waves), 0, stream, a);
    return hipGetLastError();
}

static hipError_t launch_stream(const PlanTables &pt, StreamArgs a, const uint64_t *dtab, int nsrc, Form form,
                                LaunchCfg cfg, hipStream_t stream)
{
    void (*fn)(const StreamArgs) = nullptr;
    const uint64_t traffic = (uint64_t)(nsrc + (form == kPacked ? 2 : 1)) * (a.range.hi - a.range.lo);
    const bool cached = traffic <= kCachedTraffic;
    // a capped grid (few waves, say on the host link) wants all that a wave may have in flight
    const uint32_t unroll = cfg.capped ? 4 : cached ? 1 : long_stream_unroll(nsrc);
    if (unroll < cfg.unroll) cfg.unroll = unroll;
    if (cached && !cfg.capped) cfg.nontemporal = false;
    if (nsrc > kMaxSrc && cfg.unroll > 2) cfg.unroll = 2;    // 2 KiB of 9 sources and more: 18 loads a lane
    if (form == kPacked || form == kInPlace) cfg.unroll = 1;
    a.first_step = a.range.first / cfg.unroll;
    a.nsteps = a.range.last / cfg.unroll - a.first_step + 1;
    const uint64_t mean = pt.L / pt.T;
    const uint32_t waves = cached || cfg.capped ? 4
                           : in_pairs(nsrc, mean, traffic, pt.odd, form == kPacked, dtab != nullptr, pt.windows) ? 2 : 1;
    a.off = pt.off;
    a.unit_off = pt.unit_off;
    a.unit_span = pt.unit_span;
    a.T = pt.T;
    a.unit_shift = pt.unit_shift;
    a.grid = pt.grid;
    if (a.last == kLastTable) a.last_row = a.tab + (uint64_t)(nsrc - 1) * pt.T;
    else a.last_row = pt.unit_off;
    a.ragged = dtab != nullptr;
    a.dest_row = dtab ? dtab : pt.unit_off;
    if (pt.unit == kSmallUnit) return launch_small(a, nsrc, form, cfg, stream);
    a.run = 1;
    a.spread = waves == 4 || !cfg.nontemporal || a.first_step % 32
                   ? kInOrder : spread_of(nsrc, mean, traffic, pt.odd, form == kPacked, a.ragged, pt.windows);
    const bool through = a.spread && form != kInPlace && writes_through(nsrc, mean, traffic, pt.odd, form == kPacked);
    if (form == kPlain && cfg.runs && cfg.unroll == 4) {
        a.run = run_of_units(a.nsteps, waves * (uint64_t)cfg.max_wgs, nsrc, mean);
        if (a.run > 1) form = kRuns;
    }
    switch (form) {
    case kPlain:
        if (through) {
            switch (nsrc) {
                REFT_CASES_4(REFT_PICK_THROUGH) REFT_CASES_5_8(REFT_PICK_THROUGH) REFT_CASES_9_16(REFT_PICK_THROUGH)
            default: return hipErrorInvalidValue;
            }
            break;
        }
        if (a.spread == kFarUnturned) {
            switch (nsrc) {
                REFT_CASES_4(REFT_PICK_FAR) REFT_CASES_5_8(REFT_PICK_FAR) REFT_CASES_9_16(REFT_PICK_FAR)
            default: return hipErrorInvalidValue;
            }
            break;
        }
        if (a.spread) {
            switch (nsrc) {
                REFT_CASES_4(REFT_PICK_SPREAD) REFT_CASES_5_8(REFT_PICK_SPREAD) REFT_CASES_9_16(REFT_PICK_SPREAD)
            default: return hipErrorInvalidValue;
            }
            break;
        }
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
    const uint32_t g = stream_grid((a.nsteps + a.run - 1) / a.run, waves, cfg.capped ? cfg.max_wgs : 0);
    a.waves = waves;
    a.stride = (uint64_t)g * waves;
    const uint32_t crowd = waves == 4 ? 32 : waves == 2 ? pair_waves(nsrc, mean, form == kPacked)
                           : through ? through_waves(nsrc, form == kPacked) : crowd_waves(nsrc, mean, form == kPacked);
    const uint32_t lds = waves * crowd_lds(crowd);
    hipLaunchKernelGGL(fn, dim3(g), dim3(64 * waves), lds, stream, a);
    return hipGetLastError();
}

hipError_t launch_gather(const PlanTables &pt, const uint64_t *tab, int nrows, bool acc, bool in_place,
                         const uint64_t *dtab, uint64_t dst_vbase, const StreamRange &range,
                         const LaunchCfg &cfg, hipStream_t stream)
{
    if (range.lo >= range.hi) return hipSuccess;
    if (range.hi > pt.L) return hipErrorInvalidValue;
    StreamArgs a{};
    a.tab = tab;
    a.vb = dst_vbase;
    a.range = range;
    a.last = acc ? kLastDest : kLastTable;
    return launch_stream(pt, a, dtab, nrows + (acc ? 1 : 0), in_place && !acc ? kInPlace : kPlain, cfg,
                         stream);
}

hipError_t launch_gather_pack(const PlanTables &pt, const uint64_t *tab, int nrows, uint64_t vb,
                              uint64_t vb2, const StreamRange &range, const LaunchCfg &cfg,
                              hipStream_t stream)
{
    if (range.lo >= range.hi) return hipSuccess;
    if (range.hi > pt.L) return hipErrorInvalidValue;
    StreamArgs a{};
    a.tab = tab;
    a.vb = vb;
    a.vb2 = vb2;
    a.range = range;
    a.last = kLastTable;
    return launch_stream(pt, a, nullptr, nrows, kPacked, cfg, stream);
}

hipError_t launch_scatter(const PlanTables &pt, const uint64_t *tab, uint64_t src_vbase,
                          const StreamRange &range, const LaunchCfg &cfg, hipStream_t stream)
{
    if (range.lo >= range.hi) return hipSuccess;
    if (range.hi > pt.L) return hipErrorInvalidValue;
    StreamArgs a{};
    a.cbase = src_vbase;
    a.range = range;
    a.last = kLastContig;
    return launch_stream(pt, a, tab, 1, kPlain, cfg, stream);
}

}  // namespace reft

// Grid sizes and launch rules (host arithmetic alone, without HIP, so that it can be checked at any size).
#pragma once
#include <stdint.h>

namespace reft {

// Workgroups of 64 * waves threads for a launch of one wave per unit: as many as the units need, at most
// `cap` (0: no cap), and so few that the work-items of the launch stay below 2^32, which is what HIP and
// the 32-bit grid size of a dispatch packet take (one-wave workgroups on 1 KiB units get there at 64 GiB
// of stream).  A wave takes more than one unit where there are fewer waves than units.
inline uint32_t stream_grid(uint64_t nunits, uint32_t waves, uint32_t cap)
{
    const uint64_t most = 0xffffffffull / (64ull * waves);
    uint64_t g = (nunits + waves - 1) / waves;
    if (cap && g > cap) g = cap;
    return (uint32_t)(g < most ? g : most);
}

// The stream kernel's units: every span is cut into pieces of `unit` bytes of its own.  The first one ends `head`
// bytes into the span (1 to `unit`), the last one with the span.  A unit has kUnit bytes, or, in streams of tiny spans
// (kSmallMeanSpan), kSmallUnit.
constexpr uint64_t kUnit = 1024, kSmallUnit = 256;
constexpr uint64_t units_of(uint64_t span_bytes, uint64_t head, uint64_t unit = kUnit)
{
    return span_bytes == 0 ? 0 : span_bytes <= head ? 1 : 1 + (span_bytes - head + unit - 1) / unit;
}

// At 700 bytes a span small units are better with few sources and worse with many (us, kUnit / kSmallUnit: packed 33.3 /
// 26.0, parity of 3 60 / 50, of 8 123 / 127, with the packed stream 133 / 143), below they win (k_stream_small).  At 512
// their numbers stay below 4 per span, so that each has its entry in the look-up table.
constexpr uint64_t kSmallMeanSpan = 512;
constexpr uint64_t unit_bytes(uint64_t L, uint64_t T)
{
    return L / T < kSmallMeanSpan && T < (1u << 29) ? kSmallUnit : kUnit;
}

// In streams of long spans (64 KiB on average) the units lie on the stream's own grid of KiB, and are numbered so that
// their numbers are the KiB's modulo `align` + 1 (some numbers between spans have no bytes): where a shard's tensors lie
// in memory in order, an XCD then keeps to the same address bits from span to span (see unit_of_wave; where they do not,
// turn_of sees to it inside each span).  Modulo 32 that holds for all the bits, but costs 16 numbers a span, which a
// capped grid's few waves look up in vain (spans of 70 KB, 64 workgroups, packed: 5 % more than modulo 8); so below 256
// KiB modulo 8, that is for the bits in which XCDs differ, but for one.  us, units that begin with their spans, in plain
// order / spread / on the grid modulo 8 / modulo 32 and spread: 8 x 0.6 GB in spans of 70 KB 1061 / 1007 / 971 / 964, 16 x
// 2030 / 1889 / 1825 / 1815; of 300 KB, 8 x 961 / 952 / 969 / 929, 12 x 1420 / 1384 / 1397 / 1356, 16 with the packed
// stream 2087 / 2015 / 2037 / 1983; a rotated unit and decode, 16 x 842 MB in pieces of 1.3 MB, 2481 spread, 2406 on the
// grid.  In other streams one more piece per span would cost more, and the spans' places have little to do with the units'
// numbers (8 x 132 MB in spans of 10 KB 204.6 us in plain order, 206.2 spread); and below 5 MiB no launch of 16 sources
// and two results at most leaves the cache, so that none would spread them (2 MB in spans of 300 KB 2.9 us, 3.1 on the
// grid).
constexpr uint64_t kGridMeanSpan = 64 * 1024, kWideMeanSpan = 256 * 1024, kGridMinBytes = 5 << 20;
constexpr uint32_t align_of(uint64_t L, uint64_t T)
{
    return L < kGridMinBytes || L / T < kGridMeanSpan ? 0 : L / T < kWideMeanSpan ? 7 : 31;
}
constexpr uint32_t grid_of(uint64_t L, uint64_t T) { return align_of(L, T) ? (uint32_t)kUnit - 1 : 0; }
constexpr uint64_t head_of(uint64_t off, uint64_t grid, uint64_t unit = kUnit) { return unit - (off & grid); }
constexpr uint64_t first_number(uint64_t least, uint64_t off, uint64_t align)
{
    return align ? least + ((off / kUnit - least) & align) : least;
}

// Unit j of a span moves its bytes [s, t), none if s >= t, as far as they lie in [lo, hi), which may reach below 0 or
// lie behind the span.  All units but the first start `lead` (below kMaxLead) bytes later than they otherwise would,
// the first moves those bytes as well.  Launches that turn their units move them to the KiB of the addresses, others,
// where the first unit's wave should not take twice as long as the rest, to the cache lines.
constexpr uint32_t kMaxLead = 1024, kLineLead = 128;
struct Piece {
    int64_t s, t;
};
constexpr Piece piece_of(uint64_t j, uint64_t head, uint32_t lead, int64_t lo, int64_t hi, uint64_t unit = kUnit)
{
    const int64_t t = (int64_t)(head + lead + j * unit), s = j ? t - (int64_t)unit : 0;
    return Piece{s < lo ? lo : s, t > hi ? hi : t};
}

// The first and the last of a span's units that may move its byte r, whatever its lead.
constexpr uint64_t last_unit_at(uint64_t r, uint64_t head, uint64_t unit = kUnit)
{
    return r < head ? 0 : 1 + (r - head) / unit;
}
constexpr uint64_t first_unit_at(uint64_t r, uint64_t head, uint64_t unit = kUnit)
{
    return last_unit_at(r < kMaxLead ? 0 : r - (kMaxLead - 1), head, unit);
}

// Where the 16 bytes lie that the lane at byte `at` (a multiple of 16) of a piece of `len` bytes moves: behind the
// piece's last whole 16 they are its last 16, which for len < 16 start in front of it.
constexpr int32_t lane_place(int32_t at, int32_t len) { return at + 16 <= len ? at : len - 16; }

// The unit that the w-th of n waves takes, where a wave is a workgroup of its own and has one unit of U KiB (1 or
// 2).  Workgroup w runs on XCD w mod 8, and KiB c of a buffer lies on the memory stack that bits 2 to 4 of c name, up
// to a constant that changes every half MiB to 2 MiB (bit 3 is the stack's I/O die; seen in the latencies of
// single loads from each XCD).  In plain order bits 0 to 2 are the XCD's own, so that for such a stretch it
// talks to half of the stacks.  Here it keeps bits 0, 1 and 4 (U = 2: 1, 2 and 4) and goes back and forth between the
// dies.  The units change places inside 32 KiB, the last incomplete 32 KiB stay in order.  TB/s, plain order and
// this one: 8 sources 6.02 and 6.30 (0.8 GB each), 6.30 and 6.44 (into tensors), 6.02 and 6.28 (with the packed
// stream), 16 sources 6.17 and 6.25, copies 6.37 and 6.58 (6.4 GB); 2 to 5 sources within 0.5 %.  Nothing else that
// was tried came near: the XCD on three other bits up to 12 costs up to 6 %, all stacks in turn 2 %.
template <uint32_t U>
constexpr uint64_t unit_of_wave(uint64_t w, uint64_t n)
{
    if ((w | 31) >= n) return w;
    if (U == 1) return (w & ~28ull) | (w >> 1 & 12) | (w & 4) << 2;
    return (w & ~12ull) | (w >> 1 & 4) | (w & 4) << 1;
}

// The same for odd streams (odd_stream): neighbouring steps that share cache lines meet in one L2 every second time, as the
// XCD keeps bits 1, 2 and 4 of the step.
constexpr uint64_t near_step_of_wave(uint64_t w, uint64_t n)
{
    if ((w | 31) >= n) return w;
    return (w & ~31ull) | (w << 1 & 6) | (w << 2 & 16) | (w >> 3 & 1) | (w >> 1 & 8);
}

// And where workgroups of two waves take neighbouring units (bit 0 of w is the wave), with the same bits the workgroup's.
constexpr uint64_t pair_step_of_wave(uint64_t w, uint64_t n)
{
    if ((w | 31) >= n) return w;
    return (w & ~24ull) | (w << 1 & 16) | (w >> 1 & 8);
}

// How far the units of a span are turned where steps are dealt in one of these orders: number x of the span (from 0) moves
// its unit x + turn, and behind the last one the first ones follow.  `number` is that of x = 0, `kib` the KiB of memory in
// which unit 0 would begin were it whole.  So a unit's number is its KiB's modulo 32 whatever the span's place in the stream,
// and an XCD keeps to its address bits.  In streams of odd sizes the numbers had nothing to do with the addresses: us,
// before and so, with the lead up to a whole KiB, in spans of 200 KB (log-uniform 50 : 65536) decode of 8 x 0.5 GB 741 / 707,
// of 4 409 / 400, parity of 8 754 / 743, copies 325 / 322; 1024 spans of 64 to 128 KiB, decode of 8 x 0.2 GB 341 / 337.
// Where the tensors lie in order already: 4139 / 4143 (8 x 3.1 GB), in shuffled order 3489 / 3463 (decode of 8 x 2.5 GB).
constexpr uint32_t kTurned = 32;                 // spans of as many units or fewer are not turned
constexpr uint32_t turn_of(uint64_t number, uint64_t kib) { return (uint32_t)(number - kib) & (kTurned - 1); }

// The unit from which on a step of U units is moved whose numbers u .. u + U - 1 are all of the span with the numbers u0 ..
// u1 - 1.  Whole steps change places among themselves (and turn by an even number where U is 2).
template <uint32_t U>
constexpr uint64_t turned(uint64_t u, uint64_t u0, uint64_t u1, uint32_t turn)
{
    const uint64_t first = (u0 + U - 1) / U * U, units = (u1 - first) / U * U;
    u += turn / U * U;
    return u < first + units ? u : u - units;
}

// Whether a stream is odd: most of its bytes (`bytes` of L) lie in spans whose places in it are no multiples of 64 bytes,
// which tensors' addresses are, so that the rows of a launch mostly do not lie alike.  Where a result lies otherwise than the
// sources, neighbouring units write parts of the same 64 bytes, and where a source does, they both read its line between
// them (8 x 132 MB in one span 187 us, the result 64 bytes off 190, 1 byte off 195, all eight sources apart 203).
constexpr bool odd_stream(uint64_t bytes, uint64_t L) { return bytes > L / 2; }

// The order in which a launch that streams (see kCachedTraffic) deals its steps to waves.
//
// In spans below 20 KiB on average the numbers of units mean too little (4 KB: 0 to +2 %, 7 KB 0 %, 14 KB -1 to +1 %,
// 28 KB -2 to -4 %), and copies, two units a wave, gain from 32 KiB on only (14 KB +1 %, 43 KB -2 %).
//
// Odd streams: two results, or two or three sources, in pairs (see in_pairs), a wave's neighbour in its own workgroup, so that both
// parts of a line that they share are in the same L2 at once.  Time of kFar / kNear / pairs, in spans of 14, 43 and 200 KB
// and 2 MB: with the packed stream, 2 sources 1 / .93 / .90, 1 / .92 / .92, 1 / .92 / .93 and 1 / .99 / .95, 5 sources 1 /
// .97 / .95, 1 / .97 / .95, 1 / .95 / .93 and 1 / .98 / .97, 8 sources 1 / .97 / .96, .97 / .97, .98 / .98, .98 / .99, 12
// sources 1 / 1 / 1.06, .99 / .99, .99 / .96, .99 / .95; parity of 2 1 / 1 / .96, .95 / .97, .94 / .96, .97 / .96.  One
// result and more sources, all alike but for the result: near, from 64 KiB and up to 12 sources (4 sources .99, .97, .98
// of kFar in 43 and 200 KB and 2 MB, 8 .99, .98, .98, 16 1.04, 1.05, .99); alike but for one source (decodes): far (near 0
// to 2 % more).  Rows that are windows at any offset: near up to 12 sources (3 .98, 7 and 11 .97 to .98), of 15 neither
// always (.98 to 1.03).  Copies: near up to 64 KiB (.98, far .99); in longer spans, of 4 to 12 GB of traffic, far .99 / .98, 1.00 /
// 1.00 and 1.00 / .985 of plain numbers (spans of 64 to 256 KB, up to 1 MB, longer; packed / unpacked), near .98 / 1.00, 1.04 / 1.03 and
// 1.02 / 1.00.
//
// Below 512 MiB of traffic units are not turned, and lie on the cache lines only, but where they go in pairs: a launch has few
// waves there, for which the first unit's longer way and what the kernel works out for turns come to more than the order of
// address bits saves (some of the data is in the 256 MB cache besides).  Time over that of units in plain numbers there, of
// launches one after the other on the same memory / on 4 to 8 sets in turn, turned / not turned and in a kernel that knows of no
// other order: 100 MiB 1.05 / 1.02 and 1.00 / 1.00, 130 MiB 1.04 / 1.01 and 1.00 / 1.00, 200 MiB 1.02 / 1.01 and 1.00 / 1.00, 480
// MiB 1.00 / 1.00 and 1.00 / 1.00 (the same for odd streams but for pairs; parity of 5 and more, of spans of 64 KiB and more,
// 1.04 / 1.02 and 1.00 / 1.00; copies 1.01 / 1.00 and 1.00 / 1.00, but odd ones in spans of 32 to 64 KiB .98 / .97 and .99 / .98).
// From there on, turned and not: 0.6 and 0.9 GiB .99, .99, 1.3 GiB .98, .98, 2 GiB .97, .98, 4 GiB .97, .98.
enum Spread : uint32_t {
    kInOrder = 0,
    kFar = 1,                // unit_of_wave
    kNear = 2,               // near_step_of_wave
    kPairs = 3,              // pair_step_of_wave
    kFarUnturned = 4,        // unit_of_wave
};
constexpr uint64_t kTurnTraffic = 512ull << 20;
constexpr uint64_t kSpreadMeanSpan = 20 * 1024, kSpreadMeanCopy = 32 * 1024, kNearMeanSpan = 64 * 1024;
constexpr uint64_t kShortMeanSpan = 5 * 1024, kMiddleMeanSpan = 12 * 1024;
// Whether a launch has workgroups of two waves.  In spans below 20 KiB for what pair_waves says of it, as long as that pays; time
// over that of single waves, on 132 / 400 MB a row (windows: 400 to 1200 MB a shard, cut by that), in spans of 3.5, 5, 7, 11,
// 14 and 18 KB.  Rows: 3, 4, 6 and 8 sources .95 to .995 / .91 to .95, .98 to 1.015 / .93 to .98, .97 to 1.00 / .94 to .985, .97
// to 1.00 / .97 to 1.04, .96 to 1.00 / .97 to 1.03, .97 to 1.00 / .985 to 1.02; 9 to 16 sources .95 to 1.00 / .95 to 1.00, but .97
// to 1.025 / .97 to 1.04, .99 to 1.03 / .99 to 1.04, .995 to 1.04 / 1.02 to 1.06, .98 to 1.03, .99 to 1.05.  Windows into
// tensors .91 to .98 up to 10 KB, .96 to .99 of 12 to 18 KB (up to 11 sources); into a unit, of 5 sources and more, .95 to 1.01
// up to 10 KB, 1.02 to 1.08 of 12 to 17 KB, of 3 and 4 sources .94 to .97, once 1.06.
//
// In longer spans from some traffic on.  Time over that of single waves, of launches one after the other on the same memory / on 4
// to 8 sets in turn, of 100, 130, 165, 205, 290 and 410 MiB: with the packed stream of 2 .97 / .95, .98 / .955, .95 / .94, .94 / .92,
// .92 / .92, .92 / .91, of 3 1.01 / .985, .99 / .97, .97 / .95, .98 / .95, .94 / .95, .94 / .93, of 4 to 8 1.02 to 1.05 / 1.00, 1.015 to
// 1.03 / .99 to 1.00, .99 to 1.01 / .98 to .99, .99 to 1.00 / .97 to .98, .965 to .99 / .96 to .98, .96 to .98 / .96 to .98, of 12 and 16
// 1.06 to 1.10 / 1.02 to 1.07, 1.05 / 1.02 to 1.03, 1.01 to 1.05 / 1.01 to 1.03, 1.02 to 1.03 / 1.01 to 1.02, 1.01 to 1.02 / 1.00 to
// 1.01, .99 / .99; rows, 2 sources 1.03 / 1.00, 1.02 / .99, 1.00 / .98, 1.00 / .98, .98 / .975, .985 / .975, 3 1.045 / 1.01, 1.04 / 1.00,
// 1.025 / .99, 1.005 / .99, 1.00 / .98, .985 / .975; and of 0.5, 1 GiB and more .92 to 1.00, .92 to .99, .88 to .98.
constexpr uint64_t kPairsOfMany = 4 * 1024, kPairsOfUnit = 11 * 1024;
constexpr uint64_t least_paired_traffic(uint32_t nsrc, bool packed)
{
    if (packed) return nsrc <= 3 ? 0 : nsrc <= 8 ? 160ull << 20 : 352ull << 20;
    return nsrc == 2 ? 144ull << 20 : 192ull << 20;
}
constexpr bool in_pairs(uint32_t nsrc, uint64_t mean_span, uint64_t traffic, bool odd, bool packed, bool tensors, bool windows)
{
    if (!odd) return false;
    if (mean_span >= kSpreadMeanSpan && !windows && traffic < least_paired_traffic(nsrc, packed)) return false;
    if (nsrc == 1) return !packed && mean_span >= kShortMeanSpan && mean_span < kSpreadMeanSpan;
    if (packed) return nsrc <= 8 || mean_span >= kSpreadMeanSpan;
    if (nsrc <= 3) return true;
    if (!windows) return mean_span < (nsrc <= 8 ? kSpreadMeanSpan : kPairsOfMany);
    if (!tensors) return mean_span < (nsrc == 4 ? kSpreadMeanSpan : kPairsOfUnit);
    return mean_span < (nsrc < 12 ? kSpreadMeanSpan : kMiddleMeanSpan);
}
constexpr Spread spread_of(uint32_t nsrc, uint64_t mean_span, uint64_t traffic, bool odd, bool packed, bool tensors, bool windows)
{
    if (mean_span < (nsrc == 1 && !packed ? kSpreadMeanCopy : kSpreadMeanSpan)) return kInOrder;
    if (in_pairs(nsrc, mean_span, traffic, odd, packed, tensors, windows)) return kPairs;
    if (odd && nsrc == 1 && !packed && mean_span < kNearMeanSpan) return kNear;
    if (traffic < kTurnTraffic) return kFarUnturned;
    if (!odd || packed || nsrc == 1) return kFar;
    return nsrc <= 12 && (windows || (!tensors && mean_span >= kNearMeanSpan)) ? kNear : kFar;
}

// LDS for one-wave workgroups to ask for, which they do not use, so that no more of them share a compute unit than its
// streams want (0: as many as fit): the more there are, the wider the windows in which the chip moves through memory.
// Swept from 8 to 30 requested waves on 0.1 to 14 GB, in spans of 10 KB to 10 MB (encode, decode, with packed stream,
// rotated, copies): with 4 sources and more the best is 16, 15, 14, 13, 12 (8 sources), 12, 11, 11, 10 (12), 9, 9, 8, 8,
// and one more or less costs 0.2 to 1 %.  (These are requests; in the blocks of 1280 bytes in which LDS is handed out
// 28, 24, 15, 13, 12, 11 and 10 come to 25, 21, 14, 12, 11, 10 and 9 waves.)  us, with 80 KiB in flight as the rule (22
// waves with 4 sources, 12 with 8, 8 from 12 on) / with this one: 4 sources 738 / 720, 5: 871 / 852, 9: 1392 / 1310, 10:
// 1482 / 1428, 12: 1779 / 1713.  All that fit / so many: 3 sources 582 / 575 in long spans, 370 / 342 (0.5 GB each) in
// short ones; 2 sources 273 / 263 in spans below a MiB, but 425 / 436 in longer ones; copies 3996 / 3911 and 567 / 559, in
// spans below 64 KiB 354 / 369; two copies of one source (with the packed stream) 319 / 328 (0.6 GB in spans of 70 KB).
constexpr uint32_t crowd_waves(uint32_t nsrc, uint64_t mean_span, bool packed)
{
    if (nsrc == 1) return mean_span >= 64 * 1024 && !packed ? 24 : 32;
    if (nsrc == 2) return mean_span < 1024 * 1024 ? 28 : 32;
    if (nsrc == 3) return 24;
    const uint32_t some = nsrc < 12 ? 20 - nsrc : 8, many = 17 - 5 * nsrc / 8;
    return some > many ? some : many > 8 ? many : 8;
}

// The same for workgroups of two waves.  In spans below 20 KiB a wave waits longer for its look-ups than for its data, the
// shorter they are the more, so that more waves keep as many bytes in flight; swept from 8 to 32 on 0.5 to 2 GB (what it gives
// is said at in_pairs; over pairs of waves, as many as crowd_waves says, with the packed stream of 2 .96, .97, .99, 1 in spans
// of 2.5, 3.5, 7 and 14 KB, of 4 .97, .98, 1, 1).  In longer spans, 28, 24 and 20 waves with the packed stream of 2 358 / 343
// / 333 us, of 3 447 / 429 / 418 (200 KB).
constexpr uint32_t pair_waves(uint32_t nsrc, uint64_t mean_span, bool packed)
{
    constexpr uint32_t least[3][12] = {{32, 32, 32, 28, 24, 20, 20, 16, 14, 16, 16, 16},
                                       {32, 32, 32, 28, 20, 16, 16, 14, 12, 14, 14, 14},
                                       {32, 32, 28, 24, 20, 16, 16, 14, 12, 12, 12, 12}};
    const uint32_t usual = crowd_waves(nsrc, mean_span, packed);
    if (mean_span >= kSpreadMeanSpan) return packed && nsrc <= 3 ? 20 : usual;
    if (!packed) return nsrc >= 12 ? 12 : least[mean_span < kShortMeanSpan ? 0 : mean_span < kMiddleMeanSpan ? 1 : 2][nsrc];
    if (nsrc <= 3) return nsrc == 2 && mean_span < kMiddleMeanSpan ? 28 : 24;
    return nsrc <= 6 && mean_span < kShortMeanSpan ? usual + 2 : usual;
}

// Whether a launch writes its results through the L2 (st16_through): in spans long enough for an XCD to keep to its address
// bits, and far more than the cache holds.  In odd streams partial lines from both sides go to memory one by one: 1.00 to 1.08 of
// the time.
//
// Time over that of results that wait in the L2 to be evicted, with loads as they were there, on the same memory in one process:
// tensors of a job one behind the other, each allocated by itself, in a heap full of holes, and as a benchmark's job has them,
// 0.16 to 11.8 GB a row.  Spans of 1 MB and more, parity of 2 .93 to 1.01, of 3 .92 to .98, of 4 .93 to 1.00, of 5 .93 to .99, of 6
// to 8 .96 to 1.00, of 10 to 16 .98 to 1.00; decodes of 2 and 3 .92 to .99, of 4 .94 to 1.00, of 5 .94 to .99, of 6 to 12 .98 to
// 1.00; with the packed stream of 2 .91 to .98 (1.0 MB: .96 to 1.02), of 3 .94 to .98, of 5 and 8 .93 to .98, of 12 .98 to 1.00.
// (With five sources and more stores alone, of the two changes, .97 to 1.00, loads alone .98 to 1.01, both together the least
// nearly everywhere.  In six processes, on two sets of memory each, parity and decode of 8 x 3.1 GB .982 to .988, of 8 x 2.5 GB
// .981 to .992, where one set differs from another by up to 4 %.)  Spans of 150, 200, 300 and 600 KB: parity of 2, 3 and 4 .99 to
// 1.07, .96 to 1.08 and .98 to 1.07, decodes .97 to 1.06, .95 to 1.05 and .98 to 1.04, with the packed stream of 2 .96 to 1.07; but
// parity of 5 .95 to 1.01, of 8 .95 to .99, of 10 to 16 .98 to 1.01, decodes of 5 to 12 .95 to 1.00, with the packed stream of 3, 5
// and 8 .92 to 1.01.  Below 0.5 GB of traffic 1.00 to 1.06 (some of it would have stayed in the 256 MB cache).
//
// Copies, 0.5 / 1.2 / 2.4 / 5 to 13 GB of traffic: spans of 1.2 MB 1.04 / 1.01 to 1.03 / 1.00 to 1.01 / .99 to 1.01, of 2.5 MB 1.03 /
// 1.00 to 1.02 / .99 to 1.01 / .99 to 1.01, of 8 MB 1.03 / 1.00 to 1.02 / .99 to 1.01 / .98 to 1.00, of 40 MB - / .99 to 1.01 / .99 /
// .98 to .99; of 0.15 to 0.6 MB .97 to 1.06.
//
// Where the results lie makes no difference to that: 2 to 12 sources, spans of 1 to 10 MB, results 1, 4, 16 or 32 bytes off a cache
// line .91 to 1.00, as on one; a tenth to nearly half of the stream at odd places .93 to .99; copies of 8 and 40 MB spans, 2.4 GB
// of traffic and more, .99 to 1.02 at such places (1.002 on average).
//
// How many waves then share a compute unit (see crowd_waves), swept from 6 to 32 on 1.7 to 28 GB: copies (25.8 GB) 3893 us
// with 24 as they were, 3862 / 3815 / 3823 written through with 24 / 20 / 18, 835 / 831 / 824 / 824 (5.6 GB), parity of 3
// sources 1032 / 962 us with 24 / 18, of 4 1283 / 1203 with 16 / 15; with the packed stream of 2 350 / 340 with 28 / 20,
// of 3 442 / 434 with 24 / 16, of 4 534 / 519 with 16 / 14, of 5 634 / 626 with 15 / 13, of 8 2600 / 2554 with 12 / 10.
constexpr uint64_t kThroughMeanSpan = 128 * 1024, kThroughMeanFew = 1024 * 1024, kThroughTraffic = 512ull << 20;
constexpr uint64_t kThroughMeanCopy = 4096 * 1024, kThroughTrafficCopy = 2ull << 30;
static_assert(kTurnTraffic <= kThroughTraffic);       // (no kernel that writes through knows kFarUnturned)
constexpr bool writes_through(uint32_t nsrc, uint64_t mean_span, uint64_t traffic, bool odd, bool packed)
{
    if (odd) return false;
    if (nsrc == 1) return !packed && mean_span >= kThroughMeanCopy && traffic >= kThroughTrafficCopy;
    return mean_span >= (nsrc <= (packed ? 2u : 4u) ? kThroughMeanFew : kThroughMeanSpan) && traffic >= kThroughTraffic;
}
constexpr uint32_t through_waves(uint32_t nsrc, bool packed)
{
    if (packed) return nsrc == 2 ? 20 : nsrc == 3 ? 16 : nsrc < 11 ? 18 - nsrc : crowd_waves(nsrc, kThroughMeanSpan, true);
    return nsrc == 1 || nsrc == 3 ? 18 : nsrc == 4 ? 15 : crowd_waves(nsrc, kThroughMeanSpan, false);
}
constexpr uint32_t crowd_lds(uint32_t waves) { return waves == 32 ? 0 : 160 * 1024 / waves / 512 * 512; }

// Consecutive units that a wave of a capped grid takes together.  Runs pay where a wave waits on look-ups for
// units inside long spans (spans of 70 KB by 8 workgroups: 46 us without, 51 with), with up to four sources
// (5 by 64 workgroups: 224 us without, 240 with), and up to this many waves, beyond which more windows in
// memory cost more than look-ups (1 GB copied by 192 / 256 workgroups: 445 / 361 us without, 367 / 382
// with; parity of 2 by 128 / 192: 804 / 590 without, 613 / 539 with).  Eight runs per wave keep the waves busy alike;
// beyond 16 units nothing is gained.
inline uint32_t run_of_units(uint64_t nunits, uint64_t waves, uint32_t nsrc, uint64_t mean_span)
{
    const uint64_t n = nunits / (8 * waves);
    if (nsrc > 4 || waves > (nsrc == 1 ? 896u : nsrc == 2 ? 768u : 384u) || mean_span < 256 * 1024) return 1;
    return n < 1 ? 1 : n < 16 ? (uint32_t)n : 16;
}

// Cap on the workgroups of a kernel bound by the host link: `halves` halves of link_wgs, but never more
// than the caller's (or the default) cap on any kernel.
inline uint32_t link_cap(uint64_t link_wgs, uint32_t halves, uint32_t max_wgs)
{
    const uint64_t w = link_wgs * halves / 2;
    return (uint32_t)(w < max_wgs ? w : max_wgs);
}

// "burst_min_rows" and "burst_min_bytes" where the caller has not set them, for the kernels over span tables.  Since its
// units lie in the order of unit_of_wave the stream kernel is as good or better up to about 12 GB a row.  Time of the
// burst kernel over the stream kernel's, in turn in one process, four places of memory each: parity of 8 rows of 3.1 GB
// 1.03, 1.01, 7 of 3.1 GB 1.02; 8 of 11.8 GB 1.025, 1.011, 1.000, 1.003, of 11.4 GB 0.999, 1.006, 0.996, 0.998, of 15.0 GB
// 1.001, 0.993, 0.998, 0.991, of 15.4 GB 1.003, 0.996, 0.994, 0.997; 7 of 11.8 GB 1.028 to 1.005, of 15.0 GB 1.004, 1.000,
// 0.998, 0.996, of 15.4 GB 1.010, 0.999, 0.993, 0.997.  Into tensors, 7 and 8 rows of 11.4 to 15.4 GB, 1.002 to 1.024 (so
// only from four times the bytes on, more than the memory holds).  Since results are written through (writes_through), 8
// rows of 15.0 GB 0.9985, 0.9983, 0.9979, 0.9933, 0.9970 on five sets of a Llama-shaped job's tensors, 1.010 and 1.012 on two
// made one after the other: a tie by where the tensors lie, so the rows stay.
constexpr uint64_t kBurstMinRows = 7, kBurstMinBytes = 13ull << 30;

// The same two for reft_reconstruct.  Its ordinary kernel (tiles, a persistent grid) mixes reads and writes
// worse than the one over span tables: there the burst kernel pays from five sources and 8 MiB on (5 sources
// 6.05 / 6.16 TB/s, ordinary / burst, 8 sources 5.23 / 6.47).  What the caller sets holds for both.
inline uint64_t contig_burst_min_rows(uint64_t rows) { return rows == kBurstMinRows ? 5 : rows; }
inline uint64_t contig_burst_min_bytes(uint64_t bytes) { return bytes == kBurstMinBytes ? 8ull << 20 : bytes; }

}  // namespace reft

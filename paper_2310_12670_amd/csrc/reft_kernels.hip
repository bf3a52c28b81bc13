// HIP kernels of libreft for gfx950 (CDNA4): the write-burst XOR kernels and the contiguous k-way XOR
// (single-loss decode from packed streams).  The ragged gather / scatter kernel is in reft_stream.hip.
//
// All are HBM-streaming kernels: no arithmetic beyond a 128-bit XOR per 16 bytes and source, so the
// design goal is full-width, coalesced 16-byte accesses with enough of them in flight per compute
// unit.  The contiguous kernel's workgroups (256 threads) walk tiles of 2^tile_shift bytes with a
// grid-stride loop; consecutive workgroups take consecutive tiles, so the eight XCDs (workgroups are
// dealt to them round-robin) stream through neighbouring addresses together.
#include "reft_device.hpp"

#include <map>
#include <mutex>
#include <tuple>
#include <utility>

namespace reft {

// Where the bytes of a piece go: to their global address, or into an LDS image of a destination
// range (image byte 0 stands for the 16-byte aligned address `origin`), from which another wave
// stores them later.
#define REFT_LDS __attribute__((address_space(3)))
struct ToGlobal {
    template <bool NT>
    __device__ __forceinline__ void put16(uint64_t a, u32x4 v) const { st16<NT>(as_g16(a), v); }
    __device__ __forceinline__ void put8(uint64_t a, uint8_t v) const { st8(a, v); }
};
struct ToImage {
    REFT_LDS unsigned char *img;
    uint64_t origin;
    template <bool NT>
    __device__ __forceinline__ void put16(uint64_t a, u32x4 v) const
    {
        *(REFT_LDS u32x4 *)(img + (uint32_t)(a - origin)) = v;
    }
    __device__ __forceinline__ void put8(uint64_t a, uint8_t v) const { img[(uint32_t)(a - origin)] = v; }
};

// One piece: n bytes at destination address d = XOR of the n bytes at each source address s[j].
// The whole workgroup cooperates.  Destination stores are 16-byte aligned: up to 15 head bytes
// and 15 tail bytes are moved bytewise, the body as 16-byte chunks, U in flight per thread and
// source, whatever the sources' alignment.
template <int K, int U, bool NT, class Sink = ToGlobal>
__device__ __forceinline__ void xor_piece(uint64_t d, const uint64_t (&s)[K], uint32_t n,
                                          const Sink sink = Sink())
{
    const uint32_t tid = threadIdx.x;
    uint32_t head = (uint32_t)(0 - d) & 15u;
    if (head > n) head = n;
    const uint32_t body = n - head;
    const uint32_t nb = body >> 4;
    const uint32_t tail = body & 15u;

    if (tid < 32) {
        uint32_t i = 0xffffffffu;
        if (tid < head) i = tid;
        else if (tid >= 16 && tid - 16 < tail) i = head + (nb << 4) + (tid - 16);
        if (i != 0xffffffffu) {
            uint8_t v = ld8(s[0] + i);
#pragma unroll
            for (int j = 1; j < K; ++j) v ^= ld8(s[j] + i);
            sink.put8(d + i, v);
        }
    }
    if (nb == 0) return;

    const uint64_t da = d + head;
    gcptr16 sp[K];
#pragma unroll
    for (int j = 0; j < K; ++j) sp[j] = as_gc16(s[j] + head);
    constexpr uint32_t step = kThreads * U;
    const uint32_t full = nb / step * step;
    for (uint32_t c = tid; c < full; c += step) {
        u32x4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = ld16<NT>(sp[0] + c + u * kThreads);
#pragma unroll
        for (int j = 1; j < K; ++j) {
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] ^= ld16<NT>(sp[j] + c + u * kThreads);
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            sink.template put16<NT>(da + ((uint64_t)(c + u * kThreads) << 4), v[u]);
    }
    for (uint32_t c = full + tid; c < nb; c += kThreads) {
        u32x4 v = ld16<NT>(sp[0] + c);
#pragma unroll
        for (int j = 1; j < K; ++j) v ^= ld16<NT>(sp[j] + c);
        sink.template put16<NT>(da + ((uint64_t)c << 4), v);
    }
}

// ------------------------------------------------------------------------------------------------
// Gather with write bursts (many sources, one pass).
//
// Measured on this part: a stream of reads runs at about 7 TB/s, but as soon as writes are mixed
// into it, even a few, the whole stream drops to 5.2 - 5.9 TB/s; the same bytes written in short
// chip-wide bursts cost far less.  So this variant separates the two in time.  A workgroup has
// four reader waves and one writer wave.  The readers XOR one stage (stage_bytes of the stream)
// after another into the two halves of an LDS double buffer and never touch the destination.
// The writer wave stores stage r-1 from its half while the readers fill the other half with stage
// r - but not before every workgroup of the grid has finished reading its stage r-1, so that
// all writer waves of the chip fire together.  That meeting is only a matter of timing: it is a
// counter the writer wave polls at most max_polls times per round (readers never wait for another
// workgroup), a writer that polls in vain stops waiting for the next 1, 2, 4, ... 64 rounds (so a
// slow workgroup, or one that is not resident, costs the others next to nothing), and the result
// does not depend on it.  The grid is persistent (the launch wrappers size it so that all
// workgroups are resident); workgroup b takes stages b, b + grid, ...
//
// The LDS image of a stage is laid out like the destination: the byte of stream offset o sits
// where address vb + o would fall relative to a 16-byte boundary.  For a contiguous destination
// vb is its virtual base.  For a ragged one (dtab), every span's place must have the same
// alignment relative to its stream offset, (dtab[i] - off[i]) mod 16 = vb mod 16 for all spans
// with bytes (the host checks this); then aligned 16-byte chunks of the image are aligned
// 16-byte chunks of every destination span.
//
// ctr: 9 counters kCtrStride words apart, all zero at launch.  Workgroups arrive on counter
// (blockIdx.x & 7); every arrival that completes a multiple of the group's size bumps counter 8,
// the only one polled, so counter 8 tells how many rounds the groups have completed between them.
// ------------------------------------------------------------------------------------------------
constexpr int kBurstThreads = kThreads + 64;
constexpr uint32_t kCtrStride = 64;

// One wave moves len bytes from an LDS image to global address d (img is the byte for d; img and d
// have the same alignment mod 16).
template <bool NT>
__device__ __forceinline__ void emit_piece(uint64_t d, REFT_LDS const unsigned char *img,
                                           uint32_t len, uint32_t lane)
{
    uint32_t head = (uint32_t)(0 - d) & 15u;
    if (head > len) head = len;
    const uint32_t nb = (len - head) >> 4;
    const uint32_t tail = (len - head) & 15u;
    if (lane < head) {
        st8(d + lane, img[lane]);
    } else if (lane >= 16 && lane - 16 < tail) {
        const uint32_t b = head + (nb << 4) + (lane - 16);
        st8(d + b, img[b]);
    }
    if (nb) {
        gptr16 dp = as_g16(d + head);
        REFT_LDS const u32x4 *ip = (REFT_LDS const u32x4 *)(img + head);
#pragma unroll 8
        for (uint32_t c = lane; c < nb; c += 64) st16<NT>(dp + c, ip[c]);
    }
}

// The rounds of a burst kernel.  read(st, img) is run by the 256 reader threads and puts stage st
// into the LDS image at img; emit(st, img, lane) is run by the writer wave and stores the image.
template <class Read, class Emit>
__device__ __forceinline__ void burst_rounds(uint64_t nstages, uint32_t stage, uint32_t *ctr,
                                             uint32_t max_polls, uint32_t nap, Read read, Emit emit)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char burst_lds[];
    REFT_LDS unsigned char *lds = (REFT_LDS unsigned char *)burst_lds;
    const uint32_t half = stage + 16;                  // an image may start up to 15 bytes in
    const uint32_t lane = threadIdx.x & 63;
    const bool writer = threadIdx.x >= kThreads;
    const uint32_t G = gridDim.x, g = blockIdx.x & 7;
    const uint64_t rounds = (nstages + G - 1) / G;
    const uint32_t members = (G - g + 7) >> 3;         // workgroups that arrive on counter g
    const uint32_t ngroups = G < 8 ? G : 8;
    uint32_t skip = 0, backoff = 0;                    // writer wave: rounds left without waiting
    // writer wave, lane 0: how its rounds went (met, timed out, not waited), kept in LDS behind
    // the two images so that the bookkeeping costs the kernels no registers
    REFT_LDS uint32_t *tally = (REFT_LDS uint32_t *)(lds + 2 * half);
    if (threadIdx.x == kThreads) tally[0] = tally[1] = tally[2] = 0;

    for (uint64_t r = 0; r <= rounds; ++r) {
        if (!writer) {
            const uint64_t st = r * G + blockIdx.x;
            if (r < rounds && st < nstages) read(st, lds + (uint32_t)(r & 1) * half);
        } else if (r > 0) {
            if (skip) {
                --skip;
                if (lane == 0) tally[2] += 1;
            } else if (max_polls) {
                const uint32_t want = ngroups * (uint32_t)r;   // every group done with round r-1
                for (uint32_t n = 0;;) {
                    uint32_t v = 0;
                    if (lane == 0)
                        v = __hip_atomic_load(ctr + 8 * kCtrStride, __ATOMIC_RELAXED,
                                              __HIP_MEMORY_SCOPE_AGENT);
                    v = __builtin_amdgcn_readfirstlane(v);
                    if (v >= want) {
                        backoff = 0;
                        if (lane == 0) tally[0] += 1;
                        break;
                    }
                    if (++n >= max_polls) {
                        // a straggler: write without the others for 1, 2, 4, ... 64 rounds
                        backoff = backoff == 0 ? 1 : backoff < 64 ? backoff * 2 : 64;
                        skip = backoff;
                        if (lane == 0) tally[1] += 1;
                        break;
                    }
                    for (uint32_t z = 0; z < nap; ++z) __builtin_amdgcn_s_sleep(16);
                }
            }
            const uint64_t st = (r - 1) * G + blockIdx.x;
            if (st < nstages) emit(st, lds + (uint32_t)((r - 1) & 1) * half, lane);
        }
        __syncthreads();       // stage r is complete in LDS; stage r-1 has left its half
        if (writer && lane == 0 && r < rounds && max_polls) {
            const uint32_t old = __hip_atomic_fetch_add(ctr + g * kCtrStride, 1u, __ATOMIC_RELAXED,
                                                        __HIP_MEMORY_SCOPE_AGENT);
            if ((old + 1) % members == 0)     // whichever round the arriving workgroup is in
                __hip_atomic_fetch_add(ctr + 8 * kCtrStride, 1u, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    // diagnostics (three adds per workgroup and launch): rounds in which the writer wave saw the
    // meeting complete, ran out of polls, or did not wait at all
    if (writer && lane == 0 && max_polls) {
        uint32_t *diag = ctr + kBurstDiagWord;
        __hip_atomic_fetch_add(diag + 0, tally[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_fetch_add(diag + 1, tally[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_fetch_add(diag + 2, tally[2], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

template <int K, int U, bool NT>
__global__ void __launch_bounds__(kBurstThreads)
k_gather_burst(PlanTables pt, const uint64_t *__restrict__ tab, const uint64_t *__restrict__ dtab,
               uint64_t vb, uint64_t lo, uint64_t hi, uint32_t stage, uint32_t *ctr,
               uint32_t max_polls, uint32_t nap)
{
    const uint64_t nstages = (hi - lo + stage - 1) / stage;
    burst_rounds(
        nstages, stage, ctr, max_polls, nap,
        [&](uint64_t st, REFT_LDS unsigned char *img) {
            uint64_t o = lo + st * stage;
            uint64_t e = o + stage;
            if (e > hi) e = hi;
            const ToImage sink{img, (vb + o) & ~15ull};
            uint32_t i = pt.tile_span[o >> pt.tile_shift];
            while (o < e) {
                // o < e <= L = off[T], so a span with off[i+1] > o exists at or after i
                while (pt.off[i + 1] <= o) ++i;
                const uint64_t so = pt.off[i];
                uint64_t pe = pt.off[i + 1];
                if (pe > e) pe = e;
                uint64_t s[K];
#pragma unroll
                for (int j = 0; j < K; ++j) s[j] = tab[(uint64_t)j * pt.T + i] + (o - so);
                xor_piece<K, U, NT, ToImage>(vb + o, s, (uint32_t)(pe - o), sink);
                o = pe;
            }
        },
        [&](uint64_t st, REFT_LDS const unsigned char *img, uint32_t lane) {
            uint64_t o = lo + st * stage;
            const uint64_t e = o + stage < hi ? o + stage : hi;
            // image byte of stream offset x: img0[x - o]
            REFT_LDS const unsigned char *img0 = img + ((uint32_t)(vb + o) & 15u);
            if (dtab == nullptr) {
                emit_piece<NT>(vb + o, img0, (uint32_t)(e - o), lane);
            } else {
                const uint64_t o0 = o;
                uint32_t i = pt.tile_span[o >> pt.tile_shift];
                while (o < e) {
                    while (pt.off[i + 1] <= o) ++i;
                    const uint64_t so = pt.off[i];
                    const uint64_t pe = pt.off[i + 1] < e ? pt.off[i + 1] : e;
                    emit_piece<NT>(dtab[i] + (o - so), img0 + (uint32_t)(o - o0), (uint32_t)(pe - o),
                                   lane);
                    o = pe;
                }
            }
        });
}

// dst[i] = XOR_j src.p[j][i], i in [0, L), with write bursts
template <int K, int U, bool NT>
__global__ void __launch_bounds__(kBurstThreads)
k_xor_contig_burst(SrcBases src, uint64_t dst, uint64_t L, uint32_t stage, uint32_t *ctr,
                   uint32_t max_polls, uint32_t nap)
{
    const uint64_t nstages = (L + stage - 1) / stage;
    burst_rounds(
        nstages, stage, ctr, max_polls, nap,
        [&](uint64_t st, REFT_LDS unsigned char *img) {
            const uint64_t o = st * stage;
            const uint64_t n = L - o < stage ? L - o : stage;
            uint64_t s[K];
#pragma unroll
            for (int j = 0; j < K; ++j) s[j] = src.p[j] + o;
            xor_piece<K, U, NT, ToImage>(dst + o, s, (uint32_t)n, ToImage{img, (dst + o) & ~15ull});
        },
        [&](uint64_t st, REFT_LDS const unsigned char *img, uint32_t lane) {
            const uint64_t o = st * stage;
            const uint64_t n = L - o < stage ? L - o : stage;
            emit_piece<NT>(dst + o, img + ((uint32_t)(dst + o) & 15u), (uint32_t)n, lane);
        });
}

__global__ void k_zero_words(uint32_t *p, uint32_t n)
{
    for (uint32_t i = threadIdx.x; i < n; i += blockDim.x) p[i] = 0;
}

// dst[i] = XOR_j src.p[j][i], i in [0, L)
template <int K, int U, bool NT>
__global__ void __launch_bounds__(kThreads)
k_xor_contig(SrcBases src, uint64_t dst, uint64_t L, uint32_t sh)
{
    const uint64_t ntiles = (L + (1ull << sh) - 1) >> sh;
    for (uint64_t t = blockIdx.x; t < ntiles; t += gridDim.x) {
        const uint64_t o = t << sh;
        uint64_t n = L - o;
        if (n > (1ull << sh)) n = 1ull << sh;
        uint64_t s[K];
#pragma unroll
        for (int j = 0; j < K; ++j) s[j] = src.p[j] + o;
        xor_piece<K, U, NT>(dst + o, s, (uint32_t)n);
    }
}

// ------------------------------------------------------------------------------------------------
// launch wrappers: pick the instantiation for (number of sources, unroll, non-temporal)
// ------------------------------------------------------------------------------------------------
static uint32_t grid_for(uint64_t ntiles, const LaunchCfg &cfg)
{
    uint64_t g = ntiles < cfg.max_wgs ? ntiles : cfg.max_wgs;
    return (uint32_t)(g < 1 ? 1 : g);
}

// Workgroups of the burst kernel that fit on one compute unit with `lds` bytes of LDS each
// (looked up once per instantiation; the first call also lifts the kernel's LDS limit).
static hipError_t burst_occupancy(const void *fn, size_t lds, int *per_cu)
{
    static std::mutex mu;
    static std::map<std::tuple<int, const void *, size_t>, int> known;   // per device
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    std::lock_guard<std::mutex> lock(mu);
    auto it = known.find(std::make_tuple(dev, fn, lds));
    if (it == known.end()) {
        e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        int n = 0;
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, fn, kBurstThreads, lds);
        if (e != hipSuccess) return e;
        it = known.emplace(std::make_tuple(dev, fn, lds), n).first;
    }
    *per_cu = it->second;
    return hipSuccess;
}

static bool burst_cfg_ok(const BurstCfg &bc)
{
    return bc.ctr && bc.stage_bytes >= 4096 && bc.stage_bytes % 4096 == 0 &&
           bc.stage_bytes <= 65536 && bc.wgs_per_cu >= 1 && bc.num_cus >= 1;
}

// Grid of a burst launch: every workgroup resident at once.
static hipError_t burst_grid(const void *fn, uint64_t nstages, const LaunchCfg &cfg,
                             const BurstCfg &bc, size_t *lds, uint32_t *grid)
{
    *lds = 2 * ((size_t)bc.stage_bytes + 16) + 16;         // an image per half and the writer's tally
    int per_cu = 0;
    hipError_t e = burst_occupancy(fn, *lds, &per_cu);
    if (e != hipSuccess) return e;
    if (per_cu < 1) return hipErrorInvalidValue;
    if ((uint32_t)per_cu > bc.wgs_per_cu) per_cu = (int)bc.wgs_per_cu;
    uint64_t g = (uint64_t)per_cu * bc.num_cus;
    if (g > cfg.max_wgs) g = cfg.max_wgs;
    if (g > nstages) g = nstages;
    *grid = (uint32_t)g;
    return hipSuccess;
}

hipError_t launch_gather_burst(const PlanTables &pt, const uint64_t *tab, int nrows,
                               const uint64_t *dtab, uint64_t vb, uint64_t lo, uint64_t hi,
                               const LaunchCfg &cfg, const BurstCfg &bc, hipStream_t stream)
{
    if (lo >= hi) return hipSuccess;
    if (hi > pt.L || !burst_cfg_ok(bc)) return hipErrorInvalidValue;
    void (*fn)(PlanTables, const uint64_t *, const uint64_t *, uint64_t, uint64_t, uint64_t,
               uint32_t, uint32_t *, uint32_t, uint32_t) = nullptr;
    REFT_PICK_K(k_gather_burst, fn, nrows)
    size_t lds = 0;
    uint32_t grid = 0;
    const uint64_t nstages = (hi - lo + bc.stage_bytes - 1) / bc.stage_bytes;
    hipError_t e = burst_grid((const void *)fn, nstages, cfg, bc, &lds, &grid);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_zero_words, dim3(1), dim3(256), 0, stream, bc.ctr, 9 * kCtrStride);
    hipLaunchKernelGGL(fn, dim3(grid), dim3(kBurstThreads), lds, stream, pt, tab, dtab, vb, lo, hi,
                       bc.stage_bytes, bc.ctr, bc.max_polls, bc.nap);
    return hipGetLastError();
}

hipError_t launch_xor_contig_burst(const SrcBases &src, int nsrc, uint64_t dst, uint64_t L,
                                   const LaunchCfg &cfg, const BurstCfg &bc, hipStream_t stream)
{
    if (L == 0) return hipSuccess;
    if (!burst_cfg_ok(bc)) return hipErrorInvalidValue;
    void (*fn)(SrcBases, uint64_t, uint64_t, uint32_t, uint32_t *, uint32_t, uint32_t) = nullptr;
    REFT_PICK_K(k_xor_contig_burst, fn, nsrc)
    size_t lds = 0;
    uint32_t grid = 0;
    const uint64_t nstages = (L + bc.stage_bytes - 1) / bc.stage_bytes;
    hipError_t e = burst_grid((const void *)fn, nstages, cfg, bc, &lds, &grid);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_zero_words, dim3(1), dim3(256), 0, stream, bc.ctr, 9 * kCtrStride);
    hipLaunchKernelGGL(fn, dim3(grid), dim3(kBurstThreads), lds, stream, src, dst, L,
                       bc.stage_bytes, bc.ctr, bc.max_polls, bc.nap);
    return hipGetLastError();
}

hipError_t launch_xor_contig(const SrcBases &src, int nsrc, uint64_t dst, uint64_t L,
                             uint32_t tile_shift, const LaunchCfg &cfg, hipStream_t stream)
{
    if (L == 0) return hipSuccess;
    void (*fn)(SrcBases, uint64_t, uint64_t, uint32_t) = nullptr;
    REFT_PICK_K(k_xor_contig, fn, nsrc)
    const uint64_t ntiles = (L + (1ull << tile_shift) - 1) >> tile_shift;
    hipLaunchKernelGGL(fn, dim3(grid_for(ntiles, cfg)), dim3(kThreads), 0, stream, src, dst, L,
                       tile_shift);
    return hipGetLastError();
}

}  // namespace reft

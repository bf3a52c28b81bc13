// Device helpers shared by the kernel files.
#pragma once
#include "reft_internal.hpp"

namespace reft {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// Addresses travel through the kernels as integers (a destination may be a "virtual base" that
// only becomes a valid address once a stream offset is added).  They are turned into pointers in
// the global address space here, so that the accesses compile to global_load / global_store.
#define REFT_GLOBAL __attribute__((address_space(1)))

// Loads of 16 bytes take any byte address: global memory is in unaligned access mode, one
// global_load_dwordx4 serves a lane whatever its address.  Measured as a copy whose source is 0, 4,
// 2 or 1 bytes off a 16-byte boundary: 2 GiB at 4.94, 4.91, 5.48, 5.49 TB/s, 14 MiB in 4.3, 4.3,
// 5.2, 5.2 us.  (Two aligned loads per 16 bytes and a funnel shift in registers, with one chunk in
// flight per source, was up to 2.7 times slower: the decode of one of 4 x 14.7 MB at odd offsets took
// 150 us, with these loads 56 us; the parity of 8 x 132 MB of small odd tensors 417 and 313 us.)
typedef u32x4 u32x4_any __attribute__((aligned(1)));
typedef const REFT_GLOBAL u32x4_any *gcptr16;
typedef REFT_GLOBAL u32x4 *gptr16;

__device__ __forceinline__ gcptr16 as_gc16(uint64_t a) { return (gcptr16)a; }
__device__ __forceinline__ gptr16 as_g16(uint64_t a) { return (gptr16)a; }
__device__ __forceinline__ uint8_t ld8(uint64_t a) { return *(const REFT_GLOBAL uint8_t *)a; }
__device__ __forceinline__ void st8(uint64_t a, uint8_t v) { *(REFT_GLOBAL uint8_t *)a = v; }

template <bool NT>
__device__ __forceinline__ u32x4 ld16(gcptr16 p)
{
    if constexpr (NT) return __builtin_nontemporal_load(p);
    else return *p;
}

template <bool NT>
__device__ __forceinline__ void st16(gptr16 p, u32x4 v)
{
    if constexpr (NT) __builtin_nontemporal_store(v, p);
    else *p = v;
}

// The instantiation of a kernel template for (number of sources, unroll, non-temporal).
#define REFT_PICK_UNT(KERNEL, K)                                                                  \
    (cfg.nontemporal                                                                              \
         ? (cfg.unroll == 1 ? KERNEL<K, 1, true> : cfg.unroll == 2 ? KERNEL<K, 2, true>           \
                                                                   : KERNEL<K, 4, true>)          \
         : (cfg.unroll == 1 ? KERNEL<K, 1, false> : cfg.unroll == 2 ? KERNEL<K, 2, false>         \
                                                                    : KERNEL<K, 4, false>))

#define REFT_PICK_K(KERNEL, fn, nsrc)                                                             \
    switch (nsrc) {                                                                               \
    case 1: fn = REFT_PICK_UNT(KERNEL, 1); break;                                                 \
    case 2: fn = REFT_PICK_UNT(KERNEL, 2); break;                                                 \
    case 3: fn = REFT_PICK_UNT(KERNEL, 3); break;                                                 \
    case 4: fn = REFT_PICK_UNT(KERNEL, 4); break;                                                 \
    case 5: fn = REFT_PICK_UNT(KERNEL, 5); break;                                                 \
    case 6: fn = REFT_PICK_UNT(KERNEL, 6); break;                                                 \
    case 7: fn = REFT_PICK_UNT(KERNEL, 7); break;                                                 \
    case 8: fn = REFT_PICK_UNT(KERNEL, 8); break;                                                 \
    default: return hipErrorInvalidValue;                                                         \
    }

}  // namespace reft

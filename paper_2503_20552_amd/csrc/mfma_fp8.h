// Pieces shared by the two matrix-core kernels for an fp8 cache: V operands read transposed out of LDS.
#pragma once

#include "mfma_page.h"

namespace adr {

constexpr int kFp8TileBytes = kPageSize * D; // one tile of K or of V for one row of D elements per token

__device__ __forceinline__ uint32_t lds_address(const void *p)
{
    return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void *)p;
}

// The transposed reads are written by hand, all eight of a step in one statement, and nothing waits for
// them there: the compiler would guard each one (it cannot tell the read's target from the ring
// slots that direct-to-LDS loads are still filling) with a wait for EVERY load in flight, which
// is exactly what the ring must not do.  The stage read here has landed (wait_groups); the results
// are valid after the caller's wait for the LDS (settle_copies below), which takes them as operands
// so that nothing reads them earlier.
__device__ __forceinline__ void lds_read_tr8_x8(const uint32_t (&addr)[8], u32x2 (&v)[8])
{
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("ds_read_b64_tr_b8 %0, %8 offset:%16\n\t"
                 "ds_read_b64_tr_b8 %1, %9 offset:%16\n\t"
                 "ds_read_b64_tr_b8 %2, %10 offset:%16\n\t"
                 "ds_read_b64_tr_b8 %3, %11 offset:%16\n\t"
                 "ds_read_b64_tr_b8 %4, %12 offset:%16\n\t"
                 "ds_read_b64_tr_b8 %5, %13 offset:%16\n\t"
                 "ds_read_b64_tr_b8 %6, %14 offset:%16\n\t"
                 "ds_read_b64_tr_b8 %7, %15 offset:%16"
                 : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3]), "=&v"(v[4]), "=&v"(v[5]), "=&v"(v[6]), "=&v"(v[7])
                 : "v"(addr[0]), "v"(addr[1]), "v"(addr[2]), "v"(addr[3]), "v"(addr[4]), "v"(addr[5]), "v"(addr[6]),
                   "v"(addr[7]), "n"(kFp8TileBytes)
                 : "memory");
#else
    for (int e = 0; e < 8; ++e)
        v[e] = u32x2{addr[e], 0u};
#endif
}

// The same, waited for: all LDS reads of this wave have arrived when it ends.
__device__ __forceinline__ void lds_read_tr8_x8_wait(const uint32_t (&addr)[8], u32x2 (&v)[8])
{
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("ds_read_b64_tr_b8 %0, %8\n\t"
                 "ds_read_b64_tr_b8 %1, %9\n\t"
                 "ds_read_b64_tr_b8 %2, %10\n\t"
                 "ds_read_b64_tr_b8 %3, %11\n\t"
                 "ds_read_b64_tr_b8 %4, %12\n\t"
                 "ds_read_b64_tr_b8 %5, %13\n\t"
                 "ds_read_b64_tr_b8 %6, %14\n\t"
                 "ds_read_b64_tr_b8 %7, %15\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3]), "=&v"(v[4]), "=&v"(v[5]), "=&v"(v[6]), "=&v"(v[7])
                 : "v"(addr[0]), "v"(addr[1]), "v"(addr[2]), "v"(addr[3]), "v"(addr[4]), "v"(addr[5]), "v"(addr[6]),
                   "v"(addr[7])
                 : "memory");
#else
    for (int e = 0; e < 8; ++e)
        v[e] = u32x2{addr[e], 0u};
#endif
}

// Ties K operands to a place in the program: what was read from LDS has arrived here, and no read is
// moved behind the loads that refill the stage.
__device__ __forceinline__ void settle_k(u32x2 (&a)[4], u32x2 (&b)[4])
{
    asm volatile("" : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]), "+v"(b[0]), "+v"(b[1]), "+v"(b[2]), "+v"(b[3])::"memory");
}

// A word of four bytes that clears, in a V operand, the tokens of this lane at or past t1 (tok =
// index of the lane's first token).
__device__ __forceinline__ uint32_t tail_mask_fp8(int tok, int t1)
{
    return (tok + 0 < t1 ? 0x000000ffu : 0u) | (tok + 1 < t1 ? 0x0000ff00u : 0u) | (tok + 2 < t1 ? 0x00ff0000u : 0u) |
           (tok + 3 < t1 ? 0xff000000u : 0u);
}

} // namespace adr

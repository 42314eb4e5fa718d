// LDS-DMA requests written out: one 16-byte-per-lane request copies lane l's
// bytes to lds_addr + 16 l (lds_addr the same in every lane).
//
// As inline assembly the compiler does not see an LDS write in flight: it
// would put a full vmcnt(0) in front of every later LDS read, which makes
// all requests in flight finish first.  The kernels' own vmcnt waits and
// barriers order the data.  The LDS address goes in through an "{m0}"
// operand, so the compiler itself writes m0 (and knows it does); the s_nop
// separates that write from the load that reads it.
#pragma once

#include "common.h"

namespace moe {
namespace {

typedef __attribute__((address_space(3))) void lds_void_t;
typedef __attribute__((address_space(1))) void gbl_void_t;

__device__ __forceinline__ void dma16_to_lds(const void *gptr, uint32_t lds_addr) {
    asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %0, off"
                 :
                 : "v"(gptr), "{m0}"(__builtin_amdgcn_readfirstlane(lds_addr))
                 : "memory");
}

// From base + voff + soff of a raw buffer resource (buf_rsrc of a pointer
// that is the same in every lane).
__device__ __forceinline__ void buf16_to_lds(const u32x4 &rsrc, uint32_t voff, uint32_t soff,
                                             uint32_t lds_addr) {
    asm volatile("s_nop 0\n\tbuffer_load_dwordx4 %0, %1, %2 offen lds"
                 :
                 : "v"(voff), "s"(rsrc), "s"(soff), "{m0}"(lds_addr)
                 : "memory");
}
__device__ __forceinline__ u32x4 buf_rsrc(const void *p) {
    const uint64_t b = (uint64_t)(uintptr_t)p;
    return u32x4{(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)b),
                 (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(b >> 32)), 0xFFFFFFFFu,
                 0x00020000u};
}

}  // namespace
}  // namespace moe

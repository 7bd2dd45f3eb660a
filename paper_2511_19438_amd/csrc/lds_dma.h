// Global -> LDS copies by DMA, as inline assembly (gfx950).
//
// The compiler does not know that LDS changes, and so puts no wait of its own before the LDS reads that follow (for the
// builtin it waits for ALL outstanding loads before the first read behind it, which empties the pipeline of loads once per
// turn of a loop); the memory clobbers here and at a kernel's own waits keep its LDS reads where they stand.  Nor does it
// know of m0, a reserved register that a clobber list may not name: nothing else in a kernel may use it (no LDS-DMA builtin
// beside these), which a check of the compiled code sees to.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace gptq {

// A pointer that is the same in every lane, in scalar registers (64-bit products are left in vector registers otherwise).
__device__ __forceinline__ const char *uniform(const char *p)
{
    const uint64_t bits = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)bits), hi = __builtin_amdgcn_readfirstlane((uint32_t)(bits >> 32));
    return reinterpret_cast<const char *>((uint64_t)hi << 32 | lo);
}

// Lane l's 16 bytes at base + byte_off land at lds + 16 l; base and lds are uniform over the wavefront.
template <bool STREAM = false>
__device__ __forceinline__ void dma_16(uint32_t lds, uint32_t byte_off, const char *base)
{
    if (STREAM)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt" ::"s"(lds), "v"(byte_off), "s"(base)
                     : "memory");
    else
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(byte_off), "s"(base)
                     : "memory");
}
// The same from an address per lane.
__device__ __forceinline__ void dma_16(uint32_t lds, const char *src)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds), "v"(src) : "memory");
}
// Lane l's 4 bytes land at lds + 4 l.
__device__ __forceinline__ void dma_4(uint32_t lds, const char *src)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off" ::"s"(lds), "v"(src) : "memory");
}

// All but the last N of this wavefront's loads have arrived.
template <int N>
__device__ __forceinline__ void wait_loads()
{
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

}  // namespace gptq

// Loads from memory straight to LDS (gfx950), shared by the forms that stage operands so.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace bc {

typedef int i32x4 __attribute__((ext_vector_type(4)));

// Raw buffer resource: no swizzle, 32-bit dword data format; loads at offsets beyond
// num_records return zeros instead of faulting, stores there are dropped.
constexpr int kBufferFlags = 0x00020000;
constexpr int kOutOfRange = 0x7FFFFF00;     // byte offset past every buffer (< 2^31 - 256 bytes)

// Raw buffer descriptor as the four dwords that the inline instruction takes.
__device__ __forceinline__ i32x4 raw_desc(const void *p, int bytes)
{
    const uint64_t u = (uint64_t)p;
    return i32x4{(int)(uint32_t)u, (int)(uint32_t)(u >> 32), bytes, kBufferFlags};
}

// 64 lanes x 16 bytes from memory to LDS bytes [lds, lds + 1024) (lane i at 16 i). No
// register receives data; offsets at or beyond the buffer's extent write zeros. M0, which
// takes the LDS address, cannot be named as clobbered (the compiler reserves it, keeps
// nothing there, and writes it right before each use of its own).
__device__ __forceinline__ void dma16(const i32x4 &r, uint32_t lds, int voff)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                 :: "s"(lds), "v"(voff), "s"(r) : "memory");
}

__device__ __forceinline__ uint32_t lds_addr(const void *p)
{
    return (uint32_t)(uint64_t)(__attribute__((address_space(3))) const uint8_t *)p;
}

}  // namespace bc

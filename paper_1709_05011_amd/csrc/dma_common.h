// Loads that write LDS, for the kernels of conv_dma.h, conv_dma.hip and wgrad_dma.hip (bf16 products of gfx950 whose operands go from memory straight into LDS:
// buffer loads with the lds modifier, no staging registers, no LDS store instructions, several k-steps in flight per compute unit).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "conv_common.h"

namespace {

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));

// 64 lanes x 16 bytes from base + voff + soff to LDS bytes lds .. lds + 1023 in lane order; lanes past the declared size of the buffer fetch zeros.
// (Inline assembly: behind the builtin the compiler waits for all of a wave's loads before each LDS read that might meet them.  No register is
// written, so nothing can be reused too early; whoever reads the bytes waits with wait_loads_and_barrier() first.)
// The compiler does not keep hazards apart that end inside the block: one wait state between m0 and the load, and five between a vector instruction that writes
// soff or rsrc (v_readfirstlane) and the load.  FROM_VECTOR: soff comes from one, the block waits itself; tests/test_device_code.py looks at all others.
template <bool FROM_VECTOR = false>
__device__ __forceinline__ void load_to_lds(const u32x4& rsrc, unsigned voff, int soff, unsigned lds) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop %4\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                 : : "s"(lds), "v"(voff), "s"(rsrc), "s"(soff), "n"(FROM_VECTOR ? 3 : 0) : "memory");
}
__device__ __forceinline__ void load_to_lds_nt(const u32x4& rsrc, unsigned voff, int soff, unsigned lds) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen nt lds" : : "s"(lds), "v"(voff), "s"(rsrc), "s"(soff) : "memory");
}
__device__ __forceinline__ u32x4 buffer_words(const void* base, unsigned bytes) {
    const uintptr_t a = reinterpret_cast<uintptr_t>(base);
    return u32x4{(unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)a), (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(a >> 32)),
                 (unsigned)__builtin_amdgcn_readfirstlane((int)bytes), kBufferWords3};
}
// At most N of this wave's loads are still under way (they arrive in order), its LDS reads are complete; then the workgroup barrier.
template <int N>
__device__ __forceinline__ void wait_loads_and_barrier() {
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" : : "n"(N) : "memory");
}
__device__ __forceinline__ unsigned lds_address(const void* ptr) {
    return (unsigned)(uintptr_t)(const __attribute__((address_space(3))) unsigned char*)(uintptr_t)ptr;
}

}  // namespace

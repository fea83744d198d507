// Requests that bring data from memory straight into LDS (no registers on the way), counted by the kernel itself.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sv {

// Two 1 KB pieces from memory straight into LDS (64 lanes x 16 bytes each, the second piece's place kStep bytes behind
// the first's): lane l's 16 bytes come from byte voff + soff of the buffer and land at lds + 16 l.  A voff of kOutside is
// past the buffer's end, and such a lane's bytes are zeros.  Nothing waits here: the caller counts these requests itself
// (s_waitcnt vmcnt); the compiler's own bookkeeping would wait for all of them in front of every LDS read.
// (s_nop 4: a scalar register that a vector instruction has just written may not be read by a memory instruction sooner,
// and the compiler does not look into the block; s_nop 0: one wait state between a write of m0 and its use.)
typedef int i32x4_t __attribute__((ext_vector_type(4)));
constexpr uint32_t kBufferBytes = 0xFFFFFFF0u, kOutside = 0xFFFFFFFFu;
template <int STEP>
__device__ __forceinline__ void memory_to_lds(uint32_t voff0, uint32_t voff1, i32x4_t buffer, uint32_t soff, uint32_t lds) {
    asm volatile(
        "s_nop 4\n\ts_mov_b32 m0, %4\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %2, %3 offen lds\n\t"
        "s_add_u32 m0, m0, %5\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
        :
        : "v"(voff0), "v"(voff1), "s"(buffer), "s"(soff), "s"(lds), "n"(STEP)
        : "memory", "m0", "scc");
}
// one such piece
__device__ __forceinline__ void memory_to_lds(uint32_t voff, i32x4_t buffer, uint32_t soff, uint32_t lds) {
    asm volatile("s_nop 4\n\ts_mov_b32 m0, %3\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %1, %2 offen lds"
                 :
                 : "v"(voff), "s"(buffer), "s"(soff), "s"(lds)
                 : "memory", "m0");
}
__device__ __forceinline__ i32x4_t buffer_of(const char* base) {
    const uint64_t p = reinterpret_cast<uint64_t>(base);
    // (raw buffer: stride 0, byte-addressed, 32-bit data format)
    return i32x4_t{__builtin_amdgcn_readfirstlane((int)(uint32_t)p), __builtin_amdgcn_readfirstlane((int)((uint32_t)(p >> 32) & 0xFFFFu)),
                   (int)kBufferBytes, 0x00020000};
}

}  // namespace sv

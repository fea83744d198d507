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

// The same for rows that a 32-bit offset does not reach (lists into a matrix of more than 4 GB, rows of 16 MB and more apart):
// an address per lane.
__device__ __forceinline__ void memory_to_lds_far(const char* p, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" : : "v"(p), "s"(lds) : "memory", "m0");
}
// what a lane past the end of a row reads there
__device__ __attribute__((aligned(16))) const uint32_t kZeroUnit[4] = {0u, 0u, 0u, 0u};

// Where one lane's 16 bytes of every request come from: NEAR an offset into the request's buffer, FAR an address.
template <bool FAR>
struct LaneSource;
template <>
struct LaneSource<false> {
    uint32_t at;
    __device__ __forceinline__ void set(const char* base, int64_t row, int64_t row_bytes, uint32_t byte) {
        (void)base;
        at = (uint32_t)row * (uint32_t)row_bytes + byte;
    }
};
template <>
struct LaneSource<true> {
    const char* at;
    __device__ __forceinline__ void set(const char* base, int64_t row, int64_t row_bytes, uint32_t byte) {
        at = base + row * row_bytes + byte;
    }
};
// one piece, `soff` bytes on from the lanes' sources (for a lane with `none`: zeros)
__device__ __forceinline__ void bring(const LaneSource<false>& l, bool none, const i32x4_t buffer, int64_t soff, uint32_t lds) {
    memory_to_lds(none ? kOutside : l.at, buffer, (uint32_t)soff, lds);
}
__device__ __forceinline__ void bring(const LaneSource<true>& l, bool none, const i32x4_t, int64_t soff, uint32_t lds) {
    memory_to_lds_far(none ? reinterpret_cast<const char*>(kZeroUnit) : l.at + soff, lds);
}
// two of them, the second's place STEP bytes behind the first's
template <int STEP>
__device__ __forceinline__ void bring(const LaneSource<false>& l0, const LaneSource<false>& l1, bool none0, bool none1,
                                      const i32x4_t buffer, int64_t soff, uint32_t lds) {
    memory_to_lds<STEP>(none0 ? kOutside : l0.at, none1 ? kOutside : l1.at, buffer, (uint32_t)soff, lds);
}
template <int STEP>
__device__ __forceinline__ void bring(const LaneSource<true>& l0, const LaneSource<true>& l1, bool none0, bool none1,
                                      const i32x4_t buffer, int64_t soff, uint32_t lds) {
    bring(l0, none0, buffer, soff, lds);
    bring(l1, none1, buffer, soff, lds + STEP);
}

}  // namespace sv

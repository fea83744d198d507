// Tiled matrix product on the matrix cores for MANY hidden-state rows (more than 32):
//     out[r, j] = < M[row(j), :], x[r, :] >      r < rows, j < n_items
// with row(j) = j (the full-vocabulary projection of Section 3.1, or the selector's score matrix of
// Section 3.3 Step 1 for a whole batch) or row(j) = idx[j] (Section 3.3 Step 3 over one set of rows
// shared by every hidden row).  bf16 storage only.
//
// With hundreds of hidden rows the product is a real contraction (Section 3.4 counts V d
// multiply-adds per hidden row): reading M once per 64 hidden rows, as the skinny kernel does, turns
// into many passes over M.  Here a workgroup owns a TM x TN tile of the output (TM hidden rows, TN
// rows of M) and walks the reduction in slices of 64 elements through LDS; every wavefront multiplies
// its part of the tile with v_mfma_f32_32x32x16_bf16 from there.  Workgroups that share rows of M (the different
// hidden-row tiles of one TN block) are given consecutive slots on the same XCD, so that M comes from HBM once and from
// that die's L2 afterwards (measured: HBM traffic 1.3 x the size of M at 512 hidden rows).
//
// Three forms of the main loop.  The plain one (slices through registers into LDS rows padded to 144 bytes) leaves the
// order of loads, LDS traffic and MFMAs to the compiler and relies on several workgroups per CU to overlap them: 17 to 32
// hidden rows where the ring does not win.  The ring (17 to 64 rows, bound by the one pass over M) has three slices on
// their way from memory to LDS.  In the alternating one (more rows) the two wavefronts of a SIMD take turns between
// multiplying and memory work, a barrier per turn, and slices go from memory to LDS directly.  The latter two name a lane's
// source by a 32-bit offset into a buffer; where that does not reach (rows of 16 MB and more apart -- hidden states that are
// the last positions of long sequences --, lists into matrices of more than 4 GB) by an address (FAR), which costs a 64-bit
// addition per request.
#include "sv_device.h"
#include "sv_launch.h"

#include <math.h>

#include <type_traits>

#include "memory_to_lds.h"
#include "tile_epilogue.h"

namespace sv {

namespace {

constexpr int kTK = 64;                  // reduction elements per slice (128 bytes of a row)
constexpr int kRowB = kTK * 2 + 16;      // padded LDS row (144 B = 36 words)
constexpr int kXcds = 8;
constexpr unsigned kRound = 256;         // workgroups that the part runs at a time where a CU holds one

// dst with lanes LO and HI replaced by the two halves of the wavefront-uniform mask m (two v_writelane_b32).
// The mask comes straight from a vector comparison: on this architecture a vector instruction that reads a
// scalar register written by the vector instruction just before it needs two wait states in between; the
// compiler inserts them for its own instructions, not for the operands of an asm block, hence the s_nop.
template <int LO, int HI>
__device__ __forceinline__ uint32_t write_lanes(uint32_t dst, uint64_t m) {
    static_assert(LO >= 0 && LO < 64 && HI >= 0 && HI < 64, "lanes of a 64-wide wavefront");
    asm("s_nop 1\n\tv_writelane_b32 %0, %1, %3\n\tv_writelane_b32 %0, %2, %4"
        : "+v"(dst)
        : "s"((uint32_t)m), "s"((uint32_t)(m >> 32)), "n"(LO), "n"(HI));
    return dst;
}

// 2 x + (this lane's bit of the wavefront-wide mask m): one add-with-carry whose carry-in is the mask.  The mask
// must come from a scalar instruction (see write_lanes for why not straight from a vector comparison).
__device__ __forceinline__ uint32_t shift_in_lane_bit(uint32_t x, uint64_t m) {
    uint64_t carry_out;
    asm volatile("v_addc_co_u32_e64 %0, %1, %0, %0, %2" : "+v"(x), "=s"(carry_out) : "s"(m));
    return x;
}

// LDS the bracket epilogue needs (it reuses the operand buffers after the main loop): per tile row the
// bracket and a candidate counter (16 bytes reserved), per wavefront the scores of one 32-row band
template <int GM, int GN, int WM, int WN>
constexpr size_t bracket_lds_bytes() {
    return (size_t)32 * GM * WM * 16 + (size_t)GM * GN * (16 * WN * 64) * 4;
}

enum { LOOP_PLAIN = 0, LOOP_TURNS = 1, LOOP_RING = 2 };
template <int GM, int GN, int WM, int WN, int PIPE>
constexpr size_t tile_lds_bytes() {
    return PIPE == LOOP_RING ? (size_t)4 * (32 * GM * WM + 32 * GN * WN) * kTK * 2
           : PIPE == LOOP_TURNS ? (size_t)(2 * 32 * GM * WM + 3 * 32 * GN * WN) * kTK * 2
                                : (size_t)2 * (32 * GM * WM + 32 * GN * WN) * kRowB;
}

// GM x GN wavefronts; each owns WM x WN MFMA tiles of 32 x 32: TM = 32 GM WM hidden rows, TN = 32 GN WN items.
// PIPE: the main loop (the last two are fed from memory to LDS, FAR: from addresses).  EPI: what happens to the product --
//   EPI_STORE    it is stored;
//   EPI_BRACKET  the epilogue of the bracketed selection (Section 3.3 Step 2 for a batch of hidden rows)
//                classifies it, nothing is stored;
//   EPI_PICK     Section 3.3 Step 3 for a batch of hidden rows with one index list each: only the entries
//                a row asks for are stored, straight to their place in logits_out.
enum { EPI_STORE = 0, EPI_BRACKET = 1, EPI_PICK = 2 };
template <int GM, int GN, int WM, int WN, int PIPE, int EPI, bool FAR>
__global__ __launch_bounds__(64 * GM * GN) void tile_mfma_kernel(const GemvArgs a, const BracketEpi ep, const PickEpi pk) {
    constexpr int kThreads = 64 * GM * GN;
    constexpr int kRowsPerPass = kThreads / 8;           // loader: 8 threads per 128-byte row slice
    constexpr int TM = 32 * GM * WM, TN = 32 * GN * WN;
    constexpr int QA = TM / kRowsPerPass, QB = TN / kRowsPerPass;   // 16-byte loads per thread and slice
    static_assert(TM % kRowsPerPass == 0 && TN % kRowsPerPass == 0, "tile rows must fill whole loader passes");
    constexpr int kStage = (TM + TN) * kRowB;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];   // [2][TM + TN][kRowB]
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int wr = wave / GN, wc = wave % GN;
    const int C = a.chunks;
    const int nk = (C + 7) / 8;
    const int64_t n_items = a.n_items_dev ? (int64_t)*a.n_items_dev : a.n_items;
    const int RT = (a.rows + TM - 1) / TM;
    // Width of an item tile: TN, or (a.balance_cus workgroups at a time, product stored) the smallest multiple of
    // 32 with which the list still takes as many rounds of workgroups as with TN -- 50223 items on 256 CUs: 225
    // tiles of 224 items instead of 197 of 256.  The wavefronts past that width have nothing to do.
    int64_t tn = TN;
    if (EPI == EPI_STORE && a.balance_cus > 0 && n_items > 0) {
        const int64_t per_round = (int64_t)TN * a.balance_cus;
        const int64_t rounds = (n_items + per_round - 1) / per_round;
        const int64_t lanes32 = (int64_t)32 * a.balance_cus * rounds;
        tn = 32 * ((n_items + lanes32 - 1) / lanes32);
    }
    const int64_t IT = (n_items + tn - 1) / tn;
    // block id -> (XCD, slot on that XCD); consecutive slots of one XCD: the RT hidden-row tiles of one item tile
    const int64_t slot = blockIdx.x / kXcds;
    const int rt = (int)(slot % RT);
    const int64_t it = (slot / RT) * kXcds + (blockIdx.x % kXcds);
    if (it >= IT || !gate_open(a, n_items)) return;
    const int64_t tile0 = it * tn;
    const int64_t tile_end = tile0 + tn < n_items ? tile0 + tn : n_items;

    // loader role of the plain loop: 8 threads cover the 128-byte slice of one row, 32 rows per pass
    const int piece = tid & 7, r0 = tid >> 3;
    const u32x4* pa[QA];
    const u32x4* pb[QB];
#pragma unroll
    for (int q = 0; q < QA; ++q) {
        int row = rt * TM + r0 + kRowsPerPass * q;
        if (row > a.rows - 1) row = a.rows - 1;                       // padding rows: computed, never stored
        pa[q] = reinterpret_cast<const u32x4*>(a.x + (int64_t)row * a.x_row_bytes);
    }
#pragma unroll
    for (int q = 0; q < QB; ++q) {
        int64_t item = tile0 + r0 + kRowsPerPass * q;
        if (item > tile_end - 1) item = tile_end - 1;
        const int64_t mrow = a.idx ? (int64_t)a.idx[item] : item;
        pb[q] = reinterpret_cast<const u32x4*>(a.M + mrow * a.m_row_bytes);
    }
    // Loads and stores of the pipeline are unconditional (slice and unit indices are clamped; the
    // units of a ragged last slice that lie past the row are zeroed on their way into LDS, when the
    // data has arrived anyway): without branches between them the compiler can count the loads in
    // flight and wait for exactly the oldest slice.
    // Workgroups walk the reduction in rotated order (slice ks of the walk is slice eff(ks) of the rows): rows a
    // power of two apart put the same offset of every row on the same memory channels, and workgroups that all
    // start at offset 0 keep hitting the same channels together.  With one tile of hidden rows (up to 128)
    // consecutive workgroups of one XCD start 37 slices apart (modulo the number of slices): the starts of even a
    // few dozen workgroups -- a launch of one workgroup per CU has 32 slots per XCD -- then spread over the whole
    // row.  With starts one slice apart such a
    // launch kept all its workgroups within the same 4 KB of their rows at any time: 60 rows x 50200 gathered
    // rows of 8 KB 97 us against 88, x 65536 117 against 105, all 128256 rows 201 against 192-194 (rows padded
    // to 8320 bytes had shown the same gain, which is how the channels were found out).
    // (Short reductions have nothing to spread.  a.plain_order: the place of an item in the list may vary from
    // run to run, and the order of a token's float32 additions must not.)
    // (Several tiles of hidden rows keep starts one slice apart: measured equal or better there, 512 rows 663
    // against 693 us -- the hidden-row tiles of one item tile share the rows of M through their XCD's L2, and
    // neighbouring item tiles that walk almost in step seem to help that.  One tile of 65 to 128 rows gains like
    // the smaller ones: 100 rows x 50200 items 120 -> 112 us, 128 rows x 65536 135 -> 128.)
    const int64_t rot_step = RT == 1 ? (nk % 37 ? 37 : 41) : 1;
    const int rot = nk >= 16 && !a.plain_order ? (int)((slot * rot_step) % nk) : 0;
    auto eff = [&](int ks) { const int e = min(ks, nk - 1) + rot; return e >= nk ? e - nk : e; };
    auto load = [&](int ks, u32x4 (&ga)[QA], u32x4 (&gb)[QB]) {
        const int u = min(eff(ks) * 8 + piece, C - 1);
#pragma unroll
        for (int q = 0; q < QB; ++q) gb[q] = pb[q][u];
#pragma unroll
        for (int q = 0; q < QA; ++q) ga[q] = pa[q][u];
    };
    auto store = [&](int ks, const u32x4 (&ga)[QA], const u32x4 (&gb)[QB]) {      // slice ks -> buffer ks % 2
        unsigned char* base = smem + (size_t)(ks & 1) * kStage + (size_t)r0 * kRowB + piece * 16;
        const bool past = ks >= nk || eff(ks) * 8 + piece >= C;
#pragma unroll
        for (int q = 0; q < QA; ++q)
            *reinterpret_cast<u32x4*>(base + (size_t)(kRowsPerPass * q) * kRowB) = past ? zero16() : ga[q];
#pragma unroll
        for (int q = 0; q < QB; ++q)
            *reinterpret_cast<u32x4*>(base + (size_t)(TM + kRowsPerPass * q) * kRowB) = past ? zero16() : gb[q];
    };

    f32x16_t acc[WM][WN];
#pragma unroll
    for (int m = 0; m < WM; ++m)
#pragma unroll
        for (int n = 0; n < WN; ++n)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[m][n][e] = 0.f;

    // operand role: lane = (row within the 32 x 32 tile = lane % 32, k-group = lane / 32)
    const size_t a_off = (size_t)(wr * 32 * WM + (lane & 31)) * kRowB + (lane >> 5) * 16;
    const size_t b_off = (size_t)(TM + wc * 32 * WN + (lane & 31)) * kRowB + (lane >> 5) * 16;
    auto multiply = [&](int buf) {
        const unsigned char* sa = smem + (size_t)buf * kStage + a_off;
        const unsigned char* sb = smem + (size_t)buf * kStage + b_off;
#pragma unroll
        for (int kk = 0; kk < kTK / 16; ++kk) {
            bf16x8_t af[WM], bf[WN];
#pragma unroll
            for (int m = 0; m < WM; ++m)
                af[m] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const u32x4*>(sa + (size_t)(32 * m) * kRowB + kk * 32));
#pragma unroll
            for (int n = 0; n < WN; ++n)
                bf[n] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const u32x4*>(sb + (size_t)(32 * n) * kRowB + kk * 32));
#pragma unroll
            for (int m = 0; m < WM; ++m)
#pragma unroll
                for (int n = 0; n < WN; ++n)
                    acc[m][n] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[m], bf[n], acc[m][n], 0, 0, 0);
        }
    };
    if constexpr (PIPE == LOOP_RING) {
        // Up to 64 hidden rows: one pass over M at the rate of the memory system.  A ring of four stages in LDS, three slices
        // on their way (96 KB of M per CU with 64 x 256 tiles), one barrier per slice: behind it everybody has slice ks and
        // nobody reads slice ks - 1 any more, whose stage takes slice ks + 3.  Layout and requests as in the loop below.
        constexpr int kWavesHere = GM * GN, kStageB = (TM + TN) * 128;
        constexpr int LA = TM / (8 * kWavesHere), LB = TN / (8 * kWavesHere);
        static_assert(TM % (8 * kWavesHere) == 0 && LB % 2 == 0 && kWavesHere % 2 == 0, "whole requests per wavefront; a constant swizzle");
        constexpr int kPass = 8 * kWavesHere;                // rows that one request of every wavefront covers
        const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;
        const int swave = __builtin_amdgcn_readfirstlane(wave);
        const int l8 = lane >> 3;
        const int unit = (lane & 7) ^ ((4 * (swave & 1) + (l8 >> 1)) & 7);
        const bool lane_past = (nk - 1) * 8 + unit >= C;     // of the last slice
        const char* const base_a = a.x + (int64_t)rt * TM * a.x_row_bytes;
        const char* const base_b = a.idx ? a.M : a.M + tile0 * a.m_row_bytes;
        LaneSource<FAR> src_a[LA], src_b[LB];
#pragma unroll
        for (int i = 0; i < LA; ++i)
            src_a[i].set(base_a, min(rt * TM + kPass * i + 8 * swave + l8, a.rows - 1) - rt * TM, a.x_row_bytes, (uint32_t)unit * 16u);
#pragma unroll
        for (int i = 0; i < LB; ++i) {
            int64_t item = tile0 + kPass * i + 8 * swave + l8;
            if (item > tile_end - 1) item = tile_end - 1;
            src_b[i].set(base_b, a.idx ? (int64_t)a.idx[item] : item - tile0, a.m_row_bytes, (uint32_t)unit * 16u);
        }
        const i32x4_t buf_a = buffer_of(base_a), buf_b = buffer_of(base_b);
        const int swz = ((lane >> 5) ^ ((lane >> 1) & 7)) * 16;
        const int fa0 = (TN + wr * 32 * WM + (lane & 31)) * 128 + swz, fb0 = (wc * 32 * WN + (lane & 31)) * 128 + swz;
        // What lies past the tile's width is neither requested nor multiplied (a wavefront requests the first MINE of its LB
        // pieces of M; `none`: its own items are all past the width), so a round takes what its width needs and lists of any
        // length can have this shape: unions of 12497 / 22481 / 32210 / 50313 rows, 33 to 64 hidden rows, a whole step
        // 37.3 / 53.5 / 65.8 / 105.3 -> 32.8 / 50.8 / 64.4 / 102.3 us, 3 to 5 of them a launch of the smaller tiles that short
        // unions were given before and that all others had to skip.
        constexpr bool kNarrow = GM == 1 && GN == 8 && WN == 1;      // (the shape whose width follows the list)
        const bool none = kNarrow && wc * 32 >= (int)tn;
        auto walk = [&](auto mine) {
            constexpr int MINE = decltype(mine)::value;
            auto request = [&](int ks) {
                const int s = eff(ks);
                const bool cut = s == nk - 1 && lane_past;
                const uint32_t at = lds0 + (uint32_t)((ks & 3) * kStageB + swave * 1024);
#pragma unroll
                for (int i = 0; i + 1 < MINE; i += 2)
                    bring<kPass * 128>(src_b[i], src_b[i + 1], cut, cut, buf_b, (int64_t)s * 128, at + (uint32_t)(i * kPass * 128));
                if constexpr (MINE % 2 == 1)
                    bring(src_b[MINE - 1], cut, buf_b, (int64_t)s * 128, at + (uint32_t)((MINE - 1) * kPass * 128));
#pragma unroll
                for (int i = 0; i < LA; ++i)
                    bring(src_a[i], cut, buf_a, (int64_t)s * 128, at + (uint32_t)(TN * 128 + i * kPass * 128));
            };
            request(0);
            request(1);
            request(2);
            for (int ks = 0; ks < nk; ++ks) {
                // (lgkmcnt: this wavefront's own reads of slice ks - 1 are back too -- nothing else keeps the MFMAs that consume
                // them, and with them their wait, in front of this barrier)
                asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(2 * (LA + MINE)) : "memory");
                request(ks + 3);
                if (none) continue;                          // uniform; the same barriers
                const unsigned char* base = smem + (size_t)(ks & 3) * kStageB;
#pragma unroll
                for (int kk = 0; kk < kTK / 16; ++kk) {
                    bf16x8_t af[WM], bf[WN];
#pragma unroll
                    for (int m = 0; m < WM; ++m)
                        af[m] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const u32x4*>(base + (fa0 ^ (kk * 32)) + 32 * m * 128));
#pragma unroll
                    for (int n = 0; n < WN; ++n)
                        bf[n] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const u32x4*>(base + (fb0 ^ (kk * 32)) + 32 * n * 128));
#pragma unroll
                    for (int m = 0; m < WM; ++m)
#pragma unroll
                        for (int n = 0; n < WN; ++n)
                            acc[m][n] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[m], bf[n], acc[m][n], 0, 0, 0);
                }
            }
        };
        if constexpr (kNarrow) {
            static_assert(LB == 4, "0 to 4 requests per wavefront");
            const int live = ((int)tn - 8 * swave + kPass - 1) / kPass;          // 0 .. 4
            if (live >= 4) walk(std::integral_constant<int, 4>{});
            else if (live == 3) walk(std::integral_constant<int, 3>{});
            else if (live == 2) walk(std::integral_constant<int, 2>{});
            else if (live == 1) walk(std::integral_constant<int, 1>{});
            else walk(std::integral_constant<int, 0>{});
        } else {
            walk(std::integral_constant<int, LB>{});
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // (slices past the end: requested, never read)
    } else if constexpr (PIPE == LOOP_TURNS) {
        // Two wavefronts share a SIMD and take turns, a barrier ending every turn: while one multiplies a
        // 16-element step (nothing but its MFMAs), the other issues its memory work -- the LDS reads of its NEXT step's
        // fragments and a few requests that bring a later slice from memory straight into LDS -- and waits for none of
        // it: whatever a wavefront reads in a memory turn is there at the end of its following multiply turn.  So the
        // multiplying wavefront never queues behind a memory instruction.  Both groups run the same program, the
        // second (wavefronts 4..7; w and w + 4 share a SIMD: the dispatcher deals them round robin, and a machine that
        // dealt them otherwise would lose time and nothing else) one turn behind the first.
        //   What bounds it: the matrix cores at the clock that their load leaves.  512 rows x 4096 x 151936: 2374 cycles per
        //     slice of which the MFMAs are 2048, at 1.6 GHz (2.4 when the operands do not change, 1.95 when the rows of M
        //     come from L2); 594 us in the kernel trace against 645 for a form of this loop that brought slices through
        //     registers (its LDS writes, staging registers and 64-bit addresses made the memory turn 410 cycles).
        //   LDS: three stages for the rows of M (they come from HBM: requested two slices and a half ahead), two for
        //     the hidden rows (L2-resident: one and a half); 160 KB with 256 x 256 tiles.
        //   Layout: rows of 128 bytes, unpadded -- a request's 64 x 16 bytes land next to each other -- with the 16-byte
        //     unit u of row r at place u ^ ((r >> 1) & 7): the fragment reads (32 rows x 2 adjacent units) run at 208
        //     B/clk like on padded rows (222); u ^ (r & 7) 123, unswizzled 32.  The swizzle is made by the lanes'
        //     memory addresses.
        //   Slice s starts at turn b = 8 s; the first group's memory turns are b + 2 m, the second's b + 2 m + 1.  It is read
        //     from turn b - 2 to b + 5 (its last reads are waited for within their turn), so from b + 6 on the stages it
        //     lay in are free: x of slice s + 2 is requested in memory turn 3 of slice s, M of slice s + 2 in memory turns 0
        //     and 1 of slice s (its stage was slice s - 1's).  Slice s + 1 has to be there at turn b + 6: every wavefront
        //     waits at the end of turn b + 5 until only its requests for M of slice s + 2 are outstanding.
        // A ragged last slice: units past a row's end are requested from outside the buffer and arrive as zeros.
        // A ragged last tile of hidden rows: groups of 32 that are past the end are not multiplied, and what a multiply turn does
        // not do shortens it (140 rows x 4096 x 128256 254 -> 224 us, 200 264 -> 252, 300 417 -> 401).
        static_assert(GM * GN == 8, "eight wavefronts: two per SIMD");
        constexpr int kAStage = TM * 128, kBStage = TN * 128;
        constexpr int LA = TM / 64, LB = TN / 64;            // requests per wavefront and slice (8 rows each)
        static_assert(LB % 2 == 0 && LA % 2 == 0, "requests go in pairs");
        constexpr int LB0 = (LB / 2 + 1) / 2 * 2;            // of those for M: in memory turn 0, the rest in turn 1
        const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;
        const int swave = __builtin_amdgcn_readfirstlane(wave);
        const uint32_t lds_b = lds0 + (uint32_t)swave * 1024u, lds_a = lds_b + 3u * kBStage;
        const int l8 = lane >> 3;
        const int unit = (lane & 7) ^ ((4 * (swave & 1) + (l8 >> 1)) & 7);
        const bool lane_past = (nk - 1) * 8 + unit >= C;     // of the last slice
        const char* const base_a = a.x + (int64_t)rt * TM * a.x_row_bytes;
        const char* const base_b = a.idx ? a.M : a.M + tile0 * a.m_row_bytes;
        LaneSource<FAR> src_a[LA], src_b[LB];
#pragma unroll
        for (int i = 0; i < LA; ++i) {
            const int row = rt * TM + 64 * i + 8 * swave + l8;
            src_a[i].set(base_a, min(row, a.rows - 1) - rt * TM, a.x_row_bytes, (uint32_t)unit * 16u);
            if constexpr (!FAR) {
                if (row >= a.rows) src_a[i].at = kOutside;   // zeros, from nowhere
            }
        }
#pragma unroll
        for (int i = 0; i < LB; ++i) {
            int64_t item = tile0 + 64 * i + 8 * swave + l8;
            if (item > tile_end - 1) item = tile_end - 1;
            src_b[i].set(base_b, a.idx ? (int64_t)a.idx[item] : item - tile0, a.m_row_bytes, (uint32_t)unit * 16u);
        }
        const i32x4_t buf_a = buffer_of(base_a), buf_b = buffer_of(base_b);
        auto request_a = [&](int ks, int stage) {
            const int s = eff(ks);
            const bool cut = s == nk - 1 && lane_past;
#pragma unroll
            for (int i = 0; i < LA; i += 2)
                bring<8192>(src_a[i], src_a[i + 1], cut, cut, buf_a, (int64_t)s * 128, lds_a + (uint32_t)(stage * kAStage + i * 8192));
        };
        auto request_b = [&](int ks, int stage, int lo, int hi) {
            const int s = eff(ks);
            const bool cut = s == nk - 1 && lane_past;
#pragma unroll
            for (int i = 0; i < LB; i += 2)
                if (i >= lo && i < hi)
                    bring<8192>(src_b[i], src_b[i + 1], cut, cut, buf_b, (int64_t)s * 128, lds_b + (uint32_t)(stage * kBStage + i * 8192));
        };
        // fragments: lane = (row within 32, k-group); unit 2 kk + k-group of a row, swizzled
        const int swz = ((lane >> 5) ^ ((lane >> 1) & 7)) * 16;
        const int fa0 = 3 * kBStage + (wr * 32 * WM + (lane & 31)) * 128 + swz, fb0 = (wc * 32 * WN + (lane & 31)) * 128 + swz;
        bf16x8_t fa[2][WM], fb[2][WN];
        auto read_frags = [&](int sta, int stb, int kk, bf16x8_t (&A)[WM], bf16x8_t (&B)[WN]) {
            const unsigned char* pa_ = smem + ((fa0 ^ (kk * 32)) + sta * kAStage);
            const unsigned char* pb_ = smem + ((fb0 ^ (kk * 32)) + stb * kBStage);
#pragma unroll
            for (int m = 0; m < WM; ++m) A[m] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const u32x4*>(pa_ + 32 * m * 128));
#pragma unroll
            for (int n = 0; n < WN; ++n) B[n] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const u32x4*>(pb_ + 32 * n * 128));
        };
        const bool second = swave >= 4;
        auto turn_ends = [&]() { asm volatile("s_barrier" ::: "memory"); };
        auto slice_landed = [&]() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LB) : "memory"); };
        request_b(0, 0, 0, LB);
        request_a(0, 0);
        request_b(1, 1, 0, LB);
        request_a(1, 1);
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LA + LB) : "memory");
        turn_ends();
        read_frags(0, 0, 0, fa[0], fb[0]);
        __builtin_amdgcn_s_waitcnt(0xC07F);
        if (second) turn_ends();               // the second group starts one turn later ...
        // (SOME: only the wavefront's first `live` groups of 32 hidden rows are any)
        int live = __builtin_amdgcn_readfirstlane((a.rows - (rt * TM + (swave / GN) * 32 * WM) + 31) / 32);
        // (A 128 x 256 tile that has one group of four would be done with its slices so much sooner than the whole tiles of the same rows
        // of M that these find them gone from L2: 140 rows x 4096 x 28000, 3.25 million L2 misses against 2.49, 66 us against 55 -- and 61 when
        // nothing was left out.  So it multiplies the first wavefronts' other group too, unless there is more than one round of
        // workgroups, where whoever is ahead goes on to the next: 285 rows x 60000 191 against 187.)
        if (TM == 128 && TN == 256 && swave < GN && live == 1 && gridDim.x <= kRound) live = WM;
        auto walk = [&](auto some) {
            int st0 = 0, st1 = 1, st2 = 2;         // stages of M: slice ks, ks + 1, ks + 2
            for (int ks = 0; ks < nk; ++ks) {
                const int sta = ks & 1;
                static_for<0, 4>([&](auto mc) {
                    constexpr int m = decltype(mc)::value;
                    // memory turn
                    if constexpr (m < 3) read_frags(sta, st0, m + 1, fa[(m + 1) & 1], fb[(m + 1) & 1]);
                    else read_frags(sta ^ 1, st1, 0, fa[0], fb[0]);
                    if constexpr (m == 0) request_b(ks + 2, st2, 0, LB0);
                    if constexpr (m == 1) request_b(ks + 2, st2, LB0, LB);
                    if constexpr (m == 3) request_a(ks + 2, sta);
                    if constexpr (m == 2) {
                        __builtin_amdgcn_s_waitcnt(0xC07F);      // the slice's last reads: done before this turn ends
                        if (second) slice_landed();
                    }
                    turn_ends();
                    // multiply turn
                    __builtin_amdgcn_s_setprio(1);
#pragma unroll
                    for (int i = 0; i < WM; ++i) {
                        if (decltype(some)::value && i >= live) break;           // uniform
#pragma unroll
                        for (int n = 0; n < WN; ++n)
                            acc[i][n] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[m & 1][i], fb[m & 1][n], acc[i][n], 0, 0, 0);
                    }
                    __builtin_amdgcn_s_setprio(0);
                    __builtin_amdgcn_sched_barrier(0);
                    __builtin_amdgcn_s_waitcnt(0xC07F);          // lgkmcnt(0): what the last memory turn read is there
                    if constexpr (m == 2) {
                        if (!second) slice_landed();
                    }
                    turn_ends();
                });
                const int st = st0;
                st0 = st1;
                st1 = st2;
                st2 = st;
            }
        };
        if (live >= WM) walk(std::false_type{});
        else walk(std::true_type{});       // (the same turns, and as many)
        if (!second) turn_ends();              // ... and the first ends one turn earlier: the same count for all
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // (slices past the end: requested, never read)
        turn_ends();
    } else {
        // Two register sets keep two slices in flight from global memory while a third is multiplied
        // out of LDS: on entry to step(ks, set) the set holds slice ks + 1 (the other set slice ks + 2).
        u32x4 ga0[QA], gb0[QB], ga1[QA], gb1[QB];
        auto step = [&](int ks, u32x4 (&ga)[QA], u32x4 (&gb)[QB]) {
            multiply(ks & 1);
            store(ks + 1, ga, gb);            // the other buffer: nobody reads it during this slice
            __syncthreads();                  // everyone is done with this buffer; the other is complete
            load(ks + 3, ga, gb);
        };
        load(0, ga0, gb0);
        store(0, ga0, gb0);
        load(1, ga0, gb0);
        load(2, ga1, gb1);
        __syncthreads();
        for (int ks = 0; ks < nk; ks += 2) {  // an odd slice count runs one more step, on a slice of zeros
            step(ks, ga0, gb0);
            step(ks + 1, ga1, gb1);
        }
    }

    // D[i][j]: j = lane % 32 (item), i = 8 (e / 4) + 4 (lane / 32) + e % 4 (hidden row) for element e
    const int64_t item0 = tile0 + wc * 32 * WN + (lane & 31);
    const int row0 = rt * TM + wr * 32 * WM + 4 * (lane >> 5);
    if constexpr (EPI == EPI_PICK) {
        // Band by band (the 32 GM rows that the wavefronts hold in the same accumulator group) the product goes
        // to LDS as a [32 GM x TN] tile; then 8 threads per row walk the entries of the row's index list that
        // fall into this item tile -- places pk.off[r, it] .. pk.off[r, it + 1] of the list (ascending, or a copy
        // grouped by tile: all that matters here is that a tile's entries are contiguous) -- and store the asked
        // entries at the same places of the output.
        //   The tiles of the likeliest tokens bound it: rows that draw from a skewed distribution want all 256 items of
        // them, where most tiles have a dozen entries per row.  Walked an entry at a time, 32 loads one after the other in
        // each of four bands, such a tile took up to 60 us more than the others, all of it past the end of a launch of one
        // round of workgroups.  So a thread has eight entries on their way and asks for the next ones, the next band's
        // included, before it stores these.  Lists with Zipf's distribution, a whole step: 200 rows x 600 / 40000 items
        // of 4 KB 77 -> 53 us, x 5768 / 128256 of 8 KB 319 -> 249, 100 rows x 11540 218 -> 198, 512 rows x 6260 487 -> 472;
        // evenly drawn ones within 2 % or better.
        constexpr int kBandRows = 32 * GM;
        constexpr int kPerRow = kThreads / kBandRows;
        constexpr int kBandW = TN + 8;                     // (eight rows of a wavefront's threads on banks of their own)
        constexpr int kAhead = 8;                          // entries per thread on their way
        static_assert((size_t)kBandRows * kBandW * 4 <= tile_lds_bytes<GM, GN, WM, WN, PIPE>(), "the band tile reuses the operand buffers");
        float* s_band = reinterpret_cast<float*>(smem);
        const int br = tid / kPerRow, sub = tid % kPerRow;                // this thread's row of the band
        const int tile_row0 = rt * TM + (br / 32) * 32 * WM + (br % 32);  // + 32 m: its row
        // the slices' bounds of all bands, and a band's first entries while the one before is stored
        uint32_t first[WM], end[WM];
#pragma unroll
        for (int m = 0; m < WM; ++m) {
            const int r = tile_row0 + 32 * m;
            first[m] = end[m] = 0u;
            if (r < a.rows) {
                first[m] = pk.off[(int64_t)r * pk.off_stride + it] + sub;
                end[m] = min(pk.off[(int64_t)r * pk.off_stride + it + 1], (uint32_t)pk.k);   // (a table built from an unsorted list: stay in bounds)
            }
        }
        auto ask = [&](int m, uint32_t j, int32_t (&q)[kAhead]) {
            const int32_t* list = pk.idx + (int64_t)min(tile_row0 + 32 * m, a.rows - 1) * pk.k;
            const uint32_t last = end[m] > 0u ? end[m] - 1u : 0u;
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                const uint32_t ju = j + (uint32_t)(u * kPerRow);
                if (__builtin_amdgcn_ballot_w64(ju < end[m]) == 0ull) break;      // (most slices have one or two entries per thread)
                q[u] = list[min(ju, last)];
            }
        };
        int32_t next[kAhead] = {};
        ask(0, first[0], next);
#pragma unroll
        for (int m = 0; m < WM; ++m) {
            __syncthreads();                               // the band tile (or, first, the operand buffers) is free
#pragma unroll
            for (int n = 0; n < WN; ++n)
#pragma unroll
                for (int e = 0; e < 16; ++e)
                    s_band[(wr * 32 + 8 * (e >> 2) + (e & 3) + 4 * (lane >> 5)) * kBandW + wc * 32 * WN + 32 * n + (lane & 31)] =
                        acc[m][n][e];
            __syncthreads();
            float* o = pk.out + (int64_t)(tile_row0 + 32 * m) * pk.k;
            const float* band = s_band + br * kBandW;
            int32_t now[kAhead];
            uint32_t j = first[m];
            auto put = [&]() {
#pragma unroll
                for (int u = 0; u < kAhead; ++u) {
                    const uint32_t ju = j + (uint32_t)(u * kPerRow), col = (uint32_t)(now[u] - (int32_t)(it * TN));
                    if (ju < end[m] && col < (uint32_t)TN) o[ju] = band[col];    // (the latter always for a consistent table)
                }
                j += (uint32_t)(kAhead * kPerRow);
            };
#pragma unroll
            for (int u = 0; u < kAhead; ++u) now[u] = next[u];
            if (j + (uint32_t)(kAhead * kPerRow) < end[m]) {     // a long slice: the next entries are asked for before these are stored
                do {
                    ask(m, j + (uint32_t)(kAhead * kPerRow), next);
                    put();
#pragma unroll
                    for (int u = 0; u < kAhead; ++u) now[u] = next[u];
                } while (j + (uint32_t)(kAhead * kPerRow) < end[m]);
            }
            if (m + 1 < WM) ask(m + 1, first[m + 1], next);
            if (j < end[m]) put();
        }
        return;
    }
    if constexpr (EPI == EPI_BRACKET) {
        // Nothing of the product is stored.  Per accumulator register (64 scores: 32 items of two hidden rows)
        // two comparisons with the rows' brackets give two lane masks:
        //   above hi  -> 2 x 32 bits of the rows' bit masks, gathered lane = row so that one store per wavefront
        //                and 64 rows writes them;
        //   in band   -> the (rare) lanes append (score, position) to a wavefront-private LDS list, which is
        //                emptied after every 32-row band by a dense loop that turns each entry into
        //                (key, id) in the candidate region of its (row, item tile).
        static_assert(WM % 2 == 0, "a lane collects the words of rows lane, lane + 64, ...");
        static_assert(16 * WN == 32, "the registers of a 32-row band map to the 32 bits of one word per lane");
        static_assert(bracket_lds_bytes<GM, GN, WM, WN>() <= tile_lds_bytes<GM, GN, WM, WN, PIPE>(), "the epilogue reuses the operand buffers");
        float2* s_thr = reinterpret_cast<float2*>(smem);                          // [TM] {hi, lo}
        uint32_t* s_cnt = reinterpret_cast<uint32_t*>(smem + (size_t)TM * 8);     // [TM] candidates of the row in this tile
        // per wavefront: the scores of one 32-row band, [16 WN / 4 register quads][64 lanes][4 floats]
        f32x4_t* s_dump = reinterpret_cast<f32x4_t*>(smem + (size_t)TM * 16) + (size_t)wave * (4 * WN * 64);
        __syncthreads();                                   // every wavefront is out of the operand buffers
        for (int t = tid; t < TM; t += kThreads) {
            const int row = rt * TM + t;
            // rows past the end: no score is above +inf, none compares with NaN
            s_thr[t] = row < a.rows ? reinterpret_cast<const float2*>(ep.thr)[row] : float2{INFINITY, __builtin_nanf("")};
            s_cnt[t] = 0u;
        }
        if (it == IT - 1) {                                // items past the end compare false with everything
#pragma unroll
            for (int n = 0; n < WN; ++n)
                if (item0 + 32 * n >= n_items) {
#pragma unroll
                    for (int m = 0; m < WM; ++m)
#pragma unroll
                        for (int e = 0; e < 16; ++e) acc[m][n][e] = __builtin_nanf("");
                }
        }
        __syncthreads();
        uint32_t words[WM / 2][WN];
#pragma unroll
        for (int j = 0; j < WM / 2; ++j)
#pragma unroll
            for (int n = 0; n < WN; ++n) words[j][n] = 0u;
        // candidate regions of this tile's rows: region of tile row t at cand_tile + t * row_stride (32-bit
        // arithmetic below: 64-bit multiplications per candidate cost more than everything else there)
        static_assert(TN == kKeepTileItems, "lists are kept per tile of that many items");
        constexpr uint32_t fcap = (uint32_t)kBracketFirst;
        uint64_t* cand_tile = ep.cand + ((int64_t)rt * TM * ep.item_tiles + it) * TN;
        const uint32_t row_stride = (uint32_t)(ep.item_tiles * TN);                   // < 2^24 (the vocabulary, padded)
        uint64_t* first_tile = ep.cand_first + ((int64_t)rt * TM * ep.item_tiles + it) * kBracketFirst;
        const uint32_t first_stride = (uint32_t)(ep.item_tiles * kBracketFirst);
        static_for<0, WM>([&](auto mc) {
            constexpr int m = decltype(mc)::value;
            constexpr int kHalfRows = 4;                   // lanes 32..63 hold the row four below
            float2 th[16];                                 // the brackets of this band's rows: one batch of LDS reads
#pragma unroll
            for (int e = 0; e < 16; ++e)
                th[e] = s_thr[wr * 32 * WM + 32 * m + 8 * (e >> 2) + (e & 3) + kHalfRows * (lane >> 5)];
            // the band's scores go to LDS as they are (the few lanes inside a bracket fetch theirs from there below)
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4)
#pragma unroll
                for (int n = 0; n < WN; ++n)
                    s_dump[(q4 * WN + n) * 64 + lane] = f32x4_t{acc[m][n][4 * q4], acc[m][n][4 * q4 + 1], acc[m][n][4 * q4 + 2], acc[m][n][4 * q4 + 3]};
            uint32_t inside = 0u;                          // per lane: bit 31 - (e WN + n) <=> score inside its row's bracket
            static_for<0, 16>([&](auto ec) {
                constexpr int e = decltype(ec)::value;
                constexpr int rlo = 32 * m + 8 * (e >> 2) + (e & 3);      // row within the wavefront's rows, lanes 0..31
                static_for<0, WN>([&](auto nc) {
                    constexpr int n = decltype(nc)::value;
                    const float f = acc[m][n][e];
                    const uint64_t ma = __builtin_amdgcn_ballot_w64(f > th[e].x);
                    const uint64_t mi = __builtin_amdgcn_ballot_w64(f >= th[e].y);
                    static_assert(rlo / 64 == (rlo + kHalfRows) / 64, "both rows of a register belong to the same lane group");
                    words[rlo / 64][n] = write_lanes<rlo % 64, (rlo + kHalfRows) % 64>(words[rlo / 64][n], ma);
                    // inside = 2 inside + (this lane's bit of the mask): one add-with-carry whose carry-in is the mask
                    inside = shift_in_lane_bit(inside, mi & ~ma);
                });
            });
            // The lanes with scores inside their bracket (about one per lane and band) take them out, up to four
            // per round with the four LDS reads, the four slot reservations and the four stores each issued
            // together: one round is the common case, and its latencies are paid once instead of per score.
            while (__builtin_amdgcn_ballot_w64(inside != 0u)) {
                constexpr int kPer = 4;
                int q[kPer];
                bool has[kPer];
#pragma unroll
                for (int u = 0; u < kPer; ++u) {
                    has[u] = inside != 0u;
                    q[u] = has[u] ? __clz((int)inside) : 0;               // e WN + n of the highest set bit
                    inside &= ~(0x80000000u >> q[u]);                     // (clears bit 31 of a word that is already 0)
                }
                float f[kPer];
                int row_t[kPer];
#pragma unroll
                for (int u = 0; u < kPer; ++u) {
                    const int e = q[u] / WN, n = q[u] % WN;
                    f[u] = reinterpret_cast<const float*>(s_dump)[(((e >> 2) * WN + n) * 64 + lane) * 4 + (e & 3)];
                    row_t[u] = wr * 32 * WM + 32 * m + 8 * (e >> 2) + (e & 3) + 4 * (lane >> 5);
                }
                uint32_t slot[kPer];
#pragma unroll
                for (int u = 0; u < kPer; ++u) slot[u] = has[u] ? atomicAdd(&s_cnt[row_t[u]], 1u) : 0u;   // < TN
#pragma unroll
                for (int u = 0; u < kPer; ++u) {
                    if (has[u]) {
                        const uint32_t item = (uint32_t)item0 + 32u * (uint32_t)(q[u] % WN);
                        uint64_t* dst = slot[u] < fcap
                                            ? first_tile + (__umul24((uint32_t)row_t[u], first_stride) + slot[u])
                                            : cand_tile + (__umul24((uint32_t)row_t[u], row_stride) + (slot[u] - fcap));
                        *dst = ((uint64_t)f32_to_ord(f[u]) << 32) | (uint32_t)(~item);
                    }
                }
            }
        });
        // lane l stores the words of the wavefront's rows l, l + 64, ...
#pragma unroll
        for (int j = 0; j < WM / 2; ++j) {
            const int row = rt * TM + wr * 32 * WM + 64 * j + lane;
            if (row < a.rows) {
                uint32_t* o = ep.bits + (int64_t)row * ep.words_per_row + it * (TN / 32) + wc * WN;
#pragma unroll
                for (int n = 0; n < WN; ++n) o[n] = words[j][n];
            }
        }
        __syncthreads();                                   // all candidates of the tile are counted
        for (int t = tid; t < TM; t += kThreads) {
            const int row = rt * TM + t;
            if (row < a.rows) ep.cnt[(int64_t)row * ep.item_tiles + it] = s_cnt[t];
        }
        return;
    }
#pragma unroll
    for (int m = 0; m < WM; ++m)
#pragma unroll
        for (int n = 0; n < WN; ++n) {
            const int64_t item = item0 + 32 * n;
            if (item >= tile_end) continue;
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int r = row0 + 32 * m + 8 * (e >> 2) + (e & 3);
                if (r < a.rows) a.out_f32[(int64_t)r * a.out_row_stride + item] = acc[m][n][e];
            }
        }
}

// The loops fed from memory to LDS keep byte offsets in 32 bits where these reach: from a tile's first row for a whole matrix,
// from the matrix itself for rows by list.  The same slices in the same order either way.
bool near(const GemvArgs& a) {
    constexpr int64_t kSpan = (int64_t)kBufferBytes;
    if (256 * a.x_row_bytes > kSpan || 256 * a.m_row_bytes > kSpan) return false;
    return a.idx == nullptr || (a.m_rows > 0 && a.m_rows <= kSpan / a.m_row_bytes);
}
// (the bracketed selection's operands are dense, and a W_vocab with rows of 16 MB would not fit any memory)
template <int PIPE, int EPI>
constexpr bool has_far() { return PIPE != LOOP_PLAIN && EPI != EPI_BRACKET; }

// more than 64 KiB of dynamic LDS needs an explicit opt-in per kernel instance and device
template <int GM, int GN, int WM, int WN, int PIPE, int EPI>
hipError_t opt_in_lds() {
    constexpr size_t bytes = tile_lds_bytes<GM, GN, WM, WN, PIPE>();
    if (bytes <= 64 * 1024) return hipSuccess;
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&tile_mfma_kernel<GM, GN, WM, WN, PIPE, EPI, false>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    if constexpr (has_far<PIPE, EPI>()) {
        if (e == hipSuccess)
            e = hipFuncSetAttribute(reinterpret_cast<const void*>(&tile_mfma_kernel<GM, GN, WM, WN, PIPE, EPI, true>),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    }
    return e;
}

template <int GM, int GN, int WM, int WN, int PIPE, int EPI = EPI_STORE>
hipError_t launch_tile(const GemvArgs& a, hipStream_t stream, const BracketEpi& ep = BracketEpi{},
                       const PickEpi& pk = PickEpi{}) {
    constexpr int TM = 32 * GM * WM, TN = 32 * GN * WN;
    const int64_t RT = (a.rows + TM - 1) / TM;
    int64_t IT = (a.n_items + TN - 1) / TN;
    if (EPI == EPI_STORE && a.balance_cus > 0)                  // narrower tiles: whole rounds of balance_cus workgroups
        IT = (IT + a.balance_cus - 1) / a.balance_cus * a.balance_cus;
    const int64_t groups = (IT + kXcds - 1) / kXcds;            // item tiles per XCD, rounded up
    const int64_t bx = groups * RT * kXcds;
    if (bx > 0x7fffffffLL) return hipErrorInvalidValue;         // more tiles than a grid dimension holds
    auto go = [&](auto kernel) {                                // LDS above 64 KiB: opted in by configure_tile_mfma_lds()
        hipLaunchKernelGGL(kernel, dim3((unsigned)bx), dim3(64 * GM * GN), (tile_lds_bytes<GM, GN, WM, WN, PIPE>()), stream, a, ep, pk);
        return hipGetLastError();
    };
    if (PIPE == LOOP_PLAIN || near(a)) return go(&tile_mfma_kernel<GM, GN, WM, WN, PIPE, EPI, false>);
    if constexpr (has_far<PIPE, EPI>()) return go(&tile_mfma_kernel<GM, GN, WM, WN, PIPE, EPI, true>);
    return hipErrorInvalidValue;
}

}  // namespace

// every instance launch_tile_mfma can pick, on the current device (called once per device, outside any
// stream capture, by the library's device set-up)
hipError_t configure_tile_mfma_lds() {
    hipError_t e = hipSuccess;
    auto all_epilogues = [&](auto fn) {
        if (e == hipSuccess) e = fn(std::integral_constant<int, EPI_STORE>{});
        if (e == hipSuccess) e = fn(std::integral_constant<int, EPI_BRACKET>{});
        if (e == hipSuccess) e = fn(std::integral_constant<int, EPI_PICK>{});
    };
    if (e == hipSuccess) e = opt_in_lds<1, 8, 2, 1, LOOP_RING, EPI_STORE>();
    if (e == hipSuccess) e = opt_in_lds<1, 2, 1, 1, LOOP_RING, EPI_STORE>();
    if (e == hipSuccess) e = opt_in_lds<1, 4, 1, 1, LOOP_RING, EPI_STORE>();
    if (e == hipSuccess) e = opt_in_lds<2, 2, 1, 1, LOOP_RING, EPI_STORE>();
    if (e == hipSuccess) e = opt_in_lds<2, 4, 1, 1, LOOP_RING, EPI_STORE>();
    if (e == hipSuccess) e = opt_in_lds<2, 4, 2, 1, LOOP_TURNS, EPI_STORE>();
    all_epilogues([](auto ec) { return opt_in_lds<2, 4, 2, 2, LOOP_TURNS, decltype(ec)::value>(); });
    all_epilogues([](auto ec) { return opt_in_lds<2, 4, 4, 2, LOOP_TURNS, decltype(ec)::value>(); });
    return e;
}

// Tiles of the alternating loop for more than 64 hidden rows.  A tile walks the whole reduction whatever the list's length,
// so what decides is how many rounds of workgroups a shape makes of the product and what a round costs: alone on the
// chip (latency), and with every CU busy (the MFMAs' power, the pass over M).  Measured at d = 4096, a round with few
// tiles / a full one, us: 256 x 256 70 / 117-141, 128 x 256 51 / 74-82, 128 x 128 41 / 54 (one workgroup per CU; two:
// 78-88 for twice the tiles); in between a square law fits within a few per cent, and d = 1536 scales all of them alike.
// 256 rows: 4096 items 42 us on 128 x 128 against 70 on 256 x 256, 32768 82 on 128 x 256 against 88, 65536 141 on
// 256 x 256 against 163.
enum TileShape { TILE_256x256, TILE_128x256, TILE_128x128 };
static TileShape tile_shape(int rows, int64_t n_items, int cus, bool wide_only) {
    const double rt128 = (rows + 127) / 128, rt256 = (rows + 255) / 256, it128 = (double)((n_items + 127) / 128), it256 = (double)((n_items + 255) / 256);
    auto cost = [&](double tiles, double alone, double full) {
        const double rounds = tiles / cus, whole = floor(rounds), part = rounds - whole;
        return whole * full + (part > 0 ? alone + (full - alone) * part * part : 0.0);
    };
    const double c256 = cost(rt256 * it256, 70, 125), c128 = cost(rt128 * it256, 51, 78);
    // two workgroups per CU: pairs of rounds, the first of which ends at 54
    const double tiles = rt128 * it128, pairs = floor(tiles / (2.0 * cus)), rest = tiles / cus - 2 * pairs;
    const double small = pairs * 82 + (rest > 1 ? 54 + 28 * (rest - 1) : rest > 0 ? 41 + 13 * rest * rest : 0.0);
    if (!wide_only && small < c128 && small < c256) return TILE_128x128;
    return c128 <= c256 ? TILE_128x256 : TILE_256x256;
}
static hipError_t shape_for(const GemvArgs& a, bool wide_only, TileShape* out) {
    DeviceInfo di;
    const hipError_t e = device_info(&di);
    if (e != hipSuccess) return e;
    *out = tile_shape(a.rows, a.n_items, di.cus, wide_only);
    return hipSuccess;
}

// the epilogues that keep something per item tile: tiles of kKeepTileItems items, whatever the number of hidden rows
template <int EPI>
static hipError_t launch_wide(const GemvArgs& a, hipStream_t stream, const BracketEpi& ep, const PickEpi& pk) {
    if (a.n_items <= 0 || a.rows <= 0) return hipSuccess;
    TileShape s;
    const hipError_t e = shape_for(a, true, &s);
    if (e != hipSuccess) return e;
    return s == TILE_256x256 ? launch_tile<2, 4, 4, 2, LOOP_TURNS, EPI>(a, stream, ep, pk)
                             : launch_tile<2, 4, 2, 2, LOOP_TURNS, EPI>(a, stream, ep, pk);
}

hipError_t launch_tile_mfma_bracket(const GemvArgs& a, const BracketEpi& ep, hipStream_t stream) {
    return launch_wide<EPI_BRACKET>(a, stream, ep, PickEpi{});
}

hipError_t launch_tile_mfma_pick(const GemvArgs& a, const PickEpi& pk, hipStream_t stream) {
    return launch_wide<EPI_PICK>(a, stream, BracketEpi{}, pk);
}

hipError_t launch_tile_mfma(const GemvArgs& a, hipStream_t stream) {
    if (a.n_items <= 0 || a.rows <= 0) return hipSuccess;
    // Up to 64 hidden rows (the caller decides when this beats the kernel without LDS tiles) the product is one
    // pass over M at the rate of the memory system, and what matters is how evenly the list's items spread over
    // the chip and how much of them is on its way: the ring, which has three slices in flight, on tiles of
    //   17 to 32 rows: 32 x 64 (two wavefronts, three workgroups per CU) up to 64 x CUs items (32 rows of 3840 elements x 10000
    //     items from HBM 23.5 us against 29.7 on 32 x 128 tiles, 16384 26.1 against 33.9); 32 x 128 (four wavefronts, two
    //     workgroups per CU) up to one workgroup per CU, and where two per CU are nearly full (32 rows x 24576 items 38.7
    //     against 43.6 on 32 x 64 tiles of the plain loop, 65536 96 against 98); in between those (49152: 78 against 73), and
    //     for short reductions, the plain loop's;
    //   33 to 64 rows: 64 x 256 (eight wavefronts, one workgroup per CU) when the list fills its last round of 256 x CUs
    //     items, or more than half of it (128256 items 188 us against 192 on the tiles below, 49152 75 against 82), or few of
    //     one beyond the first -- and for a count on the device, which a tree step has --, of a width that then fills whole
    //     rounds; otherwise 64 x 64
    //     (four wavefronts, two workgroups per CU) up to 64 x CUs items and 64 x 128 (eight wavefronts of 32 x 32) beyond:
    //     64 rows of 4096 elements x 9000 / 16384 items from HBM 25.6 / 28.7 us against 33.0 / 36.9 on 64 x 128 tiles, of
    //     4104 elements 36.4 / 41.0 against 51.3 / 55.3; 60 rows x 24576 / 32768 / 98304 items 42 / 50 / 149 on those.
    if (a.rows <= 64) {
        DeviceInfo di;
        const hipError_t e = device_info(&di);
        if (e != hipSuccess) return e;
        if (a.rows <= 32) {
            if (a.chunks > 64 && a.n_items <= (int64_t)di.cus * 64) return launch_tile<1, 2, 1, 1, LOOP_RING>(a, stream);
            const bool ring = a.chunks > 64 && (a.n_items <= (int64_t)di.cus * 128 || a.n_items >= (int64_t)di.cus * 224);
            return ring ? launch_tile<1, 4, 1, 1, LOOP_RING>(a, stream) : launch_tile<1, 2, 1, 1, LOOP_PLAIN>(a, stream);
        }
        const int64_t round_items = (int64_t)256 * di.cus, last = a.n_items % round_items;
        // (with a count on the device a.n_items is its upper bound: at most half a round, and the list is short for sure)
        const bool unknown = a.n_items_dev != nullptr && 2 * a.n_items > round_items;
        // (beyond a round, up to three eighths of the last one too: narrower tiles in all of them, where a second or third round of
        // a few whole ones takes as long as the others.  66000 / 81920 / 135000 / 200000 items, 60-odd rows of 8 KB, us: 122 / 131 / 220 /
        // 316 on the tiles below, 108 / 125 / 208 / 312 here, of 8208 bytes 168 / 177 / 293 / 413 and 144 / 158 / 261 / 383; 98304 151 / 150,
        // 160000 by 33 rows 229 / 230 and of 7600 bytes 257 / 262.  Rows of less than 2 KB, where a tile is mostly its start: up to an
        // eighth, 64 rows of 512 bytes x 66000 / 90000 15.7 / 17.1 on the tiles below, 14.9 / 18.5 here.)
        const bool few = a.n_items > round_items && 8 * last <= (a.chunks >= 128 ? 3 : 1) * round_items;
        if (unknown || few || last == 0 || 2 * last > round_items) {
            // (40960 items: 80 against 87 us with a width that fills whole rounds; unions of 30940 and 44831 rows: a tree
            // step in 82 and 104 us against 88 and 109)
            GemvArgs b = a;
            b.balance_cus = di.cus;
            return launch_tile<1, 8, 2, 1, LOOP_RING>(b, stream);
        }
        if (a.n_items <= (int64_t)64 * di.cus) return launch_tile<2, 2, 1, 1, LOOP_RING>(a, stream);
        return launch_tile<2, 4, 1, 1, LOOP_RING>(a, stream);
    }
    // A count on the device, up to 128 rows: the shape that is never far from the best, whatever the count turns out to be
    // (80 rows x 16384 / 32768 / 128256 items, 128 x 128: 44 / 58 / 203 us, 128 x 256: 55 / 64 / 197).
    if (a.n_items_dev != nullptr && a.rows <= 128) return launch_tile<2, 4, 2, 1, LOOP_TURNS>(a, stream);
    TileShape s;
    const hipError_t e = shape_for(a, false, &s);
    if (e != hipSuccess) return e;
    switch (s) {
        case TILE_128x128: return launch_tile<2, 4, 2, 1, LOOP_TURNS>(a, stream);
        case TILE_128x256: return launch_tile<2, 4, 2, 2, LOOP_TURNS>(a, stream);
        default: return launch_tile<2, 4, 4, 2, LOOP_TURNS>(a, stream);
    }
}

}  // namespace sv

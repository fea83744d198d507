// Products with a SHORT reduction for many hidden rows (the selector's W_vocab h', Section 3.3 Step 1, for a batch,
// and Section 3.4's distribution over the whole vocabulary):
//     s[r, j] = < M[row(j), :], x[r, :] >      r < rows (more than 64; keys also for fewer), rows of M of at most 512 elements, bf16
//
// What bounds it.  With d' = 256 a 256 x 256 output tile is four 64-element slices of main loop: the tiled kernel spends
// more time filling its pipeline, and in its epilogue, than multiplying (512 rows x 151936: 45 us of product of which
// the matrix cores need 20).  Here the hidden rows are STATIONARY:
// a wavefront keeps the fragments of its 32 WM hidden rows for the whole reduction in registers (128 of them at
// 64 rows x 256 elements), and a workgroup that owns a panel of TM = 32 WM GM hidden rows streams a long run of rows
// of M past them, 64 (32) rows at a time, from memory to a ring of three stages in LDS.  A step is then
// nothing but LDS reads of M's fragments (one per WM MFMAs), MFMAs and the epilogue; there is no prologue but the
// first tile's, and one barrier per step.  The matrix is read once per panel (once in all up to 512 hidden rows).
//
// Where the epilogue reduces or selects along the rows of M (the two that store nothing), M is the MFMA's first operand:
// a lane then holds 16 scores of ONE hidden row, whose map to codes or running maximum stays in its registers.
// (Tried and not used: the two wavefronts of a SIMD half a step apart, so that one multiplies while the other is in its
// epilogue, and a sub-tile's epilogue cut into pieces between the MFMAs of the next one: 103 and 92-95 us against 97 for
// the sums of 1024 rows x 151936 -- the matrix cores alone take 65, at the clock their load leaves.)
//
// Measured: the selection's product with its codes, 512 rows x 151936, d' = 256: 48 to 50 us (without the codes' stores 41, of
// which the matrix cores are busy 20; codes kept for a step and stored behind the next requests 58; to lines of 1 KB, rows of
// one unit side by side, 47); log-probabilities of 1024 rows x 151936 579 us on the tiled kernel, 230 here (sums 97, stored
// product 145 under a profiler: 622 MB at 4.3 TB/s).
//
// The sums are the ones the tiled kernel makes (v_mfma_f32_32x32x16_bf16 over ascending k from zero), bit for bit.
#include "sv_device.h"
#include "sv_launch.h"

#include <math.h>

#include <type_traits>

#include "memory_to_lds.h"
#include "tile_epilogue.h"

namespace sv {

namespace {

constexpr int kXcds = 8;
typedef unsigned short u16x2_t __attribute__((ext_vector_type(2)));
typedef short i16x2_t __attribute__((ext_vector_type(2)));
constexpr int kWaves = 8, kThreads = 64 * kWaves;
constexpr int kCusPerXcd = 32;           // (of the part, not asked of the device: a workspace's size follows from the runs)
constexpr int kRunUnit = 64;             // a run is a multiple of this many rows of M

// EPI_SAMPLE     row(j) = floor(j spread_V / 2^spread_shift), a sample of M's rows; the product is stored
// EPI_LOGP       the product minus a value per hidden row (the normaliser of Section 3.4) is stored
// EPI_LSE        only (maximum, sum of exponentials relative to it) per hidden row and run of rows of M
// EPI_CODES      a byte per score is stored, a monotone function of the score per hidden row (the selection of a batch)
// EPI_KEYS       two bytes per score: half precision, as a number that orders like it, of its distance from the row's middle
enum { EPI_SAMPLE = 0, EPI_LOGP = 1, EPI_LSE = 2, EPI_CODES = 3, EPI_KEYS = 4 };

template <int KS, int GM>
constexpr int step_items() { return KS > 16 ? 32 : GM > 2 ? 64 : 128; }      // rows of M per step
template <int KS, int GM>
constexpr size_t stage_bytes() { return (size_t)step_items<KS, GM>() * KS * 32; }
template <int KS, int GM>
constexpr int stages() { return stage_bytes<KS, GM>() > 32 * 1024 ? 2 : 3; }
// While the hidden rows come in, LDS holds so many steps of M ...
template <int KS, int GM>
constexpr int early_steps() { return KS > 8 ? 1 : stages<KS, GM>() - 1; }
// ... and so many hidden rows per wavefront at a time
// (keys, up to 256 elements: fewer, which leaves room for the tokens of the middle)
template <int KS, int GM, int EPI>
constexpr int fill_rows() { return EPI == EPI_KEYS && KS <= 16 ? (KS > 8 ? 16 : 32) : KS > 16 || stages<KS, GM>() == 2 ? 16 : 32; }
template <int KS, int GM, int EPI>
constexpr size_t fill_bytes() { return early_steps<KS, GM>() * stage_bytes<KS, GM>() + (size_t)kWaves * fill_rows<KS, GM, EPI>() * KS * 32; }
// The tokens that say where the middle of a row's scores lies, and where they are: behind the ring and the hidden rows on their way, or,
// more than 256 elements, in the last stage before its first step is.
template <int KS>
constexpr int middle_tokens() { return KS > 16 ? 16 : 32; }
template <int KS, int GM, int EPI>
constexpr size_t middle_at() {
    const size_t n = stages<KS, GM>() * stage_bytes<KS, GM>(), fill = fill_bytes<KS, GM, EPI>();
    return KS > 16 ? n - stage_bytes<KS, GM>() : n > fill ? n : fill;
}
template <int KS, int WM, int GM, int EPI>
constexpr size_t panel_lds_bytes() {
    size_t n = stages<KS, GM>() * stage_bytes<KS, GM>();
    if (EPI == EPI_LOGP) n += (size_t)32 * WM * GM * 4;
    if (EPI == EPI_KEYS && KS <= 16) n = middle_at<KS, GM, EPI>() + (size_t)middle_tokens<KS>() * KS * 32;
    const size_t fill = fill_bytes<KS, GM, EPI>();
    return n > fill ? n : fill;
}

// orders the LDS accesses of a wavefront's lanes for the compiler; no instruction
__device__ __forceinline__ void wavefront_fence() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// KS 16-element steps of the reduction are held (rows of M of up to 16 KS elements), WM groups of 32 hidden rows per
// wavefront, GM wavefronts along the panel; the other 8 / GM share the step's rows of M.
template <int KS, int WM, int GM, int EPI>
__global__ __launch_bounds__(kThreads) void panel_mfma_kernel(const PanelArgs a) {
    constexpr int GI = kWaves / GM;                      // wavefronts along the rows of M
    constexpr int kTI = step_items<KS, GM>();
    constexpr int SUB = kTI / (32 * GI);                 // 32-row sub-tiles per wavefront and step
    constexpr int TM = 32 * WM * GM;
    constexpr bool kSwap = EPI == EPI_LSE || EPI == EPI_CODES || EPI == EPI_KEYS;             // M is the MFMA's first operand
    constexpr int kRowB = KS * 32;                       // a staged row
    constexpr int kUnits = 2 * KS;                       // ... in units of 16 bytes
    constexpr int kPieces = kTI * kRowB / 1024;          // 1 KB pieces of a step
    constexpr int LR = kPieces / kWaves;                 // ... that a wavefront brings
    constexpr int NS = stages<KS, GM>();
    // stores of a wavefront per step whose rows are all there
    constexpr int kStores = EPI == EPI_LSE ? 0 : EPI == EPI_CODES ? SUB * WM : EPI == EPI_KEYS ? SUB * WM * 2 : SUB * WM * 16;
    static_assert(kPieces % kWaves == 0 && kTI % (32 * GI) == 0 && kUnits <= 64 && kUnits >= 16, "whole pieces, whole sub-tiles");
    static_assert(EPI != EPI_KEYS || (SUB == 1 && middle_tokens<KS>() * kRowB / 1024 % kWaves == 0), "a unit per wavefront and step; whole pieces");
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];     // [NS][kTI][kRowB], then the epilogue's
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int gm = wave % GM, gi = wave / GM;
    const int C = a.chunks;
    // block id -> (XCD, slot on that XCD); consecutive slots of one XCD: the panels of one run of rows of M
    const int RT = (a.rows + TM - 1) / TM;
    const int slot = (int)(blockIdx.x / kXcds);
    const int panel = slot % RT;
    const int run = slot / RT * kXcds + (int)(blockIdx.x % kXcds);
    const int n_items = (int)a.n_items, run_items = (int)a.run_items;        // (below 2^22: panel_supported)
    if (run >= (n_items + run_items - 1) / run_items) return;
    const int i0 = run * run_items;
    const int i1 = i0 + run_items < n_items ? i0 + run_items : n_items;
    const int nt = (i1 - i0 + kTI - 1) / kTI;

    // M goes from memory to LDS: a step in pieces of 1 KB (64 lanes x 16 bytes), NS - 1 steps on their way.  Unit u of row r
    // lies at place u ^ (r % 16) of its row, so that the 16 rows a fragment read meets at a time are in different banks; the
    // lanes' addresses make that order.  Units past a row's end arrive as zeros; rows past the run: the run's last row again,
    // never used.  (Through registers, the compiler waited for the last step's stores in front of every write to LDS: it
    // cannot know how many there were.)
    // A run is a whole number of 32 KB of M, the memory channels' period: runs that walked in step would all be at the same
    // channels, so every run starts its steps at another piece (60 rows x 128256, a byte per score: 17.6 -> 15.6 us).
    const char* m_base = EPI == EPI_SAMPLE ? a.M : a.M + (int64_t)i0 * a.m_row_bytes;
    const i32x4_t m_buf = buffer_of(m_base);
    const uint32_t m_row_bytes = (uint32_t)a.m_row_bytes;                    // n_items * m_row_bytes < 2^32: panel_supported
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;
    const int turn = run * 11 % kPieces;
    auto request = [&](int t, int stage) {
#pragma unroll
        for (int i = 0; i < LR; ++i) {
            const int piece = (i * kWaves + wave + turn) % kPieces;
            const int r = piece * (64 / kUnits) + lane / kUnits;
            const uint32_t u = (uint32_t)((lane % kUnits) ^ (r & 15));
            uint32_t row = (uint32_t)min(t * kTI + r, i1 - i0 - 1);
            if constexpr (EPI == EPI_SAMPLE) row = (uint32_t)(((uint64_t)(row + (uint32_t)i0) * (uint64_t)a.spread_V) >> a.spread_shift);
            memory_to_lds((int)u < C ? row * m_row_bytes + u * 16u : kOutside, m_buf, 0u,
                          lds0 + (uint32_t)(stage * (int)stage_bytes<KS, GM>() + piece * 1024));
        }
    };

    [[maybe_unused]] auto request_middle = [&]() {       // tokens from all of M, laid out like a step
        const i32x4_t whole = buffer_of(a.M);
#pragma unroll
        for (int i = 0; i < middle_tokens<KS>() * kRowB / 1024 / kWaves; ++i) {
            const int piece = i * kWaves + wave;
            const int r = piece * (64 / kUnits) + lane / kUnits;
            const uint32_t u = (uint32_t)((lane % kUnits) ^ (r & 15));
            // (spread over what lies between, so that they are not all multiples of something)
            const uint32_t row = min((uint32_t)(2 * r + 1) * (uint32_t)n_items / (uint32_t)(2 * middle_tokens<KS>()) + (uint32_t)(11 * r % 32),
                                     (uint32_t)n_items - 1u);
            memory_to_lds((int)u < C ? row * m_row_bytes + u * 16u : kOutside, whole, 0u, lds0 + (uint32_t)middle_at<KS, GM, EPI>() + (uint32_t)(piece * 1024));
        }
    };

    // This wavefront's hidden rows: lane = (row within a group of 32, k-group), like every operand of the MFMA.  They come
    // through LDS (a part of all of it per wavefront, before the first stage is filled): whole rows per load instruction,
    // where the operand's own shape, 32 bytes of 32 rows, took 15 us for the 256 KB of a panel.
    const int row_w = panel * TM + gm * 32 * WM;         // first hidden row of the wavefront
    bf16x8_t fx[WM][KS];
    {
        constexpr int kRows = fill_rows<KS, GM, EPI>();  // rows per round
        constexpr int kLoads = kRows * kUnits / 64, kRounds = WM * 32 / kRows;
        unsigned char* s_fill = smem + early_steps<KS, GM>() * stage_bytes<KS, GM>() + (size_t)wave * kRows * kRowB;
        auto fetch = [&](int round, u32x4 (&v)[kLoads]) {
#pragma unroll
            for (int q = 0; q < kLoads; ++q) {
                const int p = q * 64 + lane, u = p % kUnits;
                const int row = min(row_w + kRows * round + p / kUnits, a.rows - 1);   // padding rows: never stored
                v[q] = reinterpret_cast<const u32x4*>(a.x + (int64_t)row * a.x_row_bytes)[u < C ? u : C - 1];
            }
        };
        u32x4 v[kLoads];
        fetch(0, v);                                     // (in front of M's requests: loads come back in order)
        if constexpr (EPI == EPI_KEYS && KS <= 16) request_middle();
#pragma unroll
        for (int t = 0; t < early_steps<KS, GM>(); ++t)
            if (t < nt) request(t, t);
#pragma unroll
        for (int round = 0; round < kRounds; ++round) {
            const int m = round * kRows / 32, part = round % (32 / kRows);
#pragma unroll
            for (int q = 0; q < kLoads; ++q) {           // (units at the places that M's have)
                const int p = q * 64 + lane, u = p % kUnits, r = p / kUnits;
                *reinterpret_cast<u32x4*>(s_fill + r * kRowB + (u ^ (r & 15)) * 16) = u < C ? v[q] : zero16();
            }
            if (round + 1 < kRounds) fetch(round + 1, v);
            // (a wavefront's own LDS accesses stay in order in the hardware; the fences keep the compiler from moving a
            // lane's reads in front of the other lanes' writes, or the next round's writes in front of these reads)
            wavefront_fence();
            if (32 / kRows == 1 || (lane & 31) / kRows == part) {
                const unsigned char* mine = s_fill + ((lane & 31) % kRows) * kRowB;
#pragma unroll
                for (int kk = 0; kk < KS; ++kk)
                    fx[m][kk] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const u32x4*>(
                                                                 mine + (((2 * kk + (lane >> 5)) ^ ((lane & 31) % kRows & 15)) * 16)));
            }
            wavefront_fence();
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the first steps
        __syncthreads();                                 // ... are there; the fill regions are a stage from here on
    }

    // ---- per-workgroup state of the epilogues, behind the stages
    unsigned char* s_epi = smem + NS * stage_bytes<KS, GM>();
    [[maybe_unused]] float* s_sub = reinterpret_cast<float*>(s_epi);          // EPI_LOGP: [TM]
    const int half = lane >> 5;
    // EPI_CODES and EPI_KEYS, of hidden row row_w + 32 m + lane % 32: what makes a score a code or key, and where the lane's go
    [[maybe_unused]] float map_scale[WM], map_bias[WM];
    [[maybe_unused]] char* code_row[WM];
    [[maybe_unused]] uint32_t sample_at[WM];             // EPI_KEYS: where the row's sample goes that this wavefront has ...
    [[maybe_unused]] u32x4 kept[WM];                     // ... 16 bytes at a time
    if constexpr (EPI == EPI_CODES) {
#pragma unroll
        for (int m = 0; m < WM; ++m) {
            const int row = min(row_w + 32 * m + (lane & 31), a.rows - 1);
            const float2 t = reinterpret_cast<const float2*>(a.code_map)[row];
            map_scale[m] = t.x;
            map_bias[m] = t.y;
            code_row[m] = reinterpret_cast<char*>(a.codes) + (int64_t)row * a.code_stride + 16 * half;
        }
    }
    if constexpr (EPI == EPI_KEYS) {
#pragma unroll
        for (int m = 0; m < WM; ++m) {
            const int row = min(row_w + 32 * m + (lane & 31), a.rows - 1);
            code_row[m] = reinterpret_cast<char*>(a.codes) + (int64_t)row * a.code_stride + 32 * half;
            u16x2_t top = {0, 0};                        // the largest of the row's elements, without their signs
#pragma unroll
            for (int kk = 0; kk < KS; ++kk) {
                const u32x4 x = __builtin_bit_cast(u32x4, fx[m][kk]);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t w = x[i] & 0x7FFF7FFFu;
                    top = __builtin_elementwise_max(top, __builtin_bit_cast(u16x2_t, w));
                }
            }
            uint32_t e = umax32(top[0], top[1]) >> 7;
            e = umax32(e, (uint32_t)__shfl_xor((int)e, 32));
            e = e < 1u ? 1u : e > 253u ? 253u : e;
            map_scale[m] = __uint_as_float((254u - e) << 23);
            sample_at[m] = (uint32_t)row * (uint32_t)a.sample_stride + (uint32_t)((run * GI + gi) * a.sample_groups) * 16u;
        }
        // The middle of a row's scores: near the median of those of 32 (16) tokens from all of M, the same in every workgroup.  Without it
        // half precision keeps of scores with a common offset what the offset leaves: at 20 standard deviations 60 to 180 of 128256
        // tokens have the k-th one's key (k = 4096), at some hundreds thousands (60 rows, d' = 256, the whole selection: 49 us at 10
        // standard deviations, 56 at 20, 190 at 100, for the 41 of none).
        if constexpr (KS > 16) {
            request_middle();
            asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
        }
        const unsigned char* s_mid = smem + middle_at<KS, GM, EPI>() + (lane & (middle_tokens<KS>() - 1)) * kRowB;
#pragma unroll
        for (int m = 0; m < WM; ++m) {
            f32x16_t mid;
#pragma unroll
            for (int e = 0; e < 16; ++e) mid[e] = 0.f;
#pragma unroll
            for (int kk = 0; kk < KS; ++kk)
                mid = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                    __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const u32x4*>(s_mid + (((2 * kk + half) ^ (lane & 15)) * 16))),
                    fx[m][kk], mid, 0, 0, 0);
            // Of nine of the lane's tokens the median of three medians, or of three maxima where the upper tokens are wanted, and the smaller of this
            // and lane + 32's: a score that is there, and not a mean of two groups of tokens that have little in common
            float t[3];
#pragma unroll
            for (int i = 0; i < 3; ++i)
                t[i] = a.upper_wanted ? fmaxf(fmaxf(mid[3 * i], mid[3 * i + 1]), mid[3 * i + 2])
                                      : __builtin_amdgcn_fmed3f(mid[3 * i], mid[3 * i + 1], mid[3 * i + 2]);
            t[0] = __builtin_amdgcn_fmed3f(t[0], t[1], t[2]);
            const float middle = fminf(t[0], __shfl_xor(t[0], 32));
            const float bias = 0.0f - middle * map_scale[m];
            map_bias[m] = fabsf(bias) <= 1e30f ? bias : 0.0f;                 // (infinite scores, and those that are no number)
        }
        if constexpr (KS > 16) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");     // the stage is free
    }
    if constexpr (EPI == EPI_LOGP) {
        for (int t = tid; t < TM; t += kThreads) s_sub[t] = panel * TM + t < a.rows ? a.row_sub[panel * TM + t] : 0.0f;
        __syncthreads();
    }
    float run_max[WM], run_sum[WM];                      // EPI_LSE: of hidden row row_w + 32 m + lane % 32
#pragma unroll
    for (int m = 0; m < WM; ++m) {
        run_max[m] = -INFINITY;
        run_sum[m] = 0.0f;
    }

    f32x16_t acc[WM];
    // places of the lane's units 2 kk + lane / 32, kk < 8, of row lane % 32 (kk + 8: 256 bytes on)
    uint32_t b_lane[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) b_lane[j] = (uint32_t)((lane & 31) * kRowB + (((lane >> 5) ^ (lane & 15)) * 16 ^ (j * 32)));
    auto multiply = [&](int stage, int s) {
        const unsigned char* sb = smem + stage * (int)stage_bytes<KS, GM>() + (gi * SUB + s) * 32 * kRowB;
#pragma unroll
        for (int m = 0; m < WM; ++m)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[m][e] = 0.f;
        // M's fragments are read four 16-element steps ahead of their MFMAs; the fence keeps the compiler from reading all
        // of them first (registers)
        constexpr int kAhead = 4;
        static_assert(KS % kAhead == 0, "whole groups of steps");
        bf16x8_t fb[2][kAhead];
        auto read = [&](int g, bf16x8_t (&b)[kAhead]) {
#pragma unroll
            for (int i = 0; i < kAhead; ++i)
                b[i] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const u32x4*>(sb + b_lane[(g * kAhead + i) & 7] + (g * kAhead + i) / 8 * 256));
        };
        read(0, fb[0]);
#pragma unroll
        for (int g = 0; g < KS / kAhead; ++g) {
            if (g + 1 < KS / kAhead) read(g + 1, fb[(g + 1) & 1]);
#pragma unroll
            for (int i = 0; i < kAhead; ++i)
#pragma unroll
                for (int m = 0; m < WM; ++m) {
                    const bf16x8_t b = fb[g & 1][i], x = fx[m][g * kAhead + i];
                    if constexpr (kSwap) acc[m] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b, x, acc[m], 0, 0, 0);
                    else acc[m] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x, b, acc[m], 0, 0, 0);
                }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    // first row of M of the wavefront's sub-tile s of step t
    auto item_of = [&](int t, int s) { return i0 + t * kTI + (gi * SUB + s) * 32; };

    // EPI_KEYS: a step's sample leaves with the last of so many steps (less one)
    [[maybe_unused]] const int sample_mask = a.sample_words == 4 ? 0 : a.sample_words == 2 ? 1 : 3;
    auto epilogue = [&](int t, int s) {
        const int j0 = item_of(t, s);
        if constexpr (EPI == EPI_SAMPLE || EPI == EPI_LOGP) {
            // element e: hidden row 8 (e / 4) + 4 (lane / 32) + e % 4, item lane % 32: two 128-byte runs per store, at a
            // wavefront-uniform address plus a lane's offset that never changes
            int64_t stride = a.out_row_stride;
            asm volatile("" : "+s"(stride));             // the rows' addresses are made here, not kept in registers
            const uint32_t lane_off = (uint32_t)(4 * half * (int)stride + (lane & 31)) * 4u;
            auto store_all = [&](auto whole) {
#pragma unroll
                for (int m = 0; m < WM; ++m)
#pragma unroll
                    for (int q4 = 0; q4 < 4; ++q4) {
                        f32x4_t sub = {0.f, 0.f, 0.f, 0.f};
                        if constexpr (EPI == EPI_LOGP)
                            sub = *reinterpret_cast<const f32x4_t*>(s_sub + gm * 32 * WM + 32 * m + 8 * q4 + 4 * half);
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const int r = row_w + 32 * m + 8 * q4 + e;
                            char* o = reinterpret_cast<char*>(a.out + (int64_t)r * stride + j0) + lane_off;
                            float v = acc[m][4 * q4 + e];
                            if constexpr (EPI == EPI_LOGP) v -= sub[e];
                            if (decltype(whole)::value || (j0 + (lane & 31) < i1 && r + 4 * half < a.rows)) *reinterpret_cast<float*>(o) = v;
                        }
                    }
            };
            if (row_w + 32 * WM <= a.rows && j0 + 32 <= i1) store_all(std::true_type{});     // uniform
            else store_all(std::false_type{});
        }
        if constexpr (EPI == EPI_LSE) {
            // element e of acc[m]: hidden row 32 m + lane % 32, item 8 (e / 4) + 4 (lane / 32) + e % 4
            if (j0 + 32 > i1) {
                int left = i1 - j0 - 4 * (lane >> 5);
                asm volatile("" : "+v"(left));           // the comparisons stay inside this rare branch
#pragma unroll
                for (int e = 0; e < 16; ++e)
                    if (8 * (e >> 2) + (e & 3) >= left) {
#pragma unroll
                        for (int m = 0; m < WM; ++m) acc[m][e] = -INFINITY;
                    }
            }
#pragma unroll
            for (int m = 0; m < WM; ++m) {
                float mx = acc[m][0];
#pragma unroll
                for (int e = 1; e < 16; ++e) mx = fmaxf(mx, acc[m][e]);
                mx = fmaxf(mx, run_max[m]);
                const float ref = mx == -INFINITY ? 0.0f : mx;              // nothing seen yet
                float p[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int e = 0; e < 16; ++e) p[e & 3] += __expf(acc[m][e] - ref);
                run_sum[m] = run_sum[m] * __expf(run_max[m] - ref) + ((p[0] + p[1]) + (p[2] + p[3]));
                run_max[m] = mx;
            }
        }
        if constexpr (EPI == EPI_CODES) {
            // element e of acc[m]: hidden row 32 m + lane % 32, item 8 (e / 4) + 4 (lane / 32) + e % 4.  Byte b of word w of a
            // 32-item unit is the code of item 8 b + w: the lane's four words lie next to each other.
            if (j0 + 32 > i1) {                          // items past the run: below everything
                int left = i1 - j0 - 4 * half;
                asm volatile("" : "+v"(left));
#pragma unroll
                for (int e = 0; e < 16; ++e)
#pragma unroll
                    for (int m = 0; m < WM; ++m) acc[m][e] = 8 * (e >> 2) + (e & 3) >= left ? -INFINITY : acc[m][e];
            }
#pragma unroll
            for (int m = 0; m < WM; ++m) {
                u32x4 w;
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    uint32_t x = 0u;
#pragma unroll
                    for (int b = 0; b < 4; ++b)
                        x = __builtin_amdgcn_cvt_pk_u8_f32(__builtin_fmaf(acc[m][4 * b + c], map_scale[m], map_bias[m]), b, x);
                    w[c] = x;
                }
                // (j0 >= i1: a step longer than what is left of the run, whose next units are another workgroup's)
                if (row_w + 32 * m + (lane & 31) < a.rows && j0 < i1) *reinterpret_cast<u32x4*>(code_row[m] + j0) = w;
            }
        }
        if constexpr (EPI == EPI_KEYS) {
            // Elements as above.  Word 8 h + 4 g + c of a 32-item unit (64 bytes) holds the keys of items 8 g + 4 h + c, in its
            // lower half, and 16 more: the lane's eight words lie next to each other.
#pragma unroll
            for (int m = 0; m < WM; ++m) {
                u32x4 w[2];
#pragma unroll
                for (int g = 0; g < 2; ++g)
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        // (-0 and 0 are the same score: the bias is never -0)
                        const auto p = __builtin_amdgcn_cvt_pkrtz(__builtin_fmaf(acc[m][4 * g + c], map_scale[m], map_bias[m]),
                                                                  __builtin_fmaf(acc[m][4 * g + 8 + c], map_scale[m], map_bias[m]));
                        const i16x2_t x = __builtin_bit_cast(i16x2_t, p);
                        const i16x2_t sign = x >> (short)15;
                        w[g][c] = __builtin_bit_cast(uint32_t, x) ^ (__builtin_bit_cast(uint32_t, sign) | 0x80008000u);
                    }
                if (j0 + 32 > i1) {                      // items past the run: below everything
                    int left = i1 - j0 - 4 * half;
                    asm volatile("" : "+v"(left));
#pragma unroll
                    for (int g = 0; g < 2; ++g)
#pragma unroll
                        for (int c = 0; c < 4; ++c)
                            w[g][c] &= (8 * g + c < left ? 0xFFFFu : 0u) | (8 * g + 16 + c < left ? 0xFFFF0000u : 0u);
                }
                if (row_w + 32 * m + (lane & 31) < a.rows && j0 < i1) {
                    u32x4* o = reinterpret_cast<u32x4*>(code_row[m] + 2 * (int64_t)j0);
                    o[0] = w[0];
                    o[1] = w[1];
                }
                // the unit's part of the sample, from the lower half of the lanes; what a unit past the run has is zeros
                if (a.sample_words == 4) kept[m] = u32x4{w[0][0], w[0][2], w[1][0], w[1][2]};
                else if (a.sample_words == 2) {
                    if ((t & 1) == 0) kept[m] = u32x4{w[0][0], w[1][2], 0u, 0u};
                    else kept[m][2] = w[0][0], kept[m][3] = w[1][2];
                } else {
                    if ((t & 3) == 0) kept[m] = u32x4{w[0][0], 0u, 0u, 0u};
                    else if ((t & 3) == 1) kept[m][1] = w[0][0];
                    else if ((t & 3) == 2) kept[m][2] = w[0][0];
                    else kept[m][3] = w[0][0];
                }
                if ((t & sample_mask) == sample_mask || t + 1 == nt)
                    if (half == 0 && row_w + 32 * m + lane < a.rows)
                        *reinterpret_cast<u32x4*>(reinterpret_cast<char*>(a.samples) + (sample_at[m] + (uint32_t)t / (uint32_t)(sample_mask + 1) * 16u)) = kept[m];
            }
        }
    };

    // A step ends when the next one's pieces are there: all but the requests and stores that came after them (the counter
    // holds 63).  Then the barrier: everybody has read this step's stage.
    const bool all_rows = row_w + 32 * WM <= a.rows;
    auto step_ends = [&](bool requested, bool more_stores) {
        auto wait = [&](auto stores) {
            constexpr int kAll = decltype(stores)::value, kSt = kAll < 63 - LR ? kAll : 63 - LR;
            if (NS > 2 && requested) {
                if (all_rows) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LR + kSt) : "memory");
                else asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LR) : "memory");
            } else {
                if (all_rows) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kSt) : "memory");
                else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            }
        };
        if (EPI == EPI_KEYS && more_stores) wait(std::integral_constant<int, kStores + WM>{});
        else wait(std::integral_constant<int, kStores>{});
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    };
#pragma unroll
    for (int t = early_steps<KS, GM>(); t < NS - 1; ++t)
        if (t < nt) request(t, t);
    int stage = 0;
    for (int t = 0; t < nt; ++t) {
        // the stage of step t - 1 takes step t + NS - 1
        const bool more = t + NS - 1 < nt;
        if (more) request(t + NS - 1, stage == 0 ? NS - 1 : stage - 1);
#pragma unroll 1
        for (int s = 0; s < SUB; ++s) {
            multiply(stage, s);
            epilogue(t, s);
        }
        if (t + 1 < nt) step_ends(more, EPI == EPI_KEYS && (t & sample_mask) == sample_mask);
        stage = stage == NS - 1 ? 0 : stage + 1;
    }

    if constexpr (EPI == EPI_KEYS) {                     // the places of the steps that a shorter last run does not have
        for (int g = (nt + sample_mask) / (sample_mask + 1); g < a.sample_groups; ++g)
#pragma unroll
            for (int m = 0; m < WM; ++m)
                if (half == 0 && row_w + 32 * m + lane < a.rows)
                    *reinterpret_cast<u32x4*>(reinterpret_cast<char*>(a.samples) + (sample_at[m] + (uint32_t)g * 16u)) = zero16();
    }
    if constexpr (EPI == EPI_LSE) {
        // lanes l and l + 32 hold the same hidden row; one pair per hidden row, run and wavefront along the rows of M
#pragma unroll
        for (int m = 0; m < WM; ++m) {
            const float om = __shfl_xor(run_max[m], 32), os = __shfl_xor(run_sum[m], 32);
            const float mx = fmaxf(run_max[m], om), ref = mx == -INFINITY ? 0.0f : mx;
            const float sum = run_sum[m] * __expf(run_max[m] - ref) + os * __expf(om - ref);
            const int row = row_w + 32 * m + lane;
            if (lane < 32 && row < a.rows)
                reinterpret_cast<float2*>(a.partial)[(int64_t)row * a.partial_stride + run * GI + gi] = float2{mx, sum};
        }
    }
}

// lse[r] = log of the sum of exponentials behind a row's `n` (maximum, sum) pairs: one wavefront per hidden row
__global__ __launch_bounds__(256) void lse_fold_kernel(const float2* partial, int n, int rows, float* lse) {
    const int lane = threadIdx.x & 63;
    const int row = (int)blockIdx.x * 4 + (int)(threadIdx.x >> 6);
    if (row >= rows) return;
    const float2* p = partial + (int64_t)row * n;
    float mx = -INFINITY;
    for (int i = lane; i < n; i += 64) mx = fmaxf(mx, p[i].x);
    mx = wave_max_f32(mx);
    float sum = 0.0f;
    for (int i = lane; i < n; i += 64) sum += p[i].y * __expf(p[i].x - mx);
    sum = wave_sum(sum);
    if (lane == 0) lse[row] = mx + logf(sum);
}

// The instance for a shape, as an index: hidden rows per panel and steps held.
//   0  d' <= 256, panels of 512 (64 rows per wavefront)     1  ... of 256     2  ... of 128 (32 rows per wavefront)
//   3  d' <= 512, panels of 256 (32 rows per wavefront)
//   4, 5, 6  d' <= 128: as 0, 1, 2 with half the steps (512 rows x 128256, d' = 128: selection 110 -> 101 us, log-
//     probabilities 105 -> 95)
//   7, 8  panels of 64, keys only: d' <= 256, <= 128; steps of twice as many rows of M
struct Shape { int panel, gi; };
constexpr int kNShapes = 9;
constexpr Shape kShapes[kNShapes] = {{512, 1}, {256, 2}, {128, 2}, {256, 1}, {512, 1}, {256, 2}, {128, 2}, {64, 4}, {64, 4}};
inline int shape_of(int chunks, int rows) {
    if (rows <= 64) return chunks > 16 ? 7 : 8;
    if (chunks > 32) return 3;
    const int base = chunks <= 16 ? 4 : 0;
    if (rows <= 128) return base + 2;
    const int pad256 = (rows + 255) / 256, pad512 = (rows + 511) / 512;
    return base + (2 * pad512 == pad256 ? 0 : 1);        // no panel half idle
}
constexpr int kSampleShape = 2, kSampleShapeShort = 6;     // the ones that launch_panel_sample uses (and 3)
template <int EPI, typename F>
hipError_t with_shape(int shape, F&& f) {
    if constexpr (EPI != EPI_SAMPLE && EPI != EPI_KEYS) {
        switch (shape) {
            case 0: return f(std::integral_constant<int, 16>{}, std::integral_constant<int, 2>{}, std::integral_constant<int, 8>{});
            case 1: return f(std::integral_constant<int, 16>{}, std::integral_constant<int, 2>{}, std::integral_constant<int, 4>{});
            case 4: return f(std::integral_constant<int, 8>{}, std::integral_constant<int, 2>{}, std::integral_constant<int, 8>{});
            case 5: return f(std::integral_constant<int, 8>{}, std::integral_constant<int, 2>{}, std::integral_constant<int, 4>{});
            default: break;
        }
    }
    if constexpr (EPI == EPI_KEYS) {
        switch (shape) {
            case 7: return f(std::integral_constant<int, 16>{}, std::integral_constant<int, 1>{}, std::integral_constant<int, 2>{});
            case 8: return f(std::integral_constant<int, 8>{}, std::integral_constant<int, 1>{}, std::integral_constant<int, 2>{});
            default: break;
        }
    }
    if constexpr (EPI != EPI_KEYS) {
        if (shape == 6) return f(std::integral_constant<int, 8>{}, std::integral_constant<int, 1>{}, std::integral_constant<int, 4>{});
    }
    switch (shape) {
        case 2: return f(std::integral_constant<int, 16>{}, std::integral_constant<int, 1>{}, std::integral_constant<int, 4>{});
        case 3: return f(std::integral_constant<int, 32>{}, std::integral_constant<int, 1>{}, std::integral_constant<int, 8>{});
        default: return hipErrorInvalidValue;
    }
}

struct PanelRuns { int64_t items, runs; };   // rows of M per run (a multiple of kRunUnit) and number of runs

// How M is cut into runs.  A run and its panels are dealt to one XCD, a CU holds one workgroup, and a workgroup costs its
// start (the hidden rows' way into registers, about as long as 100 rows of M) and its rows: the number of runs per XCD is
// the one whose rounds of workgroups are cheapest.  One and two panels: a run per CU and one per two CUs.  Three panels:
// ten runs per XCD (a run per 256 / 3 CUs would be eleven on most of them, 33 workgroups on 32 CUs: 700 rows x 151936,
// selection 297 us against 215).  Many panels: at least one run per XCD (20000 rows x 32768, 79 panels: three runs, on
// three of the eight, took 3406 us, sixteen take 1820).
PanelRuns runs_of(int shape, int64_t rows, int64_t n_items) {
    const int64_t panels = (rows + kShapes[shape].panel - 1) / kShapes[shape].panel;
    PanelRuns best{};
    double least = 0.0;
    const bool even = panels <= kCusPerXcd && kCusPerXcd % panels == 0;        // one full round: nothing to weigh
    for (int64_t per_xcd = even ? kCusPerXcd / panels : kCusPerXcd; per_xcd >= 1; --per_xcd) {
        PanelRuns r;
        const int64_t wanted = per_xcd * kXcds;
        r.items = ((n_items + wanted - 1) / wanted + kRunUnit - 1) / kRunUnit * kRunUnit;
        r.runs = (n_items + r.items - 1) / r.items;
        const int64_t rounds = ((r.runs + kXcds - 1) / kXcds * panels + kCusPerXcd - 1) / kCusPerXcd;
        const double cost = (double)rounds * (double)(r.items + 100);
        if (best.items == 0 || cost < least) {
            best = r;
            least = cost;
        }
        if (even) break;
    }
    return best;
}

template <int EPI>
hipError_t launch_epi(const PanelArgs& a0, hipStream_t stream) {
    PanelArgs a = a0;
    // A sample of a few thousand rows of M is over in one or two steps and costs what fetching the hidden rows costs:
    // small panels (512 rows, 8192 of them: 10.8 us on panels of 128 against 14.0 on panels of 512).
    const int shape = EPI != EPI_SAMPLE ? shape_of(a.chunks, a.rows)
                      : a.chunks <= 16 ? kSampleShapeShort : a.chunks <= 32 ? kSampleShape : 3;
    const PanelRuns pr = runs_of(shape, a.rows, a.n_items);
    a.run_items = pr.items;
    a.partial_stride = pr.runs * kShapes[shape].gi;
    const int64_t RT = (a.rows + kShapes[shape].panel - 1) / kShapes[shape].panel;
    const int64_t bx = (pr.runs + kXcds - 1) / kXcds * kXcds * RT;
    if (bx > 0x7fffffffLL) return hipErrorInvalidValue;
    return with_shape<EPI>(shape, [&](auto ks, auto wm, auto gm) {
        constexpr int KS = decltype(ks)::value, WM = decltype(wm)::value, GM = decltype(gm)::value;
        hipLaunchKernelGGL((panel_mfma_kernel<KS, WM, GM, EPI>), dim3((unsigned)bx), dim3(kThreads),
                           (panel_lds_bytes<KS, WM, GM, EPI>()), stream, a);
        return hipGetLastError();
    });
}

template <int EPI>
hipError_t opt_in_epi() {
    for (int shape = 0; shape < kNShapes; ++shape) {
        if (EPI != EPI_KEYS && shape >= 7) continue;
        if (EPI == EPI_KEYS && shape != 2 && shape != 3 && shape < 7) continue;
        if (EPI == EPI_SAMPLE && shape != 3 && shape != kSampleShape && shape != kSampleShapeShort) continue;
        const hipError_t e = with_shape<EPI>(shape, [&](auto ks, auto wm, auto gm) {
            constexpr int KS = decltype(ks)::value, WM = decltype(wm)::value, GM = decltype(gm)::value;
            static_assert(panel_lds_bytes<KS, WM, GM, EPI>() <= 160 * 1024, "one workgroup per CU");
            return hipFuncSetAttribute(reinterpret_cast<const void*>(&panel_mfma_kernel<KS, WM, GM, EPI>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)panel_lds_bytes<KS, WM, GM, EPI>());
        });
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace

hipError_t configure_panel_lds() {
    hipError_t e = opt_in_epi<EPI_SAMPLE>();
    if (e == hipSuccess) e = opt_in_epi<EPI_LOGP>();
    if (e == hipSuccess) e = opt_in_epi<EPI_LSE>();
    if (e == hipSuccess) e = opt_in_epi<EPI_CODES>();
    if (e == hipSuccess) e = opt_in_epi<EPI_KEYS>();
    return e;
}

bool panel_keys_supported(int dt, int chunks, int64_t rows, int64_t n_items) {
    return dt == DT_BF16 && rows >= 1 && rows <= 256 && chunks > (rows <= 64 ? 0 : rows <= 128 ? 16 : 32) && chunks <= (rows <= 64 ? 32 : 64) &&
           n_items < ((int64_t)1 << 22);
}
bool panel_supported(int dt, int chunks, int64_t rows, int64_t n_items) {
    return dt == DT_BF16 && rows > 64 && chunks >= 1 && chunks <= 64 && n_items < ((int64_t)1 << 22);
}

hipError_t launch_panel_sample(const PanelArgs& a, hipStream_t stream) { return launch_epi<EPI_SAMPLE>(a, stream); }
// (16 bytes of a row's sample from four units of a run, a wavefront's in its steps one after the other, or from two units or one)
static int key_sample_groups(int shape, const PanelRuns& pr, int words) {
    const int ti = shape == 3 ? 32 : kShapes[shape].gi < 4 ? 64 : 128, per = 4 / words;
    const int steps = (int)((pr.items + ti - 1) / ti);
    return (steps + per - 1) / per;
}
int64_t panel_key_sample_bytes(int chunks, int64_t rows, int64_t V, int words) {
    const int shape = shape_of(chunks, (int)rows);
    const PanelRuns pr = runs_of(shape, rows, V);
    return pr.runs * kShapes[shape].gi * key_sample_groups(shape, pr, words) * 16;
}
hipError_t launch_panel_keys(const PanelArgs& a0, hipStream_t stream) {
    PanelArgs a = a0;
    const int shape = shape_of(a.chunks, a.rows);
    a.sample_groups = key_sample_groups(shape, runs_of(shape, a.rows, a.n_items), a.sample_words);
    return launch_epi<EPI_KEYS>(a, stream);
}
hipError_t launch_panel_codes(const PanelArgs& a, hipStream_t stream) { return launch_epi<EPI_CODES>(a, stream); }

// (maximum, sum) pairs of a hidden row
static int64_t pairs_of(int chunks, int64_t rows, int64_t V) {
    const int shape = shape_of(chunks, (int)rows);
    return runs_of(shape, rows, V).runs * kShapes[shape].gi;
}

size_t panel_log_softmax_ws_floats(int chunks, int64_t rows, int64_t V) {
    const int64_t pairs = pairs_of(chunks, rows, V);
    return (size_t)rows * (size_t)(2 * pairs + 1);
}

hipError_t launch_panel_log_softmax(const PanelArgs& a0, float* ws, hipStream_t stream) {
    PanelArgs a = a0;
    const int64_t pairs = pairs_of(a.chunks, a.rows, a.n_items);
    float* lse = ws + (size_t)a.rows * (size_t)pairs * 2;
    a.partial = ws;
    hipError_t e = launch_epi<EPI_LSE>(a, stream);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(lse_fold_kernel, dim3((unsigned)((a.rows + 3) / 4)), dim3(256), 0, stream,
                       reinterpret_cast<const float2*>(ws), (int)pairs, a.rows, lse);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    a.row_sub = lse;
    return launch_epi<EPI_LOGP>(a, stream);
}

}  // namespace sv

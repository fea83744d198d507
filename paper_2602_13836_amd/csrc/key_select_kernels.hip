// Candidate-vocabulary selection (Section 3.3, Steps 1 and 2) for the rows of a tree, without the score matrix: the scores leave
// the product as TWO BYTES each, and four launches do it all (the down-projection's among them).
//   keys      the product on the matrix cores, whose epilogue stores the half precision (rounded towards zero) of every score's distance
//             from a score near the row's median, after a power of two per hidden row that brings its largest element to [1, 2), as an
//             unsigned number that orders like the scores, and some keys of every unit of 32 tokens once more on their own, as a sample
//             (panel_mfma_kernels.hip);
//   bracket   keys of every 32 tokens say where the row's k-th lies, give or take; one pass turns the keys above that into bits and lists
//             those in between (2 to 7 per cent, of short rows up to 10) with their place in the bracket, one of 2048;
//   emit      the histogram of a row's lists names the place C that holds the k-th score.  Everything above C is selected; the
//             scores of C itself -- a dozen tokens, as a rule of one and the same key -- are computed once more, by the same matrix
//             instructions in the same order, and ranked by (score, smaller id first); the ids leave in ascending order.
// A row is cut into parts of 32768 tokens that as many workgroups work on as make one round on the chip: one CU pulls no more
// than 25 to 30 bytes a nanosecond, so the 128 to 256 KB of a whole row take it 6 to 10 us.  What the row needs as a whole (the bracket, C,
// the scores of C) every one of its workgroups works out for itself.
// A score is the same float32 as where it goes through memory, bit for bit: up to 256 elements all matrix-core kernels add its
// products in ascending order from zero (v_mfma_f32_16x16x32_bf16 adds its 32 as two 16s), and wider selectors come here from 65
// rows on, where the tiled kernel does too.  The result is exact with respect to those scores whatever they are, because the keys
// are monotone: a sample that misleads costs its row a walk by one workgroup over all of its keys, poor keys (scores that all lie next to each
// other in few places) more tokens at C.
//
// The sample has tokens of every unit.  Neighbours that resemble each other, as the scripts, the numbers or the unused ids of a real vocabulary do, are in it
// as often as they are in the row, and it says more about the row than one of independent tokens.  (A sample of 256 whole units missed where they
// share half of their variance, in one call out of two of 60 rows x 128256, k = 16384; a missed row took 120 us more.)  Only scores that
// depend on the token id modulo 32 mislead it: one such row of 60 x 128256 takes 28 to 34 us more, of 64 x 262144 57, all rows 34 to 45 and 66.
//
// Measured (60 rows x 128256, d' = 256, k = 4096; kernels under a profiler): h' 6.2 us, keys 17.6, bracket 9.2, emit 9.7 to 10.5; the whole
// selection 44.5 -> 40.3 us (as a case with the caller's part 46.5 -> 43.5).  The form it replaces (one byte per score: code_select_kernels.hip) had a sample's
// product and a map in front of the codes (6 and 4 us, each mostly a launch) and read the codes with one workgroup per row (17).  Two thirds of
// bracket and emit are their start and six round trips to memory.  Not used: this pass by one workgroup per row, 22.7 us
// (9.5 of them for the keys); a sample gathered from the keys, 16 bytes per thread from lines of their own (as many bytes as the part: bracket
// 11.7); sampled words stored one by one as they are made (keys 18.6 to 18.9).
#include "sv_device.h"
#include "sv_launch.h"

#include <math.h>

#include <type_traits>

#include "tile_epilogue.h"

namespace sv {

namespace {

constexpr int kThreads = 1024, kWaves = kThreads / 64;
constexpr int kBinBits = 11, kBins = 1 << kBinBits;      // two per thread
constexpr int kBinShift = 16 - kBinBits;                 // keys per bin of the sample's histogram, as a power of two
constexpr int64_t kMaxVocab = 262144 + 131072;           // a bit per token in LDS (48 KB)
constexpr int64_t kMinVocab = 16384;          // (shorter rows: row_select_kernel)
constexpr int kSampleLoads = (int)(kMaxVocab / 32 / (4 * kThreads));     // of 16 bytes per thread
static_assert(kBins == 2 * kThreads && kMaxVocab < ((int64_t)1 << (32 - kBinBits)), "an entry is an id and a bin");

constexpr int kPart = 32 * kThreads;                     // tokens of a part: a unit per thread
constexpr uint32_t kSegment = kPart / 4;                 // entries that a part's list has room for (2 to 5 % of its tokens as a rule)
__host__ __device__ inline int parts_of(int64_t V) { return (int)((V + kPart - 1) / kPart); }

struct KeyLayout {
    int64_t stride;          // bytes between rows of keys: an odd multiple of 256, off the memory channels' period
    // words of a unit (two keys each) that are sampled: 4096 to 8192 keys of a row, of the largest 24576 (twice as many up to three halves of each
    // range: the bracket's histogram and the product's stores take what shorter lists save, 40 rows x 66000 30.0 us against 29.4)
    int sample_words;
    // offsets in bytes from the scratch base (multiples of 8; the keys' of 256, the sample's of 16)
    size_t keys, parts, bits, list, ties, sample, total;
};
inline KeyLayout key_layout(int64_t V, int64_t rows) {
    KeyLayout L;
    const int64_t parts = parts_of(V), units = (V + 31) / 32;
    L.stride = (units * 64 + 255) / 256 * 256 | 256;
    L.sample_words = V <= 32768 ? 4 : V <= 65536 ? 2 : 1;
    size_t o = 0;
    L.keys = o;   o += (size_t)rows * (size_t)L.stride;
    L.parts = o;  o += (size_t)rows * (size_t)parts * 8;                         // {scores above the bracket, scores in it}
    L.bits = o;   o += (size_t)rows * (size_t)parts * kThreads * 4;
    L.list = o;   o += (size_t)rows * (size_t)parts * kSegment * 4;
    o = (o + 15) & ~(size_t)15;
    L.sample = o;                                        // (has been read when there are ties)
    L.ties = o;   o += (size_t)rows * (size_t)V * 8;     // (the sample takes 3 of 8 at most)
    L.total = o;
    return L;
}

// the list's histogram, the ties' keys from the end on downwards; later up to 64 rows of W_vocab and their keys
constexpr uint32_t kFew = 64;
__host__ __device__ constexpr uint32_t few_bytes(int chunks) { return kFew * ((uint32_t)(chunks + 1) * 16u + 8u); }
__host__ __device__ constexpr uint32_t stage_bytes(int chunks) { return few_bytes(chunks) > 34 * 1024 ? few_bytes(chunks) : 34 * 1024; }
constexpr uint32_t kTiesInLds = (34 * 1024 - 4 * kBins) / 8;

struct ResolveSmem {
    uint32_t w[kWaves], w2[kWaves];
    uint32_t out[4];
    uint32_t n_ties;
    u32x4 x[64];                                         // the hidden row
};
// dynamic LDS: a bit per token of the part, or of the row (ids that are selected) | the stage, whose end takes the ties' keys
__host__ __device__ inline size_t sel_bytes(int64_t V) {
    return (size_t)parts_of(V) * kThreads * 4;
}

constexpr uint32_t kDense = 576;                         // selected ids of 2048

typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

// a bit per key of a unit that is larger than `than` (that key in both halves): word 8 h + 4 g + c holds the keys of items
// 8 g + 4 h + c and 16 more
__device__ __forceinline__ uint32_t larger_than(const u32x4 (&q)[4], uint32_t than) {
    uint32_t m = 0u;
#pragma unroll
    for (int w = 0; w < 16; ++w) {
        const uint32_t x = q[w >> 2][w & 3];
        const u16x2 d = __builtin_elementwise_sub_sat(__builtin_bit_cast(u16x2, x), __builtin_bit_cast(u16x2, than));
        const u16x2 f = __builtin_elementwise_min(d, u16x2{1, 1});
        m |= __builtin_bit_cast(uint32_t, f) << (8 * ((w >> 2) & 1) + 4 * (w >> 3) + (w & 3));
    }
    return m;
}
// byte of an item's key in its unit
__device__ __forceinline__ uint32_t key_at_byte(uint32_t item) {
    return ((item & 4u) << 3) | ((item & 8u) << 1) | ((item & 3u) << 2) | ((item >> 3) & 2u);
}

// f(bin, entries above it, its entries) for the thread's two bins of a histogram.  Every thread of the workgroup must call.
template <typename F>
__device__ __forceinline__ void with_bins(const uint32_t* hist, uint32_t* s_w, F&& f) {
    const int tid = threadIdx.x;
    const uint32_t c0 = hist[2 * tid], c1 = hist[2 * tid + 1];
    const uint32_t above1 = block_suffix_exclusive<kWaves>(c0 + c1, s_w), above0 = above1 + c1;
    f(2u * tid + 1u, above1, c1);
    f(2u * tid, above0, c0);
}
__device__ __forceinline__ uint32_t same(uint32_t x) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)x); }     // (in a scalar register)
__device__ __forceinline__ uint32_t key_of(const unsigned char* key_row, uint32_t id) {
    return *reinterpret_cast<const uint16_t*>(key_row + (size_t)(id >> 5) * 64 + key_at_byte(id & 31u));
}

// A workgroup has some parts of a row: the bracket, from a sample of the whole row (all of the row's workgroups make the same one), and what
// of its parts lies above it (a bit each) and in it (id and bin of the bracket, in a list per part).
__global__ __launch_bounds__(kThreads) void key_bracket_kernel(const unsigned char* keys, int64_t stride, int64_t V, int parts, int per,
                                                               const u32x4* sample, int sample_units, uint32_t rank_hi, uint32_t rank_lo,
                                                               uint2* part_counts, uint32_t* bits, uint32_t* list) {
    __shared__ uint32_t s_samp[kBins];
    __shared__ uint32_t s_list[kSegment];
    __shared__ uint32_t s_w[kWaves], s_w2[kWaves];
    __shared__ uint32_t s_out[2];
    const int tid = threadIdx.x, lane = tid & 63;
    const int units = (int)((V + 31) / 32);
    const unsigned char* const key_row = keys + (int64_t)blockIdx.y * stride;
    const u32x4* const row = reinterpret_cast<const u32x4*>(key_row);
    // the sample: keys of every unit, so that tokens which lie together and have something in common are in it as often as they are there
    u32x4 samp[kSampleLoads];
#pragma unroll
    for (int i = 0; i < kSampleLoads; ++i)
        samp[i] = i * kThreads + tid < sample_units ? sample[(int64_t)blockIdx.y * sample_units + i * kThreads + tid] : zero16();
    int part = (int)blockIdx.x * per;
    const int end = min(part + per, parts);
    u32x4 q[4];
    auto fetch = [&]() {
        const int u = min(part * kThreads + tid, units - 1);
#pragma unroll
        for (int i = 0; i < 4; ++i) q[i] = row[4 * u + i];
    };
    fetch();
    s_samp[tid] = s_samp[tid + kThreads] = 0u;
    if (tid == 0) {
        s_out[0] = 0xFFFFu;
        s_out[1] = 1u;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kSampleLoads; ++i)
#pragma unroll
        for (int w = 0; w < 4; ++w)
            if (samp[i][w] != 0u) {                           // (zeros: nothing there)
                atomicAdd(&s_samp[(samp[i][w] & 0xFFFFu) >> kBinShift], 1u);
                atomicAdd(&s_samp[samp[i][w] >> (16 + kBinShift)], 1u);
            }
    __syncthreads();
    with_bins(s_samp, s_w, [&](uint32_t bin, uint32_t above, uint32_t c) {
        if (above < rank_hi && rank_hi <= above + c) s_out[0] = (bin << kBinShift) | ((1u << kBinShift) - 1u);
        if (above < rank_lo && rank_lo <= above + c && bin > 0u) s_out[1] = bin << kBinShift;
    });
    __syncthreads();
    const uint32_t hi_key = same(s_out[0]), lo_key = same(s_out[1]);
    const int shift = max(0, 32 - __builtin_clz((hi_key - lo_key) | 1u) - kBinBits);
    for (; part < end; ++part) {
        const int64_t slot = (int64_t)blockIdx.y * parts + part;
        const int u = part * kThreads + tid;
        if (u >= units) q[0] = q[1] = q[2] = q[3] = zero16();
        const uint32_t above = larger_than(q, hi_key * 0x10001u);
        uint32_t in = larger_than(q, (lo_key - 1u) * 0x10001u) ^ above;
        bits[slot * kThreads + tid] = above;
        const uint32_t c = (uint32_t)__popc(in);
        uint32_t at = block_prefix_exclusive<kWaves>(c, s_w);
        const uint32_t full = wave_sum_u32((uint32_t)__popc(above));
        if (lane == 0) s_w2[tid >> 6] = full;
        const uint32_t id0 = 32u * (uint32_t)u;
        for (; in; in &= in - 1u) {
            if (at < kSegment) s_list[at] = id0 + (uint32_t)__builtin_ctz(in);
            ++at;
        }
        __syncthreads();
        uint32_t n = 0u, n_above = 0u;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            n += s_w[w];
            n_above += s_w2[w];
        }
        if (tid == 0) part_counts[slot] = uint2{n_above, n};
        uint32_t* const mine = list + slot * (int64_t)kSegment;
        for (uint32_t i = tid; i < min(n, kSegment); i += kThreads) {
            const uint32_t id = s_list[i];
            mine[i] = (id << kBinBits) | ((key_of(key_row, id) - lo_key) >> shift);
        }
        if (part + 1 == end) break;
        ++part;
        fetch();
        --part;
        __syncthreads();                                      // the list and the sums have been read
    }
}

// A workgroup has some parts of a row: which code C holds the row's k-th score, which of the scores of C are selected, and the ids of its parts.
// Where the bracket missed, a list overflowed or C has more scores than LDS holds, the first of the row's workgroups does it all from the keys.
__global__ __launch_bounds__(kThreads) void key_emit_kernel(const unsigned char* keys, int64_t stride, int64_t V, int64_t k, const char* hp, const char* Wv,
                                                            int chunks, int parts, int per, const uint2* part_counts, const uint32_t* bits,
                                                            const uint32_t* list, uint64_t* ties, int32_t* idx_out) {
    extern __shared__ __attribute__((aligned(16))) uint32_t s_sel[];
    unsigned char* const s_stage = reinterpret_cast<unsigned char*>(s_sel) + sel_bytes(V);
    uint32_t* const s_hist = reinterpret_cast<uint32_t*>(s_stage);
    uint64_t* const s_ties = reinterpret_cast<uint64_t*>(s_stage + stage_bytes(chunks)) - kTiesInLds;
    __shared__ ResolveSmem sm;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int part = (int)blockIdx.x * per;                  // the first of its own
    const int64_t r = blockIdx.y;
    const int units = (int)((V + 31) / 32);
    const unsigned char* const key_row = keys + r * stride;
    const u32x4* const row = reinterpret_cast<const u32x4*>(key_row);
    uint64_t* const ties_mem = ties + r * V;
    const uint32_t* const lists = list + r * parts * (int64_t)kSegment;
    // (a hidden row of zeros -- a padding row of the batch -- has nothing but equal scores)
    bool zero_row = true;
    const char* const x_row = hp + r * chunks * 16;
    u32x4 xv = zero16();
    if (lane < chunks) xv = reinterpret_cast<const u32x4*>(x_row)[lane];
    const uint2 counts = lane < parts ? part_counts[r * parts + lane] : uint2{0u, 0u};
    uint32_t entry[4];                                        // the first of the first four parts, whether they are there or not
#pragma unroll
    for (int i = 0; i < 4; ++i) entry[i] = lists[(int64_t)min(i, parts - 1) * kSegment + tid];
    const uint32_t* const row_bits = bits + r * parts * (int64_t)kThreads;
    const uint32_t part_bits = row_bits[part * kThreads + tid];
    s_hist[tid] = s_hist[tid + kThreads] = 0u;
    for (int j = 0; j < per; ++j) s_sel[j * kThreads + tid] = 0u;
    if (tid == 0) sm.n_ties = 0u;
    if (lane < chunks) {
        zero_row = ((xv[0] | xv[1] | xv[2] | xv[3]) & 0x7FFF7FFFu) == 0u;
        if (wave == 0) sm.x[lane] = xv;
    }
    zero_row = __builtin_amdgcn_ballot_w64(!zero_row) == 0ull;
    int32_t* const out = idx_out + r * k;
    if (zero_row) {                                           // uniform
        for (int64_t j = (int64_t)blockIdx.x * kThreads + tid; j < k; j += (int64_t)gridDim.x * kThreads) out[j] = (int32_t)j;
        return;
    }
    const uint32_t wanted = (uint32_t)k;
    const uint32_t full = wave_sum_u32(counts.x), n_list = wave_sum_u32(counts.y), full_before = wave_sum_u32(lane < part ? counts.x : 0u);
    bool hard = wanted <= full || wanted > full + n_list || wave_max_u32(counts.y) > kSegment;
    // f(entry) for the entries of all parts
    auto for_each_entry = [&](auto&& f) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (i < parts && (uint32_t)tid < (uint32_t)__builtin_amdgcn_readlane((int)counts.y, i)) f(entry[i]);
        for (int p = 0; p < parts; ++p) {
            const uint32_t np = (uint32_t)__builtin_amdgcn_readlane((int)counts.y, p);
            for (uint32_t j = (uint32_t)tid + (p < 4 ? kThreads : 0); j < np; j += kThreads) f(lists[(int64_t)p * kSegment + j]);
        }
    };
    // the bin (the key, after a walk) of the k-th score: its number, the scores above it, its scores
    auto located = [&](uint32_t rank, uint32_t base) {
        with_bins(s_hist, sm.w, [&](uint32_t bin, uint32_t above, uint32_t c) {
            if (base + above < rank && rank <= base + above + c) {
                sm.out[0] = bin;
                sm.out[1] = base + above;
                sm.out[2] = c;
            }
        });
        __syncthreads();
    };
    __syncthreads();
    if (__builtin_expect(!hard, 1)) {                         // uniform
        for_each_entry([&](uint32_t e) { atomicAdd(&s_hist[e & (kBins - 1u)], 1u); });
        __syncthreads();
        located(wanted, full);
        const uint32_t n = same(sm.out[2]);
        hard = n > kTiesInLds && n != wanted - same(sm.out[1]);
    }
    if (hard && part > 0) return;
    // the workgroup's units: its part's, or the whole row's.  Wavefront w has `rounds` rounds of 64 units, lane l the units
    // (w rounds + j) 64 + l from the first on: ids ascend with (wavefront, round, lane, bit)
    const int first = hard ? 0 : part * kThreads;
    const int rounds = hard ? parts : min(per, parts - part);
    const int u0 = wave * rounds * 64 + lane;                 // (counted from `first`)
    auto for_each_unit = [&](auto&& f) {                      // (hard) f(unit, keys) with all lanes; units past the last: keys of 0
        for (int j = 0; j < rounds; ++j) {
            const int u = u0 + 64 * j;
            u32x4 q[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) q[i] = row[4 * min(u, units - 1) + i];
            if (u >= units) q[0] = q[1] = q[2] = q[3] = zero16();
            f(u, q);
        }
    };
    if (__builtin_expect(hard, 0)) {
        __syncthreads();
        s_hist[tid] = s_hist[tid + kThreads] = 0u;
        __syncthreads();
        // all keys by their upper bits, then those of the bin that holds the k-th by their lower ones
        uint32_t top = 0u, base = 0u;
        for (int level = 0; level < 2; ++level) {
            for_each_unit([&](int u, const u32x4 (&q)[4]) {
                const uint32_t valid = u < units ? (uint32_t)min((int64_t)32, V - 32 * (int64_t)u) : 0u;
                uint32_t bin = kBins, run = 0u;               // (equal ones in a row together)
#pragma unroll
                for (int i = 0; i < 32; ++i) {                // word i % 16 = 8 h + 4 g + c, its lower half or its upper
                    const int w = i & 15;
                    const uint32_t x = i < 16 ? q[w >> 2][w & 3] & 0xFFFFu : q[w >> 2][w & 3] >> 16;
                    const uint32_t b = level == 0 ? x >> kBinShift : x & ((1u << kBinShift) - 1u);
                    if ((uint32_t)(8 * ((w >> 2) & 1) + 4 * (w >> 3) + (w & 3) + (i & 16)) >= valid || (level == 1 && (x >> kBinShift) != top)) continue;
                    if (b != bin) {
                        if (run) atomicAdd(&s_hist[bin], run);
                        bin = b;
                        run = 0u;
                    }
                    ++run;
                }
                if (run) atomicAdd(&s_hist[bin], run);
            });
            __syncthreads();
            located(wanted, base);
            if (level == 0) {
                top = same(sm.out[0]);
                base = same(sm.out[1]);
                s_hist[tid] = s_hist[tid + kThreads] = 0u;
                __syncthreads();
            } else if (tid == 0) {
                sm.out[0] |= top << kBinShift;
            }
        }
        __syncthreads();
    }
    const uint32_t C = same(sm.out[0]), above_C = same(sm.out[1]), n = same(sm.out[2]);
    const uint32_t need = wanted - above_C;                   // of the n scores of C: 1 <= need <= n
    const bool whole = need == n, in_lds = n <= kTiesInLds;

    // Ids above C become bits, where they are this workgroup's; those of C too, if all are selected, or they go to the ties
    // (an inverted id each, with the score on top as soon as it is known)
    uint32_t before = 0u;                                     // selected ids of the parts before, without those above the bracket
    auto select_id = [&](uint32_t id) {
        const int u = (int)(id >> 5) - first;
        if (u < 0) ++before;
        else if (u < rounds * kThreads) atomicOr(&s_sel[u], 1u << (id & 31u));
    };
    auto put_tie = [&](uint32_t at, uint32_t id) {
        if (in_lds) s_ties[kTiesInLds - 1u - at] = (uint64_t)(~id);
        if (!in_lds) ties_mem[at] = (uint64_t)(~id);
    };
    if (__builtin_expect(hard, 0)) {
        for_each_unit([&](int u, const u32x4 (&q)[4]) {
            const uint32_t more = larger_than(q, C * 0x10001u);
            uint32_t equal = C > 0u ? larger_than(q, (C - 1u) * 0x10001u) ^ more : ~more;
            if (u >= units) return;
            const int64_t left = V - 32 * (int64_t)u;
            if (left < 32) equal &= (1u << left) - 1u;        // (keys of 0 follow)
            s_sel[u] = more | (whole ? equal : 0u);
            if (!whole && equal)
                for (uint32_t at = atomicAdd(&sm.n_ties, (uint32_t)__popc(equal)); equal; equal &= equal - 1u)
                    put_tie(at++, 32u * (uint32_t)u + (uint32_t)__builtin_ctz(equal));
        });
    } else {
        for_each_entry([&](uint32_t e) {
            const uint32_t c = e & (kBins - 1u), id = e >> kBinBits;
            if (c > C || (whole && c == C)) select_id(id);
            else if (c == C) put_tie(atomicAdd(&sm.n_ties, 1u), id);
        });
    }
    if (!whole) {                                             // uniform: the `need` largest scores of C are wanted
        auto choose = [&](auto lds) {
            constexpr bool LDS = decltype(lds)::value;        // the ties are there, and not in memory
            auto tie_at = [&](uint32_t i) -> uint64_t {
                if constexpr (LDS) return s_ties[kTiesInLds - 1u - i];
                else return ties_mem[i];
            };
            __threadfence_block();
            __syncthreads();
            // Their scores, 32 ids at a time as rows of the first operand; every column of the second is the hidden row
            auto multiply = [&](uint32_t at, auto&& unit) {       // unit(c): unit c of the lane's row
                f32x16_t acc;
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[e] = 0.f;
                constexpr int kAhead = 8;
#pragma unroll 1
                for (int k0 = 0; k0 < chunks; k0 += 2 * kAhead) {
                    u32x4 a[kAhead], b[kAhead];
#pragma unroll
                    for (int i = 0; i < kAhead; ++i) {
                        const int c = k0 + 2 * i + (lane >> 5);
                        a[i] = unit(min(c, chunks - 1));
                        b[i] = c < chunks ? sm.x[min(c, chunks - 1)] : zero16();
                    }
#pragma unroll
                    for (int i = 0; i < kAhead; ++i) {
                        const int c = k0 + 2 * i + (lane >> 5);
                        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, c < chunks ? a[i] : zero16()),
                                                                      __builtin_bit_cast(bf16x8_t, b[i]), acc, 0, 0, 0);
                    }
                }
                // element e of lanes l < 32 and l + 32: ids 8 (e / 4) + e % 4 and 4 more (every l the same)
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const uint32_t i = at + (uint32_t)(8 * (e >> 2) + 4 * (lane >> 5) + (e & 3));
                    if ((lane & 31) == e && i < n) {
                        if constexpr (LDS) reinterpret_cast<uint32_t*>(s_ties)[2u * (kTiesInLds - 1u - i) + 1u] = f32_to_ord(acc[e]);
                        else reinterpret_cast<uint32_t*>(ties_mem)[2 * (int64_t)i + 1] = f32_to_ord(acc[e]);
                    }
                }
            };
            if (LDS && n <= kFew) {
                // The usual handful: all threads bring the rows of W_vocab, in one round trip, and two wavefronts multiply.
                // Ranked by counting (keys are unique: they end in the id)
                u32x4* const s_rows = reinterpret_cast<u32x4*>(s_stage);
                for (uint32_t i = (uint32_t)tid; i < n * 32u; i += kThreads) {
                    const u32x4* w_row = reinterpret_cast<const u32x4*>(Wv + (int64_t)(~(uint32_t)tie_at(i >> 5)) * chunks * 16);
                    for (int c = (int)(i & 31u); c < chunks; c += 32) s_rows[(i >> 5) * (uint32_t)(chunks + 1) + c] = w_row[c];
                }
                __syncthreads();
                const uint32_t at = (uint32_t)wave * 32u;
                if (at < n) {
                    const u32x4* mine = s_rows + min(at + (uint32_t)(lane & 31), n - 1u) * (uint32_t)(chunks + 1);
                    multiply(at, [&](int c) { return mine[c]; });
                }
                __syncthreads();
                if (wave == 0) {
                    const uint64_t mine = (uint32_t)lane < n ? tie_at((uint32_t)lane) : 0ull;
                    uint32_t larger = 0u;
                    for (uint32_t i = 0; i < n; ++i) larger += readlane_u64(mine, (int)i) > mine;
                    if ((uint32_t)lane < n && larger < need) select_id(~(uint32_t)mine);
                }
                return;
            }
            for (uint32_t at = (uint32_t)wave * 32u; at < n; at += kWaves * 32u) {
                const uint32_t inv = (uint32_t)tie_at(min(at + (uint32_t)(lane & 31), n - 1u));
                const u32x4* w_row = reinterpret_cast<const u32x4*>(Wv + (int64_t)(~inv) * chunks * 16);
                multiply(at, [&](int c) { return w_row[c]; });
            }
            __threadfence_block();
            __syncthreads();
            // digit by digit from the top (the digits that all keys share take a pass like the others)
            uint64_t T = 0ull;                                // key of the last selected one
            uint32_t remain = need;
            int decided = 0;
            while (decided < 64) {
                const int w = 64 - decided < kBinBits ? 64 - decided : kBinBits, down = 64 - decided - w;
                __syncthreads();
                s_hist[tid] = s_hist[tid + kThreads] = 0u;
                __syncthreads();
                for (uint32_t i = tid; i < n; i += kThreads) {
                    const uint64_t x = tie_at(i);
                    if (decided == 0 || (x >> (64 - decided)) == (T >> (64 - decided)))
                        atomicAdd(&s_hist[(uint32_t)(x >> down) & ((1u << w) - 1u)], 1u);
                }
                __syncthreads();
                located(remain, 0u);
                T |= (uint64_t)sm.out[0] << down;
                remain -= sm.out[1];
                decided += w;
                if (remain == sm.out[2]) break;               // every key with these digits is selected
            }
            for (uint32_t i = tid; i < n; i += kThreads) {
                const uint64_t x = tie_at(i);
                if (x >= T) select_id(~(uint32_t)x);
            }
        };
        if (in_lds) choose(std::true_type{});
        else choose(std::false_type{});
    }
    __syncthreads();

    // The ids of the set bits, ascending.  A lane stores those of its own unit one after the other, each store to as many lines as
    // there are lanes; where they are many (from about a quarter of the tokens on) all lanes share two units at a time instead, and the stores
    // are whole lines: half of 128256 tokens wanted, mean of 9 to 512 rows, 108 -> 72 us; half of 262144 194 -> 121; an eighth of
    // them that way 87 -> 110.
    if (!hard) {
        s_sel[tid] |= part_bits;                              // (its own words)
        for (int j = 1; j < rounds; ++j) s_sel[j * kThreads + tid] |= row_bits[(part + j) * kThreads + tid];
        if (rounds > 1) __syncthreads();
    }
    uint32_t total = 0u;
    for (int j = 0; j < rounds; ++j) {
        const int u = u0 + 64 * j;
        total += first + u < units ? (uint32_t)__popc(s_sel[u]) : 0u;
    }
    total = wave_sum_u32(total);
    before = wave_sum_u32(before);
    if (lane == 0) {
        sm.w2[wave] = total;
        sm.w[wave] = before;
    }
    __syncthreads();
    uint32_t base = 0u, from = hard ? 0u : full_before, all = 0u;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        base += w < wave ? sm.w2[w] : 0u;
        from += sm.w[w];
        all += sm.w2[w];
    }
    if (from + all > (uint32_t)k) return;                     // never: k bits are set in all
    base += from;
    for (int j = 0; j < rounds; ++j) {
        const int u = u0 + 64 * j;
        uint32_t bits = first + u < units ? s_sel[u] : 0u;
        const uint32_t c = (uint32_t)__popc(bits);
        const uint32_t incl = wave_prefix_inclusive_u32(c), here = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
        if (here >= kDense) {                                 // uniform: a lane per token, two units at a time
            const uint32_t id = 32u * (uint32_t)(first + u - lane) + (uint32_t)lane;
            for (int i = 0; i < 64; i += 2) {
                const uint32_t b0 = (uint32_t)__builtin_amdgcn_readlane((int)bits, i), b1 = (uint32_t)__builtin_amdgcn_readlane((int)bits, i + 1);
                const uint32_t at = __builtin_amdgcn_mbcnt_hi(b1, __builtin_amdgcn_mbcnt_lo(b0, base));
                if (((lane < 32 ? b0 : b1) >> (lane & 31)) & 1u)
                    *reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(out) + at * 4u) = id + 32u * (uint32_t)i;
                base += (uint32_t)(__popc(b0) + __popc(b1));
            }
            continue;
        }
        uint32_t at = (base + incl - c) * 4u;
        base += here;
        const uint32_t id0 = 32u * (uint32_t)(first + u);
        while (bits) {
            *reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(out) + at) = id0 + (uint32_t)__builtin_ctz(bits);
            at += 4u;
            bits &= bits - 1u;
        }
    }
}

}  // namespace

// From how many rows on, and to how many.  us, the alternative / keys (runs differ by 2 to 4 %):
//   few rows    the alternative is the scores in memory.  From 9 rows on theirs is the longer chain: d' = 256, k = V / 32: 9 rows x 33000 to 262144
//               29.1 to 51.5 / 27.3 to 48.2, 16 rows 30.8 to 54.3 / 27.3 to 49.4; only many ids of few rows, which there leave by more
//               workgroups, tie or lose (k = V / 2: 16 rows x 128256 41.1 / 42 and more; V / 4: 16 x 66000 36.1 / 34.0, 9 x 128256 39.0 / 40.9, 9 x
//               262144 54.5 / 56.7; 24 rows x 128256, V / 2 45.4 / 44.2).  Up to 8 rows: d' = 128 and 64, k up to V / 8: 2 rows x 128256 31.5 /
//               28.5, x 16500 24.6 / 21.8, k = V / 8 32.1 / 31.1; x 262144 V / 32 40.4 / 36.7, V / 8 40.9 / 42.2 (8 rows 49.6 / 43.4); d' = 256
//               (where the product on panels, made for many rows, loses 3 us): 8 rows 31.3 / 33.1.
//   many rows   the alternative is a byte per score, half of what keys write and read.  d' = 256: as long as every workgroup of bracket and emit
//               has one part, 65 x 80000 39.6 / 37.0, 128 x 50000 36.0 / 36.1; two parts 100 x 66000 39.0 / 42.8, 65 x 100000 42.2 / 43.4; more
//               than 128 rows (panels of 256) tie: 160 x 16385 35.6 / 35.0, 200 x 17000 37.7 / 38.3; so does all of d' = 128: 128 x 17000
//               26.7 / 26.8, 65 x 50000 29.9 / 30.1.  d' = 512: 65 x 80000 61.1 / 51.0, 128 x 128256 76.6 / 75, 65 x 262144 110 / 114; 160 x
//               50000 61.7 / 60.6, 256 x 33000 57.8 / 57.1; d' = 264, 160 x 80000 60.3 / 62.9.
bool key_select_supported(int dt, int chunks, int64_t rows, int64_t V, int64_t k) {
    if (!panel_keys_supported(dt, chunks, rows, V) || V < kMinVocab || V > kMaxVocab || row_select_preferred(chunks, rows, V)) return false;
    if (rows > 64) return chunks > 32 ? rows * V <= (rows <= 128 ? 16800000 : 10000000) : rows * parts_of(V) <= 256;
    if (rows > 8) return chunks <= 16 || rows >= 24 || (4 * k <= V && (V <= 98304 || 8 * k <= V));
    return rows > 1 && chunks <= 16 && 8 * k <= V && (rows > 4 || V <= 196608 || 16 * k <= V);
}

// (more than 64 KB of LDS: an opt-in)
hipError_t configure_key_select_lds() {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(&key_emit_kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)(sel_bytes(kMaxVocab) + stage_bytes(64)));
}

size_t key_select_scratch_bytes(int64_t rows, int64_t V) { return key_layout(V, rows).total; }

hipError_t launch_key_select(const CodeSelectArgs& a, hipStream_t stream) {
    const KeyLayout L = key_layout(a.V, a.rows);
    PanelArgs p{};
    p.x = a.hp;
    p.x_row_bytes = (int64_t)a.chunks * 16;
    p.M = a.Wv;
    p.m_row_bytes = (int64_t)a.chunks * 16;
    p.n_items = a.V;
    p.chunks = a.chunks;
    p.rows = a.rows;
    p.codes = reinterpret_cast<uint8_t*>(a.scratch + L.keys);
    p.code_stride = L.stride;
    p.samples = reinterpret_cast<uint32_t*>(a.scratch + L.sample);
    p.sample_stride = panel_key_sample_bytes(a.chunks, a.rows, a.V, L.sample_words);
    p.sample_words = L.sample_words;
    p.upper_wanted = 8 * a.k <= 3 * a.V;
    if (p.sample_stride > kSampleLoads * kThreads * 16 || p.sample_stride > 8 * a.V) return hipErrorInvalidValue;     // (never)
    hipError_t e = launch_panel_keys(p, stream);
    if (e != hipSuccess) return e;
    // The number of sampled tokens among the row's k best is hypergeometric with mean m k / V if the scores have nothing to do with the tokens'
    // places, and varies less if neighbours resemble each other: its rank range, 6 standard deviations and 8 more on either side
    const double m = (double)((a.V + 31) / 32 * 2 * L.sample_words), share = (double)a.k / (double)a.V, mean = m * share;
    const double reach = 6.0 * sqrt(m * share * (1.0 - share)) + 8.0;
    const double rank_hi = fmax(floor(mean - reach), 0.0), rank_lo = fmin(ceil(mean + reach), m + 1.0);     // (0, m + 1: none)
    // as many workgroups per row as make one round on the chip
    DeviceInfo di;
    e = device_info(&di);
    if (e != hipSuccess) return e;
    const int parts = parts_of(a.V), most = di.cus / a.rows > 1 ? di.cus / a.rows : 1;
    const int per = (parts + most - 1) / most;
    const dim3 grid((unsigned)((parts + per - 1) / per), (unsigned)a.rows);
    const unsigned char* keys = reinterpret_cast<const unsigned char*>(p.codes);
    uint2* counts = reinterpret_cast<uint2*>(a.scratch + L.parts);
    uint32_t* bits = reinterpret_cast<uint32_t*>(a.scratch + L.bits);
    uint32_t* list = reinterpret_cast<uint32_t*>(a.scratch + L.list);
    hipLaunchKernelGGL(key_bracket_kernel, grid, dim3(kThreads), 0, stream, keys, L.stride, a.V, parts, per,
                       reinterpret_cast<const u32x4*>(p.samples), (int)(p.sample_stride / 16), (uint32_t)rank_hi, (uint32_t)rank_lo, counts, bits, list);
    hipLaunchKernelGGL(key_emit_kernel, grid, dim3(kThreads), sel_bytes(a.V) + stage_bytes(a.chunks), stream, keys, L.stride, a.V, a.k, a.hp, a.Wv,
                       a.chunks, parts, per, counts, bits, list, reinterpret_cast<uint64_t*>(a.scratch + L.ties), a.idx_out);
    return hipGetLastError();
}

}  // namespace sv

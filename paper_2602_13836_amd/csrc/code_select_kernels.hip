// Candidate-vocabulary selection (Section 3.3, Steps 1 and 2) for a batch of hidden rows, without the score matrix: the
// scores leave the product as ONE BYTE each.
//
// With hundreds of hidden rows the scores s [rows x V] are hundreds of megabytes.  Here, per hidden row:
//   sample    the scores of kSample evenly spaced tokens (a small matrix product);
//   map       the sample's order statistics say where the row's k-th largest score lies, give or take: a value lo below
//             it and hi above it become a map  code(s) = round(scale s + bias), saturated to 0 .. 255, with lo at 128
//             and hi at 254;
//   codes     the full product on the matrix cores, whose epilogue stores the codes (panel_mfma_kernels.hip);
//   resolve   one workgroup per row, the row's codes in registers: their histogram names the code C that holds the k-th
//             score.  Everything above C is selected; the scores of code C itself -- a few dozen tokens -- are computed
//             once more, by the same matrix instructions in the same order, and ranked by (score, smaller id first).
// A score is the same float32 as where it goes through memory, bit for bit: up to 256 elements all matrix-core kernels add its products in
// ascending order from zero (v_mfma_f32_16x16x32_bf16 adds its 32 as two 16s), and wider selectors come here from 65 rows on, where the
// tiled kernel does too.
// The result is exact with respect to those scores whatever the map is, because the map is monotone: a poor one only
// leaves more tokens in code C (a map that misses the k-th score altogether, as many as there are below lo or above hi).
// As many keys as fit stay in LDS; more go to memory.  All of it lies where the scores would (12 bytes per score with the lists that
// their selection keeps), in 11 of them.
//
// Measured (512 rows x 151936, d' = 256, k = 8192; kernels under a profiler): h' 11 us, sample 8, map 5, codes 50, resolve 37; the
// whole selection 133 -> 103 us.  The form it replaces kept a bit per score (above hi) and a list of (key, id) of the scores
// between lo and hi per row and run -- 40 us of comparisons, LDS and scattered stores on top of the product --, needed a
// sample twice as large for its lists to be short, and an idle launch for rows whose bracket had missed.
#include "sv_device.h"
#include "sv_launch.h"

#include <math.h>

#include <type_traits>

#include "tile_epilogue.h"

namespace sv {

namespace {

constexpr int kMapThreads = 512, kMapWaves = kMapThreads / 64;
constexpr int kSampleLog2 = 12;
constexpr int64_t kSample = (int64_t)1 << kSampleLog2;   // sampled tokens per call
constexpr int kHeld = (int)(kSample / kMapThreads);
constexpr int64_t kMaxVocab = 262144 + 131072;           // a bit per token in LDS (48 KB)
constexpr int64_t kMinVocab = 16384;          // (shorter rows: row_select_kernel)

struct CodeLayout {
    int64_t stride;          // bytes between rows of codes: an odd multiple of 256, off the memory channels' period
    int64_t entries;         // of a row's list that memory has room for (a list has 3 to 16 % of V as a rule)
    // offsets in bytes from the scratch base (multiples of 8; the codes' of 256)
    size_t samp, map, codes, keys, list, total;
};
inline CodeLayout code_layout(int64_t V, int64_t rows) {
    CodeLayout L;
    L.stride = (V + 255) / 256 * 256 | 256;
    L.entries = V / 2;
    size_t o = 0;
    L.samp = o;   o += (size_t)rows * kSample * 4;
    L.map = o;    o += ((size_t)rows * 8 + 255) & ~(size_t)255;             // (rows of codes start on lines)
    L.codes = o;  o += (size_t)rows * (size_t)L.stride;
    L.keys = o;   o += (size_t)rows * (size_t)V * 8;
    L.list = o;   o += (size_t)rows * (size_t)L.entries * 4;
    L.total = o;
    return L;
}

// ---- map: one workgroup per row, its part of the sample in registers
// map[r] = {scale, bias} from where the rank_hi-th and the rank_lo-th largest of the row's sample scores lie (1 <= rank_hi <=
// rank_lo <= kSample): in a histogram of equal steps from the smallest to the largest, so the interval is up to two steps
// wider than those two scores -- and drawn again over itself, as long as that helps, where that is much wider, as a few scores far
// from all others make it (what bounds this kernel is its chain of barriers: 60 rows 3.5 us, 512 rows 5.6, where two
// levels of the scores' bits took 6.1 and 7.5).
// Scores beyond kFar, infinite ones among them, only count as above or below all others, and those that are no number as below:
// so the map is finite, its scale is above zero, and infinite scores get the codes at its ends.  (One infinite score in the sample used
// to send all of the row's scores through memory: 40 rows x 128256, d' = 256: 2270 us against 43.  A score that is no number gets
// code 0; the matrix instructions make all of those negative, and their bits rank below minus infinity.)
// past_hi / past_lo: the wanted rank lies beyond the sample's largest / smallest score, by which the interval is stretched.
constexpr float kFar = 1e37f;
constexpr int kMaxPasses = 16;                            // a thousandth of the width each, usually
__global__ __launch_bounds__(kMapThreads) void code_map_kernel(const float* samp, int rank_hi, int rank_lo, int past_hi,
                                                               int past_lo, float2* map) {
    constexpr int kSteps = 2 * kMapThreads;
    __shared__ uint32_t s_hist[kSteps];
    __shared__ uint32_t s_w[kMapWaves];
    __shared__ float s_min[kMapWaves], s_max[kMapWaves];
    __shared__ uint32_t s_out[4];
    const int tid = threadIdx.x;
    const float* s = samp + (int64_t)blockIdx.x * kSample;
    float v[kHeld];
#pragma unroll
    for (int u = 0; u < kHeld; ++u) v[u] = s[u * kMapThreads + tid];
    float hi = v[0], lo = v[0];
#pragma unroll
    for (int u = 1; u < kHeld; ++u) {
        hi = fmaxf(hi, v[u]);
        lo = fminf(lo, v[u]);
    }
    auto widest = [&]() {                                     // of all threads'
        hi = wave_max_f32(hi);
        lo = -wave_max_f32(-lo);
        if ((tid & 63) == 0) {
            s_max[tid >> 6] = hi;
            s_min[tid >> 6] = lo;
        }
        s_hist[2 * tid] = s_hist[2 * tid + 1] = 0u;
        __syncthreads();
#pragma unroll
        for (int w = 0; w < kMapWaves; ++w) {
            hi = fmaxf(hi, s_max[w]);
            lo = fminf(lo, s_min[w]);
        }
    };
    auto above_hi = [&]() {                                   // sample scores; s_w is free before and after
        uint32_t mine = 0u, all = 0u;
#pragma unroll
        for (int u = 0; u < kHeld; ++u) mine += v[u] > hi ? 1u : 0u;
        mine = wave_sum_u32(mine);
        if ((tid & 63) == 0) s_w[tid >> 6] = mine;
        __syncthreads();
#pragma unroll
        for (int w = 0; w < kMapWaves; ++w) all += s_w[w];
        __syncthreads();
        return all;
    };
    widest();
    uint32_t over = 0u;                                       // sample scores above hi
    if (__builtin_expect(!(hi <= kFar && lo >= -kFar), 0)) {  // uniform
        hi = -kFar;
        lo = kFar;
#pragma unroll
        for (int u = 0; u < kHeld; ++u) {
            hi = fmaxf(hi, fabsf(v[u]) <= kFar ? v[u] : hi);
            lo = fminf(lo, fabsf(v[u]) <= kFar ? v[u] : lo);
        }
        __syncthreads();                                      // everybody has read the first ones
        widest();
        over = above_hi();
    }
    for (int pass = 1;; ++pass) {
        const float step = (hi - lo) * (1.0f / kSteps), inv = (float)kSteps / (hi - lo);
#pragma unroll
        for (int u = 0; u < kHeld; ++u)
            if (v[u] >= lo && v[u] <= hi)                     // (a step out of range, or of no number (equal scores): the first or last)
                atomicAdd(&s_hist[(uint32_t)fminf(fmaxf((v[u] - lo) * inv, 0.0f), (float)(kSteps - 1))], 1u);
        __syncthreads();
        const uint32_t c0 = s_hist[2 * tid], c1 = s_hist[2 * tid + 1];
        if (tid == 0) {
            s_out[0] = (uint32_t)rank_hi <= over ? kSteps - 1 : 0;            // (where no step holds the rank)
            s_out[1] = (uint32_t)rank_lo <= over ? kSteps - 1 : 0;
            s_out[2] = 0u;
            s_out[3] = (uint32_t)kSample;
        }
        const uint32_t above1 = over + block_suffix_exclusive<kMapWaves>(c0 + c1, s_w), above0 = above1 + c1;
        auto look = [&](uint32_t rank, uint32_t* out, bool with) {     // its step, and the scores above the step (with it)
            if (above1 < rank && rank <= above1 + c1) {
                out[0] = 2u * tid + 1u;
                out[2] = above1 + (with ? c1 : 0u);
            } else if (above0 < rank && rank <= above0 + c0) {
                out[0] = 2u * tid;
                out[2] = above0 + (with ? c0 : 0u);
            }
        };
        look((uint32_t)rank_hi, s_out, false);
        look((uint32_t)rank_lo, s_out + 1, true);
        __syncthreads();
        const float first = lo, width = hi - lo;
        if (s_out[0] < kSteps - 1) hi = first + (float)(s_out[0] + 1u) * step;            // (as exactly as it can be)
        lo = first + (float)s_out[1] * step;
        const uint32_t held = s_out[3] - s_out[2];
        if (held <= 2u * (uint32_t)(rank_lo - rank_hi) + 64u || !(hi - lo < width) || pass == kMaxPasses) break;    // uniform
        __syncthreads();                                      // s_w and the histogram have been read
        s_hist[2 * tid] = s_hist[2 * tid + 1] = 0u;
        over = above_hi();
    }
    if (tid == 0) {
        // (by three times the interval: the sample's largest score alone may lie well below the k-th of them all)
        const float gap = 3.0f * (hi - lo);
        if (past_hi) hi += gap;
        if (past_lo) lo -= gap;
        // (equal scores in their thousands: an interval that their common value has to itself)
        const float width = fmaxf(hi - lo, fmaxf(fabsf(lo) * 0x1p-14f, 1e-30f));
        const float scale = 126.0f / width;
        map[blockIdx.x] = float2{scale, 128.0f - lo * scale};
    }
}

// ---- resolve
constexpr int kThreads = 1024, kWaves = kThreads / 64;
constexpr int kBins = 256, kDigitBins = 2048;
// a unit of codes per thread; later the keys from its end on downwards, and the digits' histogram or up to 64 rows of W_vocab
constexpr int kStageBytes = 32 * kThreads + 2048;
constexpr uint32_t kKeysInLds = (kStageBytes - 4 * kDigitBins) / 8;
// what two workgroups of a CU may have each, and one alone
constexpr size_t kTwoLds = 78 * 1024, kOneLds = 156 * 1024;

struct ResolveSmem {
    uint32_t hist[kBins];
    uint32_t w[kWaves], w2[kWaves];
    uint32_t out[4];
    uint32_t n_list, n_keys;
    u32x4 x[64];                                         // the hidden row
};
// dynamic LDS: a bit per token (ids that are selected) | the stage, whose end takes the keys | the list
__host__ __device__ inline size_t resolve_sel_bytes(int64_t V) { return (size_t)((V + 127) / 128) * 16; }

constexpr uint32_t kDense = 576;                         // selected ids of 2048
constexpr uint32_t kLow = 0x7F7F7F7Fu, kOne = 0x01010101u;

// One workgroup per row.  Wavefront w has `rounds` rounds of 64 units of 32 codes, lane l the units (w rounds + j) 64 + l: a
// round is 2 KB of consecutive codes, and ids ascend with (wavefront, round, lane, bit).  Codes of 255 become bits at once;
// ids with codes from 128 to 254 (three or four per cent) go to a list, on which everything else works.
// What bounds it: vector arithmetic, of which the loops over a lane's set bits are the larger part (they run as long as the
// lane with the most).  512 rows x 151936, k = 8192, two workgroups per CU: 37 us, of which a workgroup's first pass over the
// codes is 11, the choice within code C 5, the ids 4 (a second pass over the codes instead of the list: 48; the codes held in
// registers: 64, they spill; a lane's place in the list by an atomic of its own: 54).
// The list holds list_cap entries in LDS and mem_cap in memory.  Where it holds too few -- or a code below 128 decides -- the codes are walked
// once more for their histogram and once for the choice (40 rows x 128256
// whose sampled tokens are their best: 2140 us, of which the scores of the 124000 tokens that share code 0 are all but 100; with a
// list that grew to all tokens, in 13 bytes of workspace per score, 2260).
// GROUP: 3 leaves room for two workgroups per CU.
template <int GROUP>
__global__ __launch_bounds__(kThreads, GROUP > 3 ? 4 : 8) void code_resolve_kernel(int64_t V, int64_t k, const uint8_t* codes, int64_t stride,
                                                                   const char* hp, const char* Wv, int chunks, uint64_t* keys,
                                                                   uint32_t* list, int32_t* idx_out, uint32_t list_cap, uint32_t mem_cap) {
    extern __shared__ __attribute__((aligned(16))) uint32_t s_sel[];
    unsigned char* const s_stage = reinterpret_cast<unsigned char*>(s_sel) + resolve_sel_bytes(V);
    uint32_t* const s_list = reinterpret_cast<uint32_t*>(s_stage + kStageBytes);
    uint32_t* const s_digits = reinterpret_cast<uint32_t*>(s_stage);
    uint64_t* const s_keys = reinterpret_cast<uint64_t*>(s_stage + 4 * kDigitBins);
    __shared__ ResolveSmem sm;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t r = blockIdx.x;
    const int units = (int)((V + 31) / 32);
    const int rounds = (units + kThreads - 1) / kThreads;
    const u32x4* const row = reinterpret_cast<const u32x4*>(codes + r * stride);
    const int u0 = wave * rounds * 64 + lane;
    uint64_t* const keys_mem = keys + r * V;
    uint32_t* const list_mem = list + r * (int64_t)mem_cap;
    // f(unit, codes) for the lane's units, with all lanes (units past the last: codes of 0); the codes of `group` rounds are
    // requested together
    auto for_each_unit = [&](auto group, auto&& f) {
        constexpr int kGroup = decltype(group)::value;
        for (int j0 = 0; j0 < rounds; j0 += kGroup) {
            u32x4 q[kGroup][2];
#pragma unroll
            for (int j = 0; j < kGroup; ++j) {
                const int u = min(u0 + 64 * (j0 + j), units - 1);
                q[j][0] = row[2 * u];
                q[j][1] = row[2 * u + 1];
            }
#pragma unroll
            for (int j = 0; j < kGroup; ++j) {
                const int u = u0 + 64 * (j0 + j);
                if (j0 + j >= rounds) return;                 // uniform
                if (u >= units) q[j][0] = q[j][1] = zero16();
                f(u, q[j]);
            }
        }
    };
    // (a hidden row of zeros -- a padding row of the batch -- has nothing but equal scores)
    bool zero_row = true;
    const char* const x_row = hp + r * chunks * 16;
    if (lane < chunks) {
        const u32x4 v = reinterpret_cast<const u32x4*>(x_row)[lane];
        zero_row = ((v[0] | v[1] | v[2] | v[3]) & 0x7FFF7FFFu) == 0u;
        if (wave == 0) sm.x[lane] = v;
    }
    zero_row = __builtin_amdgcn_ballot_w64(!zero_row) == 0ull;
    int32_t* const out = idx_out + r * k;
    if (zero_row) {                                           // uniform
        for (int64_t j = tid; j < k; j += kThreads) out[j] = (int32_t)j;
        return;
    }
    if (tid < kBins) sm.hist[tid] = 0u;
    if (tid == 0) sm.n_list = sm.n_keys = 0u;
    __syncthreads();

    // entry: id and code
    auto put_entry = [&](uint32_t at, uint32_t entry) {
        if (at < list_cap) s_list[at] = entry;
        else if (at - list_cap < mem_cap) list_mem[at - list_cap] = entry;
    };
    // (the lane's codes go to LDS as well, where a byte can be fetched by its number)
    unsigned char* const s_mine = s_stage + tid * 32;
    uint32_t full = 0u;
    for_each_unit(std::integral_constant<int, GROUP>{}, [&](int u, const u32x4 (&q)[2]) {
        reinterpret_cast<u32x4*>(s_mine)[0] = q[0];
        reinterpret_cast<u32x4*>(s_mine)[1] = q[1];
        uint32_t in = 0u, above = 0u;                         // bit 8 b + w: byte b of word w is 128 .. 254, is 255
#pragma unroll
        for (int w = 0; w < 8; ++w) {
            const uint32_t x = q[w >> 2][w & 3];
            const uint32_t all = (x & kLow) + kOne;           // top bits: the low seven bits are all ones
            in |= ((x & ~all) >> (7 - w)) & (kOne << w);
            above |= ((x & all) >> (7 - w)) & (kOne << w);
        }
        if (u < units) s_sel[u] = above;
        full += (uint32_t)__popc(above);
        // (places by wavefront: as many lanes' atomics on one address take several times the whole loop)
        const uint32_t c = (uint32_t)__popc(in), incl = wave_prefix_inclusive_u32(c);
        uint32_t at = 0u;
        if (lane == 63) at = atomicAdd(&sm.n_list, incl);
        at = (uint32_t)__builtin_amdgcn_readlane((int)at, 63);
        const uint32_t end = at + (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
        at += incl - c;
        const uint32_t id0 = 32u * (uint32_t)u;
        auto entry_of = [&](uint32_t p) { return ((id0 + p) << 8) | s_mine[(p & 7u) * 4u + (p >> 3)]; };
        if (end <= list_cap) {                                // uniform
            while (in) {
                const uint32_t p = (uint32_t)__builtin_ctz(in);
                s_list[at++] = entry_of(p);
                in &= in - 1u;
            }
        } else {
            while (in) {
                put_entry(at++, entry_of((uint32_t)__builtin_ctz(in)));
                in &= in - 1u;
            }
        }
    });
    full = wave_sum_u32(full);
    if (lane == 0) sm.w2[wave] = full;
    __threadfence_block();
    __syncthreads();
    full = 0u;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) full += sm.w2[w];
    auto same = [](uint32_t x) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)x); };     // (in a scalar register)
    full = same(full);
    const uint32_t n_list = same(sm.n_list), wanted = (uint32_t)k;
    auto for_each_entry = [&](auto&& f) {
        for (uint32_t i = tid; i < min(n_list, list_cap); i += kThreads) f(s_list[i]);
        for (uint32_t i = list_cap + tid; i < n_list; i += kThreads) f(list_mem[i - list_cap]);
    };
    // the code of the k-th score: its number, the scores above it, its scores
    const bool top = wanted <= full;                          // above hi
    const bool walk = !top && (wanted > full + n_list || n_list > list_cap + mem_cap);
    uint32_t C = 255u, above = 0u, n = full;
    if (__builtin_expect(!top, 1)) {                          // uniform
        if (__builtin_expect(!walk, 1)) {
            for_each_entry([&](uint32_t e) { atomicAdd(&sm.hist[e & 255u], 1u); });
        } else {
            for_each_unit(std::integral_constant<int, 1>{}, [&](int u, const u32x4 (&q)[2]) {   // (equal codes in a row together)
                reinterpret_cast<u32x4*>(s_mine)[0] = q[0];
                reinterpret_cast<u32x4*>(s_mine)[1] = q[1];
                const uint32_t valid = u < units ? (uint32_t)min((int64_t)32, V - 32 * (int64_t)u) : 0u;
                uint32_t code = 255u, run = 0u;
                for (uint32_t p = 0; p < valid; ++p) {
                    const uint32_t x = s_mine[(p & 7u) * 4u + (p >> 3)];
                    if (x != code) {
                        if (code != 255u) atomicAdd(&sm.hist[code], run);
                        code = x;
                        run = 0u;
                    }
                    ++run;
                }
                if (code != 255u) atomicAdd(&sm.hist[code], run);
            });
        }
        __syncthreads();
        const uint32_t c = tid < kBins ? (tid == 255 ? full : sm.hist[tid]) : 0u;
        const uint32_t higher = block_suffix_exclusive<kWaves>(c, sm.w);
        if (higher < wanted && wanted <= higher + c) {
            sm.out[0] = (uint32_t)tid;
            sm.out[1] = higher;
            sm.out[2] = c;
        }
        __syncthreads();
        C = same(sm.out[0]);
        above = same(sm.out[1]);
        n = same(sm.out[2]);
    }
    const uint32_t need = wanted - above;                     // of the n scores of code C: 1 <= need <= n
    const bool whole = need == n, in_lds = n <= kKeysInLds;

    // ids above code C become bits; those of code C too, if all are selected, or they go to the list of keys
    // (an inverted id each, with the score on top as soon as it is known)
    auto select_id = [&](uint32_t id) { atomicOr(&s_sel[id >> 5], 1u << (id & 31u)); };
    auto put_key = [&](uint32_t at, uint32_t id) {
        if (in_lds) s_keys[kKeysInLds - 1u - at] = (uint64_t)(~id);
        if (!in_lds) keys_mem[at] = (uint64_t)(~id);
    };
    auto put_keys = [&](int u, uint32_t bits) {               // of a lane's unit
        if (bits == 0u) return;
        for (uint32_t at = atomicAdd(&sm.n_keys, (uint32_t)__popc(bits)); bits; bits &= bits - 1u)
            put_key(at++, 32u * (uint32_t)u + (uint32_t)__builtin_ctz(bits));
    };
    if (__builtin_expect(top, 0)) {                           // uniform: the codes of 255 are bits already
        for (int j = 0; j < rounds && !whole; ++j) {
            const int u = u0 + 64 * j;
            if (u >= units) break;
            put_keys(u, s_sel[u]);
            s_sel[u] = 0u;
        }
    } else if (__builtin_expect(walk, 0)) {
        for_each_unit(std::integral_constant<int, 1>{}, [&](int u, const u32x4 (&q)[2]) {
            uint32_t more = 0u, equal = 0u;
#pragma unroll
            for (int p = 0; p < 32; ++p) {                    // byte p / 8 of word p % 8
                const uint32_t x = (q[(p & 7) >> 2][p & 3] >> (8 * (p >> 3))) & 255u;
                more |= x > C ? 1u << p : 0u;
                equal |= x == C ? 1u << p : 0u;
            }
            if (u >= units) return;
            const int64_t left = V - 32 * (int64_t)u;
            if (left < 32) equal &= (1u << left) - 1u;        // (codes of 0 follow)
            s_sel[u] = more | (whole ? equal : 0u);
            if (!whole) put_keys(u, equal);
        });
    } else {
        for_each_entry([&](uint32_t e) {
            const uint32_t c = e & 255u, id = e >> 8;
            if (c > C || (whole && c == C)) select_id(id);
            else if (c == C) put_key(atomicAdd(&sm.n_keys, 1u), id);
        });
    }
    if (!whole) {                                             // uniform: the `need` largest scores of code C are wanted
        auto choose = [&](auto lds) {
            constexpr bool LDS = decltype(lds)::value;        // the keys are there, and not in memory
            auto key_at = [&](uint32_t i) -> uint64_t {
                if constexpr (LDS) return s_keys[kKeysInLds - 1u - i];
                else return keys_mem[i];
            };
            __threadfence_block();
            __syncthreads();
            // Their scores, 32 ids at a time as rows of the first operand; every column of the second is the hidden row
            auto multiply = [&](uint32_t at, auto&& unit) {       // unit(c): unit c of the lane's row
                f32x16_t acc;
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[e] = 0.f;
                for (int k0 = 0; k0 < chunks; k0 += 8) {
                    u32x4 a[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) a[i] = unit(min(k0 + 2 * i + (lane >> 5), chunks - 1));
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int c = k0 + 2 * i + (lane >> 5);
                        const u32x4 b = sm.x[min(c, chunks - 1)];
                        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, c < chunks ? a[i] : zero16()),
                                                                      __builtin_bit_cast(bf16x8_t, c < chunks ? b : zero16()), acc, 0, 0, 0);
                    }
                }
                // element e of lanes l < 32 and l + 32: ids 8 (e / 4) + e % 4 and 4 more (every l the same)
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const uint32_t i = at + (uint32_t)(8 * (e >> 2) + 4 * (lane >> 5) + (e & 3));
                    if ((lane & 31) == e && i < n) {
                        if constexpr (LDS) reinterpret_cast<uint32_t*>(s_keys)[2u * (kKeysInLds - 1u - i) + 1u] = f32_to_ord(acc[e]);
                        else reinterpret_cast<uint32_t*>(keys_mem)[2 * (int64_t)i + 1] = f32_to_ord(acc[e]);
                    }
                }
            };
            if (LDS && n <= 64u && n * ((uint32_t)(chunks + 1) * 16u + 8u) <= (uint32_t)kStageBytes) {
                // The usual handful: all threads bring the rows of W_vocab, in one round trip, and two wavefronts multiply.
                // Ranked by counting (keys are unique: they end in the id)
                u32x4* const s_rows = reinterpret_cast<u32x4*>(s_stage);
                for (uint32_t i = (uint32_t)tid; i < n * 32u; i += kThreads) {
                    const u32x4* w_row = reinterpret_cast<const u32x4*>(Wv + (int64_t)(~(uint32_t)key_at(i >> 5)) * chunks * 16);
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
                    const uint64_t mine = (uint32_t)lane < n ? key_at((uint32_t)lane) : 0ull;
                    uint32_t larger = 0u;
                    for (uint32_t i = 0; i < n; ++i) larger += readlane_u64(mine, (int)i) > mine;
                    if ((uint32_t)lane < n && larger < need) select_id(~(uint32_t)mine);
                }
                return;
            }
            for (uint32_t at = (uint32_t)wave * 32u; at < n; at += kWaves * 32u) {
                const uint32_t inv = (uint32_t)key_at(min(at + (uint32_t)(lane & 31), n - 1u));
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
                const int w = 64 - decided < 11 ? 64 - decided : 11, shift = 64 - decided - w;
                __syncthreads();
                s_digits[tid] = 0u;
                s_digits[tid + kThreads] = 0u;
                __syncthreads();
                for (uint32_t i = tid; i < n; i += kThreads) {
                    const uint64_t x = key_at(i);
                    if (decided == 0 || (x >> (64 - decided)) == (T >> (64 - decided)))
                        atomicAdd(&s_digits[(uint32_t)(x >> shift) & ((1u << w) - 1u)], 1u);
                }
                __syncthreads();
                const uint32_t c0 = s_digits[2 * tid], c1 = s_digits[2 * tid + 1];
                const uint32_t above = block_suffix_exclusive<kWaves>(c0 + c1, sm.w);
                if (above < remain && remain <= above + c1) {
                    sm.out[0] = 2u * tid + 1u;
                    sm.out[1] = above;
                    sm.out[2] = c1;
                } else if (above + c1 < remain && remain <= above + c1 + c0) {
                    sm.out[0] = 2u * tid;
                    sm.out[1] = above + c1;
                    sm.out[2] = c0;
                }
                __syncthreads();
                T |= (uint64_t)sm.out[0] << shift;
                remain -= sm.out[1];
                decided += w;
                if (remain == sm.out[2]) break;               // every key with these digits is selected
            }
            for (uint32_t i = tid; i < n; i += kThreads) {
                const uint64_t x = key_at(i);
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
    uint32_t total = 0u;
    for (int j = 0; j < rounds; ++j) {
        const int u = u0 + 64 * j;
        total += u < units ? (uint32_t)__popc(s_sel[u]) : 0u;
    }
    total = wave_sum_u32(total);
    if (lane == 0) sm.w2[wave] = total;
    __syncthreads();
    uint32_t base = 0u, all = 0u;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        base += w < wave ? sm.w2[w] : 0u;
        all += sm.w2[w];
    }
    if (all != (uint32_t)k) return;                           // never: k bits are set
    for (int j = 0; j < rounds; ++j) {
        const int u = u0 + 64 * j;
        uint32_t bits = u < units ? s_sel[u] : 0u;
        const uint32_t c = (uint32_t)__popc(bits);
        const uint32_t incl = wave_prefix_inclusive_u32(c), here = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
        if (here >= kDense) {                                 // uniform: a lane per token, two units at a time
            const uint32_t first = 32u * (uint32_t)(u - lane) + (uint32_t)lane;
            for (int i = 0; i < 64; i += 2) {
                const uint32_t b0 = (uint32_t)__builtin_amdgcn_readlane((int)bits, i), b1 = (uint32_t)__builtin_amdgcn_readlane((int)bits, i + 1);
                const uint32_t at = __builtin_amdgcn_mbcnt_hi(b1, __builtin_amdgcn_mbcnt_lo(b0, base));
                if (((lane < 32 ? b0 : b1) >> (lane & 31)) & 1u)
                    *reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(out) + at * 4u) = first + 32u * (uint32_t)i;
                base += (uint32_t)(__popc(b0) + __popc(b1));
            }
            continue;
        }
        uint32_t at = (base + incl - c) * 4u;
        base += here;
        const uint32_t id0 = 32u * (uint32_t)u;
        while (bits) {
            *reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(out) + at) = id0 + (uint32_t)__builtin_ctz(bits);
            at += 4u;
            bits &= bits - 1u;
        }
    }
}

}  // namespace

// From 65 rows on (panel_supported), where two bytes per score are not the shorter way and short rows not that of row_select_kernel: both have
// their lines, with figures, beside key_select_supported and row_select_preferred.
bool code_select_supported(int dt, int chunks, int64_t rows, int64_t V, int64_t k) {
    return panel_supported(dt, chunks, rows, V) && V >= kMinVocab && V <= kMaxVocab && !key_select_supported(dt, chunks, rows, V, k) &&
           !row_select_preferred(chunks, rows, V);
}

// (more than 64 KB of LDS: an opt-in)
hipError_t configure_code_select_lds() {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&code_resolve_kernel<3>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)kOneLds);
    if (e != hipSuccess) return e;
    return hipFuncSetAttribute(reinterpret_cast<const void*>(&code_resolve_kernel<6>),
                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)kOneLds);
}

size_t code_select_scratch_bytes(int64_t rows, int64_t V) { return code_layout(V, rows).total; }

hipError_t launch_code_select(const CodeSelectArgs& a, hipStream_t stream) {
    const CodeLayout L = code_layout(a.V, a.rows);
    PanelArgs p{};
    p.x = a.hp;
    p.x_row_bytes = (int64_t)a.chunks * 16;
    p.M = a.Wv;
    p.m_row_bytes = (int64_t)a.chunks * 16;
    p.n_items = kSample;
    p.chunks = a.chunks;
    p.rows = a.rows;
    p.out = reinterpret_cast<float*>(a.scratch + L.samp);
    p.out_row_stride = kSample;
    p.spread_V = a.V;
    p.spread_shift = kSampleLog2;
    hipError_t e = launch_panel_sample(p, stream);
    if (e != hipSuccess) return e;
    // The number of sampled tokens among the row's k best is hypergeometric with mean m k / V: its rank range, 4.5 standard
    // deviations and 4 more on either side (a row in a hundred thousand lies outside, and costs tens of microseconds)
    const double share = (double)a.k / (double)a.V, mean = (double)kSample * share;
    const double reach = 4.5 * sqrt((double)kSample * share * (1.0 - share)) + 4.0;
    const double rank_hi = floor(mean - reach), rank_lo = ceil(mean + reach);
    float2* map = reinterpret_cast<float2*>(a.scratch + L.map);
    hipLaunchKernelGGL(code_map_kernel, dim3((unsigned)a.rows), dim3(kMapThreads), 0, stream, p.out,
                       (int)fmax(rank_hi, 1.0), (int)fmin(rank_lo, (double)kSample), rank_hi < 1.0 ? 1 : 0,
                       rank_lo > (double)kSample ? 1 : 0, map);
    p.n_items = a.V;
    p.out = nullptr;
    p.code_map = reinterpret_cast<const float*>(map);
    p.codes = reinterpret_cast<uint8_t*>(a.scratch + L.codes);
    p.code_stride = L.stride;
    e = launch_panel_codes(p, stream);
    if (e != hipSuccess) return e;
    // LDS for the list: what the expected number of entries needs and a sixth more, if that leaves two workgroups on a CU or if
    // there is but one row per CU; else as much as two workgroups have
    DeviceInfo di;
    e = device_info(&di);
    if (e != hipSuccess) return e;
    const double entries = (fmin(rank_lo, (double)kSample) - fmax(rank_hi, 0.0)) / (double)kSample * (double)a.V;
    const size_t fixed = resolve_sel_bytes(a.V) + kStageBytes + sizeof(ResolveSmem);
    const size_t want = ((size_t)(entries * 1.17) + 256) * 4, most = (a.rows > di.cus ? kTwoLds : kOneLds);
    size_t list_bytes = fixed + want <= most ? want : (fixed + 4096 <= most ? most - fixed : 4096);
    list_bytes &= ~(size_t)15;
    auto resolve = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)a.rows), dim3(kThreads), resolve_sel_bytes(a.V) + kStageBytes + list_bytes, stream,
                           a.V, a.k, p.codes, L.stride, a.hp, a.Wv, a.chunks, reinterpret_cast<uint64_t*>(a.scratch + L.keys),
                           reinterpret_cast<uint32_t*>(a.scratch + L.list), a.idx_out, (uint32_t)(list_bytes / 4), (uint32_t)L.entries);
    };
    if (a.rows <= di.cus) resolve(&code_resolve_kernel<6>);
    else resolve(&code_resolve_kernel<3>);
    return hipGetLastError();
}

}  // namespace sv

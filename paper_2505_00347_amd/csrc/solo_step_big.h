// The fused SOLO AdamW step for blocks of 2048 elements (the large-block setting of the paper's
// block-size comparison, Sec. 4.2), gfx950, wave64.
//
// A block of 2048 elements is held by one workgroup: of two wavefronts, 1024 elements each, sixteen
// consecutive elements per lane, or, where a launch has few blocks, of four, eight per lane
// (step_block_quad).  The shorter last block of a buffer runs in the same launch.
// The element-wise part (decode by table look-up, both EMAs, the parameter, the encoders, the
// 32-bit words of the code streams) is that of a 1024-element chunk of solo_step.h and runs
// without any exchange between the wavefronts.  What a block of this size changes is the block
// statistics:
//   * Delta_m' and Delta_v' are maxima over the wavefronts: DPP inside a row, four lane reads
//     across the rows, a few words of LDS and one barrier across the wavefronts;
//   * the p-quantile is the rank-205 element of 2048 values (p = 0.1), far too deep for rounds
//     of "extract the minimum".  It is found by histograms, first over what lies right above a bound that the
//     old state gives, then over ever narrower ranges of the bit
//     patterns, and, once a few keys are left, by comparing those (select_rank);
//   * the base alpha, the divisions and the level tables are computed by every wavefront (every
//     16 lanes) for itself: cheaper than another barrier.
// The number of workgroups on a CU is bound by LDS
// (an earlier form: 17.3 ms for 6.7e9 parameters at 3.5 wavefronts per SIMD, 15.7 ms at 5), so the histogram is
// kept small: see BigLayout.  (What the selection costs: a layer of the 7B shapes, 2-bit/3-bit, 377 us, 330 without any.)  Every wavefront stages and writes back the words of its own elements
// (whole 128-byte lines for 2- and 4-bit codes; ten-to-a-word codes by one atomic XOR per word at
// the memory side, since a wavefront's share does not end on a word).
#pragma once
#include "solo_step.h"

namespace solo {

constexpr int kBigBlock = 2048;
constexpr int kBigWaves = kBigBlock / kIter16;
static_assert(kBigWaves == 2, "one workgroup of two wavefronts per block");

// LDS of a workgroup (32-bit words).  `work` first serves the wavefronts as the staging areas of
// their layout transpositions, then, behind the barrier of the block maxima, the whole workgroup as
// the histograms of the selection.
// The second moments of a block that has been trained for a while sit in a few tight clusters, one
// per level of the previous code, so most of the 64 lanes of an instruction add to the same one or
// two bins, and LDS applies the adds to one bank one after the other (measured on MI355X with one
// counter per bin: the step slowed down by half between the first and the thousandth update of a
// state, all of it LDS bank conflicts).  Every bin therefore has 4 counters in neighbouring words, i.e.
// in different banks, and a lane always uses the one its number selects: 512 bins x 4 counters, the
// lower halves of the words for the first pass, the upper halves for the second (a count is at
// most 2048, so the halves do not carry into each other, and a wavefront that is still reading the
// lower halves is not disturbed by one that already counts the next pass in the upper ones).
constexpr uint32_t kFewKeys = 32;      // so many keys are compared instead of counted (a power of two, at most 64)
struct BigLayout {
    static constexpr int kStage = 64 * kColStride16;          // per wavefront: staging of the layout transpositions
    static constexpr int kWork = kBigWaves * kStage;
    static constexpr int kOffImgM = 0;                        // per wavefront: its words of each code stream
    static constexpr int kOffImgV = 132;
    static constexpr int kOffTv = 272;                        // level tables, 64-byte aligned
    static constexpr int kOffTm = 288;
    static constexpr int kSlab = 304;
};
static_assert(BigLayout::kWork >= 2048, "the histogram lies inside the work area");
// Exchange between the W wavefronts of a block: block maxima; ranges of two passes; counts of the guess;
// the keys that are left.
template <int W>
struct BigExchange {
    static constexpr int kMaxM = 0, kMaxV = W, kPass = 2 * W, kCounts = kPass + 10, kLeft = kCounts + 2 * W, kList = kLeft + W;
    static constexpr int kWords = kList + W * (int)kFewKeys;
};
static_assert(288 * 4 <= BigLayout::kStage, "the padded transposition (Stage16) fits a staging area");
static_assert(VarianceCodes16<3>::kImage <= 132, "images");

// Maximum over the 64 lanes of a wavefront (uniform result).
__device__ __forceinline__ uint32_t wave_max(uint32_t x)
{
    x = group_reduce<16>(x, UMax());
    const uint32_t a = (uint32_t)__builtin_amdgcn_readlane((int)x, 0), b = (uint32_t)__builtin_amdgcn_readlane((int)x, 16);
    const uint32_t c = (uint32_t)__builtin_amdgcn_readlane((int)x, 32), d = (uint32_t)__builtin_amdgcn_readlane((int)x, 48);
    return umax(umax(a, b), umax(c, d));
}

// Inclusive prefix sum over the 64 lanes of a wavefront: four shifted adds inside every row of 16
// lanes, then the last lane of a row is added to the rows behind it.
__device__ __forceinline__ uint32_t wave_inclusive_sum(uint32_t x)
{
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xF, 0xF, true);   // row_shr:1
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xF, 0xF, true);   // row_shr:2
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xF, 0xF, true);   // row_shr:4
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xF, 0xF, true);   // row_shr:8
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xA, 0xF, false);  // row_bcast:15 into rows 1 and 3
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xC, 0xF, false);  // row_bcast:31 into rows 2 and 3
    return x;
}

// Where the selection stands: the rank-th of the `count` keys in [base, base + len).  `guess`: a key
// of that range which many of them may equal (kNoGuess: none known).
struct Narrowed { uint32_t base, len, rank, count, guess; };
constexpr uint32_t kNoGuess = 0xFFFFFFFFu;
constexpr uint32_t kNoKey = 0xFFFFFFFFu;       // of an element that does not exist: outside every range

// The bin of the histogram (512 bins of 4 counters each, in the halves `half` of its words) that holds
// the rank-th key, by one wavefront: a lane sums the 32 words of its own 8 bins (128-bit reads in an
// order that starts neighbouring lanes in different banks), a prefix sum over the wavefront names
// the lane whose bins hold the rank, and that lane's words are read once more, one per lane, for a
// second prefix sum that names the bin.  Returns the bin, its rank and its count (0: the histogram holds fewer keys).
__device__ __forceinline__ uint32_t find_bin(const uint32_t *const h, const uint32_t half, uint32_t &rank, uint32_t &count,
                                             const uint32_t lane)
{
    const uint32_t first = 32u * lane + 4u * ((lane + (lane >> 2)) & 7u);
    uint32_t acc = 0;                              // (sums of the halves do not carry: 2048 keys at most)
#pragma unroll
    for (uint32_t i = 0; i < 8; ++i) {
        const uint4 c4 = *reinterpret_cast<const uint4 *>(h + (first ^ (4u * i)));
        acc += (c4.x + c4.y) + (c4.z + c4.w);
    }
    const uint32_t s = (acc >> half) & 0xFFFFu, incl = wave_inclusive_sum(s);
    if (rank > (uint32_t)__builtin_amdgcn_readlane((int)incl, 63)) { count = 0; return 0; }
    const uint32_t sel = (uint32_t)__builtin_ctzll(__builtin_amdgcn_ballot_w64(rank <= incl) | (1ull << 63));
    rank -= (uint32_t)__builtin_amdgcn_readlane((int)(incl - s), (int)sel);
    const uint32_t in_row = wave_inclusive_sum((h[32u * sel + (lane & 31u)] >> half) & 0xFFFFu);   // (lanes 0-31 matter)
    const uint32_t bin = (uint32_t)__builtin_ctzll(__builtin_amdgcn_ballot_w64(rank <= in_row) | (1ull << 31)) / 4u;
    const uint32_t before = bin ? (uint32_t)__builtin_amdgcn_readlane((int)in_row, (int)(4u * bin - 1u)) : 0u;
    count = (uint32_t)__builtin_amdgcn_readlane((int)in_row, (int)(4u * bin + 3u)) - before;
    rank -= before;
    return 8u * sel + bin;
}

// Counts a key in the histogram where `at16`, sixteen times its bin and some bits below, lies inside of it.  (All lanes
// are active.  Written out because the compiler branches around an atomic under a condition.)
__device__ __forceinline__ void count_key(const uint32_t at16, const uint32_t counters, const uint32_t one)
{
    asm volatile("v_cmp_gt_u32_e32 vcc, 0x2000, %0\n\ts_mov_b64 exec, vcc\n\tds_add_u32 %1, %2\n\ts_mov_b64 exec, -1"
                 : : "v"(at16), "v"(counters + (at16 & 0x1FF0u)), "v"(one) : "vcc", "memory");
}

// One pass of the selection: the keys in the range are counted by (key - base) >> shift, one barrier,
// one of the two wavefronts (they take turns) finds the bin of the rank and leaves the new range in
// LDS, a second barrier (it costs less than both wavefronts summing the histogram for themselves).
// FIRST: 512 bins of 2^shift patterns from at.base on; keys below it count in the first bin, keys behind the last
// one (and kNoKey) not at all: at.count = 0 says that the rank lies there, and at.rank stays.
template <int NK, bool FIRST>
__device__ __forceinline__ void narrow(Narrowed &at, const uint32_t (&key)[NK], const uint32_t lane, const bool mine,
                                       uint32_t *const h, const uint32_t half, uint32_t *const res, const uint32_t first_shift = 0)
{
    const uint32_t wide = 32u - (uint32_t)__builtin_clz(at.len - 1u);          // (len > 1)
    const uint32_t shift = FIRST ? first_shift : wide > 9u ? wide - 9u : 0u, one = 1u << half;
    const uint32_t counters = lds_addr(h) + 4u * (lane & 3u);
    if (FIRST) {
        const uint32_t base = in_vector(at.base), by = in_vector(shift - 4u);
#pragma unroll
        for (int j = 0; j < NK; ++j) count_key(__builtin_elementwise_sub_sat(key[j], base) >> by, counters, one);
    } else {
        char *const bytes = reinterpret_cast<char *>(h);
#pragma unroll
        for (int j = 0; j < NK; ++j) {
            const uint32_t d = key[j] - at.base;
            if (d < at.len) atomicAdd(reinterpret_cast<uint32_t *>(bytes + ((d >> shift) << 4 | 4u * (lane & 3u))), one);
        }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");        // (the compiler does not know of count_key's)
    __syncthreads();
    if (mine) {
        uint32_t rank = at.rank, count;
        const uint32_t bin = find_bin(h, half, rank, count, lane);
        uint32_t base = at.base, len = at.base + (1u << shift);
        if (FIRST && bin == 0) {                   // everything below the first bin's end
            base = 0;
        } else {
            const uint32_t begin = bin << shift, left = FIRST ? 1u << shift : at.len - begin;
            base += begin;
            len = left < (1u << shift) ? left : 1u << shift;
        }
        uint32_t guess = kNoGuess;
        if (FIRST) {                               // do the wavefront's first keys of the new range look all the same?
            const uint64_t in0 = __builtin_amdgcn_ballot_w64(key[0] - base < len);
            const uint32_t v = (uint32_t)__builtin_amdgcn_readlane((int)key[0], (int)__builtin_ctzll(in0 | (1ull << 63)));
            const uint64_t same = __builtin_amdgcn_ballot_w64(key[0] == v) & in0;
            if (2 * __builtin_popcountll(same) > __builtin_popcountll(in0) + 2) guess = v;
        }
        if (lane == 0) { res[0] = base; res[1] = len; res[2] = rank; res[3] = count; if (FIRST) res[4] = guess; }
    }
    __syncthreads();
    const uint32_t count = (uint32_t)__builtin_amdgcn_readfirstlane((int)res[3]);
    at.count = count;
    if (FIRST && count == 0) return;
    at.base = (uint32_t)__builtin_amdgcn_readfirstlane((int)res[0]);
    at.len = (uint32_t)__builtin_amdgcn_readfirstlane((int)res[1]);
    at.rank = (uint32_t)__builtin_amdgcn_readfirstlane((int)res[2]);
    if (FIRST) at.guess = (uint32_t)__builtin_amdgcn_readfirstlane((int)res[4]);
}

// The keys of the range below the guess and equal to it are counted (by ballot: nothing that many
// equal keys could slow down); the rank's side of it becomes the range.  Returns whether the guess
// is the answer.
template <int NK, int W>
__device__ __forceinline__ bool try_guess(Narrowed &at, const uint32_t (&key)[NK], const uint32_t lane, const uint32_t wave,
                                          uint32_t *const counts)
{
    uint32_t below = 0, same = 0;
#pragma unroll
    for (int j = 0; j < NK; ++j) {
        below += (uint32_t)__builtin_popcountll(__builtin_amdgcn_ballot_w64(key[j] - at.base < at.guess - at.base));
        same += (uint32_t)__builtin_popcountll(__builtin_amdgcn_ballot_w64(key[j] == at.guess));
    }
    if (lane == 0) { counts[2 * wave] = below; counts[2 * wave + 1] = same; }
    __syncthreads();
    below = 0; same = 0;
#pragma unroll
    for (int w = 0; w < W; ++w) { below += counts[2 * w]; same += counts[2 * w + 1]; }
    below = (uint32_t)__builtin_amdgcn_readfirstlane((int)below);
    same = (uint32_t)__builtin_amdgcn_readfirstlane((int)same);
    if (at.rank <= below) {
        at.len = at.guess - at.base;
        at.count = below;
        return false;
    }
    if (at.rank <= below + same) return true;
    at.rank -= below + same;
    at.count -= below + same;
    at.len -= at.guess + 1u - at.base;
    at.base = at.guess + 1u;
    return false;
}

// The largest v^ of the block, out of the exchange (behind a barrier).
template <int W>
__device__ __forceinline__ uint32_t largest_key(const uint32_t *const xch)
{
    uint32_t k = 0;
#pragma unroll
    for (int w = 0; w < W; ++w) k = umax(k, xch[BigExchange<W>::kMaxV + w]);
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)k);
}

// The rank-th smallest (1-based, uniform over the workgroup) of the `present` keys that the threads of
// the workgroup hold, NK each (W wavefronts; kNoKey: no key): bit patterns of non-negative floats.
// `floor`: a bound below all keys that the old state gives (0: none), beta2 times its smallest level.  Of a
// state that has been trained for a while the elements with the last code, a little more than the quantile's share,
// lie right above it, moved up by (1 - beta2) g^2.  So the first pass counts the quarter of an octave above the
// floor in 512 bins; seven of eight keys are above it and cost no LDS access.  Where the rank lies higher, or without
// a floor, a pass over sixteenths of an octave below the maximum follows (2^28 consecutive
// patterns in 512 bins); the next ones count 512ths of the bin that holds the rank.  As soon as at most
// kFewKeys are left, every wavefront compares those with each other instead: mostly after one pass on a trained state,
// after two on scattered values.  Elements without a gradient share the
// few decoded values: then, after the first pass, one of the keys that are left is tried as it is.
// A rank below that pass's range (28 octaves under the maximum, or zeros) starts over from 0.
// (Against a first pass over the 28 octaves, in turn, us: a layer of the 7B shapes 444 -> 377, as a table 472 -> 399, 2^26
// elements 4-bit/2-bit DE fp32 with a copy 203 -> 182, 4.2 million 15.96 -> 14.77; 2^25 elements over four formats, quantiles from
// 0.05 to 0.5 and idle rows 1.07 to 1.30 times as fast, without a state 1.03.  A step in which the gradients of all blocks jump takes
// the first pass for nothing: 2^25 elements, 2-bit/3-bit, ten times the gradients at once, 68 -> 74, with a hundredth of the blocks jumping 78 -> 66.  Before that, four fixed passes over
// 8 + 8 + 8 + 7 bits took 6 % longer than the 28 octaves on scattered values, 45 % with nine of ten gradients at zero.)
// BARRIER: whether the exchange's maxima still need one.
template <int NK, int W, bool BARRIER>
__device__ __forceinline__ uint32_t select_rank(const uint32_t (&key)[NK], const uint32_t floor, const uint32_t rank,
                                                const uint32_t present, const uint32_t lane, const uint32_t wave,
                                                uint32_t *const work, uint32_t *const xch)
{
    using Xch = BigExchange<W>;
    constexpr uint32_t kReach = 1u << 28, kFine = 12u, kCoarse = 19u, kBelow = 8u << kFine;   // (a few bins of room for rounding)
    uint32_t *const res = xch + Xch::kPass;
    Narrowed at = {0u, 1u << 31, rank, present, kNoGuess};
    bool lower_only = true;                        // of the histogram's words, only the lower halves have been used
    if (__builtin_expect(present > kFewKeys, 1)) {
        uint32_t shift = kFine;
        at.base = floor - umin(floor, kBelow);
        if (BARRIER && floor == 0) __syncthreads();
        for (;;) {
            if (floor == 0 || shift == kCoarse) {
                const uint32_t kmax = largest_key<W>(xch);
                at.base = umax(floor == 0 ? 0u : at.base + (512u << kFine), kmax >= kReach ? kmax - (kReach - 1u) : 0u);
                shift = kCoarse;
            }
            narrow<NK, true>(at, key, lane, wave == 0, work, lower_only ? 0u : 16u, res, shift);
            if (at.count != 0 || shift == kCoarse) break;          // (no key left: only what is not finite)
            shift = kCoarse;
            lower_only = false;
        }
        if (at.guess != kNoGuess && try_guess<NK, W>(at, key, lane, wave, xch + Xch::kCounts)) return at.guess;
    }
#pragma unroll 1
    for (uint32_t turn = 1; at.count > kFewKeys && at.len > 1u; ++turn) {
        if (!lower_only) {                         // both halves have been used
            uint4 *const z = reinterpret_cast<uint4 *>(work);
            for (uint32_t i = wave * 64u + lane; i < 512u; i += W * 64) z[i] = make_uint4(0, 0, 0, 0);
            __syncthreads();
        }
        narrow<NK, false>(at, key, lane, wave == (turn & 1u), work, lower_only ? 16u : 0u, res + 5 * (turn & 1u));
        lower_only = false;
    }
    if (at.len == 1u) return at.base;
    // few keys: every wavefront packs its own into LDS, then each lane compares one with all of
    // them: the answer is the largest key with fewer than `rank` keys below it
    uint32_t *const list = xch + Xch::kList + wave * kFewKeys;
    uint32_t mine = 0;
#pragma unroll
    for (int j = 0; j < NK; ++j) {
        const bool in = key[j] - at.base < at.len;
        const uint64_t who = __builtin_amdgcn_ballot_w64(in);
        if (who == 0) continue;
        const uint32_t to = __builtin_amdgcn_mbcnt_hi((uint32_t)(who >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)who, mine));
        if (in) list[to & (kFewKeys - 1u)] = key[j];
        mine += (uint32_t)__builtin_popcountll(who);
    }
    if (lane == 0) xch[Xch::kLeft + wave] = mine;
    __syncthreads();
    uint32_t slot = lane, from = 0;                // the lane's key: `slot` of wavefront `from`
#pragma unroll
    for (int w = 0; w + 1 < W; ++w) {
        const uint32_t theirs = (uint32_t)__builtin_amdgcn_readfirstlane((int)xch[Xch::kLeft + w]);
        const bool behind = from == (uint32_t)w && slot >= theirs;
        slot = behind ? slot - theirs : slot;
        from = behind ? w + 1u : from;
    }
    const uint32_t my = xch[Xch::kList + from * kFewKeys + (slot & (kFewKeys - 1u))];
    uint32_t below = 0;
    for (uint32_t i = 0; i < at.count; ++i)
        below += (uint32_t)__builtin_amdgcn_readlane((int)my, (int)i) < my ? 1u : 0u;
    return wave_max(lane < at.count && below < at.rank ? my : 0u);
}

// What the old state's smallest level becomes without a gradient, in the steps of ema_param(): no key is
// smaller (but by rounding, where the base is next to 1).  0 for a block without a state, and where the newest gradient is so
// large a part of the 2nd EMA, (1 - beta2) / (1 - beta2^t), that it carries the quantile out of the first pass's
// quarter octave: in the first steps and with a small beta2.  2^25 elements, 2-bit/3-bit bf16, late steps, with | without
// the floor, us: beta2 0.9 70 | 83, 0.85 85 | 87, 0.8 92 | 77, 0.5 80 | 74; beta2 0.999, steps 7-9 of a fresh state
// 82 | 73, 10-12 73 | 74, 13-16 65 | 74.  So the line lies at 0.1.
template <int BV, bool EXT>
__device__ __forceinline__ uint32_t key_floor(const StepArgs &a, const float *const my_tv)
{
    const float low = my_tv[(1 << BV) - 1], key = a.beta2 * low;
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)(low > 0.0f && a.settled ? f2u(EXT ? key + a.eps_state : key) : 0u));
}

// Elements of block `blk` that exist, and the rank of the quantile among them.
__device__ __forceinline__ uint32_t present_in(const uint64_t n, const uint64_t blk)
{
    const uint64_t left = n - blk * kBigBlock;
    return left < (uint64_t)kBigBlock ? (uint32_t)left : (uint32_t)kBigBlock;
}
__device__ __forceinline__ uint32_t rank_among(const StepArgs &a, const uint32_t present)
{
    if (present == (uint32_t)kBigBlock) return a.rank_full;
    const float x = __builtin_ceilf(a.quantile_p * (float)present);
    const uint32_t rank = x < 1.0f ? 1u : (uint32_t)x;
    return rank > present ? present : rank;
}

// The whole step for block `blk` of 2048 elements, executed by the two wavefronts of the calling
// workgroup.  What is done once per lane and block (level tables, the two divisions, the base, the
// hash of a group of eight) is spread over 16 elements.
// TAIL: also the shorter last block of a buffer.  It takes the same way with a few corrections under
// branches that are uniform for a wavefront: absent
// elements are read as zeros with the codes of a zero 1st moment, get no key, and their fields of the last
// code word are cleared again.  (Bounds checks on every element, instead, cost the full blocks of
// the same kernel registers: with fp32 gradients and the variants 106 instead of 96, i.e. four
// wavefronts per SIMD instead of five; 2-bit/3-bit AdaBelief, 42.7 million
// elements: 114 us, 108 now.)
// The variants run full blocks by this form, too: two copies of them would spill.  The plain step has a copy
// for full blocks without the corrections (2-bit/3-bit bf16: 97 us by the one form, 93 with the copy).
template <int BM, int BV, bool BF16, bool MDE, bool EXT, bool TAIL>
__device__ __forceinline__ void step_block(const StepArgs &a, const uint64_t blk, const uint32_t lane,
                                           const uint32_t wave, uint32_t *const slab, uint32_t *const work,
                                           uint32_t *const xch, const DeTable<BM, MDE, kBigWaves * 64> &de)
{
    constexpr int L = (1 << (BM - 1)) - 1;
    constexpr bool kDeTable = MDE && BM >= 3;
    using Xch = BigExchange<kBigWaves>;

    const uint64_t ew0 = blk * kBigBlock + (uint64_t)wave * kIter16;  // first element of this wavefront
    const uint32_t present = TAIL ? present_in(a.n, blk) : (uint32_t)kBigBlock, before = wave * kIter16;
    const uint32_t here = !TAIL ? (uint32_t)kIter16 : present <= before ? 0u : umin(present - before, (uint32_t)kIter16);  // of this wavefront
    const uint32_t mine = here <= lane * 16u ? 0u : umin(here - lane * 16u, 16u);                                           // of this lane
    uint32_t *const img_m = slab + BigLayout::kOffImgM, *const img_v = slab + BigLayout::kOffImgV;
    float *const my_tv = reinterpret_cast<float *>(slab + BigLayout::kOffTv);
    float *const my_tm = reinterpret_cast<float *>(slab + BigLayout::kOffTm);
    const uint32_t tv_addr = lds_addr(my_tv), tm_addr = lds_addr(my_tm);

    // ---- loads: parameters and gradients, the wavefront's code words, the block's scalars
    MomentCodes16<BM, MDE> mw;
    VarianceCodes16<BV> vw;
    mw.template load<!TAIL>(a.m_words, ew0, lane, here);
    vw.template load<!TAIL>(a.v_words, ew0, lane, here);
    const float dm_old = a.m_scale[blk], dv_old = a.v_scale[blk], al_old = a.v_base[blk];
    const RawPG16<BF16> raw = load_pg16<BF16>(a, ew0, lane, here);
    const float gscale = (EXT && a.grad_scale) ? *a.grad_scale : 1.0f;
    const Stage16 st(reinterpret_cast<float4 *>(work + wave * BigLayout::kStage), lane);
    de.store();                                    // (read behind the barrier of the maxima)
    mw.stage(img_m, lane);
    vw.stage(img_v, lane);

    // ---- level tables of the block (every wavefront its own copy)
    fill_level_tables<BM, BV, MDE, 64, false>(my_tv, my_tm, lane, dm_old, dv_old, al_old);
    wave_lds_sync();
    uint32_t mc8[2], vc8[2];
    mw.codes(img_m, lane, mc8);
    vw.codes(img_v, lane, vc8);
    uint32_t decode8[2] = {mc8[0], mc8[1]};
    if (__builtin_expect(here != kIter16, 0)) {                         // (code L is level 0 of either codebook)
        constexpr uint32_t kZeroCodes = (uint32_t)((uint64_t)L * (((1ull << (8 * BM)) - 1ull) / ((1ull << BM) - 1ull)));
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const uint32_t run = mine <= 8u * r ? 0u : umin(mine - 8u * r, 8u), keep = (uint32_t)((1ull << (BM * run)) - 1ull);
            decode8[r] = (mc8[r] & keep) | (kZeroCodes & ~keep);
        }
    }

    const uint32_t floor = key_floor<BV, EXT>(a, my_tv);

    // ---- coalesced layout -> 16 consecutive elements per lane
    float p[16], g[16];
    lane_layout16<BF16>(raw, st, p, g);
    if (EXT) {
#pragma unroll
        for (int j = 0; j < 16; ++j) g[j] = __builtin_fmaf(a.l2, p[j], g[j] * gscale);
    }

    // ---- dequantize (table look-up), EMA, parameter; new parameters streamed out
    float mh[16], vh[16];
    float m_absmax, v_max;
    ema_param<16, BM, BV, EXT, false, true>(a, tm_addr, tv_addr, decode8, vc8, nullptr, p, g, mh, vh, m_absmax, v_max);
    store_params16<EXT>(a, ew0, lane, p, st, here);
    if (__builtin_expect(here != kIter16, 0)) {                         // (kNoKey is a NaN: its code is whatever encode16() removes)
        v_max = 0.0f;
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            v_max = (uint32_t)j < mine ? __builtin_fmaxf(v_max, vh[j]) : v_max;
            vh[j] = (uint32_t)j < mine ? vh[j] : u2f(kNoKey);
        }
    }

    // ---- the work area becomes the histograms of the selection: a wavefront clears its own staging
    // area (it is done with it; the other may still be using its own)
    {
        uint4 *const own = reinterpret_cast<uint4 *>(work + wave * BigLayout::kStage);
        wave_lds_sync();
        constexpr int kOwn = BigLayout::kStage / 4;                                     // 128-bit words
#pragma unroll
        for (int i = 0; i < (kOwn + 63) / 64; ++i)
            if (lane + 64u * (uint32_t)i < (uint32_t)kOwn) own[lane + 64u * (uint32_t)i] = make_uint4(0, 0, 0, 0);
    }

    // ---- block maxima over the two wavefronts
    {
        const uint32_t wm_max = wave_max(f2u(m_absmax)), wv_max = wave_max(f2u(v_max));
        if (lane == 0) { xch[Xch::kMaxM + wave] = wm_max; xch[Xch::kMaxV + wave] = wv_max; }
    }
    __syncthreads();

    // ---- the r-th smallest v^ of the block
    uint32_t key[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) key[j] = f2u(vh[j]);
    const uint32_t xp_bits = select_rank<16, kBigWaves, false>(key, floor, rank_among(a, present), present, lane, wave, work, xch);
    float dm = u2f(umax(xch[Xch::kMaxM], xch[Xch::kMaxM + 1])), dv = u2f(largest_key<kBigWaves>(xch));
    if (dm < kTiny) dm = 0.0f;
    if (dv < kTiny) dv = 0.0f;

    // ---- encoder constants (every 16 lanes for themselves), codes, the wavefront's words
    const uint32_t lig = lane & 15u, gshift = lane & 16u;
    uint32_t de_base = 0;
    if (kDeTable) de_base = lds_addr(de.lds) - 16u * DeBuckets<BM>::kLo;
    const BlockCodec codec = block_codec<BV, 16, L, MDE>(xp_bits, dm, dv, lane, lig, gshift);
    uint32_t m8[2], v8[2];
    encode16<BM, BV, MDE>(a, ew0, lane, mh, vh, codec, de_base, mw, vw, img_m, img_v, mc8, vc8, m8, v8,
                          here == kIter16, mine);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    mw.template write_back<!TAIL>(img_m, lane, m8);
    vw.template write_back<!TAIL>(img_v, lane, v8);
    if (wave == 0 && lane == 0) { a.m_scale[blk] = dm; a.v_scale[blk] = dv; a.v_base[blk] = codec.alpha; }
}

// The same by four wavefronts, 8 consecutive elements per lane, where a launch is all latency: half
// as long a chain in every lane, and parameters and gradients that are not turned around through
// LDS.  TAIL: the shorter last block, with bounds checks.  (1000 elements, 2-bit/3-bit bf16: 8.8 us by
// the two wavefronts with bounds checks on every element, 5.4 by this form; 1,000,003: 9.7 and 7.1.)
constexpr int kQuadWaves = kBigBlock / kIter;
struct QuadLayout {
    static constexpr int kOffImgM = 0;                        // per wavefront: its words of each code stream
    static constexpr int kOffImgV = LaneCodes8<3, true>::kImage;
    static constexpr int kOffTv = 144;                        // level tables, 64-byte aligned
    static constexpr int kOffTm = 160;
    static constexpr int kSlab = 176;
};
static_assert(2 * LaneCodes8<3, true>::kImage <= QuadLayout::kOffTv, "images");

// The parameters are made behind the selection, out of the chain of the block, but for TAIL in front of it: the kernel for tables runs that form for all
// blocks, in launches of thousands of them too, and with eight values less alive across the selection it takes 64-68 registers instead of 74-85, seven or eight
// wavefronts per SIMD instead of five or six.  (4000 tensors of 1000 elements, behind | in front, us: 2-bit/3-bit bf16 23.8 | 22.7, 4-bit/2-bit DE fp32 24.5 | 23.2,
// 3-bit/3-bit DE bf16 with a copy 25.4 | 24.6; 20 tensors, 1000 blocks 9.67 | 9.92, 10.98 | 11.19; 1,000,003 elements 6.78 | 6.66.)
template <int BM, int BV, bool BF16, bool MDE, bool EXT, bool TAIL>
__device__ __forceinline__ void step_block_quad(const StepArgs &a, const uint64_t blk, const uint32_t lane,
                                                const uint32_t wave, uint32_t *const slab, uint32_t *const work,
                                                uint32_t *const xch, const DeTable<BM, MDE, kQuadWaves * 64> &de)
{
    constexpr int L = (1 << (BM - 1)) - 1;
    constexpr bool kDeTable = MDE && BM >= 3;
    using Xch = BigExchange<kQuadWaves>;

    const uint64_t ew0 = blk * kBigBlock + (uint64_t)wave * kIter;    // first element of this wavefront
    const uint64_t e0 = ew0 + lane * 8u;                              // first element of this lane
    const uint32_t present = TAIL ? present_in(a.n, blk) : (uint32_t)kBigBlock;
    uint32_t *const img_m = slab + QuadLayout::kOffImgM, *const img_v = slab + QuadLayout::kOffImgV;
    float *const my_tv = reinterpret_cast<float *>(slab + QuadLayout::kOffTv);
    float *const my_tm = reinterpret_cast<float *>(slab + QuadLayout::kOffTm);
    const uint32_t tv_addr = lds_addr(my_tv), tm_addr = lds_addr(my_tm);
    bool ok[8];                                    // the lane's elements that exist
#pragma unroll
    for (int j = 0; j < 8; ++j) ok[j] = !TAIL || e0 + j < a.n;

    // ---- every load is issued before the first one is waited for; the histogram is cleared meanwhile
    LaneCodes8<BM, TAIL> mw;
    LaneCodes8<BV, TAIL> vw;
    mw.load(a.m_words, a.n, ew0, lane);
    vw.load(a.v_words, a.n, ew0, lane);
    const float dm_old = a.m_scale[blk], dv_old = a.v_scale[blk], al_old = a.v_base[blk];
    const RawPG raw = load_pg<BF16, TAIL>(a, e0, ok[7]);
    const float gscale = (EXT && a.grad_scale) ? *a.grad_scale : 1.0f;
    {
        uint4 *const z = reinterpret_cast<uint4 *>(work);
#pragma unroll
        for (uint32_t i = 0; i < 512u / (64u * kQuadWaves); ++i) z[wave * 64u + lane + 64u * kQuadWaves * i] = make_uint4(0, 0, 0, 0);
    }
    uint32_t xi_word[1];
    XiGroups(a, ew0).words<1>(a, lane, xi_word);
    XiRun xi(a, xi_word[0]);
    xi.X = fresh(xi.X); xi.Y = fresh(xi.Y);
    mw.clear(img_m, lane);
    vw.clear(img_v, lane);
    de.store();
    fill_level_tables<BM, BV, MDE, 64, true>(my_tv, my_tm, lane, dm_old, dv_old, al_old);
    wave_lds_sync();
    const uint32_t mc8 = mw.codes(lane), vc8 = vw.codes(lane);
    const uint32_t floor = key_floor<BV, EXT>(a, my_tv);
    __syncthreads();                               // (the histogram is cleared, the DE table is there)

    // ---- dequantize (table look-up), EMA, parameter
    float p[8], g[8];
    unpack_pg<BF16>(raw, p, g);
    if (EXT) {
#pragma unroll
        for (int j = 0; j < 8; ++j) g[j] = __builtin_fmaf(a.l2, p[j], g[j] * gscale);
    }
    float mh[8], vh[8];
    float m_absmax, v_max;
    ema_param<8, BM, BV, EXT, TAIL, true>(a, tm_addr, tv_addr, &mc8, &vc8, ok, p, g, mh, vh, m_absmax, v_max);
    if (TAIL) {
        new_param8(a, mh, vh, p);
        store_params8<EXT, TAIL>(a, e0, ok[7], ok, p);
    }

    // ---- block maxima over the four wavefronts (read behind the selection's barriers)
    {
        const uint32_t wm_max = wave_max(f2u(m_absmax)), wv_max = wave_max(f2u(v_max));
        if (lane == 0) { xch[Xch::kMaxM + wave] = wm_max; xch[Xch::kMaxV + wave] = wv_max; }
    }

    // ---- the r-th smallest v^ of the block
    uint32_t key[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) key[j] = ok[j] ? f2u(vh[j]) : kNoKey;
    const uint32_t xp_bits = select_rank<8, kQuadWaves, true>(key, floor, rank_among(a, present), present, lane, wave, work, xch);
    if (!TAIL) {
        new_param8(a, mh, vh, p);
        store_params8<EXT, TAIL>(a, e0, ok[7], ok, p);
    }
    float dm = u2f(umax(umax(xch[Xch::kMaxM], xch[Xch::kMaxM + 1]), umax(xch[Xch::kMaxM + 2], xch[Xch::kMaxM + 3])));
    float dv = u2f(largest_key<kQuadWaves>(xch));
    if (dm < kTiny) dm = 0.0f;
    if (dv < kTiny) dv = 0.0f;

    // ---- encoder constants (every 16 lanes for themselves), codes, the wavefront's words
    const uint32_t lig = lane & 15u, gshift = lane & 16u;
    uint32_t de_base = 0;
    if (kDeTable) de_base = lds_addr(de.lds) - 16u * DeBuckets<BM>::kLo;
    const BlockCodec codec = block_codec<BV, 16, L, MDE>(xp_bits, dm, dv, lane, lig, gshift);
    uint32_t m8, v8;
    encode_run<BM, BV, MDE, TAIL>(xi, mh, vh, ok, codec, de_base, m8, v8);
    mw.change(img_m, lane, mc8, m8);
    vw.change(img_v, lane, vc8, v8);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    mw.write_back(img_m, lane, m8);
    vw.write_back(img_v, lane, v8);
    if (wave == 0 && lane == 0) { a.m_scale[blk] = dm; a.v_scale[blk] = dv; a.v_base[blk] = codec.alpha; }
}

// (Two wavefronts per block: five per SIMD, 79-96 registers, and LDS allows six; four: six to eight, 60-74 registers, and LDS allows thirteen.  The
// plain forms of the table kernel hold both forms of a block and spill 16 bytes per lane in 19 of 36 instantiations, 32 in three.)

#define SOLO_BIG_LDS(WAVES_, WORK_, SLAB_)                                                             \
    constexpr int kDeWords = de_words<BM, MDE>();                                                      \
    __shared__ __attribute__((aligned(64))) uint32_t lds_work[WORK_];                                  \
    __shared__ __attribute__((aligned(64))) uint32_t lds_slab[WAVES_ * SLAB_];                         \
    __shared__ __attribute__((aligned(64))) uint32_t lds_xch[BigExchange<WAVES_>::kWords];             \
    __shared__ __attribute__((aligned(64))) uint32_t lds_de[kDeWords];                                 \
    const DeTable<BM, MDE, WAVES_ * 64> de(lds_de);                                                    \
    const uint32_t lane = threadIdx.x & 63u;                                                           \
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));           \
    uint32_t *const slab = lds_slab + wave * SLAB_

// The kernel's arguments (BEHIND bytes behind the first one), loaded behind this point: loaded in front of the branch between the two forms of a
// block, the union of what they need of them is spilled for the full blocks, too.
template <typename T, int BEHIND = 0>
__device__ __forceinline__ T arguments_here()
{
    typedef const __attribute__((address_space(4))) T arg_t;
    typedef const __attribute__((address_space(4))) char byte_t;
    arg_t *p = (arg_t *)((byte_t *)__builtin_amdgcn_kernarg_segment_ptr() + BEHIND);
    asm volatile("" : "+s"(p));
    T a;
    __builtin_memcpy(&a, (const T *)p, sizeof(T));
    return a;
}

// One workgroup of two wavefronts per block; the shorter last block, if there is one, is block 0 of
// the grid.
template <int BM, int BV, bool BF16, bool MDE, bool EXT>
__global__ __launch_bounds__(kBigWaves * 64, kMinWaves)
void big_kernel(const StepArgs args)
{
    SOLO_BIG_LDS(kBigWaves, BigLayout::kWork, BigLayout::kSlab);
    const uint32_t ragged = (uint32_t)args.rest;
    if (EXT) {                                     // (see step_block)
        const uint64_t blk = blockIdx.x < ragged ? args.n / kBigBlock : blockIdx.x - ragged;
        step_block<BM, BV, BF16, MDE, EXT, true>(args, blk, lane, wave, slab, lds_work, lds_xch, de);
    } else if (blockIdx.x < ragged) {
        const StepArgs a = arguments_here<StepArgs>();
        step_block<BM, BV, BF16, MDE, EXT, true>(a, a.n / kBigBlock, lane, wave, slab, lds_work, lds_xch, de);
    } else {
        const StepArgs a = arguments_here<StepArgs>();
        step_block<BM, BV, BF16, MDE, EXT, false>(a, blockIdx.x - ragged, lane, wave, slab, lds_work, lds_xch, de);
    }
}

// Four wavefronts per block.
template <int BM, int BV, bool BF16, bool MDE, bool EXT>
__global__ __launch_bounds__(kQuadWaves * 64, kMinWaves)
void big_quad_kernel(SOLO_FIRST_ARGS, const StepRest)
{
    SOLO_BIG_LDS(kQuadWaves, 2048, QuadLayout::kSlab);
    if (blockIdx.x < whole) {
        const StepArgs a = all_args<kBigBlock>(arguments_here<StepRest, kFirstArgsBytes>(), whole, more, grad, m_words, v_words, m_scale,
                                               v_scale, v_base);
        step_block_quad<BM, BV, BF16, MDE, EXT, false>(a, blockIdx.x, lane, wave, slab, lds_work, lds_xch, de);
    } else {
        const StepArgs a = all_args<kBigBlock>(arguments_here<StepRest, kFirstArgsBytes>(), whole, more, grad, m_words, v_words, m_scale,
                                               v_scale, v_base);
        step_block_quad<BM, BV, BF16, MDE, EXT, true>(a, blockIdx.x, lane, wave, slab, lds_work, lds_xch, de);
    }
}

// The step over many tensors in one launch, blocks of 2048 elements.  The map of the table holds
// one entry per block of every tensor (the tensor's index; a shorter last block is flagged).
// Blocks never span tensors.
template <int BM, int BV, bool BF16, bool MDE, bool EXT>
__global__ __launch_bounds__(kBigWaves * 64, kMinWaves)
void multi_big_kernel(const MultiArgs args)
{
    const uint32_t me = args.unit_map[blockIdx.x];              // uniform: scalar loads
    SOLO_BIG_LDS(kBigWaves, BigLayout::kWork, BigLayout::kSlab);
    const MultiArgs ma = arguments_here<MultiArgs>();
    const TensorEntry &e = ma.entries[me & kMapTensorMask];
    const uint64_t blk = blockIdx.x - e.unit0;
    if (EXT || (me & kMapRagged))
        step_block<BM, BV, BF16, MDE, EXT, true>(tensor_args(ma, e), blk, lane, wave, slab, lds_work, lds_xch, de);
    else
        step_block<BM, BV, BF16, MDE, EXT, false>(tensor_args(ma, e), blk, lane, wave, slab, lds_work, lds_xch, de);
}

template <int BM, int BV, bool BF16, bool MDE, bool EXT>
__global__ __launch_bounds__(kQuadWaves * 64, kMinWaves)
void multi_big_quad_kernel(const MultiArgs ma)
{
    const TensorEntry &e = ma.entries[ma.unit_map[blockIdx.x] & kMapTensorMask];
    SOLO_BIG_LDS(kQuadWaves, 2048, QuadLayout::kSlab);
    step_block_quad<BM, BV, BF16, MDE, EXT, true>(tensor_args(ma, e), blockIdx.x - e.unit0, lane, wave, slab, lds_work, lds_xch, de);
}
#undef SOLO_BIG_LDS

// Up to how many blocks a launch gives four wavefronts to each: with few blocks the time is the
// chain of one, which four make shorter; the two-wavefront form has the fewer instructions and reads whole lines.  Measured on MI355X,
// us per launch, four | two wavefronts per block, three states in turn:
//   blocks                             1            128          488          750           1000          1200           1500
//   2-bit/3-bit bf16                   4.81 | 6.41  5.64 | 8.17  6.53 | 8.86  7.56 | 9.44   8.56 | 10.24  9.47 | 11.36   10.45 | 13.06
//   2-bit/3-bit AdaBelief fp32         5.05 | 7.30  6.04 | 8.07  7.30 | 9.65  8.27 | 10.41  9.28 | 11.03  10.61 | 12.66  12.11 | 14.88
//   4-bit/2-bit DE fp32                5.23 | 6.87  6.32 | 8.11  7.37 | 9.37  8.40 | 10.05  9.55 | 11.09  10.94 | 12.85  12.28 | 14.82
//   2-bit/2-bit bf16, p 0.3            4.53 | 6.33  5.58 | 7.63  6.55 | 8.51  7.47 | 9.10   8.42 | 9.92   9.31 | 11.25   10.29 | 13.02
//   3-bit/3-bit DE bf16, copy          5.34 | 7.82  6.17 | 9.08  7.20 | 9.95  8.25 | 10.57  9.18 | 11.16  10.22 | 12.44  13.43 | 14.61
//   time of four over time of two, geometric mean of these five, states of 0.7 GB in turn / three in turn / one again and again / behind 512 MB of other writes:
//   488 blocks .75 .75 .77 .80,  750 .79 .81 .84 .86,  1000 .82 .84 .89 .93,  1200 .81 .83 .86 .94,  1500 .82 .82 .84 .98
//   (With earlier kernels the two crossed between 1000 and 1800 blocks, tables first.  The line is four workgroups on each CU, the last size with a margin
//   behind other writes too, where AdaBelief is behind by 3 % already.)
//   Tables of 1000-element tensors, a block each, three in turn: 500 of them 7.3 | 10.2, 1100 9.8 | 12.7, 2000 14.1 | 16.1, 4000 22.7 | 27.3, 4-bit/2-bit DE fp32 23.2 | 29.0,
//   so a table of which at least three in four blocks are the only one of their tensor takes four at any size.
constexpr uint64_t kQuadUpTo = 1024;
constexpr bool quad_table(uint64_t blocks, uint64_t tensors) { return blocks <= kQuadUpTo || 4 * blocks <= 5 * tensors; }

template <int BM, bool MDE>
hipError_t launch_multi_big(uint32_t bits_v, bool bf16, const MultiArgs &args, hipStream_t stream);

template <int BM, bool MDE>
hipError_t launch_multi_big_impl(uint32_t bits_v, bool bf16, const MultiArgs &args, hipStream_t stream)
{
    if (args.total_units == 0 || args.count == 0) return hipErrorInvalidValue;
    const bool quad = quad_table(args.total_units, args.count);
    const uint32_t threads = (quad ? kQuadWaves : kBigWaves) * 64;
    if (args.total_units > 0xFFFFFFFFull / threads) return hipErrorInvalidValue;
    const StepArgs &c = args.common;
    const bool ext = args.any_bf16_copy || c.grad_scale || c.belief || c.l2 != 0.0f;
#define SOLO_LAUNCH(BV_, BF_)                                                                       \
    return launch(quad ? ext ? multi_big_quad_kernel<BM, BV_, BF_, MDE, true> : multi_big_quad_kernel<BM, BV_, BF_, MDE, false> \
                       : ext ? multi_big_kernel<BM, BV_, BF_, MDE, true> : multi_big_kernel<BM, BV_, BF_, MDE, false>,          \
                  (uint32_t)args.total_units, threads, stream, args)
#define SOLO_CASE(BV_) if (bits_v == BV_) { if (bf16) SOLO_LAUNCH(BV_, true); else SOLO_LAUNCH(BV_, false); }
    SOLO_CASE(2) SOLO_CASE(3) SOLO_CASE(4)
#undef SOLO_CASE
#undef SOLO_LAUNCH
    return hipErrorInvalidValue;
}

template <int BM, bool MDE>
hipError_t launch_big(uint32_t bits_v, bool bf16, const StepArgs &args, hipStream_t stream);

template <int BM, bool MDE>
hipError_t launch_big_impl(uint32_t bits_v, bool bf16, const StepArgs &args_in, hipStream_t stream)
{
    StepArgs args = args_in;
    const uint64_t blocks = (args.n + kBigBlock - 1) / kBigBlock;
    const bool quad = blocks <= kQuadUpTo;
    const uint32_t threads = (quad ? kQuadWaves : kBigWaves) * 64;
    if (blocks == 0 || blocks > 0xFFFFFFFFull / threads) return hipErrorInvalidValue;
    args.rest = args.n % kBigBlock ? 1 : 0;
    const bool ext = args.param_bf16 || args.grad_scale || args.belief || args.l2 != 0.0f;
#define SOLO_LAUNCH(BV_, BF_)                                                                       \
    return quad ? launch(ext ? big_quad_kernel<BM, BV_, BF_, MDE, true> : big_quad_kernel<BM, BV_, BF_, MDE, false>, (uint32_t)blocks, threads, stream, \
                         (uint32_t)(args.n / kBigBlock), (uint32_t)(args.n % kBigBlock), args.grad, args.m_words, args.v_words,             \
                         args.m_scale, args.v_scale, args.v_base, args)                             \
                : launch(ext ? big_kernel<BM, BV_, BF_, MDE, true> : big_kernel<BM, BV_, BF_, MDE, false>, (uint32_t)blocks, threads, stream, args)
#define SOLO_CASE(BV_) if (bits_v == BV_) { if (bf16) SOLO_LAUNCH(BV_, true); else SOLO_LAUNCH(BV_, false); }
    SOLO_CASE(2) SOLO_CASE(3) SOLO_CASE(4)
#undef SOLO_CASE
#undef SOLO_LAUNCH
    return hipErrorInvalidValue;
}

}  // namespace solo

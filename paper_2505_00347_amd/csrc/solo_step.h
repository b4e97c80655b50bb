// Device code of the fused SOLO AdamW step for gfx950 (wave64).
//
// Work decomposition.  A wavefront steps one chunk of consecutive elements on its own, from the
// first load to the last store: 1024 elements, 16 per lane (step_chunk16), or 512, 8 per lane
// (step_chunk8).  A block of 128 (64) elements is held by 8 (4) or 16 (8) neighbouring lanes, i.e.
// by half a DPP row or a row, and every per-block reduction is a few DPP steps.  Nothing is shared
// between wavefronts but a constant table: the only workgroup barrier, with dynamic-exponent codes
// of 3 and 4 bits, waits for that table while the elements' loads are under way.  No software prefetch: 70-96 registers (a few forms 105) leave room for five or six
// wavefronts per SIMD, which hide each other's memory latency, and the whole machine sweeps one
// compact window of memory.
//
// Which of the two: what is done once per lane and block (level tables, maxima, divisions, the
// base, the hash, packing) is spread over twice as many elements with 16 per lane, so that form
// needs fewer instructions, and its accesses fill whole lines: the faster one where the memory is the bound, from
// about 5 * 10^6 elements on; a shorter buffer takes the latency of a wavefront or a few one after the other, and
// 8 elements per lane have the shorter one (narrow_buffer()).  The ragged end of a
// buffer always runs the 8-per-lane form with bounds checks.  chunk8_kernel and chunk16_kernel run
// over a flat buffer, multi_chunk8_kernel and multi_chunk16_kernel over the tensors of a
// caller-built table.
//
// (Measured against one wavefront that walks a super-tile of 5120 elements in five iterations
// and prefetches one iteration ahead, the form of the large bf16 buffers before: 2^24 elements
// 2-bit/3-bit 41.8 -> 34.5 us, 2^28 elements 582 -> 520 us; at 6.7e9 elements, where HBM is the bound,
// no difference: 13.27 and 13.29 ms.)
//
// The pieces that these functions and the large-block functions of solo_step_big.h have in common
// (layout transposition, level tables, EMAs and parameter, encoders, code words) exist once, as
// inlined helpers in front of them.
//
// Large launches are bound by HBM, those of 10^6 to 10^8 elements by HBM, the last-level cache and vector issue alike,
// shorter ones by the latency of a wavefront, where every instruction counts.  What one costs (cycles of issue of a wavefront,
// measured with eight per SIMD): an fp32 add, multiplication or fused multiply-add, and / or / xor / bitop3, a right
// shift and an integer add 2.3-2.7, with a scalar register as an operand 4.4, a transcendental function 8.3, everything else
// 4.3.  (Packed FP32 is off.)  Everything below is shaped by that:
//   * both dequantizers are table look-ups: the lanes of a group compute the
//     block's level tables (alpha^q * Delta_v, (c-L) * Delta_m/L) once and park
//     them in LDS; an element costs one shift, one bitop3 and
//     one ds_read per moment; the launch's constants are in vector registers;
//   * the p-quantile is exact: each lane sorts its 8 or 16 values with min3/med3/max3
//     and merges; 8 per lane goes on to merge lanes, with as many of the smallest keys as the rank asks for
//     (merged_rth()); with 16, the group runs rounds of "row minimum by DPP, the
//     lowest lane that holds it pops its column"; scalar instructions pick
//     that lane for all groups, ties or not; it keeps the eight smallest of a lane for small ranks and
//     pops two of them at a time while the rank allows it;
//   * the two per-block divisions share one IEEE division sequence (even lanes
//     divide x_p by Delta_v, odd lanes L by Delta_m);
//   * the base alpha = rho^(1/K) is found by testing 16 consecutive binary32
//     candidates around a hardware exp2/log2 guess, spread over the group's lanes;
//   * 1st-moment codes are rounded by adding 1.5 * 2^23 and accumulated by shift and add; two 2nd-moment
//     codes share a conversion to binary16 that rounds down, a minimum and a dot product;
//   * xi is built as a float by one
//     bit-align of the element's finalized word of the xi stream (one hash
//     per 8 elements gives a start and a stride, every word is then mixed
//     on its own).
//
// Arithmetic contract (what makes the stored bytes reproducible): every value
// that decides a code or a scale is computed in binary32, one rounding per
// operation in a fixed order, no contraction except the two explicit fused
// multiply-adds of the EMAs.  Only the 2nd-moment code decision uses the
// hardware log2 (a result can differ from another implementation at an exact
// rounding tie), and the parameter update uses the hardware sqrt/rcp.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace solo {

constexpr int kTileUnit = 2560;    // lcm of the block sizes and of 16, 10 and 8 codes per word
constexpr int kIter = 512;         // elements of a chunk with 8 per lane
constexpr int kIter16 = 1024;      // elements of a chunk with 16 per lane
constexpr int kWaves = 4;          // wavefronts per workgroup
constexpr int kMinWaves = 5;       // wavefronts per SIMD that the register allocator must leave room for, 8 elements per lane
constexpr int kMinWaves16 = 4;     // and 16 per lane (70-80 registers, i.e. six, in two of three formats, 99-105, i.e. four, in eight; forcing six spills in the others)
constexpr int kColStride16 = 18;   // words per lane of the sorted columns (16 keys, two +inf; written 8 bytes at a time)
constexpr float kTiny = 0x1p-100f; // block maxima below this are stored as 0
constexpr float kRhoMin = 0x1p-64f;
constexpr uint32_t kInfBits = 0x7F800000u;
constexpr uint32_t kOneBits = 0x3F800000u;

// What the first loads of a wavefront do not need (SOLO_FIRST_ARGS).  (Apart, so that a launch copies 160 bytes of arguments instead of 224: in
// long runs of calls of 4096 elements the host takes 4.35 instead of 4.60 us for one.)
struct StepRest {
    float *param;
    uint64_t index_offset;  // global index of element 0 (multiple of 8)
    float beta1, omb1, beta2, omb2;
    float decay;            // 1 - lr * weight_decay
    float denom_scale;      // (1 / sqrt(1 - beta2^t)) / step_size, step_size = lr / (1 - beta1^t)
    float denom_eps;        // eps / step_size  (lr == 0: scale 0 and eps +inf, the update vanishes)
    float quantile_p;
    uint32_t rank_full;     // rank of the quantile in a full block
    uint32_t key0, key1, key2;
    uint32_t stochastic;    // 0: xi = 0
    // variants of the step (all uniform over the launch)
    uint16_t *param_bf16;   // bf16 copy of the new parameters, written beside them (null: none)
    const float *grad_scale;// device scalar every gradient is multiplied by first (null: 1)
    float l2;               // Adam with coupled decay: weight_decay, g <- g + l2 * p; otherwise 0
    float eps_state;        // AdaBelief: eps, added to the 2nd EMA itself at every step
    uint32_t belief;        // AdaBelief: the 2nd EMA follows (g - m^)^2 instead of g^2
    uint32_t settled;       // the newest gradient is a small part of the 2nd EMA (blocks of 2048: key_floor())
};

struct StepArgs : StepRest {
    const void *grad;
    uint32_t *m_words;
    float *m_scale;
    uint32_t *v_words;
    float *v_scale;
    float *v_base;
    uint64_t n;             // elements
    uint64_t rest;          // 512-element iterations behind the last whole chunk, up to the end of the last code word
};

// One tensor of a multi-tensor launch, as the kernel reads it from the caller's table
// (device memory; built on the host by solo_multi_table_build).
struct TensorEntry {
    float *param;
    uint16_t *param_bf16;   // may be null
    const void *grad;
    uint32_t *m_words;
    float *m_scale;
    uint32_t *v_words;
    float *v_scale;
    float *v_base;
    uint64_t n;             // elements of the tensor
    uint64_t unit0;         // index of the tensor's first unit among all units of the table
    uint64_t index_offset;  // global index of the tensor's element 0 in the xi stream
    uint32_t first16;       // pieces (pieces16) of the tensors before this one
    uint32_t first8;        // 512-element pieces of the tensors before this one
};
static_assert(sizeof(TensorEntry) == 96, "table layout");

// An entry of the unit map: the tensor's index; for the ragged end of a tensor, which has one entry
// per 512 elements, also the number of that entry and a flag.  (Blocks of 64 and 128 are cut into pieces,
// see find_tensor(): there the map is a first guess only.)
constexpr uint32_t kMapTensorMask = 0x00FFFFFFu, kMapRagged = 0x80000000u;
constexpr int kMapChunkShift = 24;
inline uint64_t multi_full_units(uint64_t n, uint64_t unit) { return n / unit; }
inline uint64_t multi_ragged_chunks(uint64_t n, uint64_t unit)
{
    return n % unit ? ((n + 79) / 80 * 80 - n / unit * unit + 511) / 512 : 0;      // (end_of_words)
}

struct MultiArgs {
    StepArgs common;              // the scalars of the step; pointers, n and index_offset come from the table
    const TensorEntry *entries;
    const uint32_t *unit_map;     // tensor index of every unit
    uint64_t total_units;
    uint64_t pieces;              // blocks of 64 and 128: of all tensors (0: the caller does not know)
    float units_per_piece;
    uint32_t count;               // tensors
    uint32_t any_bf16_copy;       // some tensor of the table has a bf16 copy to write
};

// The units of a multi-tensor table (what a map entry stands for).  fp32 gradients with the linear
// codebook: one entry per 2560 elements, a tensor's shorter end included.  Every other format: one
// entry per full unit of 5120 or 2560 elements, and one per 512-element iteration of a ragged end.
constexpr bool multi_chunked(bool bf16, bool mde) { return !bf16 && !mde; }
constexpr int unit_elems(uint32_t bits_m, uint32_t bits_v, uint32_t block_size)
{
    return bits_m + bits_v <= (block_size == 128 ? 6u : 5u) ? 2 * kTileUnit : kTileUnit;
}

// Elements up to the end of the last code word of n elements (80 = lcm of 16, 10 and 8 codes per
// word): a word's unused fields are written as zeros like every other field.
__host__ __device__ constexpr uint64_t end_of_words(uint64_t n) { return (n + 79) / 80 * 80; }

// The pieces that n elements are cut into, one wavefront each: whole chunks of 1024 and, for what is
// left behind them, up to three of 512; or 512 elements each.
__host__ __device__ constexpr uint64_t rest_pieces(uint64_t n, uint64_t whole)
{
    return n == whole * kIter16 ? 0 : (end_of_words(n) - whole * kIter16 + kIter - 1) / kIter;
}
__host__ __device__ constexpr uint64_t pieces16(uint64_t n) { return n / kIter16 + rest_pieces(n, n / kIter16); }
__host__ __device__ constexpr uint64_t pieces8(uint64_t n) { return n % kIter ? rest_pieces(n, 0) : n / kIter; }
// A unit of a table holds at most so many pieces (5120 elements: five, 2560 or a shorter end: three).
constexpr uint64_t kPiecesPerUnit = 5;
// Workgroups of a launch: the grid counts its work-items in 32 bits.
constexpr uint64_t kMaxGroups = 0xFFFFFFFFull / (kWaves * 64);

// ---------------------------------------------------------------- cross-lane

template <int CTRL>
__device__ __forceinline__ uint32_t dpp(uint32_t x)
{
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, CTRL, 0xF, 0xF, true);   // (every lane has a source: no old value to set up)
}

// Butterfly over the G (4, 8 or 16) lanes that hold one block: lane^1 and lane^2
// by quad permutes, then mirror inside the half row, then inside the row.
// Every lane ends with the result of its whole group.
template <int G, typename Op>
__device__ __forceinline__ uint32_t group_reduce(uint32_t x, Op op)
{
    x = op(x, dpp<0xB1>(x));    // quad_perm [1,0,3,2]
    x = op(x, dpp<0x4E>(x));    // quad_perm [2,3,0,1]
    if (G >= 8) x = op(x, dpp<0x141>(x));   // row_half_mirror
    if (G == 16) x = op(x, dpp<0x140>(x));  // row_mirror
    return x;
}

struct UMin { __device__ __forceinline__ uint32_t operator()(uint32_t a, uint32_t b) const { return a < b ? a : b; } };
struct UMax { __device__ __forceinline__ uint32_t operator()(uint32_t a, uint32_t b) const { return a > b ? a : b; } };

__device__ __forceinline__ uint32_t f2u(float x) { return __builtin_bit_cast(uint32_t, x); }
__device__ __forceinline__ float u2f(uint32_t x) { return __builtin_bit_cast(float, x); }
__device__ __forceinline__ uint32_t umin(uint32_t a, uint32_t b) { return a < b ? a : b; }
__device__ __forceinline__ uint32_t umax(uint32_t a, uint32_t b) { return a > b ? a : b; }
__device__ __forceinline__ uint64_t umin64(uint64_t a, uint64_t b) { return a < b ? a : b; }
// Median of three bit patterns of non-negative floats (they order like the floats).
__device__ __forceinline__ uint32_t umed3(uint32_t a, uint32_t b, uint32_t c)
{
    return f2u(__builtin_amdgcn_fmed3f(u2f(a), u2f(b), u2f(c)));
}

// (x & mask) | base as one two-cycle instruction (v_and_or_b32 takes four).
__device__ __forceinline__ uint32_t and_or(uint32_t x, uint32_t mask, uint32_t base)
{
    return __builtin_amdgcn_bitop3_b32(x, mask, base, 0xEA);
}

// The bits of a wave-wide ballot that belong to this lane's group, shifted down.
__device__ __forceinline__ uint32_t group_bits(uint64_t ballot, uint32_t lane, uint32_t gshift, uint32_t gmask)
{
    const uint32_t half = lane < 32u ? (uint32_t)ballot : (uint32_t)(ballot >> 32);
    return (half >> gshift) & gmask;
}

// (The larger key is what the exclusive or of all three leaves: two cycles instead of the four of a second comparison,
// whose shorter chain makes no difference where a launch is all latency.)
__device__ __forceinline__ void cswap(uint32_t &a, uint32_t &b)
{
    const uint32_t lo = umin(a, b), hi = __builtin_amdgcn_bitop3_b32(a, b, lo, 0x96);
    a = lo; b = hi;
}

// Sorts four keys with seven instructions: a three-sort (min3, med3, max3),
// then the fourth key is placed by one min, two med3 and one max.
__device__ __forceinline__ void sort4(uint32_t &a, uint32_t &b, uint32_t &c, uint32_t &d)
{
    const uint32_t lo = umin(umin(a, b), c), mid = umed3(a, b, c), hi = umax(umax(a, b), c);
    a = umin(lo, d); b = umed3(lo, mid, d); c = umed3(mid, hi, d); d = umax(hi, d);
}

// Eight keys: two four-sorts and Batcher's odd-even merge of the halves.
__device__ __forceinline__ void sort8(uint32_t (&k)[8])
{
    sort4(k[0], k[1], k[2], k[3]);
    sort4(k[4], k[5], k[6], k[7]);
    cswap(k[0], k[4]); cswap(k[1], k[5]); cswap(k[2], k[6]); cswap(k[3], k[7]);
    cswap(k[2], k[4]); cswap(k[3], k[5]);
    cswap(k[1], k[2]); cswap(k[3], k[4]); cswap(k[5], k[6]);
}

// ------------------------------------------------------------------- pieces

__device__ __forceinline__ uint32_t mix32(uint32_t h)
{
    h ^= h >> 16; h *= 0x85EBCA6Bu;
    h ^= h >> 13; h *= 0xC2B2AE35u;
    h ^= h >> 16;
    return h;
}

// Finalizer of an element's word of the xi stream: the group's words X + j Y lie on an arithmetic
// progression; xorshift and one 24-bit multiplication (full rate; the low 24 bits of the
// xorshifted word contain every bit of w) make the eight elements of a group jointly independent.
constexpr uint32_t kXiMul = 0xC2B2AFu;
__host__ __device__ constexpr uint32_t xi_finalize_ref(uint32_t w)
{
    return ((w ^ (w >> 15)) & 0xFFFFFFu) * kXiMul;
}
__device__ __forceinline__ uint32_t xi_finalize(uint32_t w)
{
    return __umul24(w ^ (w >> 15), kXiMul);
}
// A word whose finalized top 23 bits are 100...0, i.e. xi = 0 (deterministic rounding).
constexpr uint32_t kXiZeroWord = 0x1B29A9u;
static_assert((xi_finalize_ref(kXiZeroWord) >> 9) == 0x400000u, "xi = 0 word");

// Level alpha^q of the log codebook for a run-time q, by binary powering in the
// dequantizer's fixed order: the selected powers a, a^2, a^4, a^8 are
// multiplied from the lowest bit of q up.
template <int BV>
__device__ __forceinline__ float log_level(uint32_t q, float P1, float P2, float P4, float P8)
{
    float y = (q & 1u) ? P1 : 1.0f;
    y = (q & 2u) ? y * P2 : y;
    if (BV >= 3) y = (q & 4u) ? y * P4 : y;
    if (BV >= 4) y = (q & 8u) ? y * P8 : y;
    return y;
}

// Last level alpha^K, K = 2^BV - 1: ((a * a^2) * a^4) * a^8.
template <int BV>
__device__ __forceinline__ float last_level(float a)
{
    const float a2 = a * a;
    float r = a * a2;
    if (BV >= 3) { const float a4 = a2 * a2; r = r * a4; if (BV >= 4) { const float a8 = a4 * a4; r = r * a8; } }
    return r;
}

// Walks y (bits of a binary32 in (0, 1]) to the largest value whose last level
// does not exceed rho.  Both walks are bounded; used only when the parallel
// candidate test did not bracket the answer.
template <int BV>
__device__ __noinline__ uint32_t walk_base(uint32_t y, float rho)
{
    for (int i = 0; i < 4096 && last_level<BV>(u2f(y)) > rho; ++i) --y;
    for (int i = 0; i < 4096 && y < kOneBits && last_level<BV>(u2f(y + 1)) <= rho; ++i) ++y;
    return y;
}

// The base alpha = rho^(1/K) as stored: the largest binary32 whose last level does not exceed rho.
// The hardware exp2/log2 give a guess that is a few units in the last place off; the lanes of the
// group test the 16 consecutive binary32 values yb - 8 .. yb + 7 around it in parallel (one per
// lane in a group of 16, two or four per lane in a group of 8 or 4) and count those that fit.  Only a guess
// further off than that takes the bounded walk.  Returns the bit pattern; meaningful if rho < 1.
template <int BV, int G>
__device__ __forceinline__ uint32_t search_base(float rho, bool need, uint32_t lane, uint32_t lig, uint32_t gshift)
{
    constexpr int K = (1 << BV) - 1;
    constexpr float invK = 1.0f / (float)K;
    constexpr uint32_t GMASK = (1u << G) - 1u;
    static_assert(G == 4 || G == 8 || G == 16, "group of 4, 8 or 16 lanes");
    const float y0 = __builtin_amdgcn_exp2f(__builtin_amdgcn_logf(rho) * invK);
    const uint32_t yb = umed3(f2u(y0), 0x00800000u, kOneBits);
    uint32_t cnt;
    if (G == 16) {
        const uint32_t cand = umin(yb + lig - 8u, kOneBits);
        const bool fits = last_level<BV>(u2f(cand)) <= rho;
        cnt = (uint32_t)__builtin_popcount(group_bits(__builtin_amdgcn_ballot_w64(fits), lane, gshift, GMASK));
    } else {                                   // 16 / G candidates per lane
        cnt = 0;
#pragma unroll
        for (int c = 0; c < 16 / G; ++c) {
            const uint32_t cand = umin(yb + lig + (uint32_t)(c * G) - 8u, kOneBits);
            const bool fits = last_level<BV>(u2f(cand)) <= rho;
            cnt += (uint32_t)__builtin_popcount(group_bits(__builtin_amdgcn_ballot_w64(fits), lane, gshift, GMASK));
        }
    }
    uint32_t ab = umin(yb + cnt - 9u, kOneBits);
    // not bracketed (all or none of the candidates fit): walk from the nearest end
    const bool open = need && (cnt == 0u || cnt == 16u);
    if (__builtin_amdgcn_ballot_w64(open) != 0) {
        if (open) ab = walk_base<BV>(cnt == 0u ? yb - 8u : ab, rho);
    }
    return ab;
}

// A value that the compiler does not connect with what it has computed from `x` before: cheap arithmetic is then
// done again instead of being kept in registers.
__device__ __forceinline__ uint32_t fresh(uint32_t x)
{
    asm("" : "+v"(x));
    return x;
}

// A run of eight 3-bit codes that starts at slot `s` (0-9) of a word: `shift` = 3 s; the run may continue in the
// word behind it.
struct Run3 {
    uint32_t word, shift;
    // q: code index of the run's first code from the first staged word on (< 1040)
    __device__ __forceinline__ explicit Run3(const uint32_t q)
    {
        word = __umul24(q, 52429u) >> 19;          // q / 10
        shift = 3u * q - 30u * word;
    }
    // (the two bits of a word that no code owns are ignored)
    __device__ __forceinline__ uint32_t codes(const uint32_t w0, const uint32_t w1) const
    {
        return ((w0 & 0x3FFFFFFFu) >> shift | w1 << (30u - shift)) & 0xFFFFFFu;
    }
    // changes codes by exclusive or: what lanes that share a word own of it stays
    __device__ __forceinline__ void change(uint32_t *const img, const uint32_t x) const
    {
        atomicXor(&img[word], (x << shift) & 0x3FFFFFFFu);
        atomicXor(&img[word + 1], x >> (30u - shift));
    }
};

// Signed dynamic-exponent (DE) levels of the 1st moment (App. A of the paper): the first bit
// is the sign, the other b-1 bits spend E leading zeros on the exponent 10^-E, one indicator
// bit, and the rest on a linear fraction over [0.1, 1].  Exponent step i (scale 10^(-(b-2)+i))
// owns 2^i fraction cells, each represented by the mean of its boundaries, and the two codes
// left over are the levels 0 and 1.  Non-negative levels in increasing order:
// pos(0) = 0, pos(1..L) the cell means, pos(L+1) = 1, L = 2^(b-1) - 1; the negative side
// mirrors pos(1..L) (there is no level -1).
template <int BM>
struct DeLevels {
    static constexpr int L = (1 << (BM - 1)) - 1;
    static constexpr double pos(int j)
    {
        if (j <= 0) return 0.0;
        if (j > L) return 1.0;
        constexpr double tenth[8] = {1.0, 0.1, 0.01, 0.001, 1e-4, 1e-5, 1e-6, 1e-7};
        int i = 0, first = 1;                       // exponent step i holds cells [first, first + 2^i)
        while (j >= first + (1 << i)) { first += (1 << i); ++i; }
        const int cells = 1 << i, c = j - first;
        const double lo = 0.1 + 0.9 * (double)c / (double)cells;
        const double hi = 0.1 + 0.9 * (double)(c + 1) / (double)cells;
        return tenth[(BM - 2) - i] * (lo + hi) / 2.0;
    }
    // Tables evaluated at compile time: the signed levels by code (2L + 2 of them) and the
    // midpoints between neighbouring non-negative levels (the rounding boundaries of |z|).
    struct Tables {
        float level[2 * L + 2];
        float mid[L + 1];
        constexpr Tables() : level(), mid()
        {
            for (int c = 0; c < 2 * L + 2; ++c) level[c] = c >= L ? (float)pos(c - L) : -(float)pos(L - c);
            for (int k = 0; k <= L; ++k) mid[k] = (float)((pos(k) + pos(k + 1)) / 2.0);
        }
    };
    static constexpr Tables tab = Tables();
    // level of a run-time code (used once per wavefront): a select chain over literals
    __device__ static float level(uint32_t code)
    {
        float r = 0.0f;
#pragma unroll
        for (int c = 0; c < 2 * L + 2; ++c) r = (code == (uint32_t)c) ? tab.level[c] : r;
        return r;
    }
};

// Rounding to the DE levels by one table look-up.  |z| <= 1 is cut into buckets by the top of
// its binary32 pattern (the exponent and two fraction bits); the buckets are narrow enough that
// none holds more than one rounding boundary, so a bucket knows the two neighbouring codes its
// values can take.  One 8-byte entry per bucket and sign, { t, base }: the code is
// base + (z > t).  For z >= 0, t is the boundary and base the code at or below it.  For z < 0
// the code falls as |z| grows, so base is the code beyond the boundary and t = -nextup(boundary):
// z > t exactly when |z| <= boundary.  Buckets without a boundary (and the negative buckets
// beyond the last negative level) have t = +inf.  Entry 0 also serves every smaller magnitude.
template <int BM>
struct DeBuckets {
    static constexpr int L = DeLevels<BM>::L;
    static constexpr uint32_t bucket(float x) { return (__builtin_bit_cast(uint32_t, x) >> 21) & 0x3FFu; }
    static constexpr uint32_t kLo = bucket(DeLevels<BM>::tab.mid[0]) - 1u;
    static constexpr uint32_t kHi = bucket(1.0f);       // |z| can reach 1 + 2^-23
    static constexpr int N = (int)(kHi - kLo) + 1;
    struct Table {
        uint32_t w[2 * N][2];
        bool one_boundary_per_bucket;
        constexpr Table() : w(), one_boundary_per_bucket(true)
        {
            constexpr uint32_t kInf = 0x7F800000u;
            for (int b = 0; b < N; ++b) {
                int below = 0, inside = 0;              // boundaries in lower buckets / in this one
                uint32_t thr = kInf;
                for (int k = 0; k <= L; ++k) {
                    const uint32_t bk = bucket(DeLevels<BM>::tab.mid[k]);
                    if (bk < kLo + (uint32_t)b) ++below;
                    if (bk == kLo + (uint32_t)b) { ++inside; thr = __builtin_bit_cast(uint32_t, DeLevels<BM>::tab.mid[k]); }
                }
                if (inside > 1) one_boundary_per_bucket = false;
                const int j0 = below, j1 = below + inside;
                w[2 * b][0] = thr;                                       // z >= 0
                w[2 * b][1] = (uint32_t)(L + j0);
                const int n0 = L - (j0 < L ? j0 : L), n1 = L - (j1 < L ? j1 : L);   // z < 0: no level -1
                w[2 * b + 1][0] = n0 != n1 ? ((thr + 1u) | 0x80000000u) : kInf;
                w[2 * b + 1][1] = (uint32_t)n1;
            }
        }
    };
    static constexpr Table tab = Table();
    static_assert(tab.one_boundary_per_bucket, "two fraction bits must separate the boundaries");
};

// ------------------------------------------------------------------- kernel

// LDS accessed through 32-bit byte addresses, so that a table index can be
// OR-ed into an aligned base with one v_and_or_b32.
typedef __attribute__((address_space(3))) float lds_f32_t;
typedef __attribute__((address_space(3))) uint32_t lds_u32_t;
__device__ __forceinline__ uint32_t lds_addr(const void *p)
{
    return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void *)p;
}
__device__ __forceinline__ float lds_f32(uint32_t addr) { return *(lds_f32_t *)(uintptr_t)addr; }
__device__ __forceinline__ uint32_t lds_u32(uint32_t addr) { return *(lds_u32_t *)(uintptr_t)addr; }

// Streaming accesses: 128-bit, every instruction covers one contiguous kilobyte of the
// wavefront's chunk, non-temporal (nothing of p or g is touched twice).
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
typedef uint16_t u16x2_t __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) u32x2_t lds_u32x2_t;
__device__ __forceinline__ float4 stream_load_f4(const float *p)
{
    const f32x4_t v = __builtin_nontemporal_load(reinterpret_cast<const f32x4_t *>(p));
    return make_float4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ uint4 stream_load_u4(const void *p)
{
    const u32x4_t v = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t *>(p));
    return make_uint4(v.x, v.y, v.z, v.w);
}
// Streaming stores are non-temporal and written through at device scope (sc1): the data leaves
// the L2 at once instead of waiting for an eviction, which drains the write stream more evenly
// (0.5-1 % on the whole step over a plain non-temporal store).
// (Written as assembly because no builtin sets sc1.  The compiler keeps the distances that its own stores need but does not
// look inside an asm block: the s_nop in front is the five wait states between a vector instruction that
// writes a scalar register, a lane read for instance, and an access of memory that reads it as its base; the one behind is the
// two that a store of more than 64 bits needs before its data registers may be overwritten.)
// `base`: uniform over the wavefront; `at`: bytes behind it, per lane; OFFSET: of the instruction.  (One
// 32-bit register per lane addresses all stores of a chunk, instead of a 64-bit address for each.)
template <int OFFSET>
__device__ __forceinline__ void stream_store_f4(void *const base, const uint32_t at, float4 x)
{
    static_assert(OFFSET >= 0 && OFFSET < 4096, "offset of a global access");
    const u32x4_t v = {__builtin_bit_cast(uint32_t, x.x), __builtin_bit_cast(uint32_t, x.y),
                       __builtin_bit_cast(uint32_t, x.z), __builtin_bit_cast(uint32_t, x.w)};
    asm volatile("s_nop 4\n\tglobal_store_dwordx4 %0, %1, %2 offset:%3 sc1 nt\n\ts_nop 1" ::"v"(at), "v"(v), "s"(base), "n"(OFFSET) : "memory");
}

// Two binary32 values rounded to bfloat16 (nearest, ties to even: the hardware conversion),
// the first in the low half.
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi)
{
    const bf16x2_t v = {(__bf16)lo, (__bf16)hi};
    return __builtin_bit_cast(uint32_t, v);
}

// Parameters and gradients of a lane's 8 consecutive elements: two (bf16 gradients: one) 16-byte
// accesses per lane and stream.  A wavefront's access then covers every other 16 bytes of its two
// kilobytes, twice the requests of a coalesced one, but nothing has to be turned around through LDS:
// the code for 8 elements per lane runs where a launch is all latency (the transposition and its
// waits were 500 of the 6400-7200 cycles of a wavefront).  TAIL: unless `whole` says that
// all of them exist, element by element; a caller asks for a wavefront, whose loads
// are then all under way at once, or for every lane.  ALONE: the last element again in place of those that don't exist: under conditions the loads wait for each other,
// which a short launch feels (100,003 elements 2-bit/2-bit B 64, us in a graph: 3.95 | 3.45 with the last one again).  What a long buffer or a table has behind its
// chunks of 1024 runs between wavefronts that wait for memory anyway, and sixteen loads per lane at once go in front of theirs: there every lane whose elements all exist loads
// vectors, and the one that holds the end loads under conditions.  (Tables, 2-bit/3-bit bf16, conditions for every lane | the last one again | this, us: 256 tensors,
// 4.4 million elements 14.40 | 14.95 | 14.47, 20 tensors of them 14.73 | 15.09 | 14.72, 1000 tensors of 12.5 million 30.15 | 30.75 | 28.96, 4000 tensors of 12.2 million 37.97 | 36.12 | 33.50.)
// The parameters last: nothing needs them before the step's end (states out of HBM, in front | behind, us: 2^20 elements 4-bit/4-bit fp32 6.22 | 5.90,
// 3-bit/3-bit 5.90 | 5.59; out of the last-level cache the same).  And past the caches: a step mostly runs behind other work, whose written lines still fill the
// last-level cache, and a load that allocates there waits for one of them to be written back.  (Behind 512 MB of other writes, kernel time in us, through the
// caches | past them: 2^20 elements 4-bit/4-bit fp32 6.7 | 5.8, 3-bit/3-bit 6.8 | 5.5, 5 million 2-bit/3-bit bf16 20.9 | 16.9, 4-bit/4-bit fp32 AdaBelief 22.6 | 20.7, 2 million
// in blocks of 2048 13.0 | 10.9; states out of HBM in turn 2^20 4-bit/4-bit fp32 5.4 | 5.0; the same buffers again and again 4.30 | 4.35, 5 million 13.8 | 13.2.)
// PAST: bf16 gradients, too (in blocks of 128 and 64: behind other writes, parameters only | both, us: 2.5 million elements 2-bit/3-bit 11.1 | 10.3, 5 million 16.9 | 16.0;
// states in turn 7.1 | 7.3, 12.3 | 12.6).  Not fp32 ones (20.7 | 18.0, but three states in turn 14.6 | 15.8), nor in blocks of 2048 (8.6 | 8.7 and 9.2 | 9.6 in turn, 10.7 | 10.7 and 12.2 | 12.0).
struct RawPG { float4 p0, p1; uint4 g0, g1; };

template <bool BF16, bool TAIL, bool ALONE = true, bool PAST = false>
__device__ __forceinline__ RawPG load_pg(const StepArgs &a, const uint64_t e0, const bool whole)
{
    RawPG r;
    r.g1 = make_uint4(0, 0, 0, 0);
    if (!TAIL || whole) {
        if (BF16) {
            const u32x4_t *const gp = reinterpret_cast<const u32x4_t *>(static_cast<const uint16_t *>(a.grad) + e0);
            const u32x4_t halves = PAST ? __builtin_nontemporal_load(gp) : *gp;
            r.g0 = make_uint4(halves.x, halves.y, halves.z, halves.w);
        } else {
            const uint4 *gp = reinterpret_cast<const uint4 *>(static_cast<const float *>(a.grad) + e0);
            r.g0 = gp[0]; r.g1 = gp[1];
        }
        // (nothing so far has to wait for a scalar load, and the scheduler must not change that: 2^20 elements out of HBM, us, without | with:
        // 4-bit/4-bit fp32 5.89 | 5.43, 3-bit/3-bit 5.64 | 5.38, 2-bit/3-bit bf16 5.14 | 4.91)
        __builtin_amdgcn_sched_barrier(0);
        const f32x4_t *const pp = reinterpret_cast<const f32x4_t *>(a.param + e0);
        const f32x4_t low = __builtin_nontemporal_load(pp), high = __builtin_nontemporal_load(pp + 1);
        r.p0 = make_float4(low.x, low.y, low.z, low.w); r.p1 = make_float4(high.x, high.y, high.z, high.w);
    } else {
        float p[8]; uint32_t g[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const uint64_t e = ALONE ? umin64(e0 + j, a.n - 1u) : e0 + j;
            p[j] = 0.0f; g[j] = 0u;
            if (!ALONE && e >= a.n) continue;
            p[j] = a.param[e];
            if (BF16) g[j] = static_cast<const uint16_t *>(a.grad)[e];
            else      g[j] = static_cast<const uint32_t *>(a.grad)[e];
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            if (ALONE && e0 + j >= a.n) { p[j] = 0.0f; g[j] = 0u; }
        }
        r.p0 = make_float4(p[0], p[1], p[2], p[3]); r.p1 = make_float4(p[4], p[5], p[6], p[7]);
        if (BF16) r.g0 = make_uint4(g[0] | (g[1] << 16), g[2] | (g[3] << 16), g[4] | (g[5] << 16), g[6] | (g[7] << 16));
        else      { r.g0 = make_uint4(g[0], g[1], g[2], g[3]); r.g1 = make_uint4(g[4], g[5], g[6], g[7]); }
    }
    return r;
}

// A launch constant in a vector register.  With eight wavefronts per SIMD, MI355X issues an fp32 add,
// multiplication or fused multiply-add, an and / or / xor / bitop3, a right shift and an integer add of a
// wavefront in 2.3-2.7 cycles, but in 4.4 where an operand is a scalar register (everything else, min, max,
// conversions, left shifts and DPP among it, takes 4.3 in any case, the transcendental functions 8.3).
// The moments of an element had six such operands: with them in vector registers, and the two table addresses
// by bitop3, the 1024 elements of a wavefront take 3414 instead of 3616 cycles of issue (2-bit/3-bit bf16).
// (The block of assembly is empty and only hides that the value is the constant: the move in front of it is the
// compiler's own, which keeps the two wait states behind a vector instruction that writes the scalar register, a lane
// read that reloads a spilled one for instance.  Those it does not keep for a move inside the block.)
template <typename T>
__device__ __forceinline__ T in_vector(T x)
{
    asm("" : "+v"(x));
    return x;
}

// Wave-level ordering point for LDS traffic between lanes of one wavefront (LDS executes a
// wavefront's operations in order; this only stops the compiler from moving them).
__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

template <int BM>
constexpr int m_table_stride() { return BM == 2 ? 4 : BM == 3 ? 8 : 16; }   // a power of two >= the entries of a block's m table

// Words of the workgroup's DE bucket table (rounding by two boundaries: compares are cheaper).
template <int BM, bool MDE>
constexpr int de_words() { return MDE && BM >= 3 ? 4 * DeBuckets<BM>::N : 16; }

// Whether a flat buffer runs 8 elements per lane; `copy`: a bf16 copy of the parameters is written.  8 per lane starts sooner and takes no transposition
// through LDS, 16 needs fewer instructions and fills whole lines with every access, all of them past the caches, so 16 wins where the memory is the bound.  Measured on
// MI355X, time of 8 over time of 16: steps in a row (geometric mean of one state again and again, three in turn and states of 0.7 GB in turn) | a step behind
// other work that has written 512 MB:
//   elements / 2^18                 2            4            5            6            8            10           12           16           20           24           28
//   2-bit/3-bit bf16                .75 | .96    .81 | 1.06   .77 | 1.03   .78 | 1.02   .85 | 1.10   .81 | 1.02   .88 | 1.04   .92 | 1.07   .92 | 1.08   .97 | 1.14   .97 | 1.11
//   3-bit/3-bit DE bf16             .72 | 1.00   .78 | 1.10   .78 | 1.10   .78 | 1.08   .81 | 1.06   .81 | 1.05   .85 | 1.05   .90 | 1.12   .90 | 1.10   .96 | 1.14   .95 | 1.09
//   3-bit/4-bit bf16, B 64          .75 | .85    .83 | .97    .78 | .95    .79 | .95    .85 | .97    .82 | .91    .87 | .95    .93 | 1.02   .93 | 1.04   .98 | 1.05   .97 | 1.06
//   2-bit/3-bit bf16, copy          .78 | 1.10   .85 | 1.15   .82 | 1.14   .82 | 1.14   .90 | 1.17   .87 | 1.09   .94 | 1.09   .98 | 1.10   .97 | 1.12   1.00 | 1.13  1.00 | 1.08
//   2-bit/3-bit bf16, rank 39       .70 | .87    .78 | 1.00   .76 | 1.04   .76 | 1.04   .84 | 1.08   .79 | 1.01   .86 | 1.05   .92 | 1.08   .91 | 1.10   .97 | 1.16   .97 | 1.11
//   2-bit/2-bit bf16, B 64, rank 20 .71 | .70    .81 | .84    .77 | .85    .80 | .82    .89 | .89    .84 | .85    .90 | .89    .97 | .98    .95 | 1.00   1.00 | 1.05  1.01 | 1.06
//   2-bit/3-bit bf16, rank 39, copy .72 | 1.02   .81 | 1.05   .79 | 1.08   .79 | 1.09   .85 | 1.09   .82 | 1.05   .90 | 1.07   .94 | 1.07   .95 | 1.10   .98 | 1.12   .98 | 1.08
//   4-bit/4-bit fp32                .77 | 1.06   .83 | 1.19   .77 | 1.11   .76 | 1.09   .82 | 1.17   .78 | 1.17   .83 | 1.23   .93 | 1.25   .92 | 1.25   .95 | 1.26   .98 | 1.26
//   4-bit/4-bit fp32, AdaBelief     .76 | 1.10   .86 | 1.20   .80 | 1.14   .78 | 1.11   .85 | 1.18   .81 | 1.13   .86 | 1.19   .94 | 1.25   .93 | 1.23   .97 | 1.26   .97 | 1.23
//   2-bit/4-bit fp32, copy          .78 | .93    .87 | 1.02   .80 | 1.06   .80 | 1.07   .87 | 1.13   .83 | 1.08   .91 | 1.13   .95 | 1.17   .94 | 1.18   .96 | 1.19   .96 | 1.18
//   4-bit/4-bit fp32, rank 39       .68 | 1.03   .77 | 1.14   .73 | 1.10   .72 | 1.07   .78 | 1.14   .74 | 1.10   .80 | 1.15   .88 | 1.19   .88 | 1.22   .92 | 1.21   .94 | 1.22
// In a row 8 is ahead up to 24 * 2^18 or farther, also out of HBM; behind other work, whose written lines a load that allocates in the last-level cache has to wait
// for, it falls behind by 2 to 10 % from 4 * 2^18 on with bf16 gradients (8 to 17 % with a copy) and 10 to 25 % with fp32 ones.  A step of an optimizer is the one or
// the other, by how much of a model one call takes; a line lies where the mean of the four crosses 1.  The rank of the quantile, whose lists 8 per lane
// merges, does not move it.  (With gradients and parameters through the caches 8 was behind by 40 % there, 5 million elements 2-bit/3-bit bf16 20.9 us instead of 14.6.)
constexpr bool narrow_buffer(uint64_t n, bool bf16, bool copy)
{
    return n <= (uint64_t)(bf16 && copy ? 12 : 20) << 18;
}
// Up to how many pieces (pieces16) a table does.  Time of 8 over time of 16 as above, a table of 20 tensors of uneven sizes:
//   elements / 2^18                 2            3            4            6            8            12           16
//   2-bit/3-bit bf16                .77 | .78    .82 | .81    .81 | .80    .86 | .79    .86 | .77    .85 | .80    .92 | .91
//   3-bit/4-bit bf16, B 64          .79 | .80    .84 | .85    .80 | .80    .85 | .82    .86 | .83    .86 | .84    .92 | .91
//   2-bit/3-bit bf16, copy          .79 | .84    .86 | .89    .84 | .86    .84 | .86    .88 | .85    .85 | .85    .93 | .89
//   4-bit/4-bit fp32                .79 | .88    .83 | .89    .77 | .83    .83 | .87    .82 | .92    .86 | .96    .90 | 1.05
//   2-bit/4-bit fp32, copy          .81 | .86    .87 | .96    .80 | .90    .85 | .94    .84 | .91    .86 | .94    .91 | 1.04
//   2-bit/3-bit bf16, rank 39       .74 | .74    .79 | .77    .79 | .75    .86 | .77    .86 | .77    .84 | .80    .90 | .90
// and with kernels before, in a row only, that table | one of 256 equal tensors with a ragged end each (16 per lane took 3 % longer there than it does now):
//   elements / 2^18                 6            8            12           16           24           32           40
//   2-bit/3-bit bf16                .90 | 1.04   .90 | 1.00   .93 | .94    .93 | .94    .96 | 1.01   .99 | 1.01   1.00 | 1.07
//   2-bit/3-bit bf16, copy          .86 | 1.02   .90 | .98    .90 | .92    .85 | .86    .91 | .95    .91 | .94    .95 | .97
//   4-bit/4-bit fp32                .87 | 1.04   .87 | .97    .89 | .90    .87 | .89    .90 | .96    .93 | .97    .97 | 1.03
//   2-bit/3-bit bf16, rank 39       .89 | 1.03   .89 | 1.00   .94 | .95    .95 | .94    1.00 | 1.06  1.04 | 1.09  1.07 | 1.09
// One line for all of them (the pieces are what a caller's flags say), at 16 * 2^18 elements, where fp32 gradients behind other work are 5 % behind.
constexpr uint64_t narrow_table_up_to() { return 16ull << 8; }

// The rank-th smallest key of every group of G = 4 or 8 lanes (full blocks).  Each lane has parked its
// sorted column at `haddr` (+inf behind it) and passes its four smallest keys.  A round:
// group minimum of the heads by DPP; the lowest lane that holds it pops its column, so
// exactly one key leaves a group per round and the last minimum is the order statistic, multiplicities
// included.  (That lane is the lowest set bit of every G-bit field h of a ballot, h & (~h + 1) for all fields at once: each
// has a bit set, so the addition does not carry out of a field.)  While more than G + 1 keys are asked for, a round pops two at once: the lane whose second
// key is the smallest drops both.  In front of that key there are at most its own first one and
// one of every other lane, so both are among the first G + 1.  (Rank 13 of 128: 10 rounds instead of 12; 39: 23 instead of
// 38.)  The keys behind the head are fetched a round ahead, so that their LDS latency lies outside the chain.
// One block of assembly, because a fetch is under way across the back edges: the registers it lands in are
// the block's own until its last wait.  The popping lanes run under their own exec mask; all 64 lanes are
// active in front of the block and behind it.  (A DPP operand needs two instructions between
// the vector instruction that writes it and the one that reads it.)
template <int G>
__device__ __forceinline__ uint32_t extract_rth(uint32_t head, uint32_t behind, uint32_t next, uint32_t next2,
                                                uint32_t haddr, uint32_t rank)
{
    static_assert(G == 4 || G == 8, "group of 4 or 8 lanes");
    uint32_t mn, left = (uint32_t)__builtin_amdgcn_readfirstlane((int)rank);
#define SOLO_DPP(D_, S_, CTRL_) "v_min_u32_dpp " D_ ", " S_ ", " S_ " " CTRL_ " row_mask:0xf bank_mask:0xf\n\t"
#define SOLO_MIN4(X_) SOLO_DPP("%[mn]", X_, "quad_perm:[1,0,3,2]") "s_nop 1\n\t" SOLO_DPP("%[mn]", "%[mn]", "quad_perm:[2,3,0,1]")
#define SOLO_MIN8(X_) SOLO_MIN4(X_) "s_nop 1\n\t" SOLO_DPP("%[mn]", "%[mn]", "row_half_mirror")
    // exec: of every group's lanes that hold the minimum the lowest (the literals: kOnes - 1 in two halves)
#define SOLO_HOLDERS(X_, LOW_, HIGH_) "v_cmp_eq_u32_e32 vcc, " X_ ", %[mn]\n\t"                        \
        "s_sub_u32 exec_lo, " LOW_ ", vcc_lo\n\ts_subb_u32 exec_hi, " HIGH_ ", vcc_hi\n\ts_and_b64 exec, exec, vcc\n\t"
#define SOLO_EXTRACT(MIN_, LOW_, HIGH_)                                                                   \
    asm volatile("s_sub_u32 %[left], %[left], %[more]\n\t"          /* ranks behind the first G + 1 */    \
                 "s_cmp_lt_i32 %[left], 1\n\t"                                                           \
                 "s_cbranch_scc1 .Lone%=\n"                                                             \
                 ".Lpair%=:\n\t"                                                                        \
                 MIN_("%[behind]") SOLO_HOLDERS("%[behind]", LOW_, HIGH_)                               \
                 "s_waitcnt lgkmcnt(0)\n\t"                                                             \
                 "v_mov_b32_e32 %[head], %[next]\n\t"                                                   \
                 "v_mov_b32_e32 %[behind], %[next2]\n\t"                                                \
                 "ds_read_b32 %[next], %[haddr] offset:16\n\t"                                          \
                 "ds_read_b32 %[next2], %[haddr] offset:20\n\t"                                         \
                 "v_add_u32_e32 %[haddr], 8, %[haddr]\n\t"                                              \
                 "s_mov_b64 exec, -1\n\t"                                                               \
                 "s_sub_u32 %[left], %[left], 2\n\t"                                                    \
                 "s_cmp_gt_i32 %[left], 0\n\t"                                                          \
                 "s_cbranch_scc1 .Lpair%=\n"                                                            \
                 ".Lone%=:\n\t"                                                                         \
                 "s_add_u32 %[left], %[left], %[more]\n\t"                                              \
                 "s_sub_u32 %[left], %[left], 2\n\t"                /* rounds after the first, borrow: none at all */ \
                 "s_cbranch_scc1 .Ldone%=\n"                                                            \
                 ".Lround%=:\n\t"                                                                       \
                 MIN_("%[head]") SOLO_HOLDERS("%[head]", LOW_, HIGH_)                                   \
                 "s_waitcnt lgkmcnt(0)\n\t"                                                             \
                 "v_mov_b32_e32 %[head], %[behind]\n\t"                                                 \
                 "ds_read_b32 %[behind], %[haddr] offset:8\n\t"                                         \
                 "v_add_u32_e32 %[haddr], 4, %[haddr]\n\t"                                              \
                 "s_mov_b64 exec, -1\n\t"                                                               \
                 "s_sub_u32 %[left], %[left], 1\n\t"                                                    \
                 "s_cbranch_scc0 .Lround%=\n"                                                           \
                 ".Ldone%=:\n\t"                                                                        \
                 "s_waitcnt lgkmcnt(0)\n\t"                                                             \
                 "s_nop 1"                                                                              \
                 : [head] "+v"(head), [behind] "+v"(behind), [next] "+v"(next), [next2] "+v"(next2),    \
                   [haddr] "+v"(haddr), [left] "+s"(left), [mn] "=&v"(mn)                               \
                 : [more] "n"(G + 1)                                                                    \
                 : "vcc", "scc", "memory")
    if (G == 8) SOLO_EXTRACT(SOLO_MIN8, "0x1010100", "0x1010101");
    else        SOLO_EXTRACT(SOLO_MIN4, "0x11111110", "0x11111111");
#undef SOLO_EXTRACT
#undef SOLO_HOLDERS
#undef SOLO_MIN8
#undef SOLO_MIN4
#undef SOLO_DPP
    return group_reduce<G>(head, UMin());
}

// ---- the r-th smallest of a group's keys, 8 sorted ones per lane in registers, by merging.
//
// Neighbouring sorted lists are merged bitonically, pairs of lanes first, then fours, eights and sixteens; a list
// keeps its C smallest keys only (C >= r, a power of two), so once it has C each merge halves the keys that a lane
// holds: 8, 8, 4, 2, 1 for rank 13 of 128.  A list of S = R 2^t keys lies in 2^t lanes, R to a lane in order; merging it with the
// next one is the exchange of every key with its mirror image there (the smaller half is the result where C is reached), then exchanges
// over halving distances, between lanes while the distance is R or more and inside a lane below.
// Lanes count by coordinates (lane_coordinates()) in which the exchange partner over each one is a
// single DPP pattern, and the lists of lanes with the next coordinate set are sorted the other way round, so that a
// key's mirror image lies in the partner lane.  Which of two lanes keeps the smaller key is a third operand of the
// median: 0 for the smaller, all ones for the larger.
// No scalar instruction and no exec mask is in the chain: about 100 vector instructions, most of
// them independent of each other, for rank 13 of 128, where rounds of "minimum of the heads by DPP, the lowest lane that
// holds it shifts its column" took 12 times about 170 cycles one after the other (38 times at rank 39).  us per launch in a graph, rounds |
// merges: 4096 elements 2-bit/3-bit 3.52 | 3.15, at rank 39 5.12 | 3.40; 1000 elements 4.42 | 3.67; 2^20 4-bit/4-bit fp32
// 4.87 | 4.56, 3-bit/3-bit 5.08 | 4.85; 2^19 at rank 39 5.56 | 3.77; 1000 tensors of 600 6.70 | 5.88; 5 million, where
// the number of instructions counts, 14.1 | 13.9.
// (With 16 per lane a round pops two keys, fewer lanes share a block, and the other wavefronts of the SIMD fill the gaps: extract_rth().)

// The lane whose coordinate J differs: lane ^ 1, ^ 2, ^ 7 (mirror of the half row) and ^ 8 (rotation of the row by 8).
template <int J>
__device__ __forceinline__ uint32_t across(const uint32_t x)
{
    return dpp<J == 0 ? 0xB1 : J == 1 ? 0x4E : J == 2 ? 0x141 : 0x128>(x);
}
__device__ __forceinline__ uint32_t lane_coordinates(const uint32_t lane)       // bit J: coordinate J
{
    return (lane ^ (lane & 4u ? 3u : 0u)) & 15u;
}

// One exchange over coordinate J; `sides`: bit J set in the lanes that keep the larger keys.  MIRROR: key i meets key R - 1 - i.
template <int J, bool MIRROR, int R>
__device__ __forceinline__ void exchange(uint32_t (&k)[R], const uint32_t sides)
{
    const uint32_t upper = (uint32_t)__builtin_amdgcn_sbfe((int)sides, J, 1);
    uint32_t o[R];
#pragma unroll
    for (int i = 0; i < R; ++i) o[i] = across<J>(k[MIRROR ? R - 1 - i : i]);
#pragma unroll
    for (int i = 0; i < R; ++i) k[i] = umax(umin(k[i], o[i]), umin(umax(k[i], o[i]), upper));   // (one median)
}
// Over the coordinates of ORDER (N of them, four bits each), the highest first.
template <uint32_t ORDER, int N, int R>
__device__ __forceinline__ void exchange_lanes(uint32_t (&k)[R], const uint32_t sides)
{
    if constexpr (N > 0) {
        exchange<(ORDER >> (4 * (N - 1))) & 15, false>(k, sides);
        exchange_lanes<ORDER, N - 1>(k, sides);
    }
}
template <int R>
__device__ __forceinline__ void merge_in_lane(uint32_t (&k)[R])
{
#pragma unroll
    for (int w = R / 2; w >= 1; w /= 2)
#pragma unroll
        for (int i = 0; i < R; ++i) if ((i & w) == 0) cswap(k[i], k[i + w]);
}

// From lists over 2^T lanes on (R keys per lane; their blocks of R are ordered by the N coordinates of ORDER, the lowest four bits counting
// least) to the rank-th smallest key of the group, in all its lanes.  `rank`: 1 to C, at most the group's keys.
template <int G, int C, int T = 0, uint32_t ORDER = 0, int N = 0, int R>
__device__ __forceinline__ uint32_t merged_rth(uint32_t (&k)[R], const uint32_t coords, const uint32_t rank)
{
    static_assert(R << N <= C && C <= 8 * G, "a list holds at most C keys");
    if constexpr (1 << T < G) {
        const uint32_t sides = 2 << T == G ? coords : coords ^ (uint32_t)__builtin_amdgcn_sbfe((int)coords, T + 1, 1);
        if constexpr (R << N < C) {
            exchange<T, true>(k, sides);
            exchange_lanes<ORDER, N>(k, sides);
            merge_in_lane(k);
            return merged_rth<G, C, T + 1, ORDER | T << (4 * N), N + 1>(k, coords, rank);
        } else if constexpr (R > 1) {
            uint32_t h[R / 2];
#pragma unroll
            for (int i = 0; i < R / 2; ++i) h[i] = umin(k[i], across<T>(k[R - 1 - i]));      // (the partner makes the other half)
            exchange_lanes<ORDER, N>(h, sides);
            exchange<T, true>(h, sides);
            merge_in_lane(h);
            return merged_rth<G, C, T + 1, ORDER << 4 | T, N + 1>(h, coords, rank);
        } else {
            k[0] = umin(k[0], across<T>(k[0]));                                              // (both sides hold the result)
            exchange_lanes<ORDER, N>(k, sides);
            return merged_rth<G, C, T + 1, ORDER, N>(k, coords, rank);
        }
    } else {
        const uint32_t at = rank - 1u, in_lane = at % R, block = at / R;
        uint32_t want = 0, mask = 0;
#pragma unroll
        for (int b = 0; b < N; ++b) {
            const int j = (ORDER >> (4 * b)) & 15;
            want |= (block >> b & 1u) << j;
            mask |= 1u << j;
        }
#pragma unroll
        for (int w = R / 2; w >= 1; w /= 2)
#pragma unroll
            for (int i = 0; i < w; ++i) {
                const uint32_t low = k[i], high = k[i + w];      // (values: of two elements of an array it would be their addresses that are selected)
                k[i] = in_lane & (uint32_t)w ? high : low;
            }
        return group_reduce<G>(((coords ^ want) & mask) == 0u ? k[0] : 0u, UMax());
    }
}

// The r-th smallest key of every group of G lanes (`rank`: 1 to at_most, the same or smaller in each group), 8 sorted keys per lane.
template <int G>
__device__ __forceinline__ uint32_t merged_rth8(uint32_t (&k)[8], const uint32_t lane, const uint32_t rank, const uint32_t at_most)
{
    const uint32_t coords = lane_coordinates(lane);
    if (at_most <= 8u) return merged_rth<G, 8>(k, coords, rank);
    if (at_most <= 16u) return merged_rth<G, 16>(k, coords, rank);
    if (G == 8 || at_most <= 64u) return merged_rth<G, 64>(k, coords, rank);
    return merged_rth<G, 8 * G>(k, coords, rank);
}

// The 2nd-moment code is rounded down by the conversion of code * 2^-24 to binary16 toward zero: a binary16
// below 2^-14 counts in steps of 2^-24, so its bits are the integer.
constexpr float kCodeScale = 0x1p-24f;

// Per-block constants of the two encoders, from the new block statistics.
struct BlockCodec {
    float inv_s;     // L / Delta_m (DE: 1 / Delta_m); 0 for an all-zero block
    float alpha;     // the stored base; 1 for a degenerate block
    float inv_l2a;   // kCodeScale / log2(alpha); -kCodeScale for a degenerate block
    float rdv;       // 1 / Delta_v;      0 for a degenerate block (with bias 1 the ratio is then 1)
    float bias;
};

// rho = x_p / Delta_v (even lanes) and L / Delta_m (odd lanes) share one IEEE division, then a
// quad permute hands every lane both; alpha by search_base.
template <int BV, int G, int L, bool MDE>
__device__ __forceinline__ BlockCodec block_codec(uint32_t xp_bits, float dm, float dv, uint32_t lane,
                                                  uint32_t lig, uint32_t gshift)
{
    const float num = (lane & 1u) ? (MDE ? 1.0f : (float)L) : u2f(xp_bits);
    const float den = (lane & 1u) ? dm : dv;
    const float quo = num / den;
    float rho = u2f(dpp<0xA0>(f2u(quo)));        // quad_perm [0,0,2,2]
    float inv_s = u2f(dpp<0xF5>(f2u(quo)));      // quad_perm [1,1,3,3]
    inv_s = dm > 0.0f ? inv_s : 0.0f;
    rho = dv > 0.0f ? rho : 1.0f;
    rho = rho < kRhoMin ? kRhoMin : rho;
    BlockCodec c = {inv_s, 1.0f, -kCodeScale, 0.0f, 1.0f};
    const bool need = rho < 1.0f;
    const uint32_t ab = search_base<BV, G>(rho, need, lane, lig, gshift);
    // the two reciprocals of the 2nd-moment encoder, correctly rounded, again by one shared
    // division: 1 / log2(alpha) on the even lanes, 1 / Delta_v on the odd ones (a block that
    // does not need them divides by harmless stand-ins)
    const float den2 = (lane & 1u) ? (need ? dv : 1.0f) : __builtin_amdgcn_logf(need ? u2f(ab) : 0.5f);
    const float quo2 = 1.0f / den2;
    const float inv_l2a = u2f(dpp<0xA0>(f2u(quo2)));
    const float rdv = u2f(dpp<0xF5>(f2u(quo2)));
    if (need) {
        c.alpha = u2f(ab);
        c.inv_l2a = inv_l2a * kCodeScale;          // (exact)
        c.rdv = rdv;
        c.bias = 0.0f;
    }
    return c;
}

// The xi stream of a wavefront's share: its first group of eight (`group0`, 64 bits, uniform) and what the
// groups of a lane need of the upper half of their number.
struct XiGroups {
    uint32_t low, high;        // group0's low word; key2 times its high word
    bool wraps;                // the low word wraps inside the share (of at most 128 groups)
    __device__ __forceinline__ XiGroups(const StepArgs &a, const uint64_t first_element)
    {
        const uint64_t group0 = (a.index_offset + first_element) >> 3;
        low = (uint32_t)group0;
        high = (uint32_t)(group0 >> 32) * a.key2;
        wraps = low > 0xFFFFFFFFu - 128u;
    }
    // the hash's input for the R groups from group0 + k on
    template <int R>
    __device__ __forceinline__ void words(const StepArgs &a, const uint32_t k, uint32_t (&w)[R]) const
    {
#pragma unroll
        for (int r = 0; r < R; ++r) w[r] = ((low + k + r) ^ a.key0) + high;
        if (__builtin_expect(wraps, 0)) {
#pragma unroll
            for (int r = 0; r < R; ++r) w[r] += low + k + r < k + r ? a.key2 : 0u;
        }
    }
};

// The words of a run of 8 consecutive elements in the xi stream: element j owns X + j Y (xi_finalize()).
struct XiRun {
    uint32_t X, Y;
    // word: of the run's group (XiGroups::words)
    __device__ __forceinline__ XiRun(const StepArgs &a, const uint32_t word) : X(mix32(word)), Y(mix32(X ^ a.key1) | 1u)
    {
        if (!a.stochastic) { X = kXiZeroWord; Y = 0u; }     // xi = 0: the float is 1.5
    }
};

// Encodes a lane's run of 8 consecutive elements, `xi` of the xi stream: returns the packed 1st- and 2nd-moment codes (element j in bits [b j, b j + b)).
// xi: one hashed start and stride per 8 elements, every element's word finalized on its own;
// 2^-24 * (1.5 + xi - 2^-24) is built as a float by one bit-align of the finalized word.
// m: code - L = rint(m^ * L/Delta_m) in [-L, L], rounded to an integer by adding 1.5 * 2^23, whose low
// mantissa bits it then is; the words are accumulated by shift and add, modulo 2^32, and what the
// constant contributed is taken off at the end.
// v: code + 1 = floor(log_alpha(v^/Delta_v) + 1.5 + xi) in [1, K + 1].  The ratio is clamped to 1 by
// the multiplication that makes it (an output modifier), so nothing falls below 1; two elements share the
// conversion that rounds down (kCodeScale), the packed minimum with K + 1 (+inf, v^ = 0, takes the last
// code), and the dot product that shifts them into place.
// (Against rint / floor, med3 and a fused multiply-add for every code and conversions of the sums, 2-bit/3-bit,
// 16 per lane: 3327 instead of 3414 cycles of issue per wavefront; 2^26 elements 138.4 -> 132.3 us, 4-bit/4-bit fp32
// 150.7 -> 146.2, AdaBelief 4-bit/4-bit fp32 at 5 million elements, 8 per lane, 14.9 -> 14.5.)
// `ok` (TAIL only): the elements that exist.  What is not finite spoils codes of its own run only.
template <int BM, int BV, bool MDE, bool TAIL>
__device__ __forceinline__ void encode_run(const XiRun &xi, const float *mh, const float *vh,
                                           const bool *ok, const BlockCodec &c, uint32_t de_base,
                                           uint32_t &m8, uint32_t &v8)
{
    constexpr int L = (1 << (BM - 1)) - 1;
    constexpr int K = (1 << BV) - 1;
    constexpr bool kDeTable = MDE && BM >= 3;
    uint32_t xj = xi.X;                                 // X + j Y, walked up from j = 0
    float y[8];                                         // kCodeScale * (code + 1 + fraction)
    uint32_t t[8];                                      // m: code - L in the low bits, kRound's bits above
    uint32_t m8_de = 0;
    constexpr float kRound = 0x1.8p23f;
    constexpr uint32_t kRoundBits = 0x4B400000u;
#pragma unroll
    for (int j = 0; j < 8; ++j, xj += xi.Y) {
        const float z = mh[j] * c.inv_s;
        if (!MDE) {
            t[j] = f2u(z + kRound);
            if (TAIL && !ok[j]) t[j] = kRoundBits - (uint32_t)L;
        } else {
            // DE: nearest level on the magnitude; inv_s = 1/Delta_m
            uint32_t code;
            if (kDeTable) {
                // entry of the bucket of |z| (16 bytes per bucket: z >= 0, then z < 0)
                // (clamped on both sides: a non-finite input must not leave the table)
                const uint32_t bk = umin(umax(__builtin_amdgcn_ubfe(f2u(z), 21u, 10u), DeBuckets<BM>::kLo),
                                         DeBuckets<BM>::kHi);
                const uint32_t addr = ((f2u(z) >> 28) & 8u) | ((bk << 4) + de_base);
                const u32x2_t en = *(lds_u32x2_t *)(uintptr_t)addr;
                code = en.y + (z > u2f(en.x) ? 1u : 0u);
            } else {
                // few levels: the code is the number of rounding boundaries below z.  A value
                // on a boundary keeps the level of smaller magnitude: '>' on the positive side,
                // '>=' on the negative one (z = -0 is above every negative boundary: code L).
                code = 0;
#pragma unroll
                for (int k = 0; k < L; ++k) code += (z >= -DeLevels<BM>::tab.mid[k]) ? 1u : 0u;
#pragma unroll
                for (int k = 0; k <= L; ++k) code += (z > DeLevels<BM>::tab.mid[k]) ? 1u : 0u;
            }
            if (TAIL && !ok[j]) code = 0;
            m8_de |= code << (BM * j);
        }
        const float f = u2f(__builtin_amdgcn_alignbit(0x7Fu - 24u, xi_finalize(xj), 9u));
        const float ratio = __builtin_amdgcn_fmed3f(__builtin_fmaf(vh[j], c.rdv, c.bias), 0.0f, 1.0f);
        y[j] = __builtin_fmaf(__builtin_amdgcn_logf(ratio), c.inv_l2a, f);
        if (TAIL && !ok[j]) y[j] = kCodeScale;
    }
    // a sum of v's codes below 2^16: all eight (2-bit) or four
    constexpr int kSums = BV == 2 ? 1 : 2, kPer = 4 / kSums;
    uint32_t sum[2] = {0, 0};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const u16x2_t h = __builtin_bit_cast(u16x2_t, __builtin_amdgcn_cvt_pkrtz(y[2 * i], y[2 * i + 1]));
        const u16x2_t last = {(uint16_t)(K + 1), (uint16_t)(K + 1)};
        const int at = BV * 2 * (i % kPer);
        const u16x2_t weight = {(uint16_t)(1u << at), (uint16_t)(1u << (at + BV))};
        sum[i / kPer] = __builtin_amdgcn_udot2(__builtin_elementwise_min(h, last), weight, sum[i / kPer], false);
    }
    constexpr uint32_t kOnes = (uint32_t)(((1ull << (8 * BV)) - 1ull) / ((1ull << BV) - 1ull));     // sum of 2^(BV j)
    v8 = sum[0] + (kSums == 2 ? sum[1] << (4 * BV) : 0u) - kOnes;
    if (!MDE) {
        constexpr uint32_t kFields = (uint32_t)((1ull << (8 * BM)) - 1ull);
        constexpr uint32_t kPlaces = (uint32_t)(((1ull << (8 * BM)) - 1ull) / ((1ull << BM) - 1ull));
        uint32_t acc = t[7];
#pragma unroll
        for (int j = 6; j >= 0; --j) acc = (acc << BM) + t[j];
        m8 = (acc - (kRoundBits - (uint32_t)L) * kPlaces) & kFields;
    } else {
        m8 = m8_de;
    }
}

// ---- pieces shared by the tile functions and the large-block functions (solo_step_big.h)

// The level tables of a block that G lanes share (decode by table look-up): lane `lig` of the group
// fills entries lig, lig + G, ... of the 2nd-moment table (Delta_v alpha^q, alpha^q by binary
// powering) and of the 1st-moment table (linear: (c - L) (Delta_m / L); dynamic exponent: the
// levels times Delta_m).  ALL (where a launch is all latency): lanes beyond the entries fill one again, and the linear 1st-moment table its unused last one,
// so that nothing is conditional and the code around it stays one block for the compiler's scheduler.  (With 16 elements per lane that schedule takes
// more registers, 81-88 instead of 75-80, a wavefront per SIMD less, in 23 of 288 instantiations and fewer in about as many.  2^26 elements, us, with conditions |
// without: tables 3-bit/2-bit with a copy 145.8 | 148.6, 4-bit/2-bit DE with a copy 152.6 | 157.0, 4-bit/3-bit DE fp32 149.0 | 152.7; 3-bit/4-bit with a copy 137.8 | 142.1;
// where it took fewer, 2-bit/3-bit fp32 B 64 DE with a copy 165.6 | 164.2.)
template <int BM, int BV, bool MDE, int G, bool ALL>
__device__ __forceinline__ void fill_level_tables(float *const my_tv, float *const my_tm, const uint32_t lig,
                                                  const float dm_old, const float dv_old, const float al_old)
{
    constexpr int L = (1 << (BM - 1)) - 1;
    constexpr int VT = 1 << BV, kEntries = MDE ? 2 * L + 2 : 2 * L + 1, MT = ALL ? m_table_stride<BM>() : kEntries;
    static_assert(m_table_stride<BM>() >= kEntries, "entries");
    float level[(MT + G - 1) / G];
    if (MDE) {                                 // (ALL: while the scales are under way: nothing of them is read in front of this point)
#pragma unroll
        for (int r = 0; r < (MT + G - 1) / G; ++r) {
            level[r] = DeLevels<BM>::level(ALL ? (lig + r * G) & (uint32_t)(MT - 1) : lig + r * G);
            if (ALL) asm volatile("" : "+v"(level[r]));
        }
    }
    // (The scales are here: a load whose value is used under the conditions below only would be moved behind them, and
    // its latency with it.)
    if (!ALL) asm volatile("" : : "v"(dm_old), "v"(dv_old), "v"(al_old));
    const float s_m = (L == 1) ? dm_old : dm_old / (float)L;
    const float P1 = al_old, P2 = P1 * P1, P4 = P2 * P2, P8 = P4 * P4;
#pragma unroll
    for (int r = 0; r < (VT + G - 1) / G; ++r) {
        const uint32_t q = ALL ? (lig + r * G) & (uint32_t)(VT - 1) : lig + r * G;
        if (ALL || q < VT) my_tv[q] = log_level<BV>(q, P1, P2, P4, P8) * dv_old;
    }
#pragma unroll
    for (int r = 0; r < (MT + G - 1) / G; ++r) {
        const uint32_t c = ALL ? (lig + r * G) & (uint32_t)(MT - 1) : lig + r * G;
        if (ALL || c < MT) my_tm[c] = MDE ? level[r] * dm_old : (float)((int)c - L) * s_m;
    }
}

template <bool BF16>
__device__ __forceinline__ void unpack_pg(const RawPG &raw, float (&p)[8], float (&g)[8])
{
    p[0] = raw.p0.x; p[1] = raw.p0.y; p[2] = raw.p0.z; p[3] = raw.p0.w;
    p[4] = raw.p1.x; p[5] = raw.p1.y; p[6] = raw.p1.z; p[7] = raw.p1.w;
    if (BF16) {
        g[0] = u2f(raw.g0.x << 16); g[1] = u2f(raw.g0.x & 0xFFFF0000u);
        g[2] = u2f(raw.g0.y << 16); g[3] = u2f(raw.g0.y & 0xFFFF0000u);
        g[4] = u2f(raw.g0.z << 16); g[5] = u2f(raw.g0.z & 0xFFFF0000u);
        g[6] = u2f(raw.g0.w << 16); g[7] = u2f(raw.g0.w & 0xFFFF0000u);
    } else {
        g[0] = u2f(raw.g0.x); g[1] = u2f(raw.g0.y); g[2] = u2f(raw.g0.z); g[3] = u2f(raw.g0.w);
        g[4] = u2f(raw.g1.x); g[5] = u2f(raw.g1.y); g[6] = u2f(raw.g1.z); g[7] = u2f(raw.g1.w);
    }
}

// Parameter: decoupled decay, bias-corrected Adam direction,
// p <- p * decay - step_size * m^ / (sqrt(v^ / bc2) + eps), with step_size folded into the denominator.
__device__ __forceinline__ float new_param(const float p, const float mh, const float vh, const float decay, const float denom_scale, const float denom_eps)
{
    const float denom = __builtin_fmaf(__builtin_amdgcn_sqrtf(vh), denom_scale, denom_eps);
    return __builtin_fmaf(p, decay, -(mh * __builtin_amdgcn_rcpf(denom)));
}
// Those of a lane's 8 elements, in a place where the chain of the block's statistics leaves issue slots free.
__device__ __forceinline__ void new_param8(const StepArgs &a, const float (&mh)[8], const float (&vh)[8], float (&p)[8])
{
    const float decay = in_vector(a.decay), denom_scale = in_vector(a.denom_scale), denom_eps = in_vector(a.denom_eps);
#pragma unroll
    for (int j = 0; j < 8; ++j) p[j] = new_param(p[j], mh[j], vh[j], decay, denom_scale, denom_eps);
}

// Dequantize (table look-up: byte offset 4 * code, OR-ed into the aligned table base), both EMAs
// and the parameter for a lane's N = 8 or 16 consecutive elements; mc8 / vc8: the packed old
// codes of every run of 8.  VMAX: also the largest v^ (the callers that sort take it from the
// sorted keys).  TAIL: elements that do not exist (`ok`) leave zeros in m^ and v^.
// AdaBelief without a branch: d = g - kb * m^ is g itself when kb = 0 and fl(g - m^) when kb = 1
// (one rounding either way), and eps_state = 0 leaves v^ unchanged.
// 16 per lane also makes the new parameters here; 8 per lane later (new_param8()).
template <int N, int BM, int BV, bool EXT, bool TAIL, bool VMAX>
__device__ __forceinline__ void ema_param(const StepArgs &a, const uint32_t tm_addr, const uint32_t tv_addr,
                                          const uint32_t *mc8, const uint32_t *vc8, const bool *ok,
                                          float (&p)[N], const float (&g)[N], float (&mh)[N], float (&vh)[N],
                                          float &m_absmax, float &v_max)
{
    constexpr uint32_t MIDX = ((1u << BM) - 1u) << 2, VIDX = ((1u << BV) - 1u) << 2;   // byte-index masks
    float mt[N], vt[N];
    if (N == 8) {                              // (the narrow code fetches all levels first)
#pragma unroll
        for (int j = 0; j < N; ++j) {
            const uint32_t om = (j == 0) ? (mc8[0] << 2) : (mc8[0] >> (BM * j - 2));
            const uint32_t ov = (j == 0) ? (vc8[0] << 2) : (vc8[0] >> (BV * j - 2));
            mt[j] = lds_f32(and_or(om, MIDX, tm_addr));
            vt[j] = lds_f32(and_or(ov, VIDX, tv_addr));
        }
    }
    const float beta1 = in_vector(a.beta1), omb1 = in_vector(a.omb1), beta2 = in_vector(a.beta2), omb2 = in_vector(a.omb2);
    float denom_scale = 0.0f, denom_eps = 0.0f, decay = 0.0f;
    if (N != 8) { denom_scale = in_vector(a.denom_scale); denom_eps = in_vector(a.denom_eps); decay = in_vector(a.decay); }
    m_absmax = 0.0f;
    v_max = 0.0f;
    float kb = 0.0f, eps_state = 0.0f;
    if (EXT) { kb = in_vector(a.belief ? 1.0f : 0.0f); eps_state = in_vector(a.eps_state); }
#pragma unroll
    for (int j = 0; j < N; ++j) {
        if (N != 8) {
            const int r = j / 8, jj = j % 8;
            const uint32_t om = (jj == 0) ? (mc8[r] << 2) : (mc8[r] >> (BM * jj - 2));
            const uint32_t ov = (jj == 0) ? (vc8[r] << 2) : (vc8[r] >> (BV * jj - 2));
            mt[j] = lds_f32(and_or(om, MIDX, tm_addr));
            vt[j] = lds_f32(and_or(ov, VIDX, tv_addr));
        }
        mh[j] = __builtin_fmaf(beta1, mt[j], omb1 * g[j]);
        if (EXT) {
            const float d = __builtin_fmaf(-kb, mh[j], g[j]);
            vh[j] = __builtin_fmaf(beta2, vt[j], omb2 * (d * d)) + eps_state;
        } else {
            vh[j] = __builtin_fmaf(beta2, vt[j], omb2 * (g[j] * g[j]));
        }
        if (N != 8) p[j] = new_param(p[j], mh[j], vh[j], decay, denom_scale, denom_eps);
        if (TAIL && !ok[j]) { mh[j] = 0.0f; vh[j] = 0.0f; }
        m_absmax = __builtin_fmaxf(m_absmax, __builtin_fabsf(mh[j]));
        if (VMAX) v_max = __builtin_fmaxf(v_max, vh[j]);
    }
}

// The new parameters of a lane's 8 elements and their bf16 copy, if asked for.  (Non-temporal: the lines leave the L2 as they are
// written instead of when the kernel ends.  4-bit/4-bit fp32, one state again and again, us: 2 * 2^20 elements 6.62 -> 6.45, 2.5 7.75 -> 7.34,
// 3 9.11 -> 8.41, 5 14.5 -> 13.7, 4.5 12.9 -> 13.1; three states in turn and states out of HBM +-2 %, in the mean 0.3 % less.  Written
// through at device scope, as 16 per lane does, costs 13 to 28 % here, since a store covers every other 16 bytes only.)
template <bool EXT, bool TAIL>
__device__ __forceinline__ void store_params8(const StepArgs &a, const uint64_t e0, const bool whole, const bool *ok, const float (&p)[8])
{
    if (!TAIL || whole) {
        f32x4_t *const pp = reinterpret_cast<f32x4_t *>(a.param + e0);
        const f32x4_t low = {p[0], p[1], p[2], p[3]}, high = {p[4], p[5], p[6], p[7]};
        __builtin_nontemporal_store(low, pp);
        __builtin_nontemporal_store(high, pp + 1);
        if (EXT && a.param_bf16) {
            const u32x4_t halves = {pack_bf16(p[0], p[1]), pack_bf16(p[2], p[3]), pack_bf16(p[4], p[5]), pack_bf16(p[6], p[7])};
            __builtin_nontemporal_store(halves, reinterpret_cast<u32x4_t *>(a.param_bf16 + e0));
        }
    } else {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            if (ok[j]) {
                a.param[e0 + j] = p[j];
                if (EXT && a.param_bf16) a.param_bf16[e0 + j] = (uint16_t)pack_bf16(p[j], 0.0f);
            }
        }
    }
}

// A lane writes back what has changed of a word of 3-bit codes.  Ten-to-a-word codes do not end on a
// line (or even on a word) at the end of a wavefront's share:
// their words take this wavefront's changes by atomic XOR (the fields that two wavefronts own in
// a shared word are disjoint), which is carried out at the memory side and leaves no partly
// written line behind in the L2 of this die.
__device__ __forceinline__ void write_back_word(uint32_t *const word, const uint32_t changed)
{
    if (changed) atomicXor(word, changed);
}

// The first word of a stream of ten-to-a-word codes that the 512 elements of `chunk` (at most 2^31 of them:
// five fill whole words) touch, and the slot of the first element in it, in 32-bit arithmetic.
__device__ __forceinline__ uint64_t first_word10(const uint32_t chunk, uint32_t &slot)
{
    static_assert(5 * kIter % 10 == 0, "five chunks fill whole words");
    const uint32_t five = chunk / 5u, r = chunk - 5u * five, words = r * (uint32_t)kIter / 10u;
    slot = r * (uint32_t)kIter - 10u * words;
    return (uint64_t)five * (5 * kIter / 10) + words;
}

// The codes of the 512 elements that a wavefront steps on its own (8 consecutive elements per lane).  Eight 2- or
// 4-bit codes are a half or a whole word of the stream: the lane loads and stores it.  Eight 3-bit codes lie in one word or two
// neighbouring ones: the lane loads both, so that nothing has to be staged and waited for in LDS; what changes of a word
// is collected in LDS, in an image that starts from zeros, and lane i writes back the i-th one.  The first word may begin in the share before.
// TAIL: words behind the buffer are left alone.
template <int BITS, bool TAIL>
struct LaneCodes8 {
    static constexpr int C = 32 / BITS;                // codes per word
    static constexpr int kImage = BITS == 3 ? 64 : 0;  // words of the image (54 are used)
    uint32_t *word;                            // the first word of the share (uniform)
    bool has;                                  // this lane has a word, or half a one, to write
    uint32_t own[2];                           // as loaded
    uint32_t first;                            // 3-bit: slot of the first element in the first word

    // ew0: first element of the wavefront's share.  Issues the loads.
    __device__ __forceinline__ void load(uint32_t *const words, const uint64_t n, const uint64_t ew0, const uint32_t lane)
    {
        uint64_t lo;
        if (BITS == 3) lo = first_word10((uint32_t)(ew0 / kIter), first);
        else { lo = ew0 / C; first = 0; }
        word = words + lo;
        // (Lanes without a word load the last one again: a load under a condition whose fields are masked
        // behind it was waited for inside, in front of all the loads that follow.  2^20 elements,
        // 3-bit/3-bit fp32: 5.46 us under conditions, 5.27 without; the 1.3e9 elements of the 1.3B shapes, 3-bit/3-bit
        // bf16, 16 per lane: 2535 and 2439.)
        const uint32_t at = BITS == 2 ? lane / 2u : lane;
        uint32_t last = (first + kIter + C - 1) / C - 1;
        uint64_t from = lo;
        has = at <= last;
        if (TAIL) {
            const uint64_t end = (n - 1) / C;              // last word of the buffer
            has = has && lo + at <= end;
            from = umin64(from, end); last = (uint32_t)umin64(last, end - from);
        }
        if (BITS == 2) own[0] = reinterpret_cast<const uint16_t *>(words + from)[umin(lane, 2u * last + 1u)];
        else if (BITS == 4) own[0] = words[from + umin(lane, last)];
        else {
            const uint32_t w = Run3(first + lane * 8u).word;
            own[0] = words[from + umin(w, last)];
            own[1] = words[from + umin(w + 1u, last)];     // (a run that ends with its word does not use it)
        }
    }
    __device__ __forceinline__ void clear(uint32_t *const img, const uint32_t lane) const
    {
        if (BITS == 3) img[lane] = 0;
    }
    __device__ __forceinline__ uint32_t codes(const uint32_t lane) const
    {
        return BITS == 3 ? Run3(first + lane * 8u).codes(own[0], own[1]) : own[0];
    }
    // the lane's new codes (`old`: what codes() gave), in front of write_back()
    __device__ __forceinline__ void change(uint32_t *const img, const uint32_t lane, const uint32_t old, const uint32_t now) const
    {
        if (BITS == 3) Run3(first + fresh(lane) * 8u).change(img, old ^ now);
    }
    __device__ __forceinline__ void write_back(const uint32_t *const img, const uint32_t lane, const uint32_t now) const
    {
        if (TAIL || BITS == 3) { if (!has) return; }
        if (BITS == 2) reinterpret_cast<uint16_t *>(word)[lane] = (uint16_t)now;
        else if (BITS == 4) word[lane] = now;
        else write_back_word(&word[lane], img[lane]);
    }
};

// The DE bucket table of a workgroup, copied from constant memory.  Every thread asks for its words
// first (the constructor) and puts them into LDS, with a barrier, when the loads of its elements are
// under way (ready(), which every wavefront of the workgroup calls once): with the whole copy in
// front of those loads its latency stood in front of every 4096 elements (842 million elements,
// 3-bit/3-bit bf16: 1820 us, 1783 now; 2^24, 4-bit/2-bit: 39.3 and 37.6).
// THREADS: of the workgroup.
template <int BM, bool MDE, int THREADS = kWaves * 64>
struct DeTable {
    static constexpr bool kUsed = MDE && BM >= 3;
    static constexpr int kWords = de_words<BM, MDE>(), kPer = (kWords + THREADS - 1) / THREADS;
    uint32_t *const lds;
    uint32_t word[kPer];
    __device__ __forceinline__ explicit DeTable(uint32_t *const l) : lds(l)
    {
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const uint32_t w = threadIdx.x + (uint32_t)(i * THREADS);
            word[i] = 0;
            if (kUsed && w < (uint32_t)kWords) word[i] = (&DeBuckets<BM>::tab.w[0][0])[w];
        }
    }
    __device__ __forceinline__ void store() const       // (ready() without its barrier)
    {
        if (!kUsed) return;
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const uint32_t w = threadIdx.x + (uint32_t)(i * THREADS);
            if (w < (uint32_t)kWords) lds[w] = word[i];
        }
    }
    __device__ __forceinline__ void ready() const
    {
        store();
        if (kUsed) __syncthreads();
    }
};

// LDS of a wavefront that steps one 512-element chunk (32-bit words; offsets are compile-time
// constants, so the parts are reached with instruction offsets from very few address registers).
template <int BM, int BV, int B>
struct ChunkLayout8 {
    static constexpr int NG = kIter / B;
    static constexpr int VT = 1 << BV;
    static constexpr int MTS = m_table_stride<BM>();
    static constexpr int kOffImgM = 0;
    static constexpr int kOffImgV = kOffImgM + LaneCodes8<BM, false>::kImage;
    static constexpr int kOffTv = ((kOffImgV + LaneCodes8<BV, false>::kImage + 15) / 16) * 16;   // 64-byte aligned
    static constexpr int kOffTm = kOffTv + ((NG * VT + 15) / 16) * 16;
    static constexpr int kSlab = kOffTm + ((NG * MTS + 15) / 16) * 16;
};

// The whole step for the 512 elements from 512 * chunk on (TAIL: clipped to a.n, with bounds checks
// on every element), by the calling wavefront on its own.  `slab` is its LDS, `de` the
// workgroup's DE bucket table.
// A launch of few wavefronts is the chain of one, so what is not part of that chain is done where it waits: the hash of xi
// while the loads are under way, the parameters in the gaps of the divisions and of the base.  (With that, level tables filled without
// conditions, 3-bit codes straight from the words a lane loads and the position of those words by 32-bit arithmetic, us per launch in a
// graph, before | after: 4096 elements 2-bit/3-bit 3.15 | 3.01, 2^20 4-bit/4-bit fp32 4.55 | 4.46, 3-bit/3-bit 4.78 | 4.61, 2-bit/3-bit bf16
// 4.71 | 4.54, 5 million 4-bit/4-bit fp32 13.7 | 13.4.)
// ALONE: in a launch of such wavefronts; otherwise between wavefronts with 16 elements per lane, where the chain of one does not count: the
// parameters are then made, and stored, in front of the selection (tables as above, behind it | in front of it: 13.86 | 13.49 of 4.4 million elements).
// EXT: the code that also serves the variants of the step (gradient scale, coupled decay,
// AdaBelief, bf16 weight copy); the plain AdamW step runs the one without them.
template <int BM, int BV, int B, bool BF16, bool MDE, bool TAIL, bool EXT, bool ALONE = true>
__device__ __forceinline__ void step_chunk8(const StepArgs &a, const uint64_t chunk, const uint32_t lane,
                                            uint32_t *const slab, const DeTable<BM, MDE> &de)
{
    constexpr int G = B / 8;                       // lanes per block
    constexpr int NG = 64 / G;                     // blocks of the chunk
    constexpr int L = (1 << (BM - 1)) - 1;
    constexpr int VT = 1 << BV;
    using Lay = ChunkLayout8<BM, BV, B>;
    constexpr bool kDeTable = MDE && BM >= 3;

    const uint64_t ew0 = chunk * kIter, e0 = ew0 + lane * 8u;
    const uint32_t lig = lane & (G - 1);               // lane in group
    const uint32_t grp = lane / G;                     // group (block) inside the chunk
    const uint32_t gshift = lane & 31u & ~(uint32_t)(G - 1);   // group's first lane inside its 32-lane half
    uint32_t *const img_m = slab + Lay::kOffImgM, *const img_v = slab + Lay::kOffImgV;
    float *const my_tv = reinterpret_cast<float *>(slab + Lay::kOffTv) + grp * VT;
    float *const my_tm = reinterpret_cast<float *>(slab + Lay::kOffTm) + grp * Lay::MTS;
    const uint32_t tv_addr = lds_addr(my_tv), tm_addr = lds_addr(my_tm);   // aligned to the table size
    // elements of this lane's block that exist (B except in the last block)
    const uint64_t gb = chunk * NG + grp;
    uint32_t nb = B;
    bool blk_ok = true;
    bool ok[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) ok[j] = !TAIL || (e0 + j) < a.n;
    if (TAIL) {
        blk_ok = gb < (a.n + B - 1) / B;
        const uint64_t bstart = gb * B;
        nb = blk_ok ? (uint32_t)((a.n - bstart) < (uint64_t)B ? (a.n - bstart) : (uint64_t)B) : 0u;
    }

    // ---- every load is issued before the first one is waited for
    LaneCodes8<BM, TAIL> mw;
    LaneCodes8<BV, TAIL> vw;
    mw.load(a.m_words, a.n, ew0, lane);
    vw.load(a.v_words, a.n, ew0, lane);
    const uint64_t gb_here = TAIL ? umin64(gb, (a.n - 1u) / B) : gb;
    const float dm_old = a.m_scale[gb_here], dv_old = a.v_scale[gb_here], al_old = a.v_base[gb_here];
    const bool whole = !TAIL || (ALONE ? __builtin_expect(ew0 + kIter <= a.n, 0) : e0 + 8u <= a.n);
    const RawPG raw = load_pg<BF16, TAIL, ALONE, BF16 && ALONE>(a, e0, whole);
    const float gscale = (EXT && a.grad_scale) ? *a.grad_scale : 1.0f;      // uniform: the gradient is transformed first

    // ---- while they are under way: what does not depend on them
    uint32_t xi_word[1];
    XiGroups(a, ew0).words<1>(a, lane, xi_word);
    XiRun xi(a, xi_word[0]);
    if (ALONE) { xi.X = fresh(xi.X); xi.Y = fresh(xi.Y); }
    mw.clear(img_m, lane);
    vw.clear(img_v, lane);
    de.ready();

    // ---- level tables of this lane's block: entries lig, lig + G, ...
    const uint32_t de_base = kDeTable ? lds_addr(de.lds) - 16u * DeBuckets<BM>::kLo : 0u;    // bucket table address, less the first bucket's index
    fill_level_tables<BM, BV, MDE, G, true>(my_tv, my_tm, lig, dm_old, dv_old, al_old);
    wave_lds_sync();
    const uint32_t mc8 = mw.codes(lane), vc8 = vw.codes(lane);

    // ---- dequantize (table look-up), EMA
    float p[8], g[8];
    unpack_pg<BF16>(raw, p, g);
    if (EXT) {                                 // g <- fl(g * scale), then one fused g + l2 * p (l2 = 0: exact)
#pragma unroll
        for (int j = 0; j < 8; ++j) g[j] = __builtin_fmaf(a.l2, p[j], g[j] * gscale);
    }
    float mh[8], vh[8];
    float m_absmax, v_max;                     // (v_max of full chunks: the last sorted key below)
    ema_param<8, BM, BV, EXT, TAIL, TAIL>(a, tm_addr, tv_addr, &mc8, &vc8, ok, p, g, mh, vh, m_absmax, v_max);
    if (!ALONE) {
        new_param8(a, mh, vh, p);
        store_params8<EXT, TAIL>(a, e0, whole, ok, p);
    }

    // ---- the lane's v^ sorted (non-negative floats order like their bit patterns); block maxima
    uint32_t key[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) key[j] = (TAIL && !ok[j]) ? kInfBits : f2u(vh[j]);
    sort8(key);
    float dm = u2f(group_reduce<G>(f2u(m_absmax), UMax()));
    float dv = u2f(group_reduce<G>(TAIL ? f2u(v_max) : key[7], UMax()));
    if (dm < kTiny) dm = 0.0f;
    if (dv < kTiny) dv = 0.0f;

    // ---- the r-th smallest v^ of the block
    // (a shorter last block has a smaller rank; absent elements are +inf behind the others)
    uint32_t rank = a.rank_full;
    if (TAIL) {
        const float x = __builtin_ceilf(a.quantile_p * (float)nb);
        rank = x < 1.0f ? 1u : (uint32_t)x;
        rank = umax(umin(rank, nb), 1u);
    }
    const uint32_t xp_bits = merged_rth8<G>(key, lane, rank, a.rank_full);

    // ---- parameter; the block's encoder constants, then this lane's 8 codes of each moment
    if (ALONE) {
        new_param8(a, mh, vh, p);
        store_params8<EXT, TAIL>(a, e0, whole, ok, p);
    }
    const BlockCodec codec = block_codec<BV, G, L, MDE>(xp_bits, dm, dv, lane, lig, gshift);
    uint32_t m8, v8;
    encode_run<BM, BV, MDE, TAIL>(xi, mh, vh, ok, codec, de_base, m8, v8);
    mw.change(img_m, lane, mc8, m8);
    vw.change(img_v, lane, vc8, v8);
    if (lig == 0 && blk_ok) { a.m_scale[gb] = dm; a.v_scale[gb] = dv; a.v_base[gb] = codec.alpha; }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    mw.write_back(img_m, lane, m8);
    vw.write_back(img_v, lane, v8);
}

// Sixteen keys, two sorted halves: the eight smallest in order (the smaller of a and b's mirror image are a
// bitonic sequence).
__device__ __forceinline__ void lower_half(const uint32_t (&a)[8], const uint32_t (&b)[8], uint32_t (&k)[8])
{
#pragma unroll
    for (int i = 0; i < 8; ++i) k[i] = umin(a[i], b[7 - i]);
#pragma unroll
    for (int w = 4; w >= 1; w /= 2)
#pragma unroll
        for (int i = 0; i < 8; ++i) if ((i & w) == 0) cswap(k[i], k[i + w]);
}

// The merge of all sixteen: Batcher's odd-even merge of the halves (25 exchanges).
__device__ __forceinline__ void merge16(const uint32_t (&a)[8], const uint32_t (&b)[8], uint32_t (&k)[16])
{
#pragma unroll
    for (int i = 0; i < 8; ++i) { k[i] = a[i]; k[i + 8] = b[i]; }
#pragma unroll
    for (int i = 0; i < 8; ++i) cswap(k[i], k[i + 8]);
#pragma unroll
    for (int i = 4; i < 8; ++i) cswap(k[i], k[i + 4]);
#pragma unroll
    for (int i = 2; i < 12; i += 4) { cswap(k[i], k[i + 2]); cswap(k[i + 1], k[i + 3]); }
#pragma unroll
    for (int i = 1; i < 15; i += 2) cswap(k[i], k[i + 1]);
}

// Up to which rank the eight smallest of a lane's 16 values are enough but for one wavefront in a hundred
// (G lanes; the ranks in front of it fall on the lanes at random: at rank 13 of 128 one in a thousand, at 7 of 64 none).
template <int G>
constexpr uint32_t low_rank() { return G == 8 ? 16u : 10u; }

// The largest (dv, values below kTiny as 0) and the rank-th smallest (returned) v^ of every group of G
// lanes that hold 16 of them each.  `col`: the lane's column in LDS.
// Small ranks: the columns hold the eight smallest of every lane only, which takes a sixth off the sorting.  What is
// selected from those is the answer unless some lane's eighth is smaller than it, as leaving keys out can only
// raise it; then everything is done again with full columns.  (With pairs popped at once (extract_rth()) and exclusive
// ors in the exchanges, against full columns and one key a round, us: 2^26 elements 2-bit/3-bit bf16 133.6 -> 120.0, at
// p = 0.3, whose columns are full, 148.5 -> 127.7, 2-bit/2-bit B 64 at p = 0.3 132.5 -> 124.1; the 7B shapes 12843 -> 12586.)
template <int G>
__device__ __forceinline__ uint32_t quantile16(const float (&vh)[16], uint32_t *const col, const uint32_t rank, float &dv)
{
    uint32_t a[8], b[8];                           // (non-negative floats order like their bit patterns)
#pragma unroll
    for (int j = 0; j < 8; ++j) { a[j] = f2u(vh[j]); b[j] = f2u(vh[8 + j]); }
    sort8(a);
    sort8(b);
    dv = u2f(group_reduce<G>(umax(a[7], b[7]), UMax()));
    if (dv < kTiny) dv = 0.0f;
    uint32_t xp;
    if (__builtin_expect(rank <= low_rank<G>(), 1)) {
        uint32_t k[8];
        lower_half(a, b, k);
#pragma unroll
        for (int c = 0; c < 4; ++c) *reinterpret_cast<uint2 *>(col + 2 * c) = make_uint2(k[2 * c], k[2 * c + 1]);
        *reinterpret_cast<uint2 *>(col + 8) = *reinterpret_cast<uint2 *>(col + 10) = make_uint2(kInfBits, kInfBits);
        xp = extract_rth<G>(k[0], k[1], k[2], k[3], lds_addr(col), rank);
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(k[7] < xp) == 0, 1)) return xp;
#pragma unroll
        for (int j = 0; j < 8; ++j) { a[j] = f2u(vh[j]); b[j] = f2u(vh[8 + j]); }
        sort8(a);
        sort8(b);
    }
    uint32_t k[16];
    merge16(a, b, k);
#pragma unroll
    for (int c = 0; c < 8; ++c) *reinterpret_cast<uint2 *>(col + 2 * c) = make_uint2(k[2 * c], k[2 * c + 1]);
    *reinterpret_cast<uint2 *>(col + 16) = make_uint2(kInfBits, kInfBits);
    return extract_rth<G>(k[0], k[1], k[2], k[3], lds_addr(col), rank);
}

// Parameters and gradients of one lane and one 1024-element chunk, in the
// coalesced layout they are loaded in (vector k of a lane is vector lane + 64 k of the chunk).
template <bool BF16>
struct RawPG16 { float4 p[4]; uint4 g[BF16 ? 2 : 4]; };

// `here`: elements of the chunk that exist (uniform); absent ones read as zeros, and only the vector
// that holds the end of the buffer is read element by element.
template <bool BF16>
__device__ __forceinline__ RawPG16<BF16> load_pg16(const StepArgs &a, uint64_t chunk_e0, uint32_t lane, const uint32_t here = kIter16)
{
    RawPG16<BF16> r;
    const float *pp = a.param + chunk_e0 + lane * 4u;
    const uint16_t *hp = static_cast<const uint16_t *>(a.grad) + chunk_e0 + lane * 8u;     // bf16 gradients
    const uint32_t *gp = static_cast<const uint32_t *>(a.grad) + chunk_e0 + lane * 4u;     // fp32 gradients
    if (__builtin_expect(here == kIter16, 1)) {
#pragma unroll
        for (int k = 0; k < 4; ++k) r.p[k] = stream_load_f4(pp + 256 * k);
#pragma unroll
        for (int k = 0; k < (BF16 ? 2 : 4); ++k) r.g[k] = BF16 ? stream_load_u4(hp + 512 * k) : stream_load_u4(gp + 256 * k);
        return r;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const uint32_t i = lane * 4u + 256u * k;
        r.p[k] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        if (!BF16) r.g[k] = make_uint4(0, 0, 0, 0);
        if (i + 4u <= here) {
            r.p[k] = stream_load_f4(pp + 256 * k);
            if (!BF16) r.g[k] = stream_load_u4(gp + 256 * k);
        } else if (i < here) {
            r.p[k].x = pp[256 * k];
            if (i + 1u < here) r.p[k].y = pp[256 * k + 1];
            if (i + 2u < here) r.p[k].z = pp[256 * k + 2];
            if (!BF16) {
                r.g[k].x = gp[256 * k];
                if (i + 1u < here) r.g[k].y = gp[256 * k + 1];
                if (i + 2u < here) r.g[k].z = gp[256 * k + 2];
            }
        }
    }
    if (BF16) {
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const uint32_t i = lane * 8u + 512u * k;
            r.g[k] = make_uint4(0, 0, 0, 0);
            if (i + 8u <= here) {
                r.g[k] = stream_load_u4(hp + 512 * k);
            } else if (i < here) {
                uint32_t w[4] = {0, 0, 0, 0};
#pragma unroll
                for (int j = 0; j < 7; ++j)
                    if (i + j < here) w[j / 2] |= (uint32_t)hp[512 * k + j] << (16 * (j & 1));
                r.g[k] = make_uint4(w[0], w[1], w[2], w[3]);
            }
        }
    }
    return r;
}

// The staging slots of a lane for the layout transposition of a 1024-element iteration, 16-byte
// vectors.  Vector i of the chunk sits in slot i + i / 8 (one pad vector after every 8): eight
// neighbouring lanes then cover all banks both on the coalesced side (i = lane + 64 k) and on the
// lane's own side (fp32: i = 4 lane + c, slot 4 lane + lane / 2 + c; bf16: i = 2 lane + c,
// slot 2 lane + lane / 4 + c).  288 vectors.
struct Stage16 {
    float4 *c4, *l4, *c2, *l2;     // c4[72 k], l4[c]: 32-bit elements; c2[72 k], l2[c]: 16-bit elements
    __device__ __forceinline__ Stage16(float4 *stage, uint32_t lane)
        : c4(stage + (lane + lane / 8u)), l4(stage + (4u * lane + lane / 2u)),
          c2(stage + (lane + lane / 8u)), l2(stage + (2u * lane + lane / 4u)) {}
};

// A lane's 16 consecutive elements out of the coalesced layout they were loaded in.
template <bool BF16>
__device__ __forceinline__ void lane_layout16(const RawPG16<BF16> &raw, const Stage16 &st,
                                              float (&p)[16], float (&g)[16])
{
    float4 t[4];
    uint4 h[BF16 ? 2 : 4];
#pragma unroll
    for (int k = 0; k < 4; ++k) st.c4[72 * k] = raw.p[k];
    wave_lds_sync();                   // (also orders the level tables before their readers)
#pragma unroll
    for (int c = 0; c < 4; ++c) t[c] = st.l4[c];
    wave_lds_sync();
#pragma unroll
    for (int k = 0; k < (BF16 ? 2 : 4); ++k) {
        const float4 x = make_float4(u2f(raw.g[k].x), u2f(raw.g[k].y), u2f(raw.g[k].z), u2f(raw.g[k].w));
        if (BF16) st.c2[72 * k] = x; else st.c4[72 * k] = x;
    }
    wave_lds_sync();
#pragma unroll
    for (int c = 0; c < (BF16 ? 2 : 4); ++c) {
        const float4 x = BF16 ? st.l2[c] : st.l4[c];
        h[c] = make_uint4(f2u(x.x), f2u(x.y), f2u(x.z), f2u(x.w));
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) { p[4 * c] = t[c].x; p[4 * c + 1] = t[c].y; p[4 * c + 2] = t[c].z; p[4 * c + 3] = t[c].w; }
#pragma unroll
    for (int c = 0; c < (BF16 ? 2 : 4); ++c) {
        const uint32_t w[4] = {h[c].x, h[c].y, h[c].z, h[c].w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (BF16) { g[8 * c + 2 * i] = u2f(w[i] << 16); g[8 * c + 2 * i + 1] = u2f(w[i] & 0xFFFF0000u); }
            else g[4 * c + i] = u2f(w[i]);
        }
    }
}

// Half K of the 1024 bf16 copies of a chunk: the lane's 8 of them at byte `at`.
template <int K>
__device__ __forceinline__ void store_halves(uint16_t *const hp, const uint32_t at, const float4 x, const bool all, const uint32_t here)
{
    const uint32_t i = at / 2u + 512u * K;
    if (all || i + 8u <= here) {
        stream_store_f4<1024 * K>(hp, at, x);
    } else if (i < here) {
        const uint32_t w[4] = {f2u(x.x), f2u(x.y), f2u(x.z), f2u(x.w)};
#pragma unroll
        for (int j = 0; j < 7; ++j)
            if (i + j < here) hp[i + j] = (uint16_t)(w[j / 2] >> (16 * (j & 1)));
    }
}

// The new parameters of a lane's 16 elements (and their bf16 copy, if asked for: 32 bytes per
// lane, two vectors, first) back to the coalesced layout and streamed out; chunk_e0: first
// element of the wavefront's 1024, of which `here` exist.
template <bool EXT>
__device__ __forceinline__ void store_params16(const StepArgs &a, const uint64_t chunk_e0, const uint32_t lane,
                                               const float (&p)[16], const Stage16 &st, const uint32_t here = kIter16)
{
    wave_lds_sync();
    const bool all = __builtin_expect(here == kIter16, 1);
    const uint32_t at = lane * 16u;
    if (EXT && a.param_bf16) {
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const uint32_t h0 = pack_bf16(p[8 * c], p[8 * c + 1]), h1 = pack_bf16(p[8 * c + 2], p[8 * c + 3]);
            const uint32_t h2 = pack_bf16(p[8 * c + 4], p[8 * c + 5]), h3 = pack_bf16(p[8 * c + 6], p[8 * c + 7]);
            st.l2[c] = make_float4(u2f(h0), u2f(h1), u2f(h2), u2f(h3));
        }
        wave_lds_sync();
        uint16_t *const hp = a.param_bf16 + chunk_e0;
        store_halves<0>(hp, at, st.c2[0], all, here);
        store_halves<1>(hp, at, st.c2[72], all, here);
        wave_lds_sync();
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) st.l4[c] = make_float4(p[4 * c], p[4 * c + 1], p[4 * c + 2], p[4 * c + 3]);
    wave_lds_sync();
    float *const pp = a.param + chunk_e0;
    if (all) {
        stream_store_f4<0>(pp, at, st.c4[0]);
        stream_store_f4<1024>(pp, at, st.c4[72]);
        stream_store_f4<2048>(pp, at, st.c4[144]);
        stream_store_f4<3072>(pp, at, st.c4[216]);
        return;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const uint32_t i = lane * 4u + 256u * k;
        const float4 x = st.c4[72 * k];
        if (i + 4u <= here) {
            *reinterpret_cast<float4 *>(pp + i) = x;
        } else if (i < here) {
            pp[i] = x.x;
            if (i + 1u < here) pp[i + 1u] = x.y;
            if (i + 2u < here) pp[i + 2u] = x.z;
        }
    }
}

// The codes of the 1024 elements that a wavefront steps on its own (16 consecutive elements per lane).  Sixteen
// 2- or 4-bit codes are one or two words of the stream: the lane loads and stores them.  Words of 3-bit codes are
// staged in LDS, two of a stream per lane, as those of LaneCodes8.  STAGED: they are, and so are 4-bit ones of
// dynamic-exponent moments, whose rounding has no register to spare (4-bit/2-bit with a copy 85 instead of 75, five wavefronts
// per SIMD instead of six: 2^26 elements 152 us, 157 without staging).
template <int BITS, bool STAGED>
struct LaneCodes16 {
    static constexpr int C = 32 / BITS;                // codes per word
    static constexpr int K = BITS == 2 ? 1 : 2;        // words of the stream per lane (64 K >= words of 1024 elements)
    static constexpr int kImage = STAGED ? 132 : 0;    // words of the image (<= 128, + 4)
    static_assert(BITS == 4 || STAGED == (BITS == 3), "2-bit words are a lane's own, 3-bit ones are not");
    uint32_t *word;                            // the first word of the share (uniform)
    uint32_t nw;                               // words touched (<= 128)
    uint32_t own[K];                           // the words as they were loaded (3-bit: until they are staged)
    uint32_t first;                            // 3-bit: slot of the first element in the first word

    // which of the share's words a lane holds as own[k]
    static __device__ __forceinline__ uint32_t at(const uint32_t lane, const int k) { return BITS == 4 && !STAGED ? 2u * lane + k : lane + 64u * k; }

    // ew0: first element of the wavefront's share, of which `here` exist (0: none; FULL: all).
    // Issues the loads.  Lanes without a word load the last one again, because a load
    // under a condition is waited for inside it, with every load in front of it (see LaneCodes8; blocks of 2048,
    // 1 million elements, 2-bit/3-bit bf16: 9.6 us, 9.2 with it and the words in front of the parameters).
    template <bool FULL>
    __device__ __forceinline__ void load(uint32_t *const words, const uint64_t ew0, const uint32_t lane, const uint32_t here)
    {
        const uint64_t lo = ew0 / C;
        word = words + lo;
        first = (uint32_t)(ew0 - lo * C);
        nw = here ? (first + here + C - 1) / C : 0;
        if (FULL && BITS == 4 && !STAGED) {
            const uint2 two = *reinterpret_cast<const uint2 *>(word + 2u * lane);
            own[0] = two.x; own[K - 1] = two.y;
            return;
        }
        const uint64_t from = here ? lo : (ew0 - kIter16) / C;
        const uint32_t last = here ? nw - 1u : 0u;
#pragma unroll
        for (int k = 0; k < K; ++k) own[k] = words[from + umin(at(lane, k), last)];
    }
    __device__ __forceinline__ void stage(uint32_t *const img, const uint32_t lane)
    {
        if (!STAGED) return;
#pragma unroll
        for (int k = 0; k < K; ++k) img[lane + 64u * k] = own[k];
        if (BITS == 3 && lane < 4) img[64 * K + lane] = 0;
    }
    static __device__ __forceinline__ uint32_t run_from(const uint32_t *const img, const Run3 run) { return run.codes(img[run.word], img[run.word + 1]); }
    // the lane's old codes, eight to a run (2-bit: the upper half of the register is not clear)
    __device__ __forceinline__ void codes(uint32_t *const img, const uint32_t lane, uint32_t (&c8)[2]) const
    {
#pragma unroll
        for (int r = 0; r < 2; ++r)
            c8[r] = BITS == 3 ? run_from(img, Run3(first + lane * 16u + 8u * r)) : BITS == 2 ? own[0] >> (16 * r) : STAGED ? img[2u * lane + r] : own[r % K];
        if (BITS != 3) return;
        wave_lds_sync();
#pragma unroll
        for (int k = 0; k < K; ++k) img[lane + 64u * k] = 0;
    }
    // the lane's new codes of run r (`old`: what codes() gave), in front of write_back()
    __device__ __forceinline__ void change(uint32_t *const img, const uint32_t lane, const int r, const uint32_t old, const uint32_t now) const
    {
        if (BITS == 3) Run3(first + fresh(lane) * 16u + 8u * r).change(img, old ^ now);
        else if (STAGED) img[2u * lane + r] = now;
    }
    template <bool FULL>
    __device__ __forceinline__ void write_back(const uint32_t *const img, const uint32_t lane, const uint32_t (&now)[2]) const
    {
        if (FULL && BITS == 4 && !STAGED) {
            *reinterpret_cast<uint2 *>(word + 2u * lane) = make_uint2(now[0], now[1]);
            return;
        }
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const uint32_t i = at(lane, k);
            if ((FULL && BITS != 3) || i < nw) {
                if (BITS == 3) write_back_word(&word[i], img[i]);
                else word[i] = BITS == 2 ? now[0] | now[1] << 16 : STAGED ? img[i] : now[k];
            }
        }
    }
};

template <int BM, bool MDE> using MomentCodes16 = LaneCodes16<BM, BM == 3 || (BM == 4 && MDE)>;
template <int BV> using VarianceCodes16 = LaneCodes16<BV, BV == 3>;

// New codes of a lane's 16 elements, two runs of 8; ew0 is the wavefront's first element, mc8 / vc8 the old codes.
// `mine`: how many of them exist (fields behind the last element of the buffer become zero).
template <int BM, int BV, bool MDE>
__device__ __forceinline__ void encode16(const StepArgs &a, const uint64_t ew0, const uint32_t lane, const float *mh, const float *vh,
                                         const BlockCodec &codec, const uint32_t de_base, const MomentCodes16<BM, MDE> &mw,
                                         const VarianceCodes16<BV> &vw, uint32_t *const img_m, uint32_t *const img_v,
                                         const uint32_t (&mc8)[2], const uint32_t (&vc8)[2], uint32_t (&m8)[2], uint32_t (&v8)[2],
                                         const bool all = true, const uint32_t mine = 16)
{
    uint32_t xi_word[2];
    XiGroups(a, ew0).words<2>(a, 2u * lane, xi_word);
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        encode_run<BM, BV, MDE, false>(XiRun(a, xi_word[r]), mh + 8 * r, vh + 8 * r, nullptr, codec, de_base, m8[r], v8[r]);
        if (__builtin_expect(!all, 0)) {
            const uint32_t run = mine <= 8u * r ? 0u : umin(mine - 8u * r, 8u);
            m8[r] &= (uint32_t)((1ull << (BM * run)) - 1ull);
            v8[r] &= (uint32_t)((1ull << (BV * run)) - 1ull);
        }
        mw.change(img_m, lane, r, mc8[r], m8[r]);
        vw.change(img_v, lane, r, vc8[r], v8[r]);
    }
}

// LDS of a wavefront that steps one 1024-element chunk on its own (32-bit words).
template <int BM, int BV, int B, bool MDE>
struct ChunkLayout16 {
    static constexpr int NG = kIter16 / B;
    static constexpr int VT = 1 << BV;
    static constexpr int MTS = m_table_stride<BM>();
    static constexpr int kOffCol = 0;                          // staging of the transpositions, then the sorted columns
    static constexpr int kOffImgM = 64 * kColStride16;
    static constexpr int kOffImgV = kOffImgM + MomentCodes16<BM, MDE>::kImage;
    static constexpr int kOffTv = ((kOffImgV + VarianceCodes16<BV>::kImage + 15) / 16) * 16;      // 64-byte aligned
    static constexpr int kOffTm = kOffTv + ((NG * VT + 15) / 16) * 16;
    static constexpr int kEnd = kOffTm + ((NG * MTS + 15) / 16) * 16;
    // (a runaway column address, possible only with non-finite input, stays inside the slab)
    static constexpr int kColumns = (64 * kColStride16 + 140 + 15) / 16 * 16;
    static constexpr int kSlab = kEnd > kColumns ? kEnd : kColumns;
};

// The whole step for the 1024 elements from 1024 * chunk on (whole blocks, all of them present),
// by the calling wavefront on its own, 16 consecutive elements per lane.
template <int BM, int BV, int B, bool BF16, bool MDE, bool EXT>
__device__ __forceinline__ void step_chunk16(const StepArgs &a, const uint64_t chunk, const uint32_t lane,
                                             uint32_t *const slab, const DeTable<BM, MDE> &de)
{
    constexpr int G = B / 16;                      // lanes per block
    constexpr int NG = 64 / G;                     // blocks of the chunk
    constexpr int L = (1 << (BM - 1)) - 1;
    constexpr int VT = 1 << BV;
    using Lay = ChunkLayout16<BM, BV, B, MDE>;
    constexpr bool kDeTable = MDE && BM >= 3;

    const uint64_t ew0 = chunk * kIter16;
    const uint32_t lig = lane & (G - 1), grp = lane / G, gshift = lane & 31u & ~(uint32_t)(G - 1);
    uint32_t *const img_m = slab + Lay::kOffImgM, *const img_v = slab + Lay::kOffImgV;
    uint32_t *const col = slab + Lay::kOffCol + lane * kColStride16;
    float *const my_tv = reinterpret_cast<float *>(slab + Lay::kOffTv) + grp * VT;
    float *const my_tm = reinterpret_cast<float *>(slab + Lay::kOffTm) + grp * Lay::MTS;
    const uint32_t tv_addr = lds_addr(my_tv), tm_addr = lds_addr(my_tm);

    // ---- every load is issued before the first one is waited for
    MomentCodes16<BM, MDE> mw;
    VarianceCodes16<BV> vw;
    mw.template load<true>(a.m_words, ew0, lane, kIter16);
    vw.template load<true>(a.v_words, ew0, lane, kIter16);
    float *const m_scale = a.m_scale + chunk * NG, *const v_scale = a.v_scale + chunk * NG, *const v_base = a.v_base + chunk * NG;
    const float dm_old = m_scale[grp], dv_old = v_scale[grp], al_old = v_base[grp];
    const RawPG16<BF16> raw = load_pg16<BF16>(a, ew0, lane);
    const float gscale = (EXT && a.grad_scale) ? *a.grad_scale : 1.0f;
    const Stage16 st(reinterpret_cast<float4 *>(slab + Lay::kOffCol), lane);
    de.ready();

    mw.stage(img_m, lane);
    vw.stage(img_v, lane);
    const uint32_t de_base = kDeTable ? lds_addr(de.lds) - 16u * DeBuckets<BM>::kLo : 0u;
    fill_level_tables<BM, BV, MDE, G, false>(my_tv, my_tm, lig, dm_old, dv_old, al_old);
    wave_lds_sync();
    uint32_t mc8[2], vc8[2];
    mw.codes(img_m, lane, mc8);
    vw.codes(img_v, lane, vc8);

    float p[16], g[16];
    lane_layout16<BF16>(raw, st, p, g);
    if (EXT) {
#pragma unroll
        for (int j = 0; j < 16; ++j) g[j] = __builtin_fmaf(a.l2, p[j], g[j] * gscale);
    }
    float mh[16], vh[16];
    float m_absmax, v_unused;                   // (the largest v^ is the lane's last sorted key below)
    ema_param<16, BM, BV, EXT, false, false>(a, tm_addr, tv_addr, mc8, vc8, nullptr, p, g, mh, vh, m_absmax, v_unused);
    store_params16<EXT>(a, ew0, lane, p, st);
    wave_lds_sync();                            // the staging area becomes the column area

    float dm = u2f(group_reduce<G>(f2u(m_absmax), UMax()));
    if (dm < kTiny) dm = 0.0f;
    float dv;
    const uint32_t xp_bits = quantile16<G>(vh, col, a.rank_full, dv);

    const BlockCodec codec = block_codec<BV, G, L, MDE>(xp_bits, dm, dv, lane, lig, gshift);
    uint32_t m8[2], v8[2];
    encode16<BM, BV, MDE>(a, ew0, lane, mh, vh, codec, de_base, mw, vw, img_m, img_v, mc8, vc8, m8, v8);
    if (lig == 0) { m_scale[grp] = dm; v_scale[grp] = dv; v_base[grp] = codec.alpha; }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    mw.template write_back<true>(img_m, lane, m8);
    vw.template write_back<true>(img_v, lane, v8);
}

// What a wavefront of a short launch needs for its first loads, in front of the other arguments: the hardware puts the first 14 words of a
// kernel's arguments into scalar registers before the wavefront starts (the build asks for it), so that these loads
// don't wait for scalar ones.  (us in a graph, without | with: 4096 elements 2-bit/3-bit 3.11 | 3.03, 2^20 2-bit/3-bit bf16 4.70 | 4.61,
// 4-bit/4-bit fp32 4.58 | 4.52, out of HBM 5.46 | 5.23 and 6.20 | 6.22.)
// `whole`: chunks or blocks of UNIT elements; `more`: the elements behind them, and in the upper half how many wavefronts or blocks take those.
#define SOLO_FIRST_ARGS const uint32_t whole, const uint32_t more, const void *const grad, uint32_t *const m_words, \
                        uint32_t *const v_words, float *const m_scale, float *const v_scale, float *const v_base
typedef void first_args_t(SOLO_FIRST_ARGS);
// Where a kernel's arguments P end, each at its own alignment.
template <typename... P>
constexpr size_t args_end(void (*)(P...))
{
    size_t at = 0;
    ((at = (at + alignof(P) - 1) / alignof(P) * alignof(P) + sizeof(P)), ...);
    return at;
}
// (big_quad_kernel reads the StepRest behind them by its place)
constexpr int kFirstArgsBytes = (int)((args_end((first_args_t *)nullptr) + alignof(StepRest) - 1) / alignof(StepRest) * alignof(StepRest));
static_assert(kFirstArgsBytes <= 14 * 4, "more words than are loaded in front");
template <int UNIT>
__device__ __forceinline__ StepArgs all_args(const StepRest &rest, SOLO_FIRST_ARGS)
{
    static_assert(UNIT <= 0x10000, "the elements behind the whole units fit the lower half of `more`");
    StepArgs a;
    static_cast<StepRest &>(a) = rest;
    a.n = (uint64_t)whole * UNIT + (more & 0xFFFFu);
    a.grad = grad; a.m_words = m_words; a.v_words = v_words; a.m_scale = m_scale; a.v_scale = v_scale; a.v_base = v_base;
    return a;
}

// The step over one flat buffer, 8 elements per lane: one wavefront per 512 elements, the last
// ones (up to the end of the last code word) with bounds checks where the buffer ends.
template <int BM, int BV, int B, bool BF16, bool MDE, bool EXT>
__global__ __launch_bounds__(kWaves * 64, kMinWaves)
void chunk8_kernel(SOLO_FIRST_ARGS, const StepRest rest)
{
    using Lay = ChunkLayout8<BM, BV, B>;
    __shared__ __attribute__((aligned(64))) uint32_t lds_slab[kWaves * Lay::kSlab];
    __shared__ __attribute__((aligned(64))) uint32_t lds_de[de_words<BM, MDE>()];
    const DeTable<BM, MDE> de(lds_de);
    const uint32_t lane = threadIdx.x & 63u;
    // the wavefront index is uniform: keeping it (and every address derived from the chunk) in
    // scalar registers frees vector registers
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint32_t c = blockIdx.x * kWaves + wave;
    uint32_t *const slab = lds_slab + wave * Lay::kSlab;
    const StepArgs a = all_args<kIter>(rest, whole, more, grad, m_words, v_words, m_scale, v_scale, v_base);
    if (c < whole)
        step_chunk8<BM, BV, B, BF16, MDE, false, EXT>(a, c, lane, slab, de);
    else if (c < whole + (more >> 16))
        step_chunk8<BM, BV, B, BF16, MDE, true, EXT>(a, c, lane, slab, de);
    else
        de.ready();
}

// The step over one flat buffer, 16 elements per lane: one wavefront per 1024 elements.  The first
// a.rest wavefronts take what is left behind the last whole chunk (the slower, bounds-checked
// code, so it starts first), 512 elements each.
template <int BM, int BV, int B, bool BF16, bool MDE, bool EXT>
__global__ __launch_bounds__(kWaves * 64, kMinWaves16)
void chunk16_kernel(const StepArgs a)
{
    using Lay = ChunkLayout16<BM, BV, B, MDE>;
    static_assert(Lay::kSlab >= ChunkLayout8<BM, BV, B>::kSlab, "one slab serves both forms");
    __shared__ __attribute__((aligned(64))) uint32_t lds_slab[kWaves * Lay::kSlab];
    __shared__ __attribute__((aligned(64))) uint32_t lds_de[de_words<BM, MDE>()];
    const DeTable<BM, MDE> de(lds_de);
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint64_t c = (uint64_t)blockIdx.x * kWaves + wave;
    uint32_t *const slab = lds_slab + wave * Lay::kSlab;
    if (c >= a.rest) {
        if (c - a.rest < a.n / kIter16)
            step_chunk16<BM, BV, B, BF16, MDE, EXT>(a, c - a.rest, lane, slab, de);
        else
            de.ready();
    } else {
        step_chunk8<BM, BV, B, BF16, MDE, true, EXT, false>(a, a.n / kIter16 * (kIter16 / kIter) + c, lane, slab, de);
    }
}

// ---- many tensors in one launch.  Blocks never span tensors: each tensor is quantized on its own.

// The tensor whose pieces hold piece `s` of all tensors, first8 / first16 (FIRST) counting the pieces
// in front of each: 64 tensors are looked at per step, one by every lane, so that up to 64 tensors
// take one dependent load and up to 4096 two.  (A tensor without elements shares its count with the
// one behind it, which is the one taken.)
template <uint32_t TensorEntry::*FIRST>
__device__ __forceinline__ const TensorEntry &find_tensor(const MultiArgs &ma, const uint32_t s, const uint32_t lane)
{
    uint32_t lo = 0, len = ma.count;
    do {
        const uint32_t stride = (len + 63u) / 64u, at = lane * stride;
        const bool before = at < len && ma.entries[lo + at].*FIRST <= s;
        const uint32_t j = (uint32_t)__builtin_popcountll(__builtin_amdgcn_ballot_w64(before)) - 1u;   // (tensor 0 has 0 in front)
        lo += j * stride;
        len = umin(stride, len - j * stride);
    } while (len > 1u);
    return ma.entries[lo];
}

// A pointer of an entry, read as one to global memory.  (A pointer that comes out of a kernel's own
// arguments is known to be one; behind a pointer out of memory every access was a flat one, which
// also occupies the LDS path and its counter: 203 million elements in nine tensors, 2-bit/2-bit DE with
// a bf16 copy, 436 -> 430 us, 4-bit/4-bit AdaBelief 443 -> 429, 2-bit/3-bit fp32 B 64 418 -> 407,
// blocks of 2048 2-bit/3-bit 469 -> 454.)  Like every field of an entry it is the same for the whole wavefront;
// where the entry is read by vector loads (behind a store or a barrier) the compiler has to be told.
__device__ __forceinline__ uint64_t uniform64(const uint64_t x)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)x);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(x >> 32));
    return lo | (uint64_t)hi << 32;
}
template <typename T>
__device__ __forceinline__ T *global_field(T *const &field)
{
    typedef __attribute__((address_space(1))) T global_t;
    return (T *)(global_t *)uniform64((uint64_t)field);
}

__device__ __forceinline__ StepArgs tensor_args(const MultiArgs &ma, const TensorEntry &e)
{
    StepArgs a = ma.common;
    a.param = global_field(e.param); a.param_bf16 = global_field(e.param_bf16); a.grad = global_field(e.grad);
    a.m_words = global_field(e.m_words); a.m_scale = global_field(e.m_scale);
    a.v_words = global_field(e.v_words); a.v_scale = global_field(e.v_scale); a.v_base = global_field(e.v_base);
    a.n = uniform64(e.n); a.index_offset = uniform64(e.index_offset);
    return a;
}

// Every tensor is cut into the pieces of a flat buffer of its size, one wavefront each, and stepped by
// the same code.  (Cutting the units of the map instead - five wavefronts per 5120 elements, a ragged end
// as part of them - left most wavefronts of a table of short tensors without work, and one wavefront
// with three pieces one behind the other where a tensor ends; 1000 tensors of 600 elements,
// 2-bit/3-bit bf16: 16.2 us, 7.0 now; 20,000 of them: 160 and 77; 53 tensors of 787,050 elements,
// 3-bit/4-bit fp32 with a copy: 14.2 and 7.1.)

// 8 elements per lane, for tables of few elements.
// (The plain step has a form of its own here too: the variants' g + l2 * p turns a parameter that is
// infinite or NaN into a gradient that is, also with l2 = 0, and spoils the state of its block.)
template <int BM, int BV, int B, bool BF16, bool MDE, bool EXT>
__global__ __launch_bounds__(kWaves * 64, kMinWaves)
void multi_chunk8_kernel(const TensorEntry *const entries, const uint32_t count, const MultiArgs args)
{
    MultiArgs ma = args;                       // (the first two: as SOLO_FIRST_ARGS; those in `args` are not read)
    ma.entries = entries; ma.count = count;
    using Lay = ChunkLayout8<BM, BV, B>;
    __shared__ __attribute__((aligned(64))) uint32_t lds_slab[kWaves * Lay::kSlab];
    __shared__ __attribute__((aligned(64))) uint32_t lds_de[de_words<BM, MDE>()];
    const DeTable<BM, MDE> de(lds_de);
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint32_t s = blockIdx.x * kWaves + wave;
    const TensorEntry &e = find_tensor<&TensorEntry::first8>(ma, s, lane);
    const uint64_t c = s - e.first8;
    const StepArgs a = tensor_args(ma, e);
    uint32_t *const slab = lds_slab + wave * Lay::kSlab;
    if ((c + 1) * kIter <= a.n)
        step_chunk8<BM, BV, B, BF16, MDE, false, EXT>(a, c, lane, slab, de);
    else if (c * kIter < end_of_words(a.n))
        step_chunk8<BM, BV, B, BF16, MDE, true, EXT>(a, c, lane, slab, de);
    else
        de.ready();
}

// find_tensor() with a first try: the tensor that the map names at the same fraction of the units.  In
// a table of large tensors that is nearly always the one, and two scalar loads say so, where the
// search takes two vector loads one behind the other for the 99 tensors of the GPT-2-125M shapes
// (2-bit/2-bit, B 64: 269 us without the try, 249 with it).
__device__ __forceinline__ const TensorEntry &find_tensor_of_chunk(const MultiArgs &ma, const uint32_t s, const uint32_t lane)
{
    const uint32_t unit = umin((uint32_t)((float)s * ma.units_per_piece), (uint32_t)ma.total_units - 1u);
    const uint32_t k = ma.unit_map[unit] & kMapTensorMask;
    const uint32_t next = k + 1u < ma.count ? ma.entries[k + 1u].first16 : 0xFFFFFFFFu;
    if (ma.entries[k].first16 <= s && s < next) return ma.entries[k];
    return find_tensor<&TensorEntry::first16>(ma, s, lane);
}

// 16 elements per lane, and 8 for what a tensor has left behind its whole chunks.
template <int BM, int BV, int B, bool BF16, bool MDE, bool EXT>
__global__ __launch_bounds__(kWaves * 64, kMinWaves16)
void multi_chunk16_kernel(const MultiArgs ma)
{
    using Lay = ChunkLayout16<BM, BV, B, MDE>;
    __shared__ __attribute__((aligned(64))) uint32_t lds_slab[kWaves * Lay::kSlab];
    __shared__ __attribute__((aligned(64))) uint32_t lds_de[de_words<BM, MDE>()];
    const DeTable<BM, MDE> de(lds_de);
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint32_t s = blockIdx.x * kWaves + wave;
    const TensorEntry &e = find_tensor_of_chunk(ma, s, lane);
    const uint64_t c = s - e.first16, whole = e.n / kIter16;
    const StepArgs a = tensor_args(ma, e);
    uint32_t *const slab = lds_slab + wave * Lay::kSlab;
    if (c < whole)
        step_chunk16<BM, BV, B, BF16, MDE, EXT>(a, c, lane, slab, de);
    else if ((whole + c) * kIter < end_of_words(a.n))
        step_chunk8<BM, BV, B, BF16, MDE, true, EXT, false>(a, whole + c, lane, slab, de);
    else
        de.ready();
}

// A launch with the arguments as they are: the <<<>>> form hands grid and stream to the kernel's host stub through a stack of the
// runtime's, which costs 0.3 of 2.4 us per launch.
template <typename T> struct Same { using type = T; };
template <typename... P>
hipError_t launch(void (*const kernel)(P...), const uint32_t groups, const uint32_t threads, hipStream_t stream, typename Same<P>::type... args)
{
    void *at[] = {&args...};
    const hipError_t e = hipLaunchKernel(reinterpret_cast<const void *>(kernel), dim3(groups), dim3(threads), at, 0, stream);
    if (e != hipSuccess) (void)hipGetLastError();        // (reported here, not by the caller's next call)
    return e;
}

// Host-side launcher of one instantiation family (fixed bits_m and 1st-moment codebook);
// defined in solo_step_m{2,3,4}{,_de}.hip so that the families compile in parallel.
template <int BM, bool MDE>
hipError_t launch_step(uint32_t bits_v, uint32_t block_size, bool bf16, const StepArgs &args,
                       hipStream_t stream);

template <int BM, int BV, int B, bool BF16, bool MDE>
hipError_t launch_one(const StepArgs &args_in, hipStream_t stream)
{
    StepArgs args = args_in;                   // the tiling belongs to the instantiation
    if (args.n == 0) return hipSuccess;
    const bool narrow = narrow_buffer(args.n, BF16, args.param_bf16 != nullptr);
    const uint64_t whole = narrow ? 0 : args.n / kIter16;
    args.rest = narrow ? pieces8(args.n) : rest_pieces(args.n, whole);      // (narrow: all of them)
    const uint64_t groups = (whole + args.rest + kWaves - 1) / kWaves;
    if (groups > kMaxGroups) return hipErrorInvalidValue;
    const bool ext = args.param_bf16 || args.grad_scale || args.belief || args.l2 != 0.0f;
    const uint32_t grid = (uint32_t)groups, threads = kWaves * 64;
    if (!narrow)
        return launch(ext ? chunk16_kernel<BM, BV, B, BF16, MDE, true> : chunk16_kernel<BM, BV, B, BF16, MDE, false>, grid, threads, stream, args);
    const uint32_t whole8 = (uint32_t)(args.n / kIter), more = (uint32_t)(args.n % kIter) | (uint32_t)(args.rest - whole8) << 16;
    return launch(ext ? chunk8_kernel<BM, BV, B, BF16, MDE, true> : chunk8_kernel<BM, BV, B, BF16, MDE, false>, grid, threads, stream,
                  whole8, more, args.grad, args.m_words, args.v_words, args.m_scale, args.v_scale, args.v_base, args);
}

template <int BM, bool MDE>
hipError_t launch_multi(uint32_t bits_v, uint32_t block_size, bool bf16, const MultiArgs &args,
                        hipStream_t stream);

template <int BM, bool MDE>
hipError_t launch_multi_impl(uint32_t bits_v, uint32_t block_size, bool bf16, const MultiArgs &args,
                             hipStream_t stream)
{
    const StepArgs &c = args.common;
    const bool ext = args.any_bf16_copy || c.grad_scale || c.belief || c.l2 != 0.0f;
    // wavefronts; those behind the last piece find nothing to do (a tensor of 512-element pieces has
    // at most twice as many as of 1024-element ones)
    const uint64_t pieces = args.pieces ? args.pieces : args.total_units * kPiecesPerUnit;
    const bool narrow = pieces <= narrow_table_up_to();
    const uint64_t grid = ((narrow ? 2 * pieces : pieces) + kWaves - 1) / kWaves;
    if (grid == 0 || grid > kMaxGroups || args.count == 0) return hipErrorInvalidValue;
#define SOLO_LAUNCH(BV_, B_, BF_)                                                                       \
    return narrow ? launch(ext ? multi_chunk8_kernel<BM, BV_, B_, BF_, MDE, true> : multi_chunk8_kernel<BM, BV_, B_, BF_, MDE, false>, \
                           (uint32_t)grid, kWaves * 64, stream, args.entries, args.count, args)         \
                  : launch(ext ? multi_chunk16_kernel<BM, BV_, B_, BF_, MDE, true> : multi_chunk16_kernel<BM, BV_, B_, BF_, MDE, false>, \
                           (uint32_t)grid, kWaves * 64, stream, args)
#define SOLO_CASE(BV_, B_)                                                                              \
    if (bits_v == BV_ && block_size == B_) { if (bf16) SOLO_LAUNCH(BV_, B_, true); else SOLO_LAUNCH(BV_, B_, false); }
    SOLO_CASE(2, 64) SOLO_CASE(2, 128) SOLO_CASE(3, 64) SOLO_CASE(3, 128) SOLO_CASE(4, 64) SOLO_CASE(4, 128)
#undef SOLO_CASE
#undef SOLO_LAUNCH
    return hipErrorInvalidValue;
}

template <int BM, bool MDE>
hipError_t launch_step_impl(uint32_t bits_v, uint32_t block_size, bool bf16, const StepArgs &args,
                            hipStream_t stream)
{
#define SOLO_CASE(BV_, B_)                                                             \
    if (bits_v == BV_ && block_size == B_)                                             \
        return bf16 ? launch_one<BM, BV_, B_, true, MDE>(args, stream)                 \
                    : launch_one<BM, BV_, B_, false, MDE>(args, stream);
    SOLO_CASE(2, 64) SOLO_CASE(2, 128) SOLO_CASE(3, 64) SOLO_CASE(3, 128) SOLO_CASE(4, 64) SOLO_CASE(4, 128)
#undef SOLO_CASE
    return hipErrorInvalidValue;
}

}  // namespace solo

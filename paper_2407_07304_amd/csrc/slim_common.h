// Shared device helpers for the gfx950 kernels (wave64, CDNA4).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace slim {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kMasked = -1.0e30f;  // finite stand-in for -inf: exp2(kMasked - m) == 0 for any finite m

__device__ __forceinline__ float bf16_bits_to_f32(unsigned int bits16) { return __uint_as_float(bits16 << 16); }

// Stores of results that nothing in the launch reads again: device scope, so that they go through the L2 to memory at once.  A
// plain store leaves a dirty line, and what is dirty when a launch ends is written back before the next one starts.  Plain stores
// -> these, us (GPU alone, builds in turn): a prefill's rows, bf16, 4 sequences, 32 on 8 heads, S=777 30.7 -> 29.4, one, 32 heads,
// S=1024 19.4 -> 18.4, INT8, 2 sequences, 32 on 8 heads, S=793 27.7 -> 26.6, fp32 results, INT8, S=512 19.3 -> 17.3, bf16, 4, 16 on 2
// heads, S=500 15.1 -> 12.7; from some 50 us a call on within what two runs differ.  One sequence's decode step (the appends'
// stores) 12.2 -> 11.8, 64 on 8 heads, T=32768 (and the splits' records) 20.7 -> 20.5.
// Not for stores in small pieces or at the very end of many small workgroups, which wait for them: the cache rows that a prefill emits
// (one sequence, 8 heads, S=300 7.7 -> 8.4), its results in blocks of 32 rows (16 sequences, 32 on 8 heads, S=200 25.4 -> 26.2), the
// quantiser (32 heads, S=2048 9.7 -> 9.5 to 9.8, 4 sequences, 8 heads, S=4000 16.8 -> 17.2); nor a decode's result row, which gains nothing.
template <class T>
__device__ __forceinline__ void store_through(T* p, const T v) {
    static_assert(sizeof(T) == 4 || sizeof(T) == 8, "one register or two");
    using Bits = std::conditional_t<sizeof(T) == 8, unsigned long long, unsigned>;
    __hip_atomic_store(reinterpret_cast<Bits*>(p), __builtin_bit_cast(Bits, v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// 16 bytes at base + off + step (base and step uniform, off + step below 2^31)
__device__ __forceinline__ void store_through_b128(void* base, int off, int step, u32x4 v) {
    constexpr int kDeviceScope = 16;   // (the cache policy's sc1 bit)
    __builtin_amdgcn_raw_buffer_store_b128(v, __builtin_amdgcn_make_buffer_rsrc(base, 0, 0x7fffffff, 0x00020000), off, step, kDeviceScope);
}

// fp32 -> bf16, round to nearest even (the hardware conversion on gfx950)
__device__ __forceinline__ unsigned int pack_bf16x2(float lo, float hi) {
    bf16x2 v;
    v[0] = (__bf16)lo;
    v[1] = (__bf16)hi;
    return __builtin_bit_cast(unsigned int, v);
}

// signed byte n of a dword, widened exactly to fp32 (INT8 -> INT32 -> FP32, section 2.2)
template <int N>
__device__ __forceinline__ float i8_to_f32(unsigned int w) {
    return (float)(int)(signed char)(w >> (8 * N));
}

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
typedef short s16x8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ s16x4 lds_read_tr16(const uint16_t* p) {
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p));
}

// value of the other 32-lane half of the wave, combined with op: every lane ends with op(lo, hi)
__device__ __forceinline__ float half_max(float x) {
    const unsigned b = __float_as_uint(x);
    const auto sw = __builtin_amdgcn_permlane32_swap(b, b, false, false);
    return fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
}
__device__ __forceinline__ float half_sum(float x) {
    const unsigned b = __float_as_uint(x);
    const auto sw = __builtin_amdgcn_permlane32_swap(b, b, false, false);
    return __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
}

// max over the LPR (4, 8 or 16) adjacent lanes that hold one row, in every one of them: DPP exchanges inside a
// row of 16 lanes (the two quad permutations, then the mirror of 8 and the mirror of 16 lanes), no LDS traffic
template <int CTRL>
__device__ __forceinline__ float dpp_mov_f32(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, false));
}
template <int LPR>
__device__ __forceinline__ float row_group_max(float v) {
    static_assert(LPR == 4 || LPR == 8 || LPR == 16, "a row is held by 4, 8 or 16 adjacent lanes");
    v = fmaxf(v, dpp_mov_f32<0xB1>(v));                  // quad_perm [1,0,3,2]
    v = fmaxf(v, dpp_mov_f32<0x4E>(v));                  // quad_perm [2,3,0,1]
    if (LPR >= 8) v = fmaxf(v, dpp_mov_f32<0x141>(v));   // row_half_mirror: lane i <-> 7 - i of its 8
    if (LPR >= 16) v = fmaxf(v, dpp_mov_f32<0x140>(v));  // row_mirror: lane i <-> 15 - i of its 16
    return v;
}

// The INT8 quantiser of one K or V row (paper section 2.2), shared by the quantiser kernels and the prefill
// kernel that emits the cache.  The definition is scale = fl32(amax / 127) and code = rint(fl32(x / scale)), both
// IEEE fp32 divisions (one rounding each, denormals kept), ties to even.  An IEEE division is about a dozen vector
// instructions, and a row needs one per value, so the common case takes a shorter route that provably lands on
// the same bits, and everything else takes the divisions themselves:
//   scale: q = amax * fl32(1/127), r = fma(-q, 127, amax), scale = fma(r, fl32(1/127), q).  Equal to the IEEE
//          quotient for every bf16 amax in [kQuantFastLo, kQuantFastHi] (all 2^15 values are checked on the host).
//   code:  with y = x * rcp(scale) (v_rcp_f32: within 1 ulp; the product adds half an ulp; |y| < 128), y lies
//          within 2^-15 of the exact quotient and the IEEE quotient within 2^-17 of it, so unless y is within
//          kQuantTieGuard = 2^-14 of a half-integer both round to the same integer (swept on the host over every
//          bf16 pair and every reciprocal within 1.5 ulp).  That integer is read off
//          y + 1.5 * 2^23, whose low mantissa byte is the code in two's complement (the addition itself rounds to
//          nearest even).  (|x| <= amax keeps |code| <= 127: the fast path needs no clamp.)
//   near a tie: y is corrected by its remainder, y + (x - y scale) rcp(scale), two FMAs (Markstein's step to a correctly
//          rounded quotient): the IEEE quotient itself for every bf16 pair with x >= 2^-10 amax (no other is near a tie) and
//          every reciprocal within 1.5 ulp (swept on the host).  Such values are common: x = amax / 2 is the tie 63.5,
//          and of normally distributed rows 7 waves in 10 hold one; while each of them went through eight divisions the
//          quantiser was bound by the vector ALU (two tensors of 32 heads, 2048 tokens, D = 128: 12.7 us, now 10.0).
// A row whose amax lies outside the checked range sends its wave through the divisions.
constexpr float kQuantFastLo = 0x1p-60f, kQuantFastHi = 0x1p60f;   // rows with amax in this range take the fast scale and codes
constexpr float kQuantTieGuard = 0x1p-14f;
constexpr float kQuantMagic = 12582912.0f;   // 1.5 * 2^23

// One row: this lane's 8 values (of the LPR lanes that hold the row) -> its 8 codes and the row's scale.
template <int LPR>
__device__ __forceinline__ void quant_row_piece(const u32x4 raw, u32x2& out2, float& scale) {
    float v[8];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        v[2 * i] = bf16_bits_to_f32(raw[i] & 0xffffu);
        v[2 * i + 1] = __uint_as_float(raw[i] & 0xffff0000u);
    }
    float amax = 0.0f;
#pragma unroll
    for (int i = 0; i < 8; ++i) amax = fmaxf(amax, fabsf(v[i]));
    amax = row_group_max<LPR>(amax);
    const bool in_range = amax >= kQuantFastLo && amax <= kQuantFastHi;
    constexpr float kInv127 = 1.0f / 127.0f;
    const float q127 = amax * kInv127;
    scale = fmaf(fmaf(-q127, 127.0f, amax), kInv127, q127);
    const float inv = __builtin_amdgcn_rcpf(scale);
    unsigned int bits[8];
    float y[8];
    float off_int = 0.0f;   // largest distance of a y from its nearest integer
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        y[i] = v[i] * inv;
        const float f = y[i] + kQuantMagic;
        off_int = fmaxf(off_int, fabsf(y[i] - (f - kQuantMagic)));
        bits[i] = __float_as_uint(f);
    }
    if (__builtin_amdgcn_ballot_w64(!(off_int < 0.5f - kQuantTieGuard)) != 0) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {   // (values that were fine get the same bits again)
            const float quotient = fmaf(fmaf(-y[i], scale, v[i]), inv, y[i]);
            bits[i] = __float_as_uint(quotient + kQuantMagic);
        }
    }
    // byte 0 of four words -> one word
    out2[0] = __builtin_amdgcn_perm(__builtin_amdgcn_perm(bits[3], bits[2], 0x0c0c0400u),
                                    __builtin_amdgcn_perm(bits[1], bits[0], 0x0c0c0400u), 0x05040100u);
    out2[1] = __builtin_amdgcn_perm(__builtin_amdgcn_perm(bits[7], bits[6], 0x0c0c0400u),
                                    __builtin_amdgcn_perm(bits[5], bits[4], 0x0c0c0400u), 0x05040100u);
    if (__builtin_amdgcn_ballot_w64(!in_range) != 0) {
        // the definition itself, for every lane of the wave (lanes that were fine get the same bits again)
        scale = amax / 127.0f;   // IEEE division, one rounding
        unsigned int packed[2] = {0u, 0u};
        if (amax != 0.0f) {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                float r = rintf(v[i] / scale);   // IEEE division, then ties-to-even
                r = fminf(fmaxf(r, -127.0f), 127.0f);
                packed[i / 4] |= ((unsigned int)(int)r & 0xffu) << (8 * (i % 4));
            }
        }
        out2[0] = packed[0];
        out2[1] = packed[1];
    }
}

// Decode: how many of a call's n_split splits a sequence of T tokens uses: split_rate a token (in units of 2^-32; the plan
// for equal lengths has no more splits than tokens and a rate that gives every sequence all of them).
constexpr unsigned kAllSplits = 0xffffffffu;
__device__ __forceinline__ int splits_of(int T, int n_split, unsigned split_rate) {
    return min(n_split, (int)__umulhi((unsigned)T - 1u, split_rate) + 1);
}

// The chunks [begin, end) of split sp where n chunks are dealt evenly, in order, over n_used splits (the first ones take one
// more).  In 32 bits: n * sp / n_used in 64 is a division of some 150 scalar instructions, and a workgroup's first load waits
// for two of them.  (What that gives is within what two runs of one build differ: B=1, 64 on 8 heads, T=32768 23.6 and 23.3 us a step.)
__device__ __forceinline__ void split_span(int n, int n_used, int sp, int& begin, int& end) {
    const unsigned q = n_used == 1 ? (unsigned)n : (unsigned)n / (unsigned)n_used, r = (unsigned)n - q * (unsigned)n_used;
    begin = (int)(q * (unsigned)sp + min((unsigned)sp, r));
    end = begin + (int)q + ((unsigned)sp < r ? 1 : 0);
}

// A split's record for the launch that merges: accumulator (a thread a value), max and sum.  `through`: see store_through; the rule
// is with the plan.
template <int D>
__device__ __forceinline__ void store_record(float* ws_acc, float* ws_ml, long idx, int d, float acc, float M, float L, bool through) {
    float* const ap = ws_acc + idx * D + d;
    f32x2* const mlp = reinterpret_cast<f32x2*>(ws_ml) + idx;
    if (through) {
        store_through(ap, acc);
        if (d == 0) store_through(mlp, f32x2{M, L});
    } else {
        *ap = acc;
        if (d == 0) *mlp = f32x2{M, L};
    }
}

// sum and max over a wave, wave-uniform
__device__ __forceinline__ int wave_sum(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xf, 0xf, false);    // quad_perm [1,0,3,2]
    v += __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xf, 0xf, false);    // quad_perm [2,3,0,1]
    v += __builtin_amdgcn_update_dpp(0, v, 0x141, 0xf, 0xf, false);   // row_half_mirror
    v += __builtin_amdgcn_update_dpp(0, v, 0x140, 0xf, 0xf, false);   // row_mirror
    return __builtin_amdgcn_readlane(v, 0) + __builtin_amdgcn_readlane(v, 16) + __builtin_amdgcn_readlane(v, 32) + __builtin_amdgcn_readlane(v, 48);
}
__device__ __forceinline__ int wave_max(int v) {
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xf, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xf, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x141, 0xf, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x140, 0xf, 0xf, false));
    return max(max(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 16)), max(__builtin_amdgcn_readlane(v, 32), __builtin_amdgcn_readlane(v, 48)));
}

// Decode over `batch` (2 to kMaxRanked) sequences of different lengths, a workgroup for each of a sequence's `heads` rows: the
// row that workgroup (b0, h0) of the grid takes.  Workgroup ids go to the compute units in turn (id mod 8 is the XCD, whose
// 32 units each get one before one gets a second: the same unit for ids 256 apart).  In the order of the grid two long rows may meet
// on one unit while another has two short ones, and the call takes as long as the former.  So the rows are dealt
// longest first in layers of 256, and every other layer runs backwards: a unit's longest row meets the shortest of the next layer.
// The last layer runs forwards: where it is not full, the units it leaves out have the longest rows of the layer
// before.  (Where an id lands only decides about time: every row is worked off as it was, by one workgroup.  Forms of which fewer
// workgroups fit a unit than there are layers take the later rows where one ends, layer by layer: the figures are with the plan.)
// Lengths spread over an eighth to all of the cache, a fourth of them full and the others an eighth, all equal, us:
//   48 sequences, 32 on 8 heads, T=3001 37.9 -> 33.2, 38.2 -> 28.8, 51.0 -> 51.5; 16, 32 heads, T=3000 42.8 -> 39.8, 37.3 ->
//   26.7, 61.6 -> 61.8; 40, 8 heads, T=1000 14.6 -> 11.7, 13.8 -> 9.5, 18.1 -> 18.3; 64, 64 on 8 heads, D=64, T=2000 19.5 ->
//   19.2, 19.1 -> 17.9, 24.5 -> 24.7.
// Every wave finds its row by itself, with one load: lane l has the lengths of sequences l and l + 64 in chunks of 64 tokens, and
// the chunks of the sequence of a given rank are found bit by bit, by counting lanes.  No LDS and no barrier (ranks counted in LDS
// took 0.7 us more).  Where the longest is within 256 tokens or an eighth of the mean the rows keep their order.
constexpr int kMaxRanked = 128;
struct SequenceHead {
    int b, h, T;   // sequence, head, the sequence's length
};
__device__ __forceinline__ SequenceHead ranked_row(const int* __restrict__ kv_lens, int batch, int heads, int T_alloc, int b0, int h0) {
    constexpr int NI = kMaxRanked / 64;
    typedef int lens_t __attribute__((ext_vector_type(NI)));
    const int lane = (int)threadIdx.x & 63;
    lens_t len = 0, c;   // (0 past the last sequence)
#pragma unroll
    for (int i = 0; i < NI; ++i)
        if (64 * i < batch && lane + 64 * i < batch) len[i] = min(max(kv_lens[lane + 64 * i], 1), T_alloc);
    c = (len + 63) >> 6;
    int total = c[0], most = c[0];
#pragma unroll
    for (int i = 1; i < NI; ++i) {
        total += c[i];
        most = max(most, c[i]);
    }
    most = wave_max(most);
    total = wave_sum(total);
    auto length_of = [&](int b) {   // (b is uniform)
        int x = __builtin_amdgcn_readlane(len[0], b & 63);
        if (batch > 64) {
#pragma unroll
            for (int i = 1; i < NI; ++i) {
                const int y = __builtin_amdgcn_readlane(len[i], b & 63);
                x = (b >> 6) == i ? y : x;
            }
        }
        return x;
    };
    if (most * batch <= max(total + 4 * batch, total + total / 8)) return SequenceHead{b0, h0, length_of(b0)};
    const int id = b0 * heads + h0, layer = id >> 8, p = id & 255, last = (batch * heads - 1) >> 8;
    const int row = 256 * layer + (((last - layer) & 1) ? 255 - p : p);
    // (a row's index is small: the quotient by a reciprocal is off by less than the half that is added keeps it from an integer)
    const int rank = __builtin_amdgcn_readfirstlane((int)(((float)row + 0.5f) * __builtin_amdgcn_rcpf((float)heads)));
    // the greatest length that more than `rank` sequences have, and how many are longer
    int chunks = 0, longer = 0;
    for (int bit = 1 << (31 - __builtin_clz(most)); bit != 0; bit >>= 1) {
        int n = __builtin_popcountll(__builtin_amdgcn_ballot_w64(c[0] >= (chunks | bit)));
        if (batch > 64)
#pragma unroll
            for (int i = 1; i < NI; ++i) n += __builtin_popcountll(__builtin_amdgcn_ballot_w64(c[i] >= (chunks | bit)));
        if (n > rank) chunks |= bit;
        else longer = n;
    }
    // of those that have it, in order
    int nth = rank - longer, b = 0;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        if (64 * i >= batch) break;
        const unsigned long long same = __builtin_amdgcn_ballot_w64(c[i] == chunks);
        const int before = __builtin_amdgcn_mbcnt_hi((unsigned)(same >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)same, 0u));
        const unsigned long long here = __builtin_amdgcn_ballot_w64(c[i] == chunks && before == nth);
        if (here != 0) b = 64 * i + __builtin_ctzll(here);
        nth -= __builtin_popcountll(same);
    }
    return SequenceHead{b, row - rank * heads, length_of(b)};
}

}  // namespace slim

// Decode attention over the INT8 KV cache (paper section 2.2: next-token attention is a
// matrix-vector product bound by memory bandwidth; cached INT8 values are widened to FP32
// in registers and fed to FMAs, with one scale per token per head).
//
// HBM-bound streaming kernel.  A workgroup of 4 or 8 waves serves one (batch, query head) and
// one split of the key axis (the whole of it wherever equal rows alone fill the chip); its
// chunks of 64 tokens are dealt to the waves in turn, so that the workgroup sweeps one
// contiguous piece of the cache (on the B=16, 32 heads, T=8192 cache 8 % faster than a
// contiguous run of 512 tokens per wave, which 6.1 TB/s was the ceiling of):
//   - a token row of D codes is read by D/16 adjacent lanes ("slot") with one 128-bit
//     load each, so one load instruction of a wave fetches 64/(D/16) whole rows, and the
//     wave's loads of a chunk cover one contiguous piece of K and one of V;
//   - the K and V loads of chunk c+1 are issued before chunk c is consumed, so a wave
//     always has a chunk of 128-bit loads in flight;
//   - lane i of the wave owns token i of the chunk: it loads that token's two scales
//     (coalesced), keeps its score, and computes ONE exponential per chunk;
//   - each slot carries its own running max / sum (online softmax, fp32), so the only
//     cross-lane traffic in the loop is DPP adds inside a slot and a 256-byte LDS
//     exchange of the chunk's probabilities;
//   - slots and waves are merged in LDS at the end, and where there are several splits a second
//     kernel merges them in a fixed order (no atomics: the result does not depend on arrival order).
#include <algorithm>
#include <mutex>
#include <type_traits>

#include "slim_common.h"
#include "slim_kernels.h"

namespace slim {

constexpr int kChunk = 64;   // tokens per wave per chunk

// lane exchange inside a slot via DPP (no LDS traffic); every lane of the slot ends with the slot total
template <int CTRL>
__device__ __forceinline__ float dpp_f32(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, false));
}
template <int LPR>
__device__ __forceinline__ float slot_sum(float v) {
    v += dpp_f32<0xB1>(v);                 // quad_perm [1,0,3,2]
    v += dpp_f32<0x4E>(v);                 // quad_perm [2,3,0,1]
    if (LPR == 8) v += dpp_f32<0x141>(v);  // row_half_mirror: the other quad of the 8 lanes
    return v;
}
template <int LPR>
__device__ __forceinline__ float slot_max(float v) {
    v = fmaxf(v, dpp_f32<0xB1>(v));
    v = fmaxf(v, dpp_f32<0x4E>(v));
    if (LPR == 8) v = fmaxf(v, dpp_f32<0x141>(v));
    return v;
}

// D head dimension, W waves per workgroup
template <int D, int W>
__global__ __launch_bounds__(64 * W) void slim_decode_int8_split_kernel(
    const uint16_t* __restrict__ q, const int8_t* __restrict__ kc, const float* __restrict__ ks,
    const int8_t* __restrict__ vc, const float* __restrict__ vs, uint16_t* __restrict__ out,
    float* __restrict__ ws_acc, float* __restrict__ ws_ml, const int* __restrict__ kv_lens, int group, int Hkv, int T_alloc,
    int n_split, unsigned split_rate, int mode, float scale_log2e) {
    constexpr int LPR = D / 16;        // lanes per token row
    constexpr int SLOTS = 64 / LPR;    // token rows per load instruction of a wave
    constexpr int CH = LPR;            // rows per slot per chunk: SLOTS * CH == kChunk, one token per lane
    constexpr int PARTS = 64 * W / D;  // threads that share an output column at the merge

    __shared__ __attribute__((aligned(16))) float pvS[W][kChunk];
    __shared__ __attribute__((aligned(16))) float accS[W][SLOTS][D];
    __shared__ float lS[W];
    __shared__ float mS[W];
    __shared__ float oS[PARTS][D];

    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));   // (the wave index as a scalar: everything derived from it stays uniform)
    const int c = lane % LPR, s = lane / LPR;
    // T_alloc is the cache's allocated length (the row stride); this sequence's first T tokens count
    int h = blockIdx.y, b = blockIdx.z, T;
    const int sp = blockIdx.x;
    if (mode > 0) {   // (dealt by length; one split)
        const SequenceHead row = ranked_row(kv_lens, mode, group * Hkv, T_alloc, b, h);
        h = row.h;
        b = row.b;
        T = row.T;
    } else {
        T = kv_lens ? min(max(kv_lens[b], 1), T_alloc) : T_alloc;
    }
    const int Hq = group * Hkv, g = group == 1 ? h : h / group;   // (group query heads per KV head)
    const int n_used = splits_of(T, n_split, split_rate);
    if (sp >= n_used) return;   // (nobody reads this split's record)
    const long kvbase = ((long)b * Hkv + g) * (long)T_alloc;
    // Buffer descriptors over exactly this (batch, KV head)'s first T tokens: a row past the end reads as zeros (and
    // is masked below), an address is one 32-bit offset per lane plus a constant per row, and the descriptors live in
    // scalar registers (with pointers and clamped row indices the addresses of a chunk's loads took some eighty
    // vector instructions and a dozen more vector registers).
    const __amdgpu_buffer_rsrc_t krs = __builtin_amdgcn_make_buffer_rsrc((void*)(kc + kvbase * D), 0, (int)((unsigned)T * D), 0x00020000);
    const __amdgpu_buffer_rsrc_t vrs = __builtin_amdgcn_make_buffer_rsrc((void*)(vc + kvbase * D), 0, (int)((unsigned)T * D), 0x00020000);
    const __amdgpu_buffer_rsrc_t ksr = __builtin_amdgcn_make_buffer_rsrc((void*)(ks + kvbase), 0, (int)((unsigned)T * 4u), 0x00020000);
    const __amdgpu_buffer_rsrc_t vsr = __builtin_amdgcn_make_buffer_rsrc((void*)(vs + kvbase), 0, (int)((unsigned)T * 4u), 0x00020000);
    const int lane_off = (s * CH) * D + c * 16;   // this lane's piece of its slot's first row, relative to the chunk
    // The sequence's own chunks are dealt evenly over its splits, and a split's chunks to its waves in turn: the
    // waves of a workgroup read adjacent pieces of the cache at a time.
    const int n_all = (T + kChunk - 1) / kChunk;
    int c_begin, c_end;
    split_span(n_all, n_used, sp, c_begin, c_end);
    c_begin += w;
    const int n_chunks = c_begin < c_end ? (c_end - c_begin + W - 1) / W : 0;

    // this lane's 16 query values, fp32
    float qf[16];
    {
        const uint16_t* qp = q + ((long)b * Hq + h) * D + c * 16;
        const u32x4 q0 = *reinterpret_cast<const u32x4*>(qp);
        const u32x4 q1 = *reinterpret_cast<const u32x4*>(qp + 8);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            qf[2 * i] = bf16_bits_to_f32(q0[i] & 0xffffu);
            qf[2 * i + 1] = __uint_as_float(q0[i] & 0xffff0000u);
            qf[8 + 2 * i] = bf16_bits_to_f32(q1[i] & 0xffffu);
            qf[8 + 2 * i + 1] = __uint_as_float(q1[i] & 0xffff0000u);
        }
    }

    float acc[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = 0.0f;
    float m = kMasked, l = 0.0f;   // slot max (identical in the slot's lanes), this lane's part of the slot sum

    u32x4 kbuf[CH], vbuf[CH];
    float ksc = 0.0f, vsc = 0.0f;
    // the codes are read once per step, so their loads are non-temporal (measured: 5.6 -> 6.3 TB/s on the B=16,
    // T=8192 cache)
    auto issue_k = [&](int t_chunk0) {
        const int off = t_chunk0 * D + lane_off;
#pragma unroll
        for (int it = 0; it < CH; ++it) kbuf[it] = __builtin_amdgcn_raw_buffer_load_b128(krs, off + it * D, 0, 2 /* nt */);
        ksc = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(ksr, (t_chunk0 + lane) * 4, 0, 0));
    };
    auto issue_v = [&](int t_chunk0) {
        const int off = t_chunk0 * D + lane_off;
        // (the scale first: it is wanted before the codes, and loads complete in order, so a wait for a scale
        // issued after the codes would be a wait for the codes)
        vsc = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(vsr, (t_chunk0 + lane) * 4, 0, 0));
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int it = 0; it < CH; ++it) vbuf[it] = __builtin_amdgcn_raw_buffer_load_b128(vrs, off + it * D, 0, 2 /* nt */);
    };

    // unconditional (a wave past the end gets zeros and reads nothing): keeps the prologue free of branches
    const int t_first = n_chunks > 0 ? c_begin * kChunk : T;
    issue_k(t_first);
    issue_v(t_first);
    // one chunk; PREFETCH is a compile-time flag so the loop body has no branch around its loads
    auto chunk = [&](int ch, auto prefetch) {
        constexpr bool more = decltype(prefetch)::value;
        const int t_chunk0 = (c_begin + ch * W) * kChunk;

        // scores: the slot's CH rows; lane c of the slot keeps row c (token t_chunk0 + lane)
        float my_dot = 0.0f;
#pragma unroll
        for (int it = 0; it < CH; ++it) {
            const u32x4 kw = kbuf[it];
            float dot = 0.0f;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                dot = fmaf(qf[4 * i + 0], i8_to_f32<0>(kw[i]), dot);
                dot = fmaf(qf[4 * i + 1], i8_to_f32<1>(kw[i]), dot);
                dot = fmaf(qf[4 * i + 2], i8_to_f32<2>(kw[i]), dot);
                dot = fmaf(qf[4 * i + 3], i8_to_f32<3>(kw[i]), dot);
            }
            dot = slot_sum<LPR>(dot);
            my_dot = (c == it) ? dot : my_dot;
        }
        const bool valid = t_chunk0 + lane < T;
        const float my_s = valid ? my_dot * (ksc * scale_log2e) : kMasked;
        if constexpr (more) issue_k(t_chunk0 + W * kChunk);

        const float m_new = fmaxf(m, slot_max<LPR>(my_s));
        const float alpha = fast_exp2(m - m_new);
        float p = fast_exp2(my_s - m_new);
        p = valid ? p : 0.0f;
        l = fmaf(l, alpha, p);
        pvS[w][lane] = p * vsc;   // probability times the token's V scale
        if (__builtin_amdgcn_ballot_w64(m_new > m) != 0) {
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[i] *= alpha;
        }
        m = m_new;

        float pv[CH];
#pragma unroll
        for (int i = 0; i < CH / 4; ++i) {
            const f32x4 t4 = *reinterpret_cast<const f32x4*>(&pvS[w][s * CH + 4 * i]);
            pv[4 * i] = t4[0];
            pv[4 * i + 1] = t4[1];
            pv[4 * i + 2] = t4[2];
            pv[4 * i + 3] = t4[3];
        }
#pragma unroll
        for (int it = 0; it < CH; ++it) {
            const u32x4 vw = vbuf[it];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                acc[4 * i + 0] = fmaf(pv[it], i8_to_f32<0>(vw[i]), acc[4 * i + 0]);
                acc[4 * i + 1] = fmaf(pv[it], i8_to_f32<1>(vw[i]), acc[4 * i + 1]);
                acc[4 * i + 2] = fmaf(pv[it], i8_to_f32<2>(vw[i]), acc[4 * i + 2]);
                acc[4 * i + 3] = fmaf(pv[it], i8_to_f32<3>(vw[i]), acc[4 * i + 3]);
            }
        }
        if constexpr (more) issue_v(t_chunk0 + W * kChunk);
    };
    for (int ch = 0; ch + 1 < n_chunks; ++ch) chunk(ch, std::true_type{});
    if (n_chunks > 0) chunk(n_chunks - 1, std::false_type{});

    // Merge: the slots of a wave are brought to the wave's maximum in registers, then PARTS threads per output column
    // add up their share of the waves' slots from LDS, and one of them the parts.
    l = slot_sum<LPR>(l);
    float m_wave = m;
#pragma unroll
    for (int x = LPR; x < 64; x *= 2) m_wave = fmaxf(m_wave, __shfl_xor(m_wave, x));
    {
        const float f = fast_exp2(m - m_wave);   // an empty slot has l = 0 and acc = 0
        l *= f;
#pragma unroll
        for (int x = LPR; x < 64; x *= 2) l += __shfl_xor(l, x);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            f32x4 a4 = {acc[4 * i] * f, acc[4 * i + 1] * f, acc[4 * i + 2] * f, acc[4 * i + 3] * f};
            *reinterpret_cast<f32x4*>(&accS[w][s][c * 16 + 4 * i]) = a4;
        }
        if (lane == 0) {
            lS[w] = l;
            mS[w] = m_wave;
        }
    }
    __syncthreads();
    float M = kMasked;
#pragma unroll
    for (int ww = 0; ww < W; ++ww) M = fmaxf(M, mS[ww]);
    const int d = threadIdx.x % D, part = threadIdx.x / D;
    float o = 0.0f;
#pragma unroll
    for (int i = 0; i < W / PARTS; ++i) {
        const int ww = part * (W / PARTS) + i;
        float a = 0.0f;
#pragma unroll
        for (int ss = 0; ss < SLOTS; ++ss) a += accS[ww][ss][d];
        o = fmaf(fast_exp2(mS[ww] - M), a, o);
    }
    oS[part][d] = o;
    __syncthreads();
    if (threadIdx.x < D) {
        float L = 0.0f;
        o = 0.0f;
#pragma unroll
        for (int ww = 0; ww < W; ++ww) L = fmaf(fast_exp2(mS[ww] - M), lS[ww], L);
#pragma unroll
        for (int i = 0; i < PARTS; ++i) o += oS[i][d];
        const long bh = (long)b * Hq + h;
        if (n_used == 1) {
            out[bh * D + d] = (uint16_t)(pack_bf16x2(o / L, 0.0f) & 0xffffu);
        } else {
            store_record<D>(ws_acc, ws_ml, bh * n_split + sp, d, o, M, L, mode < 0);
        }
    }
}

// Merges the n_split partial (max, sum, accumulator) triples of one (batch, head) in a fixed order (records dealt to lane
// groups and waves, each group's in turn, then the groups by halves, then the waves) and writes the bf16 output row.  The launch is latency-bound (a few kilobytes per row, just written by the split kernel), so a row's records
// come in with few, wide loads that are all issued before anything is computed: D/4 lanes read a record with one 128-bit
// load each, a wave RPW = 256/D records at a time.  Up to U RPW records a row one wave does it, and a workgroup has four
// rows; more are shared by the four waves of a workgroup and merged through LDS.  Slots past the last split re-read the last
// one and count as empty (max = kMasked, sum = 0); runs longer than the slots take another pass with a running (max, sum,
// accumulator).  With a thread for every output value and sixteen records a thread (32-bit loads, 512 threads a row beyond sixteen
// splits) the wide form's decode took, before -> now: 64 on 8 heads, T=32768, 32 splits 18.6 -> 16.1 us, D=64 14.7 -> 12.6; 8
// heads, T=16000, 32 splits 11.8 -> 9.5; 32 heads, T=4000, 8 splits 9.5 -> 9.2; 16 sequences, 64 on 8 heads, T=8192, 2 splits 45.2 ->
// 44.6.
template <int D, int WAVES, int U>
__global__ __launch_bounds__(256) void slim_decode_combine_kernel(const float* __restrict__ ws_acc, const float* __restrict__ ws_ml,
                                                                  uint16_t* __restrict__ out, const int* __restrict__ kv_lens,
                                                                  int q_heads, long rows, int T_alloc, int n_split, unsigned split_rate) {
    constexpr int LPR = D / 4, RPW = 64 / LPR;
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int c = lane % LPR, sub = lane / LPR;
    const long bh = (long)blockIdx.x * (4 / WAVES) + (WAVES == 1 ? w : 0);
    if (bh >= rows) return;
    const int part = WAVES == 1 ? 0 : w;
    const int n_used = splits_of(kv_lens ? min(max(kv_lens[(unsigned)bh / (unsigned)q_heads], 1), T_alloc) : T_alloc, n_split, split_rate);
    if (n_used == 1) return;   // (its one workgroup has written the result)
    const f32x2* const ml = reinterpret_cast<const f32x2*>(ws_ml) + bh * n_split;
    const f32x4* const acc = reinterpret_cast<const f32x4*>(ws_acc) + bh * n_split * LPR + c;
    float M = kMasked, L = 0.0f;
    f32x4 o = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int s0 = 0; s0 < n_used; s0 += WAVES * RPW * U) {
        float m[U], l[U];
        f32x4 a[U];
#pragma unroll
        for (int i = 0; i < U; ++i) {
            const int s = s0 + (i * WAVES + part) * RPW + sub, sp = min(s, n_used - 1);
            const f32x2 t = ml[sp];
            const f32x4 av = acc[(long)sp * LPR];
            m[i] = s < n_used ? t[0] : kMasked;
            l[i] = s < n_used ? t[1] : 0.0f;
            a[i] = s < n_used ? av : f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        }
        float m_new = M;
#pragma unroll
        for (int i = 0; i < U; ++i) m_new = fmaxf(m_new, m[i]);
        const float keep = fast_exp2(M - m_new);   // first pass: L = o = 0, whatever this is
        L *= keep;
        o *= keep;
#pragma unroll
        for (int i = 0; i < U; ++i) {
            const float f = fast_exp2(m[i] - m_new);   // an empty split has sum = 0 and accumulator = 0
            L = fmaf(f, l[i], L);
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = fmaf(f, a[i][e], o[e]);
        }
        M = m_new;
    }
    // the wave's groups of lanes, by halves
#pragma unroll
    for (int x = LPR; x < 64; x *= 2) {
        const float m_other = __shfl_xor(M, x), l_other = __shfl_xor(L, x), m_new = fmaxf(M, m_other);
        const float f = fast_exp2(M - m_new), g = fast_exp2(m_other - m_new);
        L = fmaf(L, f, l_other * g);
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = fmaf(o[e], f, __shfl_xor(o[e], x) * g);
        M = m_new;
    }
    if constexpr (WAVES > 1) {
        __shared__ __attribute__((aligned(16))) f32x4 oS[WAVES][LPR];
        __shared__ float mS[WAVES], lS[WAVES];
        if (sub == 0) oS[w][c] = o;
        if (lane == 0) {
            mS[w] = M;
            lS[w] = L;
        }
        __syncthreads();
        if (w != 0) return;
        M = kMasked;
#pragma unroll
        for (int i = 0; i < WAVES; ++i) M = fmaxf(M, mS[i]);
        L = 0.0f;
        o = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int i = 0; i < WAVES; ++i) {
            const float f = fast_exp2(mS[i] - M);
            L = fmaf(f, lS[i], L);
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = fmaf(f, oS[i][c][e], o[e]);
        }
    }
    if (sub == 0) {
        u32x2 ov;
        ov[0] = pack_bf16x2(o[0] / L, o[1] / L);
        ov[1] = pack_bf16x2(o[2] / L, o[3] / L);
        *reinterpret_cast<u32x2*>(out + bh * D + 4 * c) = ov;
    }
}

static hipError_t launch_combine(const DecodeArgs& a, const float* ws_acc, const float* ws_ml, int n_split, unsigned split_rate,
                                 hipStream_t stream) {
    const long rows = (long)a.batch * a.q_heads;
    auto launch = [&](auto d_c, auto waves_c, auto u_c) {
        constexpr int D = decltype(d_c)::value, WAVES = decltype(waves_c)::value, U = decltype(u_c)::value;
        const unsigned grid = (unsigned)((rows * WAVES + 3) / 4);
        hipLaunchKernelGGL((slim_decode_combine_kernel<D, WAVES, U>), dim3(grid), dim3(256), 0, stream, ws_acc, ws_ml, (uint16_t*)a.out,
                           a.kv_lens, a.q_heads, rows, a.kv_len, n_split, split_rate);
        return hipGetLastError();
    };
    auto pick = [&](auto d_c) {
        using std::integral_constant;
        constexpr int RPW = 256 / decltype(d_c)::value;
        const integral_constant<int, 1> one{};
        const integral_constant<int, 4> four{};
        if (n_split <= 2 * RPW) return launch(d_c, one, integral_constant<int, 2>{});
        if (n_split <= 4 * RPW) return launch(d_c, one, four);
        if (n_split <= 16 * RPW) return launch(d_c, four, four);
        return launch(d_c, four, integral_constant<int, 8>{});
    };
    return a.head_dim == 128 ? pick(std::integral_constant<int, 128>{}) : pick(std::integral_constant<int, 64>{});
}

// Splits of the key axis and waves per workgroup.  Modelled time of S splits of n_bh rows on 256 compute units, the
// constants from a sweep of 17 row counts (8 to 2048) by 15 lengths (128 to 32768), K and V cold:
//   - the cache at 6.6 TB/s, or the fullest compute unit's tokens at its own pace (7.1 ns a token of 128 codes, 5.8 of
//     64: its vector ALU and its share of the memory): the longer of the two and a fifth of the
//     shorter;
//   - 6 us for the combine launch when S > 1.  Where that gives no compute unit a second workgroup and the step is long enough, the
//     splits are chosen again among those of which that holds, with 4.8 us (5.75 of 64 codes a token), and up to three splits may
//     have three chunks and leave a wave idle (4 sequences, 32 heads, T=2000 a step 19.6 -> 18.2 us, D=64 16.5 -> 14.3).
//     That is at the upper end of what splitting whole rows costs beyond the sweep as modelled: over 19 shapes of 64 to 128 rows,
//     T=1000 to 3000, cut in 2 to 4, 3.0 to 4.7 us by the GPU alone, over 7 of 64 codes 3.9 to 4.5.  (Of the grouped kernel's, less: a
//     fit of its model, not of the merge, which is one kernel: in a trace 2.0 to 5.5 us, 3.7 on average for 64 rows of 32 records, 4.6
//     for 1024 of 2.)
// Long enough (appends, decode, merge: from the host a step of four launches takes 13.4 to 13.9 us whatever it computes): rows that are
// split anyway from kDecodeLongNs on; whole ones from 9.4 us on (10 of 64 codes), lengths of their own by the longest of as many
// lengths spread over an eighth to all of the cache, which is what the call then waits for.  Over 44 shapes about those lines, D=128 and
// 64, steps that stay whole would lose 0 to 21 %, those that are split gain 1 to 11 % (21 sequences, 4 heads, T=1590, D=64, lengths
// spread: 11.3 us whole, 13.7 in three; 3, 32 heads, T=1466 13.1 and 13.7, T=1500 14.3 and 13.8).
// So a (batch, head) is split only where one workgroup each cannot load the chip evenly or soon enough, and whole
// caches go through one launch from about 150 rows on (B=16, 32 heads, T=8192: 161 us in one launch of eight-wave
// workgroups, 164 us as 4 splits).  A split has a chunk for each of four waves, but for the up to three above, and a call is not
// split into more records than the library's own scratch holds (that many are 126 workgroups per compute unit and more, where a finer
// split gains nothing): what decides whether slim_attn_decode_int8_static takes a shape is then its rows alone.
// longest: of sequences with lengths of their own, the expected part of kv_len that the longest has
static DecodePlan decode_plan(int kv_len, long n_bh, int head_dim, double longest) {
    const long n_chunks = ((long)kv_len + kChunk - 1) / kChunk;
    const double ns_token = head_dim == 128 ? 7.1 : 5.8;
    const double stream_ns = (double)kv_len * n_bh * (2 * head_dim + 8) / 6600.0;
    int best = 1, alone_best = 1;
    double best_ns = 0.0, alone_best_ns = 0.0, whole_ns = 0.0;
    for (int s : {1, 2, 3, 4, 6, 8, 12, 16, 24, 32, 48, 64, 96, 128, 192, 256}) {
        if (s > 1 && (s * 4 > n_chunks + 3 || decode_records_bytes(n_bh, s, head_dim) > kDecodeStaticScratchBytes)) break;
        const long per_wg = (n_chunks + s - 1) / s, rounds = (n_bh * s + 255) / 256;
        const double busy_ns = (double)(rounds * per_wg * kChunk) * ns_token;
        const double longer = busy_ns > stream_ns ? busy_ns : stream_ns, shorter = busy_ns > stream_ns ? stream_ns : busy_ns;
        const double sweep_ns = longer + 0.2 * shorter, ns = sweep_ns + (s > 1 ? 6000.0 : 0.0);
        if (s == 1) whole_ns = ns;
        if (s == 1 || (ns < best_ns && s * 4 <= n_chunks)) {
            best_ns = ns;
            best = s;
        }
        const double alone_ns = sweep_ns + (s == 1 ? 0.0 : head_dim == 128 ? 4800.0 : 5750.0);
        if (s == 1 || (alone_ns < alone_best_ns && n_bh * s <= 256)) {
            alone_best_ns = alone_ns;
            alone_best = s;
        }
    }
    const bool long_enough = best > 1 ? whole_ns > kDecodeLongNs : whole_ns * longest > (head_dim == 128 ? 9400.0 : 10000.0);
    if (long_enough && n_bh * best <= 256) best = alone_best;
    // eight waves share a merge where each still gets a few chunks (a chunk each, two of 64 codes a token, is
    // enough once several workgroups per compute unit overlap: 800 x 8 heads, T=500, D=64, 77.8 us with eight
    // waves, 72.4 with four, and with lengths of their own, where half of the eight had nothing, 60.6 and 45.9)
    const long per_wg = (n_chunks + best - 1) / best;
    return DecodePlan{per_wg >= (n_bh * best >= 512 ? (head_dim == 128 ? 8 : 16) : 24) ? 8 : 4, best, kAllSplits};
}

// The plan for sequences of different lengths (kv_lens; the host knows only the allocated length).  The plan for equal
// lengths cuts no finer than those need, and a sequence much longer than the others would then be a serial chain on an
// idle chip.  So, where one sequence makes fewer than 128 workgroups, all at full length get about 1536 of them (768 of
// the grouped kernel, whose tokens cost half as much) of at least 2048 tokens (the grouped kernel: 4096 of 128 codes);
// a shorter sequence takes a split per 512 tokens until it has them all, and the workgroups past that leave at once.
// Microseconds cut as for equal lengths -> now, one sequence of full length among sequences of 512 tokens, then lengths
// spread over an eighth to all of the cache, then all equal, then all of 300 tokens:
//   8 sequences, 32 heads, T=65536: 303 -> 87, 432 -> 373, 623 -> 629, 6 -> 13
//   32 sequences, 8 heads, T=16384: 78 -> 24, 113 -> 107, 160 -> 165, 7 -> 13
//   16 sequences, 32 on 8 heads, T=32768: 117 -> 47, 126 -> 108, 159 -> 167, 10 -> 9
//   4 sequences, 64 on 8 heads, T=65536: 64 -> 39, 65 -> 60, 84 -> 87, 9 -> 12
// (Two, four or eight workgroups a row are the worse choice: the long rows' workgroups meet on the same compute units.
// With lengths spread as above and a split per T / n tokens 4 a row were 2 to 7 % slower than 6 with 256 rows.)
static DecodePlan ragged_plan(DecodePlan plan, bool gqa, int batch, int q_heads, int kv_heads, int kv_len, int head_dim) {
    if (batch == 1) return plan;   // (equal cuts: a lone sequence is dealt over all of them)
    const long heads = gqa ? kv_heads : q_heads, rows = batch * heads;
    if (heads * plan.n_split < 128) {
        const long wanted = gqa ? 768 / rows : (1536 + rows - 1) / rows;
        const long room = (long)(kDecodeStaticScratchBytes / decode_records_bytes((long)batch * q_heads, 1, head_dim));
        const long n = std::min({wanted, (long)kv_len / (gqa ? 32 * head_dim : 2048), room});
        if (n > plan.n_split) plan = DecodePlan{gqa && q_heads / kv_heads <= 16 ? 4 : 8, (int)n, 1u << 23 /* 2^32 / 512 */};
    }
    // The grouped kernel's waves, 64 codes a token: eight where no compute unit has two workgroups (15 shapes of 240 to 256
    // workgroups: lengths spread over an eighth to all of the cache 1 to 40 % faster than with four, all equal 1 to 30 %, 32
    // sequences, 32 on 8 heads, T=3000 20.7 and 14.8 us, 24.5 and 19.3; all of 300 to 700 tokens 2 % slower to 15 % faster).
    // Not of 128 codes: up to 256 workgroups lengths so spread gain up to 14 %, but equal ones lose 2 to 6 % (16 sequences, 32
    // on 8 heads, T=8192 46.3 and 49.1 us), and above, where twelve waves of the smaller workgroups fit a compute unit and
    // eight of the larger, short contexts in a large cache lose (300 to 700 tokens, 32 sequences, T=8192 14.0 and 17.3 us, 16
    // of T=32768 10.7 and 14.5).
    if (gqa && head_dim == 64 && rows * plan.n_split <= 256) plan.waves = 8;
    // Records through the L2 (store_through) as long as a whole cache of that length is at most 64 MB.  Splits of different lengths end
    // while others still read, and from about there on the records' writes cost the reads more than their write-back at the end
    // costs the merge.  Through -> plain, us: 41 sequences, 16 on 2 heads, T=23692, D=64 40.9 -> 39.1, 8, 64 on 8, T=40000 82.1 ->
    // 79.8; of 93 shapes of 20 to 110 MB those of 80 and 110 are 0.9 % faster plain, those of 20 to 45 0.8 % slower (24 sequences, 16 on 2
    // heads, T=2525 14.3 -> 14.8).  Of equal lengths, which end together, none was faster plain (one, 64 on 8, T=32768 20.5 -> 20.7 to 21.4).
    plan.records_through = (double)kv_len * batch * kv_heads * (2 * head_dim + 8) <= 64e6;
    // Whole rows, more than one on some compute unit: dealt by their lengths (ranked_row).  Up to three a unit: with more, rows that end
    // early make room for others, and what finding a row takes comes again with each (64 sequences, 32 heads, T=500, lengths spread
    // 27.0 -> 29.3 us).  Of shorter caches two rows differ by less than that.  A unit holds three workgroups of the grouped kernel's
    // four waves (five of 64 codes), four or five of the other kernel's, two of its eight waves and one of two column groups: where a
    // layer does not fit, its rows go to the units that are free first, and that is still better than the grid's order.  Lengths spread / a fourth full and the others
    // an eighth / equal, us: 24 sequences, 32 heads, T=2500 (eight waves) 53.7 -> 50.9 / 40.4 -> 34.2 / 75.9 -> 76.1; 96, 8 heads,
    // T=4000, D=64 59.3 -> 48.5 / 48.1 -> 33.1 / 70.3 -> 70.9; 90, 160 on 8 heads, T=1200 (two groups) 42.1 -> 40.4 / 38.1 -> 34.1 /
    // 55.7 -> 56.5.  What it costs equal lengths is 0.3 us a layer: up to 3 % of 64 codes a token (96, 32 on 8, T=2000 35.9 -> 37.0).
    plan.ranked = plan.n_split == 1 && batch <= kMaxRanked && rows > 256 && rows <= 768 && kv_len >= 1000;
    return plan;
}

DecodePlan decode_plan_of(bool ragged, int batch, int q_heads, int kv_heads, int kv_len, int head_dim) {
    const bool gqa = decode_uses_gqa_kernel(q_heads, kv_heads);
    // (B lengths spread evenly over an eighth to all of the cache)
    const double longest = ragged && batch > 1 ? (batch + 0.125) / (batch + 1) : 1.0;
    const DecodePlan plan = gqa ? decode_gqa_plan(kv_len, (long)batch * kv_heads, q_heads / kv_heads, head_dim)
                                : decode_plan(kv_len, (long)batch * q_heads, head_dim, longest);
    return ragged ? ragged_plan(plan, gqa, batch, q_heads, kv_heads, kv_len, head_dim) : plan;
}

bool decode_uses_gqa_kernel(int q_heads, int kv_heads) {
    const int G = q_heads / kv_heads;
    return G >= 2 && G <= 32;
}

size_t decode_workspace_bytes(int batch, int q_heads, int kv_heads, int kv_len, int head_dim, bool ragged) {
    int n_split = decode_plan_of(ragged, batch, q_heads, kv_heads, kv_len, head_dim).n_split;
    // (grouped heads: never less than two records a row, so that the shapes the static scratch array is too small for stay what they were)
    if (decode_uses_gqa_kernel(q_heads, kv_heads) && n_split < 2) n_split = 2;
    return decode_records_bytes((long)batch * q_heads, n_split, head_dim);
}

// Scratch of the decode entry point that may not allocate: the same (max, sum, accumulator) partials as the
// caller-owned workspace, in one array per GPU that lives as long as the process.  In host code the array's
// name only stands for the symbol: its device address is asked for once per device and kept.
static __device__ __align__(256) unsigned char scratch[kDecodeStaticScratchBytes];

hipError_t decode_static_scratch(float** ptr) {
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static void* per_device[kMaxDevices] = {};
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (per_device[dev] == nullptr) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));   // this device's copy of the array
        if (e != hipSuccess) return e;
        if (p == nullptr) return hipErrorInvalidSymbol;
        per_device[dev] = p;
    }
    *ptr = static_cast<float*>(per_device[dev]);
    return hipSuccess;
}

hipError_t launch_decode(const DecodeArgs& a, hipStream_t stream) {
    // (the query heads of a KV head share one pass over its cache in the grouped-query kernel)
    const bool gqa = decode_uses_gqa_kernel(a.q_heads, a.kv_heads);
    const DecodePlan plan = decode_plan_of(a.ragged, a.batch, a.q_heads, a.kv_heads, a.kv_len, a.head_dim);
    const int n_split = plan.n_split;
    float* const ws_acc = a.workspace;
    float* const ws_ml = a.workspace + (size_t)a.batch * a.q_heads * n_split * a.head_dim;
    auto launch = [&](auto d_c, auto w_c) {
        constexpr int D = decltype(d_c)::value, W = decltype(w_c)::value;
        hipLaunchKernelGGL((slim_decode_int8_split_kernel<D, W>), dim3((unsigned)n_split, (unsigned)a.q_heads, (unsigned)a.batch),
                           dim3(64 * W), 0, stream, (const uint16_t*)a.q, a.k_codes, a.k_scale, a.v_codes, a.v_scale,
                           (uint16_t*)a.out, ws_acc, ws_ml, a.kv_lens, a.q_heads / a.kv_heads, a.kv_heads, a.kv_len, n_split,
                           plan.split_rate, decode_mode(plan, a.batch), a.softmax_scale * kLog2e);
        return hipGetLastError();
    };
    auto pick_w = [&](auto d_c) {
        return plan.waves == 8 ? launch(d_c, std::integral_constant<int, 8>{}) : launch(d_c, std::integral_constant<int, 4>{});
    };
    const hipError_t e = gqa                 ? launch_decode_gqa_split(a, ws_acc, ws_ml, plan, stream)
                         : a.head_dim == 128 ? pick_w(std::integral_constant<int, 128>{})
                                             : pick_w(std::integral_constant<int, 64>{});
    if (e != hipSuccess || n_split == 1) return e;
    return launch_combine(a, ws_acc, ws_ml, n_split, plan.split_rate, stream);
}

}  // namespace slim

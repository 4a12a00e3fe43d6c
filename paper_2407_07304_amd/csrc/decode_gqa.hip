// Decode attention over the INT8 KV cache when several query heads share a KV head (paper
// section 2.2 for the cache; section 2.1 names MHA and GQA side by side).  The cache is
// the bandwidth: every byte of it is read once per KV head here, not once per query head.
//
// With G query heads per KV head the step is a (G x D) by (D x T) product followed by a
// (G x T) by (T x D) one: dense enough for the matrix cores.  A workgroup sweeps a run of
// tokens of one (batch, KV head) for all G heads, its 32-token tiles dealt to the waves in
// turn:
//   - K and V tiles are read with coalesced 128-bit loads (a load instruction of a wave
//     covers whole rows) and written, as the INT8 codes they are, to a wave-private LDS tile
//     each.  No other wave touches them: no barriers, LDS runs a wave's accesses in order.
//   - scores, transposed, S^T = K Q^T with v_mfma_f32_16x16x32_bf16: the K tile as A operand
//     (lane = token, 128-bit LDS reads, widened to bf16 in registers, exact), Q^T as B operand
//     (columns = heads) as the caller gave it.  (Q cut into three INT8 digits for the INT8
//     instruction, K unwidened, took the same time and lost bits of values far below their
//     row's largest: B=16, 64 on 8 heads, T=8192 49.5 us against 49.3, 48 sequences of up to
//     3001 tokens, 32 on 8 heads 41.2 against 41.6.)
//   - a lane then holds one head's column and 4 of every 16 tokens: k_scale multiplies the
//     fp32 score, the running max is lazy (it moves when a score passes it by 2^8), the
//     probability takes the token's v_scale before it is rounded to bf16 and is the B operand
//     of O^T += V^T P^T (the same instruction) as it stands; V^T comes from the row-major
//     INT8 tile through the LDS byte transpose read and is widened to bf16 in registers.
//   - a wave's next tile is in flight while it works on one: its registers are refilled as soon
//     as they are in LDS.  At three waves per SIMD (146 vector registers) that covers the
//     memory latency; a second tile in flight took the third wave and was 5 % slower.
// (Before, K and V were widened to bf16 on their way into LDS and both products ran on
// 32-column tiles, half of them empty for 16 heads: 230 vector registers, 57.7 us for B=16,
// 64 on 8 heads, T=8192.)
// The waves of a workgroup are merged in LDS; where a (batch, KV head) is split over several
// workgroups, the combine kernel of decode.hip merges them in fixed order.
#include <type_traits>

#include "slim_common.h"
#include "slim_kernels.h"

namespace slim {

constexpr int kGqaTile = 32;    // tokens per tile
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) i32x2 lds_i32x2;

// 8 INT8 codes -> 8 bf16, exact
__device__ __forceinline__ bf16x8 widen8(const i32x2 cw) {
    u32x4 r;
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        r[2 * e] = pack_bf16x2(i8_to_f32<0>(cw[e]), i8_to_f32<1>(cw[e]));
        r[2 * e + 1] = pack_bf16x2(i8_to_f32<2>(cw[e]), i8_to_f32<3>(cw[e]));
    }
    return __builtin_bit_cast(bf16x8, r);
}

// D head dimension, W waves per workgroup, NC groups of 16 heads.
// TRAFFIC_ONLY: the measurement form of the kernel (include/slimprobe.h): the same workgroups, waves, token runs and
// loads, issued at the same points, but a tile's registers are only XORed together before they are refilled.  What it
// takes is what the memory system charges for this access pattern on this shape, arithmetic aside.
// The running max is a whole number: the token that sets it has the probability 2^(score - ceil(score)), above a half and 1 only if
// the score itself is whole (later ones have up to 2^8, until the max moves), and times its v_scale that rounds to bf16 like any
// other.  Were the max the score, it would be exactly 1, and a v_scale alone is further off than the mean (0.375 of an ulp, codes of
// N(0,1)); more waves, each with a maximum of its own, have more such tokens.  Distance from the 64-bit result, whole maxima / the
// scores themselves, over 33 shapes, 660 draws of N(0,1): 0.981 on average, 0.960 to 1.000.
template <int D, int W, int NC, bool TRAFFIC_ONLY = false>
__global__ __launch_bounds__(64 * W) void slim_decode_int8_gqa_kernel(
    const uint16_t* __restrict__ q, const int8_t* __restrict__ kc, const float* __restrict__ ks,
    const int8_t* __restrict__ vc, const float* __restrict__ vs, uint16_t* __restrict__ out, float* __restrict__ ws_acc,
    float* __restrict__ ws_ml, const int* __restrict__ kv_lens, int G, int Hkv, int T_alloc, int n_split,
    unsigned split_rate, int mode, float scale_log2e) {
    constexpr int KS = D / 64;            // 16-byte pieces of a K row per lane (two k-steps of the score MFMA each)
    constexpr int DT = D / 16;            // 16-row tiles of O^T
    constexpr int CPR = D / 16;           // 16-byte pieces per row
    constexpr int NP = kGqaTile * CPR / 64;   // 128-bit loads per lane, tile and tensor
    constexpr int PITCH = D + 16;         // LDS row pitch: 16 rows' pieces of a read fall on 16 different groups of four banks
    constexpr int TILE = kGqaTile * PITCH;
    constexpr int WAVE_LDS = 2 * TILE + 256;   // K tile, V tile, the tile's 32 + 32 scales
    constexpr int OPITCH = D + 4;         // floats per head in a wave's merge record (behind its maxima and sums)
    constexpr int MERGE_LDS = 16 * NC * (OPITCH + 2) * 4;
    constexpr int WAVE_BYTES = WAVE_LDS > MERGE_LDS ? WAVE_LDS : MERGE_LDS;

    __shared__ __attribute__((aligned(16))) char smem[W * WAVE_BYTES];

    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));   // (the wave index as a scalar: everything derived from it stays uniform)
    const int l16 = lane & 15, lq = lane >> 4;
    const int Hq = G * Hkv;   // (G query heads per KV head)
    int g = blockIdx.y, b = blockIdx.z, T;
    const int sp = blockIdx.x;
    if (mode > 0) {   // (dealt by length; one split)
        const SequenceHead row = ranked_row(kv_lens, mode, Hkv, T_alloc, b, g);
        g = row.h;
        b = row.b;
        T = row.T;
    } else {
        T = kv_lens ? min(max(kv_lens[b], 1), T_alloc) : T_alloc;
    }
    char* const kS = smem + w * WAVE_BYTES;
    char* const vS = kS + TILE;
    float* const scS = reinterpret_cast<float*>(kS + 2 * TILE);   // [0,32) k_scale * c, [32,64) v_scale

    // T_alloc is the cache's allocated length (the row stride); this sequence's first T tokens count.  The sequence's
    // own tiles are dealt evenly over its splits, and a split's tiles to its waves in turn.
    const int n_used = splits_of(T, n_split, split_rate);
    if (sp >= n_used) return;   // (nobody reads this split's record)
    const long kvrow0 = ((long)b * Hkv + g) * (long)T_alloc;
    const int n_all = (T + kGqaTile - 1) / kGqaTile;
    int first, end;
    split_span(n_all, n_used, sp, first, end);
    first += w;
    const int n_tiles = first < end ? (end - first + W - 1) / W : 0;

    // Q^T B operands: lane holds head l16 of its group of 16 (a column past the last head: the last head again),
    // d = 64 s + 16 lq + 8 e + [0,8)
    bf16x8 qB[NC][KS][2];
#pragma unroll
    for (int nc = 0; nc < NC; ++nc) {
        const uint16_t* qp = q + ((long)b * Hq + (long)g * G + min(16 * nc + l16, G - 1)) * D + 16 * lq;
#pragma unroll
        for (int s = 0; s < KS; ++s)
#pragma unroll
            for (int e = 0; e < 2; ++e) qB[nc][s][e] = *reinterpret_cast<const bf16x8*>(qp + 64 * s + 8 * e);
    }

    // Piece lane + 64 n of a tile (row-major, 16 codes each), through buffer descriptors that cover exactly this
    // (batch, KV head)'s slab: rows past the end of the cache read as zero (and are masked) and a load costs one
    // vector add.  The codes are used once: non-temporal.
    const __amdgpu_buffer_rsrc_t krs = __builtin_amdgcn_make_buffer_rsrc((void*)(kc + kvrow0 * D), 0, (int)((unsigned)T * D), 0x00020000);
    const __amdgpu_buffer_rsrc_t vrs = __builtin_amdgcn_make_buffer_rsrc((void*)(vc + kvrow0 * D), 0, (int)((unsigned)T * D), 0x00020000);
    // (the scales through descriptors as well: lanes 0-31 want the K scale of token lane, lanes 32-63 the V scale; each
    // load asks the other half's lanes for an offset past the end, which reads nothing, so a tile's loads are the
    // same instructions whether the tile is wanted or not)
    const __amdgpu_buffer_rsrc_t ksr = __builtin_amdgcn_make_buffer_rsrc((void*)(ks + kvrow0), 0, (int)((unsigned)T * 4u), 0x00020000);
    const __amdgpu_buffer_rsrc_t vsr = __builtin_amdgcn_make_buffer_rsrc((void*)(vs + kvrow0), 0, (int)((unsigned)T * 4u), 0x00020000);
    const bool k_half = lane < 32;
    const int s_off_k = k_half ? lane * 4 : (int)0x7ffffff0, s_off_v = k_half ? (int)0x7ffffff0 : (lane - 32) * 4;
    u32x4 kbuf[NP], vbuf[NP];
    float sc = 0.0f;
    auto issue = [&](const __amdgpu_buffer_rsrc_t rs, u32x4 (&buf)[NP], int t0) {
#pragma unroll
        for (int n = 0; n < NP; ++n) buf[n] = __builtin_amdgcn_raw_buffer_load_b128(rs, lane * 16 + n * 1024 + t0 * D, 0, 2 /* nt */);
    };
    auto issue_k = [&](int t0) {
        issue(krs, kbuf, t0);
        const uint32_t a = __builtin_amdgcn_raw_buffer_load_b32(ksr, s_off_k + t0 * 4, 0, 0);
        const uint32_t c = __builtin_amdgcn_raw_buffer_load_b32(vsr, s_off_v + t0 * 4, 0, 0);
        sc = __builtin_bit_cast(float, a | c);   // (the lanes a load left out received zero)
    };
    auto issue_v = [&](int t0) { issue(vrs, vbuf, t0); };
    auto stage = [&](const u32x4 (&buf)[NP], char* tile) {   // a tile's codes into LDS
#pragma unroll
        for (int n = 0; n < NP; ++n)
            *reinterpret_cast<u32x4*>(tile + ((lane + 64 * n) / CPR) * PITCH + (lane % CPR) * 16) = buf[n];
    };

    // Every load of the kernel is issued unconditionally: a tile that is not wanted (past the end of this wave's
    // run) is asked for at token T, past the end of the descriptor, so zeros arrive and no memory is read.  The
    // compiler places a wait by counting the loads issued after the one it needs, along the worst path that leads
    // there; loads under a branch are not outstanding on the path that skips them, and at the loop's head the
    // worst path may be the one from the prologue.  So the prologue's four groups keep the order the loop issues
    // them in (K, V of a tile, then the next tile's).
    auto t_of = [&](int i) { return i < n_tiles ? (first + i * W) * kGqaTile : T; };
    __builtin_amdgcn_sched_barrier(0);
    issue_k(t_of(0));
    __builtin_amdgcn_sched_barrier(0);
    issue_v(t_of(0));
    __builtin_amdgcn_sched_barrier(0);

    // K fragments of token tile tt, k-steps 2 s and 2 s + 1: row 16 tt + l16, bytes 64 s + 16 lq + [0,16).  V^T fragment of tile dt: the
    // 16 lanes of a group fetch 8 rows (2 lanes a row, 8 columns each) and lane j of the group receives column j of
    // them; the rows of group lq are the tokens its probabilities belong to: 4 lq + [0,4) and 16 + 4 lq + [0,4).
    const int k_addr = l16 * PITCH + 16 * lq;
    const int v_row = l16 >> 1;
    const int v_addr = (4 * lq + (v_row & 3) + 16 * (v_row >> 2)) * PITCH + 8 * (l16 & 1);

    f32x4 o[NC][DT];
    float M[NC], lsum[NC];   // running max of this lane's head (log2 units), this lane's part of the row sum
#pragma unroll
    for (int nc = 0; nc < NC; ++nc) {
        M[nc] = kMasked;
        lsum[nc] = 0.0f;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) o[nc][dt] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    }

    for (int i = 0; i < n_tiles; ++i) {
        const int t0 = t_of(i);
        const int t_next = t_of(i + 1);
        if constexpr (TRAFFIC_ONLY) {
            u32x4 x = {0u, 0u, 0u, 0u};
#pragma unroll
            for (int n = 0; n < NP; ++n) x ^= kbuf[n] ^ vbuf[n];
            lsum[0] += __uint_as_float((x[0] ^ x[1] ^ x[2] ^ x[3]) & 0x3fffffffu) + sc;
            issue_k(t_next);
            issue_v(t_next);
            // (each tile is consumed and refilled on its own, as in the full kernel: without this the compiler
            // folds the two tiles of a pair into one sum and waits for both at once)
            asm volatile("" : "+v"(lsum[0]));
            __builtin_amdgcn_sched_barrier(0);
            continue;
        }

        stage(kbuf, kS);
        scS[lane] = k_half ? sc * scale_log2e : sc;
        issue_k(t_next);
        i32x4 kw[2][KS];
#pragma unroll
        for (int tt = 0; tt < 2; ++tt)
#pragma unroll
            for (int s = 0; s < KS; ++s) kw[tt][s] = *reinterpret_cast<const i32x4*>(kS + k_addr + 16 * tt * PITCH + 64 * s);
        __builtin_amdgcn_sched_barrier(0);
        stage(vbuf, vS);
        issue_v(t_next);
        __builtin_amdgcn_sched_barrier(0);

        // scores: register r of token tile tt is token 16 tt + 4 lq + r, column = head l16 of the group
        bf16x8 kf[2][KS][2];
#pragma unroll
        for (int tt = 0; tt < 2; ++tt)
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                kf[tt][s][0] = widen8(i32x2{kw[tt][s][0], kw[tt][s][1]});
                kf[tt][s][1] = widen8(i32x2{kw[tt][s][2], kw[tt][s][3]});
            }
        u32x4 pw[NC];
#pragma unroll
        for (int nc = 0; nc < NC; ++nc) {
            f32x4 acc[2] = {{0.0f, 0.0f, 0.0f, 0.0f}, {0.0f, 0.0f, 0.0f, 0.0f}};
#pragma unroll
            for (int s = 0; s < KS; ++s)
#pragma unroll
                for (int e = 0; e < 2; ++e)
#pragma unroll
                    for (int tt = 0; tt < 2; ++tt)
                        acc[tt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[tt][s][e], qB[nc][s][e], acc[tt], 0, 0, 0);
            float u[8];
#pragma unroll
            for (int tt = 0; tt < 2; ++tt) {
                const f32x4 kf4 = *reinterpret_cast<const f32x4*>(&scS[16 * tt + 4 * lq]);
#pragma unroll
                for (int r = 0; r < 4; ++r) u[4 * tt + r] = acc[tt][r] * kf4[r];
            }
            if (t0 + kGqaTile > T) {   // the sequence ends inside this tile (or before it)
#pragma unroll
                for (int r = 0; r < 8; ++r) u[r] = (t0 + 16 * (r / 4) + 4 * lq + r % 4 < T) ? u[r] : kMasked;
            }
            float umax = fmaxf(u[0], u[1]);
#pragma unroll
            for (int r = 2; r < 8; r += 2) umax = fmaxf(umax, fmaxf(u[r], u[r + 1]));
            // the running max moves only when a score has passed it by 2^8 (always on a wave's first tile)
            if (__builtin_amdgcn_ballot_w64(umax - M[nc] > 8.0f) != 0) {
                float m_new = fmaxf(M[nc], umax);
                m_new = fmaxf(m_new, __shfl_xor(m_new, 16));
                m_new = ceilf(fmaxf(m_new, __shfl_xor(m_new, 32)));
                const float alpha = fast_exp2(M[nc] - m_new);
#pragma unroll
                for (int dt = 0; dt < DT; ++dt) o[nc][dt] *= alpha;
                lsum[nc] *= alpha;
                M[nc] = m_new;
            }
            float ps0 = 0.0f, ps1 = 0.0f;
#pragma unroll
            for (int r = 0; r < 8; r += 2) {
                u[r] = fast_exp2(u[r] - M[nc]);
                u[r + 1] = fast_exp2(u[r + 1] - M[nc]);
                ps0 += u[r];
                ps1 += u[r + 1];
            }
            lsum[nc] += ps0 + ps1;
            // the probabilities take their token's v_scale before they are rounded to bf16
#pragma unroll
            for (int tt = 0; tt < 2; ++tt) {
                const f32x4 vf = *reinterpret_cast<const f32x4*>(&scS[32 + 16 * tt + 4 * lq]);
                pw[nc][2 * tt] = pack_bf16x2(u[4 * tt] * vf[0], u[4 * tt + 1] * vf[1]);
                pw[nc][2 * tt + 1] = pack_bf16x2(u[4 * tt + 2] * vf[2], u[4 * tt + 3] * vf[3]);
            }
        }

        // O^T += V^T P^T over the tile's 32 tokens: element j of lane group lq is token 4 lq + j (j < 4) or 16 + 4 lq + j - 4
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) {
            const i32x2 vw = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_i32x2*)(vS + v_addr + 16 * dt));
            const bf16x8 va = widen8(vw);
#pragma unroll
            for (int nc = 0; nc < NC; ++nc)
                o[nc][dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va, __builtin_bit_cast(bf16x8, pw[nc]), o[nc][dt], 0, 0, 0);
        }
    }

    // Merge the waves: register r of tile dt is d = 16 dt + 4 lq + r of head l16.  A wave's record: 16 NC maxima (log2
    // units), as many sums, then the accumulators, a row of OPITCH floats per head (over its own tiles, which are dead).
    float* const rec = reinterpret_cast<float*>(kS);
#pragma unroll
    for (int nc = 0; nc < NC; ++nc) {
        float L = lsum[nc];
        L += __shfl_xor(L, 16);
        L += __shfl_xor(L, 32);
        if (lq == 0) {
            rec[16 * nc + l16] = M[nc];
            rec[16 * NC + 16 * nc + l16] = L;
        }
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
            *reinterpret_cast<f32x4*>(rec + 32 * NC + (16 * nc + l16) * OPITCH + 16 * dt + 4 * lq) = o[nc][dt];
    }
    __syncthreads();
    for (int x = threadIdx.x; x < G * D; x += 64 * W) {
        const int h = x / D, d = x % D;
        float m[W], top = kMasked;
#pragma unroll
        for (int ww = 0; ww < W; ++ww) {
            m[ww] = reinterpret_cast<const float*>(smem + ww * WAVE_BYTES)[h];
            top = ww == 0 ? m[ww] : fmaxf(top, m[ww]);
        }
        float L = 0.0f, acc = 0.0f;
#pragma unroll
        for (int ww = 0; ww < W; ++ww) {
            const float* r = reinterpret_cast<const float*>(smem + ww * WAVE_BYTES);
            const float f = fast_exp2(m[ww] - top);   // a wave without tiles has L = 0 and an accumulator of zeros
            L = fmaf(f, r[16 * NC + h], L);
            acc = fmaf(f, r[32 * NC + h * OPITCH + d], acc);
        }
        const long bh = (long)b * Hq + (long)g * G + h;
        if (!TRAFFIC_ONLY && n_used == 1) {   // (the measurement form has a workspace only)
            out[bh * D + d] = (uint16_t)(pack_bf16x2(acc / L, 0.0f) & 0xffffu);
        } else {
            store_record<D>(ws_acc, ws_ml, bh * n_split + sp, d, acc, top, L, mode < 0);
        }
    }
}

// Splits of the key axis and waves per workgroup, by the model of decode.hip's plan with this kernel's constants (from a sweep
// of 16 row counts, 8 to 1024, by 12 lengths, 128 to 32768, K and V cold): the cache at 6.6 TB/s, or the fullest compute
// unit's tokens at 5.9 ns each (7 where it holds several workgroups; 4.2 and 5 with 64 codes a token), the longer of the two
// and a fifth of the shorter, and 5 us and 40 ns a split for the combine launch.  Where that gives no compute unit a second
// workgroup and whole rows take longer than kDecodeLongNs, the splits are chosen again among those of which that holds, with
// 2.4 us and 25 ns a split (3.6 us and 40 ns of 64 codes a token), and up to three splits may have three tiles.  What splitting whole rows
// costs beyond the sweep as modelled, over 23 shapes of 64 to 128 rows, T=900 to 2200, cut in 2 to 4: 1.2 to 2.8 us by the GPU alone,
// over 8 of 64 codes 2.6 to 3.1.  Steps, us: 16 sequences, 64 on 8 heads, T=2000, one split 21.1, two 20.0; 14, 24 on 8 heads, T=2131
// 23.0 -> 18.8; 10, 64 on 8, T=1409 17.0 -> 14.6; 63, 16 on 2, lengths of up to 3776 29.0 -> 26.6.  (With more splits than
// compute units it does not hold: 34 sequences, 64 on 8 heads, T=1023 23.4 -> 27.9; nor in the place of such a cut: 11, 32 on 8,
// T=5328, D=64 20.3 -> 21.4.)
// Eight waves where the grid leaves compute units without a workgroup (less than 240 of them), four where it fills the chip:
// 128 rows at T=8192 take 45.3 us with 1024 waves in 256 workgroups, 49 with 2048 waves (52.9 in the form before, a split per
// wave; all with the combine launch).  8 rows at T=32768 are 256 workgroups of four waves as well: 16.6 us, with eight waves 17.2.
// With more than 16 heads a KV head (two column groups) always eight waves, a split from three tiles on, and 3 us for the
// combine launch: a compute unit has one or two such workgroups, and four waves are half as many as it wants (32 on 1
// head, T=777, K and V in the caches: 14.6 us with four waves in one split, 10.3 now; 20 on 1, 128 sequences,
// T=3000: 33.5 -> 25.8; a sweep of 8 row counts, 1 to 200, by 8 lengths, 64 to 30000, has no call where four waves win).
DecodePlan decode_gqa_plan(int kv_len, long n_bg, int group, int head_dim) {
    const long n_tiles = ((long)kv_len + kGqaTile - 1) / kGqaTile;
    const bool two_groups = group > 16;
    const double stream_ns = (double)kv_len * n_bg * (2 * head_dim + 8) / 6600.0;
    int best = 1, alone_best = 1;
    double best_ns = 0.0, alone_best_ns = 0.0, whole_ns = 0.0;
    for (int s : {1, 2, 3, 4, 5, 6, 8, 10, 12, 16, 24, 32, 48, 64, 96, 128, 192, 256}) {
        if (s > 1 && (s * (two_groups ? 3 : 4) > n_tiles + 3 || decode_records_bytes(n_bg * group, s, head_dim) > kDecodeStaticScratchBytes)) break;
        const long per_wg = (n_tiles + s - 1) / s, rounds = (n_bg * s + 255) / 256;
        const double ns_token = head_dim == 128 ? (rounds > 1 ? 7.0 : 5.9) : (rounds > 1 ? 5.0 : 4.2);
        const double busy_ns = (double)(rounds * per_wg * kGqaTile) * ns_token;
        const double longer = busy_ns > stream_ns ? busy_ns : stream_ns, shorter = busy_ns > stream_ns ? stream_ns : busy_ns;
        const double sweep_ns = longer + 0.2 * shorter, ns = sweep_ns + (s > 1 ? (two_groups ? 3000.0 : 5000.0) + 40.0 * s : 0.0);
        if (s == 1) whole_ns = ns;
        if (s == 1 || (ns < best_ns && s * (two_groups ? 3 : 4) <= n_tiles)) {
            best_ns = ns;
            best = s;
        }
        const double alone_ns = sweep_ns + (s == 1 ? 0.0 : head_dim == 128 ? 2400.0 + 25.0 * s : 3600.0 + 40.0 * s);
        if (s == 1 || (alone_ns < alone_best_ns && n_bg * s <= 256)) {
            alone_best_ns = alone_ns;
            alone_best = s;
        }
    }
    if (!two_groups && whole_ns > kDecodeLongNs && n_bg * best <= 256) best = alone_best;
    DecodePlan plan{two_groups || n_bg * best < 240 ? 8 : 4, best, kAllSplits};
    // 64 codes a token, several splits: eight waves as long as no compute unit has two workgroups (16 sequences, 64 on 8 heads, T=8192 33.8 -> 26.8 us, one at T=32768 14.8 -> 13.3).
    if (head_dim == 64 && best > 1 && n_bg * best <= 256) plan.waves = 8;
    return plan;
}

hipError_t launch_decode_gqa_split(const DecodeArgs& a, float* ws_acc, float* ws_ml, const DecodePlan& plan, hipStream_t stream,
                                   bool traffic_only) {
    const float scale_log2e = a.softmax_scale * kLog2e;
    const dim3 grid((unsigned)plan.n_split, (unsigned)a.kv_heads, (unsigned)a.batch);
    auto launch = [&](auto d_c, auto w_c, auto nc_c, auto traffic_c) {
        constexpr int D = decltype(d_c)::value, W = decltype(w_c)::value, NC = decltype(nc_c)::value;
        hipLaunchKernelGGL((slim_decode_int8_gqa_kernel<D, W, NC, decltype(traffic_c)::value>), grid, dim3(64 * W), 0, stream,
                           (const uint16_t*)a.q, a.k_codes, a.k_scale, a.v_codes, a.v_scale, (uint16_t*)a.out, ws_acc, ws_ml,
                           a.kv_lens, a.q_heads / a.kv_heads, a.kv_heads, a.kv_len, plan.n_split, plan.split_rate, decode_mode(plan, a.batch), scale_log2e);
        return hipGetLastError();
    };
    auto pick = [&](auto d_c) {
        using std::integral_constant;
        constexpr integral_constant<int, 4> w4{};
        constexpr integral_constant<int, 8> w8{};
        constexpr integral_constant<int, 1> one{};
        constexpr std::false_type no{};
        constexpr std::true_type yes{};
        if (traffic_only) return plan.waves == 8 ? launch(d_c, w8, one, yes) : launch(d_c, w4, one, yes);
        if (a.q_heads / a.kv_heads > 16) return launch(d_c, w8, integral_constant<int, 2>{}, no);
        return plan.waves == 8 ? launch(d_c, w8, one, no) : launch(d_c, w4, one, no);
    };
    return a.head_dim == 128 ? pick(std::integral_constant<int, 128>{}) : pick(std::integral_constant<int, 64>{});
}

}  // namespace slim

// Prefill attention for calls that are too small for prefill.hip's row blocks (paper section 2.1, same result): a
// workgroup owns 32 query rows of one head and its waves split the KEY tiles between them.
//
// What bounds such a call is latency and how few workgroups 128-row blocks make (8 heads, S=512: 32 workgroups that go
// through up to 16 key tiles one after the other).  Here a row block of 32 rows meets its tiles W at a time:
//   - wave w takes tiles w, w + W, ..: K and V come in with coalesced 128-bit loads, one tile ahead, and go to a
//     wave-private LDS tile each (INT8 codes are widened to bf16 on the way); no barriers, LDS runs a wave's accesses
//     in order.
//   - S^T = K Q^T and O^T += V^T P^T with v_mfma_f32_32x32x16_bf16 as in prefill.hip: a lane holds one query column and
//     16 of the tile's 32 keys, V^T comes through the LDS transpose read, the running max is lazy.
//   - the waves' (max, sum, accumulator) are merged once, in LDS, in wave order.
// K and V are read once per 32 rows instead of once per 128, from the L2: that is what limits the form to small calls
// (choose_rows in prefill.hip compares modelled times).
#include <type_traits>

#include "slim_common.h"
#include "slim_kernels.h"

namespace slim {

constexpr int kSplitRows = 32;   // query rows per workgroup
constexpr int kSplitTile = 32;   // keys per tile

struct SplitParams {
    const uint16_t* q;
    const void* k;
    const void* v;
    const float* ks;
    const float* vs;
    void* out;
    int8_t* kq;   // INT8 cache to write next to the attention (bf16 K/V only), or null
    float* kqs;
    int8_t* vq;
    float* vqs;
    int S, causal, n_rb, n_bh, group;
    float scale_log2e;
};

template <int D, bool KV_I8, bool OUT_F32, int W>
__global__ __launch_bounds__(64 * W) void slim_prefill_split_kernel(const SplitParams p) {
    constexpr int KS = D / 16;                  // k-steps of the score MFMA
    constexpr int DT = D / 32;                  // 32-row tiles of O^T
    constexpr int ROWB = KV_I8 ? D : 2 * D;     // bytes per K/V row in memory
    constexpr int CPR = ROWB / 16;              // 16-byte pieces per row
    constexpr int NP = kSplitTile * CPR / 64;   // 128-bit loads per lane, tile and tensor
    constexpr int PITCHK = 2 * D + 16, PITCHV = 2 * D + 64;   // LDS rows: padded so that row reads and transpose reads spread over the banks
    constexpr int TILEK = kSplitTile * PITCHK, TILEV = kSplitTile * PITCHV;
    constexpr int WAVE_LDS = TILEK + TILEV + 256;             // K tile, V tile, the tile's 32 + 32 scales
    constexpr int OPITCH = D + 4;               // floats per query row in a wave's merge record (behind 32 maxima and 32 sums)
    static_assert((64 + kSplitRows * OPITCH) * 4 <= WAVE_LDS, "a merge record fits over the wave's tiles");

    __shared__ __attribute__((aligned(16))) char smem[W * WAVE_LDS];

    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int l32 = lane & 31, hh = lane >> 5;
    // workgroup -> (row block, head): longest row blocks first; heads that share K/V on one XCD (ids are dealt round-robin)
    int rb, bh;
    {
        const int j = (int)blockIdx.x, blk = j / p.n_bh, r = j - blk * p.n_bh, per = p.n_bh >> 3;
        rb = p.n_rb - 1 - blk;
        bh = (p.n_bh & 7) != 0 ? r : (r & 7) * per + (r >> 3);
    }
    const int S = p.S, i0 = rb * kSplitRows;
    const int kvh = bh / p.group;
    const long kvrow0 = (long)kvh * S;
    const int kend = p.causal ? min(S, i0 + kSplitRows) : S;
    const int n_all = (kend + kSplitTile - 1) / kSplitTile;
    const int n_tiles = w < n_all ? (n_all - w + W - 1) / W : 0;
    char* const kS = smem + w * WAVE_LDS;
    char* const vS = kS + TILEK;
    float* const scS = reinterpret_cast<float*>(vS + TILEV);   // [0,32) k_scale * c, [32,64) v_scale

    // Q^T B operands: lane holds row l32, d = 16 s + 8 hh + [0,8)
    bf16x8 qB[KS];
    {
        const uint16_t* qp = p.q + ((long)bh * S + min(i0 + l32, S - 1)) * D + 8 * hh;
#pragma unroll
        for (int s = 0; s < KS; ++s) qB[s] = *reinterpret_cast<const bf16x8*>(qp + 16 * s);
    }
    // descriptors over exactly this head's slab: rows past the end read as zeros (and are masked); every load is issued
    // unconditionally, a tile that is not wanted is asked for past the end and reads nothing
    const __amdgpu_buffer_rsrc_t krs = __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)p.k + kvrow0 * ROWB), 0, (int)((unsigned)S * ROWB), 0x00020000);
    const __amdgpu_buffer_rsrc_t vrs = __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)p.v + kvrow0 * ROWB), 0, (int)((unsigned)S * ROWB), 0x00020000);
    const __amdgpu_buffer_rsrc_t ksr = __builtin_amdgcn_make_buffer_rsrc((void*)(p.ks + kvrow0), 0, KV_I8 ? (int)((unsigned)S * 4u) : 0, 0x00020000);
    const __amdgpu_buffer_rsrc_t vsr = __builtin_amdgcn_make_buffer_rsrc((void*)(p.vs + kvrow0), 0, KV_I8 ? (int)((unsigned)S * 4u) : 0, 0x00020000);
    const int s_off_k = hh == 0 ? l32 * 4 : (int)0x7ffffff0, s_off_v = hh == 1 ? l32 * 4 : (int)0x7ffffff0;
    u32x4 kbuf[NP], vbuf[NP];
    float sc = 0.0f;
    auto issue = [&](const __amdgpu_buffer_rsrc_t rs, u32x4 (&buf)[NP], int t0) {
#pragma unroll
        for (int n = 0; n < NP; ++n) buf[n] = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)((unsigned)t0 * ROWB + (unsigned)(lane * 16 + n * 1024)), 0, 0);
    };
    auto issue_k = [&](int t0) {
        issue(krs, kbuf, t0);
        if constexpr (KV_I8) {
            const uint32_t a = __builtin_amdgcn_raw_buffer_load_b32(ksr, s_off_k + t0 * 4, 0, 0);
            const uint32_t c = __builtin_amdgcn_raw_buffer_load_b32(vsr, s_off_v + t0 * 4, 0, 0);
            sc = __builtin_bit_cast(float, a | c);   // (the lanes a load left out received zero)
        }
    };
    auto stage = [&](const u32x4 (&buf)[NP], char* tile, int pitch) {
#pragma unroll
        for (int n = 0; n < NP; ++n) {
            const int row = (lane + 64 * n) / CPR, col = lane % CPR;
            if constexpr (KV_I8) {   // 16 codes -> 16 bf16, exact
                u32x4 lo, hi;
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    lo[2 * e] = pack_bf16x2(i8_to_f32<0>(buf[n][e]), i8_to_f32<1>(buf[n][e]));
                    lo[2 * e + 1] = pack_bf16x2(i8_to_f32<2>(buf[n][e]), i8_to_f32<3>(buf[n][e]));
                    hi[2 * e] = pack_bf16x2(i8_to_f32<0>(buf[n][2 + e]), i8_to_f32<1>(buf[n][2 + e]));
                    hi[2 * e + 1] = pack_bf16x2(i8_to_f32<2>(buf[n][2 + e]), i8_to_f32<3>(buf[n][2 + e]));
                }
                *reinterpret_cast<u32x4*>(tile + row * pitch + col * 32) = lo;
                *reinterpret_cast<u32x4*>(tile + row * pitch + col * 32 + 16) = hi;
            } else {
                *reinterpret_cast<u32x4*>(tile + row * pitch + col * 16) = buf[n];
            }
        }
    };
    auto t_of = [&](int i) { return i < n_tiles ? (w + i * W) * kSplitTile : S; };
    __builtin_amdgcn_sched_barrier(0);
    issue_k(t_of(0));
    __builtin_amdgcn_sched_barrier(0);
    issue(vrs, vbuf, t_of(0));
    __builtin_amdgcn_sched_barrier(0);

    const int k_addr = l32 * PITCHK + 16 * hh;   // K fragment of k-step s: row l32, bytes 32 s + 16 hh + [0,16)
    int v_addr[DT];                              // V transpose reads: 16 lanes fetch rows k..k+3, lane i receives column i of them
    {
        const int rv = 4 * hh + ((lane & 15) >> 2);
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) v_addr[dt] = rv * PITCHV + (4 * dt + 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1)) * 16 + 8 * (lane & 1);
    }
    f32x16 o[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[dt][r] = 0.0f;
    float M = kMasked, lsum = 0.0f;   // running max of this lane's row (log2 units), this lane's part of the row sum

    for (int i = 0; i < n_tiles; ++i) {
        const int t0 = t_of(i), t_next = t_of(i + 1);
        stage(kbuf, kS, PITCHK);
        if constexpr (KV_I8) scS[lane] = hh == 0 ? sc * p.scale_log2e : sc;
        issue_k(t_next);
        f32x16 acc;
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
#pragma unroll
        for (int s = 0; s < KS; ++s)
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8*>(kS + k_addr + 32 * s), qB[s], acc, 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        stage(vbuf, vS, PITCHV);
        issue(vrs, vbuf, t_next);
        __builtin_amdgcn_sched_barrier(0);

        // softmax: register r of this lane is key t0 + 8 (r/4) + 4 hh + r%4
        float u[16];
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
            f32x4 f = {p.scale_log2e, p.scale_log2e, p.scale_log2e, p.scale_log2e};
            if constexpr (KV_I8) f = *reinterpret_cast<const f32x4*>(&scS[8 * r4 + 4 * hh]);
#pragma unroll
            for (int e = 0; e < 4; ++e) u[4 * r4 + e] = acc[4 * r4 + e] * f[e];
        }
        if (t0 + kSplitTile > (p.causal ? i0 + 1 : S)) {   // the diagonal tile, or the tail of the key axis
            const int rel = (p.causal ? min(i0 + l32, S - 1) : S - 1) - (t0 + 4 * hh);   // keys of this lane up to offset rel are visible
#pragma unroll
            for (int r = 0; r < 16; ++r) u[r] = 8 * (r / 4) + r % 4 <= rel ? u[r] : kMasked;
        }
        float umax = fmaxf(u[0], u[1]);
#pragma unroll
        for (int r = 2; r < 16; r += 2) umax = fmaxf(umax, fmaxf(u[r], u[r + 1]));
        // the running max moves only when a score has passed it by 2^8 (always on a wave's first tile: the diagonal tile
        // shows every row its own key)
        if (__builtin_amdgcn_ballot_w64(umax - M > 8.0f) != 0) {
            float m_new = fmaxf(M, half_max(umax));
            if constexpr (KV_I8) m_new = ceilf(m_new);   // (whole numbers: see WHOLE in prefill.hip; of these maxima a row has four or eight)
            const float alpha = fast_exp2(M - m_new);
#pragma unroll
            for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                for (int r = 0; r < 16; ++r) o[dt][r] *= alpha;
            lsum *= alpha;
            M = m_new;
        }
        float ps0 = 0.0f, ps1 = 0.0f;
#pragma unroll
        for (int r = 0; r < 16; r += 2) {
            u[r] = fast_exp2(u[r] - M);
            u[r + 1] = fast_exp2(u[r + 1] - M);
            ps0 += u[r];
            ps1 += u[r + 1];
        }
        lsum += ps0 + ps1;
        u32x4 pw[2];
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
            // (INT8: the probabilities take their token's v_scale before they are rounded to bf16)
            f32x4 f = {1.0f, 1.0f, 1.0f, 1.0f};
            if constexpr (KV_I8) f = *reinterpret_cast<const f32x4*>(&scS[32 + 8 * r4 + 4 * hh]);
            pw[r4 >> 1][2 * (r4 & 1)] = pack_bf16x2(u[4 * r4] * f[0], u[4 * r4 + 1] * f[1]);
            pw[r4 >> 1][2 * (r4 & 1) + 1] = pack_bf16x2(u[4 * r4 + 2] * f[2], u[4 * r4 + 3] * f[3]);
        }
        // O^T += V^T P^T: k-step u2 covers keys 16 u2 + {4 hh .. 4 hh + 3} and 16 u2 + 8 + {4 hh .. 4 hh + 3} of the tile
#pragma unroll
        for (int u2 = 0; u2 < 2; ++u2)
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) {
                const char* va = vS + v_addr[dt] + 16 * u2 * PITCHV;
                const s16x4 lo = lds_read_tr16(reinterpret_cast<const uint16_t*>(va));
                const s16x4 hi = lds_read_tr16(reinterpret_cast<const uint16_t*>(va + 8 * PITCHV));
                const s16x8 av = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
                o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, av), __builtin_bit_cast(bf16x8, pw[u2]), o[dt], 0, 0, 0);
            }
    }

    // Merge the waves: register r of tile dt is d = 32 dt + 8 (r/4) + 4 hh + r%4 of row l32.  A wave's record lies over its
    // own tiles (dead by now): 32 maxima, 32 sums, then a row of OPITCH floats per query row.
    {
        float* const rec = reinterpret_cast<float*>(kS);
        const float L = half_sum(lsum);
        if (hh == 0) {
            rec[l32] = M;
            rec[32 + l32] = L;
        }
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4) {
                const f32x4 ov = {o[dt][4 * r4], o[dt][4 * r4 + 1], o[dt][4 * r4 + 2], o[dt][4 * r4 + 3]};
                *reinterpret_cast<f32x4*>(rec + 64 + l32 * OPITCH + 32 * dt + 8 * r4 + 4 * hh) = ov;
            }
    }
    __syncthreads();
    constexpr int PPR = D / 8;   // pieces of 8 values per row
#pragma unroll
    for (int pid = (int)threadIdx.x; pid < kSplitRows * PPR; pid += 64 * W) {
        const int row = pid / PPR, d0 = (pid % PPR) * 8;
        float m[W], top = kMasked;
#pragma unroll
        for (int ww = 0; ww < W; ++ww) {
            m[ww] = reinterpret_cast<const float*>(smem + ww * WAVE_LDS)[row];
            top = fmaxf(top, m[ww]);
        }
        float L = 0.0f, a[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) a[e] = 0.0f;
#pragma unroll
        for (int ww = 0; ww < W; ++ww) {
            const float* r = reinterpret_cast<const float*>(smem + ww * WAVE_LDS);
            const float f = fast_exp2(m[ww] - top);   // (a wave without tiles: sum and accumulator are zero)
            L = fmaf(f, r[32 + row], L);
            const f32x4 a0 = *reinterpret_cast<const f32x4*>(r + 64 + row * OPITCH + d0), a1 = *reinterpret_cast<const f32x4*>(r + 64 + row * OPITCH + d0 + 4);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                a[e] = fmaf(f, a0[e], a[e]);
                a[4 + e] = fmaf(f, a1[e], a[4 + e]);
            }
        }
        const float inv = 1.0f / L;
        if (i0 + row < S) {
            const long at = ((long)bh * S + i0 + row) * D + d0;
            if (OUT_F32) {
                f32x4* dst = reinterpret_cast<f32x4*>((float*)p.out + at);
                dst[0] = f32x4{a[0] * inv, a[1] * inv, a[2] * inv, a[3] * inv};
                dst[1] = f32x4{a[4] * inv, a[5] * inv, a[6] * inv, a[7] * inv};
            } else {
                const u32x4 ov = {pack_bf16x2(a[0] * inv, a[1] * inv), pack_bf16x2(a[2] * inv, a[3] * inv),
                                  pack_bf16x2(a[4] * inv, a[5] * inv), pack_bf16x2(a[6] * inv, a[7] * inv)};
                *reinterpret_cast<u32x4*>((uint16_t*)p.out + at) = ov;
            }
        }
    }
    // the INT8 cache of the row block's own K and V rows, if asked for: the head group's workgroups share them
    if constexpr (!KV_I8) {
        if (p.kq != nullptr) {
            constexpr int LPR = D / 8, RPI = 64 / LPR, UNITS = kSplitRows / RPI;   // lanes per row, rows per access, accesses per tensor
            for (int u = bh - kvh * p.group + p.group * w; u < 2 * UNITS; u += p.group * W) {
                const bool is_k = u < UNITS;
                const int row = i0 + RPI * (u % UNITS) + lane / LPR, piece = lane % LPR;
                const u32x4 raw = *reinterpret_cast<const u32x4*>((const uint16_t*)(is_k ? p.k : p.v) + (kvrow0 + min(row, S - 1)) * D + piece * 8);
                u32x2 cw;
                float scale;
                quant_row_piece<LPR>(raw, cw, scale);
                if (row < S) {
                    *reinterpret_cast<u32x2*>((is_k ? p.kq : p.vq) + (kvrow0 + row) * D + piece * 8) = cw;
                    if (piece == 0) (is_k ? p.kqs : p.vqs)[kvrow0 + row] = scale;
                }
            }
        }
    }
}

hipError_t launch_prefill_split(const PrefillArgs& a, int waves, hipStream_t stream) {
    SplitParams p;
    p.q = (const uint16_t*)a.q;
    p.k = a.k;
    p.v = a.v;
    p.ks = a.k_scale;
    p.vs = a.v_scale;
    p.out = a.out;
    p.kq = a.k_codes_out;
    p.kqs = a.k_scale_out;
    p.vq = a.v_codes_out;
    p.vqs = a.v_scale_out;
    p.S = a.seq_len;
    p.causal = a.causal ? 1 : 0;
    p.n_rb = (a.seq_len + kSplitRows - 1) / kSplitRows;
    p.n_bh = a.batch * a.q_heads;
    p.group = a.q_heads / a.kv_heads;
    p.scale_log2e = a.softmax_scale * kLog2e;
    auto launch = [&](auto d_c, auto i8_c, auto f32_c, auto w_c) {
        constexpr int W = decltype(w_c)::value;
        hipLaunchKernelGGL((slim_prefill_split_kernel<decltype(d_c)::value, decltype(i8_c)::value, decltype(f32_c)::value, W>),
                           dim3((unsigned)(p.n_rb * p.n_bh)), dim3(64 * W), 0, stream, p);
        return hipGetLastError();
    };
    using std::integral_constant;
    auto pick_w = [&](auto d_c, auto i8_c, auto f32_c) {
        return waves == 8 ? launch(d_c, i8_c, f32_c, integral_constant<int, 8>{}) : launch(d_c, i8_c, f32_c, integral_constant<int, 4>{});
    };
    auto pick_out = [&](auto d_c, auto i8_c) { return a.out_f32 ? pick_w(d_c, i8_c, std::true_type{}) : pick_w(d_c, i8_c, std::false_type{}); };
    auto pick_kv = [&](auto d_c) { return a.kv_int8 ? pick_out(d_c, std::true_type{}) : pick_out(d_c, std::false_type{}); };
    return a.head_dim == 128 ? pick_kv(integral_constant<int, 128>{}) : pick_kv(integral_constant<int, 64>{});
}

}  // namespace slim

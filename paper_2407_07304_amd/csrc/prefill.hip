// Prefill attention (paper section 2.1): one work item owns a block of query rows and the
// whole softmax direction; K/V stream through it in 32-key tiles while an fp32 running max
// and sum keep the softmax exact.  INT8 K/V (section 2.2) are widened exactly to bf16 while
// being staged; their per-token scales multiply the fp32 score column (K) and the
// probability before it is rounded to bf16 (V), so dequantisation adds no rounding.
//
// There are three forms, by the query rows of a workgroup's row block, and choose_rows says which one a call takes: 128
// rows, 256 rows (WIDE) and, in prefill_split.hip, 32 rows for small calls.
//
// Mapping of the 128- and 256-row forms on gfx950 (wave64, v_mfma_f32_32x32x16_bf16):
//   - A workgroup is 8 waves, two per SIMD, and a wave owns 32 query rows.  256 rows: every wave goes through all key
//     tiles, and nothing is merged.  128 rows: waves w and w+4 own the same rows, the first four waves (group 0) take the
//     even key tiles, the others (group 1) the odd ones, each with its own running max, sum and accumulator, merged once at
//     the end of the row block.
//   - An iteration is one tile of every wave, and a barrier ends it (every second one where six ring slots fit, see DEEP):
//     the wave issues the scores of its next tile and P V of its last one, alternately, and between two MFMAs a share of this
//     tile's softmax (a fused multiply-add, an exponential, an addition, half a conversion), the operand read that replaces
//     the one the MFMA consumed, and a ring request.  A wave's own vector work so runs in the shadow of its MFMAs: a
//     microbenchmark of 16 MFMAs with four vector instructions each takes 34 cycles an MFMA, alone 32.5 (waves that took
//     softmax and MFMAs in turn, two groups in opposite phases, needed 1590 cycles for what an iteration does in 1390: B=1,
//     32 heads, bf16, S=8192 490 us and 465).  On N(0,1) operands what is left is power: S=8192, not causal, takes 1.4 times
//     as long on them as on zeros.
//   - The score tile is computed transposed, S^T = K Q^T: the K tile is the A operand
//     (from LDS), Q^T the B operand (held in registers for the whole row block).  In the
//     result every lane holds ONE query column and 16 of the 32 keys, so the row max and
//     row sum are in-lane reductions plus one exchange between lanes l and l+32.
//   - The same registers, rounded to bf16, are directly the B operand of
//     O^T += V^T P^T; V^T comes from the row-major V tile in LDS through the LDS
//     transpose read (ds_read_b64_tr_b16), so V is never transposed in memory.
//   - O^T accumulators: lane = query column, so the online-softmax rescale is a per-lane
//     scalar multiply; the running max is lazy (it moves only when a row's max grew by more
//     than 2^8), so the rescale runs a few times per row block.
//   - K/V tiles live in an LDS ring of four or six iterations.  bf16 tiles are written by the
//     memory pipe itself (buffer loads with an LDS destination, iterations ahead, the same
//     loads and the same wait in every iteration: past the last tile they ask for zeros) as unpadded
//     rows whose 16-byte chunks are
//     XOR-swizzled by the row, so both the 128-bit K row reads and the V transpose reads are
//     free of bank conflicts; INT8 tiles pass through registers, where they are widened, into
//     padded rows.
//     The k_scales of a tile come from LDS as vectors of four; its v_scales are one register, from which each probability's
//     multiplication takes its own by a DPP broadcast (four 128-bit reads a wave and tile less: B=1, 32 heads, S=8192 566 ->
//     551 us, 64 on 8 heads, S=32768 17.26 -> 16.71 ms).
//   - A wave reads its MFMA operands from LDS half a tile ahead, each fragment right after the MFMA that consumed the
//     register it refills.
//   - A workgroup works off a list of (row block, head) items, one after the other; the lists are
//     dealt so that every workgroup meets about the same number of key tiles, whatever the number
//     of row blocks and heads (pairs of a short and a long block, as before, left up to half of the
//     last round empty: B=1, 32 heads, S=3000 took 96 us and takes 83).  Short blocks go first: the
//     key tiles they read are still in the L2 when a longer one starts over at tile 0.
#include <algorithm>
#include <type_traits>

#include "slim_common.h"
#include "slim_kernels.h"

namespace slim {

constexpr int kBR = 128;   // query rows per row block (4 row groups x 32)
constexpr int kBC = 32;    // keys per tile
constexpr int kPrefillThreads = 512;

struct PrefillParams {
    const uint16_t* q;
    const void* k;
    const void* v;
    const float* ks;
    const float* vs;
    void* out;
    float* row_max;   // the two-sweep variant's row maxima [batch, q_heads, seq_len, 2], else null
    int8_t* kq;    // INT8 cache to write next to the attention (bf16 K/V only), or null
    float* kqs;
    int8_t* vq;
    float* vqs;
    int S, causal;
    int n_rb, n_bh, row_off;     // row blocks per head, heads in all, rows that the first block lies before row 0
    int slots, rounds;           // workgroups per XCD, items a workgroup takes at most
    unsigned heads, last_heads;  // heads of a batch of items, of the last batch
    unsigned group;              // query heads per KV head
    unsigned batch_magic, heads_magic, last_heads_magic, group_magic;   // floor(2^32 / d) of n_rb * heads and of the others
    float scale_log2e;
};

// n / d for uniform n and d with m = floor(2^32 / d) from the host: scalar arithmetic only (a division by a value known
// at run time is some forty vector instructions long, and the first loads of an item wait for it)
__device__ __forceinline__ unsigned div_magic(unsigned n, unsigned d, unsigned m) {
    unsigned q = (unsigned)(((unsigned long long)n * m) >> 32);
    if (n - q * d >= d) ++q;   // (m is low by less than one part, so q is low by at most one)
    return q;
}

// The kernel's own arguments, as a pointer the compiler cannot see through: what is read through it is loaded where it
// is used.  Left to itself the compiler keeps every argument in scalar registers from the start, and those run out (14
// were spilled into the lanes of vector registers; 1 % of B=1, 32 heads, S=2048).
typedef const __attribute__((address_space(4))) PrefillParams* KernelArgs;
__device__ __forceinline__ KernelArgs kernel_args_now() {
    KernelArgs a = (KernelArgs)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(a));
    return a;
}

// lane n of this lane's row of 16, for a constant n: a DPP operand of the instruction that takes it
__device__ __forceinline__ float row_lane(float v, int n) {
    const int b = __builtin_bit_cast(int, v);
    int r = 0;
    switch (n) {
#define SLIM_ROW_LANE(N) case N: r = __builtin_amdgcn_update_dpp(0, b, 0x150 + N, 0xf, 0xf, true); break;
        SLIM_ROW_LANE(0) SLIM_ROW_LANE(1) SLIM_ROW_LANE(2) SLIM_ROW_LANE(3) SLIM_ROW_LANE(4) SLIM_ROW_LANE(5) SLIM_ROW_LANE(6) SLIM_ROW_LANE(7)
        SLIM_ROW_LANE(8) SLIM_ROW_LANE(9) SLIM_ROW_LANE(10) SLIM_ROW_LANE(11) SLIM_ROW_LANE(12) SLIM_ROW_LANE(13) SLIM_ROW_LANE(14) SLIM_ROW_LANE(15)
#undef SLIM_ROW_LANE
    }
    return __builtin_bit_cast(float, r);
}

template <int N>
using int_c = std::integral_constant<int, N>;

// MODE 1 and 2: the paper's own order of operations (section 2.1: the whole score row is there before the softmax
// is applied), for comparison.  A row block's scores do not fit on chip, so K is swept twice, by two launches
// of this kernel: MODE 1 computes the scores and keeps only the row maxima (one per row and wave group, written
// to p.row_max), MODE 2 computes them again, exponentiates against those final maxima and multiplies by V:
// no running maximum, no rescaling of the accumulator, 1.5 times the MFMAs.  MODE 0 is the kernel proper.
//
// WIDE: row blocks of 256 rows.  A staged tile meets twice the query rows (half the widening, or
// half the ring's requests, per MFMA), and there is nothing to merge at the end.  See choose_rows for when it is taken and
// what it gives.
//
// OWN (WIDE, bf16 K/V): for the last key tile of a row and the OWN (1 or 3) after the first the running maximum goes up to a
// whole number above the tile's own, so that the probability of the tile's largest key is a power of two, which rounding to
// bf16 leaves alone.  In blocks of 128 rows two maxima run, in those of 32 four, and a row's largest probability is exact
// under each; under the one of plain 256 rows it is exact once, and their results are 1 to 8 % further from the 64-bit ones
// (N(0,1), causal, D = 64, S=777, fp32 results, 2-norm of the error: 32 rows 1.166e-3, 128 1.217e-3, 256 1.267e-3, with one
// such tile 1.209e-3, with three 1.157e-3).  One such tile costs 0 to 3 % of a call, three 4 to 7 (B=16, 32 on 8 heads, that
// shape: 91, 93 and 96 us; 128 rows 117).
template <int D, bool KV_I8, bool OUT_F32, int MODE = 0, bool WIDE = false, int OWN = 0>
__global__ __launch_bounds__(kPrefillThreads) void slim_prefill_kernel(const PrefillParams p) {
    static_assert(!(MODE != 0 && (KV_I8 || WIDE)), "the two-sweep variant exists for bf16 K/V and 128 rows only");
    static_assert(OWN == 0 || (WIDE && !KV_I8), "see above");
    constexpr int BR = WIDE ? 2 * kBR : kBR;   // query rows per row block
    constexpr int NG = WIDE ? 1 : 2;           // key tiles of an iteration: wave groups that own the same rows
    constexpr bool stats_only = MODE == 1;
    // INT8 K/V in row blocks of 128 rows: the running maxima are whole numbers.  A probability of exactly 1 times its v_scale is the
    // v_scale rounded to bf16, which for codes of N(0,1) is off by more than a product is on average, and two maxima make
    // two of them a row (four or eight in 32): results of 32 and 128 rows are 2.6 to 4.5 % nearer the 64-bit ones for it in bf16,
    // D = 128, and 5 to 8.6 % in fp32 (means over 20 shapes each; D = 64 0.5 to 1 % and 1 to 2 %), in the same time.
    constexpr bool WHOLE = KV_I8 && !WIDE;
    constexpr int KS = D / 16;       // k-steps of the score MFMA
    constexpr int DT = D / 32;       // 32-row tiles of O^T
    constexpr int NS = 2 * KS;       // MFMAs of an iteration: KS of the scores, 2 DT = KS of P V
    constexpr int EPS = 16 / NS;     // probabilities of a lane per MFMA
    constexpr int KP = KS / 2, VP = DT;        // operand fragments read ahead: half a tile's
    constexpr int ROWB = KV_I8 ? D : 2 * D;    // bytes per K/V row in memory
    // LDS tile layouts.  bf16 K/V: unpadded rows (that is how the memory pipe writes them), the 16-byte
    // chunk c of row r at chunk position c ^ swz(r).  K: the 16 rows a 128-bit read touches in one pass
    // land on 16 different bank groups.  V: the 4 rows x 4 chunks a transpose read touches in one pass do.
    // INT8 K/V (written from registers): no swizzle, rows padded by 16 bytes (K) and 64 bytes (V) instead,
    // which keeps every address a base register plus a constant.
    constexpr int ROWL = 2 * D;               // bytes of data per LDS row
    constexpr int ROWLK = KV_I8 ? ROWL + 16 : ROWL, ROWLV = KV_I8 ? ROWL + 64 : ROWL;   // row pitch
    constexpr int TILEBK = kBC * ROWLK, TILEBV = kBC * ROWLV;   // bytes per tile in LDS
    constexpr int SLOTK = NG * TILEBK, SLOTV = NG * TILEBV;     // bytes per ring slot (an iteration's tiles)
    // A barrier every second iteration where six slots a tensor fit (256 rows) and the registers allow it (not INT8, D = 128:
    // 56 bytes of spills a lane, S=8192 548 -> 559 us): B=1, 32 heads, bf16, S=4096 128.1 -> 126.5 us, S=8192 466 -> 460; B=4, 32
    // on 8 heads, S=777 31.3 -> 30.4; D=64, S=4096 82.0 -> 80.2, INT8 99.1 -> 97.9.
    constexpr bool DEEP = WIDE && !(KV_I8 && D == 128);
    constexpr int RING = DEEP ? 6 : 4;        // ring depth, in iterations
    constexpr int BARRIERS = DEEP ? 2 : 1;    // iterations per barrier
    constexpr int LEADK = DEEP ? 5 : 4, LEADV = DEEP ? 3 : 2, LEADS = DEEP ? 4 : 3;   // iterations ahead that K, V and INT8 scales go to the ring
    auto ring_slot = [](int x) { return x % RING; };
    constexpr int CPL = ROWL / 16;            // 16-byte chunks per LDS row: 16 or 8
    constexpr int RPL = 256 / ROWL;           // rows per 256-byte line of banks: 1 or 2
    constexpr int K_BYTES = RING * SLOTK, V_BYTES = RING * SLOTV;
    constexpr int NV = DT / 2 * 4 + 1;        // f32x4 vectors a wave hands to its partner at the merge
    constexpr int OH = WIDE && OUT_F32 && D == 128 ? 2 : 1;   // parts that the output goes out in: 256 rows of 512 bytes do not fit beside Q
    constexpr int OPITCH = (OUT_F32 ? 4 * D : 2 * D) / OH + 16;   // output tile row pitch: spreads the column-wise writes over the banks
    constexpr int OUT_BYTES = BR * OPITCH, MERGE_BYTES = WIDE || 8 * NV * 64 * 16 < OUT_BYTES ? OUT_BYTES : 8 * NV * 64 * 16;
    // (the merge buffer and the output tile take the place of the ring, which is quiet by then)
    constexpr int RING_BYTES = K_BYTES + V_BYTES > MERGE_BYTES ? K_BYTES + V_BYTES : MERGE_BYTES;
    auto swz_k = [](int r) { return KV_I8 ? 0 : (r / RPL) & (CPL - 1); };
    auto swz_v = [](int r) { return KV_I8 ? 0 : ((r / RPL) & (CPL / 4 - 1)) << 2; };

    // The row block's Q: BR unpadded rows, the 16-byte chunk c of row r at chunk position c ^ qswz(r) (the bf16 K tile's layout)
    constexpr int ROWQ = 2 * D;                // bytes per Q row, in memory and in LDS
    constexpr int CPQ = ROWQ / 16;             // 16-byte chunks per row: 16 or 8
    constexpr int RPQ = 64 / CPQ;              // rows per wave-wide load: 4 or 8
    constexpr int NQ = BR / 8 / RPQ;           // loads per wave and row block (a wave brings in an eighth of the rows)
    constexpr int SC_BYTES = KV_I8 ? RING * NG * 2 * kBC * 4 : 0;   // INT8: per slot the k_scales * c, then the v_scales
    constexpr int Q_OFF = RING_BYTES + SC_BYTES;
    auto qswz = [](int r) { return (r / (256 / ROWQ)) & (CPQ - 1); };

    constexpr bool Q_LDS = !KV_I8;             // (the INT8 kernel keeps plain loads into the registers: measured faster there)
    __shared__ __attribute__((aligned(16))) char smem[Q_OFF + (Q_LDS ? BR * ROWQ : 0)];

    // Work items are (row block, batch*head).  They are listed in batches of `heads` heads (few enough that what an XCD
    // works on at a time keeps its K/V in the L2), longest row block first within a batch; item j goes to XCD j % 8
    // (workgroup ids are dealt round-robin over the XCDs), where `slots` workgroups deal the XCD's items out among
    // themselves back and forth (0, 1, .., slots - 1, slots - 1, .., 0, 0, ..), which gives all of them about the same
    // number of key tiles.  Where a batch is a multiple of 8 heads an XCD gets whole heads, consecutive ones: those share
    // K/V.  A workgroup works its list off from the end: what a short block read is still in the L2 when a longer one
    // starts over at tile 0.
    int k = p.rounds - 1, rb, bh;
    const int xcd = (int)__builtin_amdgcn_workgroup_id_x() & 7, slot = (int)__builtin_amdgcn_workgroup_id_x() >> 3;   // (the builtin, not a library call: stays a scalar)
    const int n_items = (p.n_rb * p.n_bh - xcd + 7) >> 3;
    auto index_of = [&](int round, int slots) { return round * slots + ((round & 1) ? slots - 1 - slot : slot); };
    auto item_at = [&](int round, int& rb_i, int& bh_i) {
        const KernelArgs a = kernel_args_now();
        const unsigned j = (unsigned)(index_of(round, a->slots) * 8 + xcd), per_batch = (unsigned)a->n_rb * a->heads;
        const unsigned batch = div_magic(j, per_batch, a->batch_magic), head0 = batch * a->heads, jj = j - batch * per_batch;
        const bool last = head0 + a->heads > (unsigned)a->n_bh;
        const unsigned heads = last ? a->last_heads : a->heads;
        const unsigned blk = div_magic(jj, heads, last ? a->last_heads_magic : a->heads_magic), r = jj - blk * heads;
        rb_i = a->n_rb - 1 - (int)blk;
        // (in odd rounds the heads run backwards where that keeps a workgroup on one head: full batches, aligned rounds)
        const unsigned per = heads >> 3, in = r >> 3;
        const bool back = (round & 1) != 0 && !last && ((unsigned)a->slots & (per - 1)) == 0 && (per & (per - 1)) == 0;
        bh_i = (int)(head0 + ((heads & 7) != 0 ? r : (r & 7) * per + (back ? per - 1 - in : in)));
    };
    if (index_of(k, p.slots) >= n_items) --k;
    if (k < 0) return;
    item_at(k, rb, bh);
    const int S = p.S;
    const float c = p.scale_log2e;

    // wave index as a scalar: everything derived from it (group, row group, last tile) stays uniform
    const int tid = (int)__builtin_amdgcn_workitem_id_x(), w8 = __builtin_amdgcn_readfirstlane(tid >> 6), grp = w8 >> 2, w = w8 & 3;
    const int rg = WIDE ? w8 : w;   // this wave's 32 rows of the block
    const int l = tid & 63, l32 = l & 31, hh = l >> 5;

    // Q^T B-operands of a row block: lane holds row my_q, d = 16 s + 8 hh + [0,8).  With bf16 K/V the rows come
    // in through LDS, by buffer loads with an LDS destination that move 64 consecutive 16-byte pieces each: loads
    // that give every lane a row of its own are taken lane by lane by the memory pipe (about 4 k cycles per row block
    // for the eight waves' fragments, with the first K and V tiles waiting behind them, against about 0.7 k this
    // way); rows outside the sequence arrive as zeros.  The INT8 kernel loads its fragments straight into
    // the registers.  The first row block's are requested here, ahead of the address tables below: they come from
    // cold memory.
    bf16x8 qreg[KS];
    const unsigned smem_base = (unsigned)(size_t)(__attribute__((address_space(3))) char*)smem;
    auto request_q = [&](int rb_q, int bh_q) {
        if constexpr (!Q_LDS) {
            const int q_row = min(max(rb_q * BR - p.row_off + 32 * rg + l32, 0), S - 1);
            const uint16_t* qp = p.q + ((long)bh_q * S + q_row) * (long)D + 8 * hh;
#pragma unroll
            for (int s = 0; s < KS; ++s) qreg[s] = *reinterpret_cast<const bf16x8*>(qp + 16 * s);
            return;
        }
        u32x4 qrs_raw;
        const unsigned long long a64 = (unsigned long long)(p.q + (long)bh_q * S * D);
        qrs_raw[0] = __builtin_amdgcn_readfirstlane((unsigned)a64);
        qrs_raw[1] = __builtin_amdgcn_readfirstlane((unsigned)(a64 >> 32) & 0xffffu);
        qrs_raw[2] = __builtin_amdgcn_readfirstlane((unsigned)S * ROWQ);
        qrs_raw[3] = 0x00020000u;
#pragma unroll
        for (int j = 0; j < NQ; ++j) {
            const int r = BR / 8 * w8 + RPQ * j + l / CPQ, pos = l % CPQ;   // row of the block, chunk position in LDS
            const unsigned voff = (unsigned)(rb_q * BR - p.row_off + r) * ROWQ + (unsigned)((pos ^ qswz(r)) * 16);
            const unsigned dst = __builtin_amdgcn_readfirstlane(smem_base + (unsigned)(Q_OFF + (BR / 8 * w8 + RPQ * j) * ROWQ));
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                         :
                         : "s"(dst), "v"(voff), "s"(qrs_raw)
                         : "memory", "m0");
        }
    };
    // this wave's fragments of the Q in LDS (once the requests have landed and a barrier has passed)
    auto read_q = [&]() {
        if constexpr (!Q_LDS) return;
#pragma unroll
        for (int s = 0; s < KS; ++s)
            qreg[s] = *reinterpret_cast<const bf16x8*>(smem + Q_OFF + (32 * rg + l32) * ROWQ + (((2 * s + hh) ^ qswz(l32)) * 16));
    };
    request_q(rb, bh);
    __builtin_amdgcn_sched_barrier(0);

    // ---- staging.  The buffer descriptors cover exactly this head's K (V) slab: pieces past the end of
    // the sequence read as zero (those keys are masked in the softmax).  An iteration's tiles are staged by all waves.
    // bf16: one buffer load with an LDS destination moves 64 consecutive 16-byte chunk positions (RPW whole
    // rows); lane i fills position i, so it asks for the chunk the swizzle puts there.  The load is
    // written as inline assembly on purpose: the compiler then keeps no book on it, and neither its
    // barriers nor its LDS reads wait for requests that are meant to stay in flight over an iteration.
    // Completion is tracked by hand (vmcnt) where a tile becomes readable.
    constexpr int RPW = 64 / CPL;              // rows per wave-wide load: 4 or 8
    constexpr int NLT = NG * kBC / RPW;        // loads per iteration and tensor: 4, 8 or 16
    constexpr int NLD = NLT >= 8 ? NLT / 8 : 1;   // of which a wave issues (four: the first waves K's, the others V's)
    auto raw_rsrc = [&](const char* base) {    // the same descriptor as four plain dwords
        const unsigned long long a64 = (unsigned long long)base;
        u32x4 d;
        d[0] = __builtin_amdgcn_readfirstlane((unsigned)a64);
        d[1] = __builtin_amdgcn_readfirstlane((unsigned)(a64 >> 32) & 0xffffu);
        d[2] = __builtin_amdgcn_readfirstlane((unsigned)S * ROWB);
        d[3] = 0x00020000u;
        return d;
    };
    unsigned d_koff, d_voff;
    const int d_idx = NLT >= 8 ? w8 : w;       // this wave's load of the tile (and every eighth after it)
    {
        const int r = RPW * d_idx + l / CPL, pos = l % CPL;
        d_koff = (unsigned)r * ROWB + (unsigned)((pos ^ swz_k(r)) * 16);
        d_voff = (unsigned)r * ROWB + (unsigned)((pos ^ swz_v(r)) * 16);
    }
    auto dma_fire = [&](const u32x4 rs, unsigned dst, unsigned voff) {
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                     :
                     : "s"(dst), "v"(voff), "s"(rs)
                     : "memory", "m0");
    };
    // load n of this wave's share of iteration tile T, to the slot at lds_off (a tile that is not wanted is requested past
    // the end of the slab: zeros arrive, no memory is read)
    auto dma_one = [&](const u32x4 rs, unsigned off, int n, int T, int lds_off, bool wanted) {
        const unsigned tbase = wanted ? (unsigned)T * (NG * kBC * ROWB) + (unsigned)n * (8 * RPW * ROWB) : (unsigned)S * ROWB;
        dma_fire(rs, __builtin_amdgcn_readfirstlane(smem_base + (unsigned)(lds_off + (d_idx + 8 * n) * 1024)), tbase + off);
    };

    // INT8: 16 codes go through registers and leave as two bf16 chunks.  A tensor's pieces are 64-piece units; a thread
    // takes one of K and one of V (TWO), or the first waves take K's and the next ones V's.
    constexpr int CPR = ROWB / 16;            // 16-byte pieces per row in memory
    constexpr int UPT = NG * kBC * CPR / 64;  // units per tensor and iteration: 8, 4 or 2
    constexpr bool TWO = UPT >= 8;
    const bool st_k = TWO || w8 < UPT;        // this wave's (first) unit is K's
    const bool has_p = 2 * UPT >= 8 || w8 < 2 * UPT;
    const int pid = (TWO ? w8 : w8 % UPT) * 64 + l, prow = pid / CPR, pcol = pid % CPR;
    const unsigned p_off = (unsigned)prow * ROWB + (unsigned)pcol * 16u;
    const int p_kdst = prow * ROWLK + 32 * pcol, p_vdst = K_BYTES + prow * ROWLV + 32 * pcol;
    const int p_dst = st_k ? p_kdst : p_vdst;
    // The iteration's scales: the last wave carries the k_scales, the one before it the v_scales (every choice here is
    // uniform over the wave).
    const bool has_s = KV_I8 && w8 >= 6;
    const bool s_is_k = w8 == 7;
    const int s_lane = l & (NG * kBC - 1);
    __amdgpu_buffer_rsrc_t srs;
    auto widen_dword = [&](unsigned cw, unsigned& lo, unsigned& hi) {   // 4 codes -> 4 bf16, exact
        lo = pack_bf16x2(i8_to_f32<0>(cw), i8_to_f32<1>(cw));
        hi = pack_bf16x2(i8_to_f32<2>(cw), i8_to_f32<3>(cw));
    };
    auto store_piece = [&](int at, const u32x4 cw) {
        u32x4 a, b;
        unsigned x, y;
        widen_dword(cw[0], x, y); a[0] = x; a[1] = y;
        widen_dword(cw[1], x, y); a[2] = x; a[3] = y;
        widen_dword(cw[2], x, y); b[0] = x; b[1] = y;
        widen_dword(cw[3], x, y); b[2] = x; b[3] = y;
        *reinterpret_cast<u32x4*>(smem + at) = a;
        *reinterpret_cast<u32x4*>(smem + at + 16) = b;
    };
    float* const scS = reinterpret_cast<float*>(smem + RING_BYTES);
    auto store_s = [&](int slot, float s) {
        if (has_s) scS[slot * (NG * 2 * kBC) + (s_is_k ? 0 : NG * kBC) + s_lane] = s_is_k ? s * c : s;
    };
    auto load_s = [&](int T) {   // (a key past the end of the sequence gets scale 0: it is masked anyway)
        return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(srs, (T * (NG * kBC) + s_lane) * 4, 0, 0));
    };

    f32x16 o[DT];
    // LDS read addresses (bytes).  K fragment of k-step s: row l32, chunk 2 s + hh.  V transpose read: the
    // 16 lanes of a group fetch rows k..k+3 (4 lanes per row, 8 bytes each) and lane i of the group
    // receives column i of those 4 rows; per 32-column tile dt the lane reads chunk 4 dt + 2 b4 + (l&3)/2.
    const int my_tile = NG == 2 ? grp : 0;   // which of an iteration's tiles is this wave's
    int k_addr[KS], v_addr[DT];
#pragma unroll
    for (int s2 = 0; s2 < KS; ++s2) k_addr[s2] = my_tile * TILEBK + l32 * ROWLK + (((2 * s2 + hh) ^ swz_k(l32)) * 16);
    {
        const int rv = 4 * hh + ((l & 15) >> 2);
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
            v_addr[dt] = K_BYTES + my_tile * TILEBV + rv * ROWLV + (((4 * dt + 2 * ((l >> 4) & 1) + ((l & 3) >> 1)) ^ swz_v(rv)) * 16) + 8 * (l & 1);
    }
    const int sc_addr = RING_BYTES + (my_tile * kBC + 4 * hh) * 4;   // this lane's k_scales: + 32 bytes per 8 keys
    const int scv_addr = sc_addr + (NG * kBC + 8 * ((l & 15) >> 2) + (l & 3)) * 4;

    for (;;) {   // the workgroup's items
        const int kvh = (int)div_magic((unsigned)bh, p.group, p.group_magic);   // (batch, KV head): heads per batch are a multiple of the group
        const long kvrow0 = (long)kvh * (long)S;
        // the buffer descriptors cover exactly this head's K (V) slab
        const char* const kslab = (const char*)p.k + kvrow0 * ROWB;
        const char* const vslab = (const char*)p.v + kvrow0 * ROWB;
        const u32x4 krs_raw = raw_rsrc(kslab), vrs_raw = raw_rsrc(vslab);
        const __amdgpu_buffer_rsrc_t krs = __builtin_amdgcn_make_buffer_rsrc((void*)(st_k ? kslab : vslab), 0, (int)((unsigned)S * ROWB), 0x00020000);   // (the first piece's tensor)
        const __amdgpu_buffer_rsrc_t vrs = __builtin_amdgcn_make_buffer_rsrc((void*)vslab, 0, (int)((unsigned)S * ROWB), 0x00020000);
        {
            const float* const sbase = KV_I8 ? ((s_is_k ? p.ks : p.vs) + kvrow0) : nullptr;
            srs = __builtin_amdgcn_make_buffer_rsrc((void*)sbase, 0, KV_I8 && has_s ? (int)((unsigned)S * 4u) : 0, 0x00020000);
        }
        const int i0 = rb * BR - p.row_off;              // (negative in a first block that starts before row 0)
        const int my_q = i0 + 32 * rg + l32;             // this lane's query row (may lie outside [0, S))
        const int wave_q_lo = i0 + 32 * rg;
        const int kend = p.causal ? min(S, i0 + BR) : S;
        const int n_tiles = (kend + kBC - 1) / kBC;
        const int n_iter = (n_tiles + NG - 1) / NG;
        // last tile of this row group: its diagonal under the causal mask, else the tail of the key axis; -1 if the row
        // group lies outside the sequence
        // (row_off is a multiple of 32: all of a row group's rows lie before row 0 or none does)
        const int t_last = wave_q_lo >= S || wave_q_lo < 0 ? -1 : (p.causal ? min(n_tiles - 1, wave_q_lo / kBC) : n_tiles - 1);
        const int last = t_last < my_tile ? -1 : (t_last - my_tile) / NG;   // the iteration of this wave's last tile, or -1
        const int lim = p.causal ? min(my_q, S - 1) : S - 1;   // last key this lane's row may see

        // (the first item's Q was requested at the top of the kernel, the next one's is before this one's merge)
        float M = kMasked, lsum = 0.0f;   // running max in scaled (log2) units; per-lane partial row sum
        if constexpr (MODE == 2) {   // the final maximum of this lane's row over this group's tiles
            M = p.row_max[(((long)bh * S + min(max(my_q, 0), S - 1)) * 2) + grp];
        }

        // ---- the ring.  Iteration i reads K tile i+1 (its second half) and i+2 (first half), V tile i-1 (second half)
        // and i (first half).  It requests K tile i+LEADK, in the slot of K tile i+LEADK-RING, and V tile i+LEADV, in that of
        // V tile i+LEADV-RING; both are waited for at the end of iteration i+1.  Four slots: a barrier ends every iteration; the
        // slots were last read in iteration i-1, and the tiles are read from iteration i+2 on.  Six: a barrier ends the odd
        // iterations; the slots were last read in iteration i-2, and the tiles are read from
        // iteration i+3 on, so there is a barrier between in both directions whatever i's parity.
        // INT8 tiles are stored from registers at those points instead, and what is stored next is loaded.
        // "V tile -1" meets the zero probabilities of iteration 0: its slot is filled with zeros.
        u32x4 sg0, sg1;
        float sgs = 0.0f;
        __syncthreads();   // the previous item has finished with the ring and the merge buffer that lies over it
        if constexpr (!KV_I8) {
            const bool does_k = NLT >= 8 || w8 < 4, does_v = !stats_only && (NLT >= 8 || w8 >= 4);
            auto k_tile = [&](int T) {
                if (does_k)
#pragma unroll
                    for (int n = 0; n < NLD; ++n) dma_one(krs_raw, d_koff, n, T, T * SLOTK, T < n_iter);
            };
            auto v_tile = [&](int T, bool wanted) {
                if (does_v)
#pragma unroll
                    for (int n = 0; n < NLD; ++n) dma_one(vrs_raw, d_voff, n, T, K_BYTES + T * SLOTV, wanted);
            };
#pragma unroll
            for (int T = 0; T < LEADK; ++T) k_tile(T);
#pragma unroll
            for (int T = 0; T < LEADV; ++T) v_tile(T, T < n_iter);
            v_tile(RING - 1, false);
            __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0): this wave's requests have landed in LDS
        } else {
            u32x4 ta[LEADK], tb[LEADV + 1];
            float sc[LEADS];
            // The addresses of these loads are put together here, from copies the compiler cannot see through: left
            // to itself it computes all of them ahead of the item loop, spills them, and reloads them one by one
            // between the loads, and a reload is a memory access that waits, in order, for the tile loads before it
            // (eight trips to cold memory one after the other instead of one).
            unsigned off_now = p_off;
            asm volatile("" : "+v"(off_now));
            constexpr unsigned TB = NG * kBC * ROWB;
            const unsigned beyond = (unsigned)S * ROWB;
            static_assert(LEADK == LEADV + 2, "V: its tiles, then the zeros, then nothing new");
            // (a wave that stages V only: its tiles, the zeros of V tile -1 in the ring's last slot, and its first tile again)
            auto slot_n = [&](int n) { return st_k || n < LEADV ? n : n == LEADV ? RING - 1 : 0; };
#pragma unroll
            for (int n = 0; n < LEADK; ++n)
                ta[n] = __builtin_amdgcn_raw_buffer_load_b128(krs, (int)((n == LEADV && !st_k ? beyond : n > LEADV && !st_k ? 0u : n * TB) + off_now), 0, 0);
            if constexpr (TWO)
#pragma unroll
                for (int n = 0; n <= LEADV; ++n)
                    tb[n] = __builtin_amdgcn_raw_buffer_load_b128(vrs, (int)((n == LEADV ? beyond : n * TB) + off_now), 0, 0);
#pragma unroll
            for (int n = 0; n < LEADS; ++n) sc[n] = load_s(n);
            sg0 = __builtin_amdgcn_raw_buffer_load_b128(krs, (int)((st_k ? LEADK * TB : LEADV * TB) + off_now), 0, 0);
            if constexpr (TWO) sg1 = __builtin_amdgcn_raw_buffer_load_b128(vrs, (int)(LEADV * TB + off_now), 0, 0);
            sgs = load_s(LEADS);
            if (has_p)
#pragma unroll
                for (int n = 0; n < LEADK; ++n) store_piece(p_dst + slot_n(n) * (st_k ? SLOTK : SLOTV), ta[n]);
            if constexpr (TWO)
#pragma unroll
                for (int n = 0; n <= LEADV; ++n) store_piece(p_vdst + (n == LEADV ? RING - 1 : n) * SLOTV, tb[n]);
#pragma unroll
            for (int n = 0; n < LEADS; ++n) store_s(n, sc[n]);
        }
        __syncthreads();
        read_q();
        // (the accumulators start here, not above: 64 registers the prologue's loads in flight can use)
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int r = 0; r < 16; ++r) o[dt][r] = 0.0f;

        // Operand fragments, read from LDS half a tile ahead:
        //   kfr: K tile as A operand, lane = key l32, d = 16 s + 8 hh + [0,8)
        //   vfr: V^T tile as A operand for keys 16u..16u+15, d = 32 dt + l32, fragment x = u DT + dt.  Transpose read: the 16
        //   lanes of a group fetch rows k..k+3 (4 lanes per row, 4 columns each) and lane i receives column i of those rows.
        bf16x8 kfr[KP];
        s16x4 vfr[VP][2];
        auto fetch_k = [&](int s, int slot_off) {   // slot_off: byte offset of the K ring slot
            kfr[s % KP] = *reinterpret_cast<const bf16x8*>(smem + k_addr[s] + slot_off);
        };
        auto fetch_v = [&](int x, int slot_off) {   // slot_off: byte offset of the V ring slot
            const char* va = smem + v_addr[x % DT] + slot_off + 16 * (x / DT) * ROWLV;
            vfr[x % VP][0] = lds_read_tr16(reinterpret_cast<const uint16_t*>(va));
            vfr[x % VP][1] = lds_read_tr16(reinterpret_cast<const uint16_t*>(va + 8 * ROWLV));
        };
        // One score MFMA, S^T[key][query] += sum over d in [16 s, 16 s + 16) of K[key][d] Q[query][d], and one
        // P V MFMA, O^T[d][query] += sum_key V[key][d] P[query][key] for d in [32 dt, 32 dt + 32); k-step u of
        // the latter covers registers 8u..8u+7 of the probabilities, i.e. keys 16u + {4hh..4hh+3} and
        // 16u + 8 + {4hh..4hh+3} of the tile.
        auto pv_mfma = [&](int x, const u32x4 (&pw)[2]) {
            const s16x4 lo = vfr[x % VP][0], hi = vfr[x % VP][1];
            const s16x8 av = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
            o[x % DT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, av), __builtin_bit_cast(bf16x8, pw[x / DT]), o[x % DT], 0, 0, 0);
        };
        // The probabilities of a lane, in a, to pn (INT8: times their token's v_scale, before they are rounded to bf16).
        auto pack_p = [&](int sc_off, float (&a)[16], u32x4 (&pn)[2]) {
            if constexpr (KV_I8) {
#pragma unroll
                for (int r4 = 0; r4 < 4; ++r4) {
                    const f32x4 vf = *reinterpret_cast<const f32x4*>(smem + sc_addr + sc_off + NG * kBC * 4 + 32 * r4);
#pragma unroll
                    for (int e = 0; e < 4; ++e) a[4 * r4 + e] *= vf[e];
                }
            }
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int i = 0; i < 4; ++i) pn[u][i] = pack_bf16x2(a[8 * u + 2 * i], a[8 * u + 2 * i + 1]);
        };
        // OWN: the least running max not below M that lies a whole number above a tile's (that has no finite score: M)
        auto own_max = [&](float m_tile) { return fmaxf(M, m_tile + ceilf(fminf(fmaxf(M - m_tile, 0.0f), 1e30f))); };
        // The softmax of tile t with the maximum taken exactly (scores in st, register r of this lane is key 32 t + 8 (r/4)
        // + 4 hh + r%4; sc_off: the tile's scales): moves the running max, rescales what there is, leaves the probabilities
        // in pn.  Keys of this lane past offset rel are masked.  (No contraction: a product that is masked cannot be one, and a
        // tile's result must not depend on whether the compiler knows that none is.)  own: the new max is own_max.
        auto exact_softmax = [&](int sc_off, int rel, bool first, bool own, const f32x16& st, u32x4 (&pn)[2]) {
#pragma clang fp contract(off)
            float a[16];
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4) {
                f32x4 kf = {c, c, c, c};
                if constexpr (KV_I8) kf = *reinterpret_cast<const f32x4*>(smem + sc_addr + sc_off + 32 * r4);
#pragma unroll
                for (int e = 0; e < 4; ++e) a[4 * r4 + e] = 8 * r4 + e <= rel ? st[4 * r4 + e] * kf[e] : kMasked;
            }
            float umax = fmaxf(a[0], a[1]);
#pragma unroll
            for (int r = 2; r < 16; r += 2) umax = fmaxf(umax, fmaxf(a[r], a[r + 1]));
            float m_new = own ? own_max(half_max(umax)) : fmaxf(M, half_max(umax));
            if constexpr (WHOLE) m_new = ceilf(m_new);
            const float alpha = fast_exp2(M - m_new);
            // (the accumulator is still zero on a wave's first tile, and on the diagonal tile the maximum has
            // usually been met already: the 16 DT multiplications are skipped when they would change nothing)
            if (!first && __builtin_amdgcn_ballot_w64(m_new > M) != 0) {
#pragma unroll
                for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                    for (int r = 0; r < 16; ++r) o[dt][r] *= alpha;
            }
            lsum *= alpha;
            M = m_new;
            float ps0 = 0.0f, ps1 = 0.0f;
#pragma unroll
            for (int r = 0; r < 16; r += 2) {
                a[r] = fast_exp2(a[r] - m_new);
                a[r + 1] = fast_exp2(a[r + 1] - m_new);
                ps0 += a[r];
                ps1 += a[r + 1];
            }
            pack_p(sc_off, a, pn);
            return ps0 + ps1;
        };
        // The same for a wave's last tile.  Where that is not its rows' last one (128 rows: the group that does not hold the
        // diagonal) nothing is masked, and like every other such tile it leaves the running max where it is unless the
        // probabilities overflow: the maximum that they are rounded against does not depend on which group a tile fell to.
        auto last_softmax = [&](int sc_off, int rel, bool masked, bool first, const f32x16& st, u32x4 (&pn)[2]) {
            if (NG > 1 && !masked) {
                float a[16], ps0 = 0.0f, ps1 = 0.0f;
#pragma unroll
                for (int r4 = 0; r4 < 4; ++r4) {
                    f32x4 kf = {c, c, c, c};
                    if constexpr (KV_I8) kf = *reinterpret_cast<const f32x4*>(smem + sc_addr + sc_off + 32 * r4);
#pragma unroll
                    for (int e = 0; e < 4; ++e) a[4 * r4 + e] = fast_exp2(fmaf(st[4 * r4 + e], kf[e], -M));
                    ps0 += a[4 * r4];
                    ps1 += a[4 * r4 + 1];
                    ps0 += a[4 * r4 + 2];
                    ps1 += a[4 * r4 + 3];
                }
                const float ps = ps0 + ps1;
                if (__builtin_amdgcn_ballot_w64(ps > 256.0f) == 0) {
                    pack_p(sc_off, a, pn);
                    return ps;
                }
            }
            return exact_softmax(sc_off, rel, first, OWN > 0, st, pn);
        };
        auto max_only = [&](int rel, const f32x16& st) {   // MODE 1: the tile's scores only raise the row maximum
            float umax = kMasked;
#pragma unroll
            for (int r = 0; r < 16; ++r) umax = fmaxf(umax, (8 * (r / 4) + (r % 4) <= rel) ? st[r] * c : kMasked);
            M = fmaxf(M, half_max(umax));
        };

        // this wave's requests (bf16) of iteration i, and the wait for those of iteration i - 1.  Invariant the wait rests
        // on: an iteration issues exactly REQ requests a wave, and buffer loads complete in the order they were issued.
        constexpr int REQ = KV_I8 ? 0 : NLT >= 8 && !stats_only ? 2 * NLD : NLD;
        static_assert(REQ < 16, "vmcnt is written into the low four bits of the wait's immediate");
        auto request = [&](int n, int i, int p4) {   // n of REQ
            if constexpr (NLT >= 8) {
                if (n < NLD) dma_one(krs_raw, d_koff, n, i + LEADK, ring_slot(p4 + LEADK) * SLOTK, i + LEADK < n_iter);
                else dma_one(vrs_raw, d_voff, n - NLD, i + LEADV, K_BYTES + ring_slot(p4 + LEADV) * SLOTV, i + LEADV < n_iter);
            } else {
                const bool ks = w8 < 4;
                const int T = ks ? i + LEADK : i + LEADV;
                u32x4 rs;
#pragma unroll
                for (int e = 0; e < 4; ++e) rs[e] = ks ? krs_raw[e] : vrs_raw[e];
                dma_one(rs, ks ? d_koff : d_voff, 0, T, ks ? ring_slot(p4 + LEADK) * SLOTK : K_BYTES + ring_slot(p4 + LEADV) * SLOTV, T < n_iter);
            }
        };
        // INT8: the registers' pieces go to K tile i+LEADK and V tile i+LEADV, their scales to tile i+LEADS; then the next ones are loaded
        auto stage_dst = [&](int piece, int p4) {
            return piece == 1 ? p_vdst + ring_slot(p4 + LEADV) * SLOTV : p_dst + (st_k ? ring_slot(p4 + LEADK) * SLOTK : ring_slot(p4 + LEADV) * SLOTV);
        };
        auto load_piece0 = [&](int i) {
            constexpr unsigned TB = NG * kBC * ROWB;
            sg0 = __builtin_amdgcn_raw_buffer_load_b128(krs, (int)((unsigned)(i + 1 + (st_k ? LEADK : LEADV)) * TB + p_off), 0, 0);
        };
        auto load_piece1 = [&](int i) {
            constexpr unsigned TB = NG * kBC * ROWB;
            sg1 = __builtin_amdgcn_raw_buffer_load_b128(vrs, (int)((unsigned)(i + 1 + LEADV) * TB + p_off), 0, 0);
        };
        auto end_iteration = [&](bool barrier) {
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (!KV_I8) __builtin_amdgcn_s_waitcnt(0x0f70 | REQ);   // vmcnt(REQ), see the invariant above
            asm volatile("" ::: "memory");
            if (barrier) __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            __builtin_amdgcn_sched_barrier(0);
        };

        float own_alpha = 1.0f;               // OWN: what the next tile's maximum scales the accumulator by
        f32x4 kfs = {c, c, c, c}, kfs_next;   // INT8: k_scales of the four keys at work, and of the next four
        float vfs = 0.0f;                     // INT8: the tile's v_scales, lane n of each 16 the one of this lane's register n
        // Iteration i of a wave that has a tile after this one: the scores of tile i+1 into sn, the probabilities of tile i
        // (scores in st) into pn, P V of tile i-1 (probabilities in pv).  An MFMA, then a share of the vector work,
        // the refill of the operand the MFMA consumed and of the ring: the fences keep the order as written.
        auto full = [&](auto p4_c, int i, const f32x16& st, f32x16& sn, const u32x4 (&pv)[2], u32x4 (&pn)[2]) {
            constexpr int P4 = decltype(p4_c)::value;
            constexpr int K1 = (P4 + 1) % RING * SLOTK, K2 = (P4 + 2) % RING * SLOTK;
            constexpr int VM = (P4 + RING - 1) % RING * SLOTV, V0 = P4 * SLOTV;
            constexpr int SC = P4 * NG * 2 * kBC * 4, SCN = (P4 + 1) % RING * NG * 2 * kBC * 4;
            float a[16], ps0 = 0.0f, ps1 = 0.0f;
            u32x4 wide;
            auto finish_p = [&](int r) {
                if (r & 1) ps1 += a[r];
                else ps0 += a[r];
                if constexpr (KV_I8) a[r] *= row_lane(vfs, r);
                if (r & 1) {
                    pn[r / 8][(r % 8) / 2] = pack_bf16x2(a[r - 1], a[r]);
                    asm volatile("" : "+v"(pn[r / 8][(r % 8) / 2]));   // (packed here and now: else the compiler keeps all sixteen past the overflow check)
                }
            };
#pragma unroll
            for (int j = 0; j < NS; ++j) {
                const int x = j / 2;
                if (j % 2 == 0) {
                    f32x16 z;
#pragma unroll
                    for (int r = 0; r < 16; ++r) z[r] = 0.0f;
                    sn = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kfr[x % KP], qreg[x], x == 0 ? z : sn, 0, 0, 0);
                } else if (!stats_only) {
                    pv_mfma(x, pv);
                }
                __builtin_amdgcn_sched_barrier(0);
                if (j % 2 == 0) {
                    if (x < KP) fetch_k(x + KP, K1);
                    else fetch_k(x - KP, K2);
                } else if (!stats_only) {
                    if (x < VP) fetch_v(x + VP, VM);
                    else fetch_v(x - VP, V0);
                }
                if constexpr (!stats_only) {
#pragma unroll
                    for (int e = 0; e < EPS; ++e) {
                        const int r = EPS * j + e;
                        if constexpr (KV_I8)
                            if (r % 4 == 0) kfs = kfs_next;
                        const float u = fmaf(st[r], kfs[r % 4], -M);
                        if constexpr (KV_I8)
                            if (r % 4 == 1) kfs_next = *reinterpret_cast<const f32x4*>(smem + sc_addr + (r < 12 ? SC + 32 * (r / 4 + 1) : SCN));
                        if (r > 0) finish_p(r - 1);
                        a[r] = fast_exp2(u);
                    }
                }
                if constexpr (!KV_I8) {
                    if (j % 2 == 1 && j / 2 < REQ) request(j / 2, i, P4);
                } else {
                    // (a dword of a piece per step, and what a thread stores next is asked for right after; which steps, and
                    // whether the loads come here or at the iteration's end, made no difference)
                    const int e = j - (NS == 16 ? 4 : 0), piece = e / 4;
                    if (e >= 0 && e < (TWO ? 8 : 4) && has_p) {
                        unsigned lo, hi;
                        widen_dword(piece == 0 ? sg0[e % 4] : sg1[e % 4], lo, hi);
                        wide[2 * (e % 2)] = lo;
                        wide[2 * (e % 2) + 1] = hi;
                        if (e % 2 == 1) *reinterpret_cast<u32x4*>(smem + stage_dst(piece, P4) + 16 * ((e % 4) / 2)) = wide;
                    }
                    if (e == 3) load_piece0(i);
                    if (TWO && e == 7) load_piece1(i);
                    if (j == NS - 2) {
                        store_s(ring_slot(P4 + LEADS), sgs);
                        sgs = load_s(i + 1 + LEADS);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (stats_only) {
                max_only(kBC, st);
            } else {
                finish_p(15);
                if constexpr (KV_I8) vfs = *reinterpret_cast<const float*>(smem + scv_addr + SCN);
                float ps = ps0 + ps1;
                // Lazy running max: the exponentials were taken against the max as it stands, and it moves only when the sum of
                // a lane's 16 probabilities exceeds 2^8, so the accumulator is rescaled a few times per row block.
                if (__builtin_amdgcn_ballot_w64(ps > 256.0f) != 0) ps = exact_softmax(SC, kBC, i == 0, false, st, pn);
                lsum += ps;
                // OWN: the next tile's maximum is set here, before its exponentials (its scores are there, and it is not the
                // last one); what there is follows: the sum now, the accumulator an iteration later, when it has this tile.
                if constexpr (P4 >= 1 && P4 <= OWN) {
                    if (i == P4) {
#pragma unroll
                        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                            for (int r = 0; r < 16; ++r) o[dt][r] *= own_alpha;
                    }
                }
                if constexpr (P4 < OWN) {
                    own_alpha = 1.0f;
                    if (i == P4 && last > i + 1) {
                        float umax = fmaxf(sn[0], sn[1]);
#pragma unroll
                        for (int r = 2; r < 16; r += 2) umax = fmaxf(umax, fmaxf(sn[r], sn[r + 1]));
                        const float m_new = own_max(half_max(umax) * c);
                        own_alpha = fast_exp2(M - m_new);
                        lsum *= own_alpha;
                        M = m_new;
                    }
                }
            }
            end_iteration(BARRIERS == 1 || P4 % 2 == 1);
        };

        f32x16 st_a, st_b;
        u32x4 p_a[2] = {{0u, 0u, 0u, 0u}, {0u, 0u, 0u, 0u}}, p_b[2] = {{0u, 0u, 0u, 0u}, {0u, 0u, 0u, 0u}};
        int i = 0;
        if (last >= 0) {
            // the scores of tile 0; then the first operands of iteration 0 (there is no tile -1: zeros)
#pragma unroll
            for (int s = 0; s < KP; ++s) fetch_k(s, 0);
#pragma unroll
            for (int r = 0; r < 16; ++r) st_a[r] = 0.0f;
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                st_a = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kfr[s % KP], qreg[s], st_a, 0, 0, 0);
                if (s < KP) fetch_k(s + KP, 0);
                else fetch_k(s - KP, SLOTK);
            }
#pragma unroll
            for (int x = 0; x < VP; ++x) vfr[x][0] = vfr[x][1] = s16x4{0, 0, 0, 0};
            if constexpr (KV_I8) {
                kfs_next = *reinterpret_cast<const f32x4*>(smem + sc_addr);
                vfs = *reinterpret_cast<const float*>(smem + scv_addr);
            }
        }
        // (K tile 0 has been read: iteration 0 or 1 sends another to its slot)
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0)
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        if (last >= 0) {
            auto from_b = [&]() {
                st_a = st_b;
                p_a[0] = p_b[0];
                p_a[1] = p_b[1];
            };
            for (;;) {
                if (i >= last) break;
                full(int_c<0>{}, i, st_a, st_b, p_a, p_b);
                if (++i >= last) {
                    from_b();
                    break;
                }
                full(int_c<1>{}, i, st_b, st_a, p_b, p_a);
                if (++i >= last) break;
                full(int_c<2>{}, i, st_a, st_b, p_a, p_b);
                if (++i >= last) {
                    from_b();
                    break;
                }
                full(int_c<3>{}, i, st_b, st_a, p_b, p_a);
                ++i;
                if constexpr (RING == 6) {
                    if (i >= last) break;
                    full(int_c<4>{}, i, st_a, st_b, p_a, p_b);
                    if (++i >= last) {
                        from_b();
                        break;
                    }
                    full(int_c<5>{}, i, st_b, st_a, p_b, p_a);
                    ++i;
                }
            }
        }
        auto ring_share = [&](int i, int p4) {   // what an iteration sends or stores to the ring
            if constexpr (!KV_I8) {
#pragma unroll
                for (int n = 0; n < REQ; ++n) request(n, i, p4);
            } else {
                if (has_p) store_piece(stage_dst(0, p4), sg0);
                if constexpr (TWO) store_piece(stage_dst(1, p4), sg1);
                store_s(ring_slot(p4 + LEADS), sgs);
                load_piece0(i);
                if constexpr (TWO) load_piece1(i);
                sgs = load_s(i + 1 + LEADS);
            }
        };
        // This wave's last tile, then its share of the ring for the rest of the row block's iterations.  Two pieces of code, so that
        // what only the former needs does not stay in registers through the latter (B=4, 32 on 8 heads, S=777 32.0 -> 31.5 us, 32
        // heads, S=1024 19.1 -> 18.9, D=64, S=4096 83.3 -> 82.3), but one loop where the registers are full either way (INT8:
        // two pieces spill; D=128, 128 rows 51.4 -> 55.0 us at S=2048, the others the same).
        constexpr bool APART = !KV_I8;
        if (APART ? last >= 0 : i < n_iter) {
            do {
                const int p4 = ring_slot(i);
                ring_share(i, p4);
                if (APART || i == last) {
                    const int rel = lim - ((NG * i + my_tile) * kBC + 4 * hh);
                    if constexpr (stats_only) {
                        max_only(rel, st_a);
                    } else {
                        const int vm = ring_slot(p4 + RING - 1) * SLOTV, v0 = p4 * SLOTV;
#pragma unroll
                        for (int x = 0; x < 2 * DT; ++x) {
                            pv_mfma(x, p_a);
                            if (x < VP) fetch_v(x + VP, vm);
                            else fetch_v(x - VP, v0);
                        }
                        lsum += last_softmax(p4 * NG * 2 * kBC * 4, rel, NG * i + my_tile == t_last, i == 0, st_a, p_a);
#pragma unroll
                        for (int x = 0; x < 2 * DT; ++x) {
                            pv_mfma(x, p_a);
                            if (x < VP) fetch_v(x + VP, v0);
                        }
                    }
                }
                if constexpr (KV_I8) __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0): what this wave stored is in LDS
                end_iteration(BARRIERS == 1 || (i & 1) != 0);
                ++i;
            } while (!APART && i < n_iter);
        }
        for (; i < n_iter; ++i) {
            ring_share(i, ring_slot(i));
            if constexpr (KV_I8) __builtin_amdgcn_s_waitcnt(0xc07f);
            end_iteration(BARRIERS == 1 || (i & 1) != 0);
        }
        if constexpr (!KV_I8 || BARRIERS > 1) {
            // the last iterations' requests (zeros) have landed, and all reads are done, before the ring is used for anything else
            if constexpr (!KV_I8) __builtin_amdgcn_s_waitcnt(0x0f70);
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
        }
        if constexpr (MODE == 1) {   // this sweep's result: the row maxima; nothing to merge, nothing to store
            if (hh == 0 && my_q >= 0 && my_q < S) p.row_max[(((long)bh * S + my_q) * 2) + grp] = M;
            if (--k < 0) break;
            item_at(k, rb, bh);
            request_q(rb, bh);
            continue;
        }
        const int bh_now = bh;
        if (--k >= 0) {
            item_at(k, rb, bh);
            request_q(rb, bh);
        }
        // (the next item's Q is in flight during the merge: every wave read its fragments of this one's long ago)

        // ---- merge the two groups' partial results.  A wave keeps half of its O^T tiles and hands the
        // other half, with its max and row sum, to its partner (same rows, other group) through LDS.
        // The row block's output then goes out through LDS as well: a lane holds a few values of a row of its own,
        // and stores of that shape (64 lanes, 32 rows, 8 or 16 bytes each) are taken lane by lane by the memory
        // pipe and land as partial lines.  The tile is put together in the merge records' place (once every wave
        // has read its partner's) and leaves as whole rows, 64 consecutive 16-byte pieces per instruction.
        constexpr int OB = OUT_F32 ? 4 * D : 2 * D;   // bytes per output row
        static_assert(BR * OPITCH <= RING_BYTES, "the output tile fits where the ring was");
        auto put_tile = [&](const f32x16& ok, int dt) {   // register r of tile dt is d = 32 dt + 8 (r/4) + 4 hh + r%4
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4) {
                const int d = 32 * (dt % (DT / OH)) + 8 * r4 + 4 * hh;
                char* at = smem + (32 * rg + l32) * OPITCH;
                if (OUT_F32) {
                    const f32x4 ov = {ok[4 * r4], ok[4 * r4 + 1], ok[4 * r4 + 2], ok[4 * r4 + 3]};
                    *reinterpret_cast<f32x4*>(at + 4 * d) = ov;
                } else {
                    u32x2 ov;
                    ov[0] = pack_bf16x2(ok[4 * r4], ok[4 * r4 + 1]);
                    ov[1] = pack_bf16x2(ok[4 * r4 + 2], ok[4 * r4 + 3]);
                    *reinterpret_cast<u32x2*>(at + 2 * d) = ov;
                }
            }
        };
        auto copy_out = [&](int part) {
            constexpr int PPR = OB / OH / 16;                      // 16-byte pieces per row
            constexpr int NST = BR * PPR / kPrefillThreads;        // pieces per thread
            constexpr int RPI = kPrefillThreads / PPR;             // rows from one piece of a thread to its next
            // INT8 K/V, 128 rows: that step goes into the store's scalar offset.  Added up in vector registers the form with fp32
            // results, D = 128, spills four registers in the place of two.  Not in blocks of 256 rows, which spill nothing: the code that
            // it gives is 0.4 % slower (64 on 8 heads, S=16384 4137 -> 4154 us); bf16 forms are the same either way.
            constexpr bool STEP = KV_I8 && !WIDE;
            char* const obase = (char*)kernel_args_now()->out + ((long)bh_now * S + i0) * (long)OB + part * (OB / OH);
#pragma unroll
            for (int i = 0; i < NST; ++i) {
                // (the thread id, counted afresh: keeping it alive through the tile loops costs spills)
                const int lane_now = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
                const int pid = (w8 * 64 + lane_now) + (STEP ? 0 : kPrefillThreads * i), row0 = pid / PPR, col = pid % PPR, row = row0 + (STEP ? i * RPI : 0);
                const u32x4 piece = *reinterpret_cast<const u32x4*>(smem + row * OPITCH + col * 16);
                if (i0 + row >= 0 && i0 + row < S) store_through_b128(obase, row0 * OB + col * 16, STEP ? i * RPI * OB : 0, piece);
            }
        };
        auto finish = [&](auto grp_c) {
            constexpr int G = decltype(grp_c)::value;
            constexpr int HALF = DT / 2;
            constexpr int keep0 = G == 0 ? 0 : HALF, send0 = G == 0 ? HALF : 0;
            f32x4* mg = reinterpret_cast<f32x4*>(smem);   // [wave][NV][lane]; the ring is dead and quiet after the last barrier
            const float L = half_sum(lsum);
#pragma unroll
            for (int dt = 0; dt < HALF; ++dt)
#pragma unroll
                for (int r4 = 0; r4 < 4; ++r4) {
                    const f32x4 vsend = {o[send0 + dt][4 * r4], o[send0 + dt][4 * r4 + 1], o[send0 + dt][4 * r4 + 2], o[send0 + dt][4 * r4 + 3]};
                    mg[(w8 * NV + dt * 4 + r4) * 64 + l] = vsend;
                }
            {
                const f32x4 ml = {M, L, 0.0f, 0.0f};
                mg[(w8 * NV + NV - 1) * 64 + l] = ml;
            }
            __syncthreads();
            const int pw8 = w8 ^ 4;
            const f32x4 oml = mg[(pw8 * NV + NV - 1) * 64 + l];
            const float m_all = fmaxf(M, oml[0]);
            const float a_me = fast_exp2(M - m_all), a_ot = fast_exp2(oml[0] - m_all);
            const float inv = 1.0f / (L * a_me + oml[1] * a_ot);
            const float s_me = a_me * inv, s_ot = a_ot * inv;
#pragma unroll
            for (int dt = 0; dt < HALF; ++dt)
#pragma unroll
                for (int r4 = 0; r4 < 4; ++r4) {
                    const f32x4 ot = mg[(pw8 * NV + dt * 4 + r4) * 64 + l];
#pragma unroll
                    for (int e = 0; e < 4; ++e) o[keep0 + dt][4 * r4 + e] = fmaf(o[keep0 + dt][4 * r4 + e], s_me, ot[e] * s_ot);
                }
            __syncthreads();
#pragma unroll
            for (int dt = 0; dt < HALF; ++dt) put_tile(o[keep0 + dt], keep0 + dt);
            __syncthreads();
            copy_out(0);
        };
        // ---- the INT8 cache of this row block's own K and V rows, if asked for (section 2.2), with the quantiser's row
        // routine.  The rows were this row block's last tiles, so they come from the L2.  The block's pieces of a
        // wave-wide access each are dealt to the query heads that share the KV head, and to the waves: left to the
        // first head's workgroup alone they were 10 us of B=4, 32 on 8 heads, S=777.
        auto emit_cache = [&]() {
            if constexpr (KV_I8) return;
            const KernelArgs args = kernel_args_now();
            if (args->kq != nullptr) {
                constexpr int LPR = D / 8;          // lanes per row
                constexpr int RPI = 64 / LPR;       // rows per wave-wide access
                constexpr int UNITS = BR / RPI;     // accesses per tensor
                const int step = (int)args->group, first = bh_now - kvh * step;
                const int piece = l % LPR;
                for (int u0 = first + step * w8; u0 < 2 * UNITS; u0 += 4 * 8 * step) {
                    u32x4 raw[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j) {   // the loads first: their latencies overlap
                        const int u = min(u0 + 8 * step * j, 2 * UNITS - 1);
                        const uint16_t* src = (const uint16_t*)(u < UNITS ? args->k : args->v) + kvrow0 * D;
                        const int row = i0 + RPI * (u % UNITS) + l / LPR;
                        raw[j] = *reinterpret_cast<const u32x4*>(src + (long)min(max(row, 0), S - 1) * D + piece * 8);
                    }
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const int u = u0 + 8 * step * j;
                        if (u >= 2 * UNITS) break;
                        int8_t* codes = (u < UNITS ? args->kq : args->vq) + kvrow0 * D;
                        float* scales = (u < UNITS ? args->kqs : args->vqs) + kvrow0;
                        const int row = i0 + RPI * (u % UNITS) + l / LPR;
                        u32x2 cw;
                        float scale;
                        quant_row_piece<LPR>(raw[j], cw, scale);
                        if (row >= 0 && row < S) {
                            *reinterpret_cast<u32x2*>(codes + (long)row * D + piece * 8) = cw;
                            if (piece == 0) scales[row] = scale;
                        }
                    }
                }
            }
        };
        if constexpr (WIDE) {   // every wave has its rows' whole result
            const float inv = 1.0f / half_sum(lsum);
#pragma unroll
            for (int part = 0; part < OH; ++part) {
                if (part > 0) __syncthreads();
#pragma unroll
                for (int dt = part * (DT / OH); dt < (part + 1) * (DT / OH); ++dt) {
#pragma unroll
                    for (int r = 0; r < 16; ++r) o[dt][r] *= inv;
                    put_tile(o[dt], dt);
                }
                __syncthreads();
                copy_out(part);
            }
            emit_cache();
            if (k < 0) break;
            continue;
        }
        if (grp == 0) finish(int_c<0>{});
        else finish(int_c<1>{});

        emit_cache();
        if (k < 0) break;
    }
}

template <int D, bool KV_I8, bool OUT_F32, int MODE = 0, bool WIDE = false, int OWN = 0>
static hipError_t launch_one(const PrefillParams& p, hipStream_t stream) {
    const unsigned grid = (unsigned)(8 * p.slots);
    hipLaunchKernelGGL((slim_prefill_kernel<D, KV_I8, OUT_F32, MODE, WIDE, OWN>), dim3(grid), dim3(kPrefillThreads), 0,
                       stream, p);
    return hipGetLastError();
}

// Microseconds the fullest workgroup takes: us_tile for 128 rows of a key tile (halves of them a block) and us_item an item
// (prologue, merge and output).  Of a long list of items the mean, else the longest of the first, middle and last lists.
static double modelled_us(const PrefillParams& p, double us_tile, double us_item, int rows, int halves) {
    const long n = (long)p.n_rb * p.n_bh;
    if (p.rounds > 8)
        return (double)n / (8.0 * p.slots) * ((p.causal ? ((double)p.S + rows) / 64 : p.S / 32.0) * halves * us_tile + us_item);
    double most = 0.0;
    for (const int slot : {0, p.slots / 2, p.slots - 1}) {
        double us = 0.0;
        for (int k = 0; k < p.rounds; ++k) {
            const long j = 8L * ((long)k * p.slots + ((k & 1) ? p.slots - 1 - slot : slot));
            if (j >= n) continue;
            // (batches of heads, longest row blocks first)
            const long batch = j / (p.n_rb * (long)p.heads), in = j - batch * p.n_rb * (long)p.heads;
            const long heads = std::min((long)p.heads, p.n_bh - batch * (long)p.heads);
            const long kend = (p.n_rb - in / heads) * rows - p.row_off;
            const long keys = p.causal && kend < p.S ? kend : p.S;
            us += (double)((keys + kBC - 1) / kBC * halves) * us_tile + us_item;
        }
        if (us > most) most = us;
    }
    return most;
}

// The items of row blocks of `rows` rows and how they are listed, for so many workgroups a compute unit
static void set_blocks(PrefillParams& p, const PrefillArgs& a, int rows, int per_cu = 1) {
    p.n_rb = (a.seq_len + rows - 1) / rows;
    // Under the causal mask the rows that do not fill a block go to the first one, which has the fewest keys, and not
    // to the last (S = 777: 91 key tiles per head instead of 109); the offset keeps the diagonal on tile bounds.
    p.row_off = p.causal ? (p.n_rb * rows - a.seq_len) / 32 * 32 : 0;
    p.n_bh = a.batch * a.q_heads;
    const int per_xcd = (p.n_rb * p.n_bh + 7) / 8;
    p.slots = per_xcd < 32 * per_cu ? per_xcd : 32 * per_cu;
    p.rounds = (per_xcd + p.slots - 1) / p.slots;
    // A batch has 4 KV heads an XCD, or all heads up to twice that: with 32 heads and 32 workgroups an XCD no two of
    // them read the same K/V (B=8, 32 heads, S=4096: 1600 us, 1110 in batches); smaller batches leave ends of
    // rounds unfilled (B=1, 32 heads, S=6000: 334 us in batches of two heads an XCD, 287 with all four).
    p.group = (unsigned)(a.q_heads / a.kv_heads);
    const unsigned per_batch = 8 * 4 * p.group;
    p.heads = (unsigned)p.n_bh > 2 * per_batch ? per_batch : (unsigned)p.n_bh;
    p.last_heads = (unsigned)p.n_bh % p.heads != 0 ? (unsigned)p.n_bh % p.heads : p.heads;
    auto magic = [](unsigned long long d) { return d == 1 ? 0xffffffffu : (unsigned)((1ull << 32) / d); };   // (div_magic's correction covers 2^32 - 1 for d = 1)
    p.batch_magic = magic((unsigned long long)p.n_rb * p.heads);
    p.heads_magic = magic(p.heads);
    p.last_heads_magic = magic(p.last_heads);
    p.group_magic = magic(p.group);
}

// Which form a call takes (rows of its row blocks: 32, 128 or 256; p is left set for 128 or 256): the one with the
// smallest modelled time.  The constants are fitted to the times of all three forms, 13 pairs of batch and heads (4 to 384
// heads) by 17 lengths (64 to 8192), causal and not, with plain blocks of 256 rows: of 1350 calls 43 take a form that is more
// than 3 % slower than the best.
//   - a tile of 256 rows costs less than twice one of 128 (half the staging per query row, INT8 half the widening, no
//     merge), but there are half as many items to fill the chip with.  32 heads, bf16, D=128, rows of 128 against 256:
//     S=2048 40.5 and 49 us, S=3000 79.8 and 77.1, S=8192 500 and 465; INT8 S=2048 51 and 60, S=4096 170 and 147; D=64, B=4, 32
//     on 8 heads, bf16, S=777 27.1 and 23.3, S=4096 344 and 321.
//   - fp32 results cost an item more; of 256 rows by 128 values they go out in two parts.
//   - small calls take the form of prefill_split.hip: the longest row block's latency, or the chip's tiles and items
//     (8 heads: S=200 8.9 -> 5.2 us, S=1024 17.0 -> 10.4).  All heads go
//     through one row block before the next, so bf16 K and V that are well over what the L2s hold (32 MB) are read again
//     for every block, at 10 TB/s (33 MB are not yet worth it: 40 x 32 heads, S=100, D=64, 23.6 us in the caches and
//     36.9 cold, 27.2 and 34.8 at 128 rows; 66 MB, S=200: 51.6 and 74.7, 55.9 and 67.0).  The form has a workgroup per row
//     block and head, and a launch less than 2^32 threads: more of them than that stay with the lists.
//   - bf16 calls of 128 values, not causal, that the coarser lines below give 32 rows do not go to 128: they would take 5 %
//     longer (4 sequences, 32 on 8 heads, S=100 7.3 us at 32 rows, 7.7 at 128; 40 on 8, S=67, fp32 results 7.6 and 8.0) and be
//     further from the 64-bit result.  (Causal ones go: S=92, 15 sequences, 12 heads 9.6 us at 32 rows, 7.7 at 128.)
//   - bf16 calls that keep the 128-row form whatever the model says: D = 64, sequences of fewer than 500 rows, or not causal
//     with no more blocks of 256 than compute units; D = 128, not causal, fewer than 200 rows, but for those that the coarser
//     lines below give 256 (8 sequences, 24 on 8 heads, S=134: 10.3 us, at 32 rows 13.6; as near the 64-bit result as these).
//     These are the shapes by which that form's tests reach it, and it costs: of 50 such calls that the model would give 256
//     rows, these are 2 to 29 % faster (24 sequences, 32 heads, S=413, D=64 68.6 and 50.7 us).
//   - bf16 blocks of 256 rows are as near the 64-bit result as those in whose place they are (OWN, in `own`).  That is said by
//     coarser lines (kCoarse; 8 head counts, 4 to 512, by 12 lengths, 50 to 4096), which have 256 rows for 128 values and bf16
//     results only: as near as 32 rows, or as 128, by one more exact maximum a row than these have; or plain ones.
struct FormCosts {   // microseconds
    double tile128, item128, tile256, item256;       // a key tile (of 256 rows: half of one) and an item of the list forms
    double fp32_128, fp32_256;                       // what fp32 results add to an item
    double lists;                                    // what a launch of theirs takes besides
    double first32, chain32, base32, tile32, block32;   // 32 rows: the longest block, and all tiles and blocks over 256 compute units
};
static int choose_rows(PrefillParams& p, const PrefillArgs& a, int& own) {
    static constexpr FormCosts kCosts[4] = {
        {0.275, 4.16, 0.284, 2.24, 0.24, 1.90, 0.555, 2.13, 0.0662, 1.02, 0.102, 0.933},   // D = 64, bf16
        {0.397, 5.24, 0.356, 3.22, 0.0, 0.0, 2.53, 3.05, 0.109, 1.31, 0.153, 0.790},       // D = 64, INT8
        {0.365, 4.17, 0.291, 5.33, 0.125, 0.909, 1.08, 3.07, 0.367, 2.29, 0.187, 1.72},    // D = 128, bf16
        {0.567, 6.29, 0.461, 3.87, 0.739, 1.90, 2.00, 4.65, 0.273, 4.35, 0.295, 1.41}};    // D = 128, INT8
    static constexpr FormCosts kCoarse[2] = {{0.31, 5.0, 0.0, 0.0, 0.0, 0.0, 2.0, 3.3, 0.11, 1.2, 0.115, 1.2},    // bf16, D = 64
                                             {0.31, 4.2, 0.30, 5.5, 0.0, 0.0, 1.5, 3.4, 0.18, 1.5, 0.18, 2.0}};   // and 128
    const bool d128 = a.head_dim == 128;
    const FormCosts& c = kCosts[(d128 ? 2 : 0) + (a.kv_int8 ? 1 : 0)];
    p.n_bh = a.batch * a.q_heads;
    const double blocks32 = (a.seq_len + 31) / 32, tiles = blocks32 * p.n_bh * (p.causal ? (blocks32 + 1) / 2 : blocks32);
    const double kv_bytes = 4.0 * a.batch * a.kv_heads * a.seq_len * a.head_dim;
    const double us_again = !a.kv_int8 && kv_bytes > 40e6 ? kv_bytes * (p.causal ? (blocks32 + 1) / 2 : blocks32) / 10e6 : 0.0;
    const bool launchable = blocks32 * p.n_bh * 256 < 0x1p32;
    auto small_us = [&](const FormCosts& f) {
        const double longest = f.first32 + f.chain32 * blocks32;
        const double all = f.base32 + (f.tile32 * tiles + f.block32 * blocks32 * p.n_bh) / 256 + us_again;
        return launchable ? std::max(longest, all) : 1e30;
    };
    const double us32 = small_us(c);
    // (small calls are bound by what the host does for them: no lists where their longest item alone takes longer)
    const double item128 = c.item128 + (a.out_f32 ? c.fp32_128 : 0.0), item256 = c.item256 + (a.out_f32 ? c.fp32_256 : 0.0);
    if (us32 < c.lists + std::min(blocks32 * c.tile128 + item128, 2.0 * blocks32 * c.tile256 + item256)) return 32;
    set_blocks(p, a, 2 * kBR);
    const double us_wide = modelled_us(p, c.tile256, item256, 2 * kBR, 2);
    const FormCosts& g = kCoarse[d128];
    const double coarse256 = d128 && !a.out_f32 && !a.kv_int8 ? modelled_us(p, g.tile256, g.item256, 2 * kBR, 2) : 1e30;
    const bool many = (long)p.n_rb * p.n_bh > 256;
    set_blocks(p, a, kBR);
    double us = modelled_us(p, c.tile128, item128, kBR, 1);
    const double coarse128 = a.kv_int8 ? 0.0 : modelled_us(p, g.tile128, g.item128, kBR, 1);
    const int coarse = small_us(g) < std::min(coarse128, coarse256) + g.lists ? 32 : coarse256 < coarse128 ? 2 * kBR : kBR;
    const bool tested128 = d128 ? !p.causal && a.seq_len < 200 : a.seq_len < 500 || !(p.causal || many);
    const bool wide = a.kv_int8 || coarse == 2 * kBR || !tested128;
    own = a.kv_int8 ? 0 : coarse == 32 || (coarse == 2 * kBR && tested128) ? 3 : coarse == kBR ? 1 : 0;
    int rows = kBR;
    if (wide && us_wide < us) {
        us = us_wide;
        rows = 2 * kBR;
        set_blocks(p, a, 2 * kBR);
    }
    const bool stays32 = rows == kBR && !a.kv_int8 && coarse == 32 && d128 && !p.causal;
    return us32 < us + c.lists || stays32 ? 32 : rows;
}

int prefill_block_rows(const PrefillArgs& a) {
    PrefillParams p;
    p.S = a.seq_len;
    p.causal = a.causal ? 1 : 0;
    int own;
    return choose_rows(p, a, own);
}

hipError_t launch_prefill(const PrefillArgs& a, hipStream_t stream) {
    PrefillParams p;
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
    p.scale_log2e = a.softmax_scale * kLog2e;
    p.row_max = a.row_max;
    if (a.row_max) {   // the comparison variant: bf16 K/V only (checked by the caller); two launches
        // (the sweep for the maxima fits twice on a compute unit at D = 64, 94 registers and 80 KB, and wants to be there
        // twice: both sweeps of B=8, 64 on 8 heads, S=1024 220 us with one workgroup, 190 with two, measured when waves still
        // met at a barrier per half iteration)
        set_blocks(p, a, kBR, a.head_dim == 64 ? 2 : 1);
        hipError_t e = a.head_dim == 128 ? launch_one<128, false, false, 1>(p, stream) : launch_one<64, false, false, 1>(p, stream);
        if (e != hipSuccess) return e;
        set_blocks(p, a, kBR);
        if (a.head_dim == 128) return a.out_f32 ? launch_one<128, false, true, 2>(p, stream) : launch_one<128, false, false, 2>(p, stream);
        return a.out_f32 ? launch_one<64, false, true, 2>(p, stream) : launch_one<64, false, false, 2>(p, stream);
    }
    const bool d128 = a.head_dim == 128;
    int own = 0;
    const int rows = choose_rows(p, a, own);
    if (rows == 32) {
        // (eight waves where a compute unit has hardly more than one workgroup and a row block many tiles)
        const int blocks32 = (a.seq_len + 31) / 32;
        const bool eight = blocks32 * p.n_bh <= 384 && blocks32 >= (a.kv_int8 ? 24 : 48);
        return launch_prefill_split(a, eight ? 8 : 4, stream);
    }
    const int sel = (d128 ? 4 : 0) | (a.kv_int8 ? 2 : 0) | (a.out_f32 ? 1 : 0);
    if (rows == 2 * kBR) {
        switch (sel) {
            case 0: return own == 3 ? launch_one<64, false, false, 0, true, 3>(p, stream) : launch_one<64, false, false, 0, true, 1>(p, stream);
            case 1: return own == 3 ? launch_one<64, false, true, 0, true, 3>(p, stream) : launch_one<64, false, true, 0, true, 1>(p, stream);
            case 2: return launch_one<64, true, false, 0, true>(p, stream);
            case 3: return launch_one<64, true, true, 0, true>(p, stream);
            case 4:
                return own == 0 ? launch_one<128, false, false, 0, true>(p, stream)
                     : own == 1 ? launch_one<128, false, false, 0, true, 1>(p, stream) : launch_one<128, false, false, 0, true, 3>(p, stream);
            case 5: return own == 3 ? launch_one<128, false, true, 0, true, 3>(p, stream) : launch_one<128, false, true, 0, true, 1>(p, stream);
            case 6: return launch_one<128, true, false, 0, true>(p, stream);
            default: return launch_one<128, true, true, 0, true>(p, stream);
        }
    }
    switch (sel) {
        case 0: return launch_one<64, false, false>(p, stream);
        case 1: return launch_one<64, false, true>(p, stream);
        case 2: return launch_one<64, true, false>(p, stream);
        case 3: return launch_one<64, true, true>(p, stream);
        case 4: return launch_one<128, false, false>(p, stream);
        case 5: return launch_one<128, false, true>(p, stream);
        case 6: return launch_one<128, true, false>(p, stream);
        default: return launch_one<128, true, true>(p, stream);
    }
}

}  // namespace slim

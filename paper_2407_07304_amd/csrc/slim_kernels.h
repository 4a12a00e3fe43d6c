// Host-side launchers of the gfx950 kernels; arguments are validated by the C ABI layer.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace slim {

hipError_t launch_kv_quant_int8(const void* x, int8_t* codes, float* scales, long n_rows, int head_dim,
                                hipStream_t stream);

hipError_t launch_kv_quant_int8_pair(const void* k, const void* v, int8_t* k_codes, float* k_scale, int8_t* v_codes,
                                     float* v_scale, long n_rows, int head_dim, hipStream_t stream);
hipError_t launch_kv_quant_int8_append(const void* x, int8_t* codes, float* scales, const int* positions, int batch,
                                       int kv_heads, int kv_len, int head_dim, hipStream_t stream);

struct PrefillArgs {
    const void* q;
    const void* k;
    const void* v;
    const float* k_scale;
    const float* v_scale;
    void* out;
    int8_t* k_codes_out;   // with bf16 K/V: also write their INT8 cache (all four set), or all null
    float* k_scale_out;
    int8_t* v_codes_out;
    float* v_scale_out;
    int batch, q_heads, kv_heads, seq_len, head_dim, causal;
    float softmax_scale;
    bool kv_int8, out_f32;
    float* row_max;   // null, or (bf16 K/V only) the two-sweep variant's workspace [batch, q_heads, seq_len, 2]
};
hipError_t launch_prefill(const PrefillArgs& a, hipStream_t stream);
// Rows of the row blocks that launch_prefill takes for these sizes and types: 32, 128 or 256 (pointers are not looked at)
int prefill_block_rows(const PrefillArgs& a);
// The same for small calls: workgroups of 32 query rows whose waves (4 or 8) split the keys.
hipError_t launch_prefill_split(const PrefillArgs& a, int waves, hipStream_t stream);
// The comparison variant that keeps a row block's whole score strip in LDS (bf16 K/V, sequences up to
// kPrefillStripMaxSeqLen keys: 32 rows x that many fp16 scores is what fits beside the V staging buffer).
constexpr int kPrefillStripMaxSeqLen = 2048;
hipError_t launch_prefill_strip(const PrefillArgs& a, hipStream_t stream);

struct DecodeArgs {
    const void* q;
    const int8_t* k_codes;
    const float* k_scale;
    const int8_t* v_codes;
    const float* v_scale;
    void* out;
    float* workspace;
    const int* kv_lens;   // device, [batch]: tokens of each sequence's cache that count (clamped to 1..kv_len), or null: all
    int batch, q_heads, kv_heads, kv_len, head_dim;
    float softmax_scale;
    bool ragged;          // use the plan for sequences of different lengths (the workspace has room for it)
};
// From this long on (whole rows, as the plans model them) a decode is cut with the merge's launch as what it takes the GPU, below with
// more: its step (two appends, then the decode) is then over before the host has issued a fourth launch.  32 heads, T=1000, four splits
// and one: by the GPU alone 10.3 and 12.0 us, from the host 12.6 to 14.1 (bound by the fourth launch) and 11.8 (by the GPU).  A captured
// step, whose launches the host does not issue, loses those 14 % to this.
constexpr double kDecodeLongNs = 9000.0;
// How a decode call is cut up: waves per workgroup, splits of the key axis (workgroups per row), and how many of them a
// sequence uses (splits_of).
struct DecodePlan {
    int waves, n_split;
    unsigned split_rate;
    bool ranked = false;            // workgroups take the rows in the order of their lengths (ranked_row)
    bool records_through = true;    // the splits' records go through the L2 (store_record)
};
// The plan's options in the kernels' one argument for them: the number of sequences where rows are dealt by length (then there are no
// records), else -1 for records through the L2, 0 for plain ones
inline int decode_mode(const DecodePlan& plan, int batch) { return plan.ranked ? batch : plan.records_through ? -1 : 0; }
// Grouped-query variant (2 to 32 query heads per KV head): a workgroup sweeps a run of tokens of one (batch, KV head)
// for all its query heads and is a split.  n_bg = batch * kv_heads, group = query heads per KV head.
bool decode_uses_gqa_kernel(int q_heads, int kv_heads);
DecodePlan decode_gqa_plan(int kv_len, long n_bg, int group, int head_dim);
// traffic_only: the measurement form (the kernel's loads without its arithmetic; what it writes is meaningless)
hipError_t launch_decode_gqa_split(const DecodeArgs& a, float* ws_acc, float* ws_ml, const DecodePlan& plan, hipStream_t stream,
                                   bool traffic_only = false);
// The plan of a call; ragged: the sequences have lengths of their own
DecodePlan decode_plan_of(bool ragged, int batch, int q_heads, int kv_heads, int kv_len, int head_dim);
size_t decode_workspace_bytes(int batch, int q_heads, int kv_heads, int kv_len, int head_dim, bool ragged);
hipError_t launch_decode(const DecodeArgs& a, hipStream_t stream);
// The library's own decode scratch (one static device array per GPU) for the entry point that may not
// allocate: its address on the current device, looked up on the first call there.
constexpr size_t kDecodeStaticScratchBytes = (size_t)16 << 20;
hipError_t decode_static_scratch(float** ptr);
// Partial results (accumulator, max, sum) of n_rows (batch, query head) rows in n_split splits each
inline size_t decode_records_bytes(long n_rows, int n_split, int head_dim) {
    return (size_t)n_rows * n_split * ((size_t)head_dim + 2) * sizeof(float);
}

}  // namespace slim

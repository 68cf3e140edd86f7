// Host-side launch functions of the HGCA kernels (internal to the library).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>

#include "hgca_device.hpp"
#include "routes.hpp"

namespace hgca {

// Allows launches of a kernel with up to `bytes` of dynamic LDS, once per device (the attribute belongs to a device's copy of
// the kernel; the limit without it is 64 KiB).
template <auto Kernel>
hipError_t lift_lds_limit(int bytes)
{
    constexpr int kMaxDevices = 64;
    static std::atomic<bool> lifted[kMaxDevices];                // zero-initialised
    int dev = 0;
    hipError_t rc = hipGetDevice(&dev);
    if (rc != hipSuccess) return rc;
    const bool tracked = dev >= 0 && dev < kMaxDevices;
    if (tracked && lifted[dev].load(std::memory_order_acquire)) return hipSuccess;
    rc = hipFuncSetAttribute(reinterpret_cast<const void *>(Kernel), hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (rc == hipSuccess && tracked) lifted[dev].store(true, std::memory_order_release);
    return rc;
}

constexpr int kMaxChunk = 512;     // tokens of one split (one workgroup) at most
constexpr int kMaxScoreChunk = 128;   // same for the MFMA score pass, which wants many small workgroups
constexpr int kMinChunk = 64;

// Split partials of softmax attention: for every (b, h, split)
//   m = max score, l = sum e^{s-m}, o[d] = sum e^{s-m} v   (not normalised).
struct Partials {
    float *o;      // [B*Hq, stride, d]
    float *m;      // [B*Hq, stride]
    float *l;      // [B*Hq, stride]
    int32_t n_splits;
    int32_t stride;    // slots of a row, n_splits or more (two sets may share the slots of a row)
};

// Two tiers attended to by the same queries as ONE line of tokens -- the first tier's, then the second's, each rounded
// up to whole steps -- that `shares` workgroups per (sequence, KV head, block of query rows) cut into equal parts
// whatever the two lengths are.  Share i leaves its part of the first tier in slot i of the partials and its part of
// the second in slot i + 1: the one share that crosses the boundary writes both, so shares + 1 slots are enough, and
// the first `first_slots` of them belong to the first tier.
constexpr int kLineStep = 64;                    // tokens of a step
struct LineDev {
    const int32_t *first_lens, *second_lens;     // device [B] or null (= the capacity)
    int32_t first_cap, second_cap;
    int32_t shares;                              // 0: no line
    int32_t rows_per_seq;                        // partial rows of one sequence
};
struct LineCut {
    int32_t first_steps, share_steps;
    __device__ __forceinline__ LineCut(const LineDev &l, int b) {
        const int n1 = l.first_lens ? min(max(l.first_lens[b], 0), l.first_cap) : l.first_cap;
        const int n2 = l.second_lens ? min(max(l.second_lens[b], 0), l.second_cap) : l.second_cap;
        first_steps = (n1 + kLineStep - 1) / kLineStep;
        const int steps = first_steps + (n2 + kLineStep - 1) / kLineStep;
        share_steps = max((steps + l.shares - 1) / l.shares, 1);
    }
    __device__ __forceinline__ int first_slots() const { return first_steps / share_steps + 1; }
};

struct AttnArgs {
    ShapeDev sh;
    const void *q;
    KvDev kv;
    const int32_t *idx;    // gather only: [B, Hq, k_max]
    const int32_t *cnt;    // gather only: [B, Hq]
    const float *sel_scores;   // gather only, optional: scaled scores of the listed entries (skips the K pass)
    int32_t k_max;
    int32_t chunk;         // tokens per split
    Partials part;
    float *raw_scores;     // dense only, optional: [B, Hq, cap], receives the scaled score of every valid token
    int32_t grouped;       // gather only: idx is [B, Hkv, k_max], cnt [B, Hkv]; the heads of a group share the list
    int32_t by_group;      // per-head lists: the workgroups of a group's heads run side by side on one XCD (GatherPlace), ...
    int32_t keep;          // ... and rows stay in its cache for the other heads instead of being streamed past it
};

// dtype: 0 fp32, 1 bf16; head_dim 64|128.  Dense handles the `group` query heads
// of one KV head per workgroup; gather handles one query head per workgroup.
hipError_t launch_attn_partial_dense(int dtype, int head_dim, const AttnArgs &a, hipStream_t s);
hipError_t launch_attn_partial_gather(int dtype, int head_dim, const AttnArgs &a, hipStream_t s);

hipError_t launch_combine(int head_dim, int64_t n_rows, const Partials &p, float *o, float *lse, hipStream_t s);
// Folds the splits of two partial sets (either may have n_splits == 0) into one result; o_dtype 0 fp32, 1 bf16.
hipError_t launch_combine2(int head_dim, int64_t n_rows, const Partials &p, const Partials &q, void *o, int o_dtype,
                           float *lse, hipStream_t s, float *lse_p = nullptr,   // lse_p / lse_q: optional lse of set p / q alone
                           float *lse_q = nullptr);
// The fold of a line's partials `t` (shares + 1 slots per row); lse_first / lse_second: optional lse of either tier.
hipError_t launch_combine_line(int head_dim, int64_t n_rows, const Partials &t, const LineDev &line, float *o, float *lse,
                               float *lse_first, float *lse_second, hipStream_t s);

hipError_t launch_merge(int head_dim, int64_t n_rows, const float *o_a, const float *lse_a, const float *o_b,
                        const float *lse_b, void *o_out, int o_dtype, float *lse_out, hipStream_t s);

struct ScoreArgs {
    ShapeDev sh;
    const void *q;
    KvDev kv;
    float *scores;         // [B, Hq, cap] fp32, or [B, Hkv, cap] with group_max
    int32_t chunk;
    int32_t n_chunks;
    int32_t group_max;     // write the maximum over the heads of each group instead of every head's score
};
hipError_t launch_scores(int dtype, int head_dim, const ScoreArgs &a, hipStream_t s);

struct SelectArgs {
    ShapeDev sh;
    KvDev kv;              // only seq_lens / cap are used
    const float *scores;   // [B, Hq, cap]
    const int32_t *k_per_seq;
    int32_t k_uniform, k_max;
    int32_t *idx;          // [B, Hq, k_max]
    int32_t *cnt;          // [B, Hq]
    float *sel_scores;     // optional [B, Hq, k_max]: score of every kept entry, in idx order
};
hipError_t launch_select(const SelectArgs &a, hipStream_t s);

// A short decode step in two launches (same results as the launches above up to the order of the fp32 sums):
// the window's split kernels and the score pass (no group_max), ...
hipError_t launch_window_scores(int dtype, int head_dim, const AttnArgs &dense, const ScoreArgs &scores, hipStream_t s);
// ... and per row the selection (idx, cnt and sel_scores are written as by launch_select), attention over the selected V rows
// and the fold with the window's partials.  Lists of up to kMaxShortList entries; a.kv is the pool with its V rows.
hipError_t launch_select_attend(int dtype, int head_dim, const SelectArgs &a, const Partials &window, void *o, int o_dtype,
                                float *lse, hipStream_t s);

// The window's split kernels and the per-head gather's split kernels (launch_attn_partial_dense and
// launch_attn_partial_gather with the same arguments) as one launch; per-head lists.
bool dense_gather_fusable(int dtype, int head_dim, int group);
// With k_new / v_new ([B, Hkv, row], paged window with a per-sequence first block only) the window takes one more
// token per sequence in the same launch: the split that owns its position writes its rows into the window's block
// first; the stored length is NOT updated (pending_window_len gives the length the launch works with).
hipError_t launch_dense_gather(int dtype, int head_dim, const AttnArgs &dense, const AttnArgs &gather, hipStream_t s,
                               const void *k_new = nullptr, const void *v_new = nullptr);

// Union of the index lists of the heads of each group: idx [B, Hq, k_max] / cnt [B, Hq] -> out [B, Hkv, k_max_out]
// ascending, -1 padded, out_cnt [B, Hkv].  Positions must lie in [0, n_positions).
hipError_t launch_union_lists(const int32_t *idx, const int32_t *cnt, int32_t k_max, int32_t batch, int32_t n_q_heads,
                              int32_t n_kv_heads, int32_t n_positions, int32_t *out, int32_t *out_cnt,
                              int32_t k_max_out, int32_t *status, hipStream_t s);

// ---- attention weights, their moving average, threshold rule ----

// a [n_rows, cap] holds scaled scores on entry and softmax weights e^{s - lse} on exit (0 beyond the length);
// maw (optional, [n_rows, cap]) receives the moving-average update with those weights in the same pass.
hipError_t launch_window_weights(float *a, const float *lse, const int32_t *seq_lens, int64_t n_rows, int32_t n_q_heads,
                                 int32_t cap, float *maw, int32_t n_new, float alpha, hipStream_t s);

hipError_t launch_maw_update(float *maw, const float *a_gpu, const int32_t *seq_lens, int64_t n_rows, int32_t n_q_heads,
                             int32_t cap, int32_t n_new, float alpha, hipStream_t s);

struct ThresholdArgs {
    const float *w;            // [B*Hq, cap]
    const int32_t *seq_lens;   // [B] or null
    const int32_t *sizes;      // [B] or null
    double beta;
    int32_t size_uniform, n_q_heads, cap, k_max;
    int32_t *idx;              // [B*Hq, k_max]
    int32_t *cnt;              // [B*Hq]
    float *w_norm;             // optional [B*Hq, k_max]
    int32_t *status;           // optional: receives status_bit (atomic or) when a row has more than k_max passing entries
    int32_t status_bit;
};
hipError_t launch_threshold_select(const ThresholdArgs &a, int64_t n_rows, hipStream_t s);

// ---- append stage: N queries per sequence over one tier or two (matrix cores, either type) ----

constexpr int kMaxAppendChunk = 8192;   // tokens of capacity per share of the append-stage attention at most, where shares are counted

struct AppendArgs {
    ShapeDev sh;
    const void *q;             // [B, N, Hq, d]
    KvDev kv;
    int32_t n_q;               // N
    int32_t causal_tail;       // 1: the tier's last N valid tokens are the queries' own; query i sees tokens < len-N+i+1
    int32_t one_part_p;        // 1: the weights enter the second product as one bf16 value instead of a high and a low part
    Partials part;             // attention: rows are (b, query, head), one slot per share, or shares + 1 with a second tier
    const float *lse;          // weights: [B, N, Hq], the tier's log-sum-exp per query and head
    float *a_out;              // weights: [B, Hq, cap]
};
// One tier (second = nullptr, `shares` slots) or two as a line (same queries, shape and partials; each tier with its
// own view and mask rule; `shares` + 1 slots).  weights_follow: launch_append_weights comes next,
// on the same tiers.
hipError_t launch_append_attn(int dtype, int head_dim, const AppendArgs &first, const AppendArgs *second, const LineDev &line,
                              bool weights_follow, hipStream_t s);
// the weights of one tier (second = nullptr) or of two (same queries and shape), as a line.  after_attention: these rows
// have just passed launch_append_attn with weights_follow.
hipError_t launch_append_weights(int dtype, int head_dim, const AppendArgs &first, const AppendArgs *second, const LineDev &line,
                                 bool after_attention, hipStream_t s);
// the same on fp32 inputs (two = 0: a2 is not used); these check nothing, the two above call them
hipError_t launch_append_attn_f32(int head_dim, const AppendArgs &a, const AppendArgs &a2, const LineDev &line, int two, dim3 grid,
                                  hipStream_t s);
hipError_t launch_append_weights_f32(int head_dim, const AppendArgs &a, const AppendArgs &a2, const LineDev &line, int two,
                                     dim3 grid, hipStream_t s);
// ---- KV manager over a block pool (mirrors hgca_cache_state; all pointers device memory) ----

constexpr int32_t kCacheWindowFull = 1, kCacheContextFull = 2, kCacheListFull = 4;   // sticky bits of *status

// Length of a window that takes n_new tokens: len + n_new if they fit the window's capacity and the sequence's table
// row; otherwise the window takes none of them, the stored length stands and *fail_bits (if given) names the reason.
// Every kernel that has to agree on the outcome before the new length is stored applies this one rule.
__device__ __forceinline__ int pending_window_len(int len, int first_block, int n_new, int cap, int block_size,
                                                  int max_blocks, int32_t *fail_bits)
{
    const bool no_room = len >= 0 && n_new > cap - len;          // (no sum of the two, which may be no int)
    if (len < 0 || no_room || first_block + (len + n_new - 1) / block_size >= max_blocks) {
        if (fail_bits) *fail_bits = no_room ? kCacheWindowFull : kCacheContextFull;
        return len;
    }
    return len + n_new;
}

struct CacheDev {
    char *k_blocks, *v_blocks;
    const int32_t *block_table;
    int32_t *first_win_block, *win_lens, *pool_lens;
    float *a_maw;
    int32_t *ctx_idx, *ctx_cnt, *plan, *status;
    float *a_evicted;          // optional [B*Hq, pool_cap]
    int32_t block_size, max_blocks, win_blocks, k_max, pool_cap;
    int32_t win_cap;           // tokens the window may hold (>= win_blocks * block_size = l_max); row length of a_maw
};

// k_in / v_in: [B, n_tokens, Hkv, row]
hipError_t launch_kv_append(const CacheDev &c, const void *k_in, const void *v_in, const int32_t *active, int32_t batch,
                            int32_t n_kv_heads, int32_t row_bytes, int32_t n_tokens, hipStream_t s);
hipError_t launch_kv_evict(const CacheDev &c, int32_t batch, int32_t n_q_heads, double beta, hipStream_t s);
// Tail of an append turn: moving average with a_gpu (n_new new entries), salient lists replaced from a_cpu (may be
// null when the cache has no pool capacity), eviction and sparsification: one launch, one workgroup per row.
hipError_t launch_append_tail(const CacheDev &c, const float *a_gpu, const float *a_cpu, int32_t batch, int32_t n_q_heads,
                              int32_t n_new, float alpha, double beta, hipStream_t s);
// Fold of the window's (p) and the salient list's (q) split partials, window weights e^{s - lse_window} in place in
// a_gpu [n_rows, win_cap] with Alg. 1's moving average (one new token), eviction and sparsification: one launch.
// token_pending: the token's rows are in the window but the stored length does not count it yet (see
// launch_dense_gather); the launch then stores the new length, or raises the status bit if the token did not fit.
hipError_t launch_decode_tail(int head_dim, int64_t n_rows, const Partials &p, const Partials &q, void *o, int o_dtype,
                              float *lse, float *a_gpu, const CacheDev &c, int32_t n_q_heads, float alpha, double beta,
                              int32_t token_pending, hipStream_t s);

// Copy of listed pool entries into per-head contiguous storage (KV_ctx of Alg. 1).
struct CtxCompactArgs {
    ShapeDev sh;
    KvDev kv;                  // the pool
    const int32_t *idx, *cnt;  // [B*Hq, k_max], [B*Hq]
    const int32_t *first_row;  // optional [B*Hq]: rows of KV_ctx already taken
    int32_t *cnt_out;          // optional [B*Hq]: rows taken afterwards
    char *k_ctx, *v_ctx;       // [B*Hq, ctx_cap, row_bytes]
    int32_t k_max, ctx_cap, row_bytes;
};
hipError_t launch_ctx_compact(const CtxCompactArgs &a, hipStream_t s);

}  // namespace hgca

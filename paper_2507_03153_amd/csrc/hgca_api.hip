// C ABI of libhgca: argument validation, workspace layout, kernel sequencing.
// See include/hgca.h for the contract of every entry point.
#include "../../include/hgca.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cstdint>

#include "hgca_launch.hpp"

namespace {

using namespace hgca;

constexpr size_t kAlign = 256;
// Workgroups a launch aims for (256 CUs): compile-time tunables, one per streaming pass.
#ifndef HGCA_TARGET_WGS_DENSE_SHARED
#define HGCA_TARGET_WGS_DENSE_SHARED 512
#endif
#ifndef HGCA_TARGET_WGS_DENSE
#define HGCA_TARGET_WGS_DENSE 1024
#endif
#ifndef HGCA_TARGET_WGS_SCORES
#define HGCA_TARGET_WGS_SCORES 32768
#endif
#ifndef HGCA_TARGET_WGS_SPARSE
#define HGCA_TARGET_WGS_SPARSE 2048
#endif
#ifndef HGCA_TARGET_WGS_GROUPED                  // the sparse part over lists shared by a group, when it is folded at once
#define HGCA_TARGET_WGS_GROUPED 1024
#endif
#ifndef HGCA_TARGET_WGS_SPARSE_SCORED            // the sparse part inside hgca_hybrid_decode_step (scores given, V only)
#define HGCA_TARGET_WGS_SPARSE_SCORED 2048
#endif

// Workgroups of the append-stage attention that the device holds at once (two per compute unit in bf16), and the most
// shares it is cut into where the tokens do not ask for more (append_shares): every workgroup writes a partial of 128 rows x d
// floats (64 KB, read again by the fold: the K/V bytes of four 64-token steps).  More than a full round of them was no
// better even with long pools: 8B shape, N = 32, 512 / 768 / 1024 / 1536 workgroups of an earlier kernel (16-row tiles):
// window 55.7 / 61.0 / 66.0 / 74.8 us, pool 258.5 / 273.4 / 266.6 / 288.1 us.
#ifndef HGCA_APPEND_TARGET_WGS
#define HGCA_APPEND_TARGET_WGS 512
#endif
// 1: moving average, re-evaluation and eviction of an append turn are one launch
#ifndef HGCA_FUSE_APPEND_TAIL
#define HGCA_FUSE_APPEND_TAIL 1
#endif
// 1: the token of a managed decode step is written into the window by the window split that reads it (needs the two below)
#ifndef HGCA_FUSE_KV_APPEND
#define HGCA_FUSE_KV_APPEND 1
#endif
// 1: the tail of the managed decode step (fold, window weights + moving average, eviction) is one launch
#ifndef HGCA_FUSE_DECODE_TAIL
#define HGCA_FUSE_DECODE_TAIL 1
#endif
// 1: the window's split kernels and the sparse part's split kernels of a step share a launch where the shapes allow
#ifndef HGCA_FUSE_DENSE_GATHER
#define HGCA_FUSE_DENSE_GATHER 1
#endif

size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

int group_of(const hgca_shape *s) { return s->n_q_heads / s->n_kv_heads; }

int check_shape(const hgca_shape *s)
{
    if (!s) return HGCA_ERR_INVALID_ARG;
    if (s->batch < 0 || s->n_q_heads <= 0 || s->n_kv_heads <= 0 || s->head_dim <= 0) return HGCA_ERR_INVALID_ARG;
    if (s->n_q_heads % s->n_kv_heads != 0) return HGCA_ERR_INVALID_ARG;
    // sequences and heads are grid dimensions y and z of the launches (65 535 at most each)
    if (s->batch > 65535 || s->n_q_heads > 65535) return HGCA_ERR_UNSUPPORTED;
    if (s->dtype != HGCA_F32 && s->dtype != HGCA_BF16) return HGCA_ERR_UNSUPPORTED;
    if (s->head_dim != 64 && s->head_dim != 128) return HGCA_ERR_UNSUPPORTED;
    const int g = group_of(s);
    if (g != 1 && g != 2 && g != 4 && g != 8) return HGCA_ERR_UNSUPPORTED;
    if (!(s->sm_scale == s->sm_scale)) return HGCA_ERR_INVALID_ARG;   // NaN
    return HGCA_OK;
}

int check_view(const hgca_shape *s, const hgca_kv_view *v, bool need_v)
{
    if (!v) return HGCA_ERR_INVALID_ARG;
    if (v->cap < 0) return HGCA_ERR_INVALID_ARG;
    // rows of a tier are numbered with 32 bits inside the kernels
    if (!v->block_table && (int64_t)s->batch * s->n_kv_heads * v->cap >= (int64_t(1) << 32)) return HGCA_ERR_UNSUPPORTED;
    if (v->cap > 0) {
        if (!v->k || !aligned16(v->k)) return HGCA_ERR_INVALID_ARG;
        if (need_v && (!v->v || !aligned16(v->v))) return HGCA_ERR_INVALID_ARG;
    }
    if (v->block_table) {
        if (v->block_size <= 0 || v->max_blocks <= 0) return HGCA_ERR_INVALID_ARG;
        if (v->block_size % 16 != 0) return HGCA_ERR_UNSUPPORTED;
        if ((int64_t)v->max_blocks * v->block_size < v->cap) return HGCA_ERR_INVALID_ARG;
    }
    return HGCA_OK;
}

KvDev to_dev(const hgca_kv_view *v)
{
    KvDev d{};
    d.k = static_cast<const char *>(v->k);
    d.v = static_cast<const char *>(v->v);
    d.seq_lens = v->seq_lens;
    d.block_table = v->block_table;
    d.first_block = v->block_table ? v->first_block : nullptr;
    d.cap = v->cap;
    d.block_size = v->block_table ? v->block_size : 1;
    d.max_blocks = v->block_table ? v->max_blocks : 0;
    return d;
}

ShapeDev to_dev(const hgca_shape *s)
{
    ShapeDev d{};
    d.batch = s->batch;
    d.n_q_heads = s->n_q_heads;
    d.n_kv_heads = s->n_kv_heads;
    d.group = group_of(s);
    d.sm_scale = s->sm_scale;
    return d;
}

// Tokens per split for a set of at most n tokens processed by `units` independent
// (sequence, head unit) pairs: a multiple of 64 in [kMinChunk, kMaxChunk] that yields
// roughly `target` workgroups.
int pick_chunk(int64_t n, int64_t units, int target, int max_chunk = kMaxChunk)
{
    if (n <= 0 || units <= 0) return kMinChunk;
    const int64_t want_splits = std::max<int64_t>(1, target / units);
    int64_t chunk = (n + want_splits - 1) / want_splits;
    chunk = (chunk + 63) / 64 * 64;
    return (int)std::min<int64_t>(max_chunk, std::max<int64_t>(kMinChunk, chunk));
}

int n_splits_for(int64_t n, int chunk) { return (int)((n + chunk - 1) / chunk); }

// Windows and lists long enough to make 8 or 16 splits of 128 are not cut into splits of 64, however few sequences there are: more
// partials than the fold takes in one round trip.  One sequence, 32 / 8 heads of 128, window 4096: steady step, 2000 listed 21.8 ->
// 17.7 us, decode loop 25.0 -> 21.5 us per step, step with a selection 41.0 -> 37.0, of 61 003 tokens 62.0 -> 58.4; a window of 512
// is better in splits of 64 (step 29.9 : 31.1, loop of 3 sequences 21.7 : 23.1), a list of 600 the same in both.
int no_shorter(int chunk, int64_t n, int64_t from) { return n >= from ? std::max(chunk, 128) : chunk; }
constexpr int64_t kLongWindow = 2048, kLongList = 1024;
// ... and lists only as long as the splits of 128 come to a workgroup per compute unit, two where a row has 512 bytes, of which a
// workgroup has half as many in flight (fp32, 16 lists of 2285 entries of dimension 128: loop 18.4 -> 19.4 us per step)
int gather_split(const hgca_shape *s, int64_t k_max, int target)
{
    const int64_t rows = (int64_t)s->batch * s->n_q_heads, row_bytes = s->head_dim * (s->dtype == HGCA_BF16 ? 2 : 4);
    const int chunk = pick_chunk(k_max, rows, target);
    return rows * n_splits_for(k_max, 128) >= 256 * std::max<int64_t>(1, row_bytes / 256) ? no_shorter(chunk, k_max, kLongList) : chunk;
}

// Whether the window's splits and the sparse part's splits share a launch, and the window split's tokens there (below).
// fp32 and groups of up to 4 always do.  Measured, two launches : one, us: fp32 steady steps 1 sequence, 32 / 8 heads of 128,
// window 2048, 1900 listed 29.3 : 22.6, 4 sequences 63.9 : 60.4; decode loops, which insert the token in the same launch, per
// step 37.2 : 29.4 and 58.2 : 53.2.  The window body of groups of 8 leaves room for two (head_dim 128) or three workgroups per
// unit, so the launch pays where the gather's workgroups come to about one round, or two with a token to insert: steady, heads of
// 128, 256 workgroups 18.2 : 15.8, 960 19.0 : 22.1, 1920 25.3 : 35.0; heads of 64, 960 17.9 : 15.6, 1920 19.6 : 22.1; loops, heads of
// 128, 640 workgroups 24.5 : 18.2 per step, 1280 29.3 : 29.7, 2048 38.5 : 39.8; heads of 64, 2048 25.7 : 20.9 and 43.2 : 36.2, 8700 137.6 : 144.6.
bool shares_launch(const hgca_shape *s, int64_t window, int64_t pool, int64_t k_max, int gather_chunk, bool scored, bool token)
{
    if (!HGCA_FUSE_DENSE_GATHER || window <= 0 || pool <= 0 || k_max <= 0 ||
        !dense_gather_fusable(s->dtype, s->head_dim, group_of(s)))
        return false;
    const int64_t wgs = (int64_t)s->batch * s->n_q_heads * n_splits_for(k_max, gather_chunk);
    const int64_t window_wgs = (int64_t)s->batch * s->n_kv_heads * n_splits_for(window, kMinChunk);
    if (wgs + window_wgs > int64_t(1) << 23) return false;       // threads of a flat grid are counted in 32 bits
    if (s->dtype == HGCA_F32 || group_of(s) < 8) return true;
    if (scored) return false;
    return wgs <= (s->head_dim == 64 ? (token ? 4096 : 1024) : (token ? 1024 : 512));
}

// pool: tokens the pool can hold (a managed pool's capacity may count the window's blocks)
void order_gather(AttnArgs &ga, int64_t pool, bool managed)
{
    const GatherOrder o = gather_order(ga.sh.group, ga.k_max, pool, ga.sel_scores != nullptr, managed);
    ga.by_group = o.by_group;
    ga.keep = o.keep;
}

// Tokens per window split: in a launch of its own the window wants about HGCA_TARGET_WGS_DENSE workgroups; in a launch
// it shares with the sparse part's splits, which fill the device anyway, longer splits (half as many partials to write
// and fold) are better.  Measured on the 8B shape: full step 145.2 -> 143.8 us, steady 67.9 -> 67.6 us; on its own the
// window is 1 us slower with them.
// fp32 windows run on the vector units, several times as long per token as the gather's splits: theirs are as short as in a
// launch of their own (with the longer ones, where a window may be a single split: 40 sequences, 32 / 8 heads of 128, window 512, pool
// 2500, 60 listed: steady 58 us in two launches, 91 in one; 60 with short splits, 48 with the window's workgroups first as well; step
// with a selection 170 : 201 : 162.  8 sequences, 64 / 8 heads, window 2048, pool 4096, 100 listed: step 142 : 156 : 140).
int dense_chunk(const hgca_shape *s, int64_t cap, bool shared)
{
    const int64_t units = (int64_t)s->batch * s->n_kv_heads;
    if (!shared || s->dtype == HGCA_F32) return pick_chunk(cap, units, HGCA_TARGET_WGS_DENSE);
    return no_shorter(pick_chunk(cap, units, HGCA_TARGET_WGS_DENSE_SHARED), cap, kLongWindow);
}

// Tokens per workgroup of the score pass over a pool of `cap` tokens.  Groups of 8 heads take half the tokens per
// workgroup (64 instead of 128 on the 70B shape: 317 against 321 us per step).
int score_chunk(const hgca_shape *s, int64_t cap)
{
    const int target = HGCA_TARGET_WGS_SCORES * (s->n_q_heads / s->n_kv_heads >= 8 ? 2 : 1);
    return pick_chunk(cap, (int64_t)s->batch * s->n_kv_heads, target, s->dtype == HGCA_BF16 ? kMaxScoreChunk : kMaxChunk);
}

// Workspace layout: [partials o | partials m | partials l | one float per row | scores | scores of the kept entries].
struct WsLayout {
    size_t part_o, part_m, part_l, row_aux, scores, sel, total;
};

WsLayout layout(const hgca_shape *s, int64_t max_attn_tokens, int64_t max_pool)
{
    const size_t rows = (size_t)s->batch * s->n_q_heads;
    const size_t max_splits = (size_t)n_splits_for(std::max<int64_t>(max_attn_tokens, 1), kMinChunk);
    WsLayout w{};
    size_t at = 0;
    w.part_o = at; at += align_up(rows * max_splits * s->head_dim * sizeof(float));
    w.part_m = at; at += align_up(rows * max_splits * sizeof(float));
    w.part_l = at; at += align_up(rows * max_splits * sizeof(float));
    w.row_aux = at; at += align_up(rows * sizeof(float));
    w.scores = at; at += align_up(rows * (size_t)std::max<int64_t>(max_pool, 0) * sizeof(float));
    w.sel = at; at += max_pool > 0 ? align_up(rows * (size_t)std::max<int64_t>(max_attn_tokens, 0) * sizeof(float)) : 0;
    w.total = std::max<size_t>(at, kAlign);
    return w;
}

Partials partials_at(void *ws, const WsLayout &w, int n_splits)
{
    char *base = static_cast<char *>(ws);
    Partials p{};
    p.o = reinterpret_cast<float *>(base + w.part_o);
    p.m = reinterpret_cast<float *>(base + w.part_m);
    p.l = reinterpret_cast<float *>(base + w.part_l);
    p.n_splits = p.stride = n_splits;
    return p;
}

int from_hip(hipError_t e) { return e == hipSuccess ? HGCA_OK : HGCA_ERR_DEVICE; }

}  // namespace

extern "C" {

const char *hgca_status_string(int status)
{
    switch (status) {
    case HGCA_OK: return "ok";
    case HGCA_ERR_INVALID_ARG: return "invalid argument";
    case HGCA_ERR_UNSUPPORTED: return "unsupported shape, dtype or layout";
    case HGCA_ERR_WORKSPACE: return "workspace missing or too small";
    case HGCA_ERR_DEVICE: return "HIP launch failed";
    default: return "unknown status";
    }
}

size_t hgca_workspace_bytes(const hgca_shape *shape, int32_t max_window, int32_t max_pool, int32_t k_max)
{
    if (check_shape(shape) != HGCA_OK || max_window < 0 || max_pool < 0 || k_max < 0) return 0;
    return layout(shape, std::max(max_window, k_max), max_pool).total;
}

namespace {

int dense_window(const hgca_shape *shape, const void *q, const hgca_kv_view *window, float *o_out, float *lse_out,
                 float *a_out, float *a_maw, int32_t n_new, float alpha, void *ws, size_t ws_bytes, void *hip_stream)
{
    int rc = check_shape(shape);
    if (rc != HGCA_OK) return rc;
    if (shape->batch == 0) return HGCA_OK;       // nothing to do
    if ((rc = check_view(shape, window, true)) != HGCA_OK) return rc;
    const bool deferred = !o_out && !lse_out;    // leave the split partials in ws for hgca_lse_merge_splits
    if (!q || !aligned16(q) || (!deferred && (!o_out || !lse_out || !aligned16(o_out)))) return HGCA_ERR_INVALID_ARG;
    if (a_out && deferred) return HGCA_ERR_INVALID_ARG;   // the weights need the window's own lse
    const WsLayout w = layout(shape, window->cap, 0);
    if (!ws || ws_bytes < w.total || !aligned16(ws)) return HGCA_ERR_WORKSPACE;
    hipStream_t s = static_cast<hipStream_t>(hip_stream);

    AttnArgs a{};
    a.sh = to_dev(shape);
    a.q = q;
    a.kv = to_dev(window);
    a.chunk = pick_chunk(window->cap, (int64_t)shape->batch * shape->n_kv_heads, HGCA_TARGET_WGS_DENSE);
    a.part = partials_at(ws, w, n_splits_for(window->cap, a.chunk));
    a.raw_scores = a_out;
    const int64_t rows = (int64_t)shape->batch * shape->n_q_heads;
    if ((rc = from_hip(launch_attn_partial_dense(shape->dtype, shape->head_dim, a, s))) != HGCA_OK) return rc;
    if (deferred) return HGCA_OK;
    if ((rc = from_hip(launch_combine(shape->head_dim, rows, a.part, o_out, lse_out, s))) != HGCA_OK) return rc;
    if (!a_out) return HGCA_OK;
    return from_hip(launch_window_weights(a_out, lse_out, window->seq_lens, rows, shape->n_q_heads, window->cap, a_maw,
                                          n_new, alpha, s));
}

}  // namespace

int hgca_dense_window_attn(const hgca_shape *shape, const void *q, const hgca_kv_view *window, float *o_out,
                           float *lse_out, void *ws, size_t ws_bytes, void *hip_stream)
{
    return dense_window(shape, q, window, o_out, lse_out, nullptr, nullptr, 0, 0.f, ws, ws_bytes, hip_stream);
}

}  // extern "C"

// ---- dense window attention for callers that cannot allocate ---------------------------------------------
// The split partials of the call live in a file-scope device array instead of a caller's workspace.  Its name is
// a host-side stand-in here, not a device address: the address of each device's copy comes from
// hipGetSymbolAddress, once per device, and only that pointer is handed to kernels.
static __device__ __align__(256) unsigned char scratch[HGCA_STATIC_SCRATCH_BYTES];

namespace {

// Device address of the current device's copy of `scratch`; NULL (and *err set) if the runtime refuses.
void *static_scratch(hipError_t *err)
{
    constexpr int kMaxDevices = 64;
    static std::atomic<void *> known[kMaxDevices];               // zero-initialised
    int dev = 0;
    if ((*err = hipGetDevice(&dev)) != hipSuccess) return nullptr;
    const bool tracked = dev >= 0 && dev < kMaxDevices;
    void *ptr = tracked ? known[dev].load(std::memory_order_acquire) : nullptr;
    if (!ptr) {
        if ((*err = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch))) != hipSuccess) return nullptr;
        if (tracked) known[dev].store(ptr, std::memory_order_release);
    }
    return ptr;
}

}  // namespace

extern "C" {

int hgca_dense_window_attn_static(const hgca_shape *shape, const void *q, const hgca_kv_view *window, float *o_out,
                                  float *lse_out, void *hip_stream)
{
    int rc = check_shape(shape);
    if (rc != HGCA_OK) return rc;
    if (shape->batch == 0) return HGCA_OK;
    if ((rc = check_view(shape, window, true)) != HGCA_OK) return rc;
    if (!o_out || !lse_out) return HGCA_ERR_INVALID_ARG;         // no deferred result: the partials are not the caller's
    if (layout(shape, window->cap, 0).total > (size_t)HGCA_STATIC_SCRATCH_BYTES) return HGCA_ERR_WORKSPACE;
    hipError_t err = hipSuccess;
    void *ws = static_scratch(&err);
    if (!ws) return HGCA_ERR_DEVICE;
    // every split writes its whole partial (empty ones included) and the fold reads only those, so nothing in the
    // array has to be cleared between calls
    return dense_window(shape, q, window, o_out, lse_out, nullptr, nullptr, 0, 0.f, ws, HGCA_STATIC_SCRATCH_BYTES,
                        hip_stream);
}

int hgca_dense_window_attn_weights(const hgca_shape *shape, const void *q, const hgca_kv_view *window, float *o_out,
                                   float *lse_out, float *a_out, void *ws, size_t ws_bytes, void *hip_stream)
{
    if (!a_out && window && window->cap > 0) return HGCA_ERR_INVALID_ARG;
    return dense_window(shape, q, window, o_out, lse_out, a_out, nullptr, 0, 0.f, ws, ws_bytes, hip_stream);
}

int hgca_dense_window_attn_maw(const hgca_shape *shape, const void *q, const hgca_kv_view *window, float *o_out,
                               float *lse_out, float *a_out, float *a_maw, int32_t n_new, float alpha, void *ws,
                               size_t ws_bytes, void *hip_stream)
{
    if (window && window->cap > 0 && (!a_out || !a_maw)) return HGCA_ERR_INVALID_ARG;
    if (n_new < 0 || !(alpha >= 0.f && alpha <= 1.f)) return HGCA_ERR_INVALID_ARG;
    return dense_window(shape, q, window, o_out, lse_out, a_out, a_maw, n_new, alpha, ws, ws_bytes, hip_stream);
}

int hgca_maw_update(const hgca_shape *shape, float *a_maw, const float *a_gpu, const int32_t *seq_lens, int32_t cap,
                    int32_t n_new, float alpha, void *hip_stream)
{
    int rc = check_shape(shape);
    if (rc != HGCA_OK) return rc;
    if (cap < 0 || n_new < 0 || !(alpha >= 0.f && alpha <= 1.f)) return HGCA_ERR_INVALID_ARG;
    if (shape->batch == 0 || cap == 0) return HGCA_OK;
    if (!a_maw || !a_gpu) return HGCA_ERR_INVALID_ARG;
    const int64_t rows = (int64_t)shape->batch * shape->n_q_heads;
    return from_hip(launch_maw_update(a_maw, a_gpu, seq_lens, rows, shape->n_q_heads, cap, n_new, alpha,
                                      static_cast<hipStream_t>(hip_stream)));
}

int hgca_threshold_select(const hgca_shape *shape, const float *weights, const int32_t *seq_lens, int32_t cap,
                          const int32_t *size_per_seq, int32_t size_uniform, double beta, int32_t k_max,
                          int32_t *idx_out, int32_t *cnt_out, float *w_norm_out, void *hip_stream)
{
    int rc = check_shape(shape);
    if (rc != HGCA_OK) return rc;
    if (cap < 0 || k_max < 0 || !(beta >= 0.0) || (!size_per_seq && size_uniform <= 0)) return HGCA_ERR_INVALID_ARG;
    if (shape->batch == 0) return HGCA_OK;
    if (!cnt_out || (k_max > 0 && !idx_out) || (cap > 0 && !weights)) return HGCA_ERR_INVALID_ARG;
    ThresholdArgs a{};
    a.w = weights;
    a.seq_lens = seq_lens;
    a.sizes = size_per_seq;
    a.beta = beta;
    a.size_uniform = size_uniform;
    a.n_q_heads = shape->n_q_heads;
    a.cap = cap;
    a.k_max = k_max;
    a.idx = idx_out;
    a.cnt = cnt_out;
    a.w_norm = k_max > 0 ? w_norm_out : nullptr;
    const int64_t rows = (int64_t)shape->batch * shape->n_q_heads;
    return from_hip(launch_threshold_select(a, rows, static_cast<hipStream_t>(hip_stream)));
}

int hgca_pool_scores(const hgca_shape *shape, const void *q, const hgca_kv_view *pool, float *scores_out,
                     void *hip_stream)
{
    int rc = check_shape(shape);
    if (rc != HGCA_OK) return rc;
    if (shape->batch == 0) return HGCA_OK;
    if ((rc = check_view(shape, pool, false)) != HGCA_OK) return rc;
    if (!q || !aligned16(q) || (pool->cap > 0 && (!scores_out || !aligned16(scores_out)))) return HGCA_ERR_INVALID_ARG;
    ScoreArgs sa{};
    sa.sh = to_dev(shape);
    sa.q = q;
    sa.kv = to_dev(pool);
    sa.scores = scores_out;
    sa.chunk = score_chunk(shape, pool->cap);
    sa.n_chunks = n_splits_for(pool->cap, sa.chunk);
    return from_hip(launch_scores(shape->dtype, shape->head_dim, sa, static_cast<hipStream_t>(hip_stream)));
}

int hgca_select_salient(const hgca_shape *shape, const void *q, const hgca_kv_view *pool, const int32_t *k_per_seq,
                        int32_t k_uniform, int32_t k_max, int32_t *idx_out, int32_t *cnt_out,
                        float *sel_scores_out, void *ws, size_t ws_bytes, void *hip_stream)
{
    int rc = check_shape(shape);
    if (rc != HGCA_OK) return rc;
    if (shape->batch == 0) return HGCA_OK;
    if ((rc = check_view(shape, pool, false)) != HGCA_OK) return rc;
    if (!q || !aligned16(q) || !cnt_out || k_max < 0 || (k_max > 0 && !idx_out)) return HGCA_ERR_INVALID_ARG;
    if (!k_per_seq && (k_uniform < 0 || std::min(k_uniform, pool->cap) > k_max)) return HGCA_ERR_INVALID_ARG;
    const WsLayout w = layout(shape, 0, pool->cap);
    if (!ws || ws_bytes < w.total || !aligned16(ws)) return HGCA_ERR_WORKSPACE;
    hipStream_t s = static_cast<hipStream_t>(hip_stream);

    ScoreArgs sa{};
    sa.sh = to_dev(shape);
    sa.q = q;
    sa.kv = to_dev(pool);
    sa.scores = reinterpret_cast<float *>(static_cast<char *>(ws) + w.scores);
    sa.chunk = score_chunk(shape, pool->cap);
    sa.n_chunks = n_splits_for(pool->cap, sa.chunk);
    if ((rc = from_hip(launch_scores(shape->dtype, shape->head_dim, sa, s))) != HGCA_OK) return rc;

    SelectArgs se{};
    se.sh = sa.sh;
    se.kv = sa.kv;
    se.scores = sa.scores;
    se.k_per_seq = k_per_seq;
    se.k_uniform = k_uniform;
    se.k_max = k_max;
    se.idx = idx_out;
    se.cnt = cnt_out;
    se.sel_scores = sel_scores_out;
    return from_hip(launch_select(se, s));
}

int hgca_select_topk(const hgca_shape *shape, const float *scores, const int32_t *seq_lens, int32_t cap,
                     const int32_t *k_per_seq, int32_t k_uniform, int32_t k_max, int32_t *idx_out, int32_t *cnt_out,
                     float *sel_scores_out, void *hip_stream)
{
    int rc = check_shape(shape);
    if (rc != HGCA_OK) return rc;
    if (cap < 0 || k_max < 0) return HGCA_ERR_INVALID_ARG;
    if (!k_per_seq && (k_uniform < 0 || std::min(k_uniform, cap) > k_max)) return HGCA_ERR_INVALID_ARG;
    if (shape->batch == 0) return HGCA_OK;
    if (!cnt_out || (k_max > 0 && !idx_out) || (cap > 0 && (!scores || !aligned16(scores)))) return HGCA_ERR_INVALID_ARG;
    SelectArgs se{};
    se.sh = to_dev(shape);
    se.kv.seq_lens = seq_lens;
    se.kv.cap = cap;
    se.scores = scores;
    se.k_per_seq = k_per_seq;
    se.k_uniform = k_uniform;
    se.k_max = k_max;
    se.idx = idx_out;
    se.cnt = cnt_out;
    se.sel_scores = sel_scores_out;
    return from_hip(launch_select(se, static_cast<hipStream_t>(hip_stream)));
}

int hgca_sparse_attn(const hgca_shape *shape, const void *q, const hgca_kv_view *pool, const int32_t *idx,
                     const int32_t *cnt, int32_t k_max, const float *sel_scores, float *o_out, float *lse_out,
                     void *ws, size_t ws_bytes, void *hip_stream)
{
    int rc = check_shape(shape);
    if (rc != HGCA_OK) return rc;
    if (shape->batch == 0) return HGCA_OK;
    if ((rc = check_view(shape, pool, true)) != HGCA_OK) return rc;
    const bool deferred = !o_out && !lse_out;
    if (!q || !aligned16(q) || (!deferred && (!o_out || !lse_out || !aligned16(o_out)))) return HGCA_ERR_INVALID_ARG;
    if (k_max < 0 || !cnt || (k_max > 0 && !idx)) return HGCA_ERR_INVALID_ARG;
    const WsLayout w = layout(shape, k_max, 0);
    if (!ws || ws_bytes < w.total || !aligned16(ws)) return HGCA_ERR_WORKSPACE;
    hipStream_t s = static_cast<hipStream_t>(hip_stream);

    AttnArgs a{};
    a.sh = to_dev(shape);
    a.q = q;
    a.kv = to_dev(pool);
    a.idx = idx;
    a.cnt = cnt;
    a.sel_scores = sel_scores;
    a.k_max = k_max;
    a.chunk = pick_chunk(k_max, (int64_t)shape->batch * shape->n_q_heads, HGCA_TARGET_WGS_SPARSE);
    a.part = partials_at(ws, w, std::max(1, n_splits_for(k_max, a.chunk)));
    const int64_t rows = (int64_t)shape->batch * shape->n_q_heads;
    if ((rc = from_hip(launch_attn_partial_gather(shape->dtype, shape->head_dim, a, s))) != HGCA_OK) return rc;
    if (deferred) return HGCA_OK;
    return from_hip(launch_combine(shape->head_dim, rows, a.part, o_out, lse_out, s));
}

int hgca_select_salient_grouped(const hgca_shape *shape, const void *q, const hgca_kv_view *pool,
                                const int32_t *k_per_seq, int32_t k_uniform, int32_t k_max, int32_t *idx_out,
                                int32_t *cnt_out, void *ws, size_t ws_bytes, void *hip_stream)
{
    int rc = check_shape(shape);
    if (rc != HGCA_OK) return rc;
    if (shape->batch == 0) return HGCA_OK;
    if ((rc = check_view(shape, pool, false)) != HGCA_OK) return rc;
    if (!q || !aligned16(q) || !cnt_out || k_max < 0 || (k_max > 0 && !idx_out)) return HGCA_ERR_INVALID_ARG;
    if (!k_per_seq && (k_uniform < 0 || std::min(k_uniform, pool->cap) > k_max)) return HGCA_ERR_INVALID_ARG;
    const WsLayout w = layout(shape, 0, pool->cap);
    if (!ws || ws_bytes < w.total || !aligned16(ws)) return HGCA_ERR_WORKSPACE;
    hipStream_t s = static_cast<hipStream_t>(hip_stream);

    ScoreArgs sa{};
    sa.sh = to_dev(shape);
    sa.q = q;
    sa.kv = to_dev(pool);
    sa.scores = reinterpret_cast<float *>(static_cast<char *>(ws) + w.scores);    // [B, Hkv, cap] of the region
    sa.group_max = 1;
    sa.chunk = score_chunk(shape, pool->cap);
    sa.n_chunks = n_splits_for(pool->cap, sa.chunk);
    if ((rc = from_hip(launch_scores(shape->dtype, shape->head_dim, sa, s))) != HGCA_OK) return rc;

    SelectArgs se{};
    se.sh = sa.sh;
    se.sh.n_q_heads = shape->n_kv_heads;         // one row of scores and one list per KV head
    se.kv = sa.kv;
    se.scores = sa.scores;
    se.k_per_seq = k_per_seq;
    se.k_uniform = k_uniform;
    se.k_max = k_max;
    se.idx = idx_out;
    se.cnt = cnt_out;
    return from_hip(launch_select(se, s));
}

int hgca_union_lists(const hgca_shape *shape, const int32_t *idx, const int32_t *cnt, int32_t k_max,
                     int32_t n_positions, int32_t *idx_out, int32_t *cnt_out, int32_t k_max_out, int32_t *status,
                     void *hip_stream)
{
    int rc = check_shape(shape);
    if (rc != HGCA_OK) return rc;
    if (k_max < 0 || k_max_out < 0 || n_positions < 0) return HGCA_ERR_INVALID_ARG;
    // one bit per position in the 64 KiB of LDS a kernel may use without asking for more (64 bytes of it are static)
    if (n_positions > HGCA_UNION_MAX_POSITIONS) return HGCA_ERR_UNSUPPORTED;
    if (shape->batch == 0) return HGCA_OK;
    if (!cnt || !cnt_out || (k_max > 0 && !idx) || (k_max_out > 0 && !idx_out)) return HGCA_ERR_INVALID_ARG;
    return from_hip(launch_union_lists(idx, cnt, k_max, shape->batch, shape->n_q_heads, shape->n_kv_heads, n_positions,
                                       idx_out, cnt_out, k_max_out, status, static_cast<hipStream_t>(hip_stream)));
}

int hgca_sparse_attn_grouped(const hgca_shape *shape, const void *q, const hgca_kv_view *pool, const int32_t *idx,
                             const int32_t *cnt, int32_t k_max, float *o_out, float *lse_out, void *ws,
                             size_t ws_bytes, void *hip_stream)
{
    int rc = check_shape(shape);
    if (rc != HGCA_OK) return rc;
    if (shape->batch == 0) return HGCA_OK;
    if ((rc = check_view(shape, pool, true)) != HGCA_OK) return rc;
    const bool deferred = !o_out && !lse_out;
    if (!q || !aligned16(q) || (!deferred && (!o_out || !lse_out || !aligned16(o_out)))) return HGCA_ERR_INVALID_ARG;
    if (k_max < 0 || !cnt || (k_max > 0 && !idx)) return HGCA_ERR_INVALID_ARG;
    const WsLayout w = layout(shape, k_max, 0);
    if (!ws || ws_bytes < w.total || !aligned16(ws)) return HGCA_ERR_WORKSPACE;
    hipStream_t s = static_cast<hipStream_t>(hip_stream);

    AttnArgs a{};
    a.sh = to_dev(shape);
    a.q = q;
    a.kv = to_dev(pool);
    a.idx = idx;
    a.cnt = cnt;
    a.k_max = k_max;
    a.grouped = 1;
    // Deferred, the split size is hgca_sparse_attn's (hgca_lse_merge_splits derives the split count from k_max alone).
    // Folded here, there are a group's times fewer lists and workgroups, so the splits are that much shorter (64 lists
    // of 2 048 entries for groups of 4: 27.0 -> 22.6 us with 1024 workgroups; with 2048, two partials per 64 rows, 26.6),
    // but no shorter than 16 KB of K each (64 lists of 900 entries of dimension 64 in bf16: 13.1 us in splits of 128, 15.6
    // in splits of 64), and the bf16 kernel for groups of 8, whose workgroups write eight rows of partials each, gets half as
    // many (64 lists of 900 entries, dimension 64 / 128: 20.8 / 26.8 us with 512 workgroups, 34.5 / 34.6 with 960).
    // Without groups there are as many lists as heads, and nothing to shorten.
    const int group = group_of(shape), row_bytes = shape->head_dim * (shape->dtype == HGCA_BF16 ? 2 : 4);
    if (deferred || group == 1) {
        a.chunk = pick_chunk(k_max, (int64_t)shape->batch * shape->n_q_heads, HGCA_TARGET_WGS_SPARSE);
    } else {
        const int target = shape->dtype == HGCA_BF16 && group == 8 ? HGCA_TARGET_WGS_GROUPED / 2 : HGCA_TARGET_WGS_GROUPED;
        a.chunk = std::max(pick_chunk(k_max, (int64_t)shape->batch * shape->n_kv_heads, target), 16384 / row_bytes);
    }
    a.part = partials_at(ws, w, std::max(1, n_splits_for(k_max, a.chunk)));
    const int64_t rows = (int64_t)shape->batch * shape->n_q_heads;
    if ((rc = from_hip(launch_attn_partial_gather(shape->dtype, shape->head_dim, a, s))) != HGCA_OK) return rc;
    if (deferred) return HGCA_OK;
    return from_hip(launch_combine(shape->head_dim, rows, a.part, o_out, lse_out, s));
}

int hgca_lse_merge_splits(const hgca_shape *shape, int32_t window_cap, const void *ws_dense, size_t ws_dense_bytes,
                          int32_t k_max, const void *ws_sparse, size_t ws_sparse_bytes, void *o_out, int32_t o_dtype,
                          float *lse_out, void *hip_stream)
{
    int rc = check_shape(shape);
    if (rc != HGCA_OK) return rc;
    if (o_dtype != HGCA_F32 && o_dtype != HGCA_BF16) return HGCA_ERR_UNSUPPORTED;
    if (shape->batch == 0) return HGCA_OK;
    if (window_cap < 0 || k_max < 0 || !o_out || !aligned16(o_out)) return HGCA_ERR_INVALID_ARG;
    // the same layouts and split counts the two deferred calls used
    Partials pd{}, ps{};
    if (ws_dense) {
        const WsLayout w = layout(shape, window_cap, 0);
        if (ws_dense_bytes < w.total || !aligned16(ws_dense)) return HGCA_ERR_WORKSPACE;
        const int chunk = pick_chunk(window_cap, (int64_t)shape->batch * shape->n_kv_heads, HGCA_TARGET_WGS_DENSE);
        pd = partials_at(const_cast<void *>(ws_dense), w, n_splits_for(window_cap, chunk));
    }
    if (ws_sparse) {
        const WsLayout w = layout(shape, k_max, 0);
        if (ws_sparse_bytes < w.total || !aligned16(ws_sparse)) return HGCA_ERR_WORKSPACE;
        const int chunk = pick_chunk(k_max, (int64_t)shape->batch * shape->n_q_heads, HGCA_TARGET_WGS_SPARSE);
        ps = partials_at(const_cast<void *>(ws_sparse), w, std::max(1, n_splits_for(k_max, chunk)));
    }
    const int64_t rows = (int64_t)shape->batch * shape->n_q_heads;
    return from_hip(launch_combine2(shape->head_dim, rows, pd, ps, o_out, o_dtype, lse_out,
                                    static_cast<hipStream_t>(hip_stream)));
}

int hgca_hybrid_decode_step(const hgca_shape *shape, const void *q, const hgca_kv_view *window,
                            const hgca_kv_view *pool, const int32_t *k_per_seq, int32_t k_uniform, int32_t k_max,
                            int32_t *idx_out, int32_t *cnt_out, void *o_out, int32_t o_dtype, float *lse_out,
                            void *ws_dense, size_t ws_dense_bytes, void *ws_sparse, size_t ws_sparse_bytes,
                            void *hip_stream)
{
    int rc = check_shape(shape);
    if (rc != HGCA_OK) return rc;
    if (o_dtype != HGCA_F32 && o_dtype != HGCA_BF16) return HGCA_ERR_UNSUPPORTED;
    if (shape->batch == 0) return HGCA_OK;
    if ((rc = check_view(shape, window, true)) != HGCA_OK) return rc;
    if ((rc = check_view(shape, pool, true)) != HGCA_OK) return rc;
    if (!q || !aligned16(q) || !o_out || !aligned16(o_out) || !cnt_out || k_max < 0 || (k_max > 0 && !idx_out))
        return HGCA_ERR_INVALID_ARG;
    if (!k_per_seq && (k_uniform < 0 || std::min(k_uniform, pool->cap) > k_max)) return HGCA_ERR_INVALID_ARG;
    const WsLayout wd = layout(shape, window->cap, 0);
    const WsLayout wsp = layout(shape, k_max, pool->cap);
    if (!ws_dense || ws_dense_bytes < wd.total || !aligned16(ws_dense)) return HGCA_ERR_WORKSPACE;
    if (!ws_sparse || ws_sparse_bytes < wsp.total || !aligned16(ws_sparse)) return HGCA_ERR_WORKSPACE;
    if (ws_dense == ws_sparse) return HGCA_ERR_WORKSPACE;       // the two parts are live at the same time
    hipStream_t s = static_cast<hipStream_t>(hip_stream);

    ScoreArgs sa{};
    sa.sh = to_dev(shape);
    sa.q = q;
    sa.kv = to_dev(pool);
    sa.scores = reinterpret_cast<float *>(static_cast<char *>(ws_sparse) + wsp.scores);
    sa.chunk = score_chunk(shape, pool->cap);
    sa.n_chunks = n_splits_for(pool->cap, sa.chunk);

    AttnArgs da{};
    da.sh = sa.sh;
    da.q = q;
    da.kv = to_dev(window);
    float *sel = k_max > 0 && pool->cap > 0 ? reinterpret_cast<float *>(static_cast<char *>(ws_sparse) + wsp.sel) : nullptr;
    SelectArgs se{};
    se.sh = sa.sh;
    se.kv = sa.kv;
    se.scores = sa.scores;
    se.k_per_seq = k_per_seq;
    se.k_uniform = k_uniform;
    se.k_max = k_max;
    se.idx = idx_out;
    se.cnt = cnt_out;
    se.sel_scores = sel;
    if (short_step(shape->dtype == HGCA_F32, shape->head_dim, (int64_t)shape->batch * shape->n_kv_heads, group_of(shape), window->cap, pool->cap, k_max)) {
        // window splits as in the launch shared with the gather; in fp32, on the vector units, half as long (4 sequences, 64 / 8
        // heads, window 8192: 146 -> 117 us; bf16, 1 sequence, 32 / 8 heads, the other way round 24.6 : 27.0)
        da.chunk = dense_chunk(shape, window->cap, true);
        da.part = partials_at(ws_dense, wd, n_splits_for(window->cap, da.chunk));
        if ((rc = from_hip(launch_window_scores(shape->dtype, shape->head_dim, da, sa, s))) != HGCA_OK) return rc;
        return from_hip(launch_select_attend(shape->dtype, shape->head_dim, se, da.part, o_out, o_dtype, lse_out, s));
    }
    // The window's splits and the sparse part's splits are two streaming passes that need nothing from each other:
    // where the shapes allow they share one launch (after the selection), so the second needs no ramp-up of its own.
    const int gather_chunk = gather_split(shape, k_max, HGCA_TARGET_WGS_SPARSE_SCORED);
    const bool fuse_gather = shares_launch(shape, window->cap, pool->cap, k_max, gather_chunk, true, false);
    da.chunk = dense_chunk(shape, window->cap, fuse_gather);
    da.part = partials_at(ws_dense, wd, n_splits_for(window->cap, da.chunk));

    // 1. split kernels of the window part (unless they go with the sparse part's), score pass over the pool
    if (!fuse_gather && (rc = from_hip(launch_attn_partial_dense(shape->dtype, shape->head_dim, da, s))) != HGCA_OK)
        return rc;
    if ((rc = from_hip(launch_scores(shape->dtype, shape->head_dim, sa, s))) != HGCA_OK) return rc;
    // 2. per-head top-k; the kept entries' scores stay in the workspace for the sparse part
    if ((rc = from_hip(launch_select(se, s))) != HGCA_OK) return rc;
    // 3. sparse part on the given scores (V rows only)
    AttnArgs ga{};
    ga.sh = sa.sh;
    ga.q = q;
    ga.kv = sa.kv;
    ga.idx = idx_out;
    ga.cnt = cnt_out;
    ga.sel_scores = sel;
    ga.k_max = k_max;
    ga.chunk = gather_chunk;
    ga.part = partials_at(ws_sparse, wsp, std::max(1, n_splits_for(k_max, ga.chunk)));
    order_gather(ga, pool->cap, false);
    if (fuse_gather) rc = from_hip(launch_dense_gather(shape->dtype, shape->head_dim, da, ga, s));
    else rc = from_hip(launch_attn_partial_gather(shape->dtype, shape->head_dim, ga, s));
    if (rc != HGCA_OK) return rc;
    // 4. one fold of all split partials = merge_state over all of them
    const int64_t rows = (int64_t)shape->batch * shape->n_q_heads;
    return from_hip(launch_combine2(shape->head_dim, rows, da.part, ga.part, o_out, o_dtype, lse_out, s));
}

int hgca_hybrid_decode_step_selected(const hgca_shape *shape, const void *q, const hgca_kv_view *window,
                                     const hgca_kv_view *pool, const int32_t *idx, const int32_t *cnt, int32_t k_max,
                                     const float *sel_scores, void *o_out, int32_t o_dtype, float *lse_out,
                                     void *ws_dense, size_t ws_dense_bytes, void *ws_sparse, size_t ws_sparse_bytes,
                                     void *hip_stream)
{
    int rc = check_shape(shape);
    if (rc != HGCA_OK) return rc;
    if (o_dtype != HGCA_F32 && o_dtype != HGCA_BF16) return HGCA_ERR_UNSUPPORTED;
    if (shape->batch == 0) return HGCA_OK;
    if ((rc = check_view(shape, window, true)) != HGCA_OK) return rc;
    if ((rc = check_view(shape, pool, true)) != HGCA_OK) return rc;
    if (!q || !aligned16(q) || !o_out || !aligned16(o_out) || !cnt || k_max < 0 || (k_max > 0 && !idx))
        return HGCA_ERR_INVALID_ARG;
    const WsLayout wd = layout(shape, window->cap, 0);
    const WsLayout wsp = layout(shape, k_max, 0);
    if (!ws_dense || ws_dense_bytes < wd.total || !aligned16(ws_dense)) return HGCA_ERR_WORKSPACE;
    if (!ws_sparse || ws_sparse_bytes < wsp.total || !aligned16(ws_sparse)) return HGCA_ERR_WORKSPACE;
    if (ws_dense == ws_sparse) return HGCA_ERR_WORKSPACE;       // the two parts are live at the same time
    hipStream_t s = static_cast<hipStream_t>(hip_stream);

    AttnArgs da{};
    da.sh = to_dev(shape);
    da.q = q;
    da.kv = to_dev(window);
    const int gather_chunk = gather_split(shape, k_max, HGCA_TARGET_WGS_SPARSE);
    const bool scored = sel_scores != nullptr;
    const bool one_launch = shares_launch(shape, window->cap, pool->cap, k_max, gather_chunk, scored, false);
    da.chunk = dense_chunk(shape, window->cap, one_launch);
    da.part = partials_at(ws_dense, wd, n_splits_for(window->cap, da.chunk));
    AttnArgs ga{};
    ga.sh = da.sh;
    ga.q = q;
    ga.kv = to_dev(pool);
    ga.idx = idx;
    ga.cnt = cnt;
    ga.sel_scores = sel_scores;
    ga.k_max = k_max;
    ga.chunk = gather_chunk;
    ga.part = partials_at(ws_sparse, wsp, std::max(1, n_splits_for(k_max, ga.chunk)));
    order_gather(ga, pool->cap, false);
    // gpu_attention over the window and cpu_attention over the listed entries: one launch where the shapes allow
    if (one_launch) {
        if ((rc = from_hip(launch_dense_gather(shape->dtype, shape->head_dim, da, ga, s))) != HGCA_OK) return rc;
    } else {
        if ((rc = from_hip(launch_attn_partial_dense(shape->dtype, shape->head_dim, da, s))) != HGCA_OK) return rc;
        if ((rc = from_hip(launch_attn_partial_gather(shape->dtype, shape->head_dim, ga, s))) != HGCA_OK) return rc;
    }
    // merge_state over all split partials of both parts
    const int64_t rows = (int64_t)shape->batch * shape->n_q_heads;
    return from_hip(launch_combine2(shape->head_dim, rows, da.part, ga.part, o_out, o_dtype, lse_out, s));
}

int hgca_lse_merge(const hgca_shape *shape, const float *o_a, const float *lse_a, const float *o_b,
                   const float *lse_b, void *o_out, int32_t o_dtype, float *lse_out, void *hip_stream)
{
    if (!shape || shape->batch < 0 || shape->n_q_heads <= 0) return HGCA_ERR_INVALID_ARG;
    if (shape->head_dim != 64 && shape->head_dim != 128) return HGCA_ERR_UNSUPPORTED;
    if (o_dtype != HGCA_F32 && o_dtype != HGCA_BF16) return HGCA_ERR_UNSUPPORTED;
    if (shape->batch == 0) return HGCA_OK;
    if (!o_a || !lse_a || !o_b || !lse_b || !o_out) return HGCA_ERR_INVALID_ARG;
    if (o_dtype == HGCA_BF16 && (o_out == (const void *)o_a || o_out == (const void *)o_b))
        return HGCA_ERR_INVALID_ARG;             // a bf16 result cannot overwrite an fp32 input in place
    const int64_t rows = (int64_t)shape->batch * shape->n_q_heads;
    return from_hip(launch_merge(shape->head_dim, rows, o_a, lse_a, o_b, lse_b, o_out, o_dtype, lse_out,
                                 static_cast<hipStream_t>(hip_stream)));
}

namespace {

int check_cache(const hgca_shape *shape, const hgca_cache_state *c, CacheDev *out)
{
    int rc = check_shape(shape);
    if (rc != HGCA_OK) return rc;
    if (!c) return HGCA_ERR_INVALID_ARG;
    if (c->block_size <= 0 || c->max_blocks <= 0 || c->win_blocks <= 0 || c->win_blocks > c->max_blocks || c->k_max < 0 ||
        c->pool_cap < 0)
        return HGCA_ERR_INVALID_ARG;
    if (c->block_size % 16 != 0) return HGCA_ERR_UNSUPPORTED;
    if (c->win_cap_blocks != 0 && (c->win_cap_blocks < c->win_blocks || c->win_cap_blocks > c->max_blocks))
        return HGCA_ERR_INVALID_ARG;
    if (shape->batch > 0 &&
        (!c->k_blocks || !c->v_blocks || !aligned16(c->k_blocks) || !aligned16(c->v_blocks) || !c->block_table ||
         !c->first_win_block || !c->win_lens || !c->pool_lens || !c->a_maw || !c->ctx_cnt || !c->plan || !c->status ||
         (c->k_max > 0 && !c->ctx_idx)))
        return HGCA_ERR_INVALID_ARG;
    out->k_blocks = static_cast<char *>(c->k_blocks);
    out->v_blocks = static_cast<char *>(c->v_blocks);
    out->block_table = c->block_table;
    out->first_win_block = c->first_win_block;
    out->win_lens = c->win_lens;
    out->pool_lens = c->pool_lens;
    out->a_maw = c->a_maw;
    out->ctx_idx = c->ctx_idx;
    out->ctx_cnt = c->ctx_cnt;
    out->plan = c->plan;
    out->status = c->status;
    out->a_evicted = c->a_evicted;
    out->block_size = c->block_size;
    out->max_blocks = c->max_blocks;
    out->win_blocks = c->win_blocks;
    out->k_max = c->k_max;
    out->pool_cap = c->pool_cap;
    out->win_cap = (c->win_cap_blocks ? c->win_cap_blocks : c->win_blocks) * c->block_size;
    return HGCA_OK;
}

}  // namespace

int hgca_kv_append_tokens(const hgca_shape *shape, const hgca_cache_state *cache, const void *k_in, const void *v_in,
                          int32_t n_tokens, const int32_t *active, void *hip_stream)
{
    CacheDev c{};
    int rc = check_cache(shape, cache, &c);
    if (rc != HGCA_OK) return rc;
    if (n_tokens < 0) return HGCA_ERR_INVALID_ARG;
    if (shape->batch == 0 || n_tokens == 0) return HGCA_OK;
    if (!k_in || !v_in || !aligned16(k_in) || !aligned16(v_in)) return HGCA_ERR_INVALID_ARG;
    const int32_t row_bytes = shape->head_dim * (shape->dtype == HGCA_BF16 ? 2 : 4);
    return from_hip(launch_kv_append(c, k_in, v_in, active, shape->batch, shape->n_kv_heads, row_bytes, n_tokens,
                                     static_cast<hipStream_t>(hip_stream)));
}

int hgca_kv_append(const hgca_shape *shape, const hgca_cache_state *cache, const void *k_in, const void *v_in,
                   const int32_t *active, void *hip_stream)
{
    return hgca_kv_append_tokens(shape, cache, k_in, v_in, 1, active, hip_stream);
}

int hgca_kv_evict(const hgca_shape *shape, const hgca_cache_state *cache, double beta, void *hip_stream)
{
    CacheDev c{};
    int rc = check_cache(shape, cache, &c);
    if (rc != HGCA_OK) return rc;
    if (!(beta >= 0.0)) return HGCA_ERR_INVALID_ARG;
    if (shape->batch == 0) return HGCA_OK;
    return from_hip(launch_kv_evict(c, shape->batch, shape->n_q_heads, beta, static_cast<hipStream_t>(hip_stream)));
}

int hgca_managed_decode_step(const hgca_shape *shape, const hgca_cache_state *cache, const void *q, const void *k_in,
                             const void *v_in, float alpha, double beta, float *a_gpu,
                             void *o_out, int32_t o_dtype, float *lse_out, void *ws_dense, size_t ws_dense_bytes,
                             void *ws_sparse, size_t ws_sparse_bytes, void *hip_stream)
{
    CacheDev c{};
    int rc = check_cache(shape, cache, &c);
    if (rc != HGCA_OK) return rc;
    if (o_dtype != HGCA_F32 && o_dtype != HGCA_BF16) return HGCA_ERR_UNSUPPORTED;
    if (!(alpha >= 0.f && alpha <= 1.f) || !(beta >= 0.0)) return HGCA_ERR_INVALID_ARG;
    if (shape->batch == 0) return HGCA_OK;
    if (!q || !aligned16(q) || !k_in || !v_in || !aligned16(k_in) || !aligned16(v_in) || !a_gpu || !o_out ||
        !aligned16(o_out))
        return HGCA_ERR_INVALID_ARG;
    // the two tiers as ranges of the sequence's block list
    hgca_kv_view window{}, pool{};
    window.k = pool.k = cache->k_blocks;
    window.v = pool.v = cache->v_blocks;
    window.block_table = pool.block_table = cache->block_table;
    window.block_size = pool.block_size = cache->block_size;
    window.max_blocks = pool.max_blocks = cache->max_blocks;
    window.seq_lens = cache->win_lens;
    window.first_block = cache->first_win_block;
    window.cap = c.win_cap;
    pool.seq_lens = cache->pool_lens;
    pool.cap = cache->pool_cap;
    if ((rc = check_view(shape, &window, true)) != HGCA_OK) return rc;
    if ((rc = check_view(shape, &pool, true)) != HGCA_OK) return rc;
    const WsLayout wd = layout(shape, window.cap, 0);
    const WsLayout wsp = layout(shape, cache->k_max, 0);
    if (!ws_dense || ws_dense_bytes < wd.total || !aligned16(ws_dense)) return HGCA_ERR_WORKSPACE;
    if (!ws_sparse || ws_sparse_bytes < wsp.total || !aligned16(ws_sparse) || ws_sparse == ws_dense) return HGCA_ERR_WORKSPACE;
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    const int64_t rows = (int64_t)shape->batch * shape->n_q_heads;
    const int32_t row_bytes = shape->head_dim * (shape->dtype == HGCA_BF16 ? 2 : 4);

    const bool token_may_join = HGCA_FUSE_KV_APPEND && HGCA_FUSE_DECODE_TAIL;
    const int gather_chunk = gather_split(shape, cache->k_max, HGCA_TARGET_WGS_SPARSE);
    const bool one_launch = shares_launch(shape, window.cap, cache->pool_cap, cache->k_max, gather_chunk, false, token_may_join);
    // Alg. 2: KV_gpu' = concat(KV_gpu, KV_in): a launch of its own, or (token_joins_in_split) the window split that
    // owns the token's position writes its rows and the step's last launch stores the new length
    const bool token_joins_in_split = token_may_join && one_launch;
    if (!token_joins_in_split &&
        (rc = from_hip(launch_kv_append(c, k_in, v_in, nullptr, shape->batch, shape->n_kv_heads, row_bytes, 1, s))) != HGCA_OK)
        return rc;
    // gpu_attention: split kernels of the window, leaving the scaled scores in a_gpu
    AttnArgs da{};
    da.sh = to_dev(shape);
    da.q = q;
    da.kv = to_dev(&window);
    da.chunk = dense_chunk(shape, window.cap, one_launch);
    da.part = partials_at(ws_dense, wd, n_splits_for(window.cap, da.chunk));
    da.raw_scores = a_gpu;
    // cpu_attention over KV_ctx: split kernels over each head's list of salient pool positions
    AttnArgs ga{};
    ga.sh = da.sh;
    ga.q = q;
    ga.kv = to_dev(&pool);
    ga.idx = cache->ctx_idx;
    ga.cnt = cache->ctx_cnt;
    ga.k_max = cache->k_max;
    ga.chunk = gather_chunk;
    ga.part = partials_at(ws_sparse, wsp, std::max(1, n_splits_for(cache->k_max, ga.chunk)));
    order_gather(ga, std::min<int64_t>(pool.cap, (int64_t)(cache->max_blocks - cache->win_blocks) * cache->block_size), true);
    // the two parts need nothing from each other: one launch where the shapes allow
    if (one_launch) {
        if ((rc = from_hip(launch_dense_gather(shape->dtype, shape->head_dim, da, ga, s, token_joins_in_split ? k_in : nullptr,
                                               token_joins_in_split ? v_in : nullptr))) != HGCA_OK)
            return rc;
    } else {
        if ((rc = from_hip(launch_attn_partial_dense(shape->dtype, shape->head_dim, da, s))) != HGCA_OK) return rc;
        if ((rc = from_hip(launch_attn_partial_gather(shape->dtype, shape->head_dim, ga, s))) != HGCA_OK) return rc;
    }
    // merge_state over all split partials; A_gpu = e^{s - lse_g} with the window's own lse from the same fold;
    // Alg. 1: A_maw <- (1 - alpha) A_maw + alpha A_gpu (the inserted token has no history); eviction and
    // sparsification where a window is full.  All three are per (sequence, head) row: one launch.
    if (HGCA_FUSE_DECODE_TAIL)
        return from_hip(launch_decode_tail(shape->head_dim, rows, da.part, ga.part, o_out, o_dtype, lse_out, a_gpu, c,
                                           shape->n_q_heads, alpha, beta, token_joins_in_split ? 1 : 0, s));
    float *lse_w = reinterpret_cast<float *>(static_cast<char *>(ws_dense) + wd.row_aux);
    if ((rc = from_hip(launch_combine2(shape->head_dim, rows, da.part, ga.part, o_out, o_dtype, lse_out, s, lse_w))) != HGCA_OK)
        return rc;
    if ((rc = from_hip(launch_window_weights(a_gpu, lse_w, window.seq_lens, rows, shape->n_q_heads, window.cap, c.a_maw, 1,
                                             alpha, s))) != HGCA_OK)
        return rc;
    return from_hip(launch_kv_evict(c, shape->batch, shape->n_q_heads, beta, s));
}

int hgca_ctx_compact(const hgca_shape *shape, const hgca_kv_view *pool, const int32_t *idx, const int32_t *cnt,
                     int32_t k_max, const int32_t *first_row, void *k_ctx, void *v_ctx, int32_t ctx_cap,
                     int32_t *cnt_out, void *hip_stream)
{
    int rc = check_shape(shape);
    if (rc != HGCA_OK) return rc;
    if (k_max < 0 || ctx_cap < 0) return HGCA_ERR_INVALID_ARG;
    if (shape->batch == 0) return HGCA_OK;
    if ((rc = check_view(shape, pool, true)) != HGCA_OK) return rc;
    if (!cnt || (k_max > 0 && !idx)) return HGCA_ERR_INVALID_ARG;
    if (ctx_cap > 0 && (!k_ctx || !v_ctx || !aligned16(k_ctx) || !aligned16(v_ctx) || k_ctx == v_ctx))
        return HGCA_ERR_INVALID_ARG;
    if (cnt_out && (cnt_out == first_row || cnt_out == cnt)) return HGCA_ERR_INVALID_ARG;   // read by other workgroups
    CtxCompactArgs a{};
    a.sh = to_dev(shape);
    a.kv = to_dev(pool);
    a.idx = idx;
    a.cnt = cnt;
    a.first_row = first_row;
    a.cnt_out = cnt_out;
    a.k_ctx = static_cast<char *>(k_ctx);
    a.v_ctx = static_cast<char *>(v_ctx);
    a.k_max = k_max;
    a.ctx_cap = ctx_cap;
    a.row_bytes = shape->head_dim * (shape->dtype == HGCA_BF16 ? 2 : 4);
    return from_hip(launch_ctx_compact(a, static_cast<hipStream_t>(hip_stream)));
}

namespace {

// Blocks of up to 128 query rows over all (sequence, KV head) pairs: each is attended to by its own workgroups.
int64_t append_units(const hgca_shape *s, int32_t n_q)
{
    const int64_t n_qb = ((int64_t)n_q * group_of(s) + 127) / 128;
    return std::max<int64_t>(1, (int64_t)s->batch * s->n_kv_heads * n_qb);
}

int64_t line_steps(int64_t tokens) { return std::max<int64_t>(1, (tokens + kLineStep - 1) / kLineStep); }

int append_want_splits(const hgca_shape *s, int32_t n_q)
{
    return (int)std::max<int64_t>(1, HGCA_APPEND_TARGET_WGS / append_units(s, n_q));
}

// Shares of the attention.  In bf16 a compute unit holds two workgroups: a 64-token step of both takes 2.8 us, of one alone
// 1.6, so two long shares are better than one of twice the length, but short ones pay for their start, 3 us, and for
// their partial, which is written and read again by the fold (64 KB for 128 rows of 128 columns, 5 TB/s).  Times in 0.1 us;
// only the smallest number of shares of each length in steps is looked at.  64 queries x 4 heads over 8 K tokens: 31.3 us
// with 16 shares per unit (one workgroup per compute unit), 34.9 with 32; 55 queries over 5.6 K tokens 15.8 with 32, 18.6
// with 45; 8 x 32 queries x 4 heads over 32 K tokens 260 with 8 (two workgroups per compute unit), 282 with 4.
// (With the weights rounded to bf16, fewer shares also mean fewer weights that are exactly 1: 55 queries over 5.6 K tokens 6.7e-4
// off with 30 shares, 6.3e-4 with 45.)
// In fp32 a compute unit holds one workgroup; what a share costs beside its steps counts as one of them (counted as two or three, 1092
// sizes are 0.7 and 1.0 % faster on average, single ones 14 % faster to 16 % slower).
int append_shares(const hgca_shape *s, int32_t n_q, int64_t tokens, int most)
{
    const int64_t units = append_units(s, n_q);
    if (s->dtype == HGCA_F32) return line_shares(units, line_steps(tokens), most, HGCA_APPEND_TARGET_WGS / 2, 1);
    constexpr int64_t kUnits = HGCA_APPEND_TARGET_WGS / 2, kStepOfTwo = 28, kStepAlone = 16, kStart = 30;
    const int64_t steps = line_steps(tokens);
    const int64_t partial = std::min<int64_t>(128, (int64_t)n_q * group_of(s)) * s->head_dim * 8;        // bytes, written and read
    int64_t best = 1, best_cost = INT64_MAX;
    for (int64_t n = 1; n <= most && n <= steps;) {
        const int64_t len = (steps + n - 1) / n, load = (n * units + kUnits - 1) / kUnits;
        const int64_t cost = load / 2 * (len * kStepOfTwo + kStart) + load % 2 * (len * kStepAlone + kStart) +
                             n * units * partial / 500000;
        if (cost < best_cost) {
            best_cost = cost;
            best = n;
        }
        if (len == 1) break;
        n = (steps + len - 2) / (len - 1);       // the smallest number whose shares are shorter
    }
    return (int)best;
}

struct AppendWs {
    size_t o, m, l, total;
    int max_splits;
};

AppendWs append_layout(const hgca_shape *s, int32_t n_q, int64_t max_tokens)
{
    AppendWs w{};
    // shares of up to kMaxAppendChunk tokens; fp32 may run on the one-query kernels, whose splits hold kMaxChunk
    w.max_splits = std::max(append_want_splits(s, n_q), n_splits_for(std::max<int64_t>(max_tokens, 1),
                                                                     s->dtype == HGCA_F32 ? kMaxChunk : kMaxAppendChunk));
    const size_t rows = (size_t)s->batch * n_q * s->n_q_heads;
    size_t at = 0;
    w.o = at; at += align_up(rows * w.max_splits * s->head_dim * sizeof(float));
    w.m = at; at += align_up(rows * w.max_splits * sizeof(float));
    w.l = at; at += align_up(rows * w.max_splits * sizeof(float));
    w.total = std::max<size_t>(at, kAlign);
    return w;
}

int check_append(const hgca_shape *shape, const void *q, int32_t n_q, const hgca_kv_view *tier, bool need_v)
{
    int rc = check_shape(shape);
    if (rc != HGCA_OK) return rc;
    if (n_q < 0 || n_q > 4096) return HGCA_ERR_INVALID_ARG;
    // the kernels keep the running maximum on the raw scores and apply the scale inside the exponent
    if (!(shape->sm_scale > 0.f) || !(shape->sm_scale < 3.0e38f)) return HGCA_ERR_INVALID_ARG;
    if ((rc = check_view(shape, tier, need_v)) != HGCA_OK) return rc;
    if (shape->batch > 0 && n_q > 0 && (!q || !aligned16(q))) return HGCA_ERR_INVALID_ARG;
    return HGCA_OK;
}

}  // namespace

size_t hgca_append_workspace_bytes(const hgca_shape *shape, int32_t n_q, int32_t max_tokens)
{
    if (check_shape(shape) != HGCA_OK || n_q < 0 || max_tokens < 0) return 0;
    return append_layout(shape, n_q, max_tokens).total;
}

int hgca_append_attn(const hgca_shape *shape, const void *q, int32_t n_q, const hgca_kv_view *tier,
                     int32_t flags, float *o_out, float *lse_out, void *ws, size_t ws_bytes, void *hip_stream)
{
    int rc = check_append(shape, q, n_q, tier, true);
    if (rc != HGCA_OK) return rc;
    if (flags & ~(HGCA_APPEND_CAUSAL_TAIL | HGCA_APPEND_ONE_PART_P)) return HGCA_ERR_INVALID_ARG;
    if (shape->batch == 0 || n_q == 0) return HGCA_OK;
    if (!o_out || !lse_out || !aligned16(o_out)) return HGCA_ERR_INVALID_ARG;
    // a limit of the interface (once the grid dimension of the (KV head, block of 128 query rows) pairs)
    if ((int64_t)shape->n_kv_heads * (((int64_t)n_q * group_of(shape) + 127) / 128) > 65535) return HGCA_ERR_UNSUPPORTED;
    const AppendWs w = append_layout(shape, n_q, tier->cap);
    if (!ws || ws_bytes < w.total || !aligned16(ws)) return HGCA_ERR_WORKSPACE;
    hipStream_t s = static_cast<hipStream_t>(hip_stream);

    if (shape->dtype == HGCA_F32) {
        // batch * n_q sequences of one query each, as one of the two routes has it, are a grid dimension
        if ((int64_t)shape->batch * n_q > 65535) return HGCA_ERR_UNSUPPORTED;
        // splits no shorter than the workspace has slots for
        const int chunk = std::max(pick_chunk(tier->cap, (int64_t)shape->batch * n_q * shape->n_kv_heads, HGCA_TARGET_WGS_DENSE),
                                   (n_splits_for(tier->cap, w.max_splits) + 63) / 64 * 64);
        const int n_splits = n_splits_for(tier->cap, chunk);
        const int64_t turns = line_turns(append_units(shape, n_q), line_steps(tier->cap),
                                         append_shares(shape, n_q, tier->cap, w.max_splits), HGCA_APPEND_TARGET_WGS / 2);
        if (tier->cap > 0 && query_by_query(shape->head_dim, shape->batch, shape->n_kv_heads, group_of(shape), n_q, tier->cap, n_splits, turns)) {
            if (chunk > kMaxChunk || n_splits > w.max_splits) return HGCA_ERR_WORKSPACE;
            AttnArgs d{};
            d.sh = to_dev(shape);
            d.sh.batch = shape->batch * n_q;
            d.q = q;
            d.kv = to_dev(tier);
            d.kv.n_q = n_q;
            d.kv.causal_tail = (flags & HGCA_APPEND_CAUSAL_TAIL) ? 1 : 0;
            d.chunk = chunk;
            char *base = static_cast<char *>(ws);
            d.part = Partials{reinterpret_cast<float *>(base + w.o), reinterpret_cast<float *>(base + w.m),
                              reinterpret_cast<float *>(base + w.l), n_splits, n_splits};
            const int64_t rows = (int64_t)d.sh.batch * shape->n_q_heads;
            if ((rc = from_hip(launch_attn_partial_dense(shape->dtype, shape->head_dim, d, s))) != HGCA_OK) return rc;
            return from_hip(launch_combine(shape->head_dim, rows, d.part, o_out, lse_out, s));
        }
    }
    AppendArgs a{};
    a.sh = to_dev(shape);
    a.q = q;
    a.kv = to_dev(tier);
    a.n_q = n_q;
    a.causal_tail = (flags & HGCA_APPEND_CAUSAL_TAIL) ? 1 : 0;
    a.one_part_p = (flags & HGCA_APPEND_ONE_PART_P) ? 1 : 0;
    const LineDev line{tier->seq_lens, nullptr, tier->cap, 0, append_shares(shape, n_q, tier->cap, w.max_splits), 0};
    char *base = static_cast<char *>(ws);
    a.part = Partials{reinterpret_cast<float *>(base + w.o), reinterpret_cast<float *>(base + w.m),
                      reinterpret_cast<float *>(base + w.l), line.shares, line.shares};
    if ((rc = from_hip(launch_append_attn(shape->dtype, shape->head_dim, a, nullptr, line, false, s))) != HGCA_OK) return rc;
    const int64_t rows = (int64_t)shape->batch * n_q * shape->n_q_heads;
    return from_hip(launch_combine(shape->head_dim, rows, a.part, o_out, lse_out, s));
}

namespace {

// Workspace of the two-tier append attention: the partials of the line of pool and window (one slot more than there
// are shares), and the two per-tier lse rows for callers that do not ask for them.
struct TiersWs {
    size_t o, m, l, lse_w, lse_p, total;
    int shares;
};

// reusable: the size the queries return, which also serves tiers of smaller capacities (these may be cut into more shares).
TiersWs tiers_layout(const hgca_shape *s, int32_t n_q, int64_t win_cap, int64_t pool_cap, bool reusable = false)
{
    TiersWs w{};
    const int64_t tokens = (win_cap + kLineStep - 1) / kLineStep * kLineStep + (pool_cap + kLineStep - 1) / kLineStep * kLineStep;
    const int most = std::max(append_want_splits(s, n_q), n_splits_for(std::max<int64_t>(tokens, 1), kMaxAppendChunk));
    w.shares = append_shares(s, n_q, tokens, most);
    const int64_t most_of_any = std::min<int64_t>(most, std::max<int64_t>(1, tokens / kLineStep));
    const size_t rows = (size_t)s->batch * n_q * s->n_q_heads, slots = (reusable ? most_of_any : w.shares) + 1;
    size_t at = 0;
    w.o = at; at += align_up(rows * slots * s->head_dim * sizeof(float));
    w.m = at; at += align_up(rows * slots * sizeof(float));
    w.l = at; at += align_up(rows * slots * sizeof(float));
    w.lse_w = at; at += align_up(rows * sizeof(float));
    w.lse_p = at; at += align_up(rows * sizeof(float));
    w.total = std::max<size_t>(at, kAlign);
    return w;
}

}  // namespace

size_t hgca_append_tiers_workspace_bytes(const hgca_shape *shape, int32_t n_q, int32_t window_cap, int32_t pool_cap)
{
    if (check_shape(shape) != HGCA_OK || n_q < 0 || window_cap < 0 || pool_cap < 0) return 0;
    return tiers_layout(shape, n_q, window_cap, pool_cap, true).total;
}

namespace {

// Both tiers of an append turn, either type (the exported call takes bf16 only; a turn over the managed cache both).
int append_attn_tiers(const hgca_shape *shape, const void *q, int32_t n_q, const hgca_kv_view *window,
                           const hgca_kv_view *pool, int32_t flags, float *o_out, float *lse_out, float *lse_window_out,
                           float *lse_pool_out, bool weights_follow, void *ws, size_t ws_bytes, void *hip_stream)
{
    int rc = check_append(shape, q, n_q, window, true);
    if (rc != HGCA_OK) return rc;
    if ((rc = check_append(shape, q, n_q, pool, true)) != HGCA_OK) return rc;
    if (flags & ~(HGCA_APPEND_CAUSAL_TAIL | HGCA_APPEND_ONE_PART_P)) return HGCA_ERR_INVALID_ARG;
    if (shape->batch == 0 || n_q == 0) return HGCA_OK;
    if (!o_out || !lse_out || !aligned16(o_out)) return HGCA_ERR_INVALID_ARG;
    if ((int64_t)shape->n_kv_heads * (((int64_t)n_q * group_of(shape) + 127) / 128) > 65535) return HGCA_ERR_UNSUPPORTED;
    const TiersWs w = tiers_layout(shape, n_q, window->cap, pool->cap);
    if (!ws || ws_bytes < w.total || !aligned16(ws)) return HGCA_ERR_WORKSPACE;
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    char *base = static_cast<char *>(ws);

    AppendArgs aw{}, ap{};
    aw.sh = ap.sh = to_dev(shape);
    aw.q = ap.q = q;
    aw.n_q = ap.n_q = n_q;
    aw.one_part_p = ap.one_part_p = (flags & HGCA_APPEND_ONE_PART_P) ? 1 : 0;
    aw.kv = to_dev(window);
    aw.causal_tail = (flags & HGCA_APPEND_CAUSAL_TAIL) ? 1 : 0;
    ap.kv = to_dev(pool);
    ap.causal_tail = 0;
    aw.part = ap.part = Partials{reinterpret_cast<float *>(base + w.o), reinterpret_cast<float *>(base + w.m),
                                 reinterpret_cast<float *>(base + w.l), w.shares + 1, w.shares + 1};
    const LineDev line{pool->seq_lens, window->seq_lens, pool->cap, window->cap, w.shares, n_q * shape->n_q_heads};
    if ((rc = from_hip(launch_append_attn(shape->dtype, shape->head_dim, ap, &aw, line, weights_follow, s))) != HGCA_OK) return rc;
    // merge_state over the partials of both tiers at once; each tier's own lse comes out of the same fold
    const int64_t rows = (int64_t)shape->batch * n_q * shape->n_q_heads;
    float *lse_w = lse_window_out ? lse_window_out : reinterpret_cast<float *>(base + w.lse_w);
    float *lse_p = lse_pool_out ? lse_pool_out : reinterpret_cast<float *>(base + w.lse_p);
    const bool want_tiers = lse_window_out || lse_pool_out;
    return from_hip(launch_combine_line(shape->head_dim, rows, ap.part, line, o_out, lse_out, want_tiers ? lse_p : nullptr,
                                        want_tiers ? lse_w : nullptr, s));
}

}  // namespace

int hgca_append_attn_tiers(const hgca_shape *shape, const void *q, int32_t n_q, const hgca_kv_view *window,
                           const hgca_kv_view *pool, int32_t flags, float *o_out, float *lse_out, float *lse_window_out,
                           float *lse_pool_out, void *ws, size_t ws_bytes, void *hip_stream)
{
    int rc = check_append(shape, q, n_q, window, true);
    if (rc != HGCA_OK) return rc;
    if ((rc = check_append(shape, q, n_q, pool, true)) != HGCA_OK) return rc;
    if (flags & ~(HGCA_APPEND_CAUSAL_TAIL | HGCA_APPEND_ONE_PART_P)) return HGCA_ERR_INVALID_ARG;
    if (shape->dtype != HGCA_BF16) return HGCA_ERR_UNSUPPORTED;      // fp32 inputs: one call per tier and hgca_lse_merge
    return append_attn_tiers(shape, q, n_q, window, pool, flags, o_out, lse_out, lse_window_out, lse_pool_out, false, ws, ws_bytes,
                             hip_stream);
}

namespace {

// Arguments of the weights pass over one tier.
AppendArgs weights_args(const hgca_shape *shape, const void *q, int32_t n_q, const hgca_kv_view *tier, int32_t causal_tail,
                        const float *lse, float *a_out)
{
    AppendArgs a{};
    a.sh = to_dev(shape);
    a.q = q;
    a.kv = to_dev(tier);
    a.n_q = n_q;
    a.causal_tail = causal_tail ? 1 : 0;
    a.lse = lse;
    a.a_out = a_out;
    return a;
}

// Workgroups per (sequence, KV head) of the weights pass: one per compute unit, each meets all query rows.
// (What a share costs beside its steps, fp32, counted as two or four of them instead of one: 179 sizes 0.3 and 0.5 % faster on average.)
int weights_shares(const hgca_shape *s, int64_t tokens)
{
    constexpr int kPlaces = 256;
    return line_shares((int64_t)s->batch * s->n_kv_heads, line_steps(tokens), kPlaces, kPlaces, s->dtype == HGCA_F32 ? 1 : 5);
}

}  // namespace

namespace {

int append_weights_tiers(const hgca_shape *shape, const void *q, int32_t n_q, const hgca_kv_view *window,
                              const hgca_kv_view *pool, int32_t causal_tail, const float *lse_window, const float *lse_pool,
                              float *a_gpu, float *a_cpu, bool after_attention, void *hip_stream)
{
    int rc = check_append(shape, q, n_q, window, false);
    if (rc != HGCA_OK) return rc;
    if ((rc = check_append(shape, q, n_q, pool, false)) != HGCA_OK) return rc;
    if (n_q == 0) return HGCA_ERR_INVALID_ARG;       // an average over no query is undefined
    if (shape->batch == 0) return HGCA_OK;
    if ((window->cap > 0 && (!lse_window || !a_gpu)) || (pool->cap > 0 && (!lse_pool || !a_cpu))) return HGCA_ERR_INVALID_ARG;
    const AppendArgs aw = weights_args(shape, q, n_q, window, causal_tail, lse_window, a_gpu);
    const AppendArgs ap = weights_args(shape, q, n_q, pool, 0, lse_pool, a_cpu);
    const LineDev line{pool->seq_lens, window->seq_lens, pool->cap, window->cap,
                       weights_shares(shape, (int64_t)pool->cap + window->cap), 0};
    return from_hip(launch_append_weights(shape->dtype, shape->head_dim, ap, &aw, line, after_attention,
                                          static_cast<hipStream_t>(hip_stream)));
}

}  // namespace

int hgca_append_weights_tiers(const hgca_shape *shape, const void *q, int32_t n_q, const hgca_kv_view *window,
                              const hgca_kv_view *pool, int32_t causal_tail, const float *lse_window, const float *lse_pool,
                              float *a_gpu, float *a_cpu, void *hip_stream)
{
    int rc = check_append(shape, q, n_q, window, false);
    if (rc != HGCA_OK) return rc;
    if ((rc = check_append(shape, q, n_q, pool, false)) != HGCA_OK) return rc;
    if (n_q == 0) return HGCA_ERR_INVALID_ARG;       // an average over no query is undefined
    if (shape->dtype != HGCA_BF16) return HGCA_ERR_UNSUPPORTED;      // fp32 inputs: one call per tier
    return append_weights_tiers(shape, q, n_q, window, pool, causal_tail, lse_window, lse_pool, a_gpu, a_cpu, false, hip_stream);
}

int hgca_append_weights(const hgca_shape *shape, const void *q, int32_t n_q, const hgca_kv_view *tier,
                        int32_t causal_tail, const float *lse, float *a_out, void *hip_stream)
{
    int rc = check_append(shape, q, n_q, tier, false);
    if (rc != HGCA_OK) return rc;
    if (n_q == 0) return HGCA_ERR_INVALID_ARG;       // an average over no query is undefined
    if (shape->batch == 0 || tier->cap == 0) return HGCA_OK;
    if (!lse || !a_out) return HGCA_ERR_INVALID_ARG;
    const AppendArgs a = weights_args(shape, q, n_q, tier, causal_tail, lse, a_out);
    const LineDev line{tier->seq_lens, nullptr, tier->cap, 0, weights_shares(shape, tier->cap), 0};
    return from_hip(launch_append_weights(shape->dtype, shape->head_dim, a, nullptr, line, false, static_cast<hipStream_t>(hip_stream)));
}

namespace {

// Workspace of hgca_managed_append_step: [scratch of the two-tier attention | lse of the window part | lse of the pool part]
struct ManagedAppendWs {
    size_t attn, lse_w, lse_p, total;
    size_t attn_bytes;
};

ManagedAppendWs managed_append_layout(const hgca_shape *s, int32_t n_q, int32_t win_cap, int32_t pool_cap, bool reusable = false)
{
    ManagedAppendWs w{};
    const size_t rows = (size_t)s->batch * n_q * s->n_q_heads;
    w.attn_bytes = tiers_layout(s, n_q, win_cap, pool_cap, reusable).total;
    size_t at = 0;
    w.attn = at; at += align_up(w.attn_bytes);
    w.lse_w = at; at += align_up(rows * sizeof(float));
    w.lse_p = at; at += align_up(rows * sizeof(float));
    w.total = std::max<size_t>(at, kAlign);
    return w;
}

}  // namespace

size_t hgca_managed_append_workspace_bytes(const hgca_shape *shape, const hgca_cache_state *cache, int32_t n_q)
{
    CacheDev c{};
    hgca_shape host_only = shape ? *shape : hgca_shape{};
    host_only.batch = shape ? std::min(shape->batch, 0) : 0;     // sizing needs no device pointers
    if (!shape || !cache || n_q < 0 || n_q > 4096 || check_shape(shape) != HGCA_OK || check_cache(&host_only, cache, &c) != HGCA_OK)
        return 0;
    return managed_append_layout(shape, n_q, c.win_cap, c.pool_cap, true).total;
}

int hgca_managed_append_step(const hgca_shape *shape, const hgca_cache_state *cache, const void *q, const void *k_in,
                             const void *v_in, int32_t n_q, float alpha, double beta, int32_t flags, float *a_gpu,
                             float *a_cpu, float *o_out, float *lse_out, void *ws, size_t ws_bytes, void *hip_stream)
{
    CacheDev c{};
    int rc = check_cache(shape, cache, &c);
    if (rc != HGCA_OK) return rc;
    if (n_q < 0 || n_q > 4096 || !(alpha >= 0.f && alpha <= 1.f) || !(beta >= 0.0) || (flags & ~HGCA_APPEND_ONE_PART_P))
        return HGCA_ERR_INVALID_ARG;
    if (shape->batch == 0 || n_q == 0) return HGCA_OK;
    // the two tiers as ranges of the sequence's block list
    hgca_kv_view window{}, pool{};
    window.k = pool.k = cache->k_blocks;
    window.v = pool.v = cache->v_blocks;
    window.block_table = pool.block_table = cache->block_table;
    window.block_size = pool.block_size = cache->block_size;
    window.max_blocks = pool.max_blocks = cache->max_blocks;
    window.seq_lens = cache->win_lens;
    window.first_block = cache->first_win_block;
    window.cap = c.win_cap;
    pool.seq_lens = cache->pool_lens;
    pool.cap = cache->pool_cap;
    if ((rc = check_append(shape, q, n_q, &window, true)) != HGCA_OK) return rc;
    if ((rc = check_append(shape, q, n_q, &pool, true)) != HGCA_OK) return rc;
    if ((int64_t)shape->batch * n_q > 65535) return HGCA_ERR_UNSUPPORTED;        // a limit of the interface
    if (!k_in || !v_in || !aligned16(k_in) || !aligned16(v_in) || !a_gpu || (cache->pool_cap > 0 && !a_cpu) || !o_out ||
        !lse_out || !aligned16(o_out))
        return HGCA_ERR_INVALID_ARG;
    const ManagedAppendWs w = managed_append_layout(shape, n_q, c.win_cap, c.pool_cap);
    if (!ws || ws_bytes < w.total || !aligned16(ws)) return HGCA_ERR_WORKSPACE;
    char *base = static_cast<char *>(ws);
    float *lse_w = reinterpret_cast<float *>(base + w.lse_w), *lse_p = reinterpret_cast<float *>(base + w.lse_p);
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    const int32_t row_bytes = shape->head_dim * (shape->dtype == HGCA_BF16 ? 2 : 4);

    // Alg. 2, append branch: KV_gpu' = concat(KV_gpu, KV_in)
    if ((rc = from_hip(launch_kv_append(c, k_in, v_in, nullptr, shape->batch, shape->n_kv_heads, row_bytes, n_q, s))) != HGCA_OK)
        return rc;
    // gpu_attention over the window (causal among the incoming tokens), cpu_attention over the complete offloaded
    // cache, merge_state per (sequence, query, head): one launch for both tiers and one fold
    if ((rc = append_attn_tiers(shape, q, n_q, &window, &pool, flags | HGCA_APPEND_CAUSAL_TAIL, o_out, lse_out, lse_w, lse_p, true,
                                base + w.attn, w.attn_bytes, hip_stream)) != HGCA_OK)
        return rc;
    // A_gpu, A_cpu: the query-averaged weights of the two parts, one launch for both
    if ((rc = append_weights_tiers(shape, q, n_q, &window, &pool, 1, lse_w, lse_p, a_gpu, a_cpu, true, hip_stream)) != HGCA_OK)
        return rc;
    // Alg. 1: moving averages (the n_q new entries take their first observed weight), re-evaluation of the salient
    // lists (Sec. 3.2.2: ids = A_cpu > beta / A_cpu.size), eviction of as many whole blocks as it takes: per row, one launch
    if (HGCA_FUSE_APPEND_TAIL)
        return from_hip(launch_append_tail(c, a_gpu, cache->pool_cap > 0 ? a_cpu : nullptr, shape->batch, shape->n_q_heads,
                                           n_q, alpha, beta, s));
    const int64_t rows = (int64_t)shape->batch * shape->n_q_heads;
    if ((rc = from_hip(launch_maw_update(c.a_maw, a_gpu, c.win_lens, rows, shape->n_q_heads, c.win_cap, n_q, alpha, s))) != HGCA_OK)
        return rc;
    // re-evaluation (Sec. 3.2.2): the salient lists are replaced by ids = A_cpu > beta / A_cpu.size
    if (cache->pool_cap > 0) {
        ThresholdArgs t{};
        t.w = a_cpu;
        t.seq_lens = c.pool_lens;
        t.sizes = c.pool_lens;
        t.beta = beta;
        t.n_q_heads = shape->n_q_heads;
        t.cap = cache->pool_cap;
        t.k_max = c.k_max;
        t.idx = c.ctx_idx;
        t.cnt = c.ctx_cnt;
        t.status = c.status;
        t.status_bit = kCacheListFull;
        if ((rc = from_hip(launch_threshold_select(t, rows, s))) != HGCA_OK) return rc;
    }
    // eviction of as many whole blocks as it takes, sparsification of what leaves
    return from_hip(launch_kv_evict(c, shape->batch, shape->n_q_heads, beta, s));
}

}  // extern "C"

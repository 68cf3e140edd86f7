// The launches of a decode step that is too short for launches of their own: two where the general path has four or five.
//
// A small step waits for launches and not for memory: window, scores, selection, attention over the selection and fold
// depend on each other in three levels only, and each kernel of a step of 4 heads over 2 K tokens takes 3 to 7 us whatever
// it does.  Here the window's splits share a launch with the score pass (they need nothing from each other), and the
// workgroup that selects a row's entries attends to them at once and folds the window's partials in.
// Measured (general path : this one, us per step; the rule and more of both sides stand where the path is chosen): fp32, 4 heads
// of 64, window 256, pool 2048, k 64: 18.9 : 13.1; fp32, 32 / 8 heads of 128, window 1024, pool 4096, k 400: 24.8 : 23.3;
// bf16, 64 / 8 heads, window 256, pool 2048, k 64: 22.7 : 16.7.
#include "attn_device.hpp"
#include "select_device.hpp"

#include <algorithm>
#include <type_traits>

namespace hgca {

namespace {

// The window's splits and the chunks of the score pass in one grid, the window's (longer) first.
template <typename T, int D, int G>
__global__ __launch_bounds__(kBlock) void window_scores_kernel(KernelArgs da, KernelArgs sa, int n_dense, int n_chunks)
{
    static_assert(kScoreBlock == kBlock, "both roles use the same workgroup");
    constexpr bool F32 = sizeof(T) == 4;
    using DV = SplitValu<T, D, G, kDense>;
    using SV = SplitValu<T, D, G, kScores>;
    using DM = DenseSplit<D, G, kBlock>;
    using SM = ScoreSplit<D, G>;
    constexpr int kLds = F32 ? (DV::kLdsBytes > SV::kLdsBytes ? DV::kLdsBytes : SV::kLdsBytes)
                             : (DM::kLdsBytes > SM::kLdsBytes ? DM::kLdsBytes : SM::kLdsBytes);
    __shared__ __attribute__((aligned(16))) char s_lds[kLds];
    const bool dense_role = (int)blockIdx.x < n_dense;           // uniform over the workgroup
    const int per_unit = dense_role ? da.part.n_splits : n_chunks;
    const int u = (int)blockIdx.x - (dense_role ? 0 : n_dense);
    const int part = u % per_unit, kvh = u / per_unit % da.sh.n_kv_heads, b = u / (per_unit * da.sh.n_kv_heads);
    if constexpr (F32) {
        if (dense_role) DV::run(da, s_lds, part, kvh, b);
        else SV::run(sa, s_lds, part, kvh, b);
    } else {
        if (!dense_role) {
            SM::run(sa, s_lds, part, kvh, b);
            return;
        }
        const int n = tier_len(da.kv, b), chunk = even_chunk(da.chunk, n, per_unit, 16384 / D), t0 = part * chunk;
        if (t0 >= n) write_empty_partial<D, G>(da.part, (int64_t)b * da.sh.n_q_heads + (int64_t)kvh * G, part);
        else DM::run(da, s_lds, part, kvh, b, t0, min(chunk, n - t0));
    }
}

// One workgroup per (sequence, query head): selection of the row's entries, softmax attention over them (V rows only, the
// scores are at hand) and the fold with the window's partials.  After the selection its dynamic LDS holds the list's weights
// and rows.  Bound by the row's chain of round trips and, for long lists, by what one compute unit takes in (kLoads
// 16-byte loads in flight per lane, 128 KB per unit).
template <typename T, int D>
__global__ __launch_bounds__(kLargeBlock) void select_attend_kernel(SelectArgs a, KvDev kv, Partials win, void *o, int o_bf16,
                                                                    float *lse, int cache_floats, int cache_bytes,
                                                                    int list_bytes)
{
    using S = Sel<kLargeBlock>;
    constexpr int EPL = Elem<T>::kPerLoad, LPR = D / EPL, RPW = kWave / LPR, NW = kLargeBlock / kWave, RPI = NW * RPW;
    constexpr int C4 = D / 4, SG = kLargeBlock / C4;             // the window's fold: four columns per thread, SG splits at a time
    constexpr size_t ROW_BYTES = D * sizeof(T);
    extern __shared__ __attribute__((aligned(16))) float s_dyn[];
    __shared__ union {
        typename S::SelShared sel;
        struct {
            float acc[NW][D];                    // every wave's sum over its list entries
            float4 win[SG][C4];
            float m[NW], l_list[NW], l_win[SG];
        } f;
    } sh;
    const int64_t bh = blockIdx.x;
    const int b = (int)(bh / a.sh.n_q_heads), kvh = (int)(bh % a.sh.n_q_heads) / a.sh.group;
    static_assert(kMaxShortList * 8 <= kMaxCacheFloats * 4, "weights and rows of a list fit where the selection had its row");
    const int tid = threadIdx.x, w = tid / kWave, lane = tid % kWave, r = lane / LPR, c = lane % LPR;

    select_one_row<kLargeBlock, 8>(a, sh.sel, s_dyn, bh, cache_floats, cache_bytes, list_bytes);

    // the window's partials travel while the list's rows are looked up
    const int sg = tid / C4, c4 = tid % C4, np = win.n_splits;
    const int64_t first = bh * win.stride;
    float pm = -INFINITY, pl = 0.f;
    float4 po = make_float4(0.f, 0.f, 0.f, 0.f);
    if (sg < np) {
        pm = win.m[first + sg];
        pl = win.l[first + sg];
        po = *reinterpret_cast<const float4 *>(win.o + (first + sg) * D + 4 * c4);
    }
    float mx = pm;
    for (int s = sg + SG; s < np; s += SG) mx = fmaxf(mx, win.m[first + s]);

    __syncthreads();                             // the list is written (by this workgroup) and the selection's LDS is free
    const int n = tier_len(a.kv, b);
    int k = a.k_per_seq ? a.k_per_seq[b] : a.k_uniform;
    k = max(0, min(min(k, n), a.k_max));
    float *s_p = s_dyn;
    uint32_t *s_row = reinterpret_cast<uint32_t *>(s_dyn + a.k_max);
    const int32_t *blocks = kv.block_table ? kv.block_table + (int64_t)b * kv.max_blocks + (kv.first_block ? kv.first_block[b] : 0)
                                           : nullptr;
    for (int j = tid; j < k; j += kLargeBlock) {
        // a position that is none of the sequence's (a row with NaN scores need not fill its list) is clamped into it, as in
        // make_row_map: no address is formed that the tier or its block table does not hold
        const int tok = min(max(a.idx[bh * a.k_max + j], 0), n - 1);
        s_row[j] = blocks ? (uint32_t)(((int64_t)blocks[tok / kv.block_size] * a.sh.n_kv_heads + kvh) * kv.block_size + tok % kv.block_size)
                          : (uint32_t)(((int64_t)b * a.sh.n_kv_heads + kvh) * kv.cap + tok);
        const float s = a.sel_scores[bh * a.k_max + j];
        s_p[j] = s;
        mx = fmaxf(mx, s);
    }
    mx = wave_max(mx);
    if (lane == 0) sh.f.m[w] = mx;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NW; ++i) mx = fmaxf(mx, sh.f.m[i]);
    const float M = mx;                          // of window and list together

    float acc[EPL], l = 0.f;
#pragma unroll
    for (int e = 0; e < EPL; ++e) acc[e] = 0.f;
    auto attend = [&](auto loads) {
        constexpr int U = decltype(loads)::value;
        for (int base = 0; base < k; base += RPI * U) {
            uint4 vr[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int j = min(base + u * RPI + w * RPW + r, k - 1);
                vr[u] = load16_stream(kv.v + s_row[j] * ROW_BYTES + c * 16);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int j = base + u * RPI + w * RPW + r;
                // -inf stays out whatever the maximum is
                const float s = j < k ? s_p[j] : -INFINITY, p = s == -INFINITY ? 0.f : __expf(s - M);
                float vf[EPL];
                Elem<T>::expand(vr[u], vf);
                l += p;
#pragma unroll
                for (int e = 0; e < EPL; ++e) acc[e] = fmaf(p, vf[e], acc[e]);
            }
        }
    };
    if (k <= 2 * RPI) attend(std::integral_constant<int, 2>{});
    else attend(std::integral_constant<int, 8>{});
#pragma unroll
    for (int e = 0; e < EPL; ++e) {
        acc[e] = strided_sum<LPR>(acc[e]);
        if (r == 0) sh.f.acc[w][c * EPL + e] = acc[e];
    }
    l = strided_sum<LPR>(l);                     // the lanes of a row hold the same
    if (lane == 0) sh.f.l_list[w] = l;
    if (sg < np) {
        const float wgt = pm == -INFINITY ? 0.f : expf(pm - M);
        pl *= wgt;
        po.x *= wgt; po.y *= wgt; po.z *= wgt; po.w *= wgt;
        for (int s = sg + SG; s < np; s += SG) {
            const float ms = win.m[first + s], ws = ms == -INFINITY ? 0.f : expf(ms - M);
            const float4 v = *reinterpret_cast<const float4 *>(win.o + (first + s) * D + 4 * c4);
            pl = fmaf(win.l[first + s], ws, pl);
            po.x = fmaf(v.x, ws, po.x); po.y = fmaf(v.y, ws, po.y);
            po.z = fmaf(v.z, ws, po.z); po.w = fmaf(v.w, ws, po.w);
        }
        sh.f.win[sg][c4] = po;
        if (c4 == 0) sh.f.l_win[sg] = pl;
    }
    __syncthreads();
    if (tid < D) {
        float L = 0.f, t = 0.f;
#pragma unroll
        for (int i = 0; i < NW; ++i) { t += sh.f.acc[i][tid]; L += sh.f.l_list[i]; }
        const float *part = reinterpret_cast<const float *>(sh.f.win);
        for (int s = 0; s < min(np, SG); ++s) { t += part[s * D + tid]; L += sh.f.l_win[s]; }
        const bool any = M != -INFINITY;
        t = any ? t * (1.f / L) : 0.f;
        if (o_bf16) {
            uint32_t u = __float_as_uint(t);
            u += 0x7fffu + ((u >> 16) & 1u);     // round to nearest even (finite values)
            reinterpret_cast<uint16_t *>(o)[bh * D + tid] = (uint16_t)(u >> 16);
        } else {
            reinterpret_cast<float *>(o)[bh * D + tid] = t;
        }
        if (tid == 0 && lse) lse[bh] = any ? M + logf(L) : -INFINITY;
    }
}

KernelArgs to_kernel_args(const AttnArgs &a)
{
    KernelArgs ka{};
    ka.sh = a.sh;
    ka.q = static_cast<const char *>(a.q);
    ka.kv = a.kv;
    ka.chunk = a.chunk;
    ka.part = a.part;
    return ka;
}

template <typename T, int D>
hipError_t launch_window_scores_group(const KernelArgs &da, const KernelArgs &sa, int n_dense, int n_chunks, dim3 grid,
                                      hipStream_t s)
{
    const dim3 block(kBlock);
    switch (da.sh.group) {
    case 1: hipLaunchKernelGGL((window_scores_kernel<T, D, 1>), grid, block, 0, s, da, sa, n_dense, n_chunks); break;
    case 2: hipLaunchKernelGGL((window_scores_kernel<T, D, 2>), grid, block, 0, s, da, sa, n_dense, n_chunks); break;
    case 4: hipLaunchKernelGGL((window_scores_kernel<T, D, 4>), grid, block, 0, s, da, sa, n_dense, n_chunks); break;
    case 8: hipLaunchKernelGGL((window_scores_kernel<T, D, 8>), grid, block, 0, s, da, sa, n_dense, n_chunks); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <typename T, int D>
hipError_t launch_select_attend_typed(const SelectArgs &a, const KvDev &kv, const Partials &win, void *o, int o_dtype,
                                      float *lse, hipStream_t s)
{
    using S = Sel<kLargeBlock>;
    const int padded = S::padded_length(a.kv.cap);
    const int cache_floats = padded <= kMaxCacheFloats ? padded : 0;
    const int cache_bytes = cache_floats == 0 && padded <= 4 * kMaxCacheFloats ? padded : 0;
    const int list_bytes = cache_floats != 0 ? 0 : kMaxCacheFloats * (int)sizeof(float);
    const size_t lds = std::max({(size_t)cache_floats * sizeof(float), (size_t)list_bytes, (size_t)a.k_max * 8});
    const hipError_t rc = lift_lds_limit<select_attend_kernel<T, D>>(kMaxCacheFloats * (int)sizeof(float));
    if (rc != hipSuccess) return rc;
    const int64_t rows = (int64_t)a.sh.batch * a.sh.n_q_heads;
    hipLaunchKernelGGL((select_attend_kernel<T, D>), dim3((unsigned)rows), dim3(kLargeBlock), lds, s, a, kv, win, o,
                       o_dtype == 1 ? 1 : 0, lse, cache_floats, cache_bytes, list_bytes);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_window_scores(int dtype, int head_dim, const AttnArgs &dense, const ScoreArgs &scores, hipStream_t s)
{
    const int64_t units = (int64_t)dense.sh.batch * dense.sh.n_kv_heads;
    const int64_t n_dense = units * dense.part.n_splits, blocks = n_dense + units * scores.n_chunks;
    if (blocks == 0) return hipSuccess;
    if (blocks > 0x7fffffff || scores.group_max) return hipErrorInvalidValue;
    const KernelArgs da = to_kernel_args(dense);
    KernelArgs sa = da;
    sa.kv = scores.kv;
    sa.chunk = scores.chunk;
    sa.scores = scores.scores;
    const dim3 grid((unsigned)blocks);
    if (dtype == 0 && head_dim == 64) return launch_window_scores_group<float, 64>(da, sa, (int)n_dense, scores.n_chunks, grid, s);
    if (dtype == 0 && head_dim == 128) return launch_window_scores_group<float, 128>(da, sa, (int)n_dense, scores.n_chunks, grid, s);
    if (dtype == 1 && head_dim == 64) return launch_window_scores_group<bf16_t, 64>(da, sa, (int)n_dense, scores.n_chunks, grid, s);
    if (dtype == 1 && head_dim == 128) return launch_window_scores_group<bf16_t, 128>(da, sa, (int)n_dense, scores.n_chunks, grid, s);
    return hipErrorInvalidValue;
}

hipError_t launch_select_attend(int dtype, int head_dim, const SelectArgs &a, const Partials &window, void *o, int o_dtype,
                                float *lse, hipStream_t s)
{
    if (a.sh.batch == 0) return hipSuccess;
    if (!a.sel_scores || a.k_max <= 0 || a.k_max > kMaxShortList) return hipErrorInvalidValue;
    if (dtype == 0 && head_dim == 64) return launch_select_attend_typed<float, 64>(a, a.kv, window, o, o_dtype, lse, s);
    if (dtype == 0 && head_dim == 128) return launch_select_attend_typed<float, 128>(a, a.kv, window, o, o_dtype, lse, s);
    if (dtype == 1 && head_dim == 64) return launch_select_attend_typed<bf16_t, 64>(a, a.kv, window, o, o_dtype, lse, s);
    if (dtype == 1 && head_dim == 128) return launch_select_attend_typed<bf16_t, 128>(a, a.kv, window, o, o_dtype, lse, s);
    return hipErrorInvalidValue;
}

}  // namespace hgca

// Independent kernels of a decode step as ONE launch.
#include "attn_device.hpp"

#include <type_traits>

namespace hgca {

namespace {

// The window's split kernels and the sparse part's split kernels:
//
// Both are streaming passes that need nothing from each other (Alg. 2 runs gpu_attention and cpu_attention side by
// side); as two launches of one stream the second waits for the last workgroup of the first, and each pays its own
// ramp-up and tail.  In one grid the workgroups of one part take over compute units as the other's drain.  Roles by
// blockIdx; which part starts first is window_first's to say.
// fp32 takes both parts on the vector units; there and in small steps a launch saved is what counts (managed decode loop of one
// sequence, fp32, 32 / 8 heads of 64, per step: insert, window, gather and tail 24.8 us, in two launches 18.2).
#ifndef HGCA_DG_OCC
#define HGCA_DG_OCC 5                            // waves per SIMD the register budget is set for
#endif
#ifndef HGCA_DG_GATHER_UNROLL
#define HGCA_DG_GATHER_UNROLL 8                  // K / V loads a lane of a sparse split keeps in flight (4 in a launch of
#endif                                           // its own, where eight 64-register workgroups share a unit; here the
                                                 // register budget is the window body's: 66.8 against 67.9 us per steady step)
#ifndef HGCA_DG_UNROLL
#define HGCA_DG_UNROLL 4                         // V loads a lane of a window split keeps in flight
#endif

// ORDER of the gather's workgroups: 0 head by head, 1 by groups of heads, 2 the same with the rows kept for each other.
template <typename T, int D, int G, int GMODE, int LD, int ORDER>
__global__ __launch_bounds__(kBlock, sizeof(T) == 2 && G < 8 ? HGCA_DG_OCC : 1) void dense_gather_kernel(KernelArgs da, KernelArgs ga, int n_dense,
                                                                          int dense_splits, int gather_splits,
                                                                          int gather_first, const char *k_new,
                                                                          const char *v_new)
{
    constexpr bool F32 = sizeof(T) == 4;
    // bf16: the window on the matrix cores, LDS sized for splits of up to LD tokens; fp32: on the vector units
    using DS = std::conditional_t<F32, SplitValu<T, D, G, kDense>, DenseSplit<D, G, kBlock, HGCA_DG_UNROLL, LD>>;
    using GS = SplitValu<T, D, 1, GMODE, F32 ? kUnroll : HGCA_DG_GATHER_UNROLL, ORDER == 2>;
    constexpr int kLds = DS::kLdsBytes > GS::kLdsBytes ? DS::kLdsBytes : GS::kLdsBytes;
    __shared__ __attribute__((aligned(16))) char s_lds[kLds];
    // one part takes the lower block numbers and starts first, the other fills in behind it (window_first)
    const int n_gather = (int)gridDim.x - n_dense;
    const bool dense_role = gather_first ? (int)blockIdx.x >= n_gather : (int)blockIdx.x < n_dense;
    const int u = (int)blockIdx.x - (dense_role ? (gather_first ? n_gather : 0) : (gather_first ? 0 : n_dense));
    if (dense_role) {                            // uniform over the workgroup
        if (ORDER > 0 && u >= da.sh.batch * da.sh.n_kv_heads * dense_splits) return;         // padding
        const int split = u % dense_splits, kvh = (u / dense_splits) % da.sh.n_kv_heads,
                  b = u / (dense_splits * da.sh.n_kv_heads);
        int n = tier_len(da.kv, b), len = 0, first = 0;
        bool takes_token = false;
        if (k_new) {                             // uniform over the launch: the window takes one more token first
            len = da.kv.seq_lens[b];
            first = da.kv.first_block[b];
            const int grown = pending_window_len(len, first, 1, da.kv.cap, da.kv.block_size, da.kv.max_blocks, nullptr);
            n = min(max(grown, 0), da.kv.cap);
            takes_token = grown > len;
        }
        const int chunk = even_chunk(da.chunk, n, dense_splits, 16384 / D), t0 = split * chunk;
        if (takes_token && len >= t0 && len < t0 + chunk) {      // uniform over the workgroup
            // this split owns the token's position: its K and V rows go into the window's block, then the split
            // reads them back like any other row (no other workgroup of the launch touches that position)
            constexpr int kRow = D * (int)sizeof(T), kPieces = kRow / 16;
            if (threadIdx.x < 2 * kPieces) {
                const bool is_v = threadIdx.x >= kPieces;
                const int piece = threadIdx.x % kPieces;
                const int64_t blk = da.kv.block_table[(int64_t)b * da.kv.max_blocks + first + len / da.kv.block_size];
                const int64_t dst = ((blk * da.sh.n_kv_heads + kvh) * da.kv.block_size + len % da.kv.block_size) * kRow;
                const int64_t src = ((int64_t)b * da.sh.n_kv_heads + kvh) * kRow;
                *reinterpret_cast<uint4 *>(const_cast<char *>(is_v ? da.kv.v : da.kv.k) + dst + 16 * piece) =
                    *reinterpret_cast<const uint4 *>((is_v ? v_new : k_new) + src + 16 * piece);
            }
            __syncthreads();
        }
        if constexpr (F32) {
            DS::run_of(da, s_lds, split, kvh, b, n);
        } else {
            if (t0 >= n) write_empty_partial<D, G>(da.part, (int64_t)b * da.sh.n_q_heads + (int64_t)kvh * G, split);
            else DS::run(da, s_lds, split, kvh, b, t0, min(chunk, n - t0));
        }
        return;
    }
    if (ORDER == 0) {
        GS::run(ga, s_lds, u % gather_splits, (u / gather_splits) % ga.sh.n_q_heads, u / (gather_splits * ga.sh.n_q_heads));
        return;
    }
    GatherPlace at;
    if (at.find(u, ga.sh, gather_splits)) GS::run(ga, s_lds, at.split, at.head, at.b);
}

}  // namespace

bool dense_gather_fusable(int dtype, int head_dim, int group)
{
    return (dtype == 0 || dtype == 1) && (head_dim == 64 || head_dim == 128) && (group == 1 || group == 2 || group == 4 || group == 8);
}

hipError_t launch_dense_gather(int dtype, int head_dim, const AttnArgs &dense, const AttnArgs &gather, hipStream_t s,
                               const void *k_new, const void *v_new)
{
    if (!dense_gather_fusable(dtype, head_dim, dense.sh.group) || gather.grouped) return hipErrorInvalidValue;
    if ((k_new != nullptr) != (v_new != nullptr)) return hipErrorInvalidValue;
    if (k_new && (!dense.kv.block_table || !dense.kv.first_block || !dense.kv.seq_lens)) return hipErrorInvalidValue;
    // by groups without keeping the rows is built for groups of 2 and for given scores; the others keep them here
    const int order = dense.sh.group == 1 || !gather.by_group ? 0 : !gather.sel_scores && (gather.keep || dense.sh.group > 2) ? 2 : 1;
    // (by groups, the first part's number is a multiple of the number of XCDs, so that the second part's go round them as they count)
    const int64_t n_window = (int64_t)dense.sh.batch * dense.sh.n_kv_heads * dense.part.n_splits;
    const int64_t n_dense = order ? (n_window + kXcds - 1) / kXcds * kXcds : n_window;
    const int64_t n_gather = order ? gather_blocks(gather.sh, gather.part.n_splits)
                                   : (int64_t)gather.sh.batch * gather.sh.n_q_heads * gather.part.n_splits;
    if (n_dense + n_gather == 0) return hipSuccess;
    if (n_dense + n_gather > 0x7fffffff) return hipErrorInvalidValue;
    auto to_ka = [](const AttnArgs &a) {
        KernelArgs ka{};
        ka.sh = a.sh;
        ka.q = static_cast<const char *>(a.q);
        ka.kv = a.kv;
        ka.idx = a.idx;
        ka.cnt = a.cnt;
        ka.sel_scores = a.sel_scores;
        ka.k_max = a.k_max;
        ka.chunk = a.chunk;
        ka.part = a.part;
        ka.scores = a.raw_scores;
        return ka;
    };
    const KernelArgs da = to_ka(dense), ga = to_ka(gather);
    const dim3 grid((unsigned)(n_dense + n_gather)), block(kBlock);
    const int g = dense.sh.group;
    const int gather_first = window_first(dtype == 0, g, dense.kv.cap, gather.k_max, gather.sel_scores != nullptr) ? 0 : 1;
    if (dtype == 1 && g == 8 && gather.sel_scores) return hipErrorInvalidValue;  // not built: its callers use two launches
    // the window's splits size the launch's LDS: the common 256-token splits leave room for seven workgroups per unit
#define HGCA_DG_LAUNCH(T, D, G, GMODE, LD, ORDER)                                                                   \
    hipLaunchKernelGGL((dense_gather_kernel<T, D, G, GMODE, LD, ORDER>), grid, block, 0, s, da, ga, (int)n_dense,   \
                       dense.part.n_splits, gather.part.n_splits, gather_first, static_cast<const char *>(k_new), \
                       static_cast<const char *>(v_new))
#define HGCA_DG_SCORED(T, D, G, LD)                                                                                 \
    do {                                                                                                            \
        if (order) HGCA_DG_LAUNCH(T, D, G, kGatherScored, LD, (G > 1 ? 1 : 0));                                     \
        else HGCA_DG_LAUNCH(T, D, G, kGatherScored, LD, 0);                                                         \
    } while (0)
#define HGCA_DG_GATHER(T, D, G, LD)                                                                                 \
    do {                                                                                                            \
        if (order == 2) HGCA_DG_LAUNCH(T, D, G, kGather, LD, (G > 1 ? 2 : 0));                                      \
        else if (order) HGCA_DG_LAUNCH(T, D, G, kGather, LD, (G == 2 ? 1 : G > 1 ? 2 : 0));                         \
        else HGCA_DG_LAUNCH(T, D, G, kGather, LD, 0);                                                               \
    } while (0)
#define HGCA_DG_CASE(D, G)                                                                                          \
    if (head_dim == D && g == G) {                                                                                  \
        if (dtype == 0) {                                                                                           \
            if (gather.sel_scores) HGCA_DG_SCORED(float, D, G, kMaxChunk);                                          \
            else HGCA_DG_GATHER(float, D, G, kMaxChunk);                                                            \
        } else if (gather.sel_scores) {                                                                             \
            if (dense.chunk <= 256) HGCA_DG_SCORED(bf16_t, D, (G < 8 ? G : 4), 256);                                \
            else HGCA_DG_SCORED(bf16_t, D, (G < 8 ? G : 4), kMaxChunk);                                             \
        } else {                                                                                                    \
            if (dense.chunk <= 256) HGCA_DG_GATHER(bf16_t, D, G, 256);                                              \
            else HGCA_DG_GATHER(bf16_t, D, G, kMaxChunk);                                                           \
        }                                                                                                           \
        return hipGetLastError();                                                                                   \
    }
    HGCA_DG_CASE(64, 1) HGCA_DG_CASE(64, 2) HGCA_DG_CASE(64, 4) HGCA_DG_CASE(64, 8)
    HGCA_DG_CASE(128, 1) HGCA_DG_CASE(128, 2) HGCA_DG_CASE(128, 4) HGCA_DG_CASE(128, 8)
#undef HGCA_DG_CASE
#undef HGCA_DG_GATHER
#undef HGCA_DG_SCORED
#undef HGCA_DG_LAUNCH
    return hipErrorInvalidValue;
}

}  // namespace hgca

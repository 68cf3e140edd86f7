// What the append kernels in bf16 and in fp32 share: where rows live, which row of the launch is which query and head, the
// layouts of the tiles in LDS that the matrix operands are read from.
#pragma once

#include "hgca_launch.hpp"
#include "row_map.hpp"

namespace hgca {

namespace {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float float2v __attribute__((ext_vector_type(2)));

constexpr int kStepBlocks = 2;                   // 32-token contraction blocks per step
constexpr int kStepTokens = 32 * kStepBlocks;
constexpr int kRowsPerBlock = 128;               // query rows of a workgroup
constexpr int kAttnWaves = kRowsPerBlock / 32, kAttnBlock = kAttnWaves * kWave;   // of the attention: a wave owns 32 of them
constexpr int kSub = kMaxChunk;                  // entries of the table of rows (paged tiers)
static_assert(kStepTokens == kLineStep, "shares of a line are whole steps");
static_assert(kSub * 16 % kStepTokens == 0, "a pass is a whole number of steps");

// Where the rows of a pass over part of a split live.  A contiguous tier is plain arithmetic.  A paged tier gets a
// table in LDS with one entry per 16 tokens (block sizes are multiples of 16: the row of the granule's first token for
// this KV head), so a lookup is a shift, whatever the block size, and one filling of kSub entries covers a whole split
// and the load pipeline is not drained for refills.
constexpr int kGranule = 16;
struct BlockRows {
    const uint32_t *table;                       // LDS; nullptr => row = base + j
    uint32_t base;
};

// tokens a pass may cover so that its granules fit the table, a multiple of the step
__device__ __forceinline__ int pass_length(const KvDev &kv, int nt_total) {
    return kv.block_table ? kSub * kGranule : max(nt_total, 1);
}

// `first` is the tier position of the pass's first token, a multiple of kGranule (splits and passes are cut at whole
// steps), nt the number of tokens; contains a barrier iff the tier is paged (uniform over the workgroup).
template <int BLOCK>
__device__ __forceinline__ BlockRows make_block_rows(uint32_t *s_tab, const KvDev &kv, int n_kv_heads, int b, int kvh,
                                                     int first, int nt)
{
    BlockRows m;
    if (!kv.block_table) {
        m.table = nullptr;
        m.base = (uint32_t)(((int64_t)b * n_kv_heads + kvh) * kv.cap + first);
        return m;
    }
    const int32_t *blocks = kv.block_table + (int64_t)b * kv.max_blocks + (kv.first_block ? kv.first_block[b] : 0);
    const int n_gr = (nt + kGranule - 1) / kGranule;             // <= kSub by pass_length
    for (int i = threadIdx.x; i < n_gr; i += BLOCK) {
        const int tok = first + i * kGranule;
        s_tab[i] = (uint32_t)(((int64_t)blocks[tok / kv.block_size] * n_kv_heads + kvh) * kv.block_size + tok % kv.block_size);
    }
    __syncthreads();
    m.table = s_tab;
    m.base = 0;
    return m;
}

// Reductions over the two halves of a wave (lanes n and n + 32 hold partial results of one query row):
// v_permlane32_swap of a register with itself returns the lower half twice and the upper half twice, one VALU
// instruction where a lane shuffle would go through the LDS pipeline.
__device__ __forceinline__ float halves_max(float x) {
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float halves_sum(float x) {
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// Where a query row of a (sequence, KV head) pair lives: query r / G, head r % G of the group.
struct RowInfo {
    bool valid;
    int query;
    int64_t out_row;                             // (b * N + query) * Hq + head
};

template <int G>
__device__ __forceinline__ RowInfo row_info(const AppendArgs &a, int b, int kvh, int r) {
    RowInfo ri;
    ri.valid = r < a.n_q * G;
    ri.query = ri.valid ? r / G : 0;
    ri.out_row = ((int64_t)b * a.n_q + ri.query) * a.sh.n_q_heads + kvh * G + (ri.valid ? r % G : 0);
    return ri;
}

constexpr int kXcds = 8;                         // workgroups of a launch are dealt to the XCDs in turn
constexpr int kWTile = 32;                       // tokens of a wave's tile in the weights pass
constexpr int kWManyRowTokens = 2048;            // tokens of a block that more than one pass over the rows goes through

// LDS stage of the attention kernel: the rows of a step are brought in by LDS-direct loads (global_load_lds, 16
// bytes per lane, no registers in between).  One such instruction fills 1024 consecutive bytes of LDS with whatever
// 64 pieces its lanes address, so the layout inside each 1 KB group is chosen by the lane -> global address map:
//   K: row-major rows with the 16-byte pieces of a row XOR-swizzled by the row, so that the 16 rows an A-operand
//      read touches land on different banks without padding;
//   V: quads of four rows, interleaved in 32-byte chunks ([quad][column chunk][row of the quad][32 bytes]), so that
//      the 4 rows x 32 bytes a 16-lane group takes with one transpose read are 128 consecutive bytes and the two
//      groups of a half wave, which take neighbouring chunks, 256.
template <int D, int NW> struct DmaStage {
    static constexpr int kRowBytes = D * 2;
    static constexpr int kPieces = kRowBytes / 16;               // 16-byte pieces per row
    static constexpr int kSwizzled = kPieces < 16 ? kPieces : 16;
    static constexpr int kGroupRows = 1024 / kRowBytes;          // rows per load instruction of a wave
    static constexpr int kGroups = kStepTokens / kGroupRows;     // per step and tensor
    static constexpr int kLoads = kGroups / NW;                  // per wave, step and tensor
    static constexpr int kBytes = kStepTokens * kRowBytes;       // per step and tensor
    static_assert(kGroups % NW == 0 && kLoads >= 1, "the waves share the groups of a step evenly");

    static __device__ __forceinline__ int k_swizzle(int row) { return (row / (16 / kSwizzled)) % kSwizzled; }
    // byte offset, in a K stage, of logical piece `piece` of step row `row`
    static __device__ __forceinline__ int k_offset(int row, int piece) {
        return row * kRowBytes + 16 * (piece ^ k_swizzle(row));
    }
    // byte offset, in a V stage, of the 32-byte column chunk `dt` of step row `row`
    static __device__ __forceinline__ int v_offset(int row, int dt) {
        return (row / 4) * (4 * kRowBytes) + dt * 128 + (row % 4) * 32;
    }
};

}  // namespace

}  // namespace hgca

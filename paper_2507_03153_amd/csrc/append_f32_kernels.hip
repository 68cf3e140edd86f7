// Append stage on fp32 inputs: the attention of N queries per sequence and the query-averaged weights, as in
// append_kernels.hip (work units, orientation of the products, lines of shares), with products on the bf16 matrix instructions.
//
// The fp32 matrix instructions do a sixteenth of the bf16 ones' work per cycle.  An fp32 value is the sum of three bf16 parts, each
// the rounding error of those before (24 bits), and of the nine products of parts the six down to 2^-18 of the whole are
// formed: what is left out is below 2^-26 of it, less than one rounding of a sum.  The products of the upper parts go to
// accumulators of their own, so that a sum that has nearly reached its size is rounded a few times only.
//
// bf16 has no bits below 2^-133 (2^-126 where subnormal numbers count as 0), so values below 2^-102 may lose lower parts:
//   queries and softmax weights are taken apart times 2^24 (kUp), which makes the sum of the parts exact whatever they are;
//   keys lose less than 2^-126, which |q| sm_scale <= 2^90 keeps out of the scores (2^-29 over 128 columns); larger queries become NaN;
//   V rows lose less than 2^-126 as well, which counts where a sum of them is below 2^-88 (kLeast; 2^-24 of it over 2^14 tokens).
// Values whose upper part rounds to infinity and values that are not finite give NaN.  Where sums are not finite, or so small,
// they are formed again with fp32 products, every row from what it sees and nothing else: one infinite V row or one NaN key in
// every share costs the attention of 2 x 24 queries on 5 K tokens 44 -> 110 us (66 with fp32 products throughout), a NaN key every
// 100 tokens their weights 26 -> 85 (38), a key with scores of -inf 26 -> 44.
//
// Errors against 64 bits are those of fp32 products (2 x 24 queries on 5 K tokens: O 3.5e-7, weights 2.6e-7 with either).  fp32
// matrix instructions : parts, us: that turn 137.7 : 93.6 (attention 76 : 45, weights 42 : 30); 8 x 24 queries of 32 / 8 heads of 64 on 17 K
// tokens 664 : 332; attention alone, 4 x 32 queries of 32 ungrouped heads on 4 K tokens 318 : 133, 8 x 32 queries of 32 / 8 heads on
// 16 K 643 : 396, 8 queries 626 : 237.  What bounds it now: a share's start (lengths, table of rows, first tiles: some 8 us of 45)
// and, per 32-token tile, products 3100 cycles of 5500 with 96 rows.
#include "append_device.hpp"

namespace hgca {

namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
struct Parts {
    u32x4 h, m, l;                               // 8 bf16 each
};

constexpr float kUp = 0x1p24f, kDown = 0x1p-24f;
constexpr float kMostQuery = 0x1p90f;            // times the scale
constexpr float kLeast = 0x1p-88f;

// the parts of x and y into element e of p: eleven vector instructions
__device__ __forceinline__ void pair_parts(Parts &p, int e, float x, float y)
{
    const float2v v = {x, y};
    p.h[e] = __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
    const float2v r = {x - __uint_as_float(p.h[e] << 16), y - __uint_as_float(p.h[e] & 0xffff0000u)};            // exact
    p.m[e] = __builtin_bit_cast(uint32_t, __builtin_convertvector(r, bf16x2));
    const float2v t = {r[0] - __uint_as_float(p.m[e] << 16), r[1] - __uint_as_float(p.m[e] & 0xffff0000u)};      // exact
    p.l[e] = __builtin_bit_cast(uint32_t, __builtin_convertvector(t, bf16x2));
}
__device__ __forceinline__ Parts parts_of(const uint4 &a, const uint4 &b)
{
    Parts p;
    pair_parts(p, 0, __uint_as_float(a.x), __uint_as_float(a.y));
    pair_parts(p, 1, __uint_as_float(a.z), __uint_as_float(a.w));
    pair_parts(p, 2, __uint_as_float(b.x), __uint_as_float(b.y));
    pair_parts(p, 3, __uint_as_float(b.z), __uint_as_float(b.w));
    return p;
}
// The power of two that queries are taken apart times, and the scale of the scores that they give (arguments of the kernels: both
// are at hand wherever they are used, without a register).
struct QueryScale {
    float up, scale;
};
QueryScale query_scale(float sm_scale)
{
    // with a scale as small as this sums of up to 2^128 may be scores of ordinary size, and nothing is lost (2^-60 2^127 2^-126)
    return sm_scale < 0x1p-60f ? QueryScale{1.f, sm_scale} : QueryScale{kUp, sm_scale * kDown};
}

// of eight columns of a query
__device__ __forceinline__ Parts query_parts(const char *src, float sm_scale, float up)
{
    const floatx4 a = __builtin_bit_cast(floatx4, load16(src)), b = __builtin_bit_cast(floatx4, load16(src + 16));
    float most = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) most = fmaxf(fmaxf(most, fabsf(a[i])), fabsf(b[i]));
    if (most * sm_scale > kMostQuery) up = __uint_as_float(0x7fc00000u);
    Parts p;
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        pair_parts(p, e, a[2 * e] * up, a[2 * e + 1] * up);
        pair_parts(p, 2 + e, b[2 * e] * up, b[2 * e + 1] * up);
    }
    return p;
}
__device__ __forceinline__ floatx4 mfma(const u32x4 &a, const u32x4 &b, floatx4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// The sums of a 16 x 16 tile: products of the upper parts in two chains, and the others.
struct TileSums {
    floatx4 up[2], lo;
    __device__ __forceinline__ void clear() { up[0] = up[1] = lo = floatx4{}; }
    // the j-th of a slice's six products
    __device__ __forceinline__ void add(const Parts &a, const Parts &b, int i, int j) {
        if (j == 0) lo = mfma(a.l, b.h, lo);
        else if (j == 1) up[i % 2] = mfma(a.h, b.h, up[i % 2]);
        else if (j == 2) lo = mfma(a.h, b.l, lo);
        else if (j == 3) lo = mfma(a.m, b.m, lo);
        else if (j == 4) lo = mfma(a.m, b.h, lo);
        else lo = mfma(a.h, b.m, lo);
    }
    __device__ __forceinline__ floatx4 sum() const { return (up[0] + up[1]) + lo; }
};

// The sums of a 16 x 16 tile with fp32 products: the lane points at its four columns (of every 16) of row n of each operand.
template <int D> __device__ __forceinline__ floatx4 scores_f32(const char *a, const char *b)
{
    floatx4 c[4] = {};                           // a quarter of the columns each
#pragma unroll 2
    for (int j = 0; j < D / 16; ++j) {
        const floatx4 x = __builtin_bit_cast(floatx4, load16(a + 64 * j)), y = __builtin_bit_cast(floatx4, load16(b + 64 * j));
#pragma unroll
        for (int e = 0; e < 4; ++e) c[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[e], y[e], c[e], 0, 0, 0);
    }
    return (c[0] + c[1]) + (c[2] + c[3]);
}

// ---- attention -------------------------------------------------------------------------------------------------

constexpr int kTile = 32;                        // tokens that go through LDS at a time
constexpr int kF32Waves = 8, kF32Block = kF32Waves * kWave, kF32Rows = kRowsPerBlock / kF32Waves;

// K and V of a tile as bf16 parts, K as in the bf16 kernel, V in quads of four rows interleaved in 32-byte chunks, those of
// every second quad exchanged in pairs (a half of a wave reads the same chunk of two quads).  A thread brings in, takes apart and
// stores one piece of 8 columns of each tensor.
template <int D> struct PartStage {
    using S = DmaStage<D, kAttnWaves>;
    static constexpr int kPart = kTile * S::kRowBytes;           // bytes of one part of one tensor
    static constexpr int kBytes = 6 * kPart;                     // K h, m, l, V h, m, l
    static constexpr int kPieces = kTile * (D / 8);
    static_assert(kPieces <= kF32Block && kPieces % kWave == 0, "one piece per thread, whole waves");
    static __device__ __forceinline__ int v_offset(int row, int chunk) {
        return 3 * kPart + row / 4 * (4 * S::kRowBytes) + (chunk ^ row / 4 % 2) * 128 + row % 4 * 32;
    }
};

// The softmax of a wave's rows over the tier positions [begin, row_end) (of each row; ascending over the wave's rows) with fp32
// products: maximum of the raw scores, sums of the weights (the lane's) and of V times them.  As in the kernel below, the four lanes
// g of row n hold the output columns 16 dt + 4 g .. + 3; all lanes of the wave take part.  Tokens that all rows see pass 16 at a
// time through the fp32 matrix instructions, the others one by one, as a weight of 0 does not keep an infinity out of a product.
template <int D>
__device__ __forceinline__ void append_rows_again(const KvDev &kv, int n_kv_heads, int b, int kvh, int begin, int row_end,
                                                  const char *q_row, int n, int g, float scale2, float &m, float &l,
                                                  floatx4 (&acc)[D / 16])
{
    m = -INFINITY;
    l = 0.f;
#pragma unroll
    for (int dt = 0; dt < D / 16; ++dt) acc[dt] = floatx4{};
    const int32_t *blocks = kv.block_table ? kv.block_table + (int64_t)b * kv.max_blocks + (kv.first_block ? kv.first_block[b] : 0)
                                           : nullptr;
    auto row_bytes = [&](int tok) {              // where the token's row begins
        return (blocks ? ((int64_t)blocks[tok / kv.block_size] * n_kv_heads + kvh) * kv.block_size + tok % kv.block_size
                       : ((int64_t)b * n_kv_heads + kvh) * kv.cap + tok) * (D * 4);
    };
    auto rescale = [&](float mx) {               // the sums to the maximum of what was seen and mx; returns the shift
        const float m_new = fmaxf(m, mx), corr = m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((m - m_new) * scale2);
        m = m_new;
        l *= corr;
#pragma unroll
        for (int dt = 0; dt < D / 16; ++dt) acc[dt] *= corr;
        return m == -INFINITY ? 0.f : m;
    };
    const int all_end = __builtin_amdgcn_readlane(row_end, 0), any_end = __builtin_amdgcn_readlane(row_end, kF32Rows - 1);
    int tok = begin;
#pragma unroll 1
    for (; tok + 16 <= all_end; tok += 16) {     // 16 tokens from a multiple of 16 lie in one block
        const int64_t at = row_bytes(tok);
        const floatx4 s = scores_f32<D>(kv.k + at + n * (D * 4) + 16 * g, q_row + 16 * g);       // of tokens 4 g + i
        const LanePair x = rows_of(fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3]))), y = halves_of(fmaxf(x.a, x.b));
        const float m0 = rescale(fmaxf(y.a, y.b));
        float p[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            p[i] = __builtin_amdgcn_exp2f((s[i] - m0) * scale2);
            l += p[i];
        }
        const char *v = kv.v + at + 4 * g * (D * 4) + 4 * n;
#pragma unroll
        for (int dt = 0; dt < D / 16; ++dt) {
            floatx4 part = {};
#pragma unroll
            for (int i = 0; i < 4; ++i)
                part = __builtin_amdgcn_mfma_f32_16x16x4f32(*reinterpret_cast<const float *>(v + i * (D * 4) + 64 * dt), p[i], part, 0, 0, 0);
            acc[dt] += part;
        }
    }
#pragma unroll 1
    for (; tok < any_end; ++tok) {
        const int64_t at = row_bytes(tok);
        float s = 0.f;
#pragma unroll 2
        for (int i = g; i < D / 4; i += 4) {
            const float4 x = *reinterpret_cast<const float4 *>(kv.k + at + 16 * i), y = *reinterpret_cast<const float4 *>(q_row + 16 * i);
            s = fmaf(x.w, y.w, fmaf(x.z, y.z, fmaf(x.y, y.y, fmaf(x.x, y.x, s))));
        }
        s = strided_sum<16>(s);
        if (tok >= row_end) continue;
        const float p = __builtin_amdgcn_exp2f((s - rescale(s)) * scale2);
        l += g ? 0.f : p;
#pragma unroll
        for (int dt = 0; dt < D / 16; ++dt) {
            const floatx4 x = __builtin_bit_cast(floatx4, load16(kv.v + at + 64 * dt + 16 * g));
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[dt][i] = fmaf(p, x[i], acc[dt][i]);
        }
    }
}

// A workgroup: eight waves of 16 query rows over one share of the tokens of one (sequence, KV head), tile by tile.  K and V
// reach LDS as parts: every value is taken apart once per workgroup (5.5 vector instructions; by each wave for itself, from an fp32
// tile in LDS, they took longer than the products).  A tile's rows travel while the tile before the one before is worked
// on, are taken apart beside the products of the tile in between and stored to the buffer that was read last a tile ago:
// one barrier per tile.  Two waves share a SIMD, and one's products hide the other's waits (four waves of 32 rows have half the
// LDS reads and the registers of one wave per SIMD: every read and every conversion then stands between two products).
template <int D, bool TWO>
__global__ __launch_bounds__(kF32Block, 2) void append_attn_f32_kernel(AppendArgs a1, AppendArgs a2, LineDev line, QueryScale qs)
{
    using P = PartStage<D>;
    using S = typename P::S;
    constexpr int KK = D / 32, DT = D / 16;      // slices of the score contraction, 16-column tiles of the output
    constexpr float kLog2e = 1.4426950408889634f;
    __shared__ __attribute__((aligned(1024))) char s_a[P::kBytes];
    __shared__ __attribute__((aligned(1024))) char s_b[P::kBytes];
    __shared__ uint32_t s_row[kSub];

    const int group = a1.sh.group, n_rows = a1.n_q * group;
    const int n_qb = (n_rows + kRowsPerBlock - 1) / kRowsPerBlock;
    int share = blockIdx.x, kvh = blockIdx.y, b = blockIdx.z, qb = 0;
    if (n_qb > 1) {                              // uniform over the launch: a flat grid, numbered as in append_attn_kernel
        const int wg = (int)blockIdx.x, stream = wg % kXcds + kXcds * (wg / kXcds / n_qb);
        if (stream >= line.shares * a1.sh.n_kv_heads * a1.sh.batch) return;      // uniform over the workgroup
        qb = wg / kXcds % n_qb;
        share = stream % line.shares;
        kvh = stream / line.shares % a1.sh.n_kv_heads;
        b = stream / line.shares / a1.sh.n_kv_heads;
    }
    const int tid = threadIdx.x, lane = tid % kWave, w = __builtin_amdgcn_readfirstlane(tid / kWave), n = lane % 16, g = lane / 16;
    const int row0 = qb * kRowsPerBlock + w * kF32Rows;          // first row of the wave
    const bool wave_live = row0 < n_rows;                        // uniform over the wave
    const bool row_exists = row0 + n < n_rows;                   // lanes without a row repeat the last one and store nothing
    const int r = min(row0 + n, n_rows - 1), query = r / group;
    const int64_t out_row = ((int64_t)b * a1.n_q + query) * a1.sh.n_q_heads + kvh * group + r % group;
    const char *q_row = static_cast<const char *>(a1.q) + out_row * (D * 4);
    Parts q[KK];                                 // B operand: columns 32 kk + 8 g .. + 7 of the lane's row
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) q[kk] = query_parts(q_row + 128 * kk + 32 * g, a1.sh.sm_scale, qs.up);
    // scores stay raw, but for the queries' power of two; e^{scale (s - m)} = 2^{(s - m) scale2}
    const float scale2 = qs.scale * kLog2e;

    // what the thread brings in: K rows as they stand, V rows in quads (the order in which their stage holds them)
    constexpr int kQuadLanes = 4 * S::kRowBytes / 16;
    const bool brings = tid < P::kPieces;        // uniform over the wave
    const int k_row = tid / (D / 8) % kTile, k_piece = tid % (D / 8);
    const int v_row = (w * S::kGroupRows + 4 * (lane / kQuadLanes) + lane % 8 / 2) % kTile;
    const int v_piece = 2 * (lane % kQuadLanes / 8) + lane % 2;
    const int k_put = S::k_offset(k_row, k_piece), v_put = P::v_offset(v_row, v_piece / 2) + 16 * (v_piece % 2);
    // where the operands of a tile's products stand: token n of 16, columns 32 kk + 8 g; four tokens of a quad, 16 columns
    int k_lane[KK];
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) k_lane[kk] = S::k_offset(n, 4 * kk + g);
    const int v_lane = P::v_offset(4 * g + n / 4, 0) + 8 * (n % 4);

    const LineCut cut(line, b);
    const int line_begin = share * cut.share_steps, line_end = line_begin + cut.share_steps;
#pragma unroll 1
    for (int tier = 0; tier < (TWO ? 2 : 1); ++tier) {
        // the tier's part of the share, see LineDev; all uniform
        if (TWO && tier == 0 && line_begin > cut.first_steps) continue;
        if (tier == 1 && line_end <= cut.first_steps && share != line.shares - 1) continue;
        const KvDev kv = tier ? a2.kv : a1.kv;
        const int causal_tail = tier ? a2.causal_tail : a1.causal_tail;
        const int before = tier ? cut.first_steps : 0, slot = share + tier;
        const int len = tier_len(kv, b);
        const int t0 = max(line_begin - before, 0) * kStepTokens;
        const int nt_total = min(max(line_end - before, 0) * kStepTokens, len) - t0;             // <= 0: nothing of the share is valid
        // tokens [0, vis) of the tier are visible to the row; tiles below vis_min, that of the wave's first row, need no mask
        const int vis = causal_tail ? min(max(len - a1.n_q + query + 1, 0), len) : len;
        const int vis_min = causal_tail ? min(max(len - a1.n_q + min(row0 / group, a1.n_q - 1) + 1, 0), len) : len;
        float m = -INFINITY, l = 0.f;            // l: over this lane's tokens only
        floatx4 acc[DT], part[DT];               // the sums, and those of the last two tiles: shorter chains of additions
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) acc[dt] = part[dt] = floatx4{};
        auto flush = [&]() __attribute__((always_inline)) {
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) {
                acc[dt] += part[dt];
                part[dt] = floatx4{};
            }
        };

        const int sub_len = pass_length(kv, nt_total);
        for (int sub0 = 0; sub0 < nt_total; sub0 += sub_len) {
            const int nsub = min(sub_len, nt_total - sub0);
            __syncthreads();                     // the previous table and tiles are no longer in use
            const BlockRows rows = make_block_rows<kF32Block>(s_row, kv, a1.sh.n_kv_heads, b, kvh, t0 + sub0, nsub);
            const int tiles = (nsub + kTile - 1) / kTile;
            uint4 raw[2][2];                     // the next tile's piece of K and of V
            auto request = [&](int tile) __attribute__((always_inline)) {
                if (!brings) return;
                auto row_of = [&](int t) {       // tokens behind the end read the last row
                    const uint32_t at = min(tile * kTile + t, nsub - 1);
                    return rows.table ? rows.table[at / kGranule] + at % kGranule : rows.base + at;
                };
                const char *k = kv.k + (size_t)row_of(k_row) * (D * 4) + 32 * k_piece;
                const char *v = kv.v + (size_t)row_of(v_row) * (D * 4) + 32 * v_piece;
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    raw[0][e] = load16(k + 16 * e);
                    raw[1][e] = load16(v + 16 * e);
                }
            };
            auto take_apart = [&](int i, char *stage) __attribute__((always_inline)) {
                const Parts p = parts_of(raw[i][0], raw[i][1]);
                char *at = stage + (i ? v_put : k_put);
                *reinterpret_cast<u32x4 *>(at) = p.h;
                *reinterpret_cast<u32x4 *>(at + P::kPart) = p.m;
                *reinterpret_cast<u32x4 *>(at + 2 * P::kPart) = p.l;
            };
            auto work = [&](int tile, const char *cur, char *next) __attribute__((always_inline)) {
                __syncthreads();                 // the tile is complete, and nobody reads the other buffer any more
                if (brings && tile + 1 < tiles) {
                    take_apart(0, next);
                    take_apart(1, next);
                    request(tile + 2);
                }
                if (!wave_live) return;
                // scores: c[t][i] belongs to token 16 t + 4 g + i of the tile and the lane's row
                TileSums ts[2];
                ts[0].clear();
                ts[1].clear();
                Parts kf[KK][2];
                auto read_k = [&](int kk) __attribute__((always_inline)) {
#pragma unroll
                    for (int t = 0; t < 2; ++t) {
                        const char *at = cur + k_lane[kk] + t * 16 * S::kRowBytes;
                        kf[kk][t].h = *reinterpret_cast<const u32x4 *>(at);
                        kf[kk][t].m = *reinterpret_cast<const u32x4 *>(at + P::kPart);
                        kf[kk][t].l = *reinterpret_cast<const u32x4 *>(at + 2 * P::kPart);
                    }
                };
                read_k(0);
#pragma unroll
                for (int kk = 0; kk < KK; ++kk) {
                    if (kk + 1 < KK) read_k(kk + 1);
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int j = 0; j < 6; ++j)
#pragma unroll
                        for (int t = 0; t < 2; ++t) ts[t].add(kf[kk][t], q[kk], kk, j);
                    __builtin_amdgcn_sched_barrier(0);
                }
                short4v half[DT][6];
                auto read_v = [&](int dt) __attribute__((always_inline)) {
#pragma unroll
                    for (int j = 0; j < 6; ++j)
                        half[dt][j] = lds_read_tr16(cur + j / 2 * P::kPart + j % 2 * 16 * S::kRowBytes + (v_lane ^ 128 * (dt % 2)) + 256 * (dt / 2));
                };
                read_v(0);                       // the first V rows travel while the weights are formed
                float c[8] = {};
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    const floatx4 x = ts[t].sum();
#pragma unroll
                    for (int i = 0; i < 4; ++i) c[4 * t + i] = x[i];
                }
                const int step0 = t0 + sub0 + tile * kTile, in_pass = nsub - tile * kTile;
                if (min(in_pass, vis_min - step0) < kTile) {         // uniform over the wave: a length or causal boundary
                    int limit = min(in_pass, vis - step0);
                    asm volatile("" : "+v"(limit));                  // a real branch
#pragma unroll
                    for (int i = 0; i < 8; ++i)
                        if (16 * (i / 4) + 4 * g + i % 4 >= limit) c[i] = -INFINITY;
                }
                float mx = c[0];
#pragma unroll
                for (int i = 1; i < 8; ++i) mx = fmaxf(mx, c[i]);
                if (__any(mx > m)) {                                 // uniform over the wave
                    const LanePair x = rows_of(mx), y = halves_of(fmaxf(x.a, x.b));
                    const float m_new = fmaxf(m, fmaxf(y.a, y.b));
                    const float corr = m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((m - m_new) * scale2);
                    m = m_new;
                    l *= corr;
                    flush();
#pragma unroll
                    for (int dt = 0; dt < DT; ++dt) acc[dt] *= corr;
                }
                const float m0 = m == -INFINITY ? 0.f : m;           // s - m first: the difference is exact to its own size
#pragma unroll
                for (int i = 0; i < 8; ++i) c[i] = __builtin_amdgcn_exp2f((c[i] - m0) * scale2);
                l += ((c[0] + c[1]) + (c[2] + c[3])) + ((c[4] + c[5]) + (c[6] + c[7]));
                Parts p;                         // contraction index 8 g + i is token 16 (i / 4) + 4 g + i % 4
#pragma unroll
                for (int e = 0; e < 4; ++e) pair_parts(p, e, c[2 * e] * kUp, c[2 * e + 1] * kUp);
#pragma unroll
                for (int dt = 0; dt < DT; ++dt) {
                    if (dt + 1 < DT) read_v(dt + 1);
                    __builtin_amdgcn_sched_barrier(0);
                    auto v_part = [&](int i) __attribute__((always_inline)) {
                        const short4v x0 = half[dt][2 * i], x1 = half[dt][2 * i + 1];
                        const short8v both = {x0[0], x0[1], x0[2], x0[3], x1[0], x1[1], x1[2], x1[3]};
                        return __builtin_bit_cast(u32x4, both);
                    };
                    part[dt] = mfma(v_part(2), p.h, part[dt]);
                    part[dt] = mfma(v_part(0), p.l, part[dt]);
                    part[dt] = mfma(v_part(1), p.m, part[dt]);
                    part[dt] = mfma(v_part(1), p.h, part[dt]);
                    part[dt] = mfma(v_part(0), p.m, part[dt]);
                    part[dt] = mfma(v_part(0), p.h, part[dt]);
                    __builtin_amdgcn_sched_barrier(0);
                }
            };
            request(0);
            if (brings) {
                take_apart(0, s_a);
                take_apart(1, s_a);
            }
            request(1);
#pragma unroll 1
            for (int tile = 0; tile < tiles; tile += 2) {
                work(tile, s_a, s_b);
                if (tile + 1 < tiles) work(tile + 1, s_b, s_a);
                flush();
            }
        }

        // A weight of 0 keeps a V row out of the products above only while the row is finite (0 * inf is NaN), and values that are
        // not finite, or too large or too small, have no parts: where sums are not finite, or next to nothing, the wave works its share
        // out again.
        m *= qs.up == kUp ? kDown : 1.f;
        if (wave_live && nt_total > 0) {         // uniform over the wave
            float not_finite = l * 0.f, least = INFINITY;            // (the product with 0 is NaN then)
#pragma unroll
            for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    acc[dt][i] *= kDown;
                    not_finite = fmaf(acc[dt][i], 0.f, not_finite);
                    least = fminf(least, fabsf(acc[dt][i]));
                }
            const int row_end = min(t0 + nt_total, vis);
            bool again = not_finite != 0.f || (m == -INFINITY && row_end > t0);      // (scores of -inf alone: sums that overflowed)
            if (__any(least < kLeast)) {         // 0 is no small one
#pragma unroll
                for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                    for (int i = 0; i < 4; ++i) again |= acc[dt][i] != 0.f && fabsf(acc[dt][i]) < kLeast;
            }
            if (__any(again)) {
                int lane_of = lane;              // nothing of this is worked out, and held in registers, before it is wanted
                int64_t at = out_row;
                asm volatile("" : "+v"(lane_of), "+v"(at));
                append_rows_again<D>(kv, a1.sh.n_kv_heads, b, kvh, t0, row_end, static_cast<const char *>(a1.q) + at * (D * 4),
                                     lane_of % 16, lane_of / 16, a1.sh.sm_scale * kLog2e, m, l, acc);
            }
        }

        // partial of every valid row: the lane holds output columns 16 dt + 4 g .. + 3 of its row
        l = strided_sum<16>(l);
        if (row_exists) {
            const int64_t at = out_row * a1.part.stride + slot;
#pragma unroll
            for (int dt = 0; dt < DT; ++dt)
                *reinterpret_cast<floatx4 *>(a1.part.o + at * D + 16 * dt + 4 * g) = acc[dt];
            if (g == 0) {
                a1.part.m[at] = (m == -INFINITY) ? -INFINITY : m * a1.sh.sm_scale;     // the shift of the weights, in scaled scores
                a1.part.l[at] = l;
            }
        }
    }
}

// ---- weights ---------------------------------------------------------------------------------------------------

// Query-averaged softmax weights of a tier, as append_weights_kernel forms them: a token per lane (A = Q, B = K), a wave takes
// 32-token tiles of its own and meets all rows.  The queries stay in LDS as parts, 128 rows at a time; a tile's K rows go from
// memory to the lanes that need them and are taken apart there, once for all rows.
template <int D> struct WeightsF32 {
    static constexpr int kWaves = 8, kBlock = kWaves * kWave;
    static constexpr int kRowBytes = D * 2, kPieces = D / 8, kSwizzled = kPieces < 16 ? kPieces : 16;
    static constexpr int kPart = kRowsPerBlock * kRowBytes;
    static __device__ __forceinline__ int offset(int row, int piece) {
        return row * kRowBytes + 16 * (piece ^ (row / (16 / kSwizzled)) % kSwizzled);
    }
};

// e^x for x <= 0 or thereabouts: 2^(x log2 e) with the rounding error of the product put right.  A few 2^-24 off where the
// product alone would be |x| 2^-24 off.
__device__ __forceinline__ float exp_of(float x)
{
    constexpr float kHi = 1.44269502162933349609f, kLo = 1.92596299112661746887e-8f, kLn2 = 0.69314718055994530942f;
    const float t = x * kHi, rest = fmaf(x, kLo, fmaf(x, kHi, -t)), e = __builtin_amdgcn_exp2f(t);
    return fmaf(e, rest * kLn2, e);
}
constexpr float kNoRow = -1e30f;                 // shift of a row that does not exist: weighs nothing, and exp_of stays a number

template <int D, int G, bool TWO>
__global__ __launch_bounds__(WeightsF32<D>::kBlock, 2) void append_weights_f32_kernel(AppendArgs a1, AppendArgs a2, LineDev line,
                                                                                 QueryScale qs)
{
    using W = WeightsF32<D>;
    constexpr int kWWaves = W::kWaves, kWBlock = W::kBlock, KK = D / 32, NS = G < 4 ? G : 4;
    constexpr int kSpreadLive = 2;               // row tiles from which dealing them out to idle waves pays
    __shared__ __attribute__((aligned(1024))) char s_q[3 * W::kPart];
    __shared__ __attribute__((aligned(16))) float s_shift[kRowsPerBlock];        // minus the rows' lse
    __shared__ float s_red[kWWaves][2 * NS][kWave];
    __shared__ uint32_t s_row[kSub];

    const int share = blockIdx.x, kvh = blockIdx.y, b = blockIdx.z;
    const int tid = threadIdx.x, lane = tid % kWave, w = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int n = lane % 16, lg = lane / 16;
    const int n_rows = a1.n_q * G, n_qb = (n_rows + kRowsPerBlock - 1) / kRowsPerBlock;
    const float inv_n = 1.f / (float)a1.n_q;
    const int frag0 = W::offset(n, lg);          // operand of row n of 16; slice kk is an exclusive-or of 64 kk away

    const LineCut cut(line, b);
    int q_held = -1;                             // block of rows that s_q holds
#pragma unroll 1
    for (int tier = 0; tier < (TWO ? 2 : 1); ++tier) {
        const KvDev kv = tier ? a2.kv : a1.kv;
        const int causal_tail = tier ? a2.causal_tail : a1.causal_tail, first_step = tier ? cut.first_steps : 0;
        const float *lse = tier ? a2.lse : a1.lse;
        const int len = tier_len(kv, b);
        float *out = (tier ? a2.a_out : a1.a_out) + ((int64_t)b * a1.sh.n_q_heads + kvh * G) * kv.cap;

        // entries beyond the sequence's length, shared out as well
        for (int g = 0; g < G; ++g)
            for (int j = len + share * kWBlock + tid; j < kv.cap; j += line.shares * kWBlock) out[(int64_t)g * kv.cap + j] = 0.f;

        const int begin = share * cut.share_steps;
        const int t0 = max(begin - first_step, 0) * kStepTokens;
        const int t_end = min(max(begin + cut.share_steps - first_step, 0) * kStepTokens, len);
        if (t0 >= t_end) continue;               // nothing of this tier in the share (uniform over the workgroup)
        const int pass_len = min(pass_length(kv, t_end - t0), n_qb > 1 ? kWManyRowTokens : INT32_MAX);
        for (int p0 = t0; p0 < t_end; p0 += pass_len) {
            const int nt = min(pass_len, t_end - p0), tiles = (nt + kWTile - 1) / kWTile;
            __syncthreads();                     // the table of the previous pass is no longer in use
            const BlockRows rows = make_block_rows<kWBlock>(s_row, kv, a1.sh.n_kv_heads, b, kvh, p0, nt);
            auto k_row = [&](int tile, int t) {  // of the lane's token of the t-th 16; tokens behind the end read the last row
                const uint32_t at = min(tile * kWTile + 16 * t + n, nt - 1);
                return kv.k + (size_t)(rows.table ? rows.table[at / kGranule] + at % kGranule : rows.base + at) * (D * 4);
            };
            uint4 raw[2][KK][2];                 // columns 32 kk + 8 lg .. + 7 of the lane's two tokens
            auto request = [&](int tile) {
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    const char *src = k_row(tile, t) + 32 * lg;
#pragma unroll
                    for (int kk = 0; kk < KK; ++kk) {
                        raw[t][kk][0] = load16(src + 128 * kk);
                        raw[t][kk][1] = load16(src + 128 * kk + 16);
                    }
                }
            };
            for (int qb = 0; qb < n_qb; ++qb) {
                __syncthreads();                 // the queries and shifts of the previous round are no longer in use
                const int live = (min(n_rows - qb * kRowsPerBlock, kRowsPerBlock) + 31) / 32;        // 32-row tiles with rows that exist
                // a block with fewer tiles than there are waves: several waves take a tile's rows in turn and add up at the end
                const int spread_bits = live < kSpreadLive ? 0 : 4 * tiles <= kWWaves ? 2 : 2 * tiles <= kWWaves ? 1 : 0;
                const int spread = 1 << spread_bits, part = w % spread, tile_first = w >> spread_bits, tile_step = kWWaves >> spread_bits;
                if (tile_first < tiles) request(tile_first);     // first: it has the longest way
                if (q_held != qb) {              // uniform over the workgroup
                    for (int i = tid; i < live * 32 * W::kPieces; i += kWBlock) {
                        const int row = i / W::kPieces, piece = i % W::kPieces, at = qb * kRowsPerBlock + row;
                        // rows that do not exist repeat the last query of their head and weigh nothing
                        const int r = at < n_rows ? at : n_rows - G + at % G;
                        const char *src = static_cast<const char *>(a1.q) +
                                          (((int64_t)b * a1.n_q + r / G) * a1.sh.n_q_heads + kvh * G + r % G) * (D * 4) + 32 * piece;
                        const Parts p = query_parts(src, a1.sh.sm_scale, qs.up);
                        char *dst = s_q + W::offset(row, piece);
                        *reinterpret_cast<u32x4 *>(dst) = p.h;
                        *reinterpret_cast<u32x4 *>(dst + W::kPart) = p.m;
                        *reinterpret_cast<u32x4 *>(dst + 2 * W::kPart) = p.l;
                    }
                    q_held = qb;
                }
                if (tid < kRowsPerBlock) {
                    const RowInfo ri = row_info<G>(a1, b, kvh, qb * kRowsPerBlock + tid);
                    const float row_lse = ri.valid ? lse[ri.out_row] : 0.f;
                    // a row that sees nothing has lse = -inf; its weights are left out below, whatever the shift
                    s_shift[tid] = !ri.valid ? kNoRow : row_lse == -INFINITY ? 0.f : -row_lse;
                }
                __syncthreads();

                // tokens that all rows of the block see (tokens behind the length are not stored and need no mask)
                const int seen_by_all = causal_tail ? len - a1.n_q + qb * kRowsPerBlock / G + 1 : INT32_MAX;
                float done[2][NS] = {};          // of the t-th 16 tokens: head i (G = 8: head 4 (lg % 2) + i)
                int done_at = -1;
                auto store = [&]() {             // every lane has the sums of its token: the groups of 16 lanes share them out
#pragma unroll
                    for (int t = 0; t < 2; ++t)
#pragma unroll
                        for (int i = 0; i < NS; ++i) {
                            if (G < 8 ? (t * NS + i) % 4 != lg : lg / 2 != t) continue;
                            const int at = done_at + 16 * t + n;
                            if (done_at < 0 || at >= t_end) continue;
                            float *dst = out + (int64_t)(G == 8 ? 4 * (lg % 2) + i : i) * kv.cap + at;
                            *dst = qb == 0 ? done[t][i] * inv_n : fmaf(done[t][i], inv_n, *dst);
                        }
                };
                for (int tile = tile_first; tile < tiles; tile += tile_step) {
                    if (tile != tile_first) request(tile);
                    Parts kf[2][KK];
#pragma unroll
                    for (int t = 0; t < 2; ++t)
#pragma unroll
                        for (int kk = 0; kk < KK; ++kk) kf[t][kk] = parts_of(raw[t][kk][0], raw[t][kk][1]);
                    const int tok0 = p0 + tile * kWTile;
                    // Row r of the block sees token k iff r / G >= k - (len - n_q): the first row that sees the lane's first token
                    const bool cut_tile = tok0 + kWTile > seen_by_all;               // uniform over the wave
                    const int first_row = cut_tile ? G * (tok0 + n - (len - a1.n_q)) - qb * kRowsPerBlock : INT32_MIN / 2;
                    float sum[2][NS] = {};
#pragma unroll 1
                    for (int x = part; x < 2 * live; x += spread) {                  // 16 rows at a time
                        // the score of row 16 x + 4 lg + i and the lane's t-th token
                        TileSums ts[2];
                        ts[0].clear();
                        ts[1].clear();
#pragma unroll
                        for (int kk = 0; kk < KK; ++kk) {
                            const char *at = s_q + x * 16 * W::kRowBytes + (frag0 ^ (64 * kk));
                            const Parts q = {*reinterpret_cast<const u32x4 *>(at), *reinterpret_cast<const u32x4 *>(at + W::kPart),
                                             *reinterpret_cast<const u32x4 *>(at + 2 * W::kPart)};
#pragma unroll
                            for (int j = 0; j < 6; ++j)
#pragma unroll
                                for (int t = 0; t < 2; ++t) ts[t].add(q, kf[t][kk], kk, j);
                        }
                        const float4 sh = *reinterpret_cast<const float4 *>(s_shift + 16 * x + 4 * lg);
                        const float s4[4] = {sh.x, sh.y, sh.z, sh.w};
#pragma unroll
                        for (int t = 0; t < 2; ++t) {
                            const floatx4 c = ts[t].sum();
#pragma unroll
                            for (int i = 0; i < 4; ++i) {                            // the head of row r is r % G
                                const float e = exp_of(fmaf(c[i], qs.scale, s4[i]));
                                sum[t][i % NS] += !cut_tile || 16 * x + 4 * lg + i >= first_row + G * 16 * t ? e : 0.f;
                            }
                        }
                    }
                    bool finite = true;
#pragma unroll
                    for (int t = 0; t < 2; ++t)
#pragma unroll
                        for (int i = 0; i < NS; ++i) finite &= fabsf(sum[t][i]) < INFINITY;
                    if (__any(!finite)) {        // values without parts: these sums again with fp32 products
                        float again[2][NS] = {};
#pragma unroll 1
                        for (int x = part; x < 2 * live; x += spread) {
                            const int at = qb * kRowsPerBlock + 16 * x + n, r = at < n_rows ? at : n_rows - G + at % G;
                            const char *q = static_cast<const char *>(a1.q) +
                                            (((int64_t)b * a1.n_q + r / G) * a1.sh.n_q_heads + kvh * G + r % G) * (D * 4);
#pragma unroll
                            for (int t = 0; t < 2; ++t) {
                                const floatx4 c = scores_f32<D>(q + 16 * lg, k_row(tile, t) + 16 * lg);
#pragma unroll
                                for (int i = 0; i < 4; ++i) {
                                    const int row = 16 * x + 4 * lg + i;
                                    const float e = expf(fmaf(c[i], a1.sh.sm_scale, s_shift[row]));
                                    again[t][i % NS] += qb * kRowsPerBlock + row < n_rows && (!cut_tile || row >= first_row + G * 16 * t) ? e : 0.f;
                                }
                            }
                        }
#pragma unroll
                        for (int t = 0; t < 2; ++t)
#pragma unroll
                            for (int i = 0; i < NS; ++i) sum[t][i] = fabsf(sum[t][i]) < INFINITY ? sum[t][i] : again[t][i];
                    }
                    // rows of a head lie in all four groups of lanes (G = 8: in every second one)
#pragma unroll
                    for (int t = 0; t < 2; ++t)
#pragma unroll
                        for (int i = 0; i < NS; ++i) done[t][i] = G < 8 ? strided_sum<16>(sum[t][i]) : halves_sum(sum[t][i]);
                    done_at = tok0;
                    if (spread == 1) store();
                }
                if (spread > 1) {                // uniform over the workgroup; a wave has met one tile at most
#pragma unroll
                    for (int i = 0; i < 2 * NS; ++i) s_red[w][i][lane] = done[i / NS][i % NS];
                    __syncthreads();
                    for (int k = 1; part == 0 && k < spread; ++k)
#pragma unroll
                        for (int i = 0; i < 2 * NS; ++i) done[i / NS][i % NS] += s_red[w + k][i][lane];
                    if (part != 0) done_at = -1;
                    store();
                }
            }
        }
    }
}

template <int D>
hipError_t launch_attn(const AppendArgs &a, const AppendArgs &a2, const LineDev &line, int two, dim3 grid, hipStream_t s)
{
    if (two) hipLaunchKernelGGL((append_attn_f32_kernel<D, true>), grid, dim3(kF32Block), 0, s, a, a2, line, query_scale(a.sh.sm_scale));
    else hipLaunchKernelGGL((append_attn_f32_kernel<D, false>), grid, dim3(kF32Block), 0, s, a, a2, line, query_scale(a.sh.sm_scale));
    return hipGetLastError();
}

template <int D, bool TWO>
hipError_t launch_weights(const AppendArgs &a, const AppendArgs &a2, const LineDev &line, dim3 grid, hipStream_t s)
{
    const dim3 block(WeightsF32<D>::kBlock);
    const QueryScale qs = query_scale(a.sh.sm_scale);
    switch (a.sh.group) {
    case 1: hipLaunchKernelGGL((append_weights_f32_kernel<D, 1, TWO>), grid, block, 0, s, a, a2, line, qs); break;
    case 2: hipLaunchKernelGGL((append_weights_f32_kernel<D, 2, TWO>), grid, block, 0, s, a, a2, line, qs); break;
    case 4: hipLaunchKernelGGL((append_weights_f32_kernel<D, 4, TWO>), grid, block, 0, s, a, a2, line, qs); break;
    case 8: hipLaunchKernelGGL((append_weights_f32_kernel<D, 8, TWO>), grid, block, 0, s, a, a2, line, qs); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace

hipError_t launch_append_attn_f32(int head_dim, const AppendArgs &a, const AppendArgs &a2, const LineDev &line, int two, dim3 grid,
                                  hipStream_t s)
{
    if (a.sh.group <= 0) return hipErrorInvalidValue;
    if (head_dim == 64) return launch_attn<64>(a, a2, line, two, grid, s);
    if (head_dim == 128) return launch_attn<128>(a, a2, line, two, grid, s);
    return hipErrorInvalidValue;
}

hipError_t launch_append_weights_f32(int head_dim, const AppendArgs &a, const AppendArgs &a2, const LineDev &line, int two,
                                     dim3 grid, hipStream_t s)
{
    if (head_dim == 64) return two ? launch_weights<64, true>(a, a2, line, grid, s) : launch_weights<64, false>(a, a2, line, grid, s);
    if (head_dim == 128) return two ? launch_weights<128, true>(a, a2, line, grid, s) : launch_weights<128, false>(a, a2, line, grid, s);
    return hipErrorInvalidValue;
}

}  // namespace hgca

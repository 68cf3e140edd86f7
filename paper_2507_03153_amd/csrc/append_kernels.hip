// Append stage: N queries per sequence attend to one KV tier (Sec. 2.1: S = Q K^T, A = softmax(S),
// O = A V with Q in R^{h x N x d}; Alg. 2, append branch), or to two.  Both contractions on the matrix
// cores; bf16 inputs (fp32 ones: append_f32_kernels.hip).
//
// Work unit of the attention kernel: one workgroup = one share of the tokens of one (sequence, KV head) and up to 128
// query rows (a row = one query x one head of the GQA group, query-major).  Every wave owns 32 rows, so nothing is
// reduced across waves.  The K and V rows of a 64-token step are brought into a double-buffered LDS stage by LDS-direct
// loads (no registers in between); the next step's loads are in flight during a step's arithmetic, one barrier per
// step; two workgroups share a CU.
//
// Orientation (per 32-row tile, per step):
//   S^T[token, row]  = K[token, :] . Q[row, :]        A = K tile (LDS, swizzled rows), B = Q (registers)
//   O^T[dcol, row]  += V^T[dcol, token] . P^T[token, row]   A = V^T (LDS transpose reads of the rows), B = P
// In both results a lane's column is the query row lane % 32, so the running maximum, the running sum and the
// rescaling factor of a row live in the lanes that hold its scores AND its output columns: the online softmax needs
// one lane exchange per row statistic and no LDS.  The probabilities go from the score registers straight into the B
// operand of the second contraction (the contraction index is matched by reading V^T in the same token order);
// they are rounded there, as a high and a low part (two MFMAs, fp32-level accuracy) or, on request, as one part.
//
// The weights kernel brings its K rows in the same way (it has no second contraction).
#include "append_device.hpp"

#include <algorithm>
#include <type_traits>

namespace hgca {

namespace {

constexpr int kNonTemporal = 2;                  // cache policy of a load: streamed once
constexpr int64_t kLastCache = int64_t(256) << 20;

// s_waitcnt vmcnt(0) (expcnt and lgkmcnt fields at their maxima = no wait): an LDS-direct load has landed in LDS
// when the wave's memory-load counter has counted it down.  Every wave does this before the barrier after which
// other waves read what it loaded.
__device__ __forceinline__ void wait_for_own_loads() { __builtin_amdgcn_s_waitcnt(0x0F70); }

// Requests the K and the V rows of a step.  A load instruction of a wave covers kGroupRows rows of one granule, so in
// a full step its address is a scalar (the granule's row) plus an offset that is the lane's for good; only a step
// that the pass's end cuts computes rows per lane (tokens behind the end read the last row).  The row numbers of a
// paged tier are looked up before the first load is issued: an LDS read placed after an LDS-direct load waits for it.
// POLICY_K and POLICY_V are the loads' cache policies: 0, or kNonTemporal where the rows are not to stay in the caches.
template <int D, int NW, int POLICY_K, int POLICY_V>
__device__ __forceinline__ void dma_step(const KvDev &kv, const BlockRows &rows, int step, int nsub, char *k_stage,
                                         char *v_stage)
{
    using S = DmaStage<D, NW>;
    static_assert(kGranule % S::kGroupRows == 0, "a load stays inside a granule");
    constexpr int kQuadLanes = 4 * S::kRowBytes / 16;
    const int lane = threadIdx.x % kWave, w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    // what lands at byte 16 * lane of the wave's u-th group: the row inside the group and the byte of the row
    const int k_row = lane / S::kPieces, v_row = 4 * (lane / kQuadLanes) + (lane % 8) / 2;
    auto k_byte = [&](int u) { return 16 * ((lane % S::kPieces) ^ S::k_swizzle((w + NW * u) * S::kGroupRows + k_row)); };
    const int v_byte = 16 * (2 * ((lane % kQuadLanes) / 8) + lane % 2);
    typedef const __attribute__((address_space(1))) void *GlobalPtr;
    typedef __attribute__((address_space(3))) void *LdsPtr;
    if ((step + 1) * kStepTokens <= nsub) {                      // uniform over the workgroup
        const int first = step * kStepTokens + w * S::kGroupRows;                        // of the wave's first load
        uint32_t row[S::kLoads];                                 // uniform over the wave
#pragma unroll
        for (int u = 0; u < S::kLoads; ++u) row[u] = rows.base + first + NW * S::kGroupRows * u;
        if (rows.table) {
#pragma unroll
            for (int u = 0; u < S::kLoads; ++u) row[u] = rows.table[(first + NW * S::kGroupRows * u) / kGranule];
#pragma unroll
            for (int u = 0; u < S::kLoads; ++u)
                row[u] = __builtin_amdgcn_readfirstlane(row[u]) + (first + NW * S::kGroupRows * u) % kGranule;
        }
#pragma unroll
        for (int u = 0; u < S::kLoads; ++u) {
            const size_t at = (size_t)row[u] * S::kRowBytes;
            const uint32_t k_off = k_row * S::kRowBytes + k_byte(u), v_off = v_row * S::kRowBytes + v_byte;
            __builtin_amdgcn_global_load_lds((GlobalPtr)(kv.k + at + k_off), (LdsPtr)(k_stage + (w + NW * u) * 1024), 16, 0, POLICY_K);
            __builtin_amdgcn_global_load_lds((GlobalPtr)(kv.v + at + v_off), (LdsPtr)(v_stage + (w + NW * u) * 1024), 16, 0, POLICY_V);
        }
        return;
    }
    uint32_t kr[S::kLoads], vr[S::kLoads];
#pragma unroll
    for (int u = 0; u < S::kLoads; ++u) {
        const int first = step * kStepTokens + (w + NW * u) * S::kGroupRows;
        const uint32_t kt = min(first + k_row, nsub - 1), vt = min(first + v_row, nsub - 1);
        kr[u] = rows.table ? rows.table[kt / kGranule] + kt % kGranule : rows.base + kt;
        vr[u] = rows.table ? rows.table[vt / kGranule] + vt % kGranule : rows.base + vt;
    }
#pragma unroll
    for (int u = 0; u < S::kLoads; ++u) {
        __builtin_amdgcn_global_load_lds((GlobalPtr)(kv.k + (size_t)kr[u] * S::kRowBytes + k_byte(u)),
                                         (LdsPtr)(k_stage + (w + NW * u) * 1024), 16, 0, 0);
        __builtin_amdgcn_global_load_lds((GlobalPtr)(kv.v + (size_t)vr[u] * S::kRowBytes + v_byte),
                                         (LdsPtr)(v_stage + (w + NW * u) * 1024), 16, 0, 0);
    }
}

// One 16-byte slice of the score contraction in bf16: C[32 x 32] += A . B over 16 columns.  A lane holds 16 bytes of row
// lane % 32 of either operand, the lower half of the wave one piece and the upper half the next.
__device__ __forceinline__ floatx16 score_mfma(const uint4 &a, const uint4 &b, floatx16 c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

constexpr int kWAhead = 2;                       // query pieces of the weights pass that are read ahead
constexpr int kAhead = 2;                        // slices of the score contraction whose K pieces are read ahead

// A workgroup: four waves of 32 query rows over one share of the tokens of one (sequence, KV head).  The scores come
// from v_mfma_f32_32x32x16_bf16, whose result gives a lane 16 scores of ONE row per 32 tokens (the other 16 are the
// lane's partner's, 32 lanes away), so a step's softmax is one chain per lane over 32 scores.  The pass is bound by power:
// the part lowers its clock to 1.7 - 2.0 GHz under it (a bare chain of these instructions runs at 1.8 GHz, 1.87 PFLOP/s,
// with four multiply-adds beside each 1.62), so what counts is work, and fewer cycles for the same work return a third
// of themselves in time.  Of 700 us for 2 x 509 queries on 32 K tokens the low parts' products take 120, the exponentials 43,
// the loads into LDS 80, the reads from LDS nothing.  Hence
//   - the maximum is reduced over the lanes, and the outputs rescaled, only in steps where some score exceeds its row's
//     maximum so far; the row sum stays per lane until the end of the share;
//   - the low part of a weight is a shift or a mask and a subtraction.  One v_dot2_f32_bf16 does the same in one instruction,
//     but it waits for the matrix pipe: 10 ns beside a matrix instruction of 14 where two multiply-adds hide;
//   - K pieces and V rows are read from LDS well before their products, and a workgroup that is ahead of the other one on its
//     unit steps back: waves in flight 79 -> 92 % on average (715 -> 697 us);
//   - a load instruction's address is a scalar plus a constant offset of the lane (dma_step);
//   about 7 vector instructions per score where the kernel with 16-row tiles took 13.
// 2 x 509 queries x 32 K tokens x 32 heads: 762 -> 712 us with the fold; 8 x 32 queries x 32 K tokens 261 -> 243;
// 48 queries, groups of 8, one part, 255 -> 249.
//
// A launch may serve TWO tiers (the complete pool and the window of an append turn: Alg. 2 runs the two attentions side
// by side) as one line of tokens cut into equal shares (LineDev): a workgroup goes through its part of the first tier
// and its part of the second, usually only one of them, each with the tier's view, mask rule and slot.
template <int D, int G, bool SPLIT_P, bool TWO>
__global__ __launch_bounds__(kAttnBlock, 2) void append_attn_kernel(AppendArgs a1, AppendArgs a2, LineDev line, int streamed,
                                                                    int kept_k)
{
    constexpr int NW = kAttnWaves, BLOCK = kAttnBlock;
    using S = DmaStage<D, NW>;
    constexpr int KK = D / 16;                  // slices of the score contraction
    constexpr int DT = D / 32, NT = kStepTokens / 32;            // 32-column tiles of the output, 32-token tiles of a step
    constexpr float kLog2e = 1.4426950408889634f;
    // two stages per tensor as separate arrays: the compiler then knows that a load into one stage does not
    // touch the other and lets the reads of the current stage go ahead while the next one is being filled
    __shared__ __attribute__((aligned(1024))) char s_k0[S::kBytes];
    __shared__ __attribute__((aligned(1024))) char s_k1[S::kBytes];
    __shared__ __attribute__((aligned(1024))) char s_v0[S::kBytes];
    __shared__ __attribute__((aligned(1024))) char s_v1[S::kBytes];
    __shared__ uint32_t s_row[kSub];

    // Workgroups are dealt to the XCDs in turn.  The row blocks of one stream of K/V rows (a split of a (sequence, KV
    // head)) read the same rows: they take numbers that are equal modulo the number of XCDs and follow each other
    // there, so that the stream passes through one L2.
    const int n_qb = (a1.n_q * G + kRowsPerBlock - 1) / kRowsPerBlock;
    int share = blockIdx.x, kvh = blockIdx.y, b = blockIdx.z, qb = 0;
    if (n_qb > 1) {                              // uniform over the launch: a flat grid
        const int wg = (int)blockIdx.x, stream = wg % kXcds + kXcds * (wg / kXcds / n_qb);
        if (stream >= line.shares * a1.sh.n_kv_heads * a1.sh.batch) return;      // uniform over the workgroup
        qb = wg / kXcds % n_qb;
        share = stream % line.shares;
        kvh = stream / line.shares % a1.sh.n_kv_heads;
        b = stream / line.shares / a1.sh.n_kv_heads;
    }
    const int tid = threadIdx.x, w = tid / kWave, lane = tid % kWave, n = lane % 32, hw = lane / 32;

    const int row0 = qb * kRowsPerBlock + __builtin_amdgcn_readfirstlane(w) * 32;        // first row of the wave
    const bool wave_live = row0 < a1.n_q * G;                    // uniform over the wave
    const bool row_exists = row0 + n < a1.n_q * G;               // lanes without a row repeat the last one and store nothing
    const RowInfo ri = row_info<G>(a1, b, kvh, min(row0 + n, a1.n_q * G - 1));
    uint4 qop[KK];                               // B operand: piece 2 kk + hw of the lane's row
#pragma unroll
    for (int kk = 0; kk < KK; ++kk)
        qop[kk] = load16(static_cast<const char *>(a1.q) + ri.out_row * S::kRowBytes + 16 * (2 * kk + hw));
    // The running maximum is kept on the RAW scores (the softmax scale is positive, so the order is the same) and
    // the scale, in units of ln 2, is applied inside the exponent: e^{scale (s - m)} = 2^{fma(s, scale2, -m scale2)},
    // one fused multiply-add and one bare v_exp_f32 per score.
    const float scale2 = a1.sh.sm_scale * kLog2e;
    // this lane's byte offsets into a stage: the A operand of the first product (row n of a 32-token tile, one
    // offset per 16-column slice because of the swizzle) and of the second.  The V^T operand (8 tokens of one column
    // per lane) comes from two transpose reads: lane j of a 16-lane group points at columns 4(j%4).. of row j/4 of a
    // quad of tokens, the two groups of a half wave at neighbouring column chunks.
    int k_lane[KK];
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) k_lane[kk] = S::k_offset(n, 2 * kk + hw);
    const int v_lane = S::v_offset(4 * hw + lane % 16 / 4, lane / 16 % 2) + 8 * (lane % 4);
    const LineCut cut(line, b);
    // one tier's part of the share: steps [step_begin, step_end) of the tier, which go to `slot` (see LineDev); all uniform
    auto serve = [&](const AppendArgs &a, int step_begin, int step_end, int slot) {
        const KvDev &kv = a.kv;
        const int causal_tail = a.causal_tail;
        const int len = tier_len(kv, b);
        const int t0 = step_begin * kStepTokens;
        const int nt_total = min(step_end * kStepTokens, len) - t0;              // <= 0: nothing of the share is valid
        // tokens [0, vis) of the tier are visible to the row; steps below vis_min, that of the wave's first row (rows are
        // query-major), need no mask
        const int vis = causal_tail ? min(max(len - a1.n_q + ri.query + 1, 0), len) : len;
        const int vis_min = causal_tail ? min(max(len - a1.n_q + min(row0 / G, a1.n_q - 1) + 1, 0), len) : len;
        float m = -INFINITY, shift = 0.f, l = 0.f;               // l: over this lane's tokens only
        floatx16 acc[DT];
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) acc[dt] = floatx16{};

        auto step_body = [&](const char *k_stage, const char *v_stage, int step0, int in_split) {
            // raw scores: c[t][r] belongs to step token 32 t + 8 (r / 4) + 4 hw + r % 4 and the lane's row
            floatx16 c[NT];
#pragma unroll
            for (int t = 0; t < NT; ++t) c[t] = floatx16{};
            auto k_piece = [&](int t, int kk) {
                return *reinterpret_cast<const uint4 *>(k_stage + t * 32 * S::kRowBytes + k_lane[kk]);
            };
            // a slice's K pieces are read kAhead slices before the matrix instructions that take them (the scheduler, left
            // alone, puts the reads right before their use, and every pair of instructions waits for LDS)
            uint4 kf[KK][NT];
            auto read_slice = [&](int kk) {
#pragma unroll
                for (int t = 0; t < NT; ++t) kf[kk][t] = k_piece(t, kk);
            };
#pragma unroll
            for (int kk = 0; kk < kAhead; ++kk) read_slice(kk);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int kk = 0; kk < KK; ++kk) {
                if (kk + kAhead < KK) read_slice(kk + kAhead);
#pragma unroll
                for (int t = 0; t < NT; ++t) c[t] = score_mfma(kf[kk][t], qop[kk], c[t]);        // the accumulators take turns
                __builtin_amdgcn_sched_barrier(0);
            }
            bf16x8 vop[2][DT];
            auto read_v = [&](int g, bf16x8 (&x)[DT]) {
                const char *v = v_stage + S::v_offset(16 * g, 0) + v_lane;
#pragma unroll
                for (int dt = 0; dt < DT; ++dt) {
                    const short4v x0 = lds_read_tr16(v + 256 * dt), x1 = lds_read_tr16(v + S::v_offset(8, 0) + 256 * dt);
                    const short8v both = {x0[0], x0[1], x0[2], x0[3], x1[0], x1[1], x1[2], x1[3]};
                    x[dt] = __builtin_bit_cast(bf16x8, both);
                }
            };
            // With the weights in two parts, heads of 64 are better without the reads ahead: the fences between the groups cost more than
            // they save where several blocks of rows share K and V (5 sequences of 40 heads, 144 queries, whole turn 497 -> 520 us, 480 without;
            // 200 queries x 4 heads 529 -> 546, 492; one block of rows the same within 1 %).  In one part heads of 64 gain 2 to 5 % from them,
            // heads of 128 1 to 3 %.
            constexpr bool kReadAheadV = D > 64 || !SPLIT_P;
            if constexpr (kReadAheadV) {             // the first V rows travel while the maxima are formed
                read_v(0, vop[0]);
                __builtin_amdgcn_sched_barrier(0);
            }
            if (min(in_split, vis_min - step0) < kStepTokens) {      // uniform over the wave: a length or causal boundary
                int limit = min(in_split, vis - step0);
                asm volatile("" : "+v"(limit));                      // a real branch: the selects below are not speculated into every step
#pragma unroll
                for (int t = 0; t < NT; ++t)
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        if (32 * t + 8 * (r / 4) + 4 * hw + r % 4 >= limit) c[t][r] = -INFINITY;
            }
            float mx = c[0][0];
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int r = 0; r < 16; ++r) mx = fmaxf(mx, c[t][r]);
            if (__any(mx > m)) {                     // uniform over the wave
                const float m_new = fmaxf(m, halves_max(mx));
                // a row that has seen nothing yet keeps m = -inf: shift by 0 then, every exponent is -inf and gives 0
                const float shift_new = (m_new == -INFINITY) ? 0.f : -m_new * scale2;
                // exactly 1 for a row whose maximum stands, however many other rows of the wave find new ones: the
                // difference of the two shifts as the weights have them (rounded)
                const float corr = (m == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(shift_new - shift);
                shift = shift_new;
                m = m_new;
                l *= corr;
#pragma unroll
                for (int dt = 0; dt < DT; ++dt) acc[dt] *= corr;
            }
            float sum[4] = {0.f, 0.f, 0.f, 0.f};     // four chains
            // 16 tokens at a time: contraction index 8 hw + i of group g stands for the token whose weight the lane holds
            // there, 16 g + 8 (i / 4) + 4 hw + i % 4 of the step
            bf16x8 ph, pl;
            auto weigh = [&](int g) {
                // round to nearest even, two weights per conversion; the low part carries the rounding error
                uint32_t hi[4], lo[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    float2v p;
#pragma unroll
                    for (int x = 0; x < 2; ++x) {                // masked scores give 0
                        p[x] = __builtin_amdgcn_exp2f(fmaf(c[g / 2][8 * (g % 2) + 2 * e + x], scale2, shift));
                        sum[(2 * e + x) % 4] += p[x];
                    }
                    hi[e] = __builtin_bit_cast(uint32_t, __builtin_convertvector(p, bf16x2));
                    lo[e] = 0u;
                    if (SPLIT_P) {
                        const float2v rest = {p[0] - __uint_as_float(hi[e] << 16), p[1] - __uint_as_float(hi[e] & 0xffff0000u)};    // exact
                        lo[e] = __builtin_bit_cast(uint32_t, __builtin_convertvector(rest, bf16x2));
                    }
                }
                ph = __builtin_bit_cast(bf16x8, make_uint4(hi[0], hi[1], hi[2], hi[3]));
                pl = __builtin_bit_cast(bf16x8, make_uint4(lo[0], lo[1], lo[2], lo[3]));
            };
            // O^T += V^T P^T: with kReadAheadV the V rows of the next group are read, and its weights formed, beside a group's products
            weigh(0);
#pragma unroll
            for (int g = 0; g < 2 * NT; ++g) {
                if constexpr (kReadAheadV) {
                    __builtin_amdgcn_sched_barrier(0);
                    if (g + 1 < 2 * NT) read_v(g + 1, vop[(g + 1) % 2]);
                } else {
                    read_v(g, vop[g % 2]);
                }
                const bf16x8 ph_g = ph, pl_g = pl;
#pragma unroll
                for (int dt = 0; dt < DT; ++dt)
                    acc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vop[g % 2][dt], ph_g, acc[dt], 0, 0, 0);
                if (SPLIT_P) {
#pragma unroll
                    for (int dt = 0; dt < DT; ++dt)
                        acc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vop[g % 2][dt], pl_g, acc[dt], 0, 0, 0);
                }
                if (g + 1 < 2 * NT) weigh(g + 1);
            }
            l += (sum[0] + sum[1]) + (sum[2] + sum[3]);
        };

        // a paged tier needs a table of block rows in LDS, which covers a whole split unless the blocks are tiny;
        // a contiguous tier is plain arithmetic
        const int sub_len = pass_length(kv, nt_total);
        for (int sub0 = 0; sub0 < nt_total; sub0 += sub_len) {
            const int nsub = min(sub_len, nt_total - sub0);
            __syncthreads();                         // the previous table and stages are no longer in use
            const BlockRows rows = make_block_rows<BLOCK>(s_row, kv, a1.sh.n_kv_heads, b, kvh, t0 + sub0, nsub);
            // Step s reads the stages of its parity and requests the rows of step s + 1 into the stages of the other
            // parity, which were last read in step s - 1: the barrier at the top of the step (before which every wave
            // waits for its own loads) orders both.
            const int steps = (nsub + kStepTokens - 1) / kStepTokens;
            auto request = [&](int s, char *k, char *v) {            // (the policy is part of the instructions)
                if (!streamed) dma_step<D, NW, 0, 0>(kv, rows, s, nsub, k, v);
                else if (16 * (steps - s) <= kept_k * steps) dma_step<D, NW, 0, kNonTemporal>(kv, rows, s, nsub, k, v);
                else dma_step<D, NW, kNonTemporal, kNonTemporal>(kv, rows, s, nsub, k, v);
            };
            request(0, s_k0, s_v0);
            auto step = [&](int s, const char *k_cur, const char *v_cur, char *k_next, char *v_next) {
                wait_for_own_loads();                // the barrier alone does not wait for LDS-direct loads
                __syncthreads();
                if (s + 1 < steps) request(s + 1, k_next, v_next);
                // Two workgroups share a unit, and the older one's waves go first: it would be done after two thirds of the
                // launch and leave the other alone.  The further a workgroup is in its pass over a tier, the lower its priority.
                // (A share is one pass, but for the one that holds the end of the pool and the start of the window and for tiers
                // in blocks so small that their table takes several passes: those start over.)
                const int left = steps - s;
                if (2 * left > steps) __builtin_amdgcn_s_setprio(3);
                else if (4 * left > steps) __builtin_amdgcn_s_setprio(2);
                else if (8 * left > steps) __builtin_amdgcn_s_setprio(1);
                else __builtin_amdgcn_s_setprio(0);
                if (wave_live) step_body(k_cur, v_cur, t0 + sub0 + s * kStepTokens, nsub - s * kStepTokens);
            };
            for (int s2 = 0; s2 < steps; s2 += 2) {
                step(s2, s_k0, s_v0, s_k1, s_v1);
                if (s2 + 1 < steps) step(s2 + 1, s_k1, s_v1, s_k0, s_v0);
            }
        }

        // (the V rows of every token of a tier have to be finite: a weight of 0 keeps a row out of the products only then)

        // partial of every valid row: the lane holds output columns 32 dt + 8 q + 4 hw .. + 3 of its row
        l = halves_sum(l);
        if (!row_exists) return;
        const int64_t at = ri.out_row * a1.part.stride + slot;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4)
                *reinterpret_cast<float4 *>(a1.part.o + at * D + 32 * dt + 8 * q4 + 4 * hw) =
                    make_float4(acc[dt][4 * q4], acc[dt][4 * q4 + 1], acc[dt][4 * q4 + 2], acc[dt][4 * q4 + 3]);
        if (hw == 0) {
            a1.part.m[at] = (m == -INFINITY) ? -INFINITY : m * a1.sh.sm_scale;         // the shift of the weights, in scaled scores
            a1.part.l[at] = l;
        }
    };
    const int begin = share * cut.share_steps, end = begin + cut.share_steps;
    if (!TWO || begin <= cut.first_steps) serve(a1, begin, end, share);
    if constexpr (TWO)
        if (end > cut.first_steps || share == line.shares - 1)
            serve(a2, max(begin - cut.first_steps, 0), max(end - cut.first_steps, 0), share + 1);
}

// Query-averaged softmax weights of a tier: a_out[b, h, t] = (1/N) sum_i e^{s_it - lse_i} over the queries i that see
// token t (lse_i is the tier's own log-sum-exp for query i), 0 beyond the length.
//
// Here the scores are wanted with a TOKEN per lane, S[row, token] = Q[row, :] . K[token, :] (A = Q, B = K): the rows of
// a tile are the result's registers, so the sum over the queries is an addition per score into one of min(G, 4)
// registers and nothing is exchanged between lanes but one last addition of the two halves of a wave.  A wave takes
// 32-token tiles of its own and meets all rows: the queries (128 rows at a time) stay in LDS for the eight waves of the
// workgroup, a tile's K rows arrive by LDS-direct loads in a slot that only its wave reads, go to registers as the B
// operand, and the slot takes the next tile at once -- no barrier and no sums through LDS in the loop.  Window and pool
// are one line of equal shares, as in the attention kernel, so that the launch is one full round of workgroups however
// the two lengths compare.  With more than 128 rows a share goes through blocks of 2048 tokens, every block once per 128
// rows (it stays in the caches meanwhile), adding to a_out: 33 / 64 / 128 queries x 4 heads on 28 K tokens, batch 8:
// 244 / 262 / 505 us with blocks of 512 tokens, two tiles per wave between barriers; 195 / 221 / 432 us.
//
// The number of rows may be any: a row that does not exist weighs nothing through its shift, so only tiles that the causal
// limit cuts compare, a compare and a select per score (with a test per score in every block that is not full, 31 queries
// x 4 heads took 147 us where 32 took 105; now 101 and 101).
// A tile's query pieces come from LDS well before their products, and a pair of row tiles is weighed beside the products of the
// next: with every read right before its use each of the 32 matrix instructions of a tile waited for LDS (whole turns: 8 x 32
// queries 387 -> 380 us, 4 x 128 queries 697 -> 677, 3 x 55 queries on 17 K tokens 173.5 -> 170.8; 8 x 9 queries unchanged).
// Both tiers of 8 x 32 queries on 32 K tokens, 32 / 8 heads: 150 us (tokens in registers, rows over the lanes: two lane
// exchanges per score and a barrier per 64 tokens, 2048-token workgroups that came out at 1.2 rounds) -> 117 us.  The
// loads alone take 101 us (124 us without the streaming policy; more of them in flight, 12 or 15 waves, change nothing).
// A launch over few tokens is a chain of latencies: K is requested before the queries, and a share with fewer tiles than
// waves deals a tile's rows to several waves, which add up through LDS (100 queries over 512 tokens 8.2 -> 4.8 us, 16
// queries x 4 heads over 3.5 K tokens 6.8 -> 5.4; workgroups of 64 tokens with a row tile per wave: 4.7 and 4.6).
template <int D> struct WeightsStage {
    static constexpr int kWaves = 8, kBlock = kWaves * kWave;
    static constexpr int kRowBytes = D * 2, kPieces = kRowBytes / 16, kGroupRows = 1024 / kRowBytes;
    static constexpr int kSwizzled = kPieces < 16 ? kPieces : 16;
    static __device__ __forceinline__ int swizzle(int row) { return (row / (16 / kSwizzled)) % kSwizzled; }
    static __device__ __forceinline__ int offset(int row, int piece) { return row * kRowBytes + 16 * (piece ^ swizzle(row)); }
};
// Heads of 64 in groups of up to 4 leave room for two workgroups on a unit (128 registers, 52 KB): row tiles are worked off pair by
// pair there.  Four at a time, a pair weighed beside the next one's products, take 166 to 175 registers and the second workgroup:
// 12 sequences, 16 / 8 heads, 14 K tokens, 48 / 100 queries 43.0 -> 47.8, 84.9 -> 96.6 us, with a window as well 54.2 -> 66.3, 109 ->
// 125; 3 sequences of 40 heads, up to 24 queries 36.1 -> 38.9; pair by pair 43.2, 84.1, 54.0, 106 and 36.1.  (Groups of 4 over two tiers and
// groups of 8 never had the room.  The registers of groups of 2 over two tiers come to 150 left alone, 125 when they are bounded; the
// others stay below by themselves, and 3 sequences of 40 heads take 38.6 us with the bound.)
template <int D, int G, bool TWO> constexpr bool kWTwoPerUnit = D == 64 && (G < 4 || (G == 4 && !TWO));
template <int D, int G, bool TWO>
__global__ __launch_bounds__(WeightsStage<D>::kBlock, D == 64 && G == 2 && TWO ? 4 : 2) void append_weights_kernel(
    AppendArgs a1, AppendArgs a2, LineDev line, int streamed, int from_end)
{
    using S = WeightsStage<D>;
    constexpr int kWWaves = S::kWaves, kWBlock = S::kBlock;
    constexpr int kSpreadLive = 3;               // row tiles from which dealing them out to idle waves pays
    constexpr int KK = S::kRowBytes / 32, RT = kRowsPerBlock / 32, NS = G < 4 ? G : 4;
    constexpr float kLog2e = 1.4426950408889634f;
    typedef const __attribute__((address_space(1))) void *GlobalPtr;
    typedef __attribute__((address_space(3))) void *LdsPtr;
    __shared__ __attribute__((aligned(1024))) char s_q[kRowsPerBlock * S::kRowBytes];
    __shared__ __attribute__((aligned(1024))) char s_k[kWWaves][kWTile * S::kRowBytes];
    __shared__ __attribute__((aligned(16))) float s_shift[kRowsPerBlock];        // minus the rows' lse, in the exponent's unit
    __shared__ uint32_t s_row[kSub];

    const int share = blockIdx.x, kvh = blockIdx.y, b = blockIdx.z;
    const int tid = threadIdx.x, lane = tid % kWave, w = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int n = lane % 32, hw = lane / 32;
    const int n_rows = a1.n_q * G, n_qb = (n_rows + kRowsPerBlock - 1) / kRowsPerBlock;
    // exponents in units of ln 2 for the bare v_exp_f32
    const float unit = kLog2e, inv_n = 1.f / (float)a1.n_q, scale = a1.sh.sm_scale * unit;
    const int frag0 = S::offset(n, hw);          // operand of row / token n; slice kk is an exclusive-or of 32 kk away
    char *const slot = s_k[w];

    const LineCut cut(line, b);
    int q_held = -1;                             // block of rows that s_q holds
    // one tier's part of the share; first_step: where the tier begins on the line.  (A loop over the tiers that chose
    // every argument by its counter took 0.7 us more of a launch with one.)
    auto serve = [&](const AppendArgs &a, int first_step) {
        const KvDev &kv = a.kv;
        const int causal_tail = a.causal_tail;
        const float *lse = a.lse;
        const int len = tier_len(kv, b);
        float *out = a.a_out + ((int64_t)b * a1.sh.n_q_heads + kvh * G) * kv.cap;

        // entries beyond the sequence's length, shared out as well
        for (int g = 0; g < G; ++g)
            for (int j = len + share * kWBlock + tid; j < kv.cap; j += line.shares * kWBlock) out[(int64_t)g * kv.cap + j] = 0.f;

        const int begin = share * cut.share_steps;
        const int t0 = max(begin - first_step, 0) * kStepTokens;
        const int t_end = min(max(begin + cut.share_steps - first_step, 0) * kStepTokens, len);
        if (t0 >= t_end) return;                 // nothing of this tier in the share (uniform over the workgroup)
        const int pass_len = min(pass_length(kv, t_end - t0), n_qb > 1 ? kWManyRowTokens : INT32_MAX);
        for (int p0 = t0; p0 < t_end; p0 += pass_len) {
            const int nt = min(pass_len, t_end - p0), tiles = (nt + kWTile - 1) / kWTile;
            __syncthreads();                     // the table of the previous pass is no longer in use
            const BlockRows rows = make_block_rows<kWBlock>(s_row, kv, a1.sh.n_kv_heads, b, kvh, p0, nt);
            // Requests the K rows of a tile: 16-byte pieces swizzled by the row, as the operand reads want them.
            auto request = [&](int tile) {
                constexpr int LOADS = kWTile / S::kGroupRows;
                const int r = lane / S::kPieces;                 // row inside a load instruction's group
                if ((tile + 1) * kWTile <= nt) {                 // uniform over the wave
                    uint32_t base[kWTile / kGranule];            // row of each granule's first token, uniform
#pragma unroll
                    for (int g = 0; g < kWTile / kGranule; ++g) base[g] = rows.base + tile * kWTile + g * kGranule;
                    if (rows.table) {
#pragma unroll
                        for (int g = 0; g < kWTile / kGranule; ++g) base[g] = rows.table[tile * (kWTile / kGranule) + g];
#pragma unroll
                        for (int g = 0; g < kWTile / kGranule; ++g) base[g] = __builtin_amdgcn_readfirstlane(base[g]);
                    }
#pragma unroll
                    for (int u = 0; u < LOADS; ++u) {
                        const int row = u * S::kGroupRows;       // of the tile
                        const uint32_t off = r * S::kRowBytes + 16 * ((lane % S::kPieces) ^ S::swizzle(row % 16 + r));
                        const char *src = kv.k + (size_t)(base[row / kGranule] + row % kGranule) * S::kRowBytes;
                        if (streamed)            // uniform over the launch (the policy is part of the instruction)
                            __builtin_amdgcn_global_load_lds((GlobalPtr)(src + off), (LdsPtr)(slot + u * 1024), 16, 0, kNonTemporal);
                        else
                            __builtin_amdgcn_global_load_lds((GlobalPtr)(src + off), (LdsPtr)(slot + u * 1024), 16, 0, 0);
                    }
                } else {                                         // tokens behind the end read the last row
                    uint32_t at[LOADS];
#pragma unroll
                    for (int u = 0; u < LOADS; ++u) {
                        const uint32_t t = min(tile * kWTile + u * S::kGroupRows + r, nt - 1);
                        at[u] = rows.table ? rows.table[t / kGranule] + t % kGranule : rows.base + t;
                    }
#pragma unroll
                    for (int u = 0; u < LOADS; ++u) {
                        const int piece = (lane % S::kPieces) ^ S::swizzle(u * S::kGroupRows + r);
                        __builtin_amdgcn_global_load_lds((GlobalPtr)(kv.k + (size_t)at[u] * S::kRowBytes + 16 * piece),
                                                         (LdsPtr)(slot + u * 1024), 16, 0, 0);
                    }
                }
            };
            for (int qb = 0; qb < n_qb; ++qb) {
                __syncthreads();                 // the queries and shifts of the previous round are no longer in use
                const int live = (min(n_rows - qb * kRowsPerBlock, kRowsPerBlock) + 31) / 32;        // 32-row tiles with rows that exist
                // a block with fewer tiles than there are waves: several waves take a tile's rows in turn and add up at the end
                const int spread_bits = live < kSpreadLive ? 0 : 4 * tiles <= kWWaves ? 2 : 2 * tiles <= kWWaves ? 1 : 0;
                const int spread = 1 << spread_bits, part = w % spread, stride = kWWaves >> spread_bits;
                const int tile_first = from_end ? tiles - 1 - (w >> spread_bits) : w >> spread_bits;
                const int tile_step = from_end ? -stride : stride;
                auto is_tile = [&](int t) { return (unsigned)t < (unsigned)tiles; };
                if (is_tile(tile_first)) request(tile_first);    // first: it has the longest way
                // rows that do not exist repeat the last query of their head with a shift of -inf: they weigh nothing, and
                // what a non-finite key gives them it gives an existing row of that head too
                auto existing = [&](int r) { return r < n_rows ? r : n_rows - G + r % G; };
                if (q_held != qb) {              // uniform over the workgroup
                    for (int g = w; g < kRowsPerBlock / S::kGroupRows; g += kWWaves) {
                        const int row = g * S::kGroupRows + lane / S::kPieces;
                        const RowInfo ri = row_info<G>(a1, b, kvh, existing(qb * kRowsPerBlock + row));
                        const char *src = static_cast<const char *>(a1.q) + ri.out_row * S::kRowBytes +
                                          16 * ((lane % S::kPieces) ^ S::swizzle(row));
                        __builtin_amdgcn_global_load_lds((GlobalPtr)src, (LdsPtr)(s_q + g * 1024), 16, 0, 0);
                    }
                    q_held = qb;
                }
                if (tid < kRowsPerBlock) {
                    const RowInfo ri = row_info<G>(a1, b, kvh, qb * kRowsPerBlock + tid);
                    const float row_lse = ri.valid ? lse[ri.out_row] : INFINITY;
                    // a row that sees nothing has lse = -inf; its weights are left out below, whatever the shift
                    s_shift[tid] = (row_lse == -INFINITY) ? 0.f : -row_lse * unit;
                }
                wait_for_own_loads();
                __syncthreads();

                // tokens that all rows of the block see (tokens behind the length are not stored and need no mask)
                const int seen_by_all = causal_tail ? len - a1.n_q + qb * kRowsPerBlock / G + 1 : INT32_MAX;
                float done[NS] = {};             // the sums of the tile before, not stored yet
                int done_at = -1;
                auto store = [&]() {             // lane (n, hw) of a half stores every other head of its token (G = 8: its half's heads)
                    const int t = done_at + n;
                    if (done_at >= 0 && t < t_end) {
#pragma unroll
                        for (int g = 0; g < NS; ++g) {
                            if (G < 8 && NS > 1 && g % 2 != hw) continue;
                            if (NS == 1 && hw) continue;
                            float *dst = out + (int64_t)(G == 8 ? 4 * hw + g : g) * kv.cap + t;
                            *dst = qb == 0 ? done[g] * inv_n : fmaf(done[g], inv_n, *dst);
                        }
                    }
                };
                for (int tile = tile_first; is_tile(tile); tile += tile_step) {
                    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");             // the tile's rows are in the slot
                    uint4 kf[KK];
#pragma unroll
                    for (int kk = 0; kk < KK; ++kk) kf[kk] = *reinterpret_cast<const uint4 *>(slot + (frag0 ^ (32 * kk)));
                    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");           // ... and in registers: the slot is free
                    if (is_tile(tile + tile_step)) request(tile + tile_step);
                    store();                     // (its write overlaps with this tile's arithmetic)
                    const int tok0 = p0 + tile * kWTile;
                    float sum[NS];
#pragma unroll
                    for (int g = 0; g < NS; ++g) sum[g] = 0.f;
                    // c[r] of row tile x is the score of row 32 x + 8 (r / 4) + 4 hw + r % 4 and the lane's token
                    auto q_piece = [&](int x, int kk) {
                        return *reinterpret_cast<const uint4 *>(s_q + x * 32 * S::kRowBytes + (frag0 ^ (32 * kk)));
                    };
                    auto shift_of = [&](int x, int q4) {         // of rows 32 x + 8 q4 + 4 hw .. + 3
                        return *reinterpret_cast<const float4 *>(s_shift + 32 * x + 8 * q4 + 4 * hw);
                    };
                    auto weigh_quad = [&](floatx16 &c, int q4, const float4 &sh) {
                        const float s4[4] = {sh.x, sh.y, sh.z, sh.w};
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            c[4 * q4 + e] = __builtin_amdgcn_exp2f(fmaf(c[4 * q4 + e], scale, s4[e]));
                    };
                    auto weigh = [&](int x, floatx16 &c) {
#pragma unroll
                        for (int q4 = 0; q4 < 4; ++q4) weigh_quad(c, q4, shift_of(x, q4));
                    };
                    // NP row tiles from x on, two at a time side by side so that their matrix instructions take turns.  The
                    // query pieces are read kWAhead before the instructions that take them (left alone the scheduler reads
                    // each right before its use, and every matrix instruction waits for LDS); a pair of tiles is weighed
                    // beside the products of the next pair.
                    auto tiles_of = [&](int x, auto count, floatx16 (&c)[decltype(count)::value]) {
                        constexpr int NP = decltype(count)::value, ALL = NP * KK, W = NP > 1 ? 2 : 1;
                        if constexpr (kWTwoPerUnit<D, G, TWO>) {
                            static_assert(NP <= W, "pair by pair");
                            uint4 qf[ALL];
                            auto read = [&](int i) {             // the i-th piece in the order of use
                                if (i < ALL) qf[i] = q_piece(x + i % W, i / W);
                            };
#pragma unroll
                            for (int i = 0; i < kWAhead; ++i) read(i);
#pragma unroll
                            for (int i = 0; i < W; ++i) c[i] = floatx16{};
#pragma unroll
                            for (int kk = 0; kk < KK; ++kk) {
                                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                                for (int i = 0; i < W; ++i) read(W * kk + i + kWAhead);
#pragma unroll
                                for (int i = 0; i < W; ++i) c[i] = score_mfma(qf[W * kk + i], kf[kk], c[i]);
                            }
                            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                            for (int i = 0; i < W; ++i) weigh(x + i, c[i]);
                        } else {
                            uint4 qf[ALL];
                            auto read = [&](int i) {             // the i-th piece in the order of use
                                if (i < ALL) qf[i] = q_piece(x + i / (W * KK) * W + i % W, i / W % KK);
                            };
#pragma unroll
                            for (int i = 0; i < kWAhead; ++i) read(i);
                            constexpr int QUADS = 4 * W > KK ? 4 * W / KK : 1;           // weighed beside a slice's products
                            float4 sh[4 * W];
#pragma unroll
                            for (int t0 = 0; t0 < NP; t0 += W) {
#pragma unroll
                                for (int i = 0; i < W; ++i) c[t0 + i] = floatx16{};
#pragma unroll
                                for (int kk = 0; kk < KK; ++kk) {
                                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                                    for (int i = 0; i < W; ++i) read(W * (t0 / W * KK + kk) + i + kWAhead);
                                    if (t0 > 0 && kk * QUADS < 4 * W) {
#pragma unroll
                                        for (int i = 0; i < QUADS; ++i) {
                                            const int j = kk * QUADS + i;
                                            weigh_quad(c[t0 - W + j / 4], j % 4, sh[j]);
                                        }
                                    }
#pragma unroll
                                    for (int i = 0; i < W; ++i)
                                        c[t0 + i] = score_mfma(qf[W * (t0 / W * KK + kk) + i], kf[kk], c[t0 + i]);
                                    if (kk == KK - 1) {          // the pair's shifts, for its turn to be weighed
#pragma unroll
                                        for (int j = 0; j < 4 * W; ++j) sh[j] = shift_of(x + t0 + j / 4, j % 4);
                                    }
                                }
                            }
                            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                            for (int j = 0; j < 4 * W; ++j) weigh_quad(c[NP - W + j / 4], j % 4, sh[j]);
                        }
                    };
                    auto add = [&](const floatx16 &c) {          // the head of row r is r % G
#pragma unroll
                        for (int r = 0; r < 16; ++r) sum[r % NS] += c[r];
                    };
                    if (live == RT && spread == 1 && tok0 + kWTile <= seen_by_all) {     // uniform over the wave: straight-line code
                        constexpr int NP = kWTwoPerUnit<D, G, TWO> ? 2 : RT;
#pragma unroll
                        for (int x = 0; x < RT; x += NP) {
                            floatx16 c[NP];
                            tiles_of(x, std::integral_constant<int, NP>{}, c);
#pragma unroll
                            for (int i = 0; i < NP; ++i) add(c[i]);
                        }
                    } else {
                        // Row r sees the lane's token iff r / G >= token - (len - n_q): the first such row, relative to the
                        // first row that the lane holds.  Tiles that all rows see whole get a limit nothing is below.
                        const int first_row = tok0 + kWTile <= seen_by_all
                                                  ? INT32_MIN / 2
                                                  : G * (tok0 + n - (len - a1.n_q)) - qb * kRowsPerBlock - 4 * hw;
                        auto mask = [&](int x, floatx16 &c) {
#pragma unroll
                            for (int r = 0; r < 16; ++r) c[r] = 8 * (r / 4) + r % 4 >= first_row - 32 * x ? c[r] : 0.f;
                        };
                        int x = part;
#pragma unroll 1
                        for (; spread == 1 && x + 1 < live; x += 2) {
                            floatx16 c[2];
                            tiles_of(x, std::integral_constant<int, 2>{}, c);
                            mask(x, c[0]);
                            mask(x + 1, c[1]);
                            add(c[0]);
                            add(c[1]);
                        }
#pragma unroll 1
                        for (; x < live; x += spread) {
                            floatx16 c[1];
                            tiles_of(x, std::integral_constant<int, 1>{}, c);
                            mask(x, c[0]);
                            add(c[0]);
                        }
                    }
#pragma unroll
                    for (int g = 0; g < NS; ++g) done[g] = G < 8 ? halves_sum(sum[g]) : sum[g];
                    done_at = tok0;
                }
                if (spread > 1) {                // uniform over the workgroup; a wave has met one tile at most, its slot is free
#pragma unroll
                    for (int g = 0; g < NS; ++g) reinterpret_cast<float *>(slot)[g * kWave + lane] = done[g];
                    __syncthreads();
                    for (int i = 1; part == 0 && i < spread; ++i)
#pragma unroll
                        for (int g = 0; g < NS; ++g) done[g] += reinterpret_cast<const float *>(s_k[w + i])[g * kWave + lane];
                    if (part != 0) done_at = -1;
                }
                store();
            }
        }
    };
    serve(a1, 0);
    if constexpr (TWO) serve(a2, cut.first_steps);
}

template <int D, bool SPLIT_P, bool TWO>
hipError_t launch_attn_tiers(const AppendArgs &a, const AppendArgs &a2, const LineDev &line, dim3 grid, int streamed, int kept_k,
                             hipStream_t s)
{
    const dim3 block(kAttnBlock);
    switch (a.sh.group) {
    case 1: hipLaunchKernelGGL((append_attn_kernel<D, 1, SPLIT_P, TWO>), grid, block, 0, s, a, a2, line, streamed, kept_k); break;
    case 2: hipLaunchKernelGGL((append_attn_kernel<D, 2, SPLIT_P, TWO>), grid, block, 0, s, a, a2, line, streamed, kept_k); break;
    case 4: hipLaunchKernelGGL((append_attn_kernel<D, 4, SPLIT_P, TWO>), grid, block, 0, s, a, a2, line, streamed, kept_k); break;
    case 8: hipLaunchKernelGGL((append_attn_kernel<D, 8, SPLIT_P, TWO>), grid, block, 0, s, a, a2, line, streamed, kept_k); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <int D, bool SPLIT_P>
hipError_t launch_attn_group(const AppendArgs &a, const AppendArgs &a2, const LineDev &line, int two, dim3 grid,
                             int streamed, int kept_k, hipStream_t s)
{
    return two ? launch_attn_tiers<D, SPLIT_P, true>(a, a2, line, grid, streamed, kept_k, s)
               : launch_attn_tiers<D, SPLIT_P, false>(a, a2, line, grid, streamed, kept_k, s);
}

template <int D, bool TWO>
hipError_t launch_weights_tiers(const AppendArgs &a, const AppendArgs &a2, const LineDev &line, dim3 grid, int streamed, int from_end,
                                hipStream_t s)
{
    const dim3 block(WeightsStage<D>::kBlock);
    switch (a.sh.group) {
    case 1: hipLaunchKernelGGL((append_weights_kernel<D, 1, TWO>), grid, block, 0, s, a, a2, line, streamed, from_end); break;
    case 2: hipLaunchKernelGGL((append_weights_kernel<D, 2, TWO>), grid, block, 0, s, a, a2, line, streamed, from_end); break;
    case 4: hipLaunchKernelGGL((append_weights_kernel<D, 4, TWO>), grid, block, 0, s, a, a2, line, streamed, from_end); break;
    case 8: hipLaunchKernelGGL((append_weights_kernel<D, 8, TWO>), grid, block, 0, s, a, a2, line, streamed, from_end); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <int D>
hipError_t launch_weights_group(const AppendArgs &a, const AppendArgs &a2, const LineDev &line, int two, dim3 grid,
                                int streamed, int from_end, hipStream_t s)
{
    return two ? launch_weights_tiers<D, true>(a, a2, line, grid, streamed, from_end, s)
               : launch_weights_tiers<D, false>(a, a2, line, grid, streamed, from_end, s);
}

int64_t k_bytes_of(const AppendArgs &a, const AppendArgs *second, int head_dim)
{
    return (int64_t)a.sh.batch * a.sh.n_kv_heads * ((int64_t)a.kv.cap + (second ? second->kv.cap : 0)) * head_dim * 2;
}

// A turn's weights pass reads again the K rows that its attention has just streamed (one block of rows).  From 512 MB of K and V
// on (by capacity; a managed cache counts its window twice), the K rows of the last sixteenths of every share, 12 at most and as
// many as the last cache holds of K, are left to the caches, and the weights pass walks its shares from the end (a paged share in
// passes of 8192 tokens: the passes in order, each from its end, in both kernels).  Whole turns,
// everything streamed : so, us: 8 x 32 queries 1.1 GB 381 : 377, 12 x 8 queries 1.7 GB 460 : 450; 4 x 32 queries 576 MB 227 : 224;
// 2 x 16 queries in groups of 8, 512 MB 218 : 212; 6 x 32 queries of 32 / 16 heads of 64, 864 MB 286 : 276.  Below, 0.99 to 1.01 times as
// fast (288 MB 140.2 : 140.4, 330 MB 149.4 : 150.6, 482 MB 198.9 : 200.6).  All of K kept, or walked from the start, gains less;
// attention alone loses 1 to 5 % (16 queries, 288 MB 65.5 : 69.3).
int kept_sixteenths(int64_t kv_bytes)
{
    return kv_bytes >= 2 * kLastCache ? (int)std::min<int64_t>(12, 32 * kLastCache / kv_bytes) : 0;
}

}  // namespace

hipError_t launch_append_attn(int dtype, int head_dim, const AppendArgs &a, const AppendArgs *second, const LineDev &line,
                              bool weights_follow, hipStream_t s)
{
    if (a.sh.batch == 0 || a.n_q == 0) return hipSuccess;
    const AppendArgs &a2 = second ? *second : a;
    if (line.shares <= 0 || a.part.stride != line.shares + (second ? 1 : 0) || a2.n_q != a.n_q || a2.q != a.q ||
        a2.one_part_p != a.one_part_p || a2.sh.group != a.sh.group || a2.sh.batch != a.sh.batch ||
        a2.sh.n_kv_heads != a.sh.n_kv_heads || a2.part.o != a.part.o || a2.part.stride != a.part.stride)
        return hipErrorInvalidValue;             // the two tiers share the queries, the launch shape and the partials
    const int n_qb = (a.n_q * a.sh.group + kRowsPerBlock - 1) / kRowsPerBlock;
    const int64_t streams = (int64_t)line.shares * a.sh.n_kv_heads * a.sh.batch;
    const int64_t blocks = (streams + kXcds - 1) / kXcds * kXcds * n_qb;
    if (blocks > 0x7fffffff) return hipErrorInvalidValue;
    const dim3 grid = n_qb == 1 ? dim3(line.shares, a.sh.n_kv_heads, a.sh.batch) : dim3((unsigned)blocks);
    const int two = second ? 1 : 0;
    if (dtype == 0) return launch_append_attn_f32(head_dim, a, a2, line, two, grid, s);
    const int64_t kv_bytes = 2 * k_bytes_of(a, second, head_dim);
    // One block of rows reads every K and V row once: past what the last cache holds (256 MB, by capacity) the loads leave the
    // caches alone.  1.07 GB, 8 x 32 queries, loads without arithmetic 217 -> 185 us, the attention of both tiers 249 -> 243;
    // 537 MB, 4 x 16 queries, whole turn 192 -> 179; 134 MB and less no difference.  Several blocks read the rows again:
    // three of them (48 queries, groups of 8) 245 -> 265 when streamed.
    // A managed cache that is filled to a part of its capacity loses nothing: 5 to 50 % of 0.9 to 1.0 GB, whole turns 0.99 to 1.07 times
    // as fast streamed, also where what is in it would fit the last cache for the weights pass.
    const int streamed = n_qb == 1 && kv_bytes >= kLastCache ? 1 : 0;
    const int kept_k = weights_follow && streamed ? kept_sixteenths(kv_bytes) : 0;
    if (dtype == 1 && head_dim == 64)
        return a.one_part_p ? launch_attn_group<64, false>(a, a2, line, two, grid, streamed, kept_k, s)
                            : launch_attn_group<64, true>(a, a2, line, two, grid, streamed, kept_k, s);
    if (dtype == 1 && head_dim == 128)
        return a.one_part_p ? launch_attn_group<128, false>(a, a2, line, two, grid, streamed, kept_k, s)
                            : launch_attn_group<128, true>(a, a2, line, two, grid, streamed, kept_k, s);
    return hipErrorInvalidValue;
}

hipError_t launch_append_weights(int dtype, int head_dim, const AppendArgs &a, const AppendArgs *second,
                                 const LineDev &line, bool after_attention, hipStream_t s)
{
    if (a.sh.batch == 0 || a.n_q == 0) return hipSuccess;
    const AppendArgs &a2 = second ? *second : a;
    if (line.shares <= 0 || a2.n_q != a.n_q || a2.q != a.q || a2.sh.group != a.sh.group || a2.sh.batch != a.sh.batch ||
        a2.sh.n_kv_heads != a.sh.n_kv_heads)
        return hipErrorInvalidValue;             // the two tiers share the queries and the launch shape
    // (a flat grid would be short of numbers: its threads are counted in 32 bits per dimension)
    const dim3 grid(line.shares, a.sh.n_kv_heads, a.sh.batch);
    const int two = second ? 1 : 0;
    if (dtype == 0) return launch_append_weights_f32(head_dim, a, a2, line, two, grid, s);
    // K rows that pass once and are too many to stay in the L2 caches anyway (32 MB, by capacity) are streamed past them:
    // 470 MB 106 -> 94 us; 11 MB, which do stay, 5.3 us as they are and 5.7 streamed.  More than
    // one pass over the rows reads K again: 33 queries x 4 heads 192 us as they are, 211 streamed.
    const bool one_pass = (int64_t)a.n_q * a.sh.group <= kRowsPerBlock;
    const int64_t k_bytes = k_bytes_of(a, second, head_dim);
    const int streamed = one_pass && k_bytes >= (int64_t(16) << 20) ? 1 : 0;
    const int from_end = after_attention && one_pass && kept_sixteenths(2 * k_bytes) > 0 ? 1 : 0;
    if (dtype == 1 && head_dim == 64) return launch_weights_group<64>(a, a2, line, two, grid, streamed, from_end, s);
    if (dtype == 1 && head_dim == 128) return launch_weights_group<128>(a, a2, line, two, grid, streamed, from_end, s);
    return hipErrorInvalidValue;
}

}  // namespace hgca

// Rules by which the entry points choose among paths that give the same results: plain functions of sizes, without HIP.
#pragma once

#include <stdint.h>

namespace hgca {

// Whether the workgroups of a gather run by groups of heads (GatherPlace), and whether the rows of K and V stay in the cache for
// the group's other heads or are streamed past it: by how much of the pool a group's lists would cover if they shared nothing,
// group * k_max / pool.  Heads of a group may list many of the same tokens or hardly any; the limits lie where lists that
// share no more than chance gives them lose nothing to speak of.  Measured, in percent of what the order head by head takes, groups
// of 4, lists that share nothing / a quarter of their entries at 7 % of the pool:
//   kept        coverage 20 % 107 / 105   29 % 101 / 89   36 % 99 / 85   48 % 102 / 95   60 % 92 / 76   (8 sequences, 28 672 tokens)
//               29 % 98 / 88   34 % 98 / 87   40 % 98 / 87                                    (64 sequences of 2 K to 16 K tokens in blocks)
//   lists of a selection on random keys, 29 %: 67.1 -> 70.9 us per step; fp32 28 % 105 / 100, 40 % 101 / 90, 60 % 95 / 84
// Groups of 8 by groups: 28 % 98 / 93, 40 % 97 / 91, 60 % 92 / 79; kept 40 % 105 / 89, 60 % 96 / 76; where the window shares their
// launch only the kept order is built: in small bf16 steps no order matters; fp32, 45 %, 16 sequences kept 99 / 86, 4 104 / 101.  Groups of 2 by groups: 16 % 100 /
// 100, 30 % 98 / 94; kept 106 / 103, 103 / 94.
// Managed lists have room to grow and are rarely full: the coverage by their capacity says less, and the limit is lower.  Loops,
// kept, lists that share nothing / a quarter: groups of 4, coverage by capacity 12 %, half full 103, 103, 100 / 100, 100, 99 and 20 %
// 103, 100, 102 / 102, 94, 98, nearly full 101, 98, 100 / 98, 86, 94, 32 % 100, 105, 96 / 96, 82, 88 (8 sequences, 28 672 tokens; 6,
// 60 032; 8, 14 336); room for a seventh of the pool, 57 %, filled to 30, 50 and 85 %: 8 sequences, 28 672 101, 99, 107 / 95, 95, 95; 6,
// 63 424 97, 105, 103 / 90, 87, 88; groups of 8, 114 %: 14 336 100, 95, 95 / 90, 85, 76, 28 672 100, 107, 105 (shared, 50 %: 92); groups
// of 2, 28 %: 8 sequences, 20 000 92, 96, 100 / 91, 93, 96, 5 sequences, 48 960 104, 101, 97 / 103, 99, 92 (by groups without keeping
// the rows within 3 % of that; fp32 loops kept 0.98 times that, 30 shapes).
// With the scores given only V comes in, behind a pass over the pool: by groups 36 % 96.5 .. 101, 45 % 96 .. 101, 90 % 92 .. 101 (groups
// of 2, 4 and 8, 2 to 32 sequences of 6 K to 40 K tokens).
struct GatherOrder {
    bool by_group, keep;
};
inline GatherOrder gather_order(int64_t group, int64_t k_max, int64_t pool, bool scored, bool managed)
{
    if (group <= 1 || pool <= 0) return {false, false};
    const int64_t covered = 100 * group * k_max;
    const bool by_group = covered >= (group == 2 && !scored ? 16 : managed ? 20 : 36) * pool;
    return {by_group, by_group && !scored && (managed || group == 4 || (group == 8 && covered >= 50 * pool))};
}

// Whether the window's splits take the lower block numbers of a launch that they share with the gather, and so start first; the
// other part fills in behind.  With the scores given the gather brings V alone and starts second.  With K and V gathered it has more
// to bring, in bf16 (8B shape, 270 MB against 134: 68.0 against 69.2 us per step).  In fp32 a window split takes longer than any of the
// gather's, and started last they are what the launch waits for: 12 sequences, 32 / 8 heads of 128, window 4096, 600 listed 133 : 107
// us, window 1024, 1900 listed 133 : 134; one sequence, 64 / 8 heads of 64, window 1024, 1900 listed 20.0 : 16.5; over 220 shapes 0.95
// times, at worst 1.05.  Without groups the two kinds of splits are alike and the bytes decide: 4 sequences, 40 heads of 128, 600
// listed, window 4096 137 : 123, loops with lists half full, window 256 34.3 : 35.8 per step, 1024 55.9 : 57.3, 2048 86.0 : 83.3.
inline bool window_first(bool f32, int64_t group, int64_t window, int64_t k_max, bool scored)
{
    return scored || (f32 && (group > 1 || window >= 2 * k_max));
}

// Whether a step with a selection runs as the two launches of short_step_kernels.hip.  They save two or three dependent
// launches of 3 to 5 us each; against that a row's list is read by one compute unit alone (its V rows at about 60 GB/s ... 512 KB
// take 8 us), and a score pass that shares its launch with the window has the window's registers and LDS.  One row per compute
// unit at most; then, general path : this one, in us (taken when reductions over a wave went through LDS; since then both sides are
// faster and the order is the same: bf16, one sequence, 32 / 8 heads of 128, pool 20000, k 500 29.3 : 27.4; 180 MB of keys, k 400
// 60.1 : 59.0; groups of 8 of 64, 29 MB, k 700 32.9 : 30.7; fp32, groups of 8 of 64, 65 MB, 256 KB 42.5 : 42.5)
//   V rows of a list, bf16: 102 KB (k 400) 21.4 : 20.0, 154 KB (k 1207) 32.9 : 33.9, 512 KB (k 2000) 25.5 : 31.8; fp32, which has one
//   launch more in the general path: 16 KB 24.7 : 15.9, 358 KB 27.9 : 26.6, 512 KB 27.7 : 30.5, 1 MB 34.4 : 43.0
//   keys of the pool, bf16, heads of 128 in groups of 2 and 4, lists of 16 to 128 KB: 100 MB 45.2 : 45.0 to 41.2 : 39.3, 180 MB 61.1 : 61.5,
//   65.5 : 64.2 and, partly filled pages, 45.8 : 46.5, 42.9 : 41.7; 240 MB 70.9 : 72.5, 76.2 : 78.4, pages 61.8 : 63.9, 55.6 : 56.9;
//   others of up to 4: 240 MB heads of 128 alone 64.3 : 63.4, heads of 64 in twos 71.6 : 67.5, pages 56.6 : 59.3;
//   keys of the pool, bf16, groups of up to 4: 164 MB 57.1 : 57.2, 205 MB 76.0 : 73.1, 410 MB 110.6 : 112.0 and 103.6 : 105.7;
//   groups of 8, whose window takes 70 KB of LDS: 20 MB 30.6 : 27.0, 33 MB 37.5 : 37.0, 51 MB 40.3 : 43.4, 82 MB 46.4 : 53.4
//   fp32, 350 MB to 1 GB: groups of up to 4, and of 8 with heads of 128, 0.98 to 1.12 times as fast, so no limit there; groups of 8
//   with heads of 64, whose window takes 84 registers and 26 KB: 100 MB, list of 16 KB 72.6 : 67.7, 160 KB 75.7 : 78.6, 320 KB 77.5 : 81.3;
//   126 MB, 35 KB 62.8 : 58.1; 200 MB, 16 KB 123.9 : 119.3; 128 MB, 100 KB 89.5 : 89.3; 80 MB, 128 KB 67.7 : 67.3, 256 KB 66.2 : 67.6; 64 MB,
//   205 KB 59.5 : 59.1, 384 KB 62.1 : 64.1; 32 MB, 384 KB 49.6 : 48.2; 312 MB, 175 KB 167.5 : 172.8: by keys times list, up to 256 MB.
constexpr int64_t kMaxShortList = 1536;          // entries that the limits in bytes leave room for (fp32, heads of 64)
inline bool short_step(bool f32, int64_t head_dim, int64_t units, int64_t group, int64_t window, int64_t pool, int64_t k_max)
{
    if (window <= 0 || pool <= 0 || k_max <= 0 || k_max > kMaxShortList || units * group > 256) return false;
    if (units * (window / 64 + pool / 64 + 2) > int64_t(1) << 23) return false;  // threads of a flat grid are counted in 32 bits
    const int64_t row = head_dim * (f32 ? 4 : 2), list = k_max * row, keys = units * pool * row;
    if (f32) return list <= 384 << 10 && (group < 8 || head_dim > 64 || (keys <= 256 << 20 && keys * list <= int64_t(13000) << 30));
    return list <= 128 << 10 && keys <= int64_t(group == 8 ? 32 : group > 1 && head_dim > 64 ? 192 : 256) << 20;
}

// Workgroups that share the `steps` of 64 tokens (by capacity) of each of `units`, at most `most`: the number for which the launch
// takes the least time, counted in steps: rounds of `places` workgroups (what the device holds at once) times
// the steps of a share and what a share costs beside them (`overhead` steps).
inline int line_shares(int64_t units, int64_t steps, int most, int places, int overhead)
{
    int best = 1;
    int64_t best_cost = INT64_MAX;
    for (int n = 1; n <= most && n <= steps; ++n) {
        const int64_t rounds = (n * units + places - 1) / places;
        const int64_t cost = rounds * ((steps + n - 1) / n + overhead);
        if (cost < best_cost) {
            best_cost = cost;
            best = n;
        }
    }
    return best;
}
// the steps that one place of such a launch goes through
inline int64_t line_turns(int64_t units, int64_t steps, int64_t shares, int64_t places)
{
    return (shares * units + places - 1) / places * ((steps + shares - 1) / shares);
}

// fp32 append attention of few queries over one tier: one-query attention per (sequence, query) with the split kernels of the decode
// path, which read K and V once per query and work out no more than its rows, against the matrix instructions, which work out 16 rows
// whatever there are.  The lower estimate has it, in us:
//   query by query 7 + 0.08 group^2, and the K and V bytes of all queries at what the vector units take (44 TB/s over the heads of a
//   group) or the rows come from, by the size of K and V: 20 TB/s up to 16 MB, 15 up to 70, 12 up to 150, 10 up to 256 MiB, which the last
//   cache holds, 7.5 beyond; 7.5 also where a split's queries, splits * kv_heads workgroups apart, are on different XCDs and find nothing in their L2;
//   on the matrix instructions 8, and the steps of a workgroup, one at a time per compute unit: 2.3 us with heads of 64, 3.4 with heads of
//   128, and up to 2.4 and 5.6 more with 128 rows (heads of 64 have half the columns and two thirds of the time).
// Fitted to 3585 sizes, 1 to 16 queries, 200 to 30 K tokens, up to 1.3 GB: the side taken is 0.4 % slower than the faster one on
// average, by more than 20 % at 5 of them (2.3 % and 139 with the constants before).  Query by query : matrix, us, 1 / 2 / 4 queries: 4 sequences, 40 heads of 64, 4 K tokens 54 : 117,
// 93 : 119, 176 : 121; 2 sequences, 32 / 8 heads of 128, 4 K tokens 18 : 23, 21 : 23, 33 : 24; 8 sequences, 8 heads of 128, 4 K tokens 44 : 64,
// 48 : 64, 94 : 66; 8 sequences, 32 / 8 heads of 64, 4 K tokens 28 : 46, 32 : 48, 52 : 48; 4 sequences, 64 / 8 heads of 64, 16 K tokens 50 : 85,
// 89 : 91, 177 : 95; 5 sequences, 2 heads of 128, 4 queries, 4608 tokens (24 splits) 17 : 19, 4736 tokens (25) 31 : 20.
inline bool query_by_query(int64_t head_dim, int64_t batch, int64_t kv_heads, int64_t group, int64_t n_q, int64_t tokens, int64_t splits,
                           int64_t turns)
{
    const double set = (double)batch * kv_heads * tokens * head_dim * 8, rows = n_q * group < 128 ? n_q * group / 128. : 1.;
    const bool apart = n_q > 1 && splits * kv_heads % 8 != 0;
    const double source = apart || set > 270e6 ? 7.5e6 : set > 150e6 ? 10e6 : set > 70e6 ? 12e6 : set > 16e6 ? 15e6 : 20e6;      // bytes per us
    const double vector = 44e6 / group;
    const double step = head_dim <= 64 ? 2.3 + 2.4 * rows : 3.4 + 5.6 * rows;
    return 7 + 0.08 * group * group + set * n_q / (vector < source ? vector : source) < 8 + turns * step;
}

}  // namespace hgca

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

}  // namespace hgca

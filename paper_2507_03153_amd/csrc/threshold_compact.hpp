// Ordered compaction of the entries of one fp32 row that exceed a threshold (the per-head rule
// "salient iff weight > beta / size"), shared by the kernels that apply it.
#pragma once

#include "hgca_device.hpp"

namespace hgca {

constexpr int kRowBlock = 256;                   // threads of a workgroup that owns one (b, h) row
constexpr int kRowWaves = kRowBlock / kWave;
constexpr int kPerThread = 4;                    // elements a thread handles per step
constexpr int kRowStep = kRowBlock * kPerThread;
constexpr int kMaxRowBlock = 1024;               // the same for passes over long rows

__device__ __forceinline__ int32_t row_len(const int32_t *seq_lens, int b, int32_t cap) {
    return seq_lens ? min(max(seq_lens[b], 0), cap) : cap;
}

// Number of lanes below this one whose bit is set in `mask`.
__device__ __forceinline__ int lanes_below_in(uint64_t mask) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

struct CompactShared {
    int cnt[2][kPerThread * (kMaxRowBlock / kWave)];             // double-buffered: one barrier per step
};

// Called by all BLOCK threads of a workgroup.  Walks wr[0 .. n) in steps of 4 * BLOCK entries; sub-round e
// of a step covers entries [e*BLOCK, (e+1)*BLOCK) so that loads are coalesced and the output order is the
// position order: sub-round after sub-round, wave after wave.  Entry j passes iff (double)wr[j] > thr: the comparison is made in fp64 on the exactly
// widened weight.  The r-th passing entry goes to out[start + r] = j + value_offset (and its weight to
// wn[start + r] if wn != nullptr) as long as start + r < k_max.  Returns start + the number of passing
// entries seen (uniform over the workgroup; may exceed k_max).  With STOP_WHEN_FULL the walk ends once the list
// is full (the return value is then only a lower bound of the count); without it the whole row is examined, so
// that the caller learns whether anything was left out.  my_sum accumulates the weights this thread stored.
template <bool STOP_WHEN_FULL, int BLOCK = kRowBlock>
__device__ __forceinline__ int threshold_compact(CompactShared &sh, const float *wr, int n, double thr, int32_t *out,
                                                 int start, int k_max, int value_offset, float *wn, float &my_sum)
{
    const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid / kWave), lane = tid % kWave;
    constexpr int NW = BLOCK / kWave, STEP = BLOCK * kPerThread;
    static_assert(kPerThread * NW <= kWave && BLOCK <= kMaxRowBlock, "one lane per (sub-round, wave) count");
    int base = start;
    int buf = 0;
    // the loads of a step are issued one step ahead, so a step does not begin with a round trip to memory
    float nx[kPerThread];
#pragma unroll
    for (int e = 0; e < kPerThread; ++e) {
        const int t = e * BLOCK + tid;
        nx[e] = t < n ? wr[t] : 0.f;
    }
    for (int t0 = 0; t0 < n && (!STOP_WHEN_FULL || base < k_max); t0 += STEP, buf ^= 1) {
        float x[kPerThread];
        bool keep[kPerThread];
        int below[kPerThread];
#pragma unroll
        for (int e = 0; e < kPerThread; ++e) {
            x[e] = nx[e];
            const int tn = t0 + STEP + e * BLOCK + tid;
            nx[e] = tn < n ? wr[tn] : 0.f;
        }
#pragma unroll
        for (int e = 0; e < kPerThread; ++e) {
            const int t = t0 + e * BLOCK + tid;
            keep[e] = t < n && (double)x[e] > thr;
            const uint64_t mask = __ballot(keep[e]);
            below[e] = lanes_below_in(mask);
            if (lane == 0) sh.cnt[buf][e * NW + w] = __popcll(mask);
        }
        __syncthreads();
        // exclusive prefix over the (sub-round, wave) counts of the step, one count per lane
        const int c = lane < kPerThread * NW ? sh.cnt[buf][lane] : 0;
        const int incl = (int)wave_inclusive_scan((uint32_t)c), excl = incl - c;
#pragma unroll
        for (int e = 0; e < kPerThread; ++e) {
            const int pos = base + __builtin_amdgcn_readlane(excl, e * NW + w) + below[e];
            if (keep[e] && pos < k_max) {
                out[pos] = t0 + e * BLOCK + tid + value_offset;
                if (wn) wn[pos] = x[e];
                my_sum += x[e];
            }
        }
        base += __builtin_amdgcn_readlane(incl, kPerThread * NW - 1);
    }
    return base;
}

}  // namespace hgca

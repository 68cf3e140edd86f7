// Device-side helpers shared by the HGCA kernels (gfx950, wave64).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace hgca {

constexpr int kWave = 64;

struct bf16_t { uint16_t bits; };   // storage tag: upper half of an IEEE fp32

// One KV tier as the kernels see it (mirrors hgca_kv_view, pointers are device memory).
struct KvDev {
    const char *k, *v;
    const int32_t *seq_lens;
    const int32_t *block_table;
    const int32_t *first_block;     // paged only: per-sequence offset into the table row, or null
    int32_t cap, block_size, max_blocks;
    // N queries per sequence on a path written for one: batch index bv of the launch stands for query bv % n_q of
    // sequence bv / n_q (n_q <= 1: off).  With causal_tail the tier's last n_q valid tokens are the queries' own and
    // query i sees the tokens before position len - n_q + i + 1.
    int32_t n_q, causal_tail;
};

// Shape scalars passed by value to kernels.
struct ShapeDev {
    int32_t batch, n_q_heads, n_kv_heads, group;
    float sm_scale;
};

template <typename T> struct Elem;

template <> struct Elem<float> {
    static constexpr int kPerLoad = 4;            // elements in one 16-byte load
    static __device__ __forceinline__ void expand(const uint4 &r, float *f) {
        f[0] = __uint_as_float(r.x); f[1] = __uint_as_float(r.y);
        f[2] = __uint_as_float(r.z); f[3] = __uint_as_float(r.w);
    }
};

template <> struct Elem<bf16_t> {
    static constexpr int kPerLoad = 8;
    static __device__ __forceinline__ void expand(const uint4 &r, float *f) {
        f[0] = __uint_as_float(r.x << 16); f[1] = __uint_as_float(r.x & 0xffff0000u);
        f[2] = __uint_as_float(r.y << 16); f[3] = __uint_as_float(r.y & 0xffff0000u);
        f[4] = __uint_as_float(r.z << 16); f[5] = __uint_as_float(r.z & 0xffff0000u);
        f[6] = __uint_as_float(r.w << 16); f[7] = __uint_as_float(r.w & 0xffff0000u);
    }
};

// The sequence whose K/V rows batch index b of a launch reads.
__device__ __forceinline__ int kv_seq(const KvDev &kv, int b) { return kv.n_q > 1 ? b / kv.n_q : b; }

__device__ __forceinline__ int32_t tier_len(const KvDev &kv, int b) {
    const int seq = kv_seq(kv, b);
    const int32_t len = kv.seq_lens ? min(max(kv.seq_lens[seq], 0), kv.cap) : kv.cap;   // never beyond the buffer
    if (kv.n_q > 1 && kv.causal_tail) return min(max(len - kv.n_q + (b - seq * kv.n_q) + 1, 0), len);
    return len;
}

__device__ __forceinline__ uint4 load16(const char *p) {
    return *reinterpret_cast<const uint4 *>(p);
}

// 16-byte load marked non-temporal: K/V rows are streamed once and should not displace
// reusable lines in the caches.
__device__ __forceinline__ uint4 load16_stream(const char *p) {
    const uint32_t *w = reinterpret_cast<const uint32_t *>(p);
    uint4 r;
    r.x = __builtin_nontemporal_load(w + 0);
    r.y = __builtin_nontemporal_load(w + 1);
    r.z = __builtin_nontemporal_load(w + 2);
    r.w = __builtin_nontemporal_load(w + 3);
    return r;
}

// ---- reductions and prefix sums over lanes -----------------------------------------------------------------
// A lane shuffle (ds_bpermute) goes through the LDS pipeline: a round trip for each of the six steps of a wave's reduction, which is
// what short kernels consist of, and LDS issue slots, which is what bounds the score products on the vector units.  Inside a
// row of 16 lanes DPP modifiers bring the other lane's value in the instruction that uses it; v_permlane16_swap /
// v_permlane32_swap exchange rows of 16 and halves of 32 lanes.  All lanes of the wave take part.  Shuffles : exchanges, us:
// a step with a selection of 4 fp32 heads over 2 K tokens 15.9 : 14.8, of 7 x 32 / 8 fp32 heads over 10 K tokens 100.7 : 80.7,
// bf16, one sequence of 61 003 tokens 58.7 : 56.5, 8 of 28 672 140.9 : 138.9; fp32 lists shared by groups 43.9 : 34.0.
template <int kCtrl>
__device__ __forceinline__ float dpp(float x) {
    return __uint_as_float(__builtin_amdgcn_mov_dpp(__float_as_uint(x), kCtrl, 0xf, 0xf, true));
}
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E;          // quad_perm [1,0,3,2] and [2,3,0,1]
constexpr int kDppHalfMirror = 0x141, kDppMirror = 0x140;        // lane 7 - i of 8, lane 15 - i of 16
constexpr int kDppRor8 = 0x128;                          // lane i ^ 8 of 16

struct LanePair {
    float a, b;
};
// {x of the lower half, of the upper half} in every lane of 64, and the same for even and odd rows of 16 lanes
__device__ __forceinline__ LanePair halves_of(float x) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return {__uint_as_float(r[0]), __uint_as_float(r[1])};
}
__device__ __forceinline__ LanePair rows_of(float x) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return {__uint_as_float(r[0]), __uint_as_float(r[1])};
}

// op over kWidth adjacent lanes, the result in each of them; op has to be commutative and associative up to rounding
template <int kWidth, typename Op>
__device__ __forceinline__ float group_reduce(float v, Op op) {
    static_assert(kWidth >= 2 && kWidth <= kWave && (kWidth & (kWidth - 1)) == 0, "a power of two");
    v = op(v, dpp<kDppXor1>(v));
    if (kWidth >= 4) v = op(v, dpp<kDppXor2>(v));
    if (kWidth >= 8) v = op(v, dpp<kDppHalfMirror>(v));          // the lanes of a quad hold the same by now
    if (kWidth >= 16) v = op(v, dpp<kDppMirror>(v));
    if (kWidth >= 32) { const LanePair p = rows_of(v); v = op(p.a, p.b); }
    if (kWidth >= 64) { const LanePair p = halves_of(v); v = op(p.a, p.b); }
    return v;
}
template <int kWidth>
__device__ __forceinline__ float group_sum(float v) { return group_reduce<kWidth>(v, [](float a, float b) { return a + b; }); }
__device__ __forceinline__ float wave_sum(float v) { return group_sum<kWave>(v); }
__device__ __forceinline__ float wave_max(float v) { return group_reduce<kWave>(v, [](float a, float b) { return fmaxf(a, b); }); }
__device__ __forceinline__ float wave_min(float v) { return group_reduce<kWave>(v, [](float a, float b) { return fminf(a, b); }); }

// The sum over the lanes that share lane % kFrom (kFrom = 8, 16 or 32), in each of them.
template <int kFrom>
__device__ __forceinline__ float strided_sum(float v) {
    static_assert(kFrom == 8 || kFrom == 16 || kFrom == 32, "rows of 8, 16 or 32 lanes");
    if (kFrom <= 8) v += dpp<kDppRor8>(v);
    if (kFrom <= 16) { const LanePair p = rows_of(v); v = p.a + p.b; }
    const LanePair p = halves_of(v);
    return p.a + p.b;
}

// Inclusive prefix sum over the lanes of a row of 16.
__device__ __forceinline__ uint32_t row_inclusive_scan(uint32_t v) {
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, true);    // row_shr 1, 2, 4, 8
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, true);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, true);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, true);
    return v;
}

// Inclusive prefix sum over the wave's lanes.
__device__ __forceinline__ uint32_t wave_inclusive_scan(uint32_t v) {
    v = row_inclusive_scan(v);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false);   // row_bcast15 into rows 1 and 3
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false);   // row_bcast31 into rows 2 and 3
    return v;
}

}  // namespace hgca

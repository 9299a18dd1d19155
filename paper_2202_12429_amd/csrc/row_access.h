// Row-granular access shared by the cache, forward and backward kernels.
//
// A row is moved as pieces of 16 bytes (8 where bf16 rows are computed with), one piece per lane.  A row of `lpr` pieces
// (lanes per row) is handled by a group of GW consecutive lanes, GW the next power of two >= lpr (so four D=48 fp32
// rows, 12 pieces each, share a wavefront); lanes with piece index >= lpr idle.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "common.h"

namespace bp {

constexpr int kRowBlock = 256;   // threads per workgroup of the row kernels

inline int group_width(int lpr) {
    int gw = 1;
    while (gw < lpr) gw <<= 1;
    return gw;
}

// bf16 <-> fp32, round-to-nearest-even on the way down (NaN stays NaN)
__device__ __forceinline__ float bf16_bits_to_f32(uint32_t h) { return __uint_as_float(h << 16); }
__device__ __forceinline__ uint32_t f32_to_bf16_bits(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (u >> 16) | 0x40u;
    u += 0x7fffu + ((u >> 16) & 1u);
    return u >> 16;
}

// A lane's piece of a weight row as fp32 values: 4 of fp32 storage (16 bytes), 4 or 8 of bf16 storage (8 or 16 bytes).  SPLIT:
// its 8 values are 4 of the row's first half and 4 of its second, so that what is 16 bytes of fp32 for a lane lies beside its
// neighbour's.
template <bool BF16_, int N_, bool SPLIT = false>
struct Piece {
    static constexpr bool BF16 = BF16_;
    static constexpr int N = N_;
    static_assert(BF16 ? N == 4 || N == 8 : N == 4, "8 or 16 bytes");
    static_assert(!SPLIT || N == 8, "halves of four");
    typedef std::conditional_t<BF16 && (N == 4 || SPLIT), uint2, uint4> Unit;         // one access to the stored row
    typedef std::conditional_t<BF16 && N == 4, uint2, uint4> Raw;         // the piece as it is stored
    static constexpr int kPerVec = 16 / (int)sizeof(Unit);                // units in 16 bytes
    float v[N];
    static __device__ __forceinline__ Raw none() {
        Raw r = {};
        return r;
    }
    __device__ __forceinline__ void zero() {
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] = 0.f;
    }
    // the piece of lane c of a stored row, `lpr` lanes a row
    static __device__ __forceinline__ Raw fetch(const Unit* row, int c, int lpr) {
        if constexpr (SPLIT) {
            const uint2 a = row[c], b = row[c + lpr];
            return make_uint4(a.x, a.y, b.x, b.y);
        } else {
            return row[c];
        }
    }
    static __device__ __forceinline__ void put(Unit* row, const Raw& raw, int c, int lpr) {
        if constexpr (SPLIT) {
            row[c] = make_uint2(raw.x, raw.y);
            row[c + lpr] = make_uint2(raw.z, raw.w);
        } else {
            row[c] = raw;
        }
    }
    // first element of the i-th four
    static __device__ __forceinline__ int element(int c, int i, int lpr) { return SPLIT ? 4 * (c + i * lpr) : c * N + 4 * i; }
    __device__ __forceinline__ void decode(const Raw& raw) {
        if constexpr (BF16) {
            uint32_t r[N / 2];
            r[0] = raw.x;
            r[1] = raw.y;
            if constexpr (N == 8) {
                r[2] = raw.z;
                r[3] = raw.w;
            }
#pragma unroll
            for (int i = 0; i < N / 2; ++i) {
                v[2 * i] = bf16_bits_to_f32(r[i] & 0xffffu);
                v[2 * i + 1] = bf16_bits_to_f32(r[i] >> 16);
            }
        } else {
            v[0] = __uint_as_float(raw.x);
            v[1] = __uint_as_float(raw.y);
            v[2] = __uint_as_float(raw.z);
            v[3] = __uint_as_float(raw.w);
        }
    }
    __device__ __forceinline__ Raw encode() const {
        if constexpr (BF16) {
            uint32_t r[N / 2];
#pragma unroll
            for (int i = 0; i < N / 2; ++i) r[i] = f32_to_bf16_bits(v[2 * i]) | (f32_to_bf16_bits(v[2 * i + 1]) << 16);
            if constexpr (N == 8) return make_uint4(r[0], r[1], r[2], r[3]);
            else return make_uint2(r[0], r[1]);
        } else {
            return make_uint4(__float_as_uint(v[0]), __float_as_uint(v[1]), __float_as_uint(v[2]), __float_as_uint(v[3]));
        }
    }
    // fp32 [.. D] array (pooled output, upstream gradient, Adagrad state, partial sums): the piece of lane c
    // starts at element(c, 0, lpr) of the row.
    __device__ __forceinline__ void load_f32(const float* row, int c, int lpr) {
#pragma unroll
        for (int i = 0; i < N / 4; ++i) {
            const float4 t = *reinterpret_cast<const float4*>(row + element(c, i, lpr));
            v[4 * i] = t.x; v[4 * i + 1] = t.y; v[4 * i + 2] = t.z; v[4 * i + 3] = t.w;
        }
    }
    __device__ __forceinline__ void store_f32(float* row, int c, int lpr) const {
#pragma unroll
        for (int i = 0; i < N / 4; ++i)
            *reinterpret_cast<float4*>(row + element(c, i, lpr)) = make_float4(v[4 * i], v[4 * i + 1], v[4 * i + 2], v[4 * i + 3]);
    }
    // Streaming variant for data touched once (pooled output): non-temporal stores leave the cache lines to the table rows
    // that are reused.
    __device__ __forceinline__ void store_f32_stream(float* row, int c) const {
        static_assert(!SPLIT, "whole pieces");
        typedef float vec4 __attribute__((ext_vector_type(4)));
        vec4* p = reinterpret_cast<vec4*>(row + (size_t)c * N);
#pragma unroll
        for (int i = 0; i < N / 4; ++i) {
            vec4 t;
            t.x = v[4 * i]; t.y = v[4 * i + 1]; t.z = v[4 * i + 2]; t.w = v[4 * i + 3];
            __builtin_nontemporal_store(t, p + i);
        }
    }
    __device__ __forceinline__ void add(const Piece& o) {
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] += o.v[i];
    }
};

// Calls f.template run<GW>() for the lane groups of rows of `lpr` 16-byte pieces.
template <typename F>
int dispatch_row(int lpr, F&& f) {
#define BP_CASE(W) \
    case W: return f.template run<W>();
    switch (group_width(lpr)) {
        BP_CASE(1) BP_CASE(2) BP_CASE(4) BP_CASE(8) BP_CASE(16) BP_CASE(32) BP_CASE(64)
        default: return fail(BP_ERR_UNSUPPORTED, "row of %d 16-byte pieces is wider than 1024 bytes", lpr);
    }
#undef BP_CASE
}

// Calls f.template run<GW, Piece>(lanes per row) for the kernels that compute with a row's values.  bf16 rows go by fours or by
// eights a lane.  By fours a lane's fp32 operands (gradients, pooled rows, state) are 16 bytes beside its neighbour's and take
// half the registers; by eights a lane group is half as wide, and a wavefront has twice the rows in flight.  Forward, us by
// eights / by fours, one lookup a bag: 1.3 M of dim 128, pooled rows written six batches in turn 187 / 177, always the same
// 293 / 120; over row records 147 / 135; 30,000 of dim 24: 4.1 / 3.7, 6.7 / 5.9.  Which is quicker depends on where the buffers
// lie, by something that their distance does not tell (cache and pooled rows in one allocation, twenty distances of 0 to 300 MB:
// 185 to 191 / 164 to 166).  In a training step on a cache of 16 M rows, twelve placements: by eights 170 to 171 in ten and 197
// and 199 in two, by fours 176 to 182; but the backward pass behind it takes 228 to 242 after eights, 216 to 243 after fours,
// both together 414 / 410 in the mean.  Pooling reads more than it writes, and 16 bytes a lane of the row come cheaper
// than 8: 65,535 bags of 25 in the mean, dim 128: 35 / 51 (pooled_by_eights has the rule).  Rows wider than 64 lanes by fours
// are taken by eights.
template <bool SPLIT, typename F>
int dispatch_values(const bp_config* cfg, bool eights, F&& f) {
    const bool bf16 = cfg->weight_dtype == BP_BF16;
    const int lanes = cfg->dim / 4;
    if (bf16 && (eights || lanes > 64)) {
#define BP_CASE(W) \
    case W: return f.template run<W, Piece<true, 8, SPLIT>>(lanes / 2);
        switch (group_width(lanes / 2)) {
            BP_CASE(1) BP_CASE(2) BP_CASE(4) BP_CASE(8) BP_CASE(16) BP_CASE(32) BP_CASE(64)
            default: return fail(BP_ERR_UNSUPPORTED, "row of %zu bytes is wider than 1024", row_bytes(cfg));
        }
#undef BP_CASE
    }
#define BP_CASE(W) \
    case W: return bf16 ? f.template run<W, Piece<true, 4>>(lanes) : f.template run<W, Piece<false, 4>>(lanes);
    switch (group_width(lanes)) {
        BP_CASE(1) BP_CASE(2) BP_CASE(4) BP_CASE(8) BP_CASE(16) BP_CASE(32) BP_CASE(64)
        default: return fail(BP_ERR_UNSUPPORTED, "row of %zu bytes is wider than 1024", row_bytes(cfg));
    }
#undef BP_CASE
}

}  // namespace bp

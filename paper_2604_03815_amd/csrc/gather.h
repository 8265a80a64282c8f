// Row gathers of the aggregate and of the backward's coefficient pass.
//
// A team of 16 lanes (one DPP row) serves a query-head.  A bf16 row of D
// values is read by D/8 neighbouring lanes, 16 bytes each, so that a load
// instruction touches each row's cache line once: the CU's cache looks up
// about one line a clock, and a lane that reads a whole row by itself makes
// D/8 lookups of it (at k = 128, d = 64 and 262k query-heads 537M lookups for
// K and V, 0.87 ms of the 0.92 ms the aggregate took that way).  The team
// takes RPT = 128/D rows per step; lane tl holds dimensions 8 c .. 8 c + 7,
// c = tl % (D/8), of the step's row tl / (D/8).
#pragma once

#include "kmip_device.h"

namespace kmip {

template <int D>
struct RowSplit {
    static constexpr int LPR = D / 8;       // lanes per row
    static constexpr int RPT = 16 / LPR;    // rows per team and step
    static constexpr int U = LPR < 8 ? LPR : 8;   // steps whose loads go out together (at most 16 rows)
    static_assert(LPR >= 2 && LPR <= 16, "row widths 16 .. 128");
};

// Eight bf16 of a row as floats.
__device__ __forceinline__ void widen8(float (&f)[8], const uint4& u) {
    const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        f[2 * e] = bf16_bits_to_f32(w[e] & 0xFFFFu);
        f[2 * e + 1] = bf16_bits_to_f32(w[e] >> 16);
    }
}

__device__ __forceinline__ float dot8(const float (&q)[8], const uint4& u) {
    const uint32_t w[4] = {u.x, u.y, u.z, u.w};
    float s = 0.0f;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        s = fmaf(q[2 * e], bf16_bits_to_f32(w[e] & 0xFFFFu), s);
        s = fmaf(q[2 * e + 1], bf16_bits_to_f32(w[e] >> 16), s);
    }
    return s;
}

__device__ __forceinline__ void axpy8(float (&acc)[8], float a, const uint4& u) {
    const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        acc[2 * e] = fmaf(a, bf16_bits_to_f32(w[e] & 0xFFFFu), acc[2 * e]);
        acc[2 * e + 1] = fmaf(a, bf16_bits_to_f32(w[e] >> 16), acc[2 * e + 1]);
    }
}

// Sum over the LPR lanes of a row, for each of them (after the quad steps a
// quad holds one value, so the mirrors' other lane order does not matter).
template <int LPR>
__device__ __forceinline__ float row_lanes_sum(float v) {
    v += step_partner<1>(v);
    if constexpr (LPR >= 4) v += step_partner<2>(v);
    if constexpr (LPR >= 8) v += step_partner<4>(v);
    if constexpr (LPR >= 16) v += step_partner<8>(v);
    return v;
}

// The value of lane tl ^ M (M = 8, 4, 2), the other bits kept.
template <int M>
__device__ __forceinline__ float xor_lane(float v) {
    static_assert(M == 8 || M == 4 || M == 2, "");
    if constexpr (M == 8) return row_perm<0x128>(v);                                   // row_ror:8
    if constexpr (M == 4) return row_perm<0x1B>(row_perm<kDppRowHalfMirror>(v));       // ^7, then ^3
    return row_perm<kDppQuadSwap2>(v);
}

// Sums acc over the team's RPT row groups, scattered: lane tl ends up with
// 8/RPT of its eight dimensions in acc[0 ..], the first of them at
// scatter_dim<D>(tl) of the row.
template <int D>
__device__ __forceinline__ void scatter_rows_sum(float (&acc)[8], int tl) {
    constexpr int RPT = RowSplit<D>::RPT;
    if constexpr (RPT >= 2) {
        const bool hi = (tl & 8) != 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float own = hi ? acc[4 + e] : acc[e], other = hi ? acc[e] : acc[4 + e];
            acc[e] = own + xor_lane<8>(other);
        }
    }
    if constexpr (RPT >= 4) {
        const bool hi = (tl & 4) != 0;
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const float own = hi ? acc[2 + e] : acc[e], other = hi ? acc[e] : acc[2 + e];
            acc[e] = own + xor_lane<4>(other);
        }
    }
    if constexpr (RPT >= 8) {
        const bool hi = (tl & 2) != 0;
        const float own = hi ? acc[1] : acc[0], other = hi ? acc[0] : acc[1];
        acc[0] = own + xor_lane<2>(other);
    }
}

template <int D>
__device__ __forceinline__ int scatter_dim(int tl) {
    constexpr int LPR = RowSplit<D>::LPR, RPT = RowSplit<D>::RPT;
    int t = 8 * (tl & (LPR - 1));
    if constexpr (RPT >= 2) t += (tl & 8) ? 4 : 0;
    if constexpr (RPT >= 4) t += (tl & 4) ? 2 : 0;
    if constexpr (RPT >= 8) t += (tl & 2) ? 1 : 0;
    return t;
}

// Writes the scattered sums, times f, to the row at p.
template <int D>
__device__ __forceinline__ void store_scattered(float* __restrict__ p, const float (&acc)[8], float f, int tl) {
    constexpr int RPT = RowSplit<D>::RPT;
    float* dst = p + scatter_dim<D>(tl);
#pragma unroll
    for (int e = 0; e < 8 / RPT; ++e) dst[e] = f * acc[e];
}

}  // namespace kmip

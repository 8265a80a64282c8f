// Gather-softmax-aggregate for k-MIP attention on gfx950.
//
// Algorithm 1 (Appendix E) of arXiv 2604.03815 after RowwiseTopK: gather the
// k selected value rows (GatherRows), take a softmax over the k kept scores
// times `scale`, and sum the weighted rows (Einsum nk,nkv->nv).  The kept
// scores are recomputed in fp32 from q_i and the gathered key rows, with the
// same routine the backward uses, so the weights of the two passes agree.
//
// Mapping: a team of 16 lanes per (query, head), 16 teams per workgroup (4 for
// k > 128), or four teams that share its rounds.  Rows are read by D/8 lanes each (gather.h), 128/D rows per team
// and step.  The team's key indices go to LDS first, and the slots after the
// last one kept are left out (graphs of fewer than k nodes: 85 nodes, 8 heads, d =
// 64, k = 512 53 us with them, 16 without); a step's lanes form
// their rows' scores, which go to LDS beside the indices; the softmax runs
// with the slots on lanes (slot = lane + 16 s); and the value rows are gathered
// with the weights read back from LDS.  A team lies within a wave, whose LDS
// instructions execute in order, so no barrier is needed.
//
// Bound by the cache lines the gathers look up (one a clock and CU), the round
// trips and, where the rows of a head do not stay in L2, the fabric.  Against a
// lane per row (us): 262k nodes, d = 64, k = 128 925 -> 340; 100k nodes, 4
// heads, d = 32, k = 32 241 -> 162; 500k nodes, 4 heads, d = 16, k = 32 520 ->
// 420; a batch of 128 graphs, d = 32, k = 16 37 -> 22.
//
// Attention dropout (keep != nullptr): slot t's weight in the sum is
// multiplied by keep_scale when keep[qh k + t] is nonzero and by 0
// otherwise; the softmax statistics (lse) are those before dropout.
//
// Order: without perm, the query-heads as they lie (neighbouring queries, all
// heads), or one head after the other (head_blocks workgroups each, where
// gather_by_head says so).  With a query order perm [H][N] (the forward's
// grouping of the queries by direction), block (b, h) takes positions 16 b ..
// 16 b + 15 of head h in that order: queries of one group select mostly the
// same keys, so the teams of a workgroup gather the same rows.
#include "gather.h"
#include "kmip_device.h"
#include "kmip_internal.h"

namespace kmip {
namespace {

// Steps whose loads go out together: the rows of S slots, at least one step
// and, at 16 slots, at most 8 loads a lane.
constexpr int round_steps(int s, int rpt) {
    const int u = s > rpt ? s / rpt : 1;
    return s == 16 && u > 8 ? 8 : u;
}

// Slots a team's area holds: k rounded up to whole rounds.
template <int S>
__host__ __device__ constexpr int slots_of(int k) {
    constexpr int r = S > 16 ? S : 16;
    return (k + r - 1) / r * r;
}

// Words between the LDS areas of two teams: {index, score or weight} of every
// slot, and 16 words so that the four teams of a wave meet different banks.
template <int S>
__host__ __device__ constexpr int attend_stride(int k) {
    return 2 * slots_of<S>(k) + 16;
}

// Maximum and sum over the lanes of P teams.
template <int P>
__device__ __forceinline__ float teams_max(float v) {
    v = group16_max(v);
#pragma unroll
    for (int m = 16; m < 16 * P; m <<= 1) v = fmaxf(v, __shfl_xor(v, m));
    return v;
}

template <int P>
__device__ __forceinline__ float teams_sum(float v) {
    v = group16_sum(v);
#pragma unroll
    for (int m = 16; m < 16 * P; m <<= 1) v += __shfl_xor(v, m);
    return v;
}

constexpr int kIdxLoads = 4;   // index loads of a lane in flight

template <int D, int DV, int S, int P>
__global__ __launch_bounds__(256) void attend_kernel(
    const uint16_t* __restrict__ Q, const uint16_t* __restrict__ K, const uint16_t* __restrict__ V,
    const int32_t* __restrict__ idx, const uint8_t* __restrict__ keep, float keep_scale, int32_t N,
    int32_t H, int32_t k, float scale, const int32_t* __restrict__ perm, int32_t head_blocks, float* __restrict__ out,
    float* __restrict__ lse) {
    extern __shared__ int32_t lds[];
    // P teams share a query-head: team `part` takes every P-th round
    constexpr int TL = 16 * P;
    const int tl = threadIdx.x & 15, team = threadIdx.x / TL, teams = blockDim.x / TL;
    const int part = P > 1 ? (threadIdx.x >> 4) & (P - 1) : 0, pl = threadIdx.x & (TL - 1);
    int64_t qh;
    int h;
    if (perm != nullptr || head_blocks > 0) {
        h = perm != nullptr ? blockIdx.y : blockIdx.x / head_blocks;
        const int64_t p = (int64_t)(perm != nullptr ? blockIdx.x : blockIdx.x - h * head_blocks) * teams + team;
        if (p >= N) return;  // whole team exits together
        qh = (perm != nullptr ? (int64_t)perm[(size_t)h * N + p] : p) * H + h;
    } else {
        qh = (int64_t)blockIdx.x * teams + team;
        if (qh >= (int64_t)N * H) return;  // whole team exits together
        h = (int)(qh % H);
    }
    int2* const sh = reinterpret_cast<int2*>(lds + (size_t)team * attend_stride<S>(k));
    auto put = [&](int slot, int32_t j) {
        const bool kept = j >= 0 && j < N;
        sh[slot].x = kept ? j : -1;
        return kept;
    };
    int last = k;   // slots past it are not looked at
    if (k <= 16) {
        if (P == 1 || part == 0) put(tl, tl < k ? idx[(size_t)qh * k + tl] : -1);
    } else {
        last = 0;
        for (int s0 = pl; s0 < slots_of<S>(k); s0 += TL * kIdxLoads) {
            int32_t j[kIdxLoads];
#pragma unroll
            for (int u = 0; u < kIdxLoads; ++u) {
                const int slot = s0 + TL * u;
                j[u] = slot < k ? idx[(size_t)qh * k + slot] : -1;
            }
#pragma unroll
            for (int u = 0; u < kIdxLoads; ++u)
                if (s0 + TL * u < slots_of<S>(k) && put(s0 + TL * u, j[u])) last = s0 + TL * u + 1;
        }
        last = (int)teams_max<P>((float)last);   // (at most 512)
    }
    __builtin_amdgcn_wave_barrier();

    using KS = RowSplit<D>;
    using VS = RowSplit<DV>;
    constexpr int KU = round_steps(S, KS::RPT), VU = round_steps(S, VS::RPT);
    {
        float q[8];
        widen8(q, *reinterpret_cast<const uint4*>(Q + (size_t)qh * D + 8 * (tl & (KS::LPR - 1))));
        const int g = tl / KS::LPR;
        const uint16_t* kcol = K + (size_t)h * D + 8 * (tl & (KS::LPR - 1));
        for (int s0 = part * KS::RPT * KU; s0 < last; s0 += P * KS::RPT * KU) {
            int32_t j[KU];
            uint4 w[KU];
#pragma unroll
            for (int u = 0; u < KU; ++u) {
                j[u] = sh[s0 + KS::RPT * u + g].x;
                w[u] = *reinterpret_cast<const uint4*>(kcol + (size_t)(j[u] >= 0 ? j[u] : 0) * ((size_t)H * D));
            }
#pragma unroll
            for (int u = 0; u < KU; ++u) {
                const float z = scale * row_lanes_sum<KS::LPR>(dot8(q, w[u]));
                if ((tl & (KS::LPR - 1)) == 0) sh[s0 + KS::RPT * u + g].y = __float_as_int(j[u] >= 0 ? z : -INFINITY);
            }
        }
    }
    __builtin_amdgcn_wave_barrier();

    // The first value rows go out before the softmax.
    const int g = tl / VS::LPR;
    const uint16_t* vcol = V + (size_t)h * DV + 8 * (tl & (VS::LPR - 1));
    auto value_rows = [&](uint4 (&w)[VU], int s0) {
#pragma unroll
        for (int u = 0; u < VU; ++u) {
            const int32_t j = sh[s0 + VS::RPT * u + g].x;
            w[u] = *reinterpret_cast<const uint4*>(vcol + (size_t)(j >= 0 ? j : 0) * ((size_t)H * DV));
        }
    };
    uint4 w[VU];
    int s0 = part * VS::RPT * VU;
    value_rows(w, P == 1 || s0 < last ? s0 : 0);

    float zmax = -INFINITY;
    for (int slot = pl; slot < last; slot += TL) zmax = fmaxf(zmax, __int_as_float(sh[slot].y));
    zmax = teams_max<P>(zmax);
    float zs = 0.0f;
    for (int slot = pl; slot < last; slot += TL) {
        const int2 e = sh[slot];
        float p = e.x >= 0 ? __expf(__int_as_float(e.y) - zmax) : 0.0f;
        zs += p;
        if (keep != nullptr && e.x >= 0) p *= keep[(size_t)qh * k + slot] != 0 ? keep_scale : 0.0f;
        sh[slot].y = __float_as_int(p);
    }
    zs = teams_sum<P>(zs);
    __builtin_amdgcn_wave_barrier();

    float acc[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] = 0.0f;
    while (s0 < last) {
#pragma unroll
        for (int u = 0; u < VU; ++u) {
            const int2 e = sh[s0 + VS::RPT * u + g];
            if (e.x >= 0) axpy8(acc, __int_as_float(e.y), w[u]);
        }
        s0 += P * VS::RPT * VU;
        if (s0 < last) value_rows(w, s0);
    }
    if constexpr (P > 1) {
#pragma unroll
        for (int e = 0; e < 8; ++e)
#pragma unroll
            for (int m = 16; m < TL; m <<= 1) acc[e] += __shfl_xor(acc[e], m);
        if (part != 0) return;
    }
    scatter_rows_sum<DV>(acc, tl);
    const bool any = zmax != -INFINITY;
    store_scattered<DV>(out + (size_t)qh * DV, acc, any ? 1.0f / zs : 0.0f, tl);
    if (tl == 0) lse[qh] = any ? zmax + __logf(zs) : -INFINITY;
}

}  // namespace

hipError_t launch_attend(const void* Q, const void* K, const void* V, const int32_t* idx,
                         const uint8_t* keep, float keep_scale, int32_t N, int32_t H, int32_t d, int32_t dv,
                         int32_t k, float scale, const int32_t* perm, bool one_graph, float* out, float* lse,
                         hipStream_t stream) {
    const int64_t nqh = (int64_t)N * H;
    if (nqh == 0) return hipSuccess;
    // 16 teams a workgroup; with more than 128 slots a team's LDS area would
    // leave few of them per CU, so a workgroup is one wave
    // Four teams (a wave, a workgroup) share a query-head while there are few of
    // them, since a team's chain of rounds takes longer than the chip's work
    // (one team, four; a lane per row in brackets; us): 931 nodes, d = 32, k = 128
    // 12.1, 6.4 [9.3]; 2,082 nodes, d = 32, k = 200 18.1, 9.6 [12.7]; 1,192 nodes, 4
    // heads, d = 128, k = 50 16.7, 12.6 [28.6]; 6,088 nodes, d = 16, k = 128 10.5,
    // 10.5 [10.3]; 7,575 nodes, 2 heads, d = 32, k = 64 10.5, 13.4 [18.0]; past 128
    // slots 9,768 nodes, d = 32, d_V = 64, k = 256 34.6, 26.7 [60.5]; 14,318 nodes, d =
    // 16, k = 200 26.4, 28.8 [26.3].
    const int parts = k > 32 && nqh <= (k > 128 ? 12288 : 6144) ? 4 : 1;
    const int teams = parts > 1 ? 1 : k > 128 ? 4 : 16;
    // Slots a round: up to four where there are no more (258k nodes, 2 heads, d =
    // 64, k = 1 87 -> 56 us; 16k nodes, 8 heads, d = 16, k = 1 14.9 -> 13.3); past
    // 256, where the LDS holds two or three waves per SIMD, 64 while a head's rows
    // stay in the L2 (12.5k nodes, 4 heads, d = 16, k = 512 263 -> 178; 10k nodes, 4
    // heads, d = 32, normal rows 247 -> 204).  Beyond, more rows in flight push each
    // other out of it (30k nodes, d = 32, k = 300, normal rows 413 -> 445; 100k, d =
    // 16, k = 512 3796 -> 4237), and wider rows cost more registers than they gain.
    const bool in_l2 = (int64_t)N * (d + dv) <= 5 << 18;   // 2.5 of the 4 MB
    const int round = k <= 4 ? 4 : k > 256 && d <= 32 && dv <= 32 && in_l2 && parts == 1 ? 64 : 16;
    const int32_t per_head = (N + teams - 1) / teams, head_blocks = perm == nullptr && gather_by_head(N, H, d, dv, k, one_graph) ? per_head : 0;
    const dim3 blocks = perm != nullptr   ? dim3((unsigned)per_head, (unsigned)H)
                        : head_blocks > 0 ? dim3((unsigned)((int64_t)per_head * H))
                                          : dim3((unsigned)((nqh + teams - 1) / teams));
    const uint16_t* q = reinterpret_cast<const uint16_t*>(Q);
    const uint16_t* kk = reinterpret_cast<const uint16_t*>(K);
    const uint16_t* v = reinterpret_cast<const uint16_t*>(V);
#define KMIP_ATTEND_ROUND(DD, DVV, SS, PP)                                                                     \
    if (round == SS && parts == PP) {                                                                          \
        hipLaunchKernelGGL((attend_kernel<DD, DVV, SS, PP>), blocks, dim3(16 * PP * teams),                    \
                           teams * attend_stride<SS>(k) * sizeof(int32_t), stream, q, kk, v, idx, keep, keep_scale, \
                           N, H, k, scale, perm, head_blocks, out, lse);                                       \
        return hipGetLastError();                                                                              \
    }
#define KMIP_ATTEND_CASE(DD, DVV)       \
    if (d == DD && dv == DVV) {         \
        KMIP_ATTEND_ROUND(DD, DVV, 4, 1)   \
        KMIP_ATTEND_ROUND(DD, DVV, 16, 1)  \
        KMIP_ATTEND_ROUND(DD, DVV, 16, 4)  \
        if constexpr (DD <= 32 && DVV <= 32) KMIP_ATTEND_ROUND(DD, DVV, 64, 1) \
    }
#define KMIP_ATTEND_D(DD) \
    KMIP_ATTEND_CASE(DD, 16) KMIP_ATTEND_CASE(DD, 32) KMIP_ATTEND_CASE(DD, 64) KMIP_ATTEND_CASE(DD, 128)
    KMIP_ATTEND_D(16)
    KMIP_ATTEND_D(32)
    KMIP_ATTEND_D(64)
    KMIP_ATTEND_D(128)
#undef KMIP_ATTEND_D
#undef KMIP_ATTEND_CASE
#undef KMIP_ATTEND_ROUND
    return hipErrorInvalidValue;
}

}  // namespace kmip

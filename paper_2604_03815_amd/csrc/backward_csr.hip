// Backward of k-MIP attention with a key-sorted segmented reduction.
//
// Same gradients as backward.hip (index set held fixed; Section 3.1, last
// paragraph, and Appendix E, last paragraph, of arXiv 2604.03815):
//   dQ_i = scale sum_j g_ij k_j,  dK_j = sum_i a_ij q_i,  dV_j = sum_i p_ij dO_i
// with a_ij = scale g_ij.  Instead of scattering every pair's rows with
// atomics, the pairs are sorted by key (a counting sort on the key row
// j*H + h), and each key's rows are summed in registers over its run:
//   1. coef:   per (query, head): p, dp, D, g; dQ_i; coefficients (a, p) of
//              each selected pair, stored in pair order;
//   2. count:  pairs per key row;
//   3. scan:   exclusive prefix sum of the counts (three small kernels);
//   4. place:  the pairs' records (key row, query, coefficients) in key
//              order (the scanned counts serve as cursors);
//   5. reduce: fixed chunks of the sorted pairs; a team of 16 lanes walks a
//              contiguous stretch, dimensions on lanes, keeps the running
//              sums of the current key in registers and adds them to dK and
//              dV with one atomic per dimension where the key changes or
//              the stretch ends.
// Counting and placing aggregate equal key rows within a workgroup of 256
// queries first, so a key that most queries select costs one global atomic
// per workgroup, not one per pair.
#include "gather.h"
#include "kmip_device.h"
#include "kmip_internal.h"

#include <algorithm>

namespace kmip {
namespace {

constexpr int kScanBlock = 1024;     // counts per block of the scan
constexpr int kChunk = 1024;         // sorted pairs per wave in the reduction

// 1. Per (query, head), a team of 16 lanes, NS slots per lane (k <= 16 NS):
// p, dp, D, g of each selected pair, dQ_i, and (QGt != nullptr) row qg_row of
// the interleaved copy of q_i and dO_i.  D is the
// query/key width, DV the value width (dp_j runs over it).  Slot tl + 16 s
// leaves its key index in jj[s] (-1: none) and its coefficients a = scale g, p
// in ca[s], cp[s].  With attention dropout (keep != nullptr, f = keep_scale or
// 0 by the slot's keep draw) dp is replaced by f dp and the dV coefficient is
// p f.
//
// The inputs of a query-head (coef_fetch) are fetched apart, so that a team
// that takes several fetches the next one's while it works on one.  Key and
// value rows are read by D/8 and DV/8 lanes each (gather.h); a step's lanes
// leave s and dp of their rows in the team's LDS area, from where each lane
// takes its slots', and g goes back the same way for dQ.  Against a lane per
// row the coefficient passes went from the cache's line lookups to the
// round trips as their bound.
template <int NS>
struct CoefIn {
    int32_t j[NS];   // this lane's key slots tl + 16 s (-1: none)
    uint4 qw, gw;    // this lane's eight dimensions of q_i and dO_i
    float l;         // lse (-inf: no key kept, or no query-head)
    int64_t qh;
    bool valid;
};

template <int D, int DV, int NS>
__device__ __forceinline__ void coef_fetch(const uint16_t* __restrict__ Q, const uint16_t* __restrict__ dO,
                                           const int32_t* __restrict__ idx, const float* __restrict__ lse,
                                           int32_t N, int32_t k, bool valid, int64_t qh, int tl, CoefIn<NS>& in) {
    in.valid = valid;
    in.qh = valid ? qh : 0;
    in.l = -INFINITY;
    in.qw = in.gw = make_uint4(0, 0, 0, 0);
#pragma unroll
    for (int s = 0; s < NS; ++s) in.j[s] = -1;
    if (valid) {
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const int slot = tl + 16 * s;
            // a pair exists wherever its index lies in [0, N), as the counting
            // pass sees it; its weight is zero if lse says no key was kept
            const int32_t j = slot < k ? idx[(size_t)qh * k + slot] : -1;
            in.j[s] = j >= 0 && j < N ? j : -1;
        }
        in.qw = *reinterpret_cast<const uint4*>(Q + (size_t)qh * D + 8 * (tl & (RowSplit<D>::LPR - 1)));
        in.gw = *reinterpret_cast<const uint4*>(dO + (size_t)qh * DV + 8 * (tl & (RowSplit<DV>::LPR - 1)));
        in.l = lse[qh];
    }
}

// Bytes of a team's LDS area: {s, dp} and the key index of every slot, and 16
// words so that the four teams of a wave meet different banks.
__host__ __device__ constexpr size_t coef_area(int ns) { return (size_t)ns * 16 * 12 + 64; }

template <int D, int DV, int NS, int KEEP_REGS>
__device__ __forceinline__ void coef_team(const CoefIn<NS>& in, const uint16_t* __restrict__ K,
                                          const uint16_t* __restrict__ V, const uint8_t* __restrict__ keep,
                                          float keep_scale, int32_t H, int32_t k, float scale, int tl, char* area,
                                          float* __restrict__ dQ, uint16_t* __restrict__ QGt, size_t qg_row,
                                          int32_t (&jj)[NS], float (&ca)[NS], float (&cp)[NS]) {
    using KS = RowSplit<D>;
    using VS = RowSplit<DV>;
    constexpr int K16 = 16 * NS;
    constexpr int KST = K16 / KS::RPT;            // steps over the key rows
    constexpr bool kKeep = 4 * KST <= KEEP_REGS;  // key rows kept in registers for dQ, else read again
    float2* const sd = reinterpret_cast<float2*>(area);        // [K16] s, dp; then .x = g
    int32_t* const js = reinterpret_cast<int32_t*>(sd + K16);  // [K16]
    const int64_t qh = in.qh;
    const int h = (int)(qh % H);
    if (QGt != nullptr && in.valid) {
        // row qg_row of the interleaved copy, q_i then dO_i, so that the
        // reduction gathers both with one load
        uint4* const row = reinterpret_cast<uint4*>(QGt + qg_row * (D + DV));
        if (tl < KS::LPR) row[tl] = in.qw;
        if (tl < VS::LPR) row[KS::LPR + tl] = in.gw;
    }
    float q[8], g[8];
    widen8(q, in.qw);
    widen8(g, in.gw);
    const bool live = in.l != -INFINITY;
    // Rows that are read twice are read up to the last slot kept (70 nodes, 8
    // heads, d = 64, k = 512 48 -> 15 us).
    int last = kKeep ? K16 : 0;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        jj[s] = in.j[s];
        js[tl + 16 * s] = live ? in.j[s] : -1;
        if (!kKeep && live && in.j[s] >= 0) last = tl + 16 * s + 1;
    }
    if constexpr (!kKeep) last = (int)group16_max((float)last);   // (at most 512)
    __builtin_amdgcn_wave_barrier();
    const int gk = tl / KS::LPR, gv = tl / VS::LPR;
    const uint16_t* kcol = K + (size_t)h * D + 8 * (tl & (KS::LPR - 1));
    const uint16_t* vcol = V + (size_t)h * DV + 8 * (tl & (VS::LPR - 1));
    auto key_row = [&](int32_t j) {
        return *reinterpret_cast<const uint4*>(kcol + (size_t)(j >= 0 ? j : 0) * ((size_t)H * D));
    };
    auto value_row = [&](int32_t j) {
        return *reinterpret_cast<const uint4*>(vcol + (size_t)(j >= 0 ? j : 0) * ((size_t)H * DV));
    };
    uint4 kw[kKeep ? KST : 1];
    auto dots = [&](int i0, auto keeps) {
        // KS::U steps from i0 (equal widths: both rows; else the key rows)
        int32_t j[KS::U];
        uint4 a[KS::U], b[KS::U];
#pragma unroll
        for (int u = 0; u < KS::U; ++u) {
            j[u] = js[KS::RPT * (i0 + u) + gk];
            a[u] = key_row(j[u]);
            if constexpr (DV == D) b[u] = value_row(j[u]);
        }
#pragma unroll
        for (int u = 0; u < KS::U; ++u) {
            const float sv = row_lanes_sum<KS::LPR>(dot8(q, a[u]));
            if constexpr (DV == D) {
                const float dv = row_lanes_sum<KS::LPR>(dot8(g, b[u]));
                if ((tl & (KS::LPR - 1)) == 0) sd[KS::RPT * (i0 + u) + gk] = make_float2(sv, dv);
            } else {
                if ((tl & (KS::LPR - 1)) == 0) sd[KS::RPT * (i0 + u) + gk].x = sv;
            }
            if constexpr (kKeep) keeps(u, a[u]);
        }
    };
    if constexpr (kKeep) {
#pragma unroll
        for (int i0 = 0; i0 < KST; i0 += KS::U) dots(i0, [&](int u, const uint4& w) { kw[i0 + u] = w; });
    } else {
#pragma unroll 1
        for (int i0 = 0; KS::RPT * i0 < last; i0 += KS::U) dots(i0, [](int, const uint4&) {});
    }
    if constexpr (DV != D) {
#pragma unroll 1
        for (int i0 = 0; VS::RPT * i0 < last; i0 += VS::U) {
            uint4 b[VS::U];
#pragma unroll
            for (int u = 0; u < VS::U; ++u) b[u] = value_row(js[VS::RPT * (i0 + u) + gv]);
#pragma unroll
            for (int u = 0; u < VS::U; ++u) {
                const float dv = row_lanes_sum<VS::LPR>(dot8(g, b[u]));
                if ((tl & (VS::LPR - 1)) == 0) sd[VS::RPT * (i0 + u) + gv].y = dv;
            }
        }
    }
    __builtin_amdgcn_wave_barrier();
    // the slots on lanes
    float p[NS], dp[NS];
    float dsum = 0.0f;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const int slot = tl + 16 * s;
        p[s] = dp[s] = cp[s] = 0.0f;
        if (jj[s] >= 0 && live) {
            const float2 e = sd[slot];
            p[s] = __expf(scale * e.x - in.l);
            dp[s] = e.y;
            cp[s] = p[s];
            if (keep != nullptr) {
                const float f = keep[(size_t)qh * k + slot] != 0 ? keep_scale : 0.0f;
                dp[s] *= f;
                cp[s] = p[s] * f;
            }
        }
        dsum = fmaf(p[s], dp[s], dsum);
    }
    dsum = group16_sum(dsum);
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const float gs = p[s] * (dp[s] - dsum);
        ca[s] = scale * gs;
        sd[tl + 16 * s].x = gs;
    }
    __builtin_amdgcn_wave_barrier();
    // dQ_i = scale sum_j g_j k_j
    float acc[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] = 0.0f;
    if constexpr (kKeep) {
#pragma unroll
        for (int i = 0; i < KST; ++i)
            if (js[KS::RPT * i + gk] >= 0) axpy8(acc, sd[KS::RPT * i + gk].x, kw[i]);
    } else {
#pragma unroll 1
        for (int i0 = 0; KS::RPT * i0 < last; i0 += KS::U) {
            int32_t j[KS::U];
            uint4 w[KS::U];
#pragma unroll
            for (int u = 0; u < KS::U; ++u) {
                j[u] = js[KS::RPT * (i0 + u) + gk];
                w[u] = key_row(j[u]);
            }
#pragma unroll
            for (int u = 0; u < KS::U; ++u)
                if (j[u] >= 0) axpy8(acc, sd[KS::RPT * (i0 + u) + gk].x, w[u]);
        }
    }
    __builtin_amdgcn_wave_barrier();   // the next query-head reuses the area
    scatter_rows_sum<D>(acc, tl);
    if (in.valid) store_scattered<D>(dQ + (size_t)qh * D, acc, scale, tl);
}

// The coefficients of every pair, in pair order (the segmented variant).
template <int D, int DV, int NS>
__global__ __launch_bounds__(256) void csr_coef_kernel(
    const uint16_t* __restrict__ Q, const uint16_t* __restrict__ K, const uint16_t* __restrict__ V,
    const uint16_t* __restrict__ dO, const int32_t* __restrict__ idx, const float* __restrict__ lse,
    int32_t N, int32_t H, int32_t k, float scale, float* __restrict__ dQ, float2* __restrict__ coef,
    const uint8_t* __restrict__ keep, float keep_scale, int32_t head_blocks) {
    extern __shared__ uint64_t lds[];
    const int tl = threadIdx.x & 15, team = threadIdx.x >> 4;
    int64_t qh = (int64_t)blockIdx.x * (blockDim.x >> 4) + team;
    if (head_blocks > 0) {
        const int h = blockIdx.x / head_blocks;
        const int64_t i = (int64_t)(blockIdx.x - h * head_blocks) * (blockDim.x >> 4) + team;
        if (i >= N) return;
        qh = i * H + h;
    }
    if (qh >= (int64_t)N * H) return;  // whole team exits together
    CoefIn<NS> in;
    coef_fetch<D, DV, NS>(Q, dO, idx, lse, N, k, true, qh, tl, in);
    int32_t jj[NS];
    float ca[NS], cp[NS];
    // Key rows in up to 64 registers (32 in the fused pass, whose records take
    // the rest).  With 32 (us): 760k nodes, d = 32, k = 50, normal rows 1769 ->
    // 1215 (a lane per row 1391 in the fused pass); 200k nodes, 2 heads, d = 32, k =
    // 64, city 446 -> 392; 100k nodes, 4 heads, d = 64, k = 32, normal rows 674 -> 481.
    // Not at unequal widths (40 graphs of 100-1000 nodes, 3 heads, d = 32, d_V = 128,
    // k = 64, whole backward 410 -> 443).
    constexpr int kKeepRegs = NS <= 4 && D == DV ? 64 : 32;
    coef_team<D, DV, NS, kKeepRegs>(in, K, V, keep, keep_scale, H, k, scale, tl,
                         reinterpret_cast<char*>(lds) + team * coef_area(NS), dQ, nullptr, 0, jj, ca, cp);
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const int slot = tl + 16 * s;
        if (slot < k) coef[(size_t)qh * k + slot] = make_float2(ca[s], cp[s]);
    }
}

// Launches csr_coef_kernel<D, DV, NS> with NS the smallest power of two >=
// k/16, 16 teams a workgroup (one wave for k > 128, whose LDS areas are large).
template <int D, int DV>
void launch_coef(int64_t nh, hipStream_t stream, const uint16_t* q, const uint16_t* kk, const uint16_t* v,
                 const uint16_t* g, const int32_t* idx, const float* lse, int32_t N, int32_t H, int32_t k,
                 float scale, float* dQ, float2* coef, const uint8_t* keep, float keep_scale) {
    const int ns = (k + 15) / 16;
#define KMIP_COEF(NSV)                                                                                          \
    {                                                                                                           \
        constexpr int teams = NSV > 8 ? 4 : 16;                                                                 \
        const int32_t per_head = (N + teams - 1) / teams, head_blocks = gather_by_head(N, H, D, DV, k, false) ? per_head : 0; \
        const int64_t blocks = head_blocks > 0 ? (int64_t)per_head * H : (nh + teams - 1) / teams;              \
        hipLaunchKernelGGL((csr_coef_kernel<D, DV, NSV>), dim3((unsigned)blocks), dim3(16 * teams),             \
                           teams * coef_area(NSV), stream, q, kk, v, g, idx, lse, N, H, k, scale, dQ, coef,     \
                           keep, keep_scale, head_blocks);                                                      \
        return;                                                                                                 \
    }
    if (ns <= 1) KMIP_COEF(1)
    if (ns <= 2) KMIP_COEF(2)
    if (ns <= 4) KMIP_COEF(4)
    if (ns <= 8) KMIP_COEF(8)
    if constexpr (D <= 64) {
        // k > 128 (d <= 64 only)
        if (ns <= 16) KMIP_COEF(16)
        KMIP_COEF(32)
    }
#undef KMIP_COEF
}

// Key row of slot s of query-head qh, or -1 (padding).
__device__ __forceinline__ int32_t pair_row(const int32_t* __restrict__ idx, int64_t qh, int s,
                                            int32_t k, int32_t N, int32_t H) {
    const int32_t j = idx[(size_t)qh * k + s];
    return (j >= 0 && j < N) ? j * H + (int32_t)(qh % H) : -1;
}

// 2 and 4.  A workgroup takes 256 query-heads (a thread each, walking its
// k slots) and first counts its pairs per key row in an LDS table, so that
// a key row most queries select costs one global atomic per workgroup.
// Rows that find no table slot count with their own global atomic.  The
// count pass adds the table's counts to cnt.  The place pass reserves a range
// of positions per table row with one atomic on the cursors (the scanned
// counts), then gives each pair the next position of its row's range and
// writes the pair's record there.
constexpr int kTab = 2048;      // table rows per workgroup
constexpr int kTabProbes = 8;

struct PairRecord {
    int32_t row;    // key row j*H + h
    int32_t qh;     // query-head i*H + h (full sort), or its head-major row h*N + i (buckets)
    float a;        // scale * g_ij
    float p;        // p_ij
};

struct CountTable {
    int32_t key[kTab];
    int32_t n[kTab];
    int32_t base[kTab];
};

// Slot of key row r in the table (claimed if absent), or -1 if every probe
// is taken by other rows.  With `claim` false, only looks up.
__device__ __forceinline__ int tab_slot(CountTable* t, int32_t r, bool claim) {
    const uint32_t hsh = ((uint32_t)r * 0x9E3779B1u) >> (32 - 11);
    for (int p = 0; p < kTabProbes; ++p) {
        const int ts = (int)((hsh + p) & (kTab - 1));
        const int32_t cur = __hip_atomic_load(&t->key[ts], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (cur == r) return ts;
        if (cur == -1) {
            if (!claim) return -1;
            const int32_t old = atomicCAS(&t->key[ts], -1, r);
            if (old == -1 || old == r) return ts;
        }
    }
    return -1;
}

template <bool kPlace>
__global__ __launch_bounds__(256) void csr_count_kernel(const int32_t* __restrict__ idx,
                                                        const float2* __restrict__ coef, int32_t N,
                                                        int32_t H, int32_t k,
                                                        int32_t* __restrict__ cnt,
                                                        PairRecord* __restrict__ rec) {
    static_assert(kTab == 1 << 11, "hash width");
    __shared__ CountTable tab;
    for (int e = threadIdx.x; e < kTab; e += 256) {
        tab.key[e] = -1;
        tab.n[e] = 0;
    }
    __syncthreads();
    const int64_t qh = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const bool live = qh < (int64_t)N * H;
    for (int s = 0; live && s < k; ++s) {
        const int32_t r = pair_row(idx, qh, s, k, N, H);
        if (r < 0) continue;
        const int ts = tab_slot(&tab, r, true);
        if (ts >= 0) {
            atomicAdd(&tab.n[ts], 1);
        } else if (kPlace) {
            const float2 c = coef[(size_t)qh * k + s];
            rec[atomicAdd(&cnt[r], 1)] = PairRecord{r, (int32_t)qh, c.x, c.y};
        } else {
            atomicAdd(&cnt[r], 1);
        }
    }
    __syncthreads();
    for (int e = threadIdx.x; e < kTab; e += 256) {
        const int32_t r = tab.key[e];
        if (r < 0 || tab.n[e] == 0) continue;
        const int32_t b = atomicAdd(&cnt[r], tab.n[e]);
        if (kPlace) tab.base[e] = b;
    }
    if constexpr (kPlace) {
        __syncthreads();
        for (int e = threadIdx.x; e < kTab; e += 256) tab.n[e] = 0;
        __syncthreads();
        for (int s = 0; live && s < k; ++s) {
            const int32_t r = pair_row(idx, qh, s, k, N, H);
            if (r < 0) continue;
            const int ts = tab_slot(&tab, r, false);
            if (ts < 0) continue;  // placed above
            const float2 c = coef[(size_t)qh * k + s];
            rec[tab.base[ts] + atomicAdd(&tab.n[ts], 1)] = PairRecord{r, (int32_t)qh, c.x, c.y};
        }
    }
}

// 3.  Exclusive scan of n counts in place: block sums, a scan of the block
// sums (one block), then each block's own scan plus its offset.
__device__ __forceinline__ int32_t block_exclusive_scan(int32_t v, int32_t* sh, int32_t* total) {
    const int t = threadIdx.x;
    sh[t] = v;
    __syncthreads();
    for (int off = 1; off < kScanBlock; off <<= 1) {
        const int32_t add = t >= off ? sh[t - off] : 0;
        __syncthreads();
        sh[t] += add;
        __syncthreads();
    }
    const int32_t incl = sh[t];
    if (total != nullptr && t == kScanBlock - 1) *total = incl;
    __syncthreads();
    return incl - v;
}

__global__ __launch_bounds__(kScanBlock) void scan_blocks_kernel(const int32_t* __restrict__ cnt,
                                                                 int64_t n, int32_t* __restrict__ sums) {
    __shared__ int32_t sh[kScanBlock];
    const int64_t i = (int64_t)blockIdx.x * kScanBlock + threadIdx.x;
    block_exclusive_scan(i < n ? cnt[i] : 0, sh, &sums[blockIdx.x]);
}

// Scans the nb block sums in place, kScanBlock at a time with a running
// carry; sums[nb] receives the grand total.
__global__ __launch_bounds__(kScanBlock) void scan_sums_kernel(int32_t* __restrict__ sums, int32_t nb) {
    __shared__ int32_t sh[kScanBlock];
    __shared__ int32_t total;
    const int t = threadIdx.x;
    int32_t carry = 0;
    for (int32_t base = 0; base < nb; base += kScanBlock) {
        const int32_t v = base + t < nb ? sums[base + t] : 0;
        const int32_t ex = block_exclusive_scan(v, sh, &total);
        if (base + t < nb) sums[base + t] = ex + carry;
        carry += total;
        __syncthreads();  // every thread has read total before it is rewritten
    }
    if (t == 0) sums[nb] = carry;
}

__global__ __launch_bounds__(kScanBlock) void scan_apply_kernel(int32_t* __restrict__ cnt, int64_t n,
                                                                const int32_t* __restrict__ sums) {
    __shared__ int32_t sh[kScanBlock];
    const int64_t i = (int64_t)blockIdx.x * kScanBlock + threadIdx.x;
    const int32_t ex = block_exclusive_scan(i < n ? cnt[i] : 0, sh, nullptr);
    if (i < n) cnt[i] = ex + sums[blockIdx.x];
}

// 5.  A wave per chunk of kChunk sorted pairs, four teams per wave, each team
// a contiguous quarter of the chunk.  `total` = number of sorted pairs.
template <int D, int DV>
__global__ __launch_bounds__(256) void csr_reduce_kernel(
    const uint16_t* __restrict__ Q, const uint16_t* __restrict__ dO,
    const PairRecord* __restrict__ rec, const int32_t* __restrict__ total,
    float* __restrict__ dK, float* __restrict__ dV) {
    constexpr int U = D / 16;
    constexpr int UV = DV / 16;
    constexpr int kTeamSpan = kChunk / 4;
    const int tl = threadIdx.x & 15;
    const int team = (int)(blockIdx.x * 16 + (threadIdx.x >> 4));
    const int64_t e0 = (int64_t)team * kTeamSpan;
    const int64_t e1 = min((int64_t)*total, e0 + kTeamSpan);
    int32_t cur = -1;
    float ak[U], av[UV];
#pragma unroll
    for (int u = 0; u < U; ++u) ak[u] = 0.0f;
#pragma unroll
    for (int u = 0; u < UV; ++u) av[u] = 0.0f;
    auto flush = [&]() {
        if (cur >= 0) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                atomicAdd(dK + (size_t)cur * D + 16 * u + tl, ak[u]);
                ak[u] = 0.0f;
            }
#pragma unroll
            for (int u = 0; u < UV; ++u) {
                atomicAdd(dV + (size_t)cur * DV + 16 * u + tl, av[u]);
                av[u] = 0.0f;
            }
        }
    };
    for (int64_t b = e0; b < e1; b += 16) {
        // Sixteen records at a time: lane t fetches record b + t, then the
        // team walks them in order with each record broadcast.
        const int64_t e = b + tl;
        PairRecord r{-1, 0, 0.0f, 0.0f};
        if (e < e1) r = rec[e];
        const int n = (int)min((int64_t)16, e1 - b);
        for (int t = 0; t < n; ++t) {
            const int32_t rt = __shfl(r.row, t, 16);
            const int32_t qt = __shfl(r.qh, t, 16);
            const float at = __shfl(r.a, t, 16);
            const float pt = __shfl(r.p, t, 16);
            if (rt != cur) {
                flush();
                cur = rt;
            }
            const size_t qrow = (size_t)qt * D + tl;
            const size_t grow = (size_t)qt * DV + tl;
#pragma unroll
            for (int u = 0; u < U; ++u) ak[u] = fmaf(at, bf16_bits_to_f32(Q[qrow + 16 * u]), ak[u]);
#pragma unroll
            for (int u = 0; u < UV; ++u) av[u] = fmaf(pt, bf16_bits_to_f32(dO[grow + 16 * u]), av[u]);
        }
    }
    flush();
}

// ---- Variant 4: pairs bucketed by blocks of key rows, sorted in LDS ----
//
// The key rows are cut into buckets of RB consecutive rows, at most
// kMaxBuckets of them: RB = 256 at d = 16, 128 at d = 32 and 64 above, doubled
// (up to kMaxBucketRows) while N*H would need more buckets.  The pairs are counting-sorted by bucket only: a
// counting pass takes ranges of consecutive pairs and counts them with an
// LDS histogram over the buckets, one global atomic per bucket it touches
// (against one per key row and workgroup for the full sort, whose per-row
// tables overflow when pairs spread over many keys); two placement passes
// (below) then write the records in bucket order.  Each bucket's records are
// cut into pieces that one workgroup sorts by key row in LDS and reduces
// like the full sort's reduction.
constexpr int kMaxBuckets = 8192;
constexpr int kMaxBucketRows = 512;

// log2 of the bucket rows for N*H key rows at width d (the bucketed variant
// takes N*H <= kMaxBuckets * kMaxBucketRows).
inline int bucket_shift(int64_t nh, int d) {
    int sh = d == 16 ? 8 : (d == 32 ? 7 : 6);
    while ((nh + (1 << sh) - 1) >> sh > kMaxBuckets && (1 << sh) < kMaxBucketRows) ++sh;
    return sh;
}

// Division of a dividend below 2^31 by a fixed divisor d >= 1 as a multiply
// and shift: with l = ceil(log2 d) and m = ceil(2^(32+l) / d) (at most 2^33),
// floor(n m / 2^(32+l)) = floor(n / d) for every n < 2^32 (the round-up
// method of Granlund and Montgomery); n < 2^31 keeps n m below 2^64.
struct FastDiv {
    uint64_t m;
    uint32_t s;
    uint32_t d;
};

inline FastDiv make_fastdiv(uint32_t d) {
    uint32_t l = 0;
    while ((1ull << l) < d) ++l;
    const unsigned __int128 num = (unsigned __int128)1 << (32 + l);
    return FastDiv{(uint64_t)((num + d - 1) / d), 32 + l, d};
}

__device__ __forceinline__ uint32_t fdiv(uint32_t n, const FastDiv& f) {
    return (uint32_t)(((uint64_t)n * f.m) >> f.s);
}

// A pair record of the bucketed sort, 12 bytes: the key row's offset in its
// bucket (below kMaxBucketRows = 2^9) in bits 22..30 and the head-major query
// row h*N + i in bits 0..21 (the bucketed variant takes N*H <= kMaxBuckets *
// kMaxBucketRows = 2^22), then the coefficients.
struct BucketRecord {
    uint32_t packed;
    float a;
    float p;
};
constexpr int kQRowBits = 22;
static_assert(sizeof(BucketRecord) == 12, "packed record");
static_assert((int64_t)kMaxBuckets * kMaxBucketRows <= (int64_t)1 << kQRowBits, "query rows fit 22 bits");
static_assert(kMaxBucketRows <= 1 << (32 - kQRowBits), "bucket offsets fit the other 10 bits");

// Takes one slot of LDS counter ctr[bk] for each lane with bk >= 0 and
// returns its number (kReturn) or nothing.  Lanes of a wave that share a bucket are served
// by one atomic while the group the wave's first pending lane belongs to
// holds at least 8 lanes (a bucket most pairs fall in: one atomic per wave
// instead of one per lane); the rest take one atomic each.
template <bool kReturn>
__device__ __forceinline__ int32_t claim_slot(int32_t* ctr, int32_t bk) {
    const int lane = threadIdx.x & 63;
    bool pending = bk >= 0;
    int32_t slot = 0;
    for (int it = 0; it < 4; ++it) {
        const uint64_t act = __ballot(pending);
        if (act == 0) break;
        int32_t grp = 0;
        if (pending) {
            const int32_t b0 = __builtin_amdgcn_readfirstlane(bk);
            const uint64_t eq = __ballot(bk == b0);
            grp = __popcll(eq);
            if (grp >= 8) {
                const int leader = __ffsll((unsigned long long)eq) - 1;
                int32_t base0 = 0;
                if (lane == leader) base0 = atomicAdd(&ctr[b0], grp);
                if (kReturn) base0 = __shfl(base0, leader, 64);
                if (bk == b0) {
                    slot = base0 + (int32_t)__popcll(eq & ((1ull << lane) - 1ull));
                    pending = false;
                }
            }
        }
        // this round's group size, as seen by its first lane
        if (__builtin_amdgcn_readlane(grp, __ffsll((unsigned long long)act) - 1) < 8) break;
    }
    if (pending) slot = atomicAdd(&ctr[bk], 1);
    return slot;
}

// Counting pass over a range of `per` consecutive pairs (pair e =
// query-head e / k, slot e % k, so that lanes read idx contiguously): the
// workgroup counts its pairs per bucket in LDS and adds the counts to the
// global ones, one atomic per bucket it touches.
__global__ __launch_bounds__(256) void bkt_count_kernel(const int32_t* __restrict__ idx, int32_t N, int32_t H,
                                                        int32_t k, FastDiv divk, FastDiv divh, int32_t shift,
                                                        int32_t nbk, uint32_t per, int32_t* __restrict__ gcnt) {
    __shared__ int32_t hist[kMaxBuckets];
    const int t = threadIdx.x;
    const uint32_t P = (uint32_t)N * (uint32_t)H * (uint32_t)k;
    const uint32_t p0 = blockIdx.x * per;
    const uint32_t p1 = min(P, p0 + per);
    auto row_of = [&](uint32_t e) -> int32_t {
        if (e >= p1) return -1;
        const int32_t j = idx[e];
        const uint32_t qh = fdiv(e, divk);
        return (j >= 0 && j < N) ? j * H + (int32_t)(qh - fdiv(qh, divh) * (uint32_t)H) : -1;
    };
    for (int e = t; e < nbk; e += 256) hist[e] = 0;
    __syncthreads();
    // every lane runs the same number of rounds (wave-wide claims); four
    // pairs' loads are issued before their claims
    for (uint32_t pb = p0; pb < p1; pb += 1024) {
        int32_t r[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) r[u] = row_of(pb + 256 * u + t);
#pragma unroll
        for (int u = 0; u < 4; ++u) claim_slot<false>(hist, r[u] >= 0 ? r[u] >> shift : -1);
    }
    __syncthreads();
    for (int e = t; e < nbk; e += 256) {
        const int32_t c = hist[e];
        if (c != 0) atomicAdd(&gcnt[e], c);
    }
}


// Placing the records in bucket order takes two passes with coalesced
// stores (a single pass that sends each pair to its bucket directly makes
// one scattered store per pair).  Pass 1, fused with the coefficient pass
// (coef_split_kernel), sorts each chunk of kSplitChunk pairs by super-bucket
// (kSupBuckets consecutive buckets, at most kMaxBuckets / kSupBuckets of
// them) in LDS, reserves each super-bucket's range with one atomic and
// writes the chunk out as runs; pass 2 does the same for each piece of
// kSplitChunk records of one super-bucket, by bucket, and writes the final
// records.
constexpr int kSplitChunk = 2048;
constexpr int kSupBuckets = 128;
constexpr int kMaxSup = kMaxBuckets / kSupBuckets;
static_assert(kMaxSup == 64 && kSupBuckets == 128, "6-bit super-bucket and 7-bit bucket digits; one-wave scans");

// Exclusive prefix sum over the 64 lanes of a wave; *total (lane 63's
// inclusive sum) for every lane.
__device__ __forceinline__ int32_t wave_exclusive_sum(int32_t v, int32_t* total) {
    const int lane = threadIdx.x & 63;
    int32_t x = v;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int32_t y = __shfl_up(x, off, 64);
        if (lane >= off) x += y;
    }
    *total = __shfl(x, 63, 64);
    return x - v;
}

// Slot of each lane with digit >= 0 (a value below 2^NB) in LDS counter
// ctr[digit]: the lanes of the wave with equal digits are found with NB
// ballots, and one leader per digit takes the group's slots with a single
// atomic (lanes with equal digits never meet at one counter in an atomic).
template <int NB>
__device__ __forceinline__ int32_t wave_rank(int32_t* ctr, int32_t digit) {
    const int lane = threadIdx.x & 63;
    uint64_t same = __ballot(digit >= 0);
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const bool bit = ((digit >> b) & 1) != 0;
        const uint64_t bb = __ballot(bit);
        same &= bit ? bb : ~bb;
    }
    const int leader = same != 0ull ? __ffsll((unsigned long long)same) - 1 : lane;
    int32_t base = 0;
    if (digit >= 0 && lane == leader) base = atomicAdd(&ctr[digit], (int32_t)__popcll(same));
    base = __shfl(base, leader, 64);
    return base + (int32_t)__popcll(same & ((1ull << lane) - 1ull));
}

// The coefficient pass fused with placement pass 1: a
// workgroup takes 128 / NS query-heads (8 / NS per team, at most 2048
// pairs), computes their coefficients, dQ and the interleaved copy, and
// writes their records in super-bucket order: one record per lane and
// round for 8 rounds, ranked by ballots, staged in LDS and written as runs
// into ranges the workgroup reserves with one atomic per super-bucket.  The
// coefficients never go to memory.  (k > 128: a team's LDS area is large, so
// the workgroup has 8 or 4 teams of one query-head each, and the records go
// out in NS / 8 chunks.)
// The query-heads are taken in the order u = h N + p, query perm[h][p] (p
// without perm) at position p of head h: with perm the grouping of the queries by direction,
// queries that share most of their keys are processed together (their key
// and value rows are gathered while in cache) and their rows of the
// interleaved copy, row u, lie side by side, so the reduction's gathers for
// one key row mostly read neighbouring rows and share cache lines.  The
// records carry u as their query row.
// (Four waves per SIMD where that costs few spills: k <= 16 at d = 32, d_V <=
// 32 62 -> 58 us in a batch of 128 graphs, k = 128 at d = 64 737 -> 655 at 262k
// nodes.  At d = 32, k = 32 it would cost 57 spilled registers, 285 -> 485 us; at
// d = 32, k = 16 and d_V = 64 or 128 45, the whole backward of 100k nodes, 4
// heads 578 against 500 and 770 against 689, of 64 graphs of about 270 nodes,
// 3 heads, d_V = 64 111 against 97.)
constexpr int split_threads(int ns) { return ns <= 8 ? 256 : 2048 / ns; }

template <int D, int DV, int NS>
__global__ __launch_bounds__(split_threads(NS), D <= 64 && (NS == 8 || (NS == 1 && D == 32 && DV <= 32)) ? 4 : 1) void coef_split_kernel(
    const uint16_t* __restrict__ Q, const uint16_t* __restrict__ K, const uint16_t* __restrict__ V,
    const uint16_t* __restrict__ dO, const int32_t* __restrict__ idx, const float* __restrict__ lse,
    const int32_t* __restrict__ perm, int32_t N, int32_t H, int32_t k, float scale, float* __restrict__ dQ,
    uint16_t* __restrict__ QGt, int32_t shift, int32_t* __restrict__ supcur, PairRecord* __restrict__ mid,
    const uint8_t* __restrict__ keep, float keep_scale) {
    constexpr int THREADS = split_threads(NS), TEAMS = THREADS / 16;
    constexpr int TQ = NS <= 8 ? 8 / NS : 1;   // query-heads per team
    constexpr int R = 8;                       // records per lane and chunk
    constexpr int CHUNKS = TQ * NS / R;
    constexpr size_t kStage = THREADS * R * sizeof(PairRecord), kAreas = TEAMS * coef_area(NS);
    __shared__ int32_t cnt[kMaxSup], lstart[kMaxSup], gbase[kMaxSup];
    __shared__ uint4 lds[(kStage > kAreas ? kStage : kAreas) / 16];   // the teams' areas, then the staged chunk
    PairRecord* const stage = reinterpret_cast<PairRecord*>(lds);
    __shared__ int32_t total;
    const int t = threadIdx.x;
    const int tl = t & 15, team = t >> 4;
    const int64_t nh = (int64_t)N * H;
    for (int i = t; i < kMaxSup; i += THREADS) cnt[i] = 0;
    char* const area = reinterpret_cast<char*>(lds) + team * coef_area(NS);
    PairRecord rr[CHUNKS * R];
    int32_t sup[CHUNKS * R];
    // the query rows of a team first, then each query-head's inputs while the
    // one before computes
    const int64_t u0 = (int64_t)blockIdx.x * (TEAMS * TQ) + team;
    int32_t qrow[TQ];
#pragma unroll
    for (int it = 0; it < TQ; ++it) {
        const int64_t u = u0 + it * TEAMS;
        qrow[it] = u >= nh ? 0 : perm != nullptr ? perm[u] : (int32_t)(u % N);
    }
    CoefIn<NS> nxt;
    coef_fetch<D, DV, NS>(Q, dO, idx, lse, N, k, u0 < nh, (int64_t)qrow[0] * H + (u0 < nh ? u0 / N : 0), tl, nxt);
#pragma unroll
    for (int it = 0; it < TQ; ++it) {
        const int64_t u = u0 + it * TEAMS;
        const int32_t h = u < nh ? (int32_t)(u / N) : 0;
        int32_t jj[NS];
        float ca[NS], cp[NS];
        const CoefIn<NS> cur = nxt;
        if (it + 1 < TQ) {
            const int64_t v = u + TEAMS;
            coef_fetch<D, DV, NS>(Q, dO, idx, lse, N, k, v < nh, (int64_t)qrow[it + 1] * H + (v < nh ? v / N : 0), tl, nxt);
        }
        coef_team<D, DV, NS, 32>(cur, K, V, keep, keep_scale, H, k, scale, tl, area, dQ, QGt, (size_t)u, jj, ca, cp);
#pragma unroll
        for (int s2 = 0; s2 < NS; ++s2) {
            const int r = it * NS + s2;
            sup[r] = -1;
            rr[r] = PairRecord{-1, 0, 0.0f, 0.0f};
            if (u < nh && jj[s2] >= 0) {
                const int32_t row = jj[s2] * H + h;
                rr[r] = PairRecord{row, (int32_t)u, ca[s2], cp[s2]};
                sup[r] = (row >> shift) / kSupBuckets;
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int ch = 0; ch < CHUNKS; ++ch) {
        int32_t slot[R];
#pragma unroll
        for (int r = 0; r < R; ++r) slot[r] = wave_rank<6>(cnt, sup[ch * R + r]);
        __syncthreads();
        if (t < 64) {
            const int32_t c = cnt[t];
            int32_t tot;
            const int32_t ex = wave_exclusive_sum(c, &tot);
            lstart[t] = ex;
            gbase[t] = c != 0 ? atomicAdd(&supcur[t], c) : 0;
            if (t == 0) total = tot;
            if (ch + 1 < CHUNKS) cnt[t] = 0;
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < R; ++r)
            if (sup[ch * R + r] >= 0) stage[lstart[sup[ch * R + r]] + slot[r]] = rr[ch * R + r];
        __syncthreads();
        const int n = total;
        for (int j = t; j < n; j += THREADS) {
            const PairRecord rec = stage[j];
            const int sp = (rec.row >> shift) / kSupBuckets;
            mid[gbase[sp] + (j - lstart[sp])] = rec;
        }
        if (ch + 1 < CHUNKS) __syncthreads();
    }
}

template <int D, int DV>
hipError_t launch_coef_split(int64_t nh, hipStream_t stream, const uint16_t* q, const uint16_t* kk,
                             const uint16_t* v, const uint16_t* g, const int32_t* idx, const float* lse,
                             const int32_t* perm, int32_t N, int32_t H, int32_t k, float scale, float* dQ,
                             uint16_t* qg, int32_t shift, int32_t* supcur, PairRecord* mid, const uint8_t* keep,
                             float keep_scale) {
    const int ns = (k + 15) / 16;
#define KMIP_COEF_SPLIT(NSV)                                                                                    \
    {                                                                                                           \
        constexpr int per = split_threads(NSV) / 16 * (NSV <= 8 ? 8 / NSV : 1);                                 \
        hipLaunchKernelGGL((coef_split_kernel<D, DV, NSV>), dim3((unsigned)((nh + per - 1) / per)),              \
                           dim3(split_threads(NSV)), 0, stream, q, kk, v, g, idx, lse, perm, N, H, k, scale, dQ, \
                           qg, shift, supcur, mid, keep, keep_scale);                                            \
        return hipGetLastError();                                                                               \
    }
    if (ns <= 1) KMIP_COEF_SPLIT(1)
    if (ns <= 2) KMIP_COEF_SPLIT(2)
    if (ns <= 4) KMIP_COEF_SPLIT(4)
    if (ns <= 8) KMIP_COEF_SPLIT(8)
    if constexpr (D <= 64) {
        if (ns <= 16) KMIP_COEF_SPLIT(16)
        KMIP_COEF_SPLIT(32)
    }
#undef KMIP_COEF_SPLIT
    return hipErrorInvalidValue;
}

constexpr int kPiece = 4096;   // records per reduction workgroup (sorted in 48 KB of LDS)

// Everything that follows from the bucket counts, in one workgroup (nbk <=
// kMaxBuckets; six scan launches and two small ones before, about 4 us each):
//   gcnt    the counts become the buckets' first records (the cursors pass 2
//           advances; entry nbk the total), sstart keeps a copy;
//   pstart  scanned number of reduction pieces of at most kPiece records;
//   supst   first record of each super-bucket (nsup + 1 entries), supcur the
//           cursors pass 1 reserves from, pstart2 the scanned number of
//           pass-2 pieces (nsup + 1).
__global__ __launch_bounds__(kScanBlock) void bkt_scan_kernel(int32_t* __restrict__ gcnt, int32_t nbk, int32_t nsup,
                                                              int32_t* __restrict__ sstart,
                                                              int32_t* __restrict__ pstart,
                                                              int32_t* __restrict__ supst,
                                                              int32_t* __restrict__ supcur,
                                                              int32_t* __restrict__ pstart2) {
    constexpr int PER = (kMaxBuckets + kScanBlock) / kScanBlock;   // counts per thread, consecutive
    __shared__ int32_t first[kMaxBuckets + kScanBlock];
    __shared__ int2 wsum[kScanBlock / 64];
    const int t = threadIdx.x, wave = t >> 6, lane = t & 63;
    int32_t c[PER], cs = 0, ps = 0;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int b = PER * t + i;
        c[i] = b < nbk ? gcnt[b] : 0;
        cs += c[i];
        ps += (c[i] + kPiece - 1) / kPiece;
    }
    int32_t ctot, ptot;
    int32_t cx = wave_exclusive_sum(cs, &ctot), px = wave_exclusive_sum(ps, &ptot);
    if (lane == 0) wsum[wave] = make_int2(ctot, ptot);
    __syncthreads();
    for (int w = 0; w < wave; ++w) {
        cx += wsum[w].x;
        px += wsum[w].y;
    }
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int b = PER * t + i;
        if (b <= nbk) {
            first[b] = cx;
            gcnt[b] = cx;
            sstart[b] = cx;
            pstart[b] = px;
        }
        cx += c[i];
        px += (c[i] + kPiece - 1) / kPiece;
    }
    __syncthreads();
    if (t < 64) {
        const int32_t a = first[min(t * kSupBuckets, nbk)], e = first[min((t + 1) * kSupBuckets, nbk)];
        const int32_t np = t < nsup ? (e - a + kSplitChunk - 1) / kSplitChunk : 0;
        int32_t tot;
        const int32_t ex = wave_exclusive_sum(np, &tot);
        if (t < nsup) {
            supst[t] = a;
            supcur[t] = a;
            pstart2[t] = ex;
        }
        if (t == 0) {
            supst[nsup] = first[nbk];
            pstart2[nsup] = tot;
        }
    }
}

// Zeroes the bucket counts and both gradients (n4, m4: float4 counts; g4: int4s).
__global__ __launch_bounds__(256) void bkt_clear_kernel(int4* __restrict__ gcnt, int64_t g4, float4* __restrict__ dK,
                                                        int64_t n4, float4* __restrict__ dV, int64_t m4) {
    const int64_t stride = (int64_t)gridDim.x * 256;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < g4 + n4 + m4; i += stride) {
        if (i < n4)
            dK[i] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        else if (i < n4 + m4)
            dV[i - n4] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        else
            gcnt[i - n4 - m4] = make_int4(0, 0, 0, 0);
    }
}

// Pass 2: one workgroup per piece of at most kSplitChunk records of one
// super-bucket; bcur holds the buckets' cursors (their starts, advanced
// here).
__global__ __launch_bounds__(256) void bkt_split2_kernel(const PairRecord* __restrict__ mid,
                                                         const int32_t* __restrict__ supst,
                                                         const int32_t* __restrict__ pstart2, int32_t nsup,
                                                         int32_t shift, int32_t* __restrict__ bcur,
                                                         BucketRecord* __restrict__ rec) {
    constexpr int R = kSplitChunk / 256;
    __shared__ int32_t cnt[kSupBuckets], lstart[kSupBuckets], gbase[kSupBuckets];
    __shared__ BucketRecord stage[kSplitChunk];
    __shared__ uint8_t sbk[kSplitChunk];
    const int t = threadIdx.x;
    const int w = blockIdx.x;
    if (w >= pstart2[nsup]) return;
    int lo = 0, hi = nsup;
    while (hi - lo > 1) {
        const int m = (lo + hi) >> 1;
        if (pstart2[m] <= w) lo = m; else hi = m;
    }
    const int32_t e0 = supst[lo] + (w - pstart2[lo]) * kSplitChunk;
    const int32_t n = min(supst[lo + 1] - e0, kSplitChunk);
    const int32_t b0 = lo * kSupBuckets;
    if (t < kSupBuckets) cnt[t] = 0;
    __syncthreads();
    BucketRecord fr[R];
    int32_t bk[R], slot[R];
    const uint32_t offmask = (1u << shift) - 1u;
#pragma unroll
    for (int u = 0; u < R; ++u) {
        const int i = u * 256 + t;
        bk[u] = -1;
        fr[u] = BucketRecord{0u, 0.0f, 0.0f};
        if (i < n) {
            const PairRecord r = mid[e0 + i];
            bk[u] = (r.row >> shift) - b0;
            fr[u] = BucketRecord{(((uint32_t)r.row & offmask) << kQRowBits) | (uint32_t)r.qh, r.a, r.p};
        }
    }
#pragma unroll
    for (int u = 0; u < R; ++u) slot[u] = wave_rank<7>(cnt, bk[u]);
    __syncthreads();
    if (t < 64) {
        // two halves of kSupBuckets = 128 counters, one wave
        const int32_t c0 = cnt[t], c1 = cnt[t + 64];
        int32_t tot0, tot1;
        const int32_t ex0 = wave_exclusive_sum(c0, &tot0);
        const int32_t ex1 = wave_exclusive_sum(c1, &tot1);
        lstart[t] = ex0;
        lstart[t + 64] = tot0 + ex1;
        gbase[t] = c0 != 0 ? atomicAdd(&bcur[b0 + t], c0) : 0;
        gbase[t + 64] = c1 != 0 ? atomicAdd(&bcur[b0 + t + 64], c1) : 0;
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < R; ++u) {
        if (bk[u] >= 0) {
            stage[lstart[bk[u]] + slot[u]] = fr[u];
            sbk[lstart[bk[u]] + slot[u]] = (uint8_t)bk[u];
        }
    }
    __syncthreads();
    for (int i = t; i < n; i += 256) {
        const int b = sbk[i];
        rec[gbase[b] + (i - lstart[b])] = stage[i];
    }
}

// The reduction of a piece (a stretch of at most kPiece records of one bucket,
// found by binary search in the scanned piece counts), one workgroup of 512
// threads:
//   1. counting sort of the piece's records by key row into LDS (claim_slot:
//      a key most pairs share costs about one LDS atomic per wave);
//   2. LG lanes take a contiguous span of the sorted records.  A record's
//      query row of the interleaved head-major copy (q then dO) is one 16-byte
//      load per lane; the lanes of q add a*q to dK, those of dO p*dO to dV,
//      four records' rows in flight.  A key row whose
//      records all lie in the span is stored, or, where the bucket has several
//      pieces, added with atomics; the row a span starts in the middle of and
//      the one it ends in go to LDS;
//   3. these partial rows, in row order, are added up sixteen at a time, an
//      atomic per element where the row changes (dK and dV are zero at the
//      start).
// Bound by the fabric on the row gathers of large problems, by the chain of
// phases of a workgroup on small ones.  Against sixteen-lane teams on 8192
// records that added every run with atomics (us): 128 graphs, d = 32, k = 16
// 117 -> 46; 16 clouds, d = 32, k = 32 178 -> 87; 100k nodes, d = 32 480 -> 321;
// 262k nodes, d = 64, k = 128 1577 -> 1124; 500k nodes, d = 16 1029 -> 988.
// The atomics of several pieces go to neighbouring addresses from neighbouring
// lanes (eight addresses 32 bytes apart before; us): 84k nodes, 16 heads, d = 32,
// k = 20, normal rows (two pieces a bucket) 2025 -> 676; 760k nodes, d = 32, k =
// 50 1255 -> 791; 200k nodes, 2 heads, d = 32, k = 64 493 -> 460; 30k nodes, 4
// heads, d = 32, k = 256 606 -> 466.
// (Sums in LDS with float atomics instead of the sort were six times slower:
// an LDS float add took about four clocks a lane.)
constexpr int kSumThreads = 512;

// Exchanges bit M of the register index with bit M of the lane.
template <int M>
__device__ __forceinline__ void exchange_bit(float (&a)[8], int lane) {
    const bool hi = (lane & M) != 0;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        if ((e & M) != 0) continue;
        const float give = hi ? a[e] : a[e | M];
        float got;
        if constexpr (M == 1) got = step_partner<1>(give); else got = xor_lane<M>(give);
        if (hi) a[e] = got; else a[e | M] = got;
    }
}

constexpr int pow2_at_least(int x) { return x <= 1 ? 1 : 2 * pow2_at_least((x + 1) / 2); }

// Waves per SIMD: six, three workgroups a CU, as the LDS allows, at the widths
// where 80 registers hold the exchange (16 clouds of 1k-4k nodes, 4 heads, d = 32,
// k = 32 100 -> 84 us; at other unequal widths that spills ten: d = 64, d_V = 128,
// k = 32, whole backward 571 -> 604).
constexpr int sum_waves(int d, int dv) { return d == dv || d + dv <= 64 ? 6 : 1; }

template <int D, int DV>
__global__ __launch_bounds__(kSumThreads, sum_waves(D, DV)) void bkt_reduce_kernel(const uint16_t* __restrict__ QG,
                                                                 const BucketRecord* __restrict__ rec,
                                                                 const int32_t* __restrict__ sstart,
                                                                 const int32_t* __restrict__ pstart, int32_t nbk,
                                                                 int32_t shift, float* __restrict__ dK,
                                                                 float* __restrict__ dV) {
    constexpr int RW = D + DV;                 // elements of a query row: q, then dO
    constexpr int LG = pow2_at_least(RW / 8);  // lanes per record (those past the row idle)
    constexpr int GR = kSumThreads / LG;       // lane groups
    constexpr int B = 4;                       // records of a group in flight
    constexpr int PER = kPiece / kSumThreads;  // records per thread in the sort
    constexpr int SEG = 16;                    // partial rows summed by one thread
    constexpr int T = LG < 8 ? LG : 8;         // lanes that exchange a row's sums
    static_assert(2 * GR * RW * sizeof(float) <= kPiece * sizeof(BucketRecord), "partial rows fit the records' area");
    static_assert(kSumThreads / (8 * LG) * SEG == 2 * GR, "every partial row has its threads");
    static_assert(kMaxBucketRows <= kSumThreads, "one counter a thread in the scan");
    __shared__ BucketRecord srt[kPiece];
    __shared__ int32_t base[kMaxBucketRows + 1];
    __shared__ int32_t wsum[kSumThreads / 64];
    __shared__ int32_t prow[2 * GR];
    const int t = threadIdx.x;
    const int w = blockIdx.x;
    if (w >= pstart[nbk]) return;
    int lo = 0, hi = nbk;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (pstart[mid] <= w) lo = mid; else hi = mid;
    }
    const int32_t e0 = sstart[lo] + (w - pstart[lo]) * kPiece;
    const int32_t n = min(sstart[lo + 1] - e0, kPiece);
    const bool alone = pstart[lo + 1] - pstart[lo] == 1;
    const int rb = 1 << shift;
    if (t < rb) base[t] = 0;
    for (int i = t; i < 2 * GR; i += kSumThreads) prow[i] = -1;
    __syncthreads();

    // 1. sort by key row
    BucketRecord r[PER];
    int32_t slot[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int i = u * kSumThreads + t;
        r[u] = BucketRecord{0u, 0.0f, 0.0f};
        if (i < n) r[u] = rec[e0 + i];
    }
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        slot[u] = 0;
        if (u * kSumThreads < n)
            slot[u] = claim_slot<true>(base, u * kSumThreads + t < n ? (int32_t)(r[u].packed >> kQRowBits) : -1);
    }
    __syncthreads();
    const int32_t mine = t < rb ? base[t] : 0;
    int32_t tot;
    int32_t ex = wave_exclusive_sum(mine, &tot);
    if ((t & 63) == 0) wsum[t >> 6] = tot;
    __syncthreads();
    for (int v = 0; v < (t >> 6); ++v) ex += wsum[v];
    if (t < rb) base[t] = ex;
    if (t == rb - 1) base[rb] = n;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < PER; ++u)
        if (u * kSumThreads + t < n) srt[base[r[u].packed >> kQRowBits] + slot[u]] = r[u];
    __syncthreads();

    // 2. spans of the sorted records
    const int c = t & (LG - 1), grp = t / LG;
    const bool isq = c < D / 8, used = c < RW / 8;
    const uint16_t* const col = QG + (used ? 8 * c : 0);
    const size_t width = isq ? D : DV;
    float* const dst = isq ? dK + ((size_t)lo << shift) * D + 8 * c : dV + ((size_t)lo << shift) * DV + (8 * c - D);
    const int span = ((n + GR - 1) / GR) | 1;   // odd: the groups' 12-byte records start in different banks
    const int p0 = min(n, grp * span), p1 = min(n, p0 + span);
    int32_t cur = -1, row0 = -1, row1 = -1;   // current row; rows of the span's partial sums
    float acc[8], acc0[8];                    // current sums; those of the row the span starts inside of
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] = acc0[e] = 0.0f;
    auto flush = [&]() {
        if (cur >= 0) {
            const int32_t f0 = base[cur], f1 = base[cur + 1];
            if (f0 < p0) {
                row0 = cur;
#pragma unroll
                for (int e = 0; e < 8; ++e) acc0[e] = acc[e];
            } else if (f1 > p1) {
                row1 = cur;   // the last row: its sums stay in acc
                return;
            } else if (alone) {
                if (used) {
                    float4* d4 = reinterpret_cast<float4*>(dst + cur * width);
                    d4[0] = make_float4(acc[0], acc[1], acc[2], acc[3]);
                    d4[1] = make_float4(acc[4], acc[5], acc[6], acc[7]);
                }
            } else {
                // the elements of T lanes are exchanged so that an atomic's
                // neighbouring lanes add to neighbouring addresses
                if constexpr (T == 8) exchange_bit<4>(acc, c);
                exchange_bit<2>(acc, c);
                exchange_bit<1>(acc, c);
                // (sum e is lane c0 + e's; q's lanes are the first D/8, all of an
                // eight's or, at D < 64, the first D/8 of the first eight)
                const int c0 = c & ~(T - 1), l = c & (T - 1);
                float* const pk = dK + (((size_t)lo << shift) + cur) * D + 8 * c0 + l;
                float* const pv = dV + (((size_t)lo << shift) + cur) * DV + 8 * c0 + l - D;
                float* const first = c0 < D / 8 ? pk : pv;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int off = 8 * (e & (T - 1)) + (e & ~(T - 1));
                    float* const to = (e & (T - 1)) < D / 8 ? first : pv;
                    if (c0 + (e & (T - 1)) < RW / 8) atomicAdd(to + off, acc[e]);
                }
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[e] = 0.0f;
        }
    };
    for (int i0 = p0; i0 < p1; i0 += B) {
        BucketRecord rr[B];
        uint4 x[B];
#pragma unroll
        for (int b = 0; b < B; ++b) {
            rr[b] = srt[min(i0 + b, p1 - 1)];
            x[b] = *reinterpret_cast<const uint4*>(col + (size_t)(rr[b].packed & ((1u << kQRowBits) - 1u)) * RW);
        }
#pragma unroll
        for (int b = 0; b < B; ++b) {
            if (i0 + b < p1) {
                const int32_t row = (int32_t)(rr[b].packed >> kQRowBits);
                if (row != cur) {
                    flush();
                    cur = row;
                }
                const float ca = rr[b].a, cp = rr[b].p;
                axpy8(acc, isq ? ca : cp, x[b]);
            }
        }
    }
    flush();
    __syncthreads();   // every record has been read: partial rows take their place
    float* const part = reinterpret_cast<float*>(srt);   // [2 GR][RW]
#pragma unroll
    for (int side = 0; side < 2; ++side) {
        const int32_t row = side == 0 ? row0 : row1;
        if (row >= 0 && used) {
            float* d8 = part + (size_t)(2 * grp + side) * RW + 8 * c;
#pragma unroll
            for (int e = 0; e < 8; ++e) d8[e] = side == 0 ? acc0[e] : acc[e];
            if (c == 0) prow[2 * grp + side] = row;
        }
    }
    __syncthreads();

    // 3. partial rows, an element a thread
    const int el = t % (8 * LG), sg = t / (8 * LG);
    if (el >= RW) return;
    const size_t ew = el < D ? D : DV;
    float* const out = el < D ? dK + ((size_t)lo << shift) * D + el : dV + ((size_t)lo << shift) * DV + (el - D);
    int32_t at = -1;
    float v = 0.0f;
    for (int i = sg * SEG; i < sg * SEG + SEG; ++i) {
        const int32_t row = prow[i];
        if (row < 0) continue;
        if (row != at) {
            if (at >= 0) atomicAdd(out + at * ew, v);
            at = row;
            v = 0.0f;
        }
        v += part[(size_t)i * RW + el];
    }
    if (at >= 0) atomicAdd(out + at * ew, v);
}

}  // namespace

bool bwd_bucket_rows(int32_t N, int32_t H, int32_t d) {
    const int64_t nh = (int64_t)N * H;
    const int sh = bucket_shift(nh, d);
    return ((nh + (1 << sh) - 1) >> sh) <= kMaxBuckets;
}

bool bwd_bucket_supported(int32_t N, int32_t H, int32_t d, int32_t k) {
    return d <= 64 && k <= 128 && bwd_bucket_rows(N, H, d);
}

size_t bwd_bucket_workspace_bytes(int32_t N, int32_t H, int32_t d, int32_t dv, int32_t k) {
    auto al = [](size_t x) { return (x + 255) / 256 * 256; };
    const size_t nh = (size_t)N * H, pairs = nh * k;
    const size_t nbk = (nh + ((size_t)1 << bucket_shift((int64_t)nh, d)) - 1) >> bucket_shift((int64_t)nh, d);
    return al(pairs * sizeof(BucketRecord)) + 3 * al((nbk + 1) * sizeof(int32_t)) +
           al(nh * (d + dv) * sizeof(uint16_t)) + al(pairs * sizeof(PairRecord)) +
           3 * al((kMaxSup + 1) * sizeof(int32_t)) + al(group_workspace_bytes(N, H, d));
}

hipError_t launch_bwd_bucket(const void* Q, const void* K, const void* V, const void* dO,
                             const int32_t* idx, const float* lse, const uint8_t* keep, float keep_scale,
                             int32_t N, int32_t H, int32_t d, int32_t dv, int32_t k, float scale, float* dQ, float* dK,
                             float* dV, void* ws, hipStream_t stream) {
    auto al = [](size_t x) { return (x + 255) / 256 * 256; };
    const int64_t nh = (int64_t)N * H;
    if (nh == 0) return hipSuccess;
    const size_t pairs = (size_t)nh * k;
    const int32_t shift = bucket_shift(nh, d);
    const int32_t rb = 1 << shift;
    const int32_t nbk = (int32_t)((nh + rb - 1) / rb);
    if (nbk > kMaxBuckets) return hipErrorInvalidValue;
    char* p = reinterpret_cast<char*>(ws);
    BucketRecord* rec = reinterpret_cast<BucketRecord*>(p);
    p += al(pairs * sizeof(BucketRecord));
    int32_t* gcnt = reinterpret_cast<int32_t*>(p);   // counts, then starts (nbk + 1 entries)
    p += al(((size_t)nbk + 1) * sizeof(int32_t));
    int32_t* sstart = reinterpret_cast<int32_t*>(p);   // kept starts
    p += al(((size_t)nbk + 1) * sizeof(int32_t));
    int32_t* pstart = reinterpret_cast<int32_t*>(p);   // pieces per bucket, then their starts
    p += al(((size_t)nbk + 1) * sizeof(int32_t));
    uint16_t* qg = reinterpret_cast<uint16_t*>(p);   // q and dO interleaved, row h N + p for query perm[h][p]
    p += al((size_t)nh * (d + dv) * sizeof(uint16_t));
    PairRecord* mid = reinterpret_cast<PairRecord*>(p);   // records in super-bucket order (pass 1)
    p += al(pairs * sizeof(PairRecord));
    int32_t* supst = reinterpret_cast<int32_t*>(p);
    p += al((kMaxSup + 1) * sizeof(int32_t));
    int32_t* supcur = reinterpret_cast<int32_t*>(p);
    p += al((kMaxSup + 1) * sizeof(int32_t));
    int32_t* pstart2 = reinterpret_cast<int32_t*>(p);
    p += al((kMaxSup + 1) * sizeof(int32_t));
    void* gws = p;   // grouping of the queries by direction (group.hip)

    const uint16_t* q = reinterpret_cast<const uint16_t*>(Q);
    const uint16_t* kk = reinterpret_cast<const uint16_t*>(K);
    const uint16_t* v = reinterpret_cast<const uint16_t*>(V);
    const uint16_t* g = reinterpret_cast<const uint16_t*>(dO);
    hipError_t e;
    // The coefficient pass takes the query-heads grouped by direction once
    // there are enough pairs for the shared rows to pay for the grouping
    // (measured: 2^24 pairs and more; below, the plain order is as fast or
    // faster, 14% at 1.7M pairs in a batch of small graphs).
    QueryGroups groups{};
    if ((int64_t)pairs >= (int64_t(1) << 24) && d <= 64 &&
        (e = launch_group_queries(Q, N, H, d, gws, &groups, stream)) != hipSuccess)
        return e;
    const int64_t g4 = ((int64_t)nbk + 1 + 3) / 4, n4 = nh * d / 4, m4 = nh * dv / 4;
    const unsigned zblocks = (unsigned)std::min<int64_t>((g4 + n4 + m4 + 255) / 256, 256 * 32);
    hipLaunchKernelGGL(bkt_clear_kernel, dim3(zblocks), dim3(256), 0, stream, reinterpret_cast<int4*>(gcnt), g4,
                       reinterpret_cast<float4*>(dK), n4, reinterpret_cast<float4*>(dV), m4);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    // pairs per counting workgroup: about 1024 workgroups, 2048 .. 65536 pairs
    // each (1.7M pairs in 209 workgroups of 8192 took 32 us)
    const uint32_t per = (uint32_t)std::min<size_t>(65536, std::max<size_t>(2048, (pairs / 1024 + 255) / 256 * 256));
    const unsigned cblocks = (unsigned)((pairs + per - 1) / per);
    const FastDiv divk = make_fastdiv((uint32_t)k), divh = make_fastdiv((uint32_t)H);
    hipLaunchKernelGGL(bkt_count_kernel, dim3(cblocks), dim3(256), 0, stream, idx, N, H, k, divk, divh, shift,
                       nbk, per, gcnt);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    const int32_t nsup = (nbk + kSupBuckets - 1) / kSupBuckets;
    hipLaunchKernelGGL(bkt_scan_kernel, dim3(1), dim3(kScanBlock), 0, stream, gcnt, nbk, nsup, sstart, pstart, supst,
                       supcur, pstart2);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    // coefficients, dQ and the interleaved copy, fused with placement pass 1
    e = hipErrorInvalidValue;
#define KMIP_SPLIT(DD, DVV)                                                                                   \
    if (d == DD && dv == DVV)                                                                                  \
        e = launch_coef_split<DD, DVV>(nh, stream, q, kk, v, g, idx, lse, groups.perm, N, H, k, scale, dQ, qg, shift, \
                                       supcur, mid, keep, keep_scale);
#define KMIP_SPLIT_D(DD) KMIP_SPLIT(DD, 16) KMIP_SPLIT(DD, 32) KMIP_SPLIT(DD, 64) KMIP_SPLIT(DD, 128)
    KMIP_SPLIT_D(16)
    KMIP_SPLIT_D(32)
    KMIP_SPLIT_D(64)
    KMIP_SPLIT_D(128)
#undef KMIP_SPLIT_D
#undef KMIP_SPLIT
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(bkt_split2_kernel, dim3((unsigned)(nsup + (pairs + kSplitChunk - 1) / kSplitChunk)), dim3(256),
                       0, stream, mid, supst, pstart2, nsup, shift, gcnt, rec);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    // at most one piece per bucket plus one per kPiece pairs; the rest exit
    const unsigned rblocks = (unsigned)(nbk + (pairs + kPiece - 1) / kPiece);
#define KMIP_BKT_REDUCE(DD, DVV)                                                                               \
    if (d == DD && dv == DVV)                                                                                  \
        hipLaunchKernelGGL((bkt_reduce_kernel<DD, DVV>), dim3(rblocks), dim3(kSumThreads), 0, stream, qg, rec, sstart, \
                           pstart, nbk, shift, dK, dV);
#define KMIP_BKT_REDUCE_D(DD) \
    KMIP_BKT_REDUCE(DD, 16) KMIP_BKT_REDUCE(DD, 32) KMIP_BKT_REDUCE(DD, 64) KMIP_BKT_REDUCE(DD, 128)
    KMIP_BKT_REDUCE_D(16)
    KMIP_BKT_REDUCE_D(32)
    KMIP_BKT_REDUCE_D(64)
    KMIP_BKT_REDUCE_D(128)
#undef KMIP_BKT_REDUCE_D
#undef KMIP_BKT_REDUCE
    return hipGetLastError();
}

size_t bwd_csr_workspace_bytes(int32_t N, int32_t H, int32_t k) {
    auto al = [](size_t x) { return (x + 255) / 256 * 256; };
    const size_t nh = (size_t)N * H, pairs = nh * k;
    const size_t nb = (nh + kScanBlock - 1) / kScanBlock;
    return al(pairs * sizeof(float2)) + al(pairs * sizeof(PairRecord)) + al(nh * sizeof(int32_t)) +
           al((nb + 1) * sizeof(int32_t));
}

hipError_t launch_bwd_csr(const void* Q, const void* K, const void* V, const void* dO,
                          const int32_t* idx, const float* lse, const uint8_t* keep, float keep_scale,
                          int32_t N, int32_t H, int32_t d, int32_t dv, int32_t k, float scale, float* dQ,
                          float* dK, float* dV, void* ws, hipStream_t stream) {
    auto al = [](size_t x) { return (x + 255) / 256 * 256; };
    const int64_t nh = (int64_t)N * H;
    if (nh == 0) return hipSuccess;
    const size_t pairs = (size_t)nh * k;
    const int32_t nb = (int32_t)((nh + kScanBlock - 1) / kScanBlock);
    char* p = reinterpret_cast<char*>(ws);
    float2* coef = reinterpret_cast<float2*>(p);
    p += al(pairs * sizeof(float2));
    PairRecord* rec = reinterpret_cast<PairRecord*>(p);
    p += al(pairs * sizeof(PairRecord));
    int32_t* cnt = reinterpret_cast<int32_t*>(p);
    p += al((size_t)nh * sizeof(int32_t));
    int32_t* sums = reinterpret_cast<int32_t*>(p);

    const uint16_t* q = reinterpret_cast<const uint16_t*>(Q);
    const uint16_t* kk = reinterpret_cast<const uint16_t*>(K);
    const uint16_t* v = reinterpret_cast<const uint16_t*>(V);
    const uint16_t* g = reinterpret_cast<const uint16_t*>(dO);
    hipError_t e;
    // counts are zeroed with the float fill (same bits); n padded to 4
    if ((e = launch_fill_zero(reinterpret_cast<float*>(cnt), ((size_t)nh + 3) / 4 * 4, stream)) != hipSuccess) return e;
    if ((e = launch_fill_zero(dK, (size_t)nh * d, stream)) != hipSuccess) return e;
    if ((e = launch_fill_zero(dV, (size_t)nh * dv, stream)) != hipSuccess) return e;
    bool launched = false;
#define KMIP_CSR_COEF(DD, DVV)                                                                          \
    if (d == DD && dv == DVV) {                                                                         \
        launch_coef<DD, DVV>(nh, stream, q, kk, v, g, idx, lse, N, H, k, scale, dQ, coef, keep, keep_scale); \
        launched = true;                                                                                \
    }
#define KMIP_CSR_COEF_D(DD) KMIP_CSR_COEF(DD, 16) KMIP_CSR_COEF(DD, 32) KMIP_CSR_COEF(DD, 64) KMIP_CSR_COEF(DD, 128)
    KMIP_CSR_COEF_D(16)
    KMIP_CSR_COEF_D(32)
    KMIP_CSR_COEF_D(64)
    KMIP_CSR_COEF_D(128)
#undef KMIP_CSR_COEF_D
#undef KMIP_CSR_COEF
    if (!launched) return hipErrorInvalidValue;
    if ((e = hipGetLastError()) != hipSuccess) return e;
    const unsigned qh_blocks = (unsigned)((nh + 255) / 256);
    hipLaunchKernelGGL(csr_count_kernel<false>, dim3(qh_blocks), dim3(256), 0, stream, idx, coef, N, H,
                       k, cnt, rec);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(scan_blocks_kernel, dim3((unsigned)nb), dim3(kScanBlock), 0, stream, cnt,
                       (int64_t)nh, sums);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(scan_sums_kernel, dim3(1), dim3(kScanBlock), 0, stream, sums, nb);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(scan_apply_kernel, dim3((unsigned)nb), dim3(kScanBlock), 0, stream, cnt,
                       (int64_t)nh, sums);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(csr_count_kernel<true>, dim3(qh_blocks), dim3(256), 0, stream, idx, coef, N, H,
                       k, cnt, rec);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    // one team per kChunk/4 sorted pairs, 16 teams per block; the grid covers
    // every pair slot, teams past the total exit at once
    const unsigned red_blocks = (unsigned)((pairs + kChunk * 4 - 1) / (kChunk * 4));
    const int32_t* total = sums + nb;
#define KMIP_CSR_REDUCE(DD, DVV)                                                                        \
    if (d == DD && dv == DVV)                                                                           \
        hipLaunchKernelGGL((csr_reduce_kernel<DD, DVV>), dim3(red_blocks), dim3(256), 0, stream, q, g, rec, \
                           total, dK, dV);
#define KMIP_CSR_REDUCE_D(DD) \
    KMIP_CSR_REDUCE(DD, 16) KMIP_CSR_REDUCE(DD, 32) KMIP_CSR_REDUCE(DD, 64) KMIP_CSR_REDUCE(DD, 128)
    KMIP_CSR_REDUCE_D(16)
    KMIP_CSR_REDUCE_D(32)
    KMIP_CSR_REDUCE_D(64)
    KMIP_CSR_REDUCE_D(128)
#undef KMIP_CSR_REDUCE_D
#undef KMIP_CSR_REDUCE
    return hipGetLastError();
}

}  // namespace kmip

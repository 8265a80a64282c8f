// Score + select without pruning for small and medium graphs, wide heads and
// large k on gfx950.
//
// RowwiseTopK of Algorithm 1 (Appendix E) of arXiv 2604.03815.  A workgroup of
// W waves takes QN queries (32 or 64, or 16 for k > 256) of one graph and head,
// and its waves share the graph's key tiles between them (wave w takes tiles w,
// w + W, ...).  Scores come from the streaming kernel's MFMA (A = 32 keys,
// B = 32 queries, fp32 accumulation over chunks of 16 dims), so they are the
// same values.  Two passes over the keys, neither of which keeps a running
// selection:
//   1. every lane keeps the maxima of GT T groups of the keys it scores (16 /
//      GT neighbouring rows of its 16 in every T-th of its tiles).
//      The k'-th largest of a query's 2 GT T W group maxima (k' = min(k, n)) is
//      a lower bound of its k'-th best score, since k' distinct keys reach
//      it; its 20-bit code prefix, found bit by bit, is the threshold theta;
//   2. the scores are formed again and the keys with s >= theta are listed in
//      LDS (score code, ~index).  Where a key's place says nothing about its
//      score, about 1.15 k' keys reach theta with four groups per kept key, and
//      1.4 k' with two.
// The list is then sorted by rank (score descending, index ascending).
//
// Nodes stored in spatial order have their best keys side by side, in few
// groups, and more keys reach theta the fewer groups a tile has.  So groups
// are narrow rather than many tiles apart: pairs of rows for k <= 32 (8 max3 a
// tile, as for any wider group) and single rows above (16 max).  Against
// groups of four rows, same number of them (select call, us; the streaming
// kernel in brackets): 30k nodes, 4 heads, d = 32, k = 128, 64 clusters one
// after the other 1900 -> 681 [1755], roads along a Morton curve 1527 -> 832
// [7338]; 100k nodes, d = 16, k = 512, clusters 11374 -> 3028 [11751]; drawn
// positions 1278 -> 1261, 6210 -> 6172.
// A graph whose tiles fit the waves' registers (R tiles a wave: 512 keys)
// is scored once and its scores stay in registers between the passes.
//
// Lists hold CAP >= k + 32 keys.  A query whose list overflows (top keys
// packed into few groups, or many ties) ranks the CAP keys it has, takes the
// k-th of them, an exact (score, index) bound now, as its new threshold and
// lists again; after kRelist attempts the block walks the tiles one at a
// time, sorting whenever a list has no room for another tile, which ends
// for any input.
//
// What bounds it: large graphs the matrix cores (two passes of 100k nodes, 4
// heads, d = 32, 64 queries a block run at 1.03 PFLOP/s, where a large bf16
// matrix product reaches 1.25 on the same card), then the listing; small
// ones the chain of phases of one block (about 14 us at 2,000 nodes).
// Measured against the streaming kernel with its pre-passes (select call of
// one graph, us): 2,000 nodes, d = 16, k = 10 99 -> 18; 9,000 452 -> 34;
// 30,000 719 -> 104; 20,000 nodes, 4 heads, d = 128, k = 32 1554 -> 890;
// 30,000 nodes, 4 heads, d = 32, k = 256 21000 -> 1820.
#include "kmip_device.h"
#include "kmip_internal.h"

namespace kmip {
namespace {

constexpr int kRelist = 3;   // listings before the tile-by-tile walk

__device__ __forceinline__ int dense_row(int r, int half) {
    return 8 * (r >> 2) + 4 * half + (r & 3);
}

// Sum and maximum over the TPQ consecutive lanes of a query's team: row
// operations within 16 lanes, LDS permutes across rows.
template <int CTRL>
__device__ __forceinline__ int row_move(int v) {
    return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, false);
}

template <int TPQ>
__device__ __forceinline__ int team_sum(int v) {
    v += row_move<0xB1>(v);     // quad_perm [1,0,3,2]
    v += row_move<0x4E>(v);     // quad_perm [2,3,0,1]
    v += row_move<0x141>(v);    // row_half_mirror
    if constexpr (TPQ >= 16) v += row_move<0x140>(v);    // row_mirror
    if constexpr (TPQ >= 32) v += __shfl_xor(v, 16);
    if constexpr (TPQ >= 64) v += __shfl_xor(v, 32);
    return v;
}

template <int TPQ>
__device__ __forceinline__ uint32_t team_max(uint32_t v) {
    v = max(v, (uint32_t)row_move<0xB1>((int)v));
    v = max(v, (uint32_t)row_move<0x4E>((int)v));
    v = max(v, (uint32_t)row_move<0x141>((int)v));
    if constexpr (TPQ >= 16) v = max(v, (uint32_t)row_move<0x140>((int)v));
    if constexpr (TPQ >= 32) v = max(v, (uint32_t)__shfl_xor((int)v, 16));
    if constexpr (TPQ >= 64) v = max(v, (uint32_t)__shfl_xor((int)v, 32));
    return v;
}

// LDS of a block: the lists (QN x CAP keys), whose space the group maxima
// (row stride QN + 1 words, so that a team's reads meet few bank conflicts)
// use before, then the counters, thresholds and bounds, then the value buckets.
constexpr int kValueBuckets = 64;
constexpr uint32_t kWideBucket = 64;   // up to this many keys of a bucket, or half the list, are compared with each other

template <int W, int T, int GT, int CAP, int QN>
constexpr size_t dense_list_bytes() {
    const size_t lists = (size_t)QN * CAP * 8, maxima = (size_t)2 * GT * T * W * (QN + 1) * 4;
    return lists > maxima ? lists : maxima;
}
template <int W, int T, int GT, int CAP, int QN>
constexpr size_t dense_lds_bytes() {
    return dense_list_bytes<W, T, GT, CAP, QN>() + QN * (8 + 4 + 4) + (CAP > 128 ? QN * kValueBuckets * 4 : 0);
}

// Waves per SIMD: with lists of 256 keys the LDS holds two blocks a CU, so four
// waves, as many as the registers are held to, at 2 to 16 spilled ones (the
// resident form at d = 128 would spill 41 and keeps three).  With lists of 128 at
// d = 64 six, three blocks a CU, which 84 registers would make two (12 clouds of
// 1.5k-3k nodes, 2 heads, k = 32 90 -> 79 us).
constexpr int dense_waves(int d, int cap, int qn, int r) {
    return cap == 256 && (d < 128 || r == 0) ? 4 : d == 64 && cap == 128 && qn == 32 && r == 0 ? 6 : 1;
}

// R > 0: resident (graphs of at most 32 W R keys, read from K itself);
// R == 0: two passes over the tiled keys kp.  tasks == nullptr: one graph of
// N nodes, task b being its b-th run of 32 queries (64 for QN = 64).
template <int D, int W, int T, int GT, int CAP, int QN, int R>
__global__ __launch_bounds__(64 * W, dense_waves(D, CAP, QN, R)) void dense_select_kernel(
    const uint4* __restrict__ kp, const uint16_t* __restrict__ K, const uint16_t* __restrict__ Q,
    const Task* __restrict__ tasks, int32_t ntasks, int32_t N, int32_t H, int32_t k, int32_t ntiles, int32_t first,
    int32_t* __restrict__ topk_idx) {
    constexpr int NC = D / 16;
    constexpr int TPQ = 64 * W / QN;          // threads per query
    constexpr int NG = 2 * GT * T * W;        // group maxima per query
    constexpr int E = CAP / TPQ;              // list entries per thread
    constexpr bool kBuckets = CAP > 128;
    constexpr int QB = QN > 32 ? QN / 32 : 1;   // blocks of 32 queries a wave scores
    static_assert(TPQ == 8 || TPQ == 16 || TPQ == 32 || TPQ == 64, "a team is a part of a wave");
    static_assert(CAP % TPQ == 0 && (R == 0 || T == R), "whole entries per thread; one group set per resident tile");
    extern __shared__ uint64_t lds[];
    uint64_t* const list = lds;                                  // [QN][CAP]
    float* const gsh = reinterpret_cast<float*>(lds);            // [NG][QN + 1]
    char* const tail = reinterpret_cast<char*>(lds) + dense_list_bytes<W, T, GT, CAP, QN>();
    uint64_t* const bound = reinterpret_cast<uint64_t*>(tail);   // [QN] keys below it are not listed
    float* const theta_sh = reinterpret_cast<float*>(bound + QN);
    int32_t* const cnt = reinterpret_cast<int32_t*>(theta_sh + QN);
    int32_t* const hist = cnt + QN;                              // [QN][kValueBuckets]

    const int t = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63;
    const int col = lane & 31, half = lane >> 5;
    // tasks hold runs of at most 32 QB queries: QN = 16 takes one in two blocks
    constexpr int kRun = 32 * QB, kSub = kRun / QN;
    const int nblk = ntasks * kSub;
    const int block = first + blockIdx.x;
    const int head = block / nblk;
    const int b = block - head * nblk;
    Task tk = tasks != nullptr ? tasks[b / kSub] : Task{b / kSub * kRun, min(kRun, N - b / kSub * kRun), 0, N};
    if constexpr (kSub > 1) {
        tk.q_begin += b % kSub * QN;
        tk.q_count = min(QN, tk.q_count - b % kSub * QN);
        if (tk.q_count <= 0) return;
    }
    const int n = tk.key_hi - tk.key_lo;
    const int kk = min(n, k);

    bf16x8 bq[QB][NC];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        const int qi = 32 * qb + col;
        const bool valid = qi < tk.q_count && qi < QN;
        const uint16_t* qrow = Q + ((size_t)(valid ? tk.q_begin + qi : 0) * H + head) * D + 8 * half;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const uint4 u = valid ? *reinterpret_cast<const uint4*>(qrow + 16 * c) : make_uint4(0, 0, 0, 0);
            bq[qb][c] = __builtin_bit_cast(bf16x8, u);
        }
    }

    // Key tiles: tile i holds rows base + 32 i .. + 31 (kp's tiles start at a
    // multiple of 32; the resident variant's at the graph's first key).
    const int base = R > 0 ? tk.key_lo : tk.key_lo & ~31;
    const int nt = (tk.key_hi - base + 31) >> 5;
    // Pass 1 takes every sample-th tile (each wave by itself: runs of tiles left
    // out would hide whole runs of neighbouring best keys; 45k nodes of a smooth
    // road network in Morton order, d = 32, k = 16 1180 -> 884 us): theta is
    // then about the (sample k')-th best score, and pass 2 lists sample times as
    // many keys (1.2 sample k' < CAP).  Worth it where the tiles left out cost more than the extra listing,
    // which grows with k: a 100k-node graph at d = 32, k = 32 5.2 -> 4.6 ms,
    // 200k nodes at d = 16, k = 10 3.1 -> 2.5 (every third: 2.3), but 45k
    // nodes at d = 32, k = 32 1.19 -> 1.28.
    const int sample = CAP > 128 || nt * NC < 128 * k ? 1 : k <= 16 && nt * NC >= 512 * k ? 3 : 2;
    const uint4* tiles = kp + ((size_t)head * (ntiles + kPadTiles) + (base >> 5)) * (NC * 64) + lane;
    auto load_tile = [&](uint4 (&w)[NC], int i) {
        if constexpr (R > 0) {
            const int j = min(base + 32 * i + col, tk.key_hi - 1);
            const uint16_t* row = K + ((size_t)j * H + head) * D + 8 * half;
#pragma unroll
            for (int c = 0; c < NC; ++c) w[c] = *reinterpret_cast<const uint4*>(row + 16 * c);
        } else {
#pragma unroll
            for (int c = 0; c < NC; ++c) w[c] = tiles[(size_t)i * (NC * 64) + c * 64];
        }
    };
    // Scores of tile i for the wave's query blocks; rows outside the graph get -inf.
    auto score_tile = [&](const uint4 (&w)[NC], int i, f32x16 (&acc)[QB]) {
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            acc[qb] = f32x16{};
#pragma unroll
            for (int c = 0; c < NC; ++c)
                acc[qb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, w[c]), bq[qb][c], acc[qb], 0, 0, 0);
        }
        const int j0 = base + 32 * i;
        if (j0 < tk.key_lo || j0 + 32 > tk.key_hi) {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int j = j0 + dense_row(r, half);
                if (j < tk.key_lo || j >= tk.key_hi) {
#pragma unroll
                    for (int qb = 0; qb < QB; ++qb) acc[qb][r] = -INFINITY;
                }
            }
        }
    };

    // Scores the wave's tiles in order, PF loads ahead (the next tiles are in
    // flight while one is scored), and hands each to f(scores, tile, u), u
    // counting the wave's tiles modulo T.  The wave takes tiles first, first +
    // step, ...
    auto stream_tiles = [&](int first, int step, auto f) {
        constexpr int PF = NC >= 4 ? 1 : 2;
        constexpr int U = T > PF ? T : PF;
        static_assert(U % T == 0 && U % PF == 0, "powers of two");
        if (first >= nt) return;
        uint4 ring[PF][NC];
#pragma unroll
        for (int p = 0; p < PF; ++p) load_tile(ring[p], min(first + step * p, nt - 1));
        for (int i = first; i < nt;) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (i < nt) {
                    f32x16 acc[QB];
                    score_tile(ring[u % PF], i, acc);
                    load_tile(ring[u % PF], min(i + step * PF, nt - 1));
                    f(acc, i, u % T);
                    i += step;
                }
            }
        }
    };

    // ---- 1. group maxima ----
    f32x16 kept[R > 0 ? R : 1][QB];
    float gm[T][QB][GT];
#pragma unroll
    for (int u = 0; u < T; ++u)
#pragma unroll
        for (int qb = 0; qb < QB; ++qb)
#pragma unroll
            for (int g = 0; g < GT; ++g) gm[u][qb][g] = -INFINITY;
    auto add_groups = [&](const f32x16 (&a)[QB], float (&m)[QB][GT]) {
#pragma unroll
        for (int qb = 0; qb < QB; ++qb)
#pragma unroll
            for (int r = 0; r < 16; ++r) m[qb][r / (16 / GT)] = fmaxf(m[qb][r / (16 / GT)], a[qb][r]);
    };
    auto tile_groups = [&](const f32x16 (&a)[QB], float (&m)[QB][4]) {
#pragma unroll
        for (int qb = 0; qb < QB; ++qb)
#pragma unroll
            for (int g = 0; g < 4; ++g)
                m[qb][g] = fmaxf(fmaxf(a[qb][4 * g], a[qb][4 * g + 1]), fmaxf(a[qb][4 * g + 2], a[qb][4 * g + 3]));
    };
    if constexpr (R > 0) {
        uint4 w[R][NC];
#pragma unroll
        for (int u = 0; u < R; ++u)
            if (wave + W * u < nt) load_tile(w[u], wave + W * u);
#pragma unroll
        for (int u = 0; u < R; ++u) {
            if (wave + W * u < nt) {
                score_tile(w[u], wave + W * u, kept[u]);
                add_groups(kept[u], gm[u]);
            }
        }
    } else {
        stream_tiles(wave * sample, W * sample, [&](const f32x16 (&acc)[QB], int, int u) { add_groups(acc, gm[u]); });
    }
    if (QN >= 32 || col < QN) {
#pragma unroll
        for (int u = 0; u < T; ++u)
#pragma unroll
            for (int qb = 0; qb < QB; ++qb)
#pragma unroll
                for (int g = 0; g < GT; ++g)
                    gsh[(((wave * 2 + half) * T + u) * GT + g) * (QN + 1) + 32 * qb + col] = gm[u][qb][g];
    }
    if (t < QN) cnt[t] = 0;
    __syncthreads();

    // theta: the largest 20-bit prefix that k' group maxima reach
    const int q = t / TPQ, s = t % TPQ;
    const bool active = q < tk.q_count;
    {
        uint32_t code[NG / TPQ];
        uint32_t mx = 0, mnc = 0;   // largest code, largest complement
        int have = 0;
#pragma unroll
        for (int i = 0; i < NG / TPQ; ++i) {
            const float g = gsh[(s + TPQ * i) * (QN + 1) + q];
            code[i] = g > -INFINITY ? score_code(g) : 0u;
            mx = max(mx, code[i]);
            if (code[i] != 0u) {
                mnc = max(mnc, ~code[i]);
                ++have;
            }
        }
        mx = team_max<TPQ>(mx);
        const uint32_t mn = ~team_max<TPQ>(mnc);
        uint32_t T20 = 0;
        if (team_sum<TPQ>(have) >= kk) {
            // all maxima share the leading bits of the largest and smallest
            const uint32_t diff = mn ^ mx;
            const int top = diff == 0u ? -1 : 31 - __clz(diff);
            T20 = top < 0 ? mx : top >= 31 ? 0u : mx & ~((2u << top) - 1u);
            T20 &= 0xFFFFF000u;
            for (int bit = top; bit >= 12; --bit) {
                const uint32_t x = T20 | (1u << bit);
                int c = 0;
#pragma unroll
                for (int i = 0; i < NG / TPQ; ++i) c += code[i] >= x ? 1 : 0;
                if (team_sum<TPQ>(c) >= kk) T20 = x;
            }
        }
        if (s == 0) {
            theta_sh[q] = T20 == 0u ? -INFINITY : score_from_code(T20);
            bound[q] = 0ull;
        }
    }
    __syncthreads();

    // ---- 2. list the keys at or above the threshold ----
    // Scores a of tile i, whose maxima over rows 4 g .. 4 g + 3 are m: a tile
    // without a key to list costs three instructions past the maxima, and
    // only the groups that hold one are looked at row by row.  Listing again, a
    // lane raises its theta past the bound's own score beyond the bound's
    // index: many equal keys are looked at once only (20k nodes, 2 heads, d =
    // 128, 50 distinct keys, k = 32: 1617 -> 1254 us, the streaming kernel
    // 1374; 30k nodes, 4 heads, d = 32, zero queries 3915 -> 2601, 12253).
    // (Stopping also once the list is full, in the first listing: 932 and 831,
    // but 3% on inputs that never overflow.)
    auto list_tile = [&](const f32x16 (&a)[QB], const float (&m)[QB][4], int i, float (&theta)[QB],
                         const uint64_t (&bnd)[QB], bool again) {
        const int j0 = base + 32 * i;
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            const float top = fmaxf(fmaxf(fmaxf(m[qb][0], m[qb][1]), m[qb][2]), m[qb][3]);
            if (__builtin_amdgcn_ballot_w64(top >= theta[qb]) == 0ull) continue;
            const int qi = 32 * qb + col;
            // (no bound: index -1, the largest unsigned value)
            if (again && (uint32_t)j0 > (uint32_t)key_index(bnd[qb]))
                theta[qb] = fmaxf(theta[qb], score_from_code((uint32_t)(bnd[qb] >> 32) + 1u));
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                if (__builtin_amdgcn_ballot_w64(m[qb][g] >= theta[qb]) == 0ull) continue;
#pragma unroll
                for (int r = 4 * g; r < 4 * g + 4; ++r) {
                    if (a[qb][r] >= theta[qb]) {
                        const int j = j0 + dense_row(r, half);
                        const uint64_t key = make_key(a[qb][r], j);
                        if (j >= tk.key_lo && j < tk.key_hi && key >= bnd[qb] && (QN >= 32 || col < QN)) {
                            const int slot = atomicAdd(&cnt[qi], 1);
                            if (slot < CAP) list[qi * CAP + slot] = key;
                        }
                    }
                }
            }
        }
    };
    // Thresholds and bounds of a lane's queries (columns past the block's
    // queries list nothing: a padded query row scores 0 everywhere).
    auto limits = [&](float (&theta)[QB], uint64_t (&bnd)[QB]) {
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            const int qi = 32 * qb + col;
            const bool valid = qi < QN && qi < tk.q_count;
            theta[qb] = valid ? theta_sh[valid ? qi : 0] : INFINITY;
            bnd[qb] = bound[valid ? qi : 0];
        }
    };

    // Whether some list counts more than x keys.  The same answer for every
    // wave only if no wave changes a count between the barrier before the call
    // and one after it: the waves branch to barriers on it.
    auto any_above = [&](int x) {
        return __builtin_amdgcn_ballot_w64(cnt[lane & (QN - 1)] > x) != 0ull;
    };
    uint64_t* const row = list + q * CAP;
    int32_t* const dst = topk_idx + ((size_t)(tk.q_begin + (active ? q : 0)) * H + head) * k;
    // Places key e of query q at its rank: the k-th best becomes the query's
    // bound, and with `write` the best k are the row.
    auto place = [&](uint64_t e, int rank, bool write) {
        if (rank == k - 1) {
            bound[q] = e;
            theta_sh[q] = key_score(e);
        }
        if (write && rank < k) dst[rank] = key_index(e);
    };
    // Rank by comparing with all m keys of the list, four keys at a time.
    auto rank_all = [&](int m, bool write) {
#pragma unroll 1
        for (int i0 = s; i0 < m; i0 += 4 * TPQ) {
            uint64_t e[4];
            int rank[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                e[i] = i0 + TPQ * i < m ? row[i0 + TPQ * i] : ~0ull;
                rank[i] = 0;
            }
#pragma unroll 2
            for (int f = 0; f < m; ++f) {
                const uint64_t x = row[f];
#pragma unroll
                for (int i = 0; i < 4; ++i) rank[i] += x > e[i] ? 1 : 0;
            }
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (i0 + TPQ * i < m) place(e[i], rank[i], write);
        }
    };
    // The need-th largest of the team's nonzero words w (0: none), bit by bit
    // below the leading bits that all of them share.
    auto kth_word = [&](const uint32_t (&w)[E], int need) {
        uint32_t mx = 0, mnc = 0;
#pragma unroll
        for (int i = 0; i < E; ++i) {
            mx = max(mx, w[i]);
            mnc = max(mnc, w[i] != 0u ? ~w[i] : 0u);
        }
        mx = team_max<TPQ>(mx);
        const uint32_t diff = mx ^ ~team_max<TPQ>(mnc);
        const int bits = 32 - __clz(diff);
        uint32_t x = bits == 0 ? mx : mx >> (bits - 1) >> 1 << (bits - 1) << 1;
#pragma unroll 1
        for (int bit = bits - 1; bit >= 0; --bit) {
            const uint32_t y = x | (1u << bit);
            int c = 0;
#pragma unroll
            for (int i = 0; i < E; ++i) c += w[i] >= y ? 1 : 0;
            if (team_sum<TPQ>(c) >= need) x = y;
        }
        return x;
    };
    // The k-th largest of the list's m >= k keys: its code, then its ~index among
    // the keys of that code.  (One word of each key in registers at a time: the
    // registers decide how many waves a CU holds.)
    auto kth_key = [&](int m) {
        uint32_t w[E];
#pragma unroll
        for (int i = 0; i < E; ++i) w[i] = s + TPQ * i < m ? (uint32_t)(row[s + TPQ * i] >> 32) : 0u;
        const uint32_t code = kth_word(w, k);
        int above = 0;
#pragma unroll
        for (int i = 0; i < E; ++i) above += w[i] > code ? 1 : 0;
#pragma unroll
        for (int i = 0; i < E; ++i) w[i] = w[i] == code ? (uint32_t)row[s + TPQ * i] : 0u;
        return ((uint64_t)code << 32) | kth_word(w, k - team_sum<TPQ>(above));
    };
    // Moves the list's keys >= b to its front and returns their number (the
    // team's reads of a round come before its writes, which go to slots already
    // read).
    auto keep_from = [&](uint64_t b, int m) {
        int run = 0;
        for (int f0 = 0; f0 < m; f0 += TPQ) {
            const uint64_t x = f0 + s < m ? row[f0 + s] : 0ull;
            const bool keep = x != 0ull && x >= b;
            const uint64_t mine = __builtin_amdgcn_ballot_w64(keep) >> (lane - s) & (~0ull >> (64 - TPQ));
            __builtin_amdgcn_wave_barrier();
            if (keep) row[run + __builtin_popcountll(mine & ((1ull << s) - 1ull))] = x;
            __builtin_amdgcn_wave_barrier();
            run += __builtin_popcountll(mine);
        }
        return run;
    };
    // Rank by value buckets: bucket v holds the scores in the v-th part of
    // [lowest, highest], highest first, and the list is reordered by bucket;
    // a key's rank is the size of the buckets before its own plus the keys of
    // its own that beat it.  Where a bucket holds many keys (ties), only the k
    // best are kept and ranked against each other.  Without `write` the k-th
    // key is all that is wanted.  Every thread of the block calls it.  (64 graphs
    // of 100 to 450 nodes, 3 heads, d = 32, zero queries: k = 64 947 us with all
    // ties compared within their bucket, 112 so; k = 100 1020 and 138.)
    auto rank_buckets = [&](int m, bool write) {
        if (!write) {
            if (m >= k) {
                const uint64_t b = kth_key(m);
                if (s == 0) {
                    bound[q] = b;
                    theta_sh[q] = key_score(b);
                }
            }
            return;
        }
        uint64_t e[E];
        int slot[E];
        uint32_t mx = 0, mnc = 0;
#pragma unroll
        for (int i = 0; i < E; ++i) {
            e[i] = s + TPQ * i < m ? row[s + TPQ * i] : 0ull;
            if (e[i] != 0ull) {
                mx = max(mx, (uint32_t)(e[i] >> 32));
                mnc = max(mnc, ~(uint32_t)(e[i] >> 32));
            }
        }
        const float hi = score_from_code(team_max<TPQ>(mx)), lo = score_from_code(~team_max<TPQ>(mnc));
        const float inv = hi > lo ? (float)kValueBuckets / (hi - lo) : 0.0f;
        auto bucket = [&](uint64_t key) {
            const float x = fminf(fmaxf((hi - key_score(key)) * inv, 0.0f), (float)(kValueBuckets - 1));
            return min(max((int)x, 0), kValueBuckets - 1);
        };
        int32_t* h = hist + q * kValueBuckets;
        for (int v = s; v < kValueBuckets; v += TPQ) h[v] = 0;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < E; ++i) {
            slot[i] = s + TPQ * i;   // one score: one bucket, as the keys lie
            if (hi > lo && e[i] != 0ull) slot[i] = atomicAdd(&h[bucket(e[i])], 1);
        }
        if (!(hi > lo) && s == 0) h[0] = m;
        __syncthreads();
        // exclusive sums over the buckets: the team's first 16 lanes take 4 each
        uint32_t widest = 0;
        if (s < 16) {
            constexpr int V = kValueBuckets / 16;
            int c[V], sum = 0;
#pragma unroll
            for (int v = 0; v < V; ++v) {
                c[v] = h[V * s + v];
                sum += c[v];
                widest = max(widest, (uint32_t)c[v]);
            }
            int x = sum;
            x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xF, 0xF, true);
            x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xF, 0xF, true);
            x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xF, 0xF, true);
            x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xF, 0xF, true);
            int run = x - sum;
#pragma unroll
            for (int v = 0; v < V; ++v) {
                h[V * s + v] = run;
                run += c[v];
            }
        }
        widest = team_max<TPQ>(widest);
        __syncthreads();
#pragma unroll
        for (int i = 0; i < E; ++i)
            if (e[i] != 0ull) row[h[bucket(e[i])] + slot[i]] = e[i];
        __syncthreads();
        if (widest > max(kWideBucket, (uint32_t)m / 2u)) {
            rank_all(m > k ? keep_from(kth_key(m), m) : m, true);
            return;
        }
#pragma unroll 1
        for (int i = s; i < m; i += TPQ) {
            const uint64_t x = row[i];
            const int v = bucket(x);
            const int f1 = v + 1 < kValueBuckets ? h[v + 1] : m;
            const int f0 = h[v];
            int rank = f0;
#pragma unroll 4
            for (int f = f0; f < f1; ++f) rank += row[f] > x ? 1 : 0;
            place(x, rank, write);
        }
    };

    if constexpr (R > 0) {
        float theta[QB];
        uint64_t bnd[QB];
        limits(theta, bnd);
#pragma unroll
        for (int u = 0; u < R; ++u)
            if (wave + W * u < nt) {
                float m[QB][4];
#pragma unroll
                for (int qb = 0; qb < QB; ++qb)
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        m[qb][g] = gm[u][qb][GT / 4 * g];
#pragma unroll
                        for (int i = 1; i < GT / 4; ++i) m[qb][g] = fmaxf(m[qb][g], gm[u][qb][GT / 4 * g + i]);
                    }
                list_tile(kept[u], m, wave + W * u, theta, bnd, false);
            }
    }
#pragma unroll 1
    for (int at = 0; at < kRelist; ++at) {
        if (R == 0 || at > 0) {
            float theta[QB];
            uint64_t bnd[QB];
            limits(theta, bnd);
            stream_tiles(wave, W, [&](const f32x16 (&acc)[QB], int i, int) {
                float m[QB][4];
                tile_groups(acc, m);
                list_tile(acc, m, i, theta, bnd, at > 0);
            });
        }
        __syncthreads();
        const bool fits = !any_above(CAP);
        const int m = active ? min(cnt[q], CAP) : 0;
        if constexpr (kBuckets)
            rank_buckets(m, fits);
        else
            rank_all(m, fits);
        if (fits) {
            if (active)
                for (int p = m + s; p < k; p += TPQ) dst[p] = -1;
            return;
        }
        __syncthreads();
        if (t < QN) cnt[t] = 0;
        __syncthreads();
    }
    // Tile by tile: a list always has room for one more tile; when some list
    // has not, every list of more than k keys drops the keys below its k-th.
#pragma unroll 1
    for (int i = 0; i < nt; ++i) {
        if (wave == i % W) {
            uint4 cur[NC];
            f32x16 acc[QB];
            float theta[QB], m[QB][4];
            uint64_t bnd[QB];
            limits(theta, bnd);
            load_tile(cur, i);
            score_tile(cur, i, acc);
            tile_groups(acc, m);
            list_tile(acc, m, i, theta, bnd, true);
        }
        __syncthreads();
        const bool full = any_above(CAP - 32);
        __syncthreads();   // every wave has read the counts: the next tile may list
        if (!full) continue;
        const int m = active ? cnt[q] : 0;
        if (m > k) rank_all(m, false);
        __syncthreads();
        if (m > k) {
            const int run = keep_from(bound[q], m);
            if (s == 0) cnt[q] = run;
        }
        __syncthreads();
    }
    const int m = active ? cnt[q] : 0;
    rank_all(m, true);
    if (active)
        for (int p = m + s; p < k; p += TPQ) dst[p] = -1;
}

template <int D, int W, int T, int GT, int CAP, int QN, int R>
hipError_t launch_dense_t(const void* kp, const void* K, const void* Q, const Task* tasks, int32_t ntasks, int32_t N,
                          int32_t H, int32_t k, int32_t ntiles, int32_t* topk_idx, hipStream_t stream) {
    constexpr size_t lds = dense_lds_bytes<W, T, GT, CAP, QN>();
    static_assert(lds <= 160 * 1024, "LDS of a gfx950 workgroup");
    const void* fn = reinterpret_cast<const void*>(dense_select_kernel<D, W, T, GT, CAP, QN, R>);
    if (lds > 65536) {
        const hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    // Many heads of a few nodes: slices of at most 2^31 threads (fewer than 2^28
    // blocks in all, as N H < 2^27)
    constexpr int64_t kSlice = (int64_t(1) << 31) / (64 * W);
    const int64_t blocks = (int64_t)ntasks * H * (QN < 32 ? 32 / QN : 1);
    for (int64_t first = 0; first < blocks; first += kSlice) {
        hipLaunchKernelGGL((dense_select_kernel<D, W, T, GT, CAP, QN, R>),
                           dim3((unsigned)(blocks - first < kSlice ? blocks - first : kSlice)), dim3(64 * W), lds, stream,
                           reinterpret_cast<const uint4*>(kp), reinterpret_cast<const uint16_t*>(K),
                           reinterpret_cast<const uint16_t*>(Q), tasks, ntasks, N, H, k, ntiles, (int32_t)first,
                           topk_idx);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace

hipError_t launch_dense_select(const void* kp, const void* K, const void* Q, const Task* tasks, int32_t ntasks,
                               int32_t N, int32_t H, int32_t d, int32_t k, int32_t ntiles, int32_t run, int32_t resident,
                               int32_t* topk_idx, hipStream_t stream) {
    if (ntasks <= 0) return hipSuccess;
#define KMIP_DENSE(DD, WW, TT, GG, CC, QQ, RR) \
    return launch_dense_t<DD, WW, TT, GG, CC, QQ, RR>(kp, K, Q, tasks, ntasks, N, H, k, ntiles, topk_idx, stream)
    // A resident graph has n / 4 groups of four rows, or n / 2 pairs.  Where k
    // comes near the number of groups, the lists of more than 256 nodes
    // overflow; where it does not, the larger number takes longer to search (up
    // to 128 nodes every key is listed either way).
    // 64 graphs, 3 heads, d = 32, four rows against pairs (us): about 277 nodes
    // k = 65 81 and 74, k = 80 119 and 78; 377 nodes k = 72 101 and 102, k = 90
    // 140 and 108; 478 nodes k = 65 115 and 122, k = 100 147 and 137.
#define KMIP_DENSE_D(DD)                                                   \
    if (d == DD && resident > 0 && run == 32) {                            \
        if (k <= 32) KMIP_DENSE(DD, 8, 2, 4, 128, 32, 2);                  \
        if (k <= 128 && resident > 128 && resident < 5 * k)                \
            KMIP_DENSE(DD, 8, 2, 8, 256, 32, 2);                           \
        if (k <= 128) KMIP_DENSE(DD, 8, 2, 4, 256, 32, 2);                 \
    }                                                                      \
    if (d == DD && resident == 0 && k <= 32) {                             \
        if (run == 64) KMIP_DENSE(DD, 8, 1, 8, 128, 64, 0);                \
        if (run == 32) KMIP_DENSE(DD, 8, 1, 8, 128, 32, 0);                \
    }                                                                      \
    if (d == DD && resident == 0 && k <= 128 && run == 32) KMIP_DENSE(DD, 8, 2, 16, 256, 32, 0);
    KMIP_DENSE_D(16)
    KMIP_DENSE_D(32)
    KMIP_DENSE_D(64)
    KMIP_DENSE_D(128)
#undef KMIP_DENSE_D
#define KMIP_DENSE_D(DD)                                                   \
    if (d == DD && resident == 0 && run == 32) {                           \
        if (k <= 256) KMIP_DENSE(DD, 16, 2, 16, 512, 32, 0);               \
        if (k <= 512) KMIP_DENSE(DD, 16, 2, 16, 1024, 16, 0);              \
    }
    KMIP_DENSE_D(16)
    KMIP_DENSE_D(32)
    KMIP_DENSE_D(64)
#undef KMIP_DENSE_D
#undef KMIP_DENSE
    return hipErrorInvalidValue;
}

}  // namespace kmip

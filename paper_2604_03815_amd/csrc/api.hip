// Host side of the kmip C ABI (declared in include/kmip.h): argument
// validation, workspace layout, the block-diagonal work list and launches.
#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <string>
#include <vector>

#include "kmip.h"
#include "kmip_internal.h"

namespace {
thread_local std::string g_last_error;
}  // namespace

namespace kmip {

kmip_status_t record_error(kmip_status_t s, const char* fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof(buf), fmt, ap);
    va_end(ap);
    g_last_error = buf;
    return s;
}

}  // namespace kmip

namespace {

using kmip::record_error;

kmip_status_t ok() {
    g_last_error.clear();
    return KMIP_OK;
}

kmip_status_t hip_fail(hipError_t e, const char* what) {
    return record_error(KMIP_ERR_HIP, "%s: %s", what, hipGetErrorString(e));
}

constexpr size_t kAlign = 256;

// Pinned host staging for the block-diagonal work list, so that its upload
// is an asynchronous copy (a copy from pageable memory blocks the caller
// until the stream reaches it).  Two buffers per device, used in turn; a
// buffer is refilled only after the copy that last read it has completed
// (an event recorded behind that copy).  Kept until the process ends.
struct Staging {
    void* buf[2] = {nullptr, nullptr};
    size_t cap[2] = {0, 0};
    hipEvent_t ev[2] = {nullptr, nullptr};
    int next = 0;
};
constexpr int kMaxDevices = 64;
std::mutex g_stage_mu;
Staging g_stage[kMaxDevices];

// Copies `bytes` from host `src` to device `dst` on `stream` through the
// calling device's staging buffers.
hipError_t upload_async(void* dst, const void* src, size_t bytes, hipStream_t stream) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipMemcpyAsync(dst, src, bytes, hipMemcpyHostToDevice, stream);
    std::lock_guard<std::mutex> lock(g_stage_mu);
    Staging& st = g_stage[dev];
    const int i = st.next;
    st.next ^= 1;
    if (st.ev[i] == nullptr) {
        if ((e = hipEventCreateWithFlags(&st.ev[i], hipEventDisableTiming)) != hipSuccess) return e;
    } else if ((e = hipEventSynchronize(st.ev[i])) != hipSuccess) {
        return e;
    }
    if (st.cap[i] < bytes) {
        if (st.buf[i] != nullptr && (e = hipHostFree(st.buf[i])) != hipSuccess) return e;
        st.buf[i] = nullptr;
        st.cap[i] = 0;
        const size_t cap = std::max<size_t>(bytes, 64 * 1024);
        if ((e = hipHostMalloc(&st.buf[i], cap, hipHostMallocDefault)) != hipSuccess) return e;
        st.cap[i] = cap;
    }
    std::memcpy(st.buf[i], src, bytes);
    if ((e = hipMemcpyAsync(dst, st.buf[i], bytes, hipMemcpyHostToDevice, stream)) != hipSuccess) return e;
    return hipEventRecord(st.ev[i], stream);
}

size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// Sizes shared by all entry points.
kmip_status_t check_sizes(int64_t N, int32_t H, int32_t d, int32_t k) {
    if (N < 0 || N >= (int64_t(1) << 31)) return record_error(KMIP_ERR_INVALID_ARG, "N=%lld out of range", (long long)N);
    if (H < 1) return record_error(KMIP_ERR_INVALID_ARG, "H=%d must be >= 1", H);
    if (k < 1) return record_error(KMIP_ERR_INVALID_ARG, "k=%d must be >= 1", k);
    if (d != 16 && d != 32 && d != 64 && d != 128)
        return record_error(KMIP_ERR_UNSUPPORTED, "d=%d not in {16, 32, 64, 128}", d);
    const int32_t kmax = d == 128 ? KMIP_MAX_K_WIDE : KMIP_MAX_K;
    if (k > kmax) return record_error(KMIP_ERR_UNSUPPORTED, "k=%d exceeds %d for d=%d", k, kmax, d);
    const int64_t wide = N * (int64_t)H * std::max<int64_t>(d, k);
    if (wide >= (int64_t(1) << 31)) return record_error(KMIP_ERR_INVALID_ARG, "N*H*max(d,k) >= 2^31");
    return KMIP_OK;
}

// The value width, besides the sizes check_sizes covers.
kmip_status_t check_value_width(int64_t N, int32_t H, int32_t dv) {
    if (dv != 16 && dv != 32 && dv != 64 && dv != 128)
        return record_error(KMIP_ERR_UNSUPPORTED, "d_V=%d not in {16, 32, 64, 128}", dv);
    if (N * (int64_t)H * dv >= (int64_t(1) << 31)) return record_error(KMIP_ERR_INVALID_ARG, "N*H*d_V >= 2^31");
    return KMIP_OK;
}

// Finite test on the bits: the sources are built with -fno-honor-nans (for
// the kernels' max3 chains), under which std::isfinite may assume no NaN.
bool finite_bits(float x) {
    uint32_t b;
    std::memcpy(&b, &x, sizeof(b));
    return (b & 0x7F800000u) != 0x7F800000u;
}

// Attention dropout: a rate in [0, 1); keep draws are needed for a rate > 0.
kmip_status_t check_dropout(const uint8_t* keep, float rate) {
    if (!finite_bits(rate) || rate < 0.0f || rate >= 1.0f)
        return record_error(KMIP_ERR_INVALID_ARG, "drop_rate must lie in [0, 1)");
    if (keep == nullptr && rate != 0.0f) return record_error(KMIP_ERR_INVALID_ARG, "drop_rate > 0 needs keep draws");
    return KMIP_OK;
}

kmip_status_t check_scale(float scale) {
    if (!finite_bits(scale) || !(scale > 0.0f)) return record_error(KMIP_ERR_INVALID_ARG, "scale must be finite and > 0");
    return KMIP_OK;
}

kmip_status_t check_offsets(const int32_t* off, int32_t G, int64_t N) {
    if (off == nullptr) return KMIP_OK;
    if (G < 1) return record_error(KMIP_ERR_INVALID_ARG, "num_graphs=%d must be >= 1 with offsets", G);
    if (off[0] != 0) return record_error(KMIP_ERR_INVALID_ARG, "graph_offsets[0]=%d must be 0", off[0]);
    for (int32_t g = 0; g < G; ++g)
        if (off[g + 1] < off[g]) return record_error(KMIP_ERR_INVALID_ARG, "graph_offsets decrease at %d", g);
    if (off[G] != N) return record_error(KMIP_ERR_INVALID_ARG, "graph_offsets[G]=%d != N=%lld", off[G], (long long)N);
    return KMIP_OK;
}

int32_t num_tiles(int64_t N) { return (int32_t)((N + 31) / 32); }

size_t packed_k_bytes(int64_t N, int32_t H, int32_t d) {
    return (size_t)H * (size_t)(num_tiles(N) + kmip::kPadTiles) * 32 * (size_t)d * 2;
}

// The tiled keys, before the counters.
size_t tiled_bytes(int64_t N, int32_t H, int32_t d) { return align_up(packed_k_bytes(N, H, d)); }

// The select kernel's per-XCD work counters and pacers, after the tiled keys.
constexpr size_t kCounterBytes = kmip::kSelectCounterBytes;

// Upper bound on the work-list length for any query-block size.
size_t max_tasks(int64_t N, int32_t G) { return (size_t)(N / 32 + G + 1); }

// Query blocks of 32 per wave: two when k and d are small and there are
// enough items to fill the chip, one otherwise (bounded by LDS per workgroup
// and, at d = 128, by registers).
// Candidate slots per lane: few, since LDS bounds the resident waves per CU
// and occupancy pays more than the extra merges cost (4 with two blocks, 8
// with one, measured on the 100k/500k/262k-node workloads).
kmip::SelectShape choose_shape(int64_t N, int32_t H, int32_t d, int32_t k, int32_t G) {
    const int64_t items = (N + 63) / 64 * H;
    if (k <= 32 && d <= 64 && items >= 8192 && G == 1) return kmip::SelectShape{2, 4};
    return kmip::SelectShape{1, 8};
}

// How a graph of n nodes is selected: scores in registers, two dense passes,
// or the streaming kernel.
enum SelectPath { kPathResident = 0, kPathDense = 1, kPathStream = 2 };
// Dense passes cost n^2 d per head; for one graph the streaming kernel's
// pre-passes cost about 0.5 ms and its time depends on how many key blocks
// the bounds rule out.  For one graph the lines lie where the dense passes
// are still faster on inputs that prune well (a point cloud, 4 heads, k = 32,
// select with pre-passes, streaming against dense: 65k nodes at d = 16 1.87
// against 1.18 ms, 46k at d = 32 1.54 against 0.95, 32k at d = 64 1.99 against
// 0.83; 100k at d = 32 2.3 against more than 3); with many heads the
// pre-passes weigh less (per head beyond the first, 45k nodes at d = 32: 157
// against 224 us, 30k: 127 against 137).  At d = 128 and in a batch
// nothing is pruned, but past 64k nodes the keys leave the L2 and the
// streaming kernel, whose waves keep to the same tiles, is as fast.  Wide keys
// (d = 128, or 64 in a batch) leave it sooner where k > 32, since a block then
// holds 32 queries, and up to k = 64 the streaming kernel's trees are still
// small (dense against streaming, us; 4 heads, d = 128: 36k nodes, k = 33 3661 and
// 3710, 40k 4357 and 4023, 64k 10742 and 8253; k = 50 6662 and 6712 at 50k, 10867
// and 8913 at 64k; k = 64 6856 and 7880, 10894 and 10499; one head, k = 33 1494
// and 1735 at 45k, 1855 and 1858 at 50k; two graphs of 60k, 4 heads, d = 64, k =
// 33 9216 and 7226, four of 30k, 8 heads 9836 and 9691).  Above
// k = 128 the streaming kernel's trees leave room for one or two waves per
// CU (k = 256, 200k nodes, 2 heads, d = 16: 27 against 14 ms).
SelectPath select_path(int64_t n, int32_t G, int32_t H, int32_t d, int32_t k) {
    if (n <= kmip::kResidentGraph && k <= KMIP_MAX_K_WIDE) return kPathResident;
    int64_t most = 65536;
    if (k > KMIP_MAX_K_WIDE)
        most = 200000;
    else if (G == 1 && d == 16)
        most = H <= 8 ? 65536 : 49152;
    else if (G == 1 && d == 32)
        most = H <= 8 ? 46000 : 30000;
    else if (G == 1 && d == 64)
        most = 32768;
    else if (d >= 64 && k > 32 && k < 64)
        most = G == 1 && H == 1 ? 49152 : 32768;
    return n <= most ? kPathDense : kPathStream;
}

// Queries are grouped by direction (group.hip) and keys stored in bounded
// superblocks (keyorder.hip) for a single graph on the streaming path of at
// least 8192 nodes, at d <= 64 (the key-order kernels are built for those
// widths).
// (The workspace holds the grouping and the order for every such graph,
// whichever path takes it.)
bool sized_for_grouping(int64_t N, int32_t G, int32_t d) { return G == 1 && N >= 8192 && d <= 64; }
bool use_grouping(int64_t N, int32_t G, int32_t H, int32_t d, int32_t k) {
    return sized_for_grouping(N, G, d) && select_path(N, G, H, d, k) == kPathStream;
}

// Queries per dense task: 64 share each key tile's load once the scan outweighs
// the per-query work after it, where fewer workgroups would leave waves idle
// (one head, d = 16: 20k nodes 65 us with 32, 77 with 64; 30k 112 and 104; one
// head, d = 64: 9k nodes 58 and 64, 14k 86 and 82).  n: the largest graph.
int32_t dense_run(int64_t n, int32_t d, int32_t k) {
    return k <= 32 && (n + 31) / 32 * (d / 16 + 1) >= 1900 ? 64 : 32;
}

// Workspace of kmip_topk_prefilter, in order: the bf16 key tiles and the
// select kernel's counters (for the query blocks it redoes), the int8 key
// tiles, the per-head quantisation figures, the candidate lists and their
// lengths, the overflow flags, the redo count and the redo task list.
struct PrefilterLayout {
    size_t tiles8, hstat, cand, ccount, flags, count, tasks, total;
};

PrefilterLayout prefilter_layout(int64_t N, int32_t H, int32_t d) {
    PrefilterLayout L{};
    const size_t nblocks = (size_t)num_tiles(N);
    size_t off = tiled_bytes(N, H, d) + kCounterBytes;
    L.tiles8 = off;
    off += align_up(kmip::prefilter_tile_bytes((int32_t)N, H, d));
    L.hstat = off;
    off += align_up((size_t)4 * H * sizeof(uint32_t));
    L.cand = off;
    off += align_up((size_t)N * H * kmip::kPrefilterCap * sizeof(int32_t));
    L.ccount = off;
    off += align_up((size_t)N * H * 2 * sizeof(int32_t));
    L.flags = off;
    off += align_up((size_t)H * nblocks * sizeof(int32_t));
    L.count = off;
    off += align_up(sizeof(int32_t));
    L.tasks = off;
    off += align_up(nblocks * sizeof(kmip::Task));
    L.total = off;
    return L;
}

// kmip_attend_ex with an optional query order (perm [H][N], the forward's
// grouping, or nullptr) for the order the aggregate takes query-heads in, and
// whether the call knows that the queries belong to one graph.
kmip_status_t attend_checked(const void* Q, const void* K, const void* V, int64_t N, int32_t H, int32_t d,
                             int32_t dv, int32_t k, float scale, const int32_t* topk_idx, const uint8_t* keep,
                             float drop_rate, const int32_t* perm, bool one_graph, float* out, float* lse, void* stream_) {
    kmip_status_t s = check_sizes(N, H, d, k);
    if (s != KMIP_OK) return s;
    if ((s = check_value_width(N, H, dv)) != KMIP_OK) return s;
    if ((s = check_scale(scale)) != KMIP_OK) return s;
    if ((s = check_dropout(keep, drop_rate)) != KMIP_OK) return s;
    if (N == 0) return ok();
    if (!Q || !K || !V || !topk_idx || !out || !lse)
        return record_error(KMIP_ERR_INVALID_ARG, "null buffer passed to kmip_attend");
    if (!aligned16(Q) || !aligned16(K) || !aligned16(V))
        return record_error(KMIP_ERR_INVALID_ARG, "Q, K and V must be 16-byte aligned");
    hipError_t e = kmip::launch_attend(Q, K, V, topk_idx, keep, 1.0f / (1.0f - drop_rate), (int32_t)N, H, d, dv,
                                       k, scale, perm, one_graph, out, lse, reinterpret_cast<hipStream_t>(stream_));
    if (e != hipSuccess) return hip_fail(e, "attend launch");
    return ok();
}

}  // namespace

extern "C" {

const char* kmip_status_string(kmip_status_t s) {
    switch (s) {
        case KMIP_OK: return "ok";
        case KMIP_ERR_INVALID_ARG: return "invalid argument";
        case KMIP_ERR_UNSUPPORTED: return "unsupported size";
        case KMIP_ERR_WORKSPACE: return "workspace missing or too small";
        case KMIP_ERR_HIP: return "HIP error";
    }
    return "unknown status";
}

const char* kmip_last_error(void) { return g_last_error.c_str(); }

size_t kmip_topk_workspace_size(int64_t N, int32_t H, int32_t d, int32_t k, int32_t num_graphs) {
    if (check_sizes(N, H, d, k) != KMIP_OK) return 0;
    const int32_t G = num_graphs < 1 ? 1 : num_graphs;
    size_t bytes = tiled_bytes(N, H, d) + kCounterBytes;
    if (G > 1) bytes += align_up(max_tasks(N, G) * sizeof(kmip::Task));
    if (sized_for_grouping(N, G, d))
        bytes += align_up(kmip::group_workspace_bytes((int32_t)N, H, d)) +
                 align_up(kmip::key_order_workspace_bytes((int32_t)N, H, d));
    return bytes;
}

size_t kmip_fwd_workspace_size(int64_t N, int32_t H, int32_t d, int32_t k, int32_t num_graphs) {
    return kmip_topk_workspace_size(N, H, d, k, num_graphs);
}

kmip_status_t kmip_topk(const void* Q, const void* K, const int32_t* graph_offsets,
                        int32_t num_graphs, int64_t N, int32_t H, int32_t d, int32_t k,
                        int32_t* topk_idx, void* workspace, size_t workspace_bytes,
                        void* stream) {
    return kmip_topk_with_events(Q, K, graph_offsets, num_graphs, N, H, d, k, topk_idx, workspace,
                                 workspace_bytes, stream, nullptr, nullptr);
}

kmip_status_t kmip_topk_with_events(const void* Q, const void* K, const int32_t* graph_offsets,
                                    int32_t num_graphs, int64_t N, int32_t H, int32_t d, int32_t k,
                                    int32_t* topk_idx, void* workspace, size_t workspace_bytes,
                                    void* stream_, void* select_start, void* select_stop) {
    kmip_status_t s = check_sizes(N, H, d, k);
    if (s != KMIP_OK) return s;
    if ((s = check_offsets(graph_offsets, num_graphs, N)) != KMIP_OK) return s;
    if (N == 0) return ok();
    if (!Q || !K || !topk_idx) return record_error(KMIP_ERR_INVALID_ARG, "null Q, K or topk_idx");
    if (!aligned16(Q) || !aligned16(K)) return record_error(KMIP_ERR_INVALID_ARG, "Q and K must be 16-byte aligned");
    const int32_t G = graph_offsets ? num_graphs : 1;
    const size_t need = kmip_topk_workspace_size(N, H, d, k, G);
    if (workspace == nullptr || workspace_bytes < need)
        return record_error(KMIP_ERR_WORKSPACE, "workspace of %zu bytes < %zu required", workspace_bytes, need);
    if ((reinterpret_cast<uintptr_t>(workspace) & (kAlign - 1)) != 0)
        return record_error(KMIP_ERR_WORKSPACE, "workspace must be 256-byte aligned");
    hipStream_t stream = reinterpret_cast<hipStream_t>(stream_);

    const int32_t n32 = (int32_t)N;
    const int32_t ntiles = num_tiles(N);
    char* ws = reinterpret_cast<char*>(workspace);
    void* kp = ws;
    const kmip::SelectShape shape = choose_shape(N, H, d, k, G);
    const int32_t qb = shape.qb;

    // the largest graph of each path
    int64_t largest[3] = {0, 0, 0};
    for (int32_t g = 0; g < G; ++g) {
        const int64_t n = G > 1 ? graph_offsets[g + 1] - graph_offsets[g] : N;
        int64_t& most = largest[select_path(n, G, H, d, k)];
        most = std::max(most, n);
    }
    const int32_t run = dense_run(largest[kPathDense], d, k);
    auto step_of = [&](int path) { return path == kPathResident ? 32 : path == kPathDense ? run : 32 * qb; };
    // Tasks by path: [0, nres) resident, then ndense, then nstream.
    const kmip::Task* dtasks = nullptr;
    int32_t count[3] = {0, 0, 0};
    if (G > 1) {
        // Block-diagonal batch: one task per run of 32 queries (32*qb on the
        // streaming path) of a graph, heaviest first within its path (cost ~
        // queries x keys) to balance the tail.
        std::vector<kmip::Task> tasks;
        tasks.reserve(max_tasks(N, G));
        for (int path = kPathResident; path <= kPathStream; ++path) {
            const size_t first = tasks.size();
            for (int32_t g = 0; g < G; ++g) {
                const int32_t lo = graph_offsets[g], hi = graph_offsets[g + 1];
                if (select_path(hi - lo, G, H, d, k) != path) continue;
                const int32_t step = step_of(path);
                for (int32_t q0 = lo; q0 < hi; q0 += step)
                    tasks.push_back(kmip::Task{q0, std::min(step, hi - q0), lo, hi});
            }
            std::stable_sort(tasks.begin() + first, tasks.end(), [](const kmip::Task& a, const kmip::Task& b) {
                return (int64_t)a.q_count * (a.key_hi - a.key_lo) > (int64_t)b.q_count * (b.key_hi - b.key_lo);
            });
            count[path] = (int32_t)(tasks.size() - first);
        }
        void* dst = ws + tiled_bytes(N, H, d) + kCounterBytes;
        hipError_t e = upload_async(dst, tasks.data(), tasks.size() * sizeof(kmip::Task), stream);
        if (e != hipSuccess) return hip_fail(e, "work list upload");
        dtasks = reinterpret_cast<const kmip::Task*>(dst);
    } else {
        const SelectPath path = select_path(N, G, H, d, k);
        const int32_t step = step_of(path);
        count[path] = (int32_t)((N + step - 1) / step);
    }

    // A single large graph: queries grouped by direction, keys stored in
    // superblock order with bounds.
    kmip::QueryGroups groups{};
    kmip::KeyOrder keys{};
    const bool grouped = use_grouping(N, G, H, d, k);
    if (grouped) {
        char* gws = ws + tiled_bytes(N, H, d) + kCounterBytes;
        hipError_t e = kmip::launch_group_queries(Q, n32, H, d, gws, &groups, stream);
        if (e != hipSuccess) return hip_fail(e, "query grouping launch");
        char* kws = gws + align_up(kmip::group_workspace_bytes(n32, H, d));
        e = kmip::launch_key_order(K, n32, H, d, ntiles, kws, &keys, stream);
        if (e != hipSuccess) return hip_fail(e, "key order launch");
    }
    hipError_t e;
    if (count[kPathDense] + count[kPathStream] > 0 &&
        (e = kmip::launch_pack_k(K, grouped ? keys.perm : nullptr, grouped ? keys.rows : nullptr, kp, n32, H, d, ntiles,
                                 stream)) != hipSuccess)
        return hip_fail(e, "pack_k launch");
    int32_t* work_ctr = reinterpret_cast<int32_t*>(ws + tiled_bytes(N, H, d));
    hipEvent_t ev_start = reinterpret_cast<hipEvent_t>(select_start);
    hipEvent_t ev_stop = reinterpret_cast<hipEvent_t>(select_stop);
    // the events bracket every select launch
    if (count[kPathResident] + count[kPathDense] > 0 && ev_start != nullptr) {
        if ((e = hipEventRecord(ev_start, stream)) != hipSuccess) return hip_fail(e, "event record");
        ev_start = nullptr;
    }
    for (int path = kPathResident; path <= kPathDense; ++path) {
        e = kmip::launch_dense_select(kp, K, Q, dtasks, count[path], n32, H, d, k, ntiles, step_of(path),
                                      path == kPathResident ? (int32_t)largest[path] : 0, topk_idx, stream);
        if (e != hipSuccess) return hip_fail(e, "dense select launch");
        if (dtasks != nullptr) dtasks += count[path];
    }
    if (count[kPathStream] > 0) {
        e = kmip::launch_select(kp, Q, K, dtasks, grouped ? &groups : nullptr, grouped ? &keys : nullptr,
                                count[kPathStream], n32, H, d, k, ntiles, shape, work_ctr, topk_idx, stream, ev_start,
                                ev_stop);
        if (e != hipSuccess) return hip_fail(e, "select launch");
    } else if (ev_stop != nullptr && (e = hipEventRecord(ev_stop, stream)) != hipSuccess) {
        return hip_fail(e, "event record");
    }
    return ok();
}


size_t kmip_topk_prefilter_workspace_size(int64_t N, int32_t H, int32_t d, int32_t k) {
    if (check_sizes(N, H, d, k) != KMIP_OK || k > kmip::kPrefilterMaxK) return 0;
    return prefilter_layout(N, H, d).total;
}

kmip_status_t kmip_topk_prefilter(const void* Q, const void* K, int64_t N, int32_t H, int32_t d, int32_t k,
                                  int32_t* topk_idx, int32_t* redone, void* workspace, size_t workspace_bytes,
                                  void* stream_) {
    kmip_status_t s = check_sizes(N, H, d, k);
    if (s != KMIP_OK) return s;
    if (k > kmip::kPrefilterMaxK)
        return record_error(KMIP_ERR_UNSUPPORTED, "the prefilter takes k <= %d (got %d)", kmip::kPrefilterMaxK, k);
    if (N == 0) {
        hipError_t e = redone != nullptr ? kmip::launch_fill_zero(reinterpret_cast<float*>(redone), 1,
                                                                 reinterpret_cast<hipStream_t>(stream_))
                                         : hipSuccess;
        return e == hipSuccess ? ok() : hip_fail(e, "redo count");
    }
    if (!Q || !K || !topk_idx) return record_error(KMIP_ERR_INVALID_ARG, "null Q, K or topk_idx");
    if (!aligned16(Q) || !aligned16(K)) return record_error(KMIP_ERR_INVALID_ARG, "Q and K must be 16-byte aligned");
    const PrefilterLayout L = prefilter_layout(N, H, d);
    if (workspace == nullptr || workspace_bytes < L.total)
        return record_error(KMIP_ERR_WORKSPACE, "workspace of %zu bytes < %zu required", workspace_bytes, L.total);
    if ((reinterpret_cast<uintptr_t>(workspace) & (kAlign - 1)) != 0)
        return record_error(KMIP_ERR_WORKSPACE, "workspace must be 256-byte aligned");
    hipStream_t stream = reinterpret_cast<hipStream_t>(stream_);
    char* ws = reinterpret_cast<char*>(workspace);
    const int32_t n32 = (int32_t)N, ntiles = num_tiles(N);
    kmip::Task* tasks = reinterpret_cast<kmip::Task*>(ws + L.tasks);
    hipError_t e = kmip::launch_prefilter(K, Q, n32, H, d, k, reinterpret_cast<uint32_t*>(ws + L.hstat),
                                          reinterpret_cast<uint4*>(ws + L.tiles8), reinterpret_cast<int32_t*>(ws + L.cand),
                                          reinterpret_cast<int32_t*>(ws + L.ccount),
                                          reinterpret_cast<int32_t*>(ws + L.flags),
                                          reinterpret_cast<int32_t*>(ws + L.count), tasks, topk_idx, stream);
    if (e != hipSuccess) return hip_fail(e, "prefilter launch");
    // the query blocks whose candidate lists overflowed, through the select
    // kernel (every other entry of the list is a zero-query task it skips)
    if ((e = kmip::launch_pack_k(K, nullptr, nullptr, ws, n32, H, d, ntiles, stream)) != hipSuccess)
        return hip_fail(e, "pack_k launch");
    int32_t* work_ctr = reinterpret_cast<int32_t*>(ws + tiled_bytes(N, H, d));
    e = kmip::launch_select(ws, Q, K, tasks, nullptr, nullptr, ntiles, n32, H, d, k, ntiles, kmip::SelectShape{1, 8},
                            work_ctr, topk_idx, stream, nullptr, nullptr);
    if (e != hipSuccess) return hip_fail(e, "select launch");
    if (redone != nullptr &&
        (e = hipMemcpyAsync(redone, ws + L.count, sizeof(int32_t), hipMemcpyDeviceToDevice, stream)) != hipSuccess)
        return hip_fail(e, "redo count copy");
    return ok();
}

kmip_status_t kmip_attend_ex(const void* Q, const void* K, const void* V, int64_t N, int32_t H,
                             int32_t d, int32_t dv, int32_t k, float scale, const int32_t* topk_idx,
                             const uint8_t* keep, float drop_rate, float* out, float* lse, void* stream_) {
    return attend_checked(Q, K, V, N, H, d, dv, k, scale, topk_idx, keep, drop_rate, nullptr, false, out, lse,
                          stream_);
}

kmip_status_t kmip_attend(const void* Q, const void* K, const void* V, int64_t N, int32_t H,
                          int32_t d, int32_t k, float scale, const int32_t* topk_idx, float* out,
                          float* lse, void* stream) {
    return kmip_attend_ex(Q, K, V, N, H, d, d, k, scale, topk_idx, nullptr, 0.0f, out, lse, stream);
}

kmip_status_t kmip_fwd_ex(const void* Q, const void* K, const void* V, const int32_t* graph_offsets,
                          int32_t num_graphs, int64_t N, int32_t H, int32_t d, int32_t dv, int32_t k,
                          float scale, const uint8_t* keep, float drop_rate, float* out, int32_t* topk_idx,
                          float* lse, void* workspace, size_t workspace_bytes, void* stream) {
    return kmip_fwd_ex_with_events(Q, K, V, graph_offsets, num_graphs, N, H, d, dv, k, scale, keep, drop_rate, out,
                                   topk_idx, lse, workspace, workspace_bytes, stream, nullptr, nullptr, nullptr);
}

kmip_status_t kmip_fwd_ex_with_events(const void* Q, const void* K, const void* V, const int32_t* graph_offsets,
                                      int32_t num_graphs, int64_t N, int32_t H, int32_t d, int32_t dv, int32_t k,
                                      float scale, const uint8_t* keep, float drop_rate, float* out,
                                      int32_t* topk_idx, float* lse, void* workspace, size_t workspace_bytes,
                                      void* stream, void* select_start, void* select_stop, void* attend_start) {
    kmip_status_t s = check_sizes(N, H, d, k);
    if (s != KMIP_OK) return s;
    if ((s = check_value_width(N, H, dv)) != KMIP_OK) return s;
    if ((s = check_scale(scale)) != KMIP_OK) return s;
    if ((s = check_dropout(keep, drop_rate)) != KMIP_OK) return s;
    if (N > 0 && (!V || !out || !lse)) return record_error(KMIP_ERR_INVALID_ARG, "null V, out or lse");
    if (N > 0 && !aligned16(V)) return record_error(KMIP_ERR_INVALID_ARG, "V must be 16-byte aligned");
    s = kmip_topk_with_events(Q, K, graph_offsets, num_graphs, N, H, d, k, topk_idx, workspace,
                              workspace_bytes, stream, select_start, select_stop);
    if (s != KMIP_OK) return s;
    if (N > 0 && attend_start != nullptr) {
        const hipError_t e = hipEventRecord(reinterpret_cast<hipEvent_t>(attend_start),
                                            reinterpret_cast<hipStream_t>(stream));
        if (e != hipSuccess) return hip_fail(e, "event record");
    }
    // one graph grouped by direction: the aggregate takes the queries in
    // that order too (the grouping is still in the workspace)
    const int32_t G = graph_offsets ? num_graphs : 1;
    const int32_t* perm = nullptr;
    if (N > 0 && use_grouping(N, G, H, d, k))
        perm = kmip::group_perm_in(reinterpret_cast<char*>(workspace) + tiled_bytes(N, H, d) + kCounterBytes,
                                   (int32_t)N, H, d);
    return attend_checked(Q, K, V, N, H, d, dv, k, scale, topk_idx, keep, drop_rate, perm, G == 1, out, lse,
                          stream);
}

kmip_status_t kmip_fwd(const void* Q, const void* K, const void* V, const int32_t* graph_offsets,
                       int32_t num_graphs, int64_t N, int32_t H, int32_t d, int32_t k,
                       float scale, float* out, int32_t* topk_idx, float* lse, void* workspace,
                       size_t workspace_bytes, void* stream) {
    return kmip_fwd_ex(Q, K, V, graph_offsets, num_graphs, N, H, d, d, k, scale, nullptr, 0.0f, out, topk_idx,
                       lse, workspace, workspace_bytes, stream);
}

// Backward variant the library picks (KMIP_BWD_AUTO): the bucketed reduction
// where the key rows fit its bucket table, the sizes are its own and the
// value width equals the key width, else the full key sort (for which the
// bucketed reduction may stand in, see wide_buckets).
static int32_t default_bwd_variant(int64_t N, int32_t H, int32_t d, int32_t dv, int32_t k) {
    return dv == d && kmip::bwd_bucket_supported((int32_t)N, H, d, k) ? KMIP_BWD_BUCKETED : KMIP_BWD_SEGMENTED;
}

// Whether KMIP_BWD_AUTO runs the bucketed reduction where it would pick the
// key sort (unequal widths, d = 128, k > 128): its workspace is larger
// (28 against 24 bytes a pair, and the interleaved query rows), and a caller
// whose workspace holds only the key sort's gets that.  Up to 2^20 pairs with
// equal widths, and 2^16 with unequal ones, the key sort and its smaller
// workspace stay (its passes over the index rows cost little there).  Whole
// backward, key sort against buckets (us): 1,500 nodes, 3 heads, d = 32, d_V =
// 64, k = 16 149 and 76; 60,000 nodes of the same 359 and 305; 10,000 nodes, 4
// heads, d = 128, k = 32 404 and 262; 3,000 nodes, 2 heads, d = 32, k = 256
// 1066 and 157; 30,000 nodes, 2 heads, d = 128, k = 100 1512 and 1391.
static bool wide_buckets(int64_t N, int32_t H, int32_t d, int32_t dv, int32_t k) {
    const int64_t pairs = N * (int64_t)H * k;
    return default_bwd_variant(N, H, d, dv, k) == KMIP_BWD_SEGMENTED && pairs > (dv == d ? 1 << 20 : 1 << 16) &&
           kmip::bwd_bucket_rows((int32_t)N, H, d);
}

size_t kmip_bwd_ex_workspace_size(int64_t N, int32_t H, int32_t d, int32_t dv, int32_t k, int32_t variant) {
    if (check_sizes(N, H, d, k) != KMIP_OK || check_value_width(N, H, dv) != KMIP_OK) return 0;
    const int32_t v = variant == KMIP_BWD_AUTO ? default_bwd_variant(N, H, d, dv, k) : variant;
    if (v == KMIP_BWD_KEY_AGGREGATED) return align_up(kmip::bwd_agg_workspace_bytes((int32_t)N, H, d));
    if (variant == KMIP_BWD_AUTO && wide_buckets(N, H, d, dv, k))
        return std::max(align_up(kmip::bwd_bucket_workspace_bytes((int32_t)N, H, d, dv, k)),
                        align_up(kmip::bwd_csr_workspace_bytes((int32_t)N, H, k)));
    if (v == KMIP_BWD_SEGMENTED) return align_up(kmip::bwd_csr_workspace_bytes((int32_t)N, H, k));
    if (v == KMIP_BWD_BUCKETED) return dv == d && kmip::bwd_bucket_supported((int32_t)N, H, d, k)
                                         ? align_up(kmip::bwd_bucket_workspace_bytes((int32_t)N, H, d, dv, k))
                                         : 0;
    return 0;
}

size_t kmip_bwd_workspace_size(int64_t N, int32_t H, int32_t d, int32_t k, int32_t variant) {
    return kmip_bwd_ex_workspace_size(N, H, d, d, k, variant);
}

kmip_status_t kmip_bwd_ex(const void* Q, const void* K, const void* V, const void* dOut,
                          const int32_t* topk_idx, const float* lse, const uint8_t* keep, float drop_rate,
                          int64_t N, int32_t H, int32_t d, int32_t dv, int32_t k, float scale, float* dQ,
                          float* dK, float* dV, int32_t variant, void* workspace, size_t workspace_bytes,
                          void* stream_) {
    kmip_status_t s = check_sizes(N, H, d, k);
    if (s != KMIP_OK) return s;
    if ((s = check_value_width(N, H, dv)) != KMIP_OK) return s;
    if ((s = check_scale(scale)) != KMIP_OK) return s;
    if ((s = check_dropout(keep, drop_rate)) != KMIP_OK) return s;
    const float keep_scale = 1.0f / (1.0f - drop_rate);
    if (variant < KMIP_BWD_AUTO || variant > KMIP_BWD_KEY_AGGREGATED)
        return record_error(KMIP_ERR_UNSUPPORTED, "backward variant %d", variant);
    if (variant == KMIP_BWD_BUCKETED && dv != d)
        return record_error(KMIP_ERR_UNSUPPORTED, "the bucketed variant needs d_V == d_K (got %d, %d)", dv, d);
    if (N == 0) return ok();
    if (!Q || !K || !V || !dOut || !topk_idx || !lse || !dQ || !dK || !dV)
        return record_error(KMIP_ERR_INVALID_ARG, "null buffer passed to kmip_bwd");
    if (!aligned16(Q) || !aligned16(K) || !aligned16(V) || !aligned16(dOut))
        return record_error(KMIP_ERR_INVALID_ARG, "Q, K, V and dOut must be 16-byte aligned");
    if (!aligned16(dK) || !aligned16(dV)) return record_error(KMIP_ERR_INVALID_ARG, "dK and dV must be 16-byte aligned");
    const int32_t v = variant == KMIP_BWD_AUTO ? default_bwd_variant(N, H, d, dv, k) : variant;
    hipStream_t stream = reinterpret_cast<hipStream_t>(stream_);
    hipError_t e;
    if (v != KMIP_BWD_ATOMIC) {
        const size_t need = kmip_bwd_ex_workspace_size(N, H, d, dv, k, v);
        if (workspace == nullptr || workspace_bytes < need)
            return record_error(KMIP_ERR_WORKSPACE, "workspace of %zu bytes < %zu required", workspace_bytes, need);
        if ((reinterpret_cast<uintptr_t>(workspace) & (kAlign - 1)) != 0)
            return record_error(KMIP_ERR_WORKSPACE, "workspace must be 256-byte aligned");
    }
    if (v == KMIP_BWD_KEY_AGGREGATED) {
        e = kmip::launch_bwd_agg(Q, K, V, dOut, topk_idx, lse, keep, keep_scale, (int32_t)N, H, d, dv, k, scale,
                                 dQ, dK, dV, workspace, stream);
    } else if (variant == KMIP_BWD_AUTO && wide_buckets(N, H, d, dv, k) &&
               workspace_bytes >= kmip::bwd_bucket_workspace_bytes((int32_t)N, H, d, dv, k)) {
        e = kmip::launch_bwd_bucket(Q, K, V, dOut, topk_idx, lse, keep, keep_scale, (int32_t)N, H, d, dv, k, scale,
                                    dQ, dK, dV, workspace, stream);
    } else if (v == KMIP_BWD_BUCKETED) {
        if (!kmip::bwd_bucket_supported((int32_t)N, H, d, k))
            return record_error(KMIP_ERR_UNSUPPORTED,
                                "the bucketed variant needs d <= 64, k <= 128 and N*H <= 8192*512 (key-row "
                                "buckets of at most 512 rows)");
        e = kmip::launch_bwd_bucket(Q, K, V, dOut, topk_idx, lse, keep, keep_scale, (int32_t)N, H, d, dv, k, scale,
                                    dQ, dK, dV, workspace, stream);
    } else if (v == KMIP_BWD_SEGMENTED) {
        e = kmip::launch_bwd_csr(Q, K, V, dOut, topk_idx, lse, keep, keep_scale, (int32_t)N, H, d, dv, k, scale,
                                 dQ, dK, dV, workspace, stream);
    } else {
        e = kmip::launch_bwd_atomic(Q, K, V, dOut, topk_idx, lse, keep, keep_scale, (int32_t)N, H, d, dv, k,
                                    scale, dQ, dK, dV, stream);
    }
    if (e != hipSuccess) return hip_fail(e, "backward launch");
    return ok();
}

kmip_status_t kmip_bwd(const void* Q, const void* K, const void* V, const void* dOut,
                       const int32_t* topk_idx, const float* lse, int64_t N, int32_t H,
                       int32_t d, int32_t k, float scale, float* dQ, float* dK, float* dV,
                       int32_t variant, void* workspace, size_t workspace_bytes, void* stream) {
    return kmip_bwd_ex(Q, K, V, dOut, topk_idx, lse, nullptr, 0.0f, N, H, d, d, k, scale, dQ, dK, dV, variant,
                       workspace, workspace_bytes, stream);
}

}  // extern "C"

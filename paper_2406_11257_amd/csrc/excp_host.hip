// Host side of the ExCP library: argument checks, grouping of tensors, workspace, launch order
// (Alg. 1 and Alg. 2), result collection.  No computation of the method happens here.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdio.h>
#include <string.h>

#include <new>
#include <algorithm>
#include <mutex>
#include <vector>

#include "../../include/excp.h"
#include "excp_device.h"

namespace {

constexpr u32 kMaxGroupTensors = 1024;   // tensors processed together (== EXCP_MAX_GROUP_TENSORS of the kernels)
constexpr u32 kMaxBatchTensors = 4096;   // tensors per compress / decompress call
constexpr u64 kAccSegCentres = 3ull * kMaxGroupTensors * 85;   // streams x centres whose accumulators the workspace holds
// GroupParams::alone_work (see the Lloyd iterations in k_kmeans.hip): groups that go together; others, by the number of centres.
constexpr u32 kAloneTogether = 24576, kAloneCells = 98304, kAloneFew = 196608, kAloneMany = 131072;
constexpr u64 kNoLimit = ~0ull;

enum Stage {
    ST_SAMPLE = 0, ST_STATS, ST_SELECT, ST_MASK_COMPACT, ST_MASK_SCAN, ST_MASK_GATHER, ST_LAYOUT, ST_KM_SAMPLE, ST_KM_SCAN,
    ST_KM_SCATTER, ST_KM_BUCKET_STATS, ST_KM_INIT, ST_KM_ITER, ST_ASSIGN_PACK, ST_FINALIZE,
    ST_DECODE_PREP, ST_DECODE_MAIN, ST_EXPORT_DENSE, ST_DECODE_DENSE, ST_MISC, ST_COUNT
};
const char *kStageNames[ST_COUNT] = {
    "median_sample", "stats_stream", "select_candidates", "mask_slots", "mask_scan", "mask_gather", "layout", "km_sample", "km_scan",
    "km_scatter", "km_bucket_stats", "km_init", "km_iter", "assign_pack", "finalize",
    "decode_prep", "decode_main", "export_dense", "decode_dense", "misc"};

struct Span { int stage; hipEvent_t a, b; };
struct Group { u32 first, count, ntiles; };
struct CGroup { u32 first, count, first_desc, ndescs, ntiles, tb_desc, tb_chain; };

constexpr size_t kEventPool = 8192;      // events made by excp_set_profiling: 4096 timed stages per batch

}  // namespace

struct excp_ctx {
    int device = 0;
    hipStream_t stream = nullptr;
    SideStream side{nullptr, nullptr, nullptr};
    u64 max_tensor = 0, max_group = 0, max_tiles = 0;
    Workspace w{};
    // per-batch arrays (device) and their pinned staging (host)
    TState *st_all = nullptr; u32 *cand_ctr_all = nullptr;
    DDesc *ddesc_all = nullptr; DState *dst_all = nullptr;       // (ddesc_all: of the blobs that a compress call decodes itself)
    // descriptors and tile tables of a call, one after the other (see Staged): pinned, and the device's copy
    unsigned char *h_stage = nullptr, *d_stage = nullptr;
    HostRec *h_rec = nullptr;
    u64 ws_bytes = 0;
    std::vector<void *> allocs;
    // pending batch
    int pending = 0;      // 0 none, 1 compress, 2 decompress
    int pending_count = 0;
    bool broken = false;  // a HIP call failed while a batch was being enqueued: the context takes no more work
    // per-call lists; their storage is reserved in excp_create so that no call allocates
    std::vector<Group> groups;
    std::vector<CGroup> cgroups;
    std::vector<u32> tb_offsets, order, big;
    // size thresholds of the kernel forms (excp_set_param)
    u64 wide_elems = 1ull << 28;        // a group with a tensor this large takes the sixteen-wave per-bucket kernels
    u64 cand_list_elems = 1ull << 20;   // one median-candidate list per this many elements of a tensor (1 .. 16 lists)
    // profiling
    bool profiling = false;
    std::vector<Span> spans;
    std::vector<hipEvent_t> free_events;
    double stage_ms[ST_COUNT] = {0};
    int stage_launches[ST_COUNT] = {0};
};

namespace {

// What a call stages lies back to back, so that it is one copy whatever its parts; a call about one tensor whose first
// kernel takes the description as an argument copies nothing.
constexpr size_t kStageBytes = kMaxBatchTensors * (sizeof(DDesc) + sizeof(CDesc) > sizeof(TDesc) ? sizeof(DDesc) + sizeof(CDesc) : sizeof(TDesc)) +
                               (kMaxBatchTensors * 2 + 16) * sizeof(u32) + 64;
template <class T>
struct Staged { T *h, *d; };
struct Staging {
    excp_ctx *c;
    size_t used = 0;
    template <class T>
    Staged<T> take(size_t count) {
        const size_t at = used;
        used = (used + count * sizeof(T) + 15) & ~(size_t)15;
        return {(T *)(c->h_stage + at), (T *)(c->d_stage + at)};
    }
    bool copy() const { return used == 0 || hipMemcpyAsync(c->d_stage, c->h_stage, used, hipMemcpyHostToDevice, c->stream) == hipSuccess; }
};

template <class T>
bool dev_alloc(excp_ctx *c, T **p, u64 count) {
    u64 bytes = count * sizeof(T);
    if (bytes == 0) bytes = 16;
    void *q = nullptr;
    if (hipMalloc(&q, bytes) != hipSuccess) return false;
    c->allocs.push_back(q);
    c->ws_bytes += bytes;
    *p = (T *)q;
    return true;
}

struct StageTimer {
    excp_ctx *c; int stage; hipStream_t on; hipEvent_t a = nullptr, b = nullptr;
    StageTimer(excp_ctx *ctx, int st) : StageTimer(ctx, st, ctx->stream) {}
    StageTimer(excp_ctx *ctx, int st, hipStream_t stream) : c(ctx), stage(st), on(stream) {
        if (!c->profiling) return;
        // events come from the pool excp_set_profiling made; a batch with more stages than the pool
        // holds leaves the rest untimed rather than create events in the middle of a step
        if (c->free_events.size() < 2) return;
        a = c->free_events.back(); c->free_events.pop_back();
        b = c->free_events.back(); c->free_events.pop_back();
        (void)hipEventRecord(a, on);
    }
    ~StageTimer() {
        if (!c->profiling || !a || !b) return;
        (void)hipEventRecord(b, on);
        c->spans.push_back({stage, a, b});
    }
};

// A HIP call failed after part of a batch was enqueued.  The copies already queued read the pinned
// staging arrays, so the stream is drained before anything may overwrite them, and the context takes
// no further work: what state the device tables are in is unknown.
int enqueue_failed(excp_ctx *c) {
    (void)hipStreamSynchronize(c->stream);
    (void)hipStreamSynchronize(c->side.stream);
    (void)hipGetLastError();
    for (auto &sp : c->spans) { c->free_events.push_back(sp.a); c->free_events.push_back(sp.b); }
    c->spans.clear();
    c->pending = 0;
    c->broken = true;
    return EXCP_E_HIP;
}

u64 blob_size_host(u64 n, u64 nw, u64 no, int nbits, u32 flags = 0) {
    u64 s = EXCP_HEADER + excp_books_bytes((u32)nbits);
    s += excp_pad16(8 * excp_words(n));
    s += excp_pad16(8 * excp_words((flags & EXCP_FLAG_NO_W2M) ? n : nw));
    s += excp_pad16(8 * excp_words(nw * (u64)nbits));
    s += 2 * excp_pad16(8 * excp_words(no * (u64)nbits));
    return s;
}

// Split [0, count) into groups: at most kMaxGroupTensors tensors, cap_elems elements, and cap_some of the tensors that
// `some` holds for.
template <class GetN, class Some>
void make_groups(int count, u64 cap_elems, GetN get_n, u64 cap_some, Some some, std::vector<Group> &out) {
    u32 i = 0;
    while (i < (u32)count) {
        Group g{i, 0, 0};
        u64 elems = 0, of_some = 0;
        while (i < (u32)count && g.count < kMaxGroupTensors) {
            u64 n = get_n(i);
            const bool is_some = some(i);
            if (g.count && (elems + n > cap_elems || (is_some && of_some >= cap_some))) break;
            elems += n; of_some += is_some ? 1 : 0;
            g.ntiles += (u32)((n + EXCP_TILE - 1) / EXCP_TILE);
            ++g.count; ++i;
        }
        out.push_back(g);
    }
}

// `w32`, `w16`: the group has tensors of fp32 / of 16-bit weights (blobs of the other kind are refused).
void run_decode_main(excp_ctx *c, const Workspace &w, u32 ntensors, u32 ntiles, bool small, bool moments, bool w32, bool w16) {
    StageTimer t(c, ST_DECODE_MAIN);
    if (small && w32 != w16) { launch_decode_small(w, ntensors, ntiles, moments, w16, c->stream); return; }
    if (w32) launch_decode_main(w, ntensors, ntiles, moments, c->stream);
    if (w16) launch_decode_main16(w, ntensors, ntiles, moments, c->stream);
    launch_decode_raw(w, ntensors, ntiles, moments, c->stream);     // blobs written without quantisation, if any
}

// The most tiles a tensor of [first, first + count) has.
u32 largest_tiles(const DDesc *d, u32 count) {
    u32 largest = 0;
    for (u32 q = 0; q < count; ++q) largest = std::max(largest, d[q].tile_count);
    return largest;
}

// Shared by the two calls that work on the per-element code tensors of Sec. 4.2.  `fill` writes the
// descriptor of tensor i (everything but the tile fields).
template <class Fill>
int run_dense(excp_ctx *c, int count, bool exporting, Fill fill) {
    if (hipSetDevice(c->device) != hipSuccess) return EXCP_E_HIP;
    std::vector<Group> &groups = c->groups;
    std::vector<u32> &tb_offsets = c->tb_offsets;
    groups.clear(); tb_offsets.clear();
    make_groups(count, c->max_group, [&](u32 i) { DDesc d; fill(i, d); return (u64)d.n; }, kNoLimit, [](u32) { return false; }, groups);
    Staging stage{c};
    const Staged<DDesc> descs = stage.take<DDesc>(count);
    const Staged<u32> tiles = stage.take<u32>(count + groups.size());
    u32 tb_off = 0;
    for (const Group &g : groups) {
        u32 tile = 0;
        tb_offsets.push_back(tb_off);
        for (u32 q = 0; q < g.count; ++q) {
            DDesc &d = descs.h[g.first + q];
            fill(g.first + q, d);
            d.tile_begin = tile; d.tile_count = (u32)((d.n + EXCP_TILE - 1) / EXCP_TILE);
            tiles.h[tb_off + q] = tile;
            tile += d.tile_count;
        }
        tiles.h[tb_off + g.count] = tile;
        tb_off += g.count + 1;
    }
    hipStream_t s = c->stream;
    if (count && !stage.copy()) return enqueue_failed(c);
    for (size_t gi = 0; gi < groups.size(); ++gi) {
        const Group &g = groups[gi];
        Workspace w = c->w;
        w.ddesc = descs.d + g.first;
        w.dst = c->dst_all + g.first;
        w.tile_begin = tiles.d + tb_offsets[gi];
        w.rec_dev = c->w.rec_dev + g.first;
        w.rec_base = 0;
        if (exporting) {
            bool moments = false;
            for (u32 q = 0; q < g.count; ++q)
                moments = moments || descs.h[g.first + q].cm != nullptr || descs.h[g.first + q].cv != nullptr;
            {
                StageTimer t(c, ST_DECODE_PREP);
                launch_decode_prep(w, g.count, g.ntiles, largest_tiles(descs.h + g.first, g.count), false, moments, true, nullptr, s);
            }
            { StageTimer t(c, ST_EXPORT_DENSE); launch_export_dense(w, g.count, g.ntiles, s); }
        } else {
            { StageTimer t(c, ST_MISC); launch_dense_parse(w, g.count, s); }
            { StageTimer t(c, ST_DECODE_DENSE); launch_decode_dense(w, g.count, g.ntiles, s); }
            { StageTimer t(c, ST_MISC); launch_decode_finish(w, g.count, s); }      // (codes out of range are found by the pass)
        }
    }
    if (hipGetLastError() != hipSuccess) return enqueue_failed(c);
    c->pending = 2;
    c->pending_count = count;
    return EXCP_OK;
}

// ---- Alg. 2 for one tensor without any allocation -------------------------------------------------
// Everything the decoders keep between their kernels -- the descriptor and state of the tensor, its
// two-entry tile table, the per-tile survivor counts of both bitmaps, the sums of their runs, the
// result record -- lives in one file-scope device array instead of a context's workspace.  Every GPU
// has its own copy of the array at its own address: the address is asked for once per device and kept.
constexpr u64 kStaticMaxTiles = EXCP_STATIC_MAX_ELEMS / EXCP_TILE;
struct StaticOffsets {
    static constexpr u64 ddesc = 0, dst = 256, tile_begin = 512, dec_kinds = 768, rec = 1024, dec_part = 1280,
                         cnt_w = 2048, cnt_o = cnt_w + 4 * (kStaticMaxTiles + 64), end = cnt_o + 4 * (kStaticMaxTiles + 64);
};
static_assert(sizeof(DDesc) <= 256 && sizeof(DState) <= 256 && sizeof(HostRec) <= 256, "scratch slots are 256 bytes");
constexpr u32 kStaticRuns = (StaticOffsets::cnt_w - StaticOffsets::dec_part) / (2 * sizeof(u32));
static_assert(1 + kStaticMaxTiles / EXCP_SCAN_TILES <= kStaticRuns, "the runs of the largest tensor have their sums");
static_assert(StaticOffsets::cnt_w % 256 == 0 && StaticOffsets::cnt_o % 256 == 0, "tables start on 256-byte boundaries");
constexpr u64 kScratchBytes = StaticOffsets::end;

}  // namespace

static __device__ __align__(256) unsigned char scratch[kScratchBytes];

namespace {

constexpr int kMaxDevices = 64;
struct StaticDevice { unsigned char *ptr = nullptr; int cus = 0; bool ready = false; };
StaticDevice g_static[kMaxDevices];
std::mutex g_static_mutex;

// The device's copy of `scratch` and its compute-unit count, looked up on the first call per device
// (with that device current).  The array's name is only a handle on the host; kernels and copies are
// given the address returned here.
int static_device(int device, StaticDevice &out) {
    std::lock_guard<std::mutex> lock(g_static_mutex);
    StaticDevice &d = g_static[device];
    if (!d.ready) {
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return EXCP_E_HIP;
        hipDeviceProp_t prop;
        if (hipGetDeviceProperties(&prop, device) != hipSuccess || prop.multiProcessorCount <= 0) return EXCP_E_HIP;
        d.ptr = (unsigned char *)p; d.cus = prop.multiProcessorCount; d.ready = true;
    }
    out = d;
    return EXCP_OK;
}

}  // namespace

extern "C" {

const char *excp_strerror(int code) {
    switch (code) {
        case EXCP_OK: return "ok";
        case EXCP_E_ARG: return "invalid argument";
        case EXCP_E_CAP: return "blob capacity too small";
        case EXCP_E_NONFINITE: return "non-finite input";
        case EXCP_E_BLOB: return "malformed compressed tensor";
        case EXCP_E_HIP: return "HIP error";
        case EXCP_E_STATE: return "call order violated";
        case EXCP_E_INTERNAL: return "internal work list overflowed";
        default: return "unknown error";
    }
}

uint64_t excp_blob_size(uint64_t n, uint64_t n_w, uint64_t n_o, int nbits) {
    if (((nbits < 2 || nbits > 8) && nbits != (int)EXCP_RAW_BITS) || n_w > n || n_o > n_w) return 0;
    return blob_size_host(n, n_w, n_o, nbits);
}

uint64_t excp_blob_size_ex(uint64_t n, uint64_t n_w, uint64_t n_o, int nbits, uint32_t flags) {
    const bool raw = (flags & EXCP_FLAG_NO_QUANT) != 0, nw2m = (flags & EXCP_FLAG_NO_W2M) != 0;
    if (flags > 63u || (flags & 0x30u) == 0x30u || (raw ? nbits != (int)EXCP_RAW_BITS : (nbits < 2 || nbits > 8))) return 0;
    if (n_w > n || n_o > (nw2m ? n : n_w)) return 0;
    return blob_size_host(n, n_w, n_o, nbits, flags);
}

uint64_t excp_blob_bound(uint64_t n, int nbits) {
    if ((nbits < 2 || nbits > 8) && nbits != (int)EXCP_RAW_BITS) return 0;
    return blob_size_host(n, n, n, nbits);
}

int excp_stage_count(void) { return ST_COUNT; }
const char *excp_stage_name(int i) { return (i >= 0 && i < ST_COUNT) ? kStageNames[i] : ""; }

int excp_create(excp_ctx **out, int hip_device, void *hip_stream, uint64_t max_tensor_elems,
                uint64_t max_group_elems) {
    if (!out) return EXCP_E_ARG;
    *out = nullptr;
    if (max_tensor_elems == 0 || max_tensor_elems > EXCP_MAX_TENSOR_ELEMS) return EXCP_E_ARG;
    if (max_group_elems < max_tensor_elems) return EXCP_E_ARG;
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || hip_device < 0 || hip_device >= ndev) return EXCP_E_HIP;
    if (hipSetDevice(hip_device) != hipSuccess) return EXCP_E_HIP;
    excp_ctx *c = new (std::nothrow) excp_ctx();
    if (!c) return EXCP_E_HIP;
    c->device = hip_device;
    c->stream = (hipStream_t)hip_stream;
    c->max_tensor = max_tensor_elems;
    c->max_group = max_group_elems;
    try {                                     // every list a later call fills is reserved here, at its largest
        c->groups.reserve(kMaxBatchTensors);
        c->cgroups.reserve(kMaxBatchTensors);
        c->tb_offsets.reserve(kMaxBatchTensors);
        c->order.reserve(kMaxBatchTensors);
        c->big.reserve(kMaxBatchTensors);
        c->spans.reserve(kEventPool / 2);
        c->free_events.reserve(kEventPool);
    } catch (...) { delete c; return EXCP_E_HIP; }
    Workspace &w = c->w;
    const u64 G = excp_survivor_elems(max_group_elems, kMaxGroupTensors);
    const u64 max_tiles = G / EXCP_TILE + kMaxGroupTensors + 1;
    const u64 chunks_group = 3 * (G / EXCP_CHUNK) + 3 * kMaxGroupTensors + 3;
    c->max_tiles = max_tiles;
    bool ok = true;
    ok = ok && dev_alloc(c, &c->d_stage, kStageBytes);
    ok = ok && dev_alloc(c, &c->st_all, kMaxBatchTensors);
    ok = ok && dev_alloc(c, &c->cand_ctr_all, (u64)kMaxBatchTensors * 512);
    ok = ok && dev_alloc(c, &c->ddesc_all, kMaxBatchTensors);
    ok = ok && dev_alloc(c, &c->dst_all, kMaxBatchTensors);
    ok = ok && dev_alloc(c, &w.seg, 3ull * kMaxGroupTensors);
    ok = ok && dev_alloc(c, &w.xw, G);
    ok = ok && dev_alloc(c, &w.xm, G);
    ok = ok && dev_alloc(c, &w.xv, G);
    ok = ok && dev_alloc(c, &w.med_hist, (u64)kMaxGroupTensors * 2048);
    ok = ok && dev_alloc(c, &w.sample, (u64)kMaxGroupTensors * 8192);
    ok = ok && dev_alloc(c, &w.sample_mmax, (u64)kMaxGroupTensors * EXCP_SAMPLE_PARTS);
    ok = ok && dev_alloc(c, &w.sel_ticket, kMaxGroupTensors);
    ok = ok && dev_alloc(c, &w.cand, excp_cand_words(G, kMaxGroupTensors));
    ok = ok && dev_alloc(c, &w.tile_status, 2 * max_tiles);      // one word per 2048-element sub-tile
    ok = ok && dev_alloc(c, &w.mask_prefix, 2 * max_tiles);
    ok = ok && dev_alloc(c, &w.mask_part, (u64)kMaxGroupTensors * 16);
    ok = ok && dev_alloc(c, &w.mask_bo, 2 * max_tiles * 32);
    ok = ok && dev_alloc(c, &w.chunk_total, 4);
    ok = ok && dev_alloc(c, &w.seg_chunk_begin, 3ull * kMaxGroupTensors + 4);
    ok = ok && dev_alloc(c, &w.scan_ticket, 1);
    ok = ok && dev_alloc(c, &w.lloyd_shared, 1);
    ok = ok && dev_alloc(c, &w.no_cells, 1);
    ok = ok && dev_alloc(c, &w.seg_unit_begin, 3ull * kMaxGroupTensors + 4);
    const u64 nseg_max = 3ull * kMaxGroupTensors;
    const u64 acc_words = kAccSegCentres * 3 * (EXCP_ABSM_BINS + 1);
    ok = ok && dev_alloc(c, &w.pw, G);
    ok = ok && dev_alloc(c, &w.pm, G);
    ok = ok && dev_alloc(c, &w.pv, G);
    ok = ok && dev_alloc(c, &w.km_split, nseg_max * EXCP_KM_MAP_WORDS);
    ok = ok && dev_alloc(c, &w.km_cnt, excp_count_rows(G, kMaxGroupTensors) * 256);
    ok = ok && dev_alloc(c, &w.km_begin, nseg_max * 257);
    ok = ok && dev_alloc(c, &w.km_bsum, nseg_max * 257 * EXCP_ABSM_BINS);
    ok = ok && dev_alloc(c, &w.km_min, nseg_max * 256);
    ok = ok && dev_alloc(c, &w.km_max, nseg_max * 256);
    ok = ok && dev_alloc(c, &w.km_mag, nseg_max * 256);
    ok = ok && dev_alloc(c, &w.km_dom, nseg_max * 256);
    ok = ok && dev_alloc(c, &w.km_less, nseg_max * 256);
    ok = ok && dev_alloc(c, &w.km_fine, nseg_max * 256);
    w.fine_stride = excp_fine_words(G, kMaxGroupTensors);
    ok = ok && dev_alloc(c, &w.fine_begin, 3 * w.fine_stride);
    ok = ok && dev_alloc(c, &w.fine_above, 3 * w.fine_stride);
    ok = ok && dev_alloc(c, &w.km_acc, acc_words);
    ok = ok && dev_alloc(c, &w.part_obj, chunks_group);
    // per-tile survivor counts of decode; a chain reconstruction keeps those of all its checkpoints
    ok = ok && dev_alloc(c, &w.dec_cnt_w, max_tiles * EXCP_MAX_CHAIN);
    ok = ok && dev_alloc(c, &w.dec_cnt_o, max_tiles * EXCP_MAX_CHAIN);
    ok = ok && dev_alloc(c, &w.dec_kinds, 4);
    w.dec_part_stride = excp_scan_runs(kMaxBatchTensors, (u32)std::min<u64>(max_tiles * EXCP_MAX_CHAIN, 0xffffffffull - EXCP_SCAN_TILES));
    ok = ok && dev_alloc(c, &w.dec_part, 2ull * w.dec_part_stride);
    if (ok) {
        // (the kernels write the results where the host reads them: no copy back)
        ok = hipHostMalloc((void **)&c->h_stage, kStageBytes) == hipSuccess &&
             hipHostMalloc((void **)&c->h_rec, sizeof(HostRec) * kMaxBatchTensors) == hipSuccess &&
             hipHostGetDevicePointer((void **)&w.rec_dev, c->h_rec, 0) == hipSuccess;
    }
    if (ok) {
        hipDeviceProp_t prop;
        ok = hipGetDeviceProperties(&prop, hip_device) == hipSuccess && prop.multiProcessorCount > 0;
        w.cus = ok ? prop.multiProcessorCount : 0;
    }
    ok = ok && hipStreamCreateWithFlags(&c->side.stream, hipStreamNonBlocking) == hipSuccess &&
         hipEventCreateWithFlags(&c->side.fork, hipEventDisableTiming) == hipSuccess &&
         hipEventCreateWithFlags(&c->side.join, hipEventDisableTiming) == hipSuccess;
    ok = ok && dev_alloc(c, &w.stat_part, 2ull * excp_grid(w, EXCP_STATS_PER_CU));
    if (ok) {
        launch_zero_u32(w.med_hist, (u64)kMaxGroupTensors * 2048, c->stream);
        launch_zero_u32(w.sel_ticket, kMaxGroupTensors, c->stream);
        launch_zero_u32(w.scan_ticket, 1, c->stream);
        launch_zero_u32(w.dec_kinds, 4, c->stream);
        ok = hipStreamSynchronize(c->stream) == hipSuccess;
    }
    if (!ok) { excp_destroy(c); return EXCP_E_HIP; }
    *out = c;
    return EXCP_OK;
}

void excp_destroy(excp_ctx *c) {
    if (!c) return;
    (void)hipSetDevice(c->device);
    (void)hipStreamSynchronize(c->stream);
    if (c->side.stream) { (void)hipStreamSynchronize(c->side.stream); (void)hipStreamDestroy(c->side.stream); }
    if (c->side.fork) (void)hipEventDestroy(c->side.fork);
    if (c->side.join) (void)hipEventDestroy(c->side.join);
    for (void *p : c->allocs) (void)hipFree(p);
    if (c->h_stage) (void)hipHostFree(c->h_stage);
    if (c->h_rec) (void)hipHostFree(c->h_rec);
    for (auto &s : c->spans) { (void)hipEventDestroy(s.a); (void)hipEventDestroy(s.b); }
    for (auto e : c->free_events) (void)hipEventDestroy(e);
    delete c;
}

uint64_t excp_workspace_bytes(const excp_ctx *c) { return c ? c->ws_bytes : 0; }

int excp_copy_probe(excp_ctx *c, void *dst, const void *src, uint64_t nbytes) {
    if (!c || !dst || !src || (nbytes & 15u) || (((uintptr_t)dst | (uintptr_t)src) & 15u)) return EXCP_E_ARG;
    if (hipSetDevice(c->device) != hipSuccess) return EXCP_E_HIP;
    launch_copy_probe(src, dst, nbytes, c->stream);
    return hipGetLastError() == hipSuccess ? EXCP_OK : EXCP_E_HIP;
}

int excp_set_profiling(excp_ctx *c, int enabled) {
    if (!c) return EXCP_E_ARG;
    if (c->pending) return EXCP_E_STATE;
    if (c->broken) return EXCP_E_HIP;
    if (enabled && c->free_events.empty()) {
        // the event pool is made here, once, so that no timed step creates events
        if (hipSetDevice(c->device) != hipSuccess) return EXCP_E_HIP;
        for (size_t i = 0; i < kEventPool; ++i) {
            hipEvent_t e = nullptr;
            if (hipEventCreate(&e) != hipSuccess) return EXCP_E_HIP;
            c->free_events.push_back(e);
        }
    }
    c->profiling = enabled != 0;
    return EXCP_OK;
}

int excp_set_param(excp_ctx *c, int param, uint64_t value) {
    if (!c || value == 0) return EXCP_E_ARG;
    if (c->pending) return EXCP_E_STATE;
    switch (param) {
        case EXCP_PARAM_WIDE_ELEMS: c->wide_elems = value; return EXCP_OK;
        case EXCP_PARAM_CAND_LIST_ELEMS: c->cand_list_elems = value; return EXCP_OK;
        default: return EXCP_E_ARG;
    }
}

int excp_stage_ms(excp_ctx *c, int i, double *ms, int *launches) {
    if (!c || i < 0 || i >= ST_COUNT) return EXCP_E_ARG;
    if (ms) *ms = c->stage_ms[i];
    if (launches) *launches = c->stage_launches[i];
    return EXCP_OK;
}

int excp_compress_tensors(excp_ctx *c, int count, const excp_tensor *tensors, float alpha, float beta,
                          int nbits, int lloyd_iters, uint32_t flags) {
    if (!c || count < 0 || (count && !tensors)) return EXCP_E_ARG;
    if (c->pending) return EXCP_E_STATE;
    if (c->broken) return EXCP_E_HIP;
    if ((u32)count > kMaxBatchTensors) return EXCP_E_ARG;
    if (nbits < 2 || nbits > 8 || lloyd_iters < 0 || (flags & ~63u) != 0 || (flags & 0x30u) == 0x30u) return EXCP_E_ARG;
    if (!(alpha >= 0.f) || !(beta >= 0.f) || isinf(alpha) || isinf(beta)) return EXCP_E_ARG;
    const bool raw = (flags & EXCP_FLAG_NO_QUANT) != 0;     // survivors stored as fp32: no codebook stage at all
    if (raw) nbits = (int)EXCP_RAW_BITS;
    const int K = raw ? 0 : (1 << nbits) - 1;
    for (int i = 0; i < count; ++i) {
        const excp_tensor &t = tensors[i];
        if (t.n > c->max_tensor) return EXCP_E_ARG;
        if (!t.blob || ((uintptr_t)t.blob & 15u)) return EXCP_E_ARG;
        if (t.n && (!t.W_prev_recon || !t.W_t || !t.m_t || !t.v_t)) return EXCP_E_ARG;
        // the part of the blob whose place does not depend on the data must fit
        if (t.blob_cap < EXCP_HEADER + excp_books_bytes((u32)nbits) + excp_pad16(8 * excp_words(t.n))) return EXCP_E_CAP;
    }
    if (hipSetDevice(c->device) != hipSuccess) return EXCP_E_HIP;
    const u64 cap_elems = c->max_group;
    // (the accumulators of the Lloyd iterations hold 3 x 1024 streams of up to 85 centres -- six-bit codes and fewer --
    // or 341 tensors of 255; small tensors have none)
    const u64 acc_slots = kAccSegCentres / (3ull * (u64)std::max(K, 1));
    auto small = [&](u32 i) { return raw || excp_lloyd_small(tensors[i].n, (u32)K); };
    std::vector<Group> &groups = c->groups;
    std::vector<u32> &tb_offsets = c->tb_offsets;
    groups.clear(); tb_offsets.clear();
    make_groups(count, cap_elems, [&](u32 i) { return (u64)tensors[i].n; }, acc_slots, [&](u32 i) { return !small(i); }, groups);

    // Groups with larger tensors beside no more streams than compute units take all of them the same way through the
    // Lloyd iterations (see k_kmeans.hip).
    auto lloyd_together = [&](const Group &g, u32 count) {
        bool any = false;
        for (u32 q = 0; q < g.count; ++q) any = any || !small(g.first + q);
        return any && 3u * count <= (u32)c->w.cus;
    };
    // In a group the tensors that a workgroup holds (k_small.hip) come last; the general kernels see only those before.  (The
    // ablations of the median, of quantisation and of the momentum check take the general kernels in any case.)
    const bool usual = (flags & ~(EXCP_FLAG_NO_M2W | 0x30u)) == 0;
    std::vector<u32> &order = c->order, &big = c->big;
    order.clear(); big.clear();
    for (Group &g : groups) {
        for (u32 q = 0; q < g.count; ++q) if (!usual || tensors[g.first + q].n > EXCP_SMALL_ELEMS) order.push_back(g.first + q);
        big.push_back((u32)order.size() - g.first);
        if (usual) for (u32 q = 0; q < g.count; ++q) if (tensors[g.first + q].n <= EXCP_SMALL_ELEMS) order.push_back(g.first + q);
    }
    Staging stage{c};
    const Staged<TDesc> descs = stage.take<TDesc>(count);
    const Staged<u32> tiles = stage.take<u32>(count + groups.size());
    u32 tb_off = 0;
    for (size_t gi = 0; gi < groups.size(); ++gi) {
        Group &g = groups[gi];
        const u32 nbig = big[gi];
        u64 elem_off = 0, cand_off = 0; u32 tile = 0, slot = 0;
        tb_offsets.push_back(tb_off);
        const bool together = lloyd_together(g, nbig);
        for (u32 q = 0; q < g.count; ++q) {
            const u32 i = order[g.first + q];
            const excp_tensor &t = tensors[i];
            TDesc &d = descs.h[g.first + q];
            d.Wp = (const float *)t.W_prev_recon; d.W = (const float *)t.W_t; d.m = t.m_t; d.v = t.v_t; d.n = t.n;
            d.blob = (unsigned char *)t.blob; d.blob_cap = t.blob_cap; d.W_out = (float *)t.W_recon_out;
            d.elem_off = elem_off; d.tile_begin = tile;
            d.cand_lists = excp_cand_lists(t.n, c->cand_list_elems);
            d.cand_off = cand_off; d.cand_cap = excp_cand_cap(t.n, d.cand_lists);
            cand_off += d.cand_cap;
            d.tile_count = (u32)((t.n + EXCP_TILE - 1) / EXCP_TILE);
            d.acc_slot = q < nbig && t.n && (together || !small(i)) ? slot++ : EXCP_NO_SLOT; d.rec = i - g.first;
            elem_off += excp_area_elems(t.n);
            if (q >= nbig) continue;
            tiles.h[tb_off + q] = tile;
            tile += d.tile_count;
        }
        g.ntiles = tile;
        // the tensors by size, powers of two apart, the largest first
        u32 at[65] = {0};
        auto size_class = [&](u32 q) { const u64 n = descs.h[g.first + q].n; return n ? (u32)__builtin_clzll(n) : 64u; };
        for (u32 q = 0; q < nbig; ++q) ++at[size_class(q)];
        for (u32 k = 0, sum = 0; k < 65; ++k) { const u32 here = at[k]; at[k] = sum; sum += here; }
        for (u32 q = 0; q < nbig; ++q) descs.h[g.first + at[size_class(q)]++].turn = q;
        tiles.h[tb_off + nbig] = tile;
        tb_off += nbig + 1;
    }
    hipStream_t s = c->stream;
    const bool single = count == 1;
    if (!single && !stage.copy()) return enqueue_failed(c);
    for (size_t gi = 0; gi < groups.size(); ++gi) {
        const Group &g = groups[gi];
        Workspace w = c->w;
        w.desc = descs.d + g.first;
        w.st = c->st_all + g.first;
        w.cand_ctr = c->cand_ctr_all + (u64)g.first * 512;
        w.ddesc = c->ddesc_all + g.first;
        w.dst = c->dst_all + g.first;
        w.tile_begin = tiles.d + tb_offsets[gi];
        w.rec_base = 0;
        w.rec_dev = c->w.rec_dev + g.first;
        GroupParams p{};
        p.alpha = alpha; p.beta = beta; p.nbits = nbits; p.K = K; p.iters = lloyd_iters; p.flags = flags;
        const u32 nbig = big[gi];
        p.ntensors = nbig; p.ntiles = g.ntiles;
        u64 largest = 0, elems = 0;
        bool any_out = false;
        for (u32 q = 0; q < nbig; ++q) {
            const TDesc &d = descs.h[g.first + q];
            largest = std::max(largest, d.n); elems += d.n; any_out = any_out || d.W_out != nullptr;
        }
        const bool w16 = (flags & 0x30u) != 0;
        if (!raw) {
            p.together = lloyd_together(g, nbig) ? 1u : 0u;
            const u32 whole = (alpha == 0.f ? 1u : 0u) + (beta == 0.f && (alpha == 0.f || (flags & EXCP_FLAG_NO_W2M)) ? 2u : 0u);
            const bool cells = p.together && !w16 && excp_cells_group(elems, largest, nbig, (u32)K, whole);
            for (u32 q = 0; q < nbig; ++q) p.fine += cells && excp_fine_tensor(descs.h[g.first + q].n) ? 1u : 0u;
            p.alone_work = p.fine ? kAloneCells : (p.together ? kAloneTogether : (K < 63 ? kAloneFew : kAloneMany));
            for (u32 q = 0; q < nbig; ++q) p.slots += descs.h[g.first + q].acc_slot != EXCP_NO_SLOT ? 1u : 0u;
        }
        p.unit_shift = excp_unit_shift(elems, nbig, excp_gather_subs(g.ntiles, (u32)w.cus), (u32)w.cus, excp_count_rows(c->max_group, kMaxGroupTensors));
        p.fine_size = excp_fine_size(largest); p.fine_chunks = excp_cells_chunks(elems); p.largest = largest;
        p.samples = excp_samples(p.fine != 0u, largest);
        p.wide = largest >= c->wide_elems ? 2u : ((flags & 0x30u) != 0 ? 1u : 0u);
        { StageTimer t(c, ST_LAYOUT); }                      // (made inside the mask scan and the kernels for small tensors: the span, one a group, is empty)
        // The small tensors: one launch or two (excp_small_once), beside the larger ones on the context's own stream.  (They depend on nothing but what was
        // enqueued before this group; the 14M shape has 50 of them among 76: 535 -> 526 us; the 410M shape 194 among 292: 5337 -> 5027.
        // They are enqueued when the larger ones have something to do for a while: calls of the runtime take time too.)
        const u32 nsmall = g.count - nbig;
        if (nsmall && nbig) (void)hipEventRecord(c->side.fork, s);
        auto launch_small = [&]() {
            if (!nsmall) return;
            Workspace ws = w;
            GroupParams ps = p;
            ws.desc = w.desc + nbig; ws.st = w.st + nbig;
            ps.ntensors = nsmall;
            const hipStream_t to = nbig ? c->side.stream : s;
            if (nbig) (void)hipStreamWaitEvent(c->side.stream, c->side.fork, 0);
            StageTimer t(c, ST_MISC, to);
            ::launch_small(ws, ps, single ? descs.h : nullptr, excp_small_once(descs.h + g.first + nbig, nsmall, (u32)w.cus, w16 ? 2u : 4u), to);
        };
        if (!nbig) { launch_small(); continue; }
        { StageTimer t(c, ST_SAMPLE); launch_stats(w, p, 0, single ? descs.h : nullptr, s); }
        { StageTimer t(c, ST_STATS); launch_stats(w, p, 1, nullptr, s); }
        { StageTimer t(c, ST_SELECT); launch_stats(w, p, 2, nullptr, s); }
        { StageTimer t(c, ST_MASK_COMPACT); launch_mask_compact(w, p, 0, s); }
        launch_small();
        { StageTimer t(c, ST_MASK_SCAN); launch_mask_compact(w, p, 1, s); }
        // the value -> bucket maps come from the slots, before the pass that makes the dense survivor arrays:
        // that pass also takes the bucket counts
        if (!raw) { StageTimer t(c, ST_KM_SAMPLE); launch_km_partition(w, p, 0, s); }
        { StageTimer t(c, ST_MASK_GATHER); launch_mask_compact(w, p, 2, s); }
        if (raw) {
            StageTimer t(c, ST_ASSIGN_PACK); launch_store_raw(w, p, s); launch_bitmap_o(w, p, s);
        } else {
            { StageTimer t(c, ST_KM_SCAN); launch_km_partition(w, p, 1, s); }
            { StageTimer t(c, ST_KM_SCATTER); launch_km_partition(w, p, 2, s); }
            { StageTimer t(c, ST_KM_BUCKET_STATS); launch_km_partition(w, p, 3, s); launch_km_cells(w, p, s); }
            { StageTimer t(c, ST_KM_INIT); launch_km_init(w, p, s); }
            { StageTimer t(c, ST_KM_ITER); launch_km_iter(w, p, s, c->side); }
            { StageTimer t(c, ST_ASSIGN_PACK); launch_assign_pack(w, p, s); }
        }
        { StageTimer t(c, ST_FINALIZE); launch_finalize(w, p, any_out, s); }
        if (any_out) {
            StageTimer t(c, ST_DECODE_MAIN);
            if (raw) launch_decode_raw(w, nbig, g.ntiles, false, s);
            else if (flags & 0x30u) launch_decode_main16(w, nbig, g.ntiles, false, s);
            else launch_decode_main(w, nbig, g.ntiles, false, s);
        }
        if (nsmall && !p.slots) {                            // (else the stream was joined by the Lloyd iterations)
            (void)hipEventRecord(c->side.join, c->side.stream);
            (void)hipStreamWaitEvent(s, c->side.join, 0);
        }
    }
    if (hipGetLastError() != hipSuccess) return enqueue_failed(c);
    c->pending = 1;
    c->pending_count = count;
    return EXCP_OK;
}

int excp_decompress_tensors(excp_ctx *c, int count, const excp_blob *blobs) {
    if (!c || count < 0 || (count && !blobs)) return EXCP_E_ARG;
    if (c->pending) return EXCP_E_STATE;
    if (c->broken) return EXCP_E_HIP;
    if ((u32)count > kMaxBatchTensors) return EXCP_E_ARG;
    for (int i = 0; i < count; ++i) {
        const excp_blob &b = blobs[i];
        if ((b.flags & ~0x30u) || (b.flags & 0x30u) == 0x30u) return EXCP_E_ARG;
        if (b.n > c->max_tensor) return EXCP_E_ARG;
        if (!b.blob || ((uintptr_t)b.blob & 15u)) return EXCP_E_ARG;
        if (b.n && !b.W_prev_recon) return EXCP_E_ARG;
    }
    if (hipSetDevice(c->device) != hipSuccess) return EXCP_E_HIP;
    std::vector<Group> &groups = c->groups;
    std::vector<u32> &tb_offsets = c->tb_offsets;
    groups.clear(); tb_offsets.clear();
    make_groups(count, c->max_group, [&](u32 i) { return (u64)blobs[i].n; }, kNoLimit, [](u32) { return false; }, groups);
    Staging stage{c};
    const Staged<DDesc> descs = stage.take<DDesc>(count);
    const Staged<u32> tiles = stage.take<u32>(count + groups.size());
    u32 tb_off = 0;
    for (const Group &g : groups) {
        u32 tile = 0;
        tb_offsets.push_back(tb_off);
        for (u32 q = 0; q < g.count; ++q) {
            const excp_blob &b = blobs[g.first + q];
            DDesc &d = descs.h[g.first + q];
            d.Wp = (const float *)b.W_prev_recon; d.blob = (const unsigned char *)b.blob; d.blob_bytes = b.blob_bytes; d.n = b.n;
            d.W_out = (float *)b.W_recon_out; d.m_out = b.m_out; d.v_out = b.v_out;
            d.cw = d.cm = d.cv = d.head = nullptr; d.wtype = (b.flags >> 4) & 3u; d.pad = 0;
            d.tile_begin = tile; d.tile_count = (u32)((b.n + EXCP_TILE - 1) / EXCP_TILE);
            tiles.h[tb_off + q] = tile;
            tile += d.tile_count;
        }
        tiles.h[tb_off + g.count] = tile;
        tb_off += g.count + 1;
    }
    hipStream_t s = c->stream;
    const bool single = count == 1;
    if (!single && !stage.copy()) return enqueue_failed(c);
    for (size_t gi = 0; gi < groups.size(); ++gi) {
        const Group &g = groups[gi];
        Workspace w = c->w;
        w.ddesc = descs.d + g.first;
        w.dst = c->dst_all + g.first;
        w.tile_begin = tiles.d + tb_offsets[gi];
        w.rec_dev = c->w.rec_dev + g.first;
        w.rec_base = 0;
        bool moments = false, w32 = false, w16 = false;
        for (u32 q = 0; q < g.count; ++q) {
            const excp_blob &b = blobs[g.first + q];
            moments = moments || b.m_out != nullptr || b.v_out != nullptr;
            if (b.flags & 0x30u) w16 = true; else w32 = true;
        }
        const u32 largest = largest_tiles(descs.h + g.first, g.count);
        {
            StageTimer t(c, ST_DECODE_PREP);
            launch_decode_prep(w, g.count, g.ntiles, largest, true, moments, true, single ? descs.h : nullptr, s);
        }
        run_decode_main(c, w, g.count, g.ntiles, excp_prep_small(largest), moments, w32, w16);
    }
    if (hipGetLastError() != hipSuccess) return enqueue_failed(c);
    c->pending = 2;
    c->pending_count = count;
    return EXCP_OK;
}

uint64_t excp_dense_bytes(uint64_t n, int nbits) { return nbits <= 4 ? (n + 1) / 2 : n; }
uint64_t excp_head_bytes(int nbits) { return (nbits < 2 || nbits > 8) ? 0 : EXCP_HEADER + 12ull * (1ull << nbits); }

int excp_export_dense(excp_ctx *c, int count, const excp_dense_export *items) {
    if (!c || count < 0 || (count && !items)) return EXCP_E_ARG;
    if (c->pending) return EXCP_E_STATE;
    if (c->broken) return EXCP_E_HIP;
    if ((u32)count > kMaxBatchTensors) return EXCP_E_ARG;
    for (int i = 0; i < count; ++i) {
        const excp_dense_export &e = items[i];
        if (e.n > c->max_tensor) return EXCP_E_ARG;
        if (!e.blob || ((uintptr_t)e.blob & 15u)) return EXCP_E_ARG;
        if (((uintptr_t)e.head | (uintptr_t)e.codes_w | (uintptr_t)e.codes_m | (uintptr_t)e.codes_v) & 15u) return EXCP_E_ARG;
    }
    return run_dense(c, count, true, [&](u32 i, DDesc &d) {
        const excp_dense_export &e = items[i];
        d.Wp = nullptr; d.blob = (const unsigned char *)e.blob; d.blob_bytes = e.blob_bytes; d.n = e.n;
        d.W_out = d.m_out = d.v_out = nullptr;
        d.cw = e.codes_w; d.cm = e.codes_m; d.cv = e.codes_v; d.head = (unsigned char *)e.head;
        d.wtype = 3u; d.pad = 0;
    });
}

int excp_decompress_dense(excp_ctx *c, int count, const excp_dense_blob *items) {
    if (!c || count < 0 || (count && !items)) return EXCP_E_ARG;
    if (c->pending) return EXCP_E_STATE;
    if (c->broken) return EXCP_E_HIP;
    if ((u32)count > kMaxBatchTensors) return EXCP_E_ARG;
    for (int i = 0; i < count; ++i) {
        const excp_dense_blob &e = items[i];
        if ((e.flags & ~0x30u) || (e.flags & 0x30u) == 0x30u) return EXCP_E_ARG;
        if (e.n > c->max_tensor) return EXCP_E_ARG;
        if (!e.head || ((uintptr_t)e.head & 15u)) return EXCP_E_ARG;
        if (((uintptr_t)e.codes_w | (uintptr_t)e.codes_m | (uintptr_t)e.codes_v) & 15u) return EXCP_E_ARG;
        if (e.n && e.W_recon_out && (!e.W_prev_recon || !e.codes_w)) return EXCP_E_ARG;
        if (e.n && ((e.m_out && !e.codes_m) || (e.v_out && !e.codes_v))) return EXCP_E_ARG;
    }
    return run_dense(c, count, false, [&](u32 i, DDesc &d) {
        const excp_dense_blob &e = items[i];
        d.Wp = (const float *)e.W_prev_recon; d.blob = (const unsigned char *)e.head; d.blob_bytes = e.head_bytes; d.n = e.n;
        d.W_out = (float *)e.W_recon_out; d.m_out = e.m_out; d.v_out = e.v_out;
        d.cw = (unsigned char *)e.codes_w; d.cm = (unsigned char *)e.codes_m; d.cv = (unsigned char *)e.codes_v; d.head = nullptr;
        d.wtype = (e.flags >> 4) & 3u; d.pad = 0;
    });
}

int excp_reconstruct_chain(excp_ctx *c, int count, const excp_chain *chains) {
    if (!c || count < 0 || (count && !chains)) return EXCP_E_ARG;
    if (c->pending) return EXCP_E_STATE;
    if (c->broken) return EXCP_E_HIP;
    if ((u32)count > kMaxBatchTensors) return EXCP_E_ARG;
    u64 total_descs = 0;
    for (int i = 0; i < count; ++i) {
        const excp_chain &ch = chains[i];
        if ((ch.flags & ~0x30u) || (ch.flags & 0x30u) == 0x30u) return EXCP_E_ARG;
        if (ch.n > c->max_tensor || ch.steps < 1 || ch.steps > EXCP_MAX_CHAIN) return EXCP_E_ARG;
        if (!ch.blobs || !ch.blob_bytes) return EXCP_E_ARG;
        if (ch.n && !ch.W0) return EXCP_E_ARG;
        for (int j = 0; j < ch.steps; ++j)
            if (!ch.blobs[j] || ((uintptr_t)ch.blobs[j] & 15u)) return EXCP_E_ARG;
        total_descs += (u64)ch.steps;
    }
    if (total_descs > kMaxBatchTensors) return EXCP_E_ARG;
    if (hipSetDevice(c->device) != hipSuccess) return EXCP_E_HIP;

    // Groups: at most kMaxGroupTensors tensors and as many
    // descriptor tiles (a descriptor per tensor and checkpoint) as the per-tile count tables hold (EXCP_MAX_CHAIN times a group's tiles, so
    // any tensor the context accepts fits with its whole chain).
    std::vector<CGroup> &groups = c->cgroups;
    groups.clear();
    Staging stage{c};
    const Staged<DDesc> descs = stage.take<DDesc>(total_descs);
    const Staged<CDesc> cdescs = stage.take<CDesc>(count);
    const Staged<u32> tiles = stage.take<u32>(kMaxBatchTensors * 2 + 16);
    u32 tb_off = 0, desc_off = 0;
    for (u32 i = 0; i < (u32)count;) {
        CGroup g{i, 0, desc_off, 0, 0, 0, 0};
        u64 dtiles = 0;
        while (i < (u32)count) {
            const excp_chain &ch = chains[i];
            const u64 tiles = (ch.n + EXCP_TILE - 1) / EXCP_TILE;
            if (g.count && (g.count == kMaxGroupTensors || dtiles + tiles * ch.steps > c->max_tiles * EXCP_MAX_CHAIN)) break;
            dtiles += tiles * ch.steps; g.ndescs += (u32)ch.steps; g.ntiles += (u32)tiles; ++g.count; ++i;
        }
        if (tb_off + g.ndescs + g.count + 2 > kMaxBatchTensors * 2 + 16) return EXCP_E_ARG;
        g.tb_desc = tb_off; g.tb_chain = tb_off + g.ndescs + 1;
        u32 dtile = 0, ctile = 0, d = 0;
        for (u32 q = 0; q < g.count; ++q) {
            const excp_chain &ch = chains[g.first + q];
            const u32 ntiles = (u32)((ch.n + EXCP_TILE - 1) / EXCP_TILE);
            CDesc &cd = cdescs.h[g.first + q];
            cd.W0 = (const float *)ch.W0; cd.W_out = (float *)ch.W_out; cd.n = ch.n; cd.first_desc = d; cd.steps = (u32)ch.steps;
            cd.tile_begin = ctile; cd.tile_count = ntiles;
            tiles.h[g.tb_chain + q] = ctile;
            ctile += ntiles;
            for (int j = 0; j < ch.steps; ++j, ++d) {
                DDesc &dd = descs.h[desc_off + d];
                const bool last = j + 1 == ch.steps;
                dd.Wp = nullptr; dd.blob = (const unsigned char *)ch.blobs[j]; dd.blob_bytes = ch.blob_bytes[j]; dd.n = ch.n;
                dd.W_out = nullptr; dd.m_out = last ? ch.m_out : nullptr; dd.v_out = last ? ch.v_out : nullptr;
                dd.cw = dd.cm = dd.cv = dd.head = nullptr; dd.wtype = (ch.flags >> 4) & 3u; dd.pad = 0;
                dd.tile_begin = dtile; dd.tile_count = ntiles;
                tiles.h[g.tb_desc + d] = dtile;
                dtile += ntiles;
            }
        }
        tiles.h[g.tb_desc + g.ndescs] = dtile;
        tiles.h[g.tb_chain + g.count] = ctile;
        tb_off += g.ndescs + g.count + 2;
        desc_off += g.ndescs;
        groups.push_back(g);
    }
    hipStream_t s = c->stream;
    stage.used = (size_t)((unsigned char *)(tiles.h + tb_off) - c->h_stage);
    if (count && !stage.copy()) return enqueue_failed(c);
    for (const CGroup &g : groups) {
        Workspace w = c->w;
        w.ddesc = descs.d + g.first_desc;
        w.dst = c->dst_all + g.first_desc;
        w.tile_begin = tiles.d + g.tb_desc;
        w.cdesc = cdescs.d + g.first;
        w.chain_tile_begin = tiles.d + g.tb_chain;
        w.rec_dev = c->w.rec_dev + g.first;
        w.rec_base = 0;
        const u32 dtiles = tiles.h[g.tb_desc + g.ndescs];
        bool moments = false;
        for (u32 q = 0; q < g.count; ++q)
            moments = moments || chains[g.first + q].m_out != nullptr || chains[g.first + q].v_out != nullptr;
        {
            StageTimer t(c, ST_DECODE_PREP);
            launch_decode_prep(w, g.ndescs, dtiles, largest_tiles(descs.h + g.first_desc, g.ndescs), false, moments, false, nullptr, s);
        }
        bool w16[2] = {false, false};                      // weight storage met in the group (a blob that says otherwise is refused)
        for (u32 q = 0; q < g.count; ++q) w16[(chains[g.first + q].flags & 0x30u) != 0] = true;
        for (int k = 0; k < 2; ++k)
            if (w16[k]) { StageTimer t(c, ST_DECODE_MAIN); launch_decode_chain(w, g.count, g.ntiles, k == 1, s); }
        if (moments) {      // the last checkpoints' moments
            StageTimer t(c, ST_DECODE_MAIN);
            Workspace wl = w;
            wl.tile_begin = w.chain_tile_begin;
            if (w16[0]) launch_decode_main(wl, g.count, g.ntiles, true, s);
            if (w16[1]) launch_decode_main16(wl, g.count, g.ntiles, true, s);
        }
        { StageTimer t(c, ST_MISC); launch_chain_finish(w, g.count, s); }
    }
    if (hipGetLastError() != hipSuccess) return enqueue_failed(c);
    c->pending = 2;
    c->pending_count = count;
    return EXCP_OK;
}

int excp_collect(excp_ctx *c, excp_stats *stats) {
    if (!c) return EXCP_E_ARG;
    if (!c->pending) return EXCP_E_STATE;
    if (hipSetDevice(c->device) != hipSuccess) return EXCP_E_HIP;
    hipError_t e = hipStreamSynchronize(c->stream);
    c->pending = 0;
    for (int i = 0; i < ST_COUNT; ++i) { c->stage_ms[i] = 0; c->stage_launches[i] = 0; }
    for (auto &sp : c->spans) {
        float ms = 0.f;
        if (e == hipSuccess && hipEventElapsedTime(&ms, sp.a, sp.b) == hipSuccess) {
            c->stage_ms[sp.stage] += ms;
            c->stage_launches[sp.stage] += 1;
        }
        c->free_events.push_back(sp.a);
        c->free_events.push_back(sp.b);
    }
    c->spans.clear();
    if (e != hipSuccess) return EXCP_E_HIP;
    int first = EXCP_OK;
    for (int i = 0; i < c->pending_count; ++i) {
        const HostRec &r = c->h_rec[i];
        if (stats) {
            excp_stats &o = stats[i];
            memset(&o, 0, sizeof(o));
            o.n = r.n; o.n_w = r.n_w; o.n_o = r.n_o; o.blob_bytes = r.blob_bytes; o.nonfinite = r.nonfinite;
            o.abs_sum_m = r.abs_sum; o.obj_w = r.obj[0]; o.obj_m = r.obj[1]; o.obj_v = r.obj[2];
            o.median_abs_dw = r.med; o.mean_abs_m = r.mean32; o.t_w = r.t_w; o.r_o = r.r_o;
            o.status = r.status;
        }
        if (first == EXCP_OK && r.status != 0) first = r.status;
    }
    return first;
}

int excp_compress_step(excp_ctx *c, const void *W_prev_recon, const void *W_t, const float *m_t,
                       const float *v_t, uint64_t n, float alpha, float beta, int nbits, int lloyd_iters,
                       uint32_t flags, void *blob_out, uint64_t blob_cap, uint64_t *blob_bytes,
                       void *W_recon_out, excp_stats *stats) {
    excp_tensor t{W_prev_recon, W_t, m_t, v_t, n, blob_out, blob_cap, W_recon_out};
    int rc = excp_compress_tensors(c, 1, &t, alpha, beta, nbits, lloyd_iters, flags);
    if (rc != EXCP_OK) return rc;
    excp_stats st;
    memset(&st, 0, sizeof(st));
    rc = excp_collect(c, &st);
    if (rc == EXCP_E_HIP || rc == EXCP_E_STATE) return rc;      // nothing was collected: the outputs stay untouched
    if (blob_bytes) *blob_bytes = st.blob_bytes;
    if (stats) *stats = st;
    return rc;
}

int excp_decompress_step(excp_ctx *c, const void *W_prev_recon, const void *blob, uint64_t blob_bytes,
                         uint64_t n, void *W_recon_out, float *m_out, float *v_out, uint32_t flags) {
    excp_blob b{W_prev_recon, blob, blob_bytes, n, W_recon_out, m_out, v_out, flags, 0};
    int rc = excp_decompress_tensors(c, 1, &b);
    if (rc != EXCP_OK) return rc;
    return excp_collect(c, nullptr);
}

int excp_decompress_step_static(int hip_device, void *hip_stream, const void *W_prev_recon, const void *blob,
                                uint64_t blob_bytes, uint64_t n, void *W_recon_out, float *m_out, float *v_out,
                                uint32_t flags) {
    if ((flags & ~0x30u) || (flags & 0x30u) == 0x30u) return EXCP_E_ARG;
    if (n > EXCP_STATIC_MAX_ELEMS) return EXCP_E_ARG;           // the static tables hold no more tiles than that
    if (!blob || ((uintptr_t)blob & 15u) || (n && !W_prev_recon)) return EXCP_E_ARG;
    if (hip_device < 0 || hip_device >= kMaxDevices) return EXCP_E_ARG;
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || hip_device >= ndev) return EXCP_E_HIP;
    if (hipSetDevice(hip_device) != hipSuccess) return EXCP_E_HIP;
    StaticDevice sd;
    int rc = static_device(hip_device, sd);
    if (rc != EXCP_OK) return rc;
    hipStream_t s = (hipStream_t)hip_stream;

    Workspace w{};
    w.ddesc = (DDesc *)(sd.ptr + StaticOffsets::ddesc);
    w.dst = (DState *)(sd.ptr + StaticOffsets::dst);
    w.tile_begin = (u32 *)(sd.ptr + StaticOffsets::tile_begin);
    w.dec_kinds = (u32 *)(sd.ptr + StaticOffsets::dec_kinds);
    w.rec_dev = (HostRec *)(sd.ptr + StaticOffsets::rec);
    w.dec_part = (u32 *)(sd.ptr + StaticOffsets::dec_part);
    w.dec_part_stride = kStaticRuns;
    w.dec_cnt_w = (u32 *)(sd.ptr + StaticOffsets::cnt_w);
    w.dec_cnt_o = (u32 *)(sd.ptr + StaticOffsets::cnt_o);
    w.rec_base = 0;
    w.cus = sd.cus;

    DDesc d{};
    d.Wp = (const float *)W_prev_recon; d.blob = (const unsigned char *)blob; d.blob_bytes = blob_bytes; d.n = n;
    d.W_out = (float *)W_recon_out; d.m_out = m_out; d.v_out = v_out;
    d.cw = d.cm = d.cv = d.head = nullptr; d.wtype = (flags >> 4) & 3u; d.pad = 0;
    d.tile_begin = 0; d.tile_count = (u32)((n + EXCP_TILE - 1) / EXCP_TILE);
    const u32 ntiles = d.tile_count;
    const bool moments = m_out != nullptr || v_out != nullptr;

    // Nothing of the previous call is relied on: the descriptor, the tile table and the kinds word are written by the first launch,
    // the state, every count of the tiles in use and the record by the kernels before they are read.
    launch_decode_prep(w, 1, ntiles, ntiles, true, moments, true, &d, s);
    if (excp_prep_small(ntiles)) {
        launch_decode_small(w, 1, ntiles, moments, d.wtype != 0u, s);
    } else {
        if (d.wtype == 0u) launch_decode_main(w, 1, ntiles, moments, s);
        else launch_decode_main16(w, 1, ntiles, moments, s);
        launch_decode_raw(w, 1, ntiles, moments, s);
    }
    if (hipGetLastError() != hipSuccess) { (void)hipStreamSynchronize(s); return EXCP_E_HIP; }
    HostRec rec;
    memset(&rec, 0, sizeof(rec));
    if (hipMemcpyAsync(&rec, w.rec_dev, sizeof(HostRec), hipMemcpyDeviceToHost, s) != hipSuccess) {
        (void)hipStreamSynchronize(s);
        return EXCP_E_HIP;
    }
    if (hipStreamSynchronize(s) != hipSuccess) return EXCP_E_HIP;
    return rec.status;
}

}  // extern "C"

// Non-uniform quantisation of the surviving values (Sec. 3.3): per stream, K = 2^nbits - 1
// centres by Lloyd's algorithm, then codes = 1 + nearest centre packed nbits each (Sec. 4.2).
//
// One-dimensional Lloyd has structure that makes re-reading every value in every iteration
// unnecessary: clusters are intervals, and the assignment is monotone in the value.  So each stream
// is first PARTITIONED into 256 value-ordered buckets of roughly equal population, and for every
// bucket the exact count, exact sum, minimum and maximum are stored.  The bucket of a value comes
// from arithmetic and one table look-up: the magnitude's bit pattern, offset and shifted, names one
// of 2048 cells per sign (bit patterns of floats are ordered like the values, roughly
// logarithmically), and a sample of the stream decides which run of cells forms which bucket.
// In an iteration a bucket whose minimum and maximum go to the same centre contributes its stored
// totals; only the (at most K-1) buckets that a cluster border cuts are read element by element.
// The same buckets give the initial centres (order statistics of rank ((2k+1) len)/(2K)) with a
// radix select inside one bucket per rank.
//
// All sums are exact: a value is mant * 2^(pos-149); values that are neighbours in magnitude (inside
// a window of 24 binary orders) are whole multiples of one unit, small enough that sixteen of them add
// exactly in fp64; those partial sums go on as integers and end in signed 64-bit bins 8 binary orders
// apart (the representation of the exact sum of |m| in the statistics pass, here with sign); a value
// outside the window is filed into the bins by itself.  A centre is therefore
// fp32(round-once-fp64(exact sum) / count), independent of the order in which values were met, so
// integer atomics may be used freely and the partition need not be stable.
//
// The survivor passes walk one chunk list (8192 values per chunk) spanning every stream of every
// tensor of the group; its length is known only on the device.
#include "excp_util.h"

namespace {

constexpr u32 NBKT = 256;
constexpr u32 PER_THREAD = EXCP_CHUNK / EXCP_THREADS;   // 32

__device__ __forceinline__ const float *seg_data(const Workspace &w, u32 sidx) {
    const u32 t = sidx / 3u, which = sidx % 3u;
    const float *basep = which == 0 ? w.xw : (which == 1 ? w.xm : w.xv);
    return basep + w.desc[t].elem_off;
}
__device__ __forceinline__ float *seg_part(const Workspace &w, u32 sidx) {
    const u32 t = sidx / 3u, which = sidx % 3u;
    float *basep = which == 0 ? w.pw : (which == 1 ? w.pm : w.pv);
    return basep + w.desc[t].elem_off;
}

// A launch over some of the group's streams: all of them, the residual streams, or the moment streams.
enum { STREAMS_ALL = 0, STREAMS_W = 1, STREAMS_MV = 2 };
__device__ __forceinline__ u32 stream_of(u32 idx, u32 sel) {
    return sel == STREAMS_ALL ? idx : (sel == STREAMS_W ? 3u * idx : 3u * (idx >> 1) + 1u + (idx & 1u));
}
// The stream whose turn is `turn` where those of large tensors go first: what is long and starts last keeps a few
// compute units working while the others are done.  (410M-shaped checkpoint: bucket totals 469 -> 327 us, part of which
// is owed to the shorter rounds of small buckets, initial centres 188 -> 121, Lloyd iterations of the streams that one
// workgroup takes 387 -> 244.)
__device__ __forceinline__ u32 stream_in_turn(const Workspace &w, u32 turn) {
    return 3u * ((const EXCP_CONSTANT TDesc *)(uintptr_t)(w.desc + turn / 3u))->turn + turn % 3u;
}
static u32 stream_count(u32 ntensors, u32 sel) { return ntensors * (sel == STREAMS_ALL ? 3u : (sel == STREAMS_W ? 1u : 2u)); }

// Four consecutive floats at an address that is only known to be 4-byte aligned.
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));

// ---------------------------------------------------------------- exact signed accumulation
// Adds v * 2^(bitpos - 149) to a set of signed bins (bin g has weight 2^(8g - 149)), with integer atomics.
__device__ __forceinline__ void file_i64(u64 *bins, long long v, u32 bitpos) {
    const bool neg = v < 0;
    const u64 mag = neg ? (u64)0 - (u64)v : (u64)v;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const u64 piece = (mag >> (32 * q)) & 0xffffffffull;
        const u32 p = bitpos + 32u * q;
        const u64 d = piece << (p & 7u);
        if (piece) atomicAdd(&bins[p >> 3], neg ? (u64)0 - d : d);
    }
}

// Exact summation of values that are neighbours in magnitude.  A value inside the window of 24 bit
// positions [B, B + 24) is a whole multiple of the unit 2^(B-149) below 2^47 units, so up to sixteen of
// them add exactly in fp64, whatever their signs; such a partial sum is then split into two integers
// -- units below 2^32, and signed multiples of 2^32 units -- that go on in 64-bit integer counters.
struct WindowSum {
    double part = 0.0;             // at most sixteen values since the last fold
    long long lo = 0, hi = 0;      // sum = (lo + 2^32 hi) units
    __device__ __forceinline__ void fold(u32 B) {
        const double units = ldexp(part, 149 - (int)B);                  // an integer, |units| < 2^51
        const double h = floor(units * 2.3283064365386963e-10);          // floor(units / 2^32), |h| < 2^19
        lo += (long long)(u32)(units - h * 4294967296.0);
        hi += (long long)(int)h;
        part = 0.0;
    }
};
// magnitudes (bit patterns without the sign) inside the window: lo <= pattern < lo + span
__device__ __forceinline__ void window_range(u32 B, u32 &lo, u32 &span) {
    lo = B ? ((B + 1u) << 23) : 0u;
    span = ((B + 25u) << 23) - lo;
}

// ---------------------------------------------------------------- P0: value -> bucket map from a sample
// The sample is drawn by sixteen workgroups per stream: a survivor's address is a chain of look-ups, each of its own cache
// line, and one compute unit takes about a line a cycle.  (One workgroup that did all: 32 us for a 16.8 M-element tensor.)
// The stream is read where the mask pass left it, in the sub-tile slots (the dense copy is made
// afterwards, by the pass that also counts the buckets this map defines): survivor p of the stream
// sits in the sub-tile whose scanned count is the last one <= p.  The samples lie in the array that the dense copy
// will take, which has room for them: a stream has no fewer places than values.
constexpr u32 DRAW_PARTS = 16;
__device__ __forceinline__ float *seg_sample(const Workspace &w, u32 sidx) { return const_cast<float *>(seg_data(w, sidx)); }

template <u32 DRAW_PER>                                    // samples of a thread
__global__ __launch_bounds__(EXCP_THREADS) void k_km_draw(Workspace w, GroupParams g) {
    constexpr u32 COARSE = 256;
    __shared__ u32 s_coarse[COARSE];
    const u32 sidx = blockIdx.x / DRAW_PARTS, part = blockIdx.x % DRAW_PARTS, tid = threadIdx.x;
    const u64 len = w.seg[sidx].len;
    const u32 ns = (u32)min(len, (u64)g.samples);
    {   // the stream's rows of the count table start at zero (the counts are taken by k_mask_gather)
        const u32 rows = (u32)((len + (1ull << g.unit_shift) - 1u) >> g.unit_shift);
        u32 *row0 = w.km_cnt + (u64)w.seg[sidx].row_begin * NBKT;
        for (u64 i = part * EXCP_THREADS + tid; i < (u64)rows * NBKT; i += DRAW_PARTS * EXCP_THREADS) row0[i] = 0;
    }
    const u32 i0 = (u32)(((u64)ns * part) / DRAW_PARTS), i1 = (u32)(((u64)ns * (part + 1u)) / DRAW_PARTS);
    if (i0 >= i1) return;
    const u32 ts = sidx / 3u, which = sidx % 3u;
    const u32 sub_first = 2u * w.tile_begin[ts], nsub = 2u * w.tile_begin[ts + 1u] - sub_first;
    const u64 *pre = w.mask_prefix + sub_first;
    const float *__restrict__ slots = (which == 0 ? w.pw : (which == 1 ? w.pm : w.pv)) + w.desc[ts].elem_off;
    auto at_of = [&](u64 packed) { return which == 0 ? (u32)(packed >> 32) : (u32)packed; };
    // every (nsub / 256)-th scanned count is fetched first; a search then takes eight steps in LDS and only the rest in memory
    auto coarse_sub = [&](u32 k) { return (u32)(((u64)k * nsub) / COARSE); };
    s_coarse[tid] = at_of(pre[coarse_sub(tid)]);
    __syncthreads();
    u32 pos[DRAW_PER], lo[DRAW_PER], hi[DRAW_PER];
#pragma unroll
    for (u32 k = 0; k < DRAW_PER; ++k) {
        const u32 i = min(i0 + tid + k * EXCP_THREADS, i1 - 1u);
        pos[k] = (u32)(((u64)i * len) / ns);
        lo[k] = 0;
    }
#pragma unroll
    for (u32 step = COARSE / 2; step >= 1u; step >>= 1) {
#pragma unroll
        for (u32 k = 0; k < DRAW_PER; ++k) if (s_coarse[lo[k] + step] <= pos[k]) lo[k] += step;
    }
#pragma unroll
    for (u32 k = 0; k < DRAW_PER; ++k) {            // invariant: prefix(lo) <= pos < prefix(hi)
        hi[k] = lo[k] + 1u < COARSE ? max(coarse_sub(lo[k] + 1u), coarse_sub(lo[k]) + 1u) : nsub;
        lo[k] = coarse_sub(lo[k]);
    }
    bool more = true;
    while (more) {
        more = false;
        u32 mid[DRAW_PER];
        u64 pv[DRAW_PER];
#pragma unroll
        for (u32 k = 0; k < DRAW_PER; ++k) { mid[k] = (lo[k] + hi[k]) >> 1; pv[k] = hi[k] - lo[k] > 1u ? pre[mid[k]] : 0ull; }
#pragma unroll
        for (u32 k = 0; k < DRAW_PER; ++k) {
            if (hi[k] - lo[k] > 1u) {
                if (at_of(pv[k]) <= pos[k]) lo[k] = mid[k]; else hi[k] = mid[k];
                more = more || hi[k] - lo[k] > 1u;
            }
        }
    }
    u32 at[DRAW_PER];
#pragma unroll
    for (u32 k = 0; k < DRAW_PER; ++k) at[k] = at_of(pre[lo[k]]);
    float *smp = seg_sample(w, sidx);
#pragma unroll
    for (u32 k = 0; k < DRAW_PER; ++k) {
        const float x = slots[(u64)lo[k] * 2048u + (pos[k] - at[k])];
        if (i0 + tid + k * EXCP_THREADS < i1) smp[i0 + tid + k * EXCP_THREADS] = x;
    }
}

// One workgroup per stream.  The sample fixes the magnitude range of each sign (hence offset and
// shift of the cells); the cells' sample counts, scanned, give every cell its bucket so that the
// buckets hold about equal shares of the sample.
constexpr u32 SM_THREADS = 1024;

__global__ __launch_bounds__(SM_THREADS) void k_km_sample(Workspace w, GroupParams g) {
    __shared__ u32 cnt[EXCP_KM_CELLS];
    __shared__ u32 s_map[4];
    __shared__ u32 s_ext[4];                       // min / max magnitude of the negative, of the positive samples
    __shared__ u32 s_wave[SM_THREADS / 64];
    constexpr u32 PER_S = EXCP_SAMPLES_MANY / SM_THREADS;
    const u32 sidx = blockIdx.x, tid = threadIdx.x;
    const u64 len = w.seg[sidx].len;
    if (len == 0) return;
    const u32 ns = (u32)min(len, (u64)g.samples);
    const float *smp = seg_sample(w, sidx);
    if (tid < 4) s_ext[tid] = (tid & 1u) ? 0u : 0xffffffffu;
    for (u32 c = tid; c < EXCP_KM_CELLS; c += SM_THREADS) cnt[c] = 0;
    float v[PER_S];
#pragma unroll
    for (u32 k = 0; k < PER_S; ++k) v[k] = tid + k * SM_THREADS < ns ? smp[tid + k * SM_THREADS] : 0.f;
    u32 mn[2] = {0xffffffffu, 0xffffffffu}, mx[2] = {0u, 0u};
#pragma unroll
    for (u32 k = 0; k < PER_S; ++k) {
        if (tid + k * SM_THREADS < ns) {
            const u32 bits = f2u(v[k]), a = bits & 0x7fffffffu, sg = bits >> 31;
            if (sg) { mn[0] = min(mn[0], a); mx[0] = max(mx[0], a); } else { mn[1] = min(mn[1], a); mx[1] = max(mx[1], a); }
        }
    }
    __syncthreads();
#pragma unroll
    for (int sg = 0; sg < 2; ++sg) {
        const u32 lo = wave_min_u32(mn[sg]), hi = wave_max_u32(mx[sg]);
        if ((tid & 63u) == 0) { atomicMin(&s_ext[2 * sg], lo); atomicMax(&s_ext[2 * sg + 1], hi); }
    }
    __syncthreads();
    if (tid < 2) {
        const u32 lo = s_ext[2 * tid], hi = s_ext[2 * tid + 1];
        u32 amin = 0, sh = 20;                     // no sample of this sign: exponent and 3 mantissa bits
        if (lo <= hi) {
            const u32 width = hi - lo;             // (width >> sh) must stay below 2048
            const u32 bits = width ? 32u - (u32)__clz((int)width) : 0u;
            amin = lo;
            sh = bits > 11u ? bits - 11u : 0u;
        }
        s_map[2 * tid] = amin; s_map[2 * tid + 1] = sh;
    }
    __syncthreads();
#pragma unroll
    for (u32 k = 0; k < PER_S; ++k) if (tid + k * SM_THREADS < ns) atomicAdd(&cnt[cell_of(v[k], s_map)], 1u);
    __syncthreads();
    // Exclusive scan over the cells (four consecutive cells per thread), then bucket = share of the sample
    // below.  A cell that alone holds more than 1/64 of the sample is a tied value (a continuous
    // distribution never fills one of 4096 cells like that): it gets a bucket of its own, so that a bucket
    // is either one repeated value -- which neither the initial order statistics nor the Lloyd
    // iterations ever have to read again -- or an even share of the rest.  With H such cells the others
    // are spread over S = 255 - 2 H buckets; a heavy cell sits one above the light cells before it and
    // one below those after it.
    constexpr u32 PER = EXCP_KM_CELLS / SM_THREADS;       // 4
    const u32 heavy_min = max(ns / 64u, 32u);
    u32 local[PER], sum = 0;                               // sum: heavy cells << 16 | samples in light cells
#pragma unroll
    for (u32 q = 0; q < PER; ++q) {
        local[q] = cnt[tid * PER + q];
        sum += local[q] >= heavy_min ? (1u << 16) : local[q];
    }
    u32 incl = wave_incl_scan_u32(sum);
    if (lane_id() == 63u) s_wave[tid >> 6] = incl;
    __syncthreads();
    u32 run = incl - sum, total = 0;
    for (u32 q = 0; q < SM_THREADS / 64u; ++q) { if (q < (tid >> 6)) run += s_wave[q]; total += s_wave[q]; }
    const u32 H = total >> 16, ns_light = total & 0xffffu;
    const u32 S = NBKT - 1u - 2u * H;                      // H <= 64, so S >= 127
    u32 *out = w.km_split + (u64)sidx * EXCP_KM_MAP_WORDS;
    if (tid < 4) out[tid] = s_map[tid];
#pragma unroll
    for (u32 q4 = 0; q4 < PER / 4; ++q4) {
        u32 word = 0;
#pragma unroll
        for (u32 q = 0; q < 4; ++q) {
            const u32 c = local[q4 * 4 + q];
            const bool heavy = c >= heavy_min;
            const u32 light_before = run & 0xffffu, heavy_before = run >> 16;
            const u32 share = ns_light ? min((u32)(((u64)light_before * S) / ns_light), S - 1u) : 0u;
            const u32 bkt = share + 2u * heavy_before + (heavy ? 1u : 0u);
            word |= bkt << (8u * q);
            run += heavy ? (1u << 16) : c;
        }
        out[4 + tid * (PER / 4) + q4] = word;
    }
}

// Loads the 32 values a thread owns in a chunk: eight groups of four consecutive values (group it
// starts at element (it * 256 + tid) * 4).  Values past the chunk's end are returned as NaN.
__device__ __forceinline__ void load_chunk(const EXCP_GLOBAL float *gx, u32 clen, float (&v)[PER_THREAD]) {
    const u32 tid = threadIdx.x;
    if (clen == EXCP_CHUNK) {
#pragma unroll
        for (u32 it = 0; it < PER_THREAD / 4; ++it) {
            const f4u q = *(const EXCP_GLOBAL f4u *)(gx + (it * EXCP_THREADS + tid) * 4u);
            v[4 * it] = q.x; v[4 * it + 1] = q.y; v[4 * it + 2] = q.z; v[4 * it + 3] = q.w;
        }
    } else {
#pragma unroll
        for (u32 it = 0; it < PER_THREAD; ++it) {
            const u32 e = ((it >> 2) * EXCP_THREADS + tid) * 4u + (it & 3u);
            v[it] = e < clen ? gx[e] : __uint_as_float(0x7fc00000u);
        }
    }
}
__device__ __forceinline__ u32 chunk_elem(u32 it) { return ((it >> 2) * EXCP_THREADS + threadIdx.x) * 4u + (it & 3u); }

// ---------------------------------------------------------------- P1, P2: bucket counts, positions
// The counts are taken by the pass that makes the dense survivor arrays (k_mask_gather), per unit of a
// stream (2 to 16 chunks, by the size of the group), a row each.  One workgroup per stream turns them into positions:
// bucket totals, their scan, then every row's first position in every bucket.  A wave reads a row, four buckets to
// a lane, and owns a sixteenth of the rows; what bounds it is the number of loads that wait for one another.  (With a bucket
// to a thread and a quarter of the rows each, 354 rows of a 16.8 M-element tensor took 14.4 us; with each row read twice 13.3, with up to 24 rows a wave held in registers 10.)
constexpr u32 SCAN_PARTS = 16, SCAN_HELD = 24, CROWD_MOST = 8192;
__global__ __launch_bounds__(SCAN_PARTS * 64) void k_km_scan(Workspace w, GroupParams g) {
    __shared__ __attribute__((aligned(16))) u32 tot[SCAN_PARTS][NBKT];
    __shared__ __attribute__((aligned(16))) u32 first[NBKT];
    __shared__ u32 s_wave[4], s_most[4];
    typedef u32 u4 __attribute__((ext_vector_type(4)));
    const u32 sidx = blockIdx.x, tid = threadIdx.x, lane = tid & 63u;
    const u32 part = (u32)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
    const u64 len = w.seg[sidx].len;
    if (len == 0) return;
    const u32 rows = (u32)((len + (1ull << g.unit_shift) - 1u) >> g.unit_shift);
    const u32 per = (rows + SCAN_PARTS - 1u) / SCAN_PARTS, a0 = min(part * per, rows), a1 = min(a0 + per, rows);
    EXCP_GLOBAL u4 *cnt = gptr((u4 *)(w.km_cnt + (u64)w.seg[sidx].row_begin * NBKT)) + lane;      // (rows are 1 KB)
    u4 s = {0u, 0u, 0u, 0u}, held[SCAN_HELD];
    const bool once = per <= SCAN_HELD;                    // the wave's rows stay in registers
    if (once) {
#pragma unroll
        for (u32 c = 0; c < SCAN_HELD; ++c) held[c] = a0 + c < a1 ? cnt[(u64)(a0 + c) * (NBKT / 4u)] : (u4){0u, 0u, 0u, 0u};
#pragma unroll
        for (u32 c = 0; c < SCAN_HELD; ++c) s += held[c];
    } else {
#pragma unroll 8
        for (u32 c = a0; c < a1; ++c) s += cnt[(u64)c * (NBKT / 4u)];
    }
    *(u4 *)&tot[part][4u * lane] = s;
    __syncthreads();
    u32 total = 0, incl = 0;
    if (tid < NBKT) {
        for (u32 q = 0; q < SCAN_PARTS; ++q) total += tot[q][tid];
        incl = wave_incl_scan_u32(total);
        const u32 most = wave_max_u32(total);
        if (lane == 63u) { s_wave[part] = incl; s_most[part] = most; }
    }
    __syncthreads();
    if (tid == 0) {
        const u32 most = max(max(s_most[0], s_most[1]), max(s_most[2], s_most[3]));
        const bool crowded = (u64)most > 3ull * (len / NBKT) + 1024ull;
        w.seg[sidx].crowded = crowded ? 1u : 0u;
        // A stream whose buckets do not fit the workgroups, or of which one bucket holds so many values that an iteration takes one
        // workgroup as long as a launch, is what is waited for: cells in the buckets of others would gain nothing.  (Sixty tensors
        // of a sign-like update, 20 M elements: 1606 -> 1555 us.)
        if (most > (crowded ? CROWD_MOST : excp_cells_most(g.fine_size))) *w.no_cells = 1u;
    }
    if (tid < NBKT) {
        u32 run = incl - total;
        for (u32 v = 0; v < part; ++v) run += s_wave[v];
        first[tid] = run;
        w.km_begin[(u64)sidx * (NBKT + 1) + tid] = run;
        if (tid == NBKT - 1u) w.km_begin[(u64)sidx * (NBKT + 1) + NBKT] = run + total;
    }
    __syncthreads();
    u4 run = *(const u4 *)&first[4u * lane];
    for (u32 q = 0; q < part; ++q) run += *(const u4 *)&tot[q][4u * lane];
    if (once) {
#pragma unroll
        for (u32 c = 0; c < SCAN_HELD; ++c) {
            if (a0 + c < a1) cnt[(u64)(a0 + c) * (NBKT / 4u)] = run;
            run += held[c];
        }
        return;
    }
#pragma unroll 8
    for (u32 c = a0; c < a1; ++c) {
        const u4 v = cnt[(u64)c * (NBKT / 4u)];
        cnt[(u64)c * (NBKT / 4u)] = run;
        run += v;
    }
}

// ---------------------------------------------------------------- P3: scatter into buckets
// A workgroup takes a contiguous range of chunks; inside one stream the runs that consecutive chunks
// contribute to a bucket are neighbours in memory, so the workgroup keeps, per bucket, a ring of up to
// 128 values in LDS and writes a bucket's values as whole, aligned 128-byte lines (partial lines reach
// memory at a fraction of the rate of whole ones: a run of about 32 values that starts anywhere costs
// twice a run that starts on a line).  Partial lines are written only where a workgroup's range or a
// stream begins or ends.  Values arrive 8192 at a time (eight per thread): a value takes the next place
// of its bucket's ring (one LDS atomic on a counter that also carries the ring's read position); then
// thread b looks at bucket b and lists the lines that are complete; then groups of eight lanes write
// the listed lines, sixteen bytes per lane.  A value's ring index is its place inside its memory line,
// so a whole line is one aligned quarter of the ring.  When more values arrive for a bucket in one step
// than its ring holds (tied data: one bucket takes most of a stream), those beyond the ring go straight
// to their places in memory -- consecutive arrivals, consecutive addresses -- and the ring is emptied.
// The order of values inside a bucket is that of arrival, which no reader of a bucket depends on
// (its sum, count, extremes and order statistics are those of a multiset).
constexpr u32 SC_THREADS = 1024, SC_STEP = 8192, SC_PER = SC_STEP / SC_THREADS, SC_RING = 128, SC_LIST = 1536;

__global__ __launch_bounds__(SC_THREADS, 1) void k_km_scatter(Workspace w, GroupParams g) {
    __shared__ __attribute__((aligned(16))) float ring[NBKT][SC_RING];
    __shared__ u32 cells[EXCP_KM_CELLS / 4u];
    __shared__ u32 ctr[NBKT];                            // (ring index of the oldest value) << 16 | values waiting
    __shared__ u32 gpos[NBKT];                           // place of the oldest value in the bucket-ordered array
    __shared__ __attribute__((aligned(8))) u32 list[2 * SC_LIST];   // lines to write: (bucket | ring index << 8 | count << 16), place
    __shared__ u32 nlist;
    const u32 tid = threadIdx.x, grp = tid >> 3, gl = tid & 7u;    // groups of eight lanes write a line each
    const u32 total = *w.chunk_total;
    const u32 G = gridDim.x, bid = blockIdx.x;
    const u32 nseg = 3u * g.ntensors;
    // Equal shares of the chunk list, their ends moved back to where the bucket counts were taken: the first
    // chunk of a unit.
    const u32 unit_chunks = (1u << g.unit_shift) / EXCP_CHUNK;
    auto snapped = [&](u32 c) -> u32 {
        if (c >= total) return total;
        const u32 c0 = w.seg_chunk_begin[find_owner(w.seg_chunk_begin, nseg, c)];
        return c0 + ((c - c0) & ~(unit_chunks - 1u));
    };
    const u32 lo = snapped((u32)(((u64)bid * total) / G)), hi = snapped((u32)(((u64)(bid + 1) * total) / G));
    if (lo >= hi) return;
    if (tid == 0) nlist = 0;

    for (u32 c = lo; c < hi;) {
        // the chunks [c, c_end) of this workgroup that belong to one stream
        __syncthreads();
        const u32 sidx = find_owner(w.seg_chunk_begin, nseg, c);
        const u32 c_end = min(hi, w.seg_chunk_begin[sidx + 1]);
        const u64 len = w.seg[sidx].len;
        const u32 chunk0 = w.seg[sidx].chunk_begin;
        const EXCP_GLOBAL float *data = gptr(seg_data(w, sidx));
        EXCP_GLOBAL float *part = gptr(seg_part(w, sidx));
        const u32 misalign = (u32)(((uintptr_t)seg_part(w, sidx) >> 2) & 31u);   // (place + misalign) % 32 == 0: a line starts
        // the value -> bucket table stays in global memory (4 KB, read through the vector cache): the LDS unit
        // is what this kernel is short of
        const u32 *mp = w.km_split + (u64)sidx * EXCP_KM_MAP_WORDS;
        const u32 neg_min = mp[0], neg_sh = mp[1], pos_min = mp[2], pos_sh = mp[3];
        for (u32 i = tid; i < EXCP_KM_CELLS / 4u; i += SC_THREADS) cells[i] = mp[4u + i];
        const unsigned char *cellmap = (const unsigned char *)cells;
        auto bucket = [&](float x) -> u32 {
            const u32 bits = f2u(x), a = bits & 0x7fffffffu;
            const bool neg = bits >> 31;
            const u32 amin = neg ? neg_min : pos_min, sh = neg ? neg_sh : pos_sh;
            const u32 cc = min((max(a, amin) - amin) >> sh, HALF_CELLS - 1u);
            return cellmap[neg ? (cc ^ (HALF_CELLS - 1u)) : (cc | HALF_CELLS)];
        };
        if (tid < NBKT) {
            // a ring index is the value's place inside its line, so that whole lines sit in one quarter of the ring
            const u32 gp = w.km_cnt[(u64)(w.seg[sidx].row_begin + (c - chunk0) / unit_chunks) * NBKT + tid];
            gpos[tid] = gp;
            ctr[tid] = ((gp + misalign) & 31u) << 16;
        }
        const u64 e_begin = (u64)(c - chunk0) * EXCP_CHUNK;
        const u64 e_stop = min(len, (u64)(c_end - chunk0) * EXCP_CHUNK);
        __syncthreads();

        // thread b: which lines of bucket b can be written now (at the end of the range: everything)
        auto plan = [&](bool final) {
            if (tid >= NBKT) return;                    // (whole waves)
            const u32 b = tid;
            const u32 cv = ctr[b];
            const u32 arrived = cv & 0xffffu;           // since the last look: more than the ring holds if the bucket is crowded
            const bool over = arrived > SC_RING;        // the values beyond the ring went straight to their places
            const bool all = final || over;
            const u32 f0 = min(arrived, SC_RING), h0 = cv >> 16, gp0 = gpos[b];
            // what leaves: the values up to the next line start, then whole lines, and (all) the rest
            const u32 mis = (gp0 + misalign) & 31u;
            u32 f = f0, head_cnt = 0;
            if (f && mis && (f >= 32u - mis || all)) { head_cnt = min(32u - mis, f); f -= head_cnt; }
            const bool aligned = ((gp0 + head_cnt + misalign) & 31u) == 0u;
            const u32 nfull = aligned ? f >> 5 : 0u;
            f -= nfull << 5;
            const u32 tail_cnt = (aligned && all) ? f : 0u;
            f -= tail_cnt;
            const u32 ne = (head_cnt ? 1u : 0u) + nfull + (tail_cnt ? 1u : 0u);
            const u32 gone = f0 - f;
            if (over) {                                 // the ring is empty and starts again behind everything that arrived
                gpos[b] = gp0 + arrived;
                ctr[b] = ((gp0 + arrived + misalign) & 31u) << 16;
            } else {
                ctr[b] = (((h0 + gone) & (SC_RING - 1u)) << 16) | f; gpos[b] = gp0 + gone;
            }
            // places in the list: one atomic per wave, the lanes' shares by counting the set bits below them
            const u64 b0 = ballot64(ne & 1u), b1 = ballot64(ne & 2u), b2 = ballot64(ne & 4u);
            const u32 wave_total = (u32)__popcll(b0) + 2u * (u32)__popcll(b1) + 4u * (u32)__popcll(b2);
            if (wave_total) {
                u32 base = 0;
                if ((tid & 63u) == 0u) base = atomicAdd(&nlist, wave_total);
                base = (u32)__builtin_amdgcn_readfirstlane((int)base);
                u32 at = base + lanes_below(b0) + 2u * lanes_below(b1) + 4u * lanes_below(b2);
                u32 h = h0, gp = gp0;
                auto emit = [&](u32 cnt) {
                    list[2u * at] = b | (h << 8) | (cnt << 16); list[2u * at + 1u] = gp; ++at;
                    h = (h + cnt) & (SC_RING - 1u); gp += cnt;
                };
                if (head_cnt) emit(head_cnt);
                for (u32 k = 0; k < nfull; ++k) emit(32u);
                if (tail_cnt) emit(tail_cnt);
            }
        };
        // groups of eight lanes write the listed lines, four values per lane
        auto write_lines = [&]() {
            const u32 n = nlist;
            constexpr u32 GROUPS = SC_THREADS / 8u;
            for (u32 i = grp; i < n; i += GROUPS) {
                const u64 ev = *(const u64 *)&list[2u * i];
                const u32 e0 = (u32)ev, b = e0 & 255u, off = (e0 >> 8) & 255u, cnt = e0 >> 16, gp = (u32)(ev >> 32);
                if (cnt == 32u) {                       // a whole line: it sits in one half of the ring, and on a line in memory
                    typedef float f4a __attribute__((ext_vector_type(4)));      // 16-byte aligned on both sides
                    const f4a x = *(const f4a *)&ring[b][off + 4u * gl];
                    *(EXCP_GLOBAL f4a *)(part + (u64)gp + 4u * gl) = x;
                } else {
#pragma unroll
                    for (u32 k = 0; k < 4; ++k) {
                        const u32 idx = 4u * gl + k;
                        if (idx < cnt) part[(u64)gp + idx] = ring[b][(off + idx) & (SC_RING - 1u)];
                    }
                }
            }
        };

        float nx[SC_PER];
        auto load_step = [&](u64 e, float (&v)[SC_PER]) {
            const u32 nval = (e_stop - e) < (u64)SC_STEP ? (u32)(e_stop - e) : SC_STEP;
            if (nval == SC_STEP) {
#pragma unroll
                for (u32 q = 0; q < SC_PER / 4; ++q) {
                    const f4u x = *(const EXCP_GLOBAL f4u *)(data + e + (q * SC_THREADS + tid) * 4u);
                    v[4 * q] = x.x; v[4 * q + 1] = x.y; v[4 * q + 2] = x.z; v[4 * q + 3] = x.w;
                }
            } else {
#pragma unroll
                for (u32 j = 0; j < SC_PER; ++j) {
                    const u32 el = ((j >> 2) * SC_THREADS + tid) * 4u + (j & 3u);
                    v[j] = el < nval ? data[e + el] : 0.f;
                }
            }
        };
        if (e_begin < e_stop) load_step(e_begin, nx);
        for (u64 e = e_begin; e < e_stop; e += SC_STEP) {
            const u32 nval = (e_stop - e) < (u64)SC_STEP ? (u32)(e_stop - e) : SC_STEP;
            float v[SC_PER];
#pragma unroll
            for (u32 j = 0; j < SC_PER; ++j) v[j] = nx[j];
            if (e + SC_STEP < e_stop) load_step(e + SC_STEP, nx);      // the next step's values are on their way
            u32 bb[SC_PER], cv[SC_PER];
#pragma unroll
            for (u32 j = 0; j < SC_PER; ++j) bb[j] = bucket(v[j]);
            if (tid == 0) nlist = 0;
            // a value takes the next place of its bucket: in the ring, or, when more than the ring holds have
            // arrived since the bucket was last looked at (tied data: one bucket takes most of a stream),
            // straight in the bucket-ordered array
            if (nval == SC_STEP) {
#pragma unroll
                for (u32 j = 0; j < SC_PER; ++j) cv[j] = atomicAdd(&ctr[bb[j]], 1u);
#pragma unroll
                for (u32 j = 0; j < SC_PER; ++j) {
                    const u32 pos = cv[j] & 0xffffu;
                    if (pos < SC_RING) ring[bb[j]][((cv[j] >> 16) + pos) & (SC_RING - 1u)] = v[j];
                    else part[(u64)gpos[bb[j]] + pos] = v[j];
                }
            } else {
#pragma unroll
                for (u32 j = 0; j < SC_PER; ++j) {
                    if (((j >> 2) * SC_THREADS + tid) * 4u + (j & 3u) < nval) {
                        const u32 c1 = atomicAdd(&ctr[bb[j]], 1u), pos = c1 & 0xffffu;
                        if (pos < SC_RING) ring[bb[j]][((c1 >> 16) + pos) & (SC_RING - 1u)] = v[j];
                        else part[(u64)gpos[bb[j]] + pos] = v[j];
                    }
                }
            }
            __syncthreads();
            plan(false);
            __syncthreads();
            write_lines();
            __syncthreads();
        }
        // the end of the stream or of this workgroup's range: what is left goes out as it is
        if (tid == 0) nlist = 0;
        __syncthreads();
        plan(true);
        __syncthreads();
        write_lines();
        c = c_end;
    }
}

// ---------------------------------------------------------------- P4: exact totals per bucket
// A workgroup takes four neighbouring buckets of a stream (or one): a wave each
// where they are small, and otherwise its waves share every bucket, so that one very large bucket (tied values)
// does not leave a single wave working alone.  The large tensors' sets come first (in a 410M-shaped checkpoint, whose
// last tensor is one of the two large ones, compute units stood idle for a third of the time).  Values of a bucket
// are neighbours in value, hence in exponent: a window of 24 bit positions placed from the first
// values met holds practically all of them; inside it a lane adds sixteen values at a time exactly in
// fp64 and keeps the running total in two integer counters, with no cross-lane traffic; the rest
// (rare) is filed one by one.
// (sixteen waves for the residuals of 16-bit weights, which are heavily tied, and for groups with a tensor so large
// that its buckets alone are millions of values; four otherwise, which is faster when the buckets are
// small and even)
constexpr u32 BESIDE_MAX = 1024;                           // values per wave up to which a set's buckets go side by side
template <u32 BS_WAVES, u32 BPW>
__global__ __launch_bounds__(BS_WAVES * 64, BS_WAVES == 16u ? 8 : 5) void k_km_bucket_stats(Workspace w, GroupParams g, u32 sel, u32 nseg) {
    __shared__ u64 bins[BPW][EXCP_ABSM_BINS];
    __shared__ u32 s_min[BPW], s_max[BPW], s_mag[BPW], s_ndom[BPW], s_less[BPW];
    constexpr bool TIED = BS_WAVES == 16u;
    const u32 tid = threadIdx.x, lane = tid & 63u;
    const u32 wave = (u32)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
    // a workgroup walks over sets of BPW buckets (many sets are tiny: one workgroup each would be
    // bound by the rate at which workgroups can be started)
    for (u32 set = blockIdx.x; set < nseg * (NBKT / BPW); set += gridDim.x) {
    const u32 sets = NBKT / BPW, b0 = set % sets * BPW;
    const u32 sidx = stream_in_turn(w, stream_of(set / sets, sel));
    const EXCP_CONSTANT SegState *seg = (const EXCP_CONSTANT SegState *)(uintptr_t)(w.seg + sidx);
    const EXCP_CONSTANT u32 *begin = (const EXCP_CONSTANT u32 *)(uintptr_t)(w.km_begin + (u64)sidx * (NBKT + 1));
    if (seg->len == 0) continue;                           // the same for the whole workgroup
    __syncthreads();                                       // the previous set has left the LDS tables
    for (u32 i = tid; i < BPW * EXCP_ABSM_BINS; i += BS_WAVES * 64u) (&bins[0][0])[i] = 0;
    if (tid < BPW) { s_min[tid] = 0xffffffffu; s_max[tid] = 0; s_mag[tid] = 0xffffffffu; s_ndom[tid] = 0; s_less[tid] = 0; }
    const EXCP_GLOBAL float *part = gptr(seg_part(w, sidx));
    // Small buckets: all of them side by side, a wave each (four in the sixteen-wave form), instead of a round of
    // memory round trips for each.
    const bool beside = BPW > 1u && begin[b0 + BPW] - begin[b0] <= BESIDE_MAX * BS_WAVES;
    constexpr u32 FEW = BS_WAVES / BPW;
    __syncthreads();
    for (u32 jj = 0; jj < (beside ? 1u : BPW); ++jj) {
        const u32 j = beside ? wave / FEW : jj, share = beside ? wave % FEW : wave;
        const u32 q0 = begin[b0 + j], q1 = begin[b0 + j + 1];
        // this wave's share, cut at multiples of 256 values from the bucket's start
        const u32 blocks = (q1 - q0 + 255u) >> 8, per = beside ? (blocks + FEW - 1u) / FEW : (blocks + BS_WAVES - 1u) / BS_WAVES;
        const u32 p0 = min(q0 + share * per * 256u, q1), p1 = min(p0 + per * 256u, q1);
        if (p0 >= p1) continue;
        u64 *mybins = bins[j];
        // Rounds of 1024 values, sixteen per lane, in four 16-byte loads (the other waves hide their latency).  A
        // lane's values past the end are the share's first one again, and are not taken.
        f4u q[4];
        auto load = [&](u32 p) {
            if (p + 1024u <= p1) {
#pragma unroll
                for (u32 r = 0; r < 4; ++r) q[r] = *(const EXCP_GLOBAL f4u *)(part + p + r * 256u + lane * 4u);
            } else {
#pragma unroll
                for (u32 r = 0; r < 4; ++r) {
                    if (p + r * 256u >= p1) { q[r] = q[0]; continue; }       // (the same in the whole wave)
                    const u32 i = p + r * 256u + lane * 4u;
#pragma unroll
                    for (u32 e = 0; e < 4; ++e) q[r][e] = part[i + e < p1 ? i + e : p0];
                }
            }
        };
        load(p0);
        // Tied data (the sixteen-wave form): a large bucket is mostly one value.  The bucket's first value is taken
        // for that one; its repetitions are only counted, and count times value joins the sums at the end.  How
        // many there are, and how many values are smaller, also answers most questions for an order statistic
        // of the bucket (k_km_init).
        u32 dom = 0, ndom = 0, less = 0;                   // bit pattern of the repeated value; this lane's counts
        if (TIED) dom = (u32)__builtin_amdgcn_readfirstlane((int)f2u(part[q0]));
        const u32 domkey = key_of(u2f(dom));
        // window base from the first round: top 4 binary orders above its largest value
        u32 top = 0;
#pragma unroll
        for (u32 r = 0; r < 4; ++r)
#pragma unroll
            for (u32 e = 0; e < 4; ++e) top = max(top, f2u(q[r][e]) & 0x7fffffffu);
        const u32 pm = bit_pos(wave_max_u32(top));
        const u32 B = pm + 4u > 23u ? pm + 4u - 23u : 0u;
        u32 thr_lo, span;
        window_range(B, thr_lo, span);
        const bool apart = (dom & 0x7fffffffu) - thr_lo < span;    // inside the window: summed by its count
        WindowSum S;
        u32 kmin = 0xffffffffu, kmax = 0, mag = 0xffffffffu;       // mag: smallest magnitude less one (zero wraps to the largest)
        auto take = [&](float xv) {
            const u32 u = f2u(xv), mb = u & 0x7fffffffu;
            if (TIED && u == dom) { ++ndom; if (apart) return; }
            const u32 k = key_of(xv);
            if (TIED) less += k < domkey;
            kmin = min(kmin, k); kmax = max(kmax, k);
            mag = min(mag, mb - 1u);
            if (mb - thr_lo < span) {
                S.part += (double)xv;
            } else if (mb) {
                const u32 e = mb >> 23;
                const u32 mant = (mb & 0x7fffffu) | (e ? 0x800000u : 0u);
                const u32 pos = bit_pos(mb);
                const u64 d = (u64)mant << (pos & 7u);
                atomicAdd(&mybins[pos >> 3], (u >> 31) ? (u64)0 - d : d);
            }
        };
        u32 p = p0;
        for (; p + 1024u <= p1; p += 1024u) {
#pragma unroll
            for (u32 r = 0; r < 4; ++r) { take(q[r].x); take(q[r].y); take(q[r].z); take(q[r].w); }
            S.fold(B);
            if (p + 1024u < p1) load(p + 1024u);
        }
        if (p < p1) {
#pragma unroll
            for (u32 r = 0; r < 4; ++r) {
                if (p + r * 256u >= p1) break;             // (most buckets of a small tensor hold a handful of values)
                const u32 i = p + r * 256u + lane * 4u;
#pragma unroll
                for (u32 e = 0; e < 4; ++e) if (i + e < p1) take(q[r][e]);
            }
            S.fold(B);
        }
        if (TIED && ndom && apart) {
            const u32 mb = dom & 0x7fffffffu, e = mb >> 23;
            const u32 mant = (mb & 0x7fffffu) | (e ? 0x800000u : 0u);
            const u64 term = (u64)mant << (((e ? e : 1u) - 1u) - B);                      // below 2^47 units
            const long long tl = (long long)((term & 0xffffffffull) * ndom), th = (long long)((term >> 32) * ndom);   // a lane sees < 2^20 values
            if (dom >> 31) { S.lo -= tl; S.hi -= th; } else { S.lo += tl; S.hi += th; }
            const u32 k = key_of(u2f(dom));
            kmin = min(kmin, k); kmax = max(kmax, k);
            mag = min(mag, mb - 1u);
        }
        const long long tL = (long long)wave_sum_u64((u64)S.lo), tH = (long long)wave_sum_u64((u64)S.hi);
        kmin = wave_min_u32(kmin); kmax = wave_max_u32(kmax); mag = wave_min_u32(mag);
        if (TIED) { ndom = wave_sum_u32(ndom); less = wave_sum_u32(less); }
        if (lane == 0) {
            if (TIED) { atomicAdd(&s_ndom[j], ndom); atomicAdd(&s_less[j], less); }
            atomicMin(&s_min[j], kmin); atomicMax(&s_max[j], kmax); atomicMin(&s_mag[j], mag);
            file_i64(mybins, tL, B); file_i64(mybins, tH, B + 32u);
        }
    }
    __syncthreads();
    for (u32 i = tid; i < BPW * EXCP_ABSM_BINS; i += BS_WAVES * 64u)
        w.km_bsum[((u64)sidx * EXCP_ABSM_BINS + i / BPW) * (NBKT + 1) + b0 + i % BPW] = bins[i % BPW][i / BPW];
    if (tid < BPW) {
        const u64 at = (u64)sidx * NBKT + b0 + tid;
        w.km_min[at] = s_min[tid]; w.km_max[at] = s_max[tid];
        w.km_mag[at] = s_mag[tid] + 1u;                    // (0: nothing but zeros, or nothing at all)
        if (TIED) { w.km_less[at] = s_less[tid]; w.km_dom[at] = s_ndom[tid]; }
    }
    }
}

// ---------------------------------------------------------------- P4b: cells inside the buckets
// What a Lloyd iteration reads is a bucket for every border, and an initial centre a bucket for its rank.  Where a group has
// no more streams than the GPU has compute units, its larger buckets are therefore put in order once more, in up to 512 cells of
// 64 to 128 values, with the exact sum of what lies above every cell: then one workgroup takes a stream through
// all its iterations, whatever its length, instead of a launch per iteration in which many read the buckets.  (One
// 16.8 M-element tensor, 4 bits, ten iterations: cells 33 us; iterations 154 -> 43, initial centres 35 -> 12.  Where the line
// lies: excp_fine_tensor.)
//
// A workgroup per bucket: its values are read into registers, counted and added up per cell in LDS, and written back through
// LDS in the order of their cells.  The cells are equal ranges of the (order-preserving) key between the bucket's extremes,
// without the gap round zero that a bucket of both signs has.  Sums are in units of the bucket's lowest bit position, so the
// bucket may span FINE_SPAN binary orders (24 of the mantissa, 16 of the number of values, 23: 63 bits).  A bucket that
// spans more gets no cells and is read as a whole; with a bucket larger than the workgroup's registers the group has none (k_km_scan).
constexpr u32 FINE_SPAN = 23, FINE_LEAST = 256;            // smaller buckets are one cell without any table
// km_fine: cells' log2 | shift << 4 | largest cell << 9 | FINE_NEAR: the values span eight binary orders at most | FINE_VALID
constexpr u32 FINE_VALID = 1u << 31, FINE_NEAR = 1u << 30, NEAR_SPAN = 8;
// Values over more than eight binary orders lie bunched in a few cells, and add up in integers, thirty-five instructions each: with a
// cell of more than so many the bucket is read as a whole by the workgroup sooner than a cell by its border's few lanes.  (500 000
// elements, all kept, 8 bits, a middle bucket of 2000 values in 21 binary orders: 600 us with its cells, 492 without, 495 before there
// were any.)
constexpr u32 FAR_MOST = 256;
__device__ __forceinline__ u32 fine_log2(u32 info) { return info & 15u; }
__device__ __forceinline__ u32 fine_shift(u32 info) { return (info >> 4) & 31u; }
__device__ __forceinline__ u32 fine_most(u32 info) { return (info >> 9) & 0xffffu; }
// A value of magnitude pattern mb in units of 2^(pos_lo - 149).
__device__ __forceinline__ u64 value_units(u32 bits, u32 pos_lo) {
    const u32 mb = bits & 0x7fffffffu, e = mb >> 23;
    const u64 d = mb ? (u64)((mb & 0x7fffffu) | (e ? 0x800000u : 0u)) << (bit_pos(mb) - pos_lo) : 0ull;
    return (bits >> 31) ? (u64)0 - d : d;
}

template <u32 THREADS, u32 STAGE>
struct CellsShared {
    float stage[STAGE];                                    // values on their way back
    u64 sum[512];
    u32 cnt[512];
    u32 wave_cnt[8];
    u64 wave_sum[8];
    u32 most;
};
// A bucket of at most THREADS x PER values.
template <u32 THREADS, u32 STAGE, u32 PER>
__device__ __forceinline__ void cells_of_bucket(EXCP_GLOBAL float *part, u32 size, u32 kmin, u32 kmax, u32 mag, u32 *info, u32 *begin, u64 *above, CellsShared<THREADS, STAGE> &A) {
    const u32 tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6, pos_lo = bit_pos(mag);
    float v[PER];
#pragma unroll
    for (u32 j = 0; j < PER; ++j) v[j] = j * THREADS + tid < size ? part[j * THREADS + tid] : 0.f;
    const u32 lg = excp_fine_cells_log2(size);
    const CellMap map = excp_cell_map(kmin, kmax, mag, lg);
    if (tid < 512u) { A.cnt[tid] = 0; A.sum[tid] = 0; }
    if (tid == 0) A.most = 0;
    __syncthreads();
    auto cell_in = [&](float x) { return excp_cell_of_bits(map, f2u(x)); };
    // Where the bucket spans eight binary orders and has values of one sign and no zero, as nearly all do, a cell's sum of
    // magnitudes (24 + 8 + 16 bits) and its number of values share a word and an atomic.
    const bool near = bit_pos(max(f2u(val_of(kmin)) & 0x7fffffffu, f2u(val_of(kmax)) & 0x7fffffffu)) - pos_lo <= NEAR_SPAN, packed = near && !map.gap;
    u32 place[PER / 2u];                                   // arrivals in the cells, then places in the bucket, two to a register
#pragma unroll
    for (u32 j = 0; j < PER; ++j) {
        if (j % 2u == 0u) place[j / 2u] = 0;
        asm volatile("" : "+v"(v[j]));
        if (j * THREADS + tid < size) {
            const u32 cell = cell_in(v[j]);
            if (packed) {
                place[j / 2u] |= (u32)(atomicAdd(&A.sum[cell], value_units(f2u(v[j]) & 0x7fffffffu, pos_lo) | 1ull << 48) >> 48) << (16u * (j % 2u));
            } else {
                place[j / 2u] |= atomicAdd(&A.cnt[cell], 1u) << (16u * (j % 2u));
                atomicAdd(&A.sum[cell], value_units(f2u(v[j]), pos_lo));
            }
        }
        if (j % 2u == 1u) asm volatile("" : "+v"(place[j / 2u]));
    }
    __syncthreads();
    u32 cnt = 0, incl = 0;
    u64 incls = 0;
    if (tid < 512u) {
        u64 sum = A.sum[tid];
        cnt = A.cnt[tid];
        if (packed) { cnt = (u32)(sum >> 48); sum &= (1ull << 48) - 1ull; if (kmin < 0x80000000u) sum = (u64)0 - sum; }
        incl = wave_incl_scan_u32(cnt); incls = wave_incl_scan_u64(sum);
        const u32 most = wave_max_u32(cnt);
        if (lane == 63u) { A.wave_cnt[wave] = incl; A.wave_sum[wave] = incls; atomicMax(&A.most, most); }
    }
    __syncthreads();
    if (!near && A.most > FAR_MOST) {                      // (the same in the whole workgroup)
        if (tid == 0) *info = 0u;
        return;
    }
    if (tid < 512u) {
        u64 all = 0;
#pragma unroll
        for (u32 q = 0; q < 8; ++q) { if (q < wave) { incl += A.wave_cnt[q]; incls += A.wave_sum[q]; } all += A.wave_sum[q]; }
        A.cnt[tid] = incl - cnt;
        if (tid < 1u << lg) { begin[tid] = incl - cnt; above[tid] = all - incls; }
        if (tid == 0) { begin[1u << lg] = size; *info = FINE_VALID | (near ? FINE_NEAR : 0u) | lg | map.shift << 4 | A.most << 9; }
    }
    __syncthreads();
#pragma unroll
    for (u32 j = 0; j < PER; ++j) {
        // (past the end: a place that no round has, as the largest bucket is smaller.  The cell is worked out again: kept, the
        // forty-eight of them would not fit the registers.)
        asm volatile("" : "+v"(v[j]));
        const u32 to = j * THREADS + tid < size ? A.cnt[cell_in(v[j])] : 0xffffu;
        place[j / 2u] += to << (16u * (j % 2u));
        if (j % 2u == 1u) asm volatile("" : "+v"(place[j / 2u]));
    }
#pragma unroll 1
    for (u32 r0 = 0; r0 < size; r0 += STAGE) {
        if (r0) __syncthreads();
#pragma unroll
        for (u32 j = 0; j < PER; ++j) {
            const u32 to = (place[j / 2u] >> (16u * (j % 2u)) & 0xffffu) - r0;
            if (to < STAGE) A.stage[to] = v[j];
        }
        __syncthreads();
        const u32 n = min(size - r0, STAGE);
        for (u32 i = tid; i < n; i += THREADS) part[r0 + i] = A.stage[i];
    }
}

template <u32 THREADS, u32 MOST, u32 STAGE>
__global__ __launch_bounds__(THREADS) void k_km_cells(Workspace w, GroupParams g) {
    __shared__ CellsShared<THREADS, STAGE> A;
    const u32 sidx = stream_in_turn(w, blockIdx.x / NBKT), b = blockIdx.x % NBKT, tid = threadIdx.x, t = sidx / 3u;
    if (w.seg[sidx].len == 0) return;
    const u32 at = sidx * NBKT + b;
    const EXCP_CONSTANT u32 *ends = (const EXCP_CONSTANT u32 *)(uintptr_t)(w.km_begin + (u64)sidx * (NBKT + 1u));
    const u32 q0 = ends[b], size = ends[b + 1u] - q0;
    const u32 kmin = w.km_min[at], kmax = w.km_max[at], mag = w.km_mag[at];
    const u32 top = max(f2u(val_of(kmin)) & 0x7fffffffu, f2u(val_of(kmax)) & 0x7fffffffu);
    static_assert(MOST / STAGE * STAGE == MOST && MOST < 0xffffu, "places have 16 bits");
    // (the values of a crowded stream are not spread by keys either, and the many workgroups that share its iterations would meet at
    // the same centres if its buckets were in order: 300 000 residuals of a sign-like update, 8 bits, 386 -> 821 us)
    if (size < FINE_LEAST || size > MOST || kmin >= kmax || *w.no_cells || w.seg[sidx].crowded || bit_pos(top) - bit_pos(mag) > FINE_SPAN) {
        if (tid == 0) w.km_fine[at] = 0u;
        return;
    }
    const u64 e = (u64)(sidx % 3u) * w.fine_stride + excp_fine_at(w.desc[t].elem_off, t, q0, b);
    EXCP_GLOBAL float *part = gptr(seg_part(w, sidx)) + q0;
    // (registers by the size of the bucket: with those of the largest for all of them, the 5000 values of a moment bucket
    // took as long as the 22 700 of a residual one)
#define EXCP_CELLS(PER) cells_of_bucket<THREADS, STAGE, PER>(part, size, kmin, kmax, mag, &w.km_fine[at], &w.fine_begin[e], &w.fine_above[e], A)
    if (size <= 2u * THREADS) EXCP_CELLS(2);
    else if (size <= 6u * THREADS) EXCP_CELLS(6);
    else if (size <= 16u * THREADS) EXCP_CELLS(16);
    else if (MOST > 16u * THREADS) {
        if (size <= 24u * THREADS) EXCP_CELLS(24);
        else if (size <= 40u * THREADS) EXCP_CELLS(40);
        else if (MOST > 40u * THREADS) {
            if (size <= 56u * THREADS) EXCP_CELLS(56);
            else if (size <= 76u * THREADS) EXCP_CELLS(76);
            else EXCP_CELLS(MOST / THREADS);
        }
    }
#undef EXCP_CELLS
}

// ---------------------------------------------------------------- P5: initial centres, bucket prefix sums
// Per stream K workgroups, one per initial centre, and one that makes the prefix sums of the bucket totals.
//
// A centre: radix select inside the bucket that holds its rank, 11 bits a digit (the bits that the bucket's
// smallest and largest key share are known and skipped), the digit's histogram scanned by the whole
// workgroup.  Values that fit the workgroup's registers are read once.
// (1024 threads for the residuals of 16-bit weights -- a bucket of tied values can be most of a stream -- for
// groups with a tensor of 2^28 elements, whose buckets' repetitions have been counted as well (TIED), and for few large tensors; 256 otherwise: with 1024 for everybody the 14 000 workgroups of a 410M-shaped
// checkpoint took 347 us instead of 167, and 22 instead of 33 for a 16.8 M-element tensor)
//
// The prefix sums turn the total of any run of buckets into one difference; the workgroup that makes them also decides
// how the stream goes through the Lloyd iterations, and the workgroup of centre k clears its share of their accumulators.
// The cells of bucket `at` as a Lloyd iteration sees them: those of its table, one (the bucket itself) where it has few
// values, or 0.  `span`: binary orders between its values.
__device__ __forceinline__ u32 fine_info(const Workspace &w, const GroupParams &g, u32 sidx, u32 at, u32 size, u32 span) {
    if (size < FINE_LEAST) return span <= FINE_SPAN ? FINE_VALID | (span <= NEAR_SPAN ? FINE_NEAR : 0u) | size << 9 : 0u;
    return g.fine && excp_fine_tensor(w.desc[sidx / 3u].n) ? w.km_fine[at] : 0u;
}
constexpr u32 FINE_COST = 24;                             // a value of a cell, which sixteen lanes read, in SegState::work

template <u32 INIT_THREADS, bool TIED>
__global__ __launch_bounds__(INIT_THREADS) void k_km_init(Workspace w, GroupParams g, u32 sel) {
    __shared__ __attribute__((aligned(16))) u32 hist[2048];
    __shared__ u32 s_wave[INIT_THREADS / 64], s_pick[2];
    const u32 K = (u32)g.K;
    const u32 sidx = stream_in_turn(w, stream_of(blockIdx.x / (K + 1u), sel)), k = blockIdx.x % (K + 1u), tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    SegState &S = w.seg[sidx];
    const u64 len = S.len;
    const u32 slot = ((const EXCP_CONSTANT TDesc *)(uintptr_t)(w.desc + sidx / 3u))->acc_slot;
    if (len == 0) return;
    if (k == K) {
        // a wave takes a bin: four consecutive buckets per lane
        u64 *bs = w.km_bsum + (u64)sidx * EXCP_ABSM_BINS * (NBKT + 1);
        __shared__ u32 s_whole, s_cell;
        if (tid < 2) { s_pick[tid] = tid ? 0u : 64u; s_wave[tid] = tid ? 0u : 255u; s_wave[2] = 0u; s_whole = 0u; s_cell = 0u; }
        __syncthreads();
        if (tid < NBKT) {                      // lowest and highest bit position of any value, largest bucket of several
            const u32 at = sidx * NBKT + tid, kn = w.km_min[at], kx = w.km_max[at], low = w.km_mag[at];
            const u32 b0 = w.km_begin[sidx * (NBKT + 1u) + tid], b1 = w.km_begin[sidx * (NBKT + 1u) + tid + 1u];
            // (of tied data: what is not a repetition of the bucket's first value; a bucket of one value is never cut)
            const u32 most = b1 - b0 - (TIED ? w.km_dom[at] : 0u);
            const bool any = kn <= kx;         // (an empty bucket has no extremes)
            const u32 a = f2u(val_of(kn)) & 0x7fffffffu, c = f2u(val_of(kx)) & 0x7fffffffu;
            // a border in a bucket with cells costs a cell, in another the bucket
            const u32 info = fine_info(w, g, sidx, at, b1 - b0, any ? bit_pos(max(a, c)) - bit_pos(low) : 0u);
            const u32 whole = info ? 0u : b1 - b0, ps = wave_sum_u32(whole), pc = wave_max_u32(kn < kx && info ? fine_most(info) : 0u);
            // (reduced in the wave first: an atomic whose lanes differ is a loop over them: three of those, 3000 streams 476 us, now 329)
            const u32 p0 = wave_min_u32(any ? bit_pos(low) : 255u), p1 = wave_max_u32(any ? bit_pos(max(a, c)) : 0u), p2 = wave_max_u32(kn < kx && !info ? most : 0u);
            if (lane == 0u) { atomicMin(&s_wave[0], p0); atomicMax(&s_wave[1], p1); atomicMax(&s_wave[2], p2); atomicAdd(&s_whole, ps); atomicMax(&s_cell, pc); }
        }
        for (u32 bin = wave; bin < EXCP_ABSM_BINS; bin += INIT_THREADS / 64u) {
            u64 *row = bs + (u64)bin * (NBKT + 1);
            u64 v[4], sum = 0;
#pragma unroll
            for (u32 q = 0; q < 4; ++q) { v[q] = row[4u * lane + q]; sum += v[q]; }
            if (!__any((v[0] | v[1] | v[2] | v[3]) != 0ull)) {      // nothing in this bin: it is its own prefix sum
                if (lane == 63u) row[NBKT] = 0;
                continue;
            }
            const u64 incl = wave_incl_scan_u64(sum);
            u64 run = incl - sum;
#pragma unroll
            for (u32 q = 0; q < 4; ++q) { row[4u * lane + q] = run; run += v[q]; }
            if (lane == 63u) { row[NBKT] = run; atomicMin(&s_pick[0], bin); atomicMax(&s_pick[1], bin); }
        }
        __syncthreads();
        if (tid == 0) {
            S.bin_lo = s_pick[0]; S.bin_hi = s_pick[1];
            // (windows begin up to 19 positions below a value, and sums reach up to 64 positions above one)
            S.acc_lo = s_wave[0] > 19u ? (s_wave[0] - 19u) >> 3 : 0u;
            S.acc_hi = min(s_wave[1] / 8u + 9u, EXCP_ABSM_BINS - 1u);
            // one workgroup or many (see P6)
            const u64 even = ((u64)s_whole * (K - 1u)) / NBKT, crowded = (u64)s_wave[2] * (K > 3u && (!g.fine || (u64)s_wave[2] > 3ull * (len / NBKT + 1ull)) ? 8u : 1u), cells = (u64)s_cell * FINE_COST;
            S.work = (u32)min(max(max(even, crowded), cells), 0xffffffffull);
            if (S.work > g.alone_work && slot != EXCP_NO_SLOT) {
                atomicOr(&w.st[sidx / 3u].lloyd_shared, 1u);
                atomicOr(w.lloyd_shared, 1u);
            }
        }
        return;
    }
    {
        constexpr u32 SHARE = 3u * (EXCP_ABSM_BINS + 1u);
        if (slot != EXCP_NO_SLOT && tid < SHARE) w.km_acc[((3ull * slot + sidx % 3u) * K + k) * SHARE + tid] = 0;
    }
    const u32 *begin = w.km_begin + (u64)sidx * (NBKT + 1);
    const u32 r = (u32)(((u64)(2 * k + 1) * len) / (2ull * K));
    // the bucket that holds the rank: begin[b] <= r < begin[b + 1] (empty buckets repeat an entry)
    if (tid < NBKT) { if (begin[tid] <= r && r < begin[tid + 1]) s_pick[0] = tid; }
    __syncthreads();
    // (the same in every lane, and through the scalar unit: left to the compiler, whether it is depends on stores nearby)
    const u32 b = (u32)__builtin_amdgcn_readfirstlane((int)s_pick[0]);
    const EXCP_CONSTANT u32 *ends = (const EXCP_CONSTANT u32 *)(uintptr_t)begin;
    u32 p0 = ends[b], cntb = ends[b + 1] - p0, rank = r - p0;
    const u32 kmin = ((const EXCP_CONSTANT u32 *)(uintptr_t)w.km_min)[(u64)sidx * NBKT + b], kmax = ((const EXCP_CONSTANT u32 *)(uintptr_t)w.km_max)[(u64)sidx * NBKT + b];
    u32 diff = kmin ^ kmax;
    float *out = &S.C[1][k];                 // (read by iteration 0, whose predecessor has parity 1)
    if (diff == 0) { if (tid == 0) *out = val_of(kmin); return; }
    // Tied data: the rank usually falls among the repetitions of the bucket's first value, which have been counted.
    // (The K ranks of a stream often ask for the same few large buckets: reading those for each of them took most
    // of this kernel's time: a 410M-shaped checkpoint in bf16 468 us, 164 now.)
    // (k_km_cells moves values within a bucket: the first one is no longer the one that was counted where it has run.)
    const u32 info = g.fine && excp_fine_tensor(((const EXCP_CONSTANT TDesc *)(uintptr_t)(w.desc + sidx / 3u))->n)
                         ? ((const EXCP_CONSTANT u32 *)(uintptr_t)w.km_fine)[(u64)sidx * NBKT + b] : 0u;
    if (TIED && !info && rank - w.km_less[(u64)sidx * NBKT + b] < w.km_dom[(u64)sidx * NBKT + b]) { if (tid == 0) *out = gptr(seg_part(w, sidx))[p0]; return; }
    if (info) {                                           // the cell that holds the rank
        __shared__ u32 s_ends[2];                         // (not s_pick: a wave may still have to read the bucket from there)
        const u64 e = (u64)(sidx % 3u) * w.fine_stride + excp_fine_at(w.desc[sidx / 3u].elem_off, sidx / 3u, p0, b);
        for (u32 c = tid; c < 1u << fine_log2(info); c += INIT_THREADS) {
            const u32 c0 = w.fine_begin[e + c], c1 = w.fine_begin[e + c + 1u];
            if (c0 <= rank && rank < c1) { s_ends[0] = c0; s_ends[1] = c1; }
        }
        __syncthreads();
        const u32 c0 = (u32)__builtin_amdgcn_readfirstlane((int)s_ends[0]), c1 = (u32)__builtin_amdgcn_readfirstlane((int)s_ends[1]);
        p0 += c0; cntb = c1 - c0; rank -= c0;
    }
    const EXCP_GLOBAL float *gpart = gptr(seg_part(w, sidx)) + p0;
    if (cntb <= 256u) {
        // few values: each counts those before it in the order
        const u32 mine = tid < cntb ? key_of(gpart[tid]) : 0xffffffffu;
        if (tid < 256u) hist[tid] = mine;
        __syncthreads();
        if (tid < cntb) {
            u32 less = 0;
            typedef u32 u4 __attribute__((ext_vector_type(4)));
#pragma unroll 2
            for (u32 j = 0; j < cntb; j += 4u) {
                const u4 o = *(const u4 *)&hist[j];
#pragma unroll
                for (u32 e = 0; e < 4; ++e) less += (o[e] < mine || (o[e] == mine && j + e < tid)) ? 1u : 0u;
            }
            if (less == rank) *out = val_of(mine);
        }
        return;
    }
    // A bucket far above the average size holds tied values (a continuous distribution fills the
    // buckets evenly).  Such a bucket is mostly ONE value, its smallest or its largest key, with a few
    // strays beside it: one cheap pass counts the two extremes, and if the rank falls among them the
    // answer is known without any digit-by-digit selection.
    const bool crowded = (u64)cntb > 3ull * (len / NBKT + 1ull);
    if (crowded) {
        __shared__ u32 s_ext[2];
        if (tid == 0) { s_ext[0] = 0u; s_ext[1] = 0u; }
        __syncthreads();
        u32 c_lo = 0, c_hi = 0;
        for (u32 q0 = 0; q0 < cntb; q0 += 16u * INIT_THREADS) {
            if (q0 + 16u * INIT_THREADS <= cntb) {
                f4u q[4];
#pragma unroll
                for (u32 j = 0; j < 4; ++j) q[j] = *(const EXCP_GLOBAL f4u *)(gpart + q0 + (j * INIT_THREADS + tid) * 4u);
#pragma unroll
                for (u32 j = 0; j < 4; ++j) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const u32 key = key_of(q[j][e]);
                        c_lo += key == kmin; c_hi += key == kmax;
                    }
                }
            } else {
                for (u32 p = q0 + tid; p < cntb; p += INIT_THREADS) {
                    const u32 key = key_of(gpart[p]);
                    c_lo += key == kmin; c_hi += key == kmax;
                }
            }
        }
        c_lo = wave_sum_u32(c_lo); c_hi = wave_sum_u32(c_hi);
        if (lane == 0u) { atomicAdd(&s_ext[0], c_lo); atomicAdd(&s_ext[1], c_hi); }
        __syncthreads();
        if (rank < s_ext[0]) { if (tid == 0) *out = val_of(kmin); return; }
        if (rank >= cntb - s_ext[1]) { if (tid == 0) *out = val_of(kmax); return; }
    }
    const u32 hb = 31u - (u32)__clz((int)diff);           // highest bit in which keys of this bucket differ
    u32 prefix = hb == 31u ? 0u : kmin >> (hb + 1u);
    int top = (int)hb;                                    // bits [0, top] still unknown
    const bool once = cntb <= 16u * INIT_THREADS;         // all of it in registers
    u32 held[16];
    if (once) {
#pragma unroll
        for (u32 j = 0; j < 16; ++j) { const u32 p = j * INIT_THREADS + tid; held[j] = p < cntb ? key_of(gpart[p]) : 0u; }
    }
    while (top >= 0) {
        const u32 width = top + 1 < 11 ? (u32)top + 1u : 11u, shift = (u32)top + 1u - width;
        for (u32 i = tid; i < 2048u; i += INIT_THREADS) hist[i] = 0;
        __syncthreads();
        // (in a crowded bucket the lanes mostly hit the same bin: the increments are grouped per wave)
        auto tally = [&](u32 key, bool in) {
            const bool match = in && ((top == 31) ? true : ((key >> (top + 1)) == prefix));
            const u32 bin = (key >> shift) & ((1u << width) - 1u);
            if (crowded) hist_add_tied(hist, bin, match);
            else if (match) atomicAdd(&hist[bin], 1u);
        };
        if (once) {
#pragma unroll
            for (u32 j = 0; j < 16; ++j) if (j * INIT_THREADS < cntb) tally(held[j], j * INIT_THREADS + tid < cntb);
        } else {
            // sixteen values per thread and round, every load of a round issued before its use
            for (u32 q0 = 0; q0 < cntb; q0 += 16u * INIT_THREADS) {
                if (q0 + 16u * INIT_THREADS <= cntb) {
                    f4u q[4];
#pragma unroll
                    for (u32 j = 0; j < 4; ++j) q[j] = *(const EXCP_GLOBAL f4u *)(gpart + q0 + (j * INIT_THREADS + tid) * 4u);
#pragma unroll
                    for (u32 j = 0; j < 4; ++j) {
#pragma unroll
                        for (int e = 0; e < 4; ++e) tally(key_of(q[j][e]), true);
                    }
                } else {
                    u32 x[16];
#pragma unroll
                    for (u32 j = 0; j < 16; ++j) { const u32 p = q0 + j * INIT_THREADS + tid; x[j] = p < cntb ? key_of(gpart[p]) : 0u; }
#pragma unroll
                    for (u32 j = 0; j < 16; ++j) if (q0 + j * INIT_THREADS < cntb) tally(x[j], q0 + j * INIT_THREADS + tid < cntb);
                }
            }
        }
        __syncthreads();
        constexpr u32 PER = 2048u / INIT_THREADS;
        u32 c[PER], local = 0;
#pragma unroll
        for (u32 i = 0; i < PER; ++i) { c[i] = hist[tid * PER + i]; local += c[i]; }
        u32 incl = wave_incl_scan_u32(local);
        if (lane == 63u) s_wave[wave] = incl;
        __syncthreads();
        u32 before = incl - local;
        for (u32 q = 0; q < wave; ++q) before += s_wave[q];
        if (rank >= before && rank < before + local) {                  // exactly one thread
            u32 rr = rank - before, i = 0;
#pragma unroll
            for (u32 q = 0; q + 1u < PER; ++q) if (i == q && rr >= c[q]) { rr -= c[q]; ++i; }
            s_pick[0] = tid * PER + i; s_pick[1] = rr;
        }
        __syncthreads();
        prefix = (prefix << width) | s_pick[0];
        rank = s_pick[1];
        top = (int)shift - 1;
    }
    if (tid == 0) *out = val_of(prefix);
}

// ---------------------------------------------------------------- P6: Lloyd iterations
// An iteration assigns every value to its nearest centre and adds it, exactly, to that centre's total -- where a
// cluster border cuts a bucket by reading the bucket, and otherwise not at all: the buckets lying wholly in a
// centre's cell are one difference of prefix sums.  What it costs is the chain of dependent steps (centres from
// totals, cut keys, which buckets are cut, their values, sums), so a stream goes through it in one of two ways:
//
//   one workgroup per stream, all iterations in one launch (k_km_lloyd): no launch gaps, totals in LDS;
//   one launch per iteration, many workgroups per stream (k_km_iter), where the cut buckets hold so many values that
//   one compute unit would read them for longer than a launch takes.
//
// What decides is the number of values that an iteration is expected to read (SegState::work, from the filled buckets): K - 1
// even shares of 256, or the largest bucket that holds more than one value, if that is more.  The values of a crowded
// bucket (residuals of a sign-like update, values bunched beside outliers) count eight times from four centres on, since
// most centres then lie in that bucket, and its values go one by one; of tied data only what is not a repetition of a
// bucket's first value counts.  A tensor's streams go the same way, unless buckets have cells; then each by itself, buckets
// with cells count by their largest cell, and the line lies at 98 304 (one bucket of 50 000 values without cells costs an
// iteration 8 us, a launch 14).  The host launches the iterations of the second way wherever a tensor is too large for
// excp_lloyd_small; where no stream takes it they are empty.  (2^17 elements: one workgroup needs 0.43 ms for 130 000 residuals
// of a sign-like update, the former work lists needed 0.81; 2^22 for three centres, of whose borders a bucket holds two at most.)
//   Without cells (excp_cells_group), up to 85 tensors on 256 compute units go together, the line at 24 576.  (One tensor, ten
//   iterations, us alone / shared: 4 bits, 500 000 elements 152 / 181, 1.5 M 174 / 190, 2.5 M 194 / 178, 10 M 343 / 172; 8 bits,
//   300 000 elements 834 / 750, 1 M 1056 / 227, 10 M 4020 / 222.)
//   More tensors fill the GPU as they are, one workgroup a stream, and the line lies at 196 608 (4 bits: 300 tensors of 600 000
//   elements 289 alone, 536 shared; the 410M shape 312, 326 with the line at 65 536, 1207 all alone, 285 all shared), from six bits
//   on at 131 072 (7 bits: 300 tensors of 600 000 elements 1531 alone, 2498 shared; the 410M shape 1494, 1604 with the line at
//   196 608, 9501 all alone).
//   Not in the rule: how the values of a crowded bucket are spread.  A 410M shape of bunched values, all kept, is the one
//   input met that the former work lists took through these iterations faster (2.0 against 2.7 ms each; the call 116 and 113).
constexpr u32 LLOYD_THREADS = 512, LLOYD_WAVES = LLOYD_THREADS / 64;
constexpr u32 LLOYD_FEW = 4 * LLOYD_THREADS;              // up to here a value per thread is quicker than a bucket per wave

// Workgroups of the form for up to KMAX centres that a compute unit holds, and values in cut buckets that are worth one
// (more centres, more borders to a bucket: 5 bits, 1.5 M elements 236 us with 8192, 169 with 4096).
constexpr u32 lloyd_per_cu(u32 KMAX) { return KMAX > 63u ? 1u : 2u; }        // (two waves per SIMD each)
constexpr u32 lloyd_unit(u32 KMAX) { return KMAX > 15u ? 4096u : 8192u; }

// Whether many workgroups take the stream's iterations.
__device__ __forceinline__ bool lloyd_shared(const Workspace &w, const GroupParams &g, u32 sidx) {
    if (g.fine) return w.seg[sidx].work > g.alone_work;
    return (g.together ? *w.lloyd_shared : w.st[sidx / 3u].lloyd_shared) != 0u;
}

struct LloydShared {
    float C[EXCP_MAX_K + 1], fresh[EXCP_MAX_K + 1];
    u32 cut[EXCP_MAX_K + 1];
    u32 first[EXCP_MAX_K + 1], last[EXCP_MAX_K + 1];      // per centre: the buckets whose smallest value goes to it
    u32 begin[NBKT + 1];                                  // first position of every bucket
    u32 off[NBKT + 1];                                    // cut buckets back to back: first place of every bucket
    u32 range[NBKT];                                      // per bucket: centres at its two ends, lowest and highest bit position
                                                          // (alo | ahi << 8 | pos_lo << 16 | pos_hi << 24)
    u32 wave[4];
    u32 unsorted;
};

// A stream as a workgroup keeps it through an iteration: thread b < 256 owns bucket b (its extremes, and the
// positions of its smallest non-zero and its largest magnitude: lo | hi << 8).
struct LloydStream { u32 kmin, kmax, pos, alo, acc_lo, acc_hi, bin_lo, bin_hi; const u64 *bs; };

// `slot`: the parity of the centres (and, with cuts, the cut keys) to begin with.  All loads first, then LDS.
__device__ __forceinline__ LloydStream lloyd_open(const Workspace &w, u32 sidx, u32 K, u32 slot, bool cuts, LloydShared &L) {
    const u32 tid = threadIdx.x;
    const SegState &S = w.seg[sidx];
    LloydStream st;
    st.bs = w.km_bsum + (u64)sidx * EXCP_ABSM_BINS * (NBKT + 1);
    const u32 b = min(tid, NBKT - 1u);
    const u32 *begin = w.km_begin + (u64)sidx * (NBKT + 1);
    st.kmin = w.km_min[(u64)sidx * NBKT + b]; st.kmax = w.km_max[(u64)sidx * NBKT + b];
    const u32 b0 = begin[b], b1 = begin[b + 1u], mag = w.km_mag[(u64)sidx * NBKT + b];
    const float c = S.C[slot][b];
    const u32 cut = S.cut[slot][b];
    st.acc_lo = (u32)__builtin_amdgcn_readfirstlane((int)S.acc_lo); st.acc_hi = (u32)__builtin_amdgcn_readfirstlane((int)S.acc_hi);
    st.bin_lo = (u32)__builtin_amdgcn_readfirstlane((int)S.bin_lo); st.bin_hi = (u32)__builtin_amdgcn_readfirstlane((int)S.bin_hi);
    st.alo = 0; st.pos = 0;
    if (tid < NBKT) {
        L.begin[tid] = b0;
        if (tid == NBKT - 1u) L.begin[NBKT] = b1;
        if (tid < K) L.C[tid] = c;
        if (cuts) L.cut[tid] = cut;
        if (b1 > b0) {
            const u32 a = f2u(val_of(st.kmin)) & 0x7fffffffu, z = f2u(val_of(st.kmax)) & 0x7fffffffu;
            st.pos = bit_pos(mag) | (bit_pos(max(a, z)) << 8);
        }
    }
    return st;
}

// The accumulators' bins that the stream can use, and the counts, set to zero.
__device__ __forceinline__ void lloyd_clear(u64 *acc, const LloydStream &st, u32 K) {
    for (u32 j = st.acc_lo * K + threadIdx.x; j < (st.acc_hi + 1u) * K; j += LLOYD_THREADS) acc[j] = 0;
    if (threadIdx.x < K) acc[EXCP_ABSM_BINS * K + threadIdx.x] = 0;
}

// Centres and cut keys of iteration i from L.C and, for i >= 1, st.alo (the centre that the smallest value of
// the thread's bucket went to in iteration i - 1) and `acc` (LDS, [bin][K], then [K] counts: what iteration i - 1 moved
// between centres).  A bucket counts wholly for its alo -- one difference of prefix sums for all of a centre's
// buckets -- and the values of a cut bucket above a border are moved on by acc.  Thread k owns centre k.
// An empty cluster keeps its centre; afterwards the centres are put back in ascending order (stable; nothing
// moves unless a run of equal centres was torn apart: the lowest of them takes all their members and may pass
// the ones left behind).  Begins and ends with a barrier.
__device__ __forceinline__ void lloyd_centres(const LloydStream &st, u32 K, u32 i, u64 *acc, LloydShared &L) {
    const u32 tid = threadIdx.x, g0 = st.bin_lo, g1 = st.bin_hi, alo = st.alo;
    const u64 *bs = st.bs;
    __syncthreads();
    if (i > 0u) {
        if (tid < K) { L.first[tid] = 0xffffffffu; L.last[tid] = 0u; }
        if (tid == 0) L.unsorted = 0u;
        __syncthreads();
        if (tid < NBKT && L.begin[tid + 1u] > L.begin[tid]) { atomicMin(&L.first[alo], tid); atomicMax(&L.last[alo], tid); }
        __syncthreads();
        if (g0 <= g1) {
            for (u32 j = tid; j < (g1 - g0 + 1u) * K; j += LLOYD_THREADS) {
                const u32 q = g0 + j / K, k = j % K;
                const u32 f = L.first[k], l = L.last[k] + 1u;
                if (f < l) acc[q * K + k] += bs[q * (NBKT + 1u) + l] - bs[q * (NBKT + 1u) + f];
            }
        }
        __syncthreads();
        float c = 0.f;
        if (tid < K) {
            c = L.C[tid];
            const u32 f = L.first[tid], l = L.last[tid] + 1u;      // (first = 2^32 - 1: no bucket)
            u64 cnt = acc[EXCP_ABSM_BINS * K + tid];
            if (f < l) cnt += L.begin[l] - L.begin[f];
            if (cnt) c = (float)(signed_bins_to_double(acc + tid, K, st.acc_lo, st.acc_hi) / (double)cnt);
            L.fresh[tid] = c;
        }
        __syncthreads();
        if (tid + 1u < K && !(c <= L.fresh[tid + 1u])) L.unsorted = 1u;
        lloyd_clear(acc, st, K);
        __syncthreads();
        u32 rank = tid;
        if (L.unsorted && tid < K) {
            rank = 0;
#pragma unroll 1
            for (u32 j = 0; j < K; ++j) {
                const float cj = L.fresh[j];
                rank += (cj < c || (cj == c && j < tid)) ? 1u : 0u;
            }
        }
        if (tid < K) L.C[rank] = c;
        __syncthreads();
    }
    compute_cut_keys(L.C, (int)K, L.cut);
    __syncthreads();
}

// Which buckets the present cut keys cut, laid back to back; returns how many values those hold.  `fine`: those with cells are
// left out.
__device__ __forceinline__ u32 lloyd_cut_buckets(LloydStream &st, u32 kp2, LloydShared &L, const u32 *fine) {
    const u32 tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    u32 size = 0, incl = 0;
    if (tid < NBKT) {
        const u32 cntb = L.begin[tid + 1u] - L.begin[tid];
        u32 alo = 0, ahi = 0;
        if (cntb) { alo = centre_by_cuts(L.cut, kp2, st.kmin); ahi = centre_by_cuts(L.cut, kp2, st.kmax); }
        if (alo != ahi && !(fine && fine[tid])) size = cntb;
        st.alo = alo;
        L.range[tid] = alo | (ahi << 8) | (st.pos << 16);
        incl = wave_incl_scan_u32(size);
        if (lane == 63u) L.wave[wave] = incl;
    }
    __syncthreads();
    if (tid < NBKT) {
        u32 before = incl - size;
        for (u32 v = 0; v < wave; ++v) before += L.wave[v];
        L.off[tid] = before;
        if (tid == NBKT - 1u) L.off[NBKT] = before + size;
    }
    __syncthreads();
    return L.off[NBKT];
}

// The same for a whole workgroup and few values (places [x0, x1), some per thread): every thread looks its value's bucket up.
__device__ __forceinline__ void lloyd_few(const EXCP_GLOBAL float *part, u32 x0, u32 x1, u32 K, u32 kp2, u64 *acc, const LloydShared &L) {
    for (u32 q = x0 + threadIdx.x; q < x1; q += LLOYD_THREADS) {
        u32 b = 0;
#pragma unroll
        for (u32 step = NBKT / 2; step >= 1u; step >>= 1) if (L.off[b + step] <= q) b += step;
        const u32 bits = f2u(part[L.begin[b] + (q - L.off[b])]), mb = bits & 0x7fffffffu;
        const u32 c_lo = L.range[b] & 255u, cl = centre_by_cuts(L.cut, kp2, key_of(u2f(bits)));
        if (cl == c_lo) continue;
        const u32 e = mb >> 23, pb = bit_pos(mb);
        const u64 d = (u64)((mb & 0x7fffffu) | (e ? 0x800000u : 0u)) << (pb & 7u), dd = (bits >> 31) ? (u64)0 - d : d;
        atomicAdd(&acc[(pb >> 3) * K + cl], dd);
        atomicAdd(&acc[(pb >> 3) * K + c_lo], (u64)0 - dd);
        atomicAdd(&acc[EXCP_ABSM_BINS * K + cl], 1ull);
        atomicAdd(&acc[EXCP_ABSM_BINS * K + c_lo], ~0ull);
    }
}

__device__ __forceinline__ void lloyd_file(u64 *acc, u32 K, u32 cl, long long v, u32 bitpos) {      // v * 2^(bitpos - 149) onto cluster cl
    const bool neg = v < 0;
    const u64 mag = neg ? (u64)0 - (u64)v : (u64)v;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const u64 piece = (mag >> (32 * h)) & 0xffffffffull;
        const u32 p = bitpos + 32u * (u32)h;
        const u64 d = piece << (p & 7u);
        if (piece) atomicAdd(&acc[(p >> 3) * K + cl], neg ? (u64)0 - d : d);
    }
}

// One wave, values [p0, p1) of a bucket that one or two borders cut (centres c_lo .. c_lo + 1 or c_lo + 2): the sum
// and number of the values above each border.  Values compare with a border as floats: no border lies between -0
// and +0, which are equally far from any centre.
// WIDE = false: the bucket's magnitudes span at most eight binary orders.  A value is then a whole multiple below
// 2^32 of the unit 2^(pos_lo - 149), and the 2^21 values a piece may hold add exactly in fp64 in any order.
// WIDE = true: sixteen values at a time are added in a window of 24 positions below the largest magnitude (see
// WindowSum); values below it are filed one by one.
template <bool WIDE>
__device__ __forceinline__ void lloyd_borders(const EXCP_GLOBAL float *part, u32 p0, u32 p1, u32 c_lo, bool two, u32 pos_lo, u32 pos_hi, u32 K,
                                              u64 *acc, const LloydShared &L) {
    const u32 lane = lane_id();
    const float inf = __uint_as_float(0x7f800000u);
    const float t1 = val_of(L.cut[c_lo + 1u]), t2 = two ? val_of(L.cut[c_lo + 2u]) : inf;
    const u32 B = WIDE ? (pos_hi > 23u ? pos_hi - 23u : 0u) : pos_lo;
    u32 thr_lo, span;
    window_range(B, thr_lo, span);
    WindowSum S1, S2;
    u32 cnt1 = 0, cnt2 = 0;
    auto take = [&](float x) {
        const bool u1 = x >= t1;
        cnt1 += u1;
        if (!WIDE) {
            S1.part += (double)(u1 ? x : 0.f);
            if (two) { const bool u2 = x >= t2; cnt2 += u2; S2.part += (double)(u2 ? x : 0.f); }
        } else {
            const u32 bits = f2u(x), mb = bits & 0x7fffffffu;
            const bool in = mb - thr_lo < span, u2 = x >= t2;
            cnt2 += u2;
            S1.part += (double)(u1 && in ? x : 0.f);
            S2.part += (double)(u2 && in ? x : 0.f);
            if (u1 && !in && mb) {
                const u32 e = mb >> 23, pb = bit_pos(mb), cl = c_lo + (u2 ? 2u : 1u);
                const u64 d = (u64)((mb & 0x7fffffu) | (e ? 0x800000u : 0u)) << (pb & 7u), dd = (bits >> 31) ? (u64)0 - d : d;
                atomicAdd(&acc[(pb >> 3) * K + cl], dd);
                atomicAdd(&acc[(pb >> 3) * K + c_lo], (u64)0 - dd);
            }
        }
    };
    u32 p = p0;
    if (p + 1024u <= p1) {
        // four 16-byte loads in flight per lane, the next four asked for before these are used
        f4u nx[4];
#pragma unroll
        for (u32 j = 0; j < 4; ++j) nx[j] = *(const EXCP_GLOBAL f4u *)(part + p + j * 256u + lane * 4u);
#pragma unroll 1
        for (; p + 1024u <= p1; p += 1024u) {
            f4u q[4];
#pragma unroll
            for (u32 j = 0; j < 4; ++j) q[j] = nx[j];
            if (p + 2048u <= p1) {
#pragma unroll
                for (u32 j = 0; j < 4; ++j) nx[j] = *(const EXCP_GLOBAL f4u *)(part + p + 1024u + j * 256u + lane * 4u);
            }
#pragma unroll
            for (u32 j = 0; j < 4; ++j) { take(q[j].x); take(q[j].y); take(q[j].z); take(q[j].w); }
            if (WIDE) { S1.fold(B); S2.fold(B); }
        }
    }
    if (p < p1) {                                         // fewer than 1024 left: sixteen per lane at most, side by side
        float x[16];
#pragma unroll
        for (u32 j = 0; j < 16; ++j) if (p + j * 64u < p1) x[j] = p + j * 64u + lane < p1 ? part[p + j * 64u + lane] : -inf;
#pragma unroll
        for (u32 j = 0; j < 16; ++j) if (p + j * 64u < p1) take(x[j]);
        if (WIDE) { S1.fold(B); S2.fold(B); }
    }
    cnt1 = wave_sum_u32(cnt1); cnt2 = wave_sum_u32(cnt2);
    // lane j files what cluster c_lo + j receives
    const u32 n = lane == 0u ? 0u - cnt1 : (lane == 1u ? cnt1 - cnt2 : cnt2);
    if (!WIDE) {
        S1.part = wave_sum_f64(S1.part);
        if (two) S2.part = wave_sum_f64(S2.part);
        const long long m1 = (long long)ldexp(S1.part, 149 - (int)B), m2 = (long long)ldexp(S2.part, 149 - (int)B);
        const long long v = lane == 0u ? -m1 : (lane == 1u ? m1 - m2 : m2);
        if (lane < 3u && v) lloyd_file(acc, K, c_lo + lane, v, B);
    } else {
        const long long l1 = (long long)wave_sum_u64((u64)S1.lo), h1 = (long long)wave_sum_u64((u64)S1.hi);
        const long long l2 = (long long)wave_sum_u64((u64)S2.lo), h2 = (long long)wave_sum_u64((u64)S2.hi);
        const long long vl = lane == 0u ? -l1 : (lane == 1u ? l1 - l2 : l2), vh = lane == 0u ? -h1 : (lane == 1u ? h1 - h2 : h2);
        if (lane < 3u && vl) lloyd_file(acc, K, c_lo + lane, vl, B);
        if (lane < 3u && vh) lloyd_file(acc, K, c_lo + lane, vh, B + 32u);
    }
    if (lane < 3u && n) atomicAdd(&acc[EXCP_ABSM_BINS * K + c_lo + lane], (u64)(long long)(int)n);
}

// One wave, values [p0, p1) of a bucket that three or more borders cut: value by value.  Where the bucket spans at most
// seven binary orders a value is below 2^31 units of its lowest position; its centre's sum and number then share a
// word of the wave's own table (sum in the low 48 bits, number above), one LDS atomic a value instead of two, and what the
// centres received leaves c_lo when the table is emptied, every 8192 values at the latest.  (Atomics on LDS bound this:
// a 410M shape of bunched values, all kept, 3.8 -> 2.7 ms an iteration; ten of 9 M residuals of a sign-like update 251 ->
// 230 us.)  Elsewhere what leaves c_lo is kept per lane where the bucket spans at most 39 binary orders (in two 32-bit
// halves), because all lanes would queue at that one centre.
__device__ __forceinline__ void lloyd_many(const EXCP_GLOBAL float *part, u32 p0, u32 p1, u32 c_lo, u32 c_hi, u32 pos_lo, u32 pos_hi, u32 K,
                                           u64 *acc, u64 *mine, const LloydShared &L) {
    const u32 lane = lane_id();
    const bool near = pos_hi - pos_lo <= 39u, packed = pos_hi - pos_lo <= 7u;
    u32 top = 1; while (2u * top <= c_hi - c_lo) top <<= 1;
    if (packed) {
        for (u32 c = c_lo + 1u + lane; c <= c_hi; c += 64u) mine[c] = 0;
        wave_lds_fence();
    }
    long long outL = 0, outH = 0;
    u32 n_out = 0;
    // the wave's table goes to the centres, and as much leaves c_lo
    auto empty = [&]() {
        wave_lds_fence();
        for (u32 c = c_lo + 1u + lane; c <= c_hi; c += 64u) {
            const u64 word = mine[c];
            if (!word) continue;
            const long long sum = (long long)(word << 16) >> 16;
            const u32 n = (u32)((word - (u64)sum) >> 48);
            mine[c] = 0;
            if (sum) lloyd_file(acc, K, c, sum, pos_lo);
            atomicAdd(&acc[EXCP_ABSM_BINS * K + c], (u64)n);
            outL += sum; n_out += n;
        }
        wave_lds_fence();
    };
    u32 held = 0;                                         // values that may be in the table
#pragma unroll 1
    for (u32 p = p0; p < p1; p += 256u) {
        float x[4];
        u32 cl[4];
#pragma unroll
        for (u32 j = 0; j < 4; ++j) { const u32 at = p + j * 64u + lane; x[j] = at < p1 ? part[at] : 0.f; cl[j] = c_lo; }
#pragma unroll 1
        for (u32 step = top; step >= 1u; step >>= 1) {    // number of cut keys <= key, beginning at c_lo
#pragma unroll
            for (u32 j = 0; j < 4; ++j) { const u32 c = cl[j] + step; if (c <= c_hi && L.cut[c] <= key_of(x[j])) cl[j] = c; }
        }
        if (packed) {
            held += 256u;
            if (held > 8192u) { empty(); held = 256u; }
        }
#pragma unroll
        for (u32 j = 0; j < 4; ++j) {
            if (p + j * 64u + lane >= p1 || cl[j] == c_lo) continue;
            const u32 bits = f2u(x[j]), mb = bits & 0x7fffffffu;
            const u32 e = mb >> 23, pb = bit_pos(mb), mant = (mb & 0x7fffffu) | (e ? 0x800000u : 0u);
            const bool neg = bits >> 31;
            if (packed) {
                const u64 term = mant ? (u64)mant << (pb - pos_lo) : 0ull;
                atomicAdd(&mine[cl[j]], (neg ? (u64)0 - term : term) + (1ull << 48));
                continue;
            }
            ++n_out;
            atomicAdd(&acc[EXCP_ABSM_BINS * K + cl[j]], 1ull);
            if (!mant) continue;
            const u64 d = (u64)mant << (pb & 7u), dd = neg ? (u64)0 - d : d;
            atomicAdd(&acc[(pb >> 3) * K + cl[j]], dd);
            if (near) {
                const u64 term = (u64)mant << (pb - pos_lo);
                const long long tl = (long long)(term & 0xffffffffull), th = (long long)(term >> 32);
                outL += neg ? -tl : tl; outH += neg ? -th : th;
            } else {
                atomicAdd(&acc[(pb >> 3) * K + c_lo], (u64)0 - dd);
            }
        }
    }
    if (packed) empty();
    outL = (long long)wave_sum_u64((u64)outL); outH = (long long)wave_sum_u64((u64)outH);
    n_out = wave_sum_u32(n_out);
    if (lane == 0u && n_out) {
        if (outL) lloyd_file(acc, K, c_lo, -outL, pos_lo);
        if (outH) lloyd_file(acc, K, c_lo, -outH, pos_lo + 32u);
        atomicAdd(&acc[EXCP_ABSM_BINS * K + c_lo], (u64)0 - (u64)n_out);
    }
}

// One wave moves the values at places [q0, q1) of the cut buckets on to their centres in `acc` (LDS): the sum and
// number of the values above a border go from the centre below it to the one above it.
__device__ __forceinline__ void lloyd_share(const EXCP_GLOBAL float *part, u32 q0, u32 q1, u32 K, u64 *acc, u64 *mine, const LloydShared &L) {
    while (q0 < q1) {
        u32 b = 0;                                        // last bucket with off[b] <= q0: it holds place q0
#pragma unroll 1
        for (u32 step = NBKT / 2; step >= 1u; step >>= 1) if (L.off[b + step] <= q0) b += step;
        b = (u32)__builtin_amdgcn_readfirstlane((int)b);
        const u32 stop = min(q1, min(L.off[b + 1u], q0 + (1u << 21)));
        const u32 p0 = L.begin[b] + (q0 - L.off[b]), p1 = p0 + (stop - q0);
        const u32 r = (u32)__builtin_amdgcn_readfirstlane((int)L.range[b]);
        const u32 c_lo = r & 255u, c_hi = (r >> 8) & 255u, pos_lo = (r >> 16) & 255u, pos_hi = r >> 24;
        q0 = stop;
        if (c_hi - c_lo > 2u) lloyd_many(part, p0, p1, c_lo, c_hi, pos_lo, pos_hi, K, acc, mine, L);
        else if (pos_hi - pos_lo <= 8u) lloyd_borders<false>(part, p0, p1, c_lo, c_hi - c_lo == 2u, pos_lo, pos_hi, K, acc, L);
        else lloyd_borders<true>(part, p0, p1, c_lo, c_hi - c_lo == 2u, pos_lo, pos_hi, K, acc, L);
    }
}

// The work units of the streams that many workgroups take (one workgroup makes the table): lloyd_unit values of cut buckets
// each, more where that would make more units than the GPU holds at once (one more costs a second round: 8 bits, 2.5 M
// elements 300 instead of 194 us), and one at least for every stream.
template <u32 KMAX>
__device__ __forceinline__ void lloyd_units(const Workspace &w, const GroupParams &g) {
    __shared__ u64 s_work[LLOYD_WAVES];
    __shared__ u32 s_streams[LLOYD_WAVES], s_units[LLOYD_WAVES];
    const u32 tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6, nseg = 3u * g.ntensors;
    const u32 per = (nseg + LLOYD_THREADS - 1u) / LLOYD_THREADS, s0 = min(tid * per, nseg), s1 = min(s0 + per, nseg);
    auto work_of = [&](u32 s) { return w.seg[s].len != 0 && lloyd_shared(w, g, s) ? max(w.seg[s].work, 1u) : 0u; };
    u64 work = 0;
    u32 streams = 0;
    for (u32 s = s0; s < s1; ++s) { const u32 x = work_of(s); work += x; streams += x != 0u; }
    work = wave_sum_u64(work); streams = wave_sum_u32(streams);
    if (lane == 0u) { s_work[wave] = work; s_streams[wave] = streams; }
    __syncthreads();
    work = 0; streams = 0;
#pragma unroll
    for (u32 v = 0; v < LLOYD_WAVES; ++v) { work += s_work[v]; streams += s_streams[v]; }
    const u64 unit = excp_lloyd_unit(work, streams, lloyd_per_cu(KMAX) * (u32)w.cus, lloyd_unit(KMAX));
    auto units_of = [&](u32 s) { return (u32)((work_of(s) + unit - 1u) / unit); };
    u32 units = 0;
    for (u32 s = s0; s < s1; ++s) units += units_of(s);
    const u32 incl = wave_incl_scan_u32(units);
    if (lane == 63u) s_units[wave] = incl;
    __syncthreads();
    u32 run = incl - units;
    for (u32 v = 0; v < wave; ++v) run += s_units[v];
    for (u32 s = s0; s < s1; ++s) { w.seg_unit_begin[s] = run; run += units_of(s); }
    if (tid == LLOYD_THREADS - 1u) w.seg_unit_begin[nseg] = run;
}

// One workgroup takes a stream through all its iterations; the final centres and cut keys end in the slots of
// parity `iters`.  KMAX: the centres the LDS accumulators are laid out for.
//
// Centre k has the buckets whose smallest value goes to it, [first[k], first[k + 1]): one difference of prefix sums.  What
// border k, the one below centre k, cuts off the bucket before first[k] -- the sum and number of its values from the cut key up
// -- goes from centre k - 1 to centre k: of a bucket with cells the stored sum of the higher cells and the values of one
// cell.  Sixteen lanes take a border (eight beyond 63 centres).  Buckets without cells go the way of k_km_iter.
// What bounds an iteration is its chain of steps, so there is little in it: two round trips to memory (a cell's place, its
// values), prefix sums out of LDS, as integers of 128 bits where the stream's binary orders allow, and for up to 63 centres
// everything from the sums to the next cut keys in one wave, without barriers.
// (us, ten iterations: 1414 values, 15 centres 57 -> 31; 5.8 M values, 154 in eleven launches -> 43; 8.7 M, 255 centres 247
// -> 158.)
constexpr u32 P128_BINS = 15;                             // acc_hi - acc_lo up to which sums fit 127 bits (see lloyd_wide)
template <u32 KMAX>
struct LloydAlone {
    LloydShared L;
    u64 acc[(EXCP_ABSM_BINS + 1u) * KMAX], mine[LLOYD_WAVES][KMAX + 1u];
    __int128 before[NBKT + 1u];                           // sum of the buckets before, in units of 2^(8 acc_lo - 149)
    u64 sum[KMAX + 1u];                                   // per border: what goes to centre k, in units of 2^(pos - 149)
    u32 cnt[KMAX + 1u], pos[KMAX + 1u], first[KMAX + 1u];
    u64 up[KMAX > 63u ? KMAX + 1u : 1u];                  // beyond 63 centres: the border's cell, values and sum of the higher ones
    u32 p0[KMAX > 63u ? KMAX + 1u : 1u], p1[KMAX > 63u ? KMAX + 1u : 1u], above[KMAX > 63u ? KMAX + 1u : 1u];     // p1: top bit set where FINE_NEAR
    u32 fine[NBKT], kmin[NBKT], kmax[NBKT], mag[NBKT];    // per bucket: cells (fine_info), extremes (an empty one: the next one's smallest key)
    u32 edge[4];
    u32 coarse, disorder;
};
// v * 2^(bitpos - 149) onto one column of the accumulators, which only the calling thread uses.
__device__ __forceinline__ void column_add(u64 *col, u32 stride, long long v, u32 bitpos) {
    const bool neg = v < 0;
    const u64 mag = neg ? (u64)0 - (u64)v : (u64)v;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const u64 piece = (mag >> (32 * h)) & 0xffffffffull;
        const u32 p = bitpos + 32u * (u32)h;
        const u64 d = piece << (p & 7u);
        if (piece) col[(p >> 3) * stride] += neg ? (u64)0 - d : d;
    }
}
// Bins [g0, g1] as one integer in units of 2^(8 g0 - 149), which it must fit.
__device__ __forceinline__ __int128 bins_to_i128(const u64 *bins, u32 stride, u32 g0, u32 g1) {
    unsigned __int128 t = 0;
    for (u32 q = g1 + 1u; q-- > g0;) t = (t << 8) + (unsigned __int128)(__int128)(long long)bins[q * stride];
    return (__int128)t;
}
template <u32 KMAX>
__global__ __launch_bounds__(LLOYD_THREADS, 2u * lloyd_per_cu(KMAX)) void k_km_lloyd(Workspace w, GroupParams g) {
    constexpr bool ONE_WAVE = KMAX <= 63u;
    constexpr u32 ROW = ONE_WAVE ? 16u : 8u, BATCH = 8u;  // lanes to a border, loads of a lane in flight
    __shared__ LloydAlone<KMAX> A;
    LloydShared &L = A.L;
    const u32 sidx = stream_in_turn(w, blockIdx.x), tid = threadIdx.x, lane = tid & 63u, K = (u32)g.K, iters = (u32)g.iters;
    const u32 wave = (u32)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
    SegState &S = w.seg[sidx];
    if (S.len == 0 || lloyd_shared(w, g, sidx)) return;
    u32 kp2 = 1; while (kp2 < K) kp2 <<= 1;
    const bool centre = tid < K;
    LloydStream st = lloyd_open(w, sidx, K, 1u, false, L);
    const EXCP_GLOBAL float *part = gptr(seg_part(w, sidx));
    const u64 e0 = (u64)(sidx % 3u) * w.fine_stride + excp_fine_at(w.desc[sidx / 3u].elem_off, sidx / 3u, 0u, 0u);
    const EXCP_GLOBAL u32 *fb = gptr((const u32 *)w.fine_begin) + e0;
    const EXCP_GLOBAL u64 *fa = gptr((const u64 *)w.fine_above) + e0;
    // Prefix sums in 128 bits: the highest value's lowest bit is at 8 (acc_hi - 9) + 7, six more where acc_hi is the last bin,
    // the unit's at 8 acc_lo, and 24 + 31 bits come on top for the mantissa and the number of values.
    const bool narrow = st.acc_hi - st.acc_lo <= P128_BINS;
    const u32 base = 8u * st.acc_lo;
    if (narrow && tid <= NBKT) {
        __int128 t = 0;
        if (st.bin_lo <= st.bin_hi) {
            unsigned __int128 u = 0;
#pragma unroll 4
            for (u32 q = st.bin_hi + 1u; q-- > st.bin_lo;) u = (u << 8) + (unsigned __int128)(__int128)(long long)st.bs[q * (NBKT + 1u) + tid];
            t = (__int128)(u << (8u * (st.bin_lo - st.acc_lo)));
        }
        A.before[tid] = t;
    }
    if (tid < NBKT) { A.kmin[tid] = st.kmin; A.kmax[tid] = st.kmax; A.mag[tid] = w.km_mag[(u64)sidx * NBKT + tid]; }
    if (tid <= KMAX) { A.sum[tid] = 0; A.cnt[tid] = 0; A.first[tid] = tid ? NBKT : 0u; A.pos[tid] = base; }
    if (tid <= EXCP_MAX_K) L.cut[tid] = 0xffffffffu;
    if (tid == 0) { A.coarse = 0; A.disorder = 0; }
    __syncthreads();
    u32 least = 0xffffffffu;
    if (tid < NBKT) {
        const u32 b = NBKT - 1u - tid, size = L.begin[b + 1u] - L.begin[b];     // from the last bucket to the first
        least = size ? A.kmin[b] : 0xffffffffu;
        const u32 top = size ? max(f2u(val_of(A.kmin[b])) & 0x7fffffffu, f2u(val_of(A.kmax[b])) & 0x7fffffffu) : 0u;
        A.fine[b] = fine_info(w, g, sidx, sidx * NBKT + b, size, size ? bit_pos(top) - bit_pos(A.mag[b]) : 0u);
#define EXCP_MOVE(CTRL, ROWS) dpp_u32<CTRL, ROWS>(0xffffffffu, least)
        EXCP_WAVE_SCAN(least, EXCP_FOLD_MIN, EXCP_MOVE);
#undef EXCP_MOVE
        if (lane == 63u) A.edge[wave] = least;
    }
    __syncthreads();
    if (tid < NBKT) {
        for (u32 v = 0; v < wave; ++v) least = min(least, A.edge[v]);
        A.kmin[NBKT - 1u - tid] = least;
    }
    __syncthreads();
    for (u32 i = 0;; ++i) {
        // (a) the cut keys
        if ((!ONE_WAVE || wave == 0u) && centre && tid) L.cut[tid] = cut_key(L.C, K, tid);
        if (i == iters) break;
        if ((!ONE_WAVE || wave == 0u) && tid == 0) A.coarse = 0;
        // The cell that a border c cuts: its values [p0, p1), and what lies above it in its bucket.  f: the first bucket whose
        // smallest key is not below c.
        auto find_cell = [&](u32 c, u32 f, u32 &p0, u32 &p1, bool &near, u32 &pos, u64 &up, u32 &above) {
            if (!(f && c <= A.kmax[f - 1u])) return;
            const u32 b = f - 1u, info = A.fine[b], mag = A.mag[b], q0 = L.begin[b], q1 = L.begin[b + 1u];
            if (info == 0u) { A.coarse = 1u; return; }
            p0 = q0; p1 = q1; near = (info & FINE_NEAR) != 0u;
            pos = bit_pos(mag);
            if (q1 - q0 >= FINE_LEAST) {
                const u32 e = (q0 >> EXCP_FINE_SHIFT) + b + ((excp_closed_key(c, mag) - excp_closed_key(A.kmin[b], mag)) >> fine_shift(info));
                const u32 c0 = fb[e], c1 = fb[e + 1u];
                up = fa[e];
                p0 = q0 + c0; p1 = q0 + c1; above = q1 - p1;
            }
        };
        if (!ONE_WAVE) {
            // (a thread per border: the look-ups of all borders are one round trip.  The barrier: A.coarse is set from here on.)
            __syncthreads();
            if (centre && tid) {
                const u32 c = L.cut[tid];
                u32 f = 0, p0 = 0, p1 = 0, pos = base, above = 0;
                u64 up = 0;
                bool near = true;
#pragma unroll
                for (u32 step = NBKT / 2; step >= 1u; step >>= 1) if (A.kmin[f + step - 1u] < c) f += step;
                if (f == NBKT - 1u && A.kmin[f] < c) f = NBKT;
                find_cell(c, f, p0, p1, near, pos, up, above);
                A.first[tid] = f; A.p0[tid] = p0; A.p1[tid] = p1 | (near ? 1u << 31 : 0u); A.pos[tid] = pos; A.up[tid] = up; A.above[tid] = above;
            }
        }
        __syncthreads();
        // (b) what the borders cut off
        const u32 l = tid & (ROW - 1u);
        for (u32 k0 = 1; k0 < K; k0 += LLOYD_THREADS / ROW) {
            const u32 k = k0 + tid / ROW;
            u64 sum = 0, up = 0;
            u32 cnt = 0, above = 0, f = NBKT, pos = base;
            if (k < K) {
                const u32 c = L.cut[k];
                u32 p0 = 0, p1 = 0;
                bool near = true;
                if (ONE_WAVE) {
                    // the bucket by two steps of sixteen
                    const u32 shift = lane & ~(ROW - 1u);
                    f = 16u * (u32)__popc((u32)(ballot64(A.kmin[16u * l + 15u] < c) >> shift) & 0xffffu);
                    if (f < NBKT) f += (u32)__popc((u32)(ballot64(A.kmin[f + l] < c) >> shift) & 0xffffu);
                    find_cell(c, f, p0, p1, near, pos, up, above);
                } else {
                    p0 = A.p0[k]; p1 = A.p1[k] & 0x7fffffffu; near = A.p1[k] >> 31; pos = A.pos[k]; up = A.up[k]; above = A.above[k];
                }
                // Values below 2^32 units (eight binary orders) add exactly in fp64, and compare with the border as floats: none
                // lies between -0 and +0, which are equally far from any centre.  (Eight instructions a value; as integers it was
                // thirty-five, and with 255 centres that was what an iteration waited for: 27 us, now 14.)
                const float t = val_of(c), inf = u2f(0x7f800000u);
                double part_sum = 0.0;
                if (near) {
                    for (u32 p = p0 + l; p < p1; p += BATCH * ROW) {
                        float x[BATCH];
#pragma unroll
                        for (u32 j = 0; j < BATCH; ++j) x[j] = part[min(p + ROW * j, p1 - 1u)];
#pragma unroll
                        for (u32 j = 0; j < BATCH; ++j) {
                            const bool in = (p + ROW * j < p1 ? x[j] : -inf) >= t;
                            part_sum += (double)(in ? x[j] : 0.f);
                            cnt += in;
                        }
                    }
                    sum = (u64)(long long)ldexp(part_sum, 149 - (int)pos);
                } else {
                    for (u32 p = p0 + l; p < p1; p += BATCH / 2u * ROW) {
                        float x[BATCH / 2u];
#pragma unroll
                        for (u32 j = 0; j < BATCH / 2u; ++j) x[j] = part[min(p + ROW * j, p1 - 1u)];
#pragma unroll
                        for (u32 j = 0; j < BATCH / 2u; ++j)
                            if (p + ROW * j < p1 && x[j] >= t) { sum += value_units(f2u(x[j]), pos); ++cnt; }
                    }
                }
            }
            // the row's sum, in its last lane
            sum += dpp_u64<0x111, 0xf>(sum); sum += dpp_u64<0x112, 0xf>(sum); sum += dpp_u64<0x114, 0xf>(sum);
            cnt += dpp_u32<0x111, 0xf>(0u, cnt); cnt += dpp_u32<0x112, 0xf>(0u, cnt); cnt += dpp_u32<0x114, 0xf>(0u, cnt);
            if (ROW == 16u) { sum += dpp_u64<0x118, 0xf>(sum); cnt += dpp_u32<0x118, 0xf>(0u, cnt); }
            if (l == ROW - 1u && k < K) {
                if (ONE_WAVE) { A.first[k] = f; A.pos[k] = pos; }
                A.sum[k] = sum + up; A.cnt[k] = cnt + above;
            }
        }
        if (!narrow) {
            __syncthreads();
            // (a wave takes a bin, a lane every 64th centre: the loads of a bin are on their way together)
            for (u32 q = st.acc_lo + wave; q <= st.acc_hi; q += LLOYD_WAVES) {
                const bool any = q >= st.bin_lo && q <= st.bin_hi;
                const u64 *row = st.bs + q * (NBKT + 1u);
#pragma unroll
                for (u32 j = 0; j < (KMAX + 63u) / 64u; ++j) {
                    const u32 k = j * 64u + lane;
                    if (k < K) A.acc[q * K + k] = any ? row[k + 1u < K ? A.first[k + 1u] : NBKT] - row[A.first[k]] : 0ull;
                }
            }
        }
        __syncthreads();
        const bool coarse = A.coarse != 0u;               // some border cuts a bucket without cells
        if (coarse) {
            if (narrow) for (u32 j = tid; j < (st.acc_hi + 1u - st.acc_lo) * K; j += LLOYD_THREADS) A.acc[st.acc_lo * K + j] = 0;
            if (centre) A.acc[EXCP_ABSM_BINS * K + tid] = 0;
            const u32 T = lloyd_cut_buckets(st, kp2, L, A.fine);         // (its barriers are passed before anything is added)
            if (T <= LLOYD_FEW) {
                lloyd_few(part, 0u, T, K, kp2, A.acc, L);
            } else {
                const u32 q0 = (u32)(((u64)T * wave) / LLOYD_WAVES), q1 = (u32)(((u64)T * (wave + 1u)) / LLOYD_WAVES);
                lloyd_share(part, q0, q1, K, A.acc, A.mine[wave], L);
            }
            __syncthreads();
        }
        // (c) the centres.  An empty cluster keeps its centre; afterwards the centres are put back in ascending order (stable;
        // nothing moves unless a run of equal centres was torn apart).
        if (!ONE_WAVE || wave == 0u) {
            float c = 0.f;
            if (centre) {
                const u32 f = A.first[tid], l1 = tid + 1u < K ? A.first[tid + 1u] : NBKT;
                u64 cnt = (u64)(L.begin[l1] - L.begin[f]) + A.cnt[tid] - A.cnt[tid + 1u];
                if (coarse) cnt += A.acc[EXCP_ABSM_BINS * K + tid];
                const long long in = (long long)A.sum[tid], out = (long long)A.sum[tid + 1u];
                c = L.C[tid];
                if (cnt) {
                    double total;
                    if (narrow) {
                        unsigned __int128 t = (unsigned __int128)(A.before[l1] - A.before[f]);
                        t += (unsigned __int128)(__int128)in << (A.pos[tid] - base);
                        t -= (unsigned __int128)(__int128)out << (A.pos[tid + 1u] - base);
                        if (coarse) t += (unsigned __int128)bins_to_i128(A.acc + tid, K, st.acc_lo, st.acc_hi);
                        total = i128_to_double((__int128)t, base);
                    } else {
                        column_add(A.acc + tid, K, in, A.pos[tid]);
                        column_add(A.acc + tid, K, -out, A.pos[tid + 1u]);
                        total = signed_bins_to_double(A.acc + tid, K, st.acc_lo, st.acc_hi);
                    }
                    c = (float)(total / (double)cnt);
                }
                L.fresh[tid] = c;
            }
            if (ONE_WAVE) wave_lds_fence(); else __syncthreads();
            bool unsorted = tid + 1u < K && !(c <= L.fresh[tid + 1u]);
            if (ONE_WAVE) {
                unsorted = __any(unsorted);
            } else {
                if (unsorted) A.disorder = 1u;
                __syncthreads();
                unsorted = A.disorder != 0u;
            }
            if (centre) {
                u32 rank = tid;
                if (unsorted) {
                    rank = 0;
#pragma unroll 1
                    for (u32 j = 0; j < K; ++j) {
                        const float cj = L.fresh[j];
                        rank += (cj < c || (cj == c && j < tid)) ? 1u : 0u;
                    }
                }
                L.C[rank] = c;
            }
            if (ONE_WAVE) wave_lds_fence();
            else { __syncthreads(); if (tid == 0) A.disorder = 0u; }
        }
    }
    __syncthreads();
    if (centre) S.C[iters & 1u][tid] = L.C[tid];
    if (tid <= EXCP_MAX_K) S.cut[iters & 1u][tid] = tid ? L.cut[tid] : 0u;
}

// What the streams that many workgroups take are cut into.
template <u32 KMAX>
__global__ __launch_bounds__(LLOYD_THREADS) void k_km_units(Workspace w, GroupParams g) { lloyd_units<KMAX>(w, g); }

// One iteration of the streams that many workgroups take: a workgroup for each work unit, which is an even share of the
// stream's cut buckets (the grid is the most units the group can have; those beyond the units there are have nothing
// to do).  Every workgroup of a stream computes the centres for itself, adds its share up in LDS, and hands the sums over.
// The launch after the last iteration (i == iters) only makes the final centres.
template <u32 KMAX>
__global__ __launch_bounds__(LLOYD_THREADS, 2u * lloyd_per_cu(KMAX)) void k_km_iter(Workspace w, GroupParams g, u32 i) {
    __shared__ LloydShared L;
    __shared__ u64 acc[(EXCP_ABSM_BINS + 1u) * KMAX], mine[LLOYD_WAVES][KMAX + 1u];
    const u32 tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6, u = blockIdx.x;
    const u32 K = (u32)g.K, nseg = 3u * g.ntensors, accw = (EXCP_ABSM_BINS + 1u) * K;
    if (u >= w.seg_unit_begin[nseg]) return;
    // the stream that holds unit u: 64 entries of the table are compared at once
    u32 sidx = 0;
#pragma unroll 1
    for (u32 span = nseg; span > 1u;) {
        const u32 step = (span + 63u) / 64u;
        const u64 le = ballot64(lane * step < span && w.seg_unit_begin[min(sidx + lane * step, nseg)] <= u);
        const u32 pick = (u32)__popcll(le) - 1u;          // (entry 0 of the span is <= u)
        span = min(step, span - pick * step);
        sidx += pick * step;
    }
    sidx = (u32)__builtin_amdgcn_readfirstlane((int)sidx);
    const u32 u_first = u - w.seg_unit_begin[sidx], nu = w.seg_unit_begin[sidx + 1u] - (u - u_first);
    if (i == (u32)g.iters && u_first != 0u) return;
    u32 kp2 = 1; while (kp2 < K) kp2 <<= 1;
    SegState &S = w.seg[sidx];
    u64 *gacc = w.km_acc + (3ull * w.desc[sidx / 3u].acc_slot + sidx % 3u) * 3u * accw;      // [3][bins + count][K]
    LloydStream st = lloyd_open(w, sidx, K, (i + 1u) & 1u, i > 0u, L);
    if (i == 0u) {
        lloyd_clear(acc, st, K);
    } else {
        const u64 *old = gacc + ((i - 1u) % 3u) * accw;
        const u32 j1 = (st.acc_hi + 1u) * K;
        for (u32 j0 = st.acc_lo * K + tid; j0 < j1; j0 += 4u * LLOYD_THREADS) {
            u64 v[4];
#pragma unroll
            for (u32 q = 0; q < 4; ++q) v[q] = j0 + q * LLOYD_THREADS < j1 ? old[j0 + q * LLOYD_THREADS] : 0ull;
#pragma unroll
            for (u32 q = 0; q < 4; ++q) if (j0 + q * LLOYD_THREADS < j1) acc[j0 + q * LLOYD_THREADS] = v[q];
        }
        if (tid < K) acc[EXCP_ABSM_BINS * K + tid] = old[EXCP_ABSM_BINS * K + tid];
        __syncthreads();
        if (tid < NBKT && L.begin[tid + 1u] > L.begin[tid]) st.alo = centre_by_cuts(L.cut, kp2, st.kmin);
    }
    lloyd_centres(st, K, i, acc, L);
    if (u_first == 0u) {
        // one workgroup per stream keeps what the next iteration starts from, and clears the accumulators
        // of the iteration after it (they were read by the previous launch for the last time)
        if (tid < K) S.C[i & 1u][tid] = L.C[tid];
        if (tid <= EXCP_MAX_K) S.cut[i & 1u][tid] = tid ? L.cut[tid] : 0u;
        u64 *nxt = gacc + ((i + 1u) % 3u) * accw;
        for (u32 j = st.acc_lo * K + tid; j < (st.acc_hi + 1u) * K; j += LLOYD_THREADS) nxt[j] = 0;
        if (tid < K) nxt[EXCP_ABSM_BINS * K + tid] = 0;
    }
    if (i == (u32)g.iters) return;
    const u32 T = lloyd_cut_buckets(st, kp2, L, nullptr);
    const u32 x0 = (u32)(((u64)T * u_first) / nu), x1 = (u32)(((u64)T * (u_first + 1u)) / nu);
    if (x1 - x0 <= LLOYD_FEW) {
        lloyd_few(gptr(seg_part(w, sidx)), x0, x1, K, kp2, acc, L);
    } else {
        const u32 q0 = x0 + (u32)(((u64)(x1 - x0) * wave) / LLOYD_WAVES), q1 = x0 + (u32)(((u64)(x1 - x0) * (wave + 1u)) / LLOYD_WAVES);
        lloyd_share(gptr(seg_part(w, sidx)), q0, q1, K, acc, mine[wave], L);
    }
    __syncthreads();
    u64 *now = gacc + (i % 3u) * accw;
    for (u32 j = st.acc_lo * K + tid; j < (st.acc_hi + 1u) * K; j += LLOYD_THREADS) { const u64 v = acc[j]; if (v) atomicAdd(&now[j], v); }
    if (tid < K) { const u64 v = acc[EXCP_ABSM_BINS * K + tid]; if (v) atomicAdd(&now[EXCP_ABSM_BINS * K + tid], v); }
}

// The codes of a thread's 32 values of a whole chunk, ORed into the chunk's bit stream in LDS; returns
// the thread's share of the objective.  The four values of a group go through the bisection over the
// cut keys side by side, so that four table reads are in flight at every step instead of one.
__device__ __forceinline__ double assign_whole_chunk(const float (&v)[PER_THREAD], const u32 *s_cut, const float *s_C, u32 kp2,
                                                     u32 nbits, u32 *s_pack) {
    double obj = 0.0;
    u32 tid = threadIdx.x;
    asm volatile("" : "+v"(tid));                  // bit positions are worked out where they are used, not kept from chunk to chunk
    const unsigned char *cut_b = (const unsigned char *)s_cut, *cen_b = (const unsigned char *)s_C;
#pragma unroll
    for (u32 q = 0; q < PER_THREAD / 4; ++q) {
        u32 key[4], p4[4];                         // p4: four times the number of cut keys <= key found so far (a byte offset)
#pragma unroll
        for (u32 j = 0; j < 4; ++j) { key[j] = key_of(v[4 * q + j]); p4[j] = 0; }
        for (u32 step4 = kp2 << 1; step4 >= 4u; step4 >>= 1) {  // as centre_by_cuts, on byte offsets
            u32 a[4], c[4];
#pragma unroll
            for (u32 j = 0; j < 4; ++j) { a[j] = p4[j] + step4; c[j] = *(const u32 *)(cut_b + a[j]); }
#pragma unroll
            for (u32 j = 0; j < 4; ++j) p4[j] = c[j] <= key[j] ? a[j] : p4[j];
        }
        float cen[4];
#pragma unroll
        for (u32 j = 0; j < 4; ++j) cen[j] = *(const float *)(cen_b + p4[j]);
        // the codes (index + 1) of four consecutive values, nbits each: p4 + 4 is four times the code
        u32 field = (p4[0] + 4u) >> 2;
#pragma unroll
        for (u32 j = 1; j < 4; ++j) field |= (p4[j] + 4u) << (nbits * j - 2u);
#pragma unroll
        for (u32 j = 0; j < 4; ++j) {
            float x = v[4 * q + j];
            asm volatile("" : "+v"(x));            // widened here, not when the value arrived (thirty-two doubles would not fit)
            const double d = (double)x - (double)cen[j];
            obj += d * d;
        }
        // into the chunk's bit stream at bit (first element) * nbits: at most two 32-bit words
        const u32 bitpos = (q * EXCP_THREADS + tid) * 4u * nbits, wi = bitpos >> 5, sh = bitpos & 31u;
        atomicOr(&s_pack[wi], field << sh);
        if (sh && (field >> (32u - sh))) atomicOr(&s_pack[wi + 1], field >> (32u - sh));
        __builtin_amdgcn_sched_barrier(0);         // one group at a time: nothing of the next is started early
    }
    return obj;
}

// ---------------------------------------------------------------- final assignment + packing
// A chunk's codes are ORed, four at a time, into the chunk's bit stream in LDS and leave as whole
// 64-bit words.
__global__ __launch_bounds__(EXCP_THREADS, 5) void k_assign_pack(Workspace w, GroupParams g) {
    __shared__ float s_C[EXCP_MAX_K + 1];
    __shared__ u32 s_cut[EXCP_MAX_K + 1];
    __shared__ u32 s_pack2[2][EXCP_CHUNK * 8 / 32 + 2];  // a chunk's packed codes (up to 8 bits each); chunks alternate between the two
    __shared__ double s_red[EXCP_THREADS / 64];
    const u32 tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    const u32 total = *w.chunk_total;
    const u32 G = gridDim.x, b = blockIdx.x;
    const u32 lo = (u32)(((u64)b * total) / G), hi = (u32)(((u64)(b + 1) * total) / G);
    if (lo >= hi) return;
    const u32 nseg = 3u * g.ntensors;
    const int K = g.K;
    u32 kp2 = 1; while (kp2 < (u32)K) kp2 <<= 1;
    const u32 nbits = (u32)g.nbits;
    const u32 words_per_chunk = EXCP_CHUNK * nbits / 64u;

    u32 sidx = 0xffffffffu, s_end = 0;
    u64 len = 0, nwords = 0;                       // of the stream in hand: fetched when the stream changes, not per chunk
    u32 chunk0 = 0;
    const EXCP_GLOBAL float *data = nullptr;
    u64 *out = nullptr;
    double obj = 0.0;                              // this thread's share of the objective over the chunks of the stream in hand
    // The workgroup's total for the stream goes into the entry of the last of its chunks (the others hold 0).
    auto close_stream = [&](u32 last_chunk) {
#pragma unroll
        for (int mm = 32; mm >= 1; mm >>= 1) obj += shfl_xor_f64(obj, mm);
        if (lane == 0) s_red[wave] = obj;
        __syncthreads();
        if (tid == 0) w.part_obj[last_chunk] = (s_red[0] + s_red[1]) + (s_red[2] + s_red[3]);
        obj = 0.0;
    };
    for (u32 c = lo; c < hi; ++c) {
        u32 *s_pack = s_pack2[c & 1u];
        if (sidx == 0xffffffffu || c >= s_end) {
            if (sidx != 0xffffffffu) close_stream(c - 1u);
            __syncthreads();
            sidx = find_owner(w.seg_chunk_begin, nseg, c);
            s_end = w.seg_chunk_begin[sidx + 1];
            const u32 t = sidx / 3u, which = sidx % 3u;
            const TState &T = w.st[t];
            len = w.seg[sidx].len; chunk0 = w.seg[sidx].chunk_begin; data = gptr(seg_data(w, sidx));
            nwords = excp_words(len * nbits);
            out = (u64 *)(w.desc[t].blob + (which == 0 ? T.off_cw : (which == 1 ? T.off_cm : T.off_cv)));
            if (tid < (u32)K) s_C[tid] = w.seg[sidx].C[g.iters & 1][tid];        // the final centres and their cut keys
            s_cut[tid] = w.seg[sidx].cut[g.iters & 1][tid];
            __syncthreads();
        }
        const u64 ebase = (u64)(c - chunk0) * EXCP_CHUNK;
        const u32 clen = (len - ebase) < EXCP_CHUNK ? (u32)(len - ebase) : EXCP_CHUNK;
        const u64 wbase = (u64)(c - chunk0) * words_per_chunk;
        float v[PER_THREAD];
        load_chunk(data + ebase, clen, v);
        for (u32 i = tid; i < 2u * words_per_chunk + 2u; i += EXCP_THREADS) s_pack[i] = 0;
        __syncthreads();
        if (clen == EXCP_CHUNK) {
            obj += assign_whole_chunk(v, s_cut, s_C, kp2, nbits, s_pack);
        } else {
            // a stream's ragged last chunk: value by value
#pragma unroll
            for (u32 q = 0; q < PER_THREAD / 4; ++q) {
                u32 field = 0;
#pragma unroll
                for (u32 j = 0; j < 4; ++j) {
                    const u32 it = 4 * q + j;
                    if (chunk_elem(it) < clen) {
                        const u32 pick = centre_by_cuts(s_cut, kp2, key_of(v[it]));
                        const double d = (double)v[it] - (double)s_C[pick];
                        obj += d * d;
                        field |= (1u + pick) << (nbits * j);
                    }
                }
                const u32 bitpos = chunk_elem(4 * q) * nbits, wi = bitpos >> 5, sh = bitpos & 31u;
                if (field) {
                    atomicOr(&s_pack[wi], field << sh);
                    if (sh && (field >> (32u - sh))) atomicOr(&s_pack[wi + 1], field >> (32u - sh));
                }
            }
        }
        __syncthreads();
        for (u32 wl = tid; wl < words_per_chunk; wl += EXCP_THREADS) {
            const u64 wg = wbase + wl;
            if (wg >= nwords) break;
            out[wg] = (u64)s_pack[2 * wl] | ((u64)s_pack[2 * wl + 1] << 32);
            if (wg == nwords - 1 && (nwords & 1ull)) out[nwords] = 0ull;     // 16-byte padding
        }
        if (tid == 0) w.part_obj[c] = 0.0;
        // (no barrier here: the next chunk uses the other buffer, and this one is zeroed again only after
        // the two barriers of that chunk)
    }
    close_stream(hi - 1u);
}

// ---------------------------------------------------------------- no quantisation: the streams as they are
// Prune-only mode (Table "abl"): every survivor stream goes into its blob section as fp32, in index
// order; the section's padding (up to 16 bytes) is zeroed.  One chunk of 8192 values per step.
__global__ __launch_bounds__(EXCP_THREADS) void k_store_raw(Workspace w, GroupParams g) {
    const u32 tid = threadIdx.x;
    const u32 total = *w.chunk_total;
    const u32 nseg = 3u * g.ntensors;
    for (u32 c = blockIdx.x; c < total; c += gridDim.x) {
        const u32 sidx = find_owner(w.seg_chunk_begin, nseg, c);
        const SegState &S = w.seg[sidx];
        const u32 t = sidx / 3u, which = sidx % 3u;
        const TState &T = w.st[t];
        const u64 len = S.len;
        const u64 base = (u64)(c - S.chunk_begin) * EXCP_CHUNK;
        const u32 clen = (len - base) < EXCP_CHUNK ? (u32)(len - base) : EXCP_CHUNK;
        const u64 off = which == 0 ? T.off_cw : (which == 1 ? T.off_cm : T.off_cv);
        const EXCP_GLOBAL float *src = gptr(seg_data(w, sidx)) + base;
        EXCP_GLOBAL float *dst = gptr((float *)(w.desc[t].blob + off)) + base;
        const u32 padded = (clen + 3u) & ~3u;              // a chunk starts on a 16-byte boundary of the section
        for (u32 i = tid * 4u; i < padded; i += EXCP_THREADS * 4u) {
            f4u o;
            if (i + 4u <= clen) {
                const f4u q = *(const EXCP_GLOBAL f4u *)(src + i);
                o = q;
            } else {
                o.x = i < clen ? src[i] : 0.f; o.y = i + 1u < clen ? src[i + 1u] : 0.f;
                o.z = i + 2u < clen ? src[i + 2u] : 0.f; o.w = 0.f;
            }
            *(EXCP_GLOBAL f4u *)(dst + i) = o;
        }
    }
}

// ---------------------------------------------------------------- header, codebooks, results
// A workgroup per tensor; `decode`: and what the decoders need to make W_hat of the blob just written, without parsing it -- its
// state, and, by the workgroups beyond, how many survivors precede every tile, which the scan of the mask pass knows.
__global__ __launch_bounds__(EXCP_THREADS) void k_finalize(Workspace w, GroupParams g, u32 rec_base, u32 decode) {
    __shared__ double s_obj[3];
    if (blockIdx.x >= g.ntensors) {
        const u32 tile = (blockIdx.x - g.ntensors) * EXCP_THREADS + threadIdx.x;
        if (tile < g.ntiles) w.dec_cnt_w[tile] = (u32)(w.mask_prefix[2ull * tile] >> 32);
        return;
    }
    if (decode && threadIdx.x == EXCP_THREADS - 1u) {
        const u32 t = blockIdx.x;
        const TDesc &C = w.desc[t];
        const TState &T = w.st[t];
        DDesc D{};
        DState S{};
        D.Wp = C.Wp; D.blob = C.blob; D.blob_bytes = T.blob_bytes; D.n = C.n; D.W_out = C.W_out;
        D.wtype = excp_wtype(g.flags); D.tile_begin = C.tile_begin; D.tile_count = C.tile_count;
        S.n_w = T.n_w; S.n_o = T.n_o; S.blob_bytes = T.blob_bytes; S.nbits = (u32)g.nbits;
        S.off_bw = EXCP_HEADER + excp_books_bytes((u32)g.nbits);
        S.off_bo = T.off_bo; S.off_cw = T.off_cw; S.off_cm = T.off_cm; S.off_cv = T.off_cv;
        S.status = (T.status == 0 && C.W_out != nullptr) ? 0 : 1;    // 1 = skip silently
        S.flags = g.flags;
        w.ddesc[t] = D; w.dst[t] = S;
        if (t == 0) *w.dec_kinds = blob_kind((u32)g.nbits, g.flags);
    }
    const u32 t = blockIdx.x, tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    const TDesc &D = w.desc[t];
    TState &T = w.st[t];
    const bool raw = (u32)g.nbits >= EXCP_RAW_BITS;          // no quantisation: no codebooks, no objective
    const u32 E = raw ? 0u : 1u << g.nbits;
    if (wave < 3) {
        const u32 sidx = 3u * t + wave;
        double acc = 0.0;
        if (!raw && w.seg[sidx].len) {
            const u32 c0 = w.seg[sidx].chunk_begin, c1 = w.seg_chunk_begin[sidx + 1];
            // (eight at a time: one after the other, this kernel took 7.6 us for a 16.8 M-element tensor's 700 chunks, 17.7 for the 410M shape,
            // now 5.1 and 8.1)
            for (u32 c = c0 + lane; c < c1; c += 8u * 64u) {
                double x[8];
#pragma unroll
                for (u32 q = 0; q < 8u; ++q) x[q] = c + q * 64u < c1 ? w.part_obj[c + q * 64u] : 0.0;
#pragma unroll
                for (u32 q = 0; q < 8u; ++q) acc += x[q];
            }
        }
#pragma unroll
        for (int mm = 32; mm >= 1; mm >>= 1) acc += shfl_xor_f64(acc, mm);
        if (lane == 0) s_obj[wave] = acc;
    }
    __syncthreads();
    // codebooks: entry 0 is +0, then the K centres
    float *books = (float *)(D.blob + EXCP_HEADER);
    for (u32 i = tid; i < 3u * E; i += EXCP_THREADS) {
        u32 which = i / E, e = i % E;
        const SegState &S = w.seg[3u * t + which];
        books[i] = (e == 0 || S.len == 0) ? 0.f : S.C[g.iters & 1][e - 1];
    }
    if (tid == 0) {
        T.obj[0] = s_obj[0]; T.obj[1] = s_obj[1]; T.obj[2] = s_obj[2];
        u32 *h = (u32 *)D.blob;
        u64 *h64 = (u64 *)D.blob;
        float *hf = (float *)D.blob;
        h[0] = EXCP_MAGIC; h[1] = EXCP_VERSION; h[2] = (u32)g.nbits; h[3] = g.flags;
        h64[2] = D.n; h64[3] = T.n_w; h64[4] = T.n_o;
        hf[10] = g.alpha; hf[11] = g.beta; hf[12] = u2f(T.med_bits); hf[13] = T.mean32;
        hf[14] = T.t_w; hf[15] = T.r_o;
        h64[8] = T.blob_bytes;
        h[18] = (u32)g.iters; h[19] = 0u;
        HostRec &R = w.rec_dev[rec_base + D.rec];
        R.n = D.n; R.n_w = T.n_w; R.n_o = T.n_o; R.blob_bytes = T.blob_bytes; R.nonfinite = T.nonfinite;
        R.abs_sum = T.abs_sum; R.obj[0] = s_obj[0]; R.obj[1] = s_obj[1]; R.obj[2] = s_obj[2];
        R.med = u2f(T.med_bits); R.mean32 = T.mean32; R.t_w = T.t_w; R.r_o = T.r_o;
        R.status = T.status; R.pad = 0;
    }
}

}  // namespace

void launch_km_partition(const Workspace &w, const GroupParams &g, int phase, hipStream_t s) {
    if (!g.ntensors) return;
    const u32 nseg = 3 * g.ntensors;
    switch (phase) {
        case 0:
            if (g.samples > EXCP_SAMPLES_FEW) hipLaunchKernelGGL(k_km_draw<EXCP_SAMPLES_MANY / (DRAW_PARTS * EXCP_THREADS)>, dim3(nseg * DRAW_PARTS), dim3(EXCP_THREADS), 0, s, w, g);
            else hipLaunchKernelGGL(k_km_draw<EXCP_SAMPLES_FEW / (DRAW_PARTS * EXCP_THREADS)>, dim3(nseg * DRAW_PARTS), dim3(EXCP_THREADS), 0, s, w, g);
            hipLaunchKernelGGL(k_km_sample, dim3(nseg), dim3(SM_THREADS), 0, s, w, g); break;
        case 1: hipLaunchKernelGGL(k_km_scan, dim3(nseg), dim3(SCAN_PARTS * 64), 0, s, w, g); break;
        case 2: hipLaunchKernelGGL(k_km_scatter, dim3(excp_grid(w, 1)), dim3(SC_THREADS), 0, s, w, g); break;
        default:
            if (g.wide == 2u) {
                hipLaunchKernelGGL((k_km_bucket_stats<16, 1>), dim3(nseg * NBKT), dim3(1024), 0, s, w, g, (u32)STREAMS_ALL, nseg);
            } else {
                const u32 sel = g.wide ? STREAMS_MV : STREAMS_ALL, ns = stream_count(g.ntensors, sel);
                if (g.wide) hipLaunchKernelGGL((k_km_bucket_stats<16, 4>), dim3(g.ntensors * (NBKT / 4)), dim3(1024), 0, s, w, g, (u32)STREAMS_W, g.ntensors);
                // (sets of four buckets, unless that leaves compute units without work: the 192 sets of one 16.8 M-element
                // tensor took 34 us, its 768 buckets 15)
                if (ns * (NBKT / 4) < excp_grid(w, 4))
                    hipLaunchKernelGGL((k_km_bucket_stats<4, 1>), dim3(ns * NBKT), dim3(256), 0, s, w, g, sel, ns);
                else
                    hipLaunchKernelGGL((k_km_bucket_stats<4, 4>), dim3(std::min(ns * (NBKT / 4), excp_grid(w, 40))), dim3(256), 0, s, w, g, sel, ns);
            }
            break;
    }
}

// Cells for the group's larger tensors, by the largest (EXCP_FINE_): registers for buckets of 8192 values, which the tensors
// are not expected to exceed, of 40 960 in sixteen waves, or of 53 248 in eight, which take longer (16.8 M elements 40
// instead of 31 us).
void launch_km_cells(const Workspace &w, const GroupParams &g, hipStream_t s) {
    if (!g.fine) return;
    const dim3 grid(3u * g.fine * NBKT);
    if (g.fine_size == 0u) hipLaunchKernelGGL((k_km_cells<512, excp_cells_most(0u), 8192>), grid, dim3(512), 0, s, w, g);
    else if (g.fine_size == 1u) hipLaunchKernelGGL((k_km_cells<1024, excp_cells_most(1u), 20480>), grid, dim3(1024), 0, s, w, g);
    else hipLaunchKernelGGL((k_km_cells<512, excp_cells_most(2u), 26624>), grid, dim3(512), 0, s, w, g);
}

void launch_km_init(const Workspace &w, const GroupParams &g, hipStream_t s) {
    if (!g.ntensors) return;
    const u32 per = (u32)g.K + 1u;
    if (g.wide == 2u) {
        hipLaunchKernelGGL((k_km_init<1024, true>), dim3(3 * g.ntensors * per), dim3(1024), 0, s, w, g, (u32)STREAMS_ALL);
    } else {
        const u32 sel = g.wide ? STREAMS_MV : STREAMS_ALL;
        if (g.wide) hipLaunchKernelGGL((k_km_init<1024, true>), dim3(g.ntensors * per), dim3(1024), 0, s, w, g, (u32)STREAMS_W);
        // A workgroup reads a bucket, of which those of few large tensors hold a hundred thousand values: sixteen waves, if there are no
        // more than eight workgroups to a compute unit and the tensors are of 2^24 elements on average (us with four waves / sixteen, 4 bits:
        // one of 100 M elements 138 / 79, 40 M 61 / 33, four layers of the 7B shape 209 / 126, 8 x 16.8 M 46 / 38, 8 x 8 M 29 / 29, 20 x 3 M 22 / 40; 8 bits:
        // 100 M 192 / 99, 40 M 80 / 65, but 8 x 16.8 M, 6144 workgroups, 120 / 269).
        const u32 grid = stream_count(g.ntensors, sel) * per;
        if (!g.fine && (u64)g.ntiles * EXCP_TILE >= (u64)g.ntensors << 24 && grid <= excp_grid(w, 8)) hipLaunchKernelGGL((k_km_init<1024, false>), dim3(grid), dim3(1024), 0, s, w, g, sel);
        else hipLaunchKernelGGL((k_km_init<256, false>), dim3(grid), dim3(256), 0, s, w, g, sel);
    }
}

// All iterations: the streams that one workgroup takes through them, and, if the group may have others, a launch per
// iteration and one for the final centres.  The two kinds have nothing to do with each other and neither fills the GPU, so one
// goes to a stream of its own: the launches, where cells make it likely that no stream takes them (then they are empty, 4.5 us
// each, which pass beside the first kind), otherwise the single one (the 410M shape: 219 us beside 186), because what begins on
// the other stream begins some 15 us later.  Nothing of this needs bitmap_o, which is made beside, where there is less to do.
template <u32 KMAX>
static void launch_lloyd(const Workspace &w, const GroupParams &g, hipStream_t s, const SideStream &side) {
    const hipStream_t many = g.fine ? side.stream : s, one = g.fine || !g.slots ? s : side.stream;
    if (g.slots) {
        (void)hipEventRecord(side.fork, s);
        (void)hipStreamWaitEvent(side.stream, side.fork, 0);
    }
    // (first: the others are a dozen calls of the runtime, during which it would not yet have begun)
    hipLaunchKernelGGL(k_km_lloyd<KMAX>, dim3(3 * g.ntensors), dim3(LLOYD_THREADS), 0, one, w, g);
    launch_bitmap_o(w, g, one);
    if (!g.slots) return;
    hipLaunchKernelGGL(k_km_units<KMAX>, dim3(1), dim3(LLOYD_THREADS), 0, many, w, g);
    const u32 units = excp_lloyd_grid(excp_grid(w, lloyd_per_cu(KMAX)), g.slots);
    for (u32 i = 0; i <= (u32)g.iters; ++i) hipLaunchKernelGGL(k_km_iter<KMAX>, dim3(units), dim3(LLOYD_THREADS), 0, many, w, g, i);
    (void)hipEventRecord(side.join, side.stream);
    (void)hipStreamWaitEvent(s, side.join, 0);
}
void launch_km_iter(const Workspace &w, const GroupParams &g, hipStream_t s, const SideStream &side) {
    if (!g.ntensors) return;
    if (g.K <= 15) launch_lloyd<15>(w, g, s, side);
    else if (g.K <= 63) launch_lloyd<63>(w, g, s, side);
    else launch_lloyd<EXCP_MAX_K>(w, g, s, side);
}

void launch_assign_pack(const Workspace &w, const GroupParams &g, hipStream_t s) {
    hipLaunchKernelGGL(k_assign_pack, dim3(excp_grid(w, 5)), dim3(EXCP_THREADS), 0, s, w, g);
}

void launch_store_raw(const Workspace &w, const GroupParams &g, hipStream_t s) {
    if (!g.ntensors) return;
    hipLaunchKernelGGL(k_store_raw, dim3(excp_grid(w, 16)), dim3(EXCP_THREADS), 0, s, w, g);
}

void launch_finalize(const Workspace &w, const GroupParams &g, bool decode, hipStream_t s) {
    if (!g.ntensors) return;
    const u32 counts = decode ? (g.ntiles + EXCP_THREADS - 1u) / EXCP_THREADS : 0u;
    hipLaunchKernelGGL(k_finalize, dim3(g.ntensors + counts), dim3(EXCP_THREADS), 0, s, w, g, w.rec_base, decode ? 1u : 0u);
}

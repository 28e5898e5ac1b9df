// Reconstruction (Alg. 2): bitmap rank -> packed code -> codebook -> W_hat = W_prev + C_w[code],
// m_hat / v_hat = C[code] (zero where pruned).
//
// A tile of 4096 elements needs (a) the number of residual survivors before it, and (b) the number
// of moment survivors before its first residual survivor.  Both come from popcounts: per-tile
// counts of bitmap_w, an exclusive scan per tensor, then per-tile popcounts of the matching bit
// range of bitmap_o and a second scan.  The main pass is then independent per tile.
#include "excp_util.h"

#include <algorithm>

namespace {

// Weights and moments go through once in either direction, sixteen bytes a lane and neighbours side by side: past the caches.  (The
// main pass of the 410M shape 719 -> 654 us, of 24 ragged tensors with their moments 825 -> 711, eight chained checkpoints 1142 ->
// 1064; loads alone past them 721, 819 and 1102, stores alone 699, 785 and 1094.)
#define READ_ONCE(T, p) __builtin_nontemporal_load((const EXCP_GLOBAL T *)p)
#define WRITE_ONCE(T, p, x) __builtin_nontemporal_store(x, (EXCP_GLOBAL T *)p)

__device__ __forceinline__ u64 range_mask(u32 lo_bit, u32 hi_bit) {   // bits [lo_bit, hi_bit), hi_bit <= 64
    u64 hi = (hi_bit >= 64u) ? ~0ull : ((1ull << hi_bit) - 1ull);
    u64 lo = (lo_bit >= 64u) ? ~0ull : ((1ull << lo_bit) - 1ull);
    return hi & ~lo;
}

// popcount of bits [p0, p1) of a bitmap
__device__ __forceinline__ u32 popcount_range_lane(const u64 *__restrict__ bm, u64 p0, u64 p1, u32 lane) {
    // the calling wave covers up to 65 words: lane l takes word (p0 >> 6) + l, lane 0 also the 65th
    if (p1 <= p0) return 0;
    const u64 w0 = p0 >> 6, w1 = (p1 - 1) >> 6;
    u32 cnt = 0;
    for (u64 wi = w0 + lane; wi <= w1; wi += 64) {
        u64 word = bm[wi];
        u32 lo = (wi == w0) ? (u32)(p0 & 63ull) : 0u;
        u32 hi = (wi == w1) ? (u32)((p1 - 1) & 63ull) + 1u : 64u;
        cnt += __popcll(word & range_mask(lo, hi));
    }
    return cnt;
}

__device__ __forceinline__ bool wants_moments(const DDesc &D) {
    return D.m_out != nullptr || D.v_out != nullptr || D.cm != nullptr || D.cv != nullptr;
}

// Validates the header of a blob and derives the section offsets.  Returns the kind of blob, 0 if it is damaged.
__device__ __forceinline__ u32 parse_header(const DDesc &D, DState &S, bool allow_raw) {
    S.status = 0; S.pop_w = 0; S.pop_o = 0;
    S.n_w = 0; S.n_o = 0; S.nbits = 4; S.blob_bytes = 0; S.flags = 0; S.pad = 0;
    if (D.blob_bytes < EXCP_HEADER) { S.status = -4; return 0u; }
    const u32 *h = (const u32 *)D.blob;
    const u64 *h64 = (const u64 *)D.blob;
    const u32 nbits = h[2];
    const u64 n = h64[2], nw = h64[3], no = h64[4], total = h64[8];
    const bool raw = (h[3] & 4u) != 0u;                   // written without quantisation: fp32 values, no codebooks
    const bool nw2m = (h[3] & 8u) != 0u;                  // bitmap_o over all elements, not over the kept residuals
    bool ok = h[0] == EXCP_MAGIC && h[1] == EXCP_VERSION && h[3] < 64u && (h[3] & 0x30u) != 0x30u;
    ok = ok && (raw ? (nbits == EXCP_RAW_BITS && allow_raw) : (nbits >= 2u && nbits <= 8u));
    ok = ok && n == D.n && nw <= n && no <= (nw2m ? n : nw);
    ok = ok && (D.wtype == 3u || D.wtype == excp_wtype(h[3]));      // the caller's arrays are what the blob expects
    u64 off = EXCP_HEADER;
    if (ok) {
        off += excp_books_bytes(nbits);
        S.off_bw = off; off += excp_pad16(8ull * excp_words(n));
        S.off_bo = off; off += excp_pad16(8ull * excp_words(nw2m ? n : nw));
        S.off_cw = off; off += excp_pad16(8ull * excp_words(nw * nbits));
        S.off_cm = off; off += excp_pad16(8ull * excp_words(no * nbits));
        S.off_cv = off; off += excp_pad16(8ull * excp_words(no * nbits));
        ok = (off == total) && (total <= D.blob_bytes);
    }
    if (!ok) { S.status = -4; return 0u; }
    S.n_w = nw; S.n_o = no; S.nbits = nbits; S.blob_bytes = total; S.flags = h[3];
    return blob_kind(nbits, h[3]);
}
// The first launch of a larger group: headers, kinds of blob, sums of counts at zero.  `single`: the only tensor's
// description comes as an argument and is left where the others look for it.  (Blobs lie in as many pages, so many compute units
// take a share: 2336 of them 49 us in one workgroup.  Its last workgroup, by ticket, hands the kinds over.)
constexpr u32 PARSE_THREADS = 64;
__global__ __launch_bounds__(PARSE_THREADS) void k_decode_parse(Workspace w, u32 ntensors, u32 parts, u32 allow_raw, DDesc one, u32 single) {
    const u32 tid = threadIdx.x, i = blockIdx.x * PARSE_THREADS + tid;
    if (single && i == 0u) { w.ddesc[0] = one; w.tile_begin[0] = 0u; w.tile_begin[1] = one.tile_count; }
    for (u32 k = i; k < parts; k += gridDim.x * PARSE_THREADS) { w.dec_part[k] = 0u; w.dec_part[w.dec_part_stride + k] = 0u; }
    u32 kind = 0;
    if (i < ntensors) kind = single ? parse_header(one, w.dst[i], allow_raw != 0u) : parse_header(w.ddesc[i], w.dst[i], allow_raw != 0u);
    u32 kinds = 0;
#pragma unroll
    for (u32 k = 1u; k <= 4u; k <<= 1) kinds |= ballot64(kind == k) ? k : 0u;
    if (tid != 0) return;
    if (gridDim.x == 1u) { w.dec_kinds[0] = kinds; return; }
    if (kinds) atomicOr(&w.dec_kinds[1], kinds);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // (it has arrived before the ticket is drawn)
    if (atomicAdd(&w.dec_kinds[2], 1u) == gridDim.x - 1u) {
        w.dec_kinds[0] = atomicExch(&w.dec_kinds[1], 0u);
        w.dec_kinds[2] = 0u;
    }
}

__device__ __forceinline__ void decode_record(const Workspace &w, u32 t, u64 n, const DState &S) {
    HostRec R{};
    R.n = n; R.n_w = S.n_w; R.n_o = S.n_o; R.blob_bytes = S.blob_bytes; R.status = S.status;
    w.rec_dev[w.rec_base + t] = R;
}

// All that has to be known before the main pass, for groups of tensors of at most PREP_TILES tiles each, in one
// launch: a workgroup per tensor parses the header, counts, and scans the counts.  Small tensors are bound by the
// number of launches: parsing, counting and scanning are three (five with the moments), of 2 to 4 us each and
// as much again between them (a restore of 65 536 elements 66-75 -> 55 us when they were five and eight).  Four tiles to a wave, so that a tensor is
// one round of loads; larger tensors would leave the one workgroup behind the general path's many.
constexpr u32 PREP_WAVES = 8, PREP_TILES = 4 * PREP_WAVES;

// `single`: the only tensor's description comes as an argument and is left where the main pass looks for it.  `records`: the
// results for the host are known here and written at once.
__global__ __launch_bounds__(PREP_WAVES * 64) void k_decode_prep(Workspace w, u32 allow_raw, u32 moments, u32 records, DDesc one, u32 single) {
    __shared__ DDesc D;
    __shared__ DState S;
    __shared__ u32 s_cnt[PREP_TILES], s_excl[PREP_TILES + 1];
    const u32 t = blockIdx.x, tid = threadIdx.x, lane = tid & 63u;
    const u32 wave = (u32)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
    if (tid == 0) {
        if (single) { D = one; w.ddesc[0] = one; w.tile_begin[0] = 0u; w.tile_begin[1] = one.tile_count; }
        else D = w.ddesc[t];
        (void)parse_header(D, S, allow_raw != 0u);
        if (t == 0) *w.dec_kinds = 7u;                     // (the main passes look at every tensor)
    }
    __syncthreads();
    const u32 ntiles = D.tile_count;
    const u64 n = D.n;
    // exclusive scan of s_cnt into s_excl and the table; returns the total (in the first wave)
    auto scan = [&](u32 *table) {
        __syncthreads();
        u32 total = 0;
        if (wave == 0u) {
            const u32 c = lane < ntiles ? s_cnt[lane] : 0u, incl = wave_incl_scan_u32(c);
            if (lane < ntiles) { s_excl[lane] = incl - c; table[D.tile_begin + lane] = incl - c; }
            total = last_lane_u32(incl);
            if (lane == 0u) s_excl[ntiles] = total;
        }
        return total;
    };
    {
        u64 v[4] = {0ull, 0ull, 0ull, 0ull};
        if (S.status == 0) {
            const EXCP_GLOBAL u64 *bm = gptr((const u64 *)(D.blob + S.off_bw));
#pragma unroll
            for (u32 k = 0; k < 4; ++k) {
                const u64 word = (wave * 4u + k) * 64u + lane;
                if (word < excp_words(n)) {
                    v[k] = bm[word];
                    if (n - word * 64u < 64u) v[k] &= (1ull << (n - word * 64u)) - 1ull;       // (bits beyond n are ignored)
                }
            }
        }
#pragma unroll
        for (u32 k = 0; k < 4; ++k) {
            const u32 c = wave_sum_u32((u32)__popcll(v[k]));
            if (lane == 0u) s_cnt[wave * 4u + k] = c;
        }
        const u32 total = scan(w.dec_cnt_w);
        if (tid == 0) { S.pop_w = total; if (S.status == 0 && total != S.n_w) S.status = -4; }
    }
    __syncthreads();
    if (moments && wants_moments(D)) {
#pragma unroll
        for (u32 k = 0; k < 4; ++k) {
            const u32 tile = wave * 4u + k;
            u32 c = 0;
            if (tile < ntiles && S.status == 0) {
                u64 p0 = s_excl[tile], p1 = s_excl[tile + 1u];
                if (S.flags & 8u) {                        // one bit per element: the tile's own range
                    p0 = (u64)tile * EXCP_TILE;
                    p1 = (n - p0 < (u64)EXCP_TILE) ? n : p0 + EXCP_TILE;
                }
                c = popcount_range_lane((const u64 *)(D.blob + S.off_bo), p0, p1, lane);
            }
            c = wave_sum_u32(c);
            if (lane == 0u) s_cnt[tile] = c;
        }
        __syncthreads();                                   // (the counts above are read before they are scanned over)
        const u32 total = scan(w.dec_cnt_o);
        if (tid == 0) { S.pop_o = total; if (S.status == 0 && total != S.n_o) S.status = -4; }
    }
    if (tid == 0) {
        w.dst[t] = S;
        if (records) decode_record(w, t, D.n, S);
    }
}

// which == 0: per-tile popcount of bitmap_w.  which == 1: per-tile popcount of the bitmap_o bits
// that belong to the tile's survivors (needs the scanned bitmap_w counts).  A wave takes a contiguous range of tiles, eight at a
// time, each with eight lanes of its own that look their tensor up when it changes.  The bitmap is 1/128 of what the main pass moves, so what
// bounds this one is latency, and what matters is that neighbouring tiles of different tensors do not wait for each other.  (Eight
// checkpoints of the 410M shape, 405 MB of bitmaps, two thirds of the tensors one tile: with a wave for eight tiles of one tensor 234 us in
// three launches, some of the waves with thirty-two tensors to look up one after the other; now 87 in one.)
// The counts of a run of tiles, the first of a tensor up to a multiple of SCAN_BLOCK or SCAN_BLOCK more, are also added up in
// dec_part, where the scan finds what lies before its run.
constexpr u32 SCAN_BLOCK = EXCP_SCAN_TILES;
// The run that a tile of a tensor beginning at `first` belongs to: the tensor's number, or that of the block behind all tensors.
__device__ __forceinline__ u32 run_of(u32 tile, u32 t, u32 first, u32 ntensors) {
    return tile / SCAN_BLOCK == first / SCAN_BLOCK ? t : ntensors + tile / SCAN_BLOCK;
}
__device__ __forceinline__ u32 sum_of_eight(u32 x) {       // in all of them: neighbours, pairs, then the two quads
    x += dpp_u32<0xb1, 0xf>(0u, x);           // quad_perm 1 0 3 2
    x += dpp_u32<0x4e, 0xf>(0u, x);           // quad_perm 2 3 0 1
    x += dpp_u32<0x141, 0xf>(0u, x);          // row_half_mirror
    return x;
}
template <int WHICH>
__global__ __launch_bounds__(EXCP_THREADS) void k_decode_count(Workspace w, u32 ntensors, u32 ntiles) {
    extern __shared__ u32 s_begin[];                       // [ntensors + 1]
    __shared__ u32 s_run[EXCP_THREADS / 64], s_sum[EXCP_THREADS / 64];
    const u32 lane = threadIdx.x & 63u, group = lane >> 3, l = lane & 7u;
    const u32 wave = (u32)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    load_tile_table(s_begin, w.tile_begin, ntensors);
    const u32 nwaves = gridDim.x * (EXCP_THREADS / 64), wid = blockIdx.x * (EXCP_THREADS / 64) + wave;
    const u32 t_lo = (u32)(((u64)wid * ntiles) / nwaves), t_hi = (u32)(((u64)(wid + 1u) * ntiles) / nwaves);
    u32 *part = w.dec_part + (WHICH == 0 ? 0u : w.dec_part_stride), *table = WHICH == 0 ? w.dec_cnt_w : w.dec_cnt_o;
    u32 t = 0, first = 0, end = 0;                         // the group's tensor, its first tile, one past its last
    u64 n = 0, most = 0, pop = 0;                          // its elements; of its survivors: bits in bitmap_o, counted
    bool good = false, per_element = false;
    const EXCP_GLOBAL u64 *bm = nullptr;
    u32 run = 0xffffffffu, sum = 0;                        // counts not yet handed over, and the run they belong to
    for (u32 tile0 = t_lo; tile0 < t_hi; tile0 += 8u) {
        const u32 tile = tile0 + group;
        const bool have = tile < t_hi;
        if (have && tile >= end) {
            t = find_owner(s_begin, ntensors, tile);
            first = s_begin[t]; end = s_begin[t + 1u];
            const DDesc &D = w.ddesc[t];
            const DState &S = w.dst[t];
            n = D.n;
            good = S.status == 0 && (WHICH == 0 || wants_moments(D));          // (bitmap_o only where moments are wanted)
            bm = gptr((const u64 *)(D.blob + (WHICH == 0 ? S.off_bw : S.off_bo)));
            if (WHICH == 1) { most = S.n_w; pop = S.pop_w; per_element = (S.flags & 8u) != 0u; }
        }
        u32 cnt = 0;
        if (have && good) {
            const u64 base = (u64)(tile - first) * EXCP_TILE;
            if (WHICH == 0) {
                const u64 word0 = (base >> 6) + 2u * l;
                if (base + EXCP_TILE <= n) {
                    typedef u64 pair __attribute__((ext_vector_type(2)));       // (sections begin at multiples of 16 bytes)
                    pair v[4];
#pragma unroll
                    for (u32 k = 0; k < 4; ++k) v[k] = *(const EXCP_GLOBAL pair *)(bm + word0 + 16u * k);
#pragma unroll
                    for (u32 k = 0; k < 4; ++k) cnt += (u32)(__popcll(v[k].x) + __popcll(v[k].y));
                } else {
                    // bits beyond n must be clear in a well-formed blob; ignore them here
                    const u64 nwords = excp_words(n);
#pragma unroll
                    for (u32 k = 0; k < 8; ++k) {
                        const u64 word = word0 + 16u * (k >> 1) + (k & 1u);
                        if (word < nwords) cnt += (u32)__popcll(bm[word] & (n - word * 64u < 64u ? (1ull << (n - word * 64u)) - 1ull : ~0ull));
                    }
                }
            } else {
                u64 p0 = w.dec_cnt_w[tile], p1 = tile + 1u < end ? (u64)w.dec_cnt_w[tile + 1u] : pop;
                p1 = min(p1, most);                        // damaged blob: stay inside the bitmap
                p0 = min(p0, p1);
                if (per_element) { p0 = base; p1 = min(n, base + EXCP_TILE); }      // one bit per element: the tile's own range
                if (p0 < p1) {
                    const u64 w0 = p0 >> 6, w1 = (p1 - 1u) >> 6;
                    for (u64 wi = w0 + l; wi <= w1; wi += 32u) {
                        u64 v[4];
#pragma unroll
                        for (u32 k = 0; k < 4; ++k) v[k] = wi + 8u * k <= w1 ? bm[wi + 8u * k] : 0ull;
#pragma unroll
                        for (u32 k = 0; k < 4; ++k) {
                            const u64 at = wi + 8u * k;
                            cnt += (u32)__popcll(v[k] & range_mask(at == w0 ? (u32)(p0 & 63u) : 0u, at == w1 ? (u32)((p1 - 1u) & 63u) + 1u : 64u));
                        }
                    }
                }
            }
        }
        cnt = sum_of_eight(cnt);
        if (have) {
            if (l == 0u) table[tile] = cnt;
            const u32 r = run_of(tile, t, first, ntensors);
            if (r != run) {
                if (l == 0u && sum) atomicAdd(&part[run], sum);
                run = r; sum = 0;
            }
            sum += cnt;
        }
    }
    // Usually the workgroup's tiles are all of one run: then one atomic.  (One from every wave: 512 at the same address, 24 ragged
    // tensors 53 instead of 8 us.)
    const u32 first_run = (u32)__builtin_amdgcn_readfirstlane((int)run);
    const bool one_run = __all(run == first_run || sum == 0u);
    const u32 total = wave_sum_u32(l == 0u ? sum : 0u);
    if (!one_run && l == 0u && sum) atomicAdd(&part[run], sum);
    if (lane == 0u) { s_run[wave] = first_run; s_sum[wave] = one_run ? total : 0u; }
    __syncthreads();
    if (threadIdx.x != 0) return;
#pragma unroll
    for (u32 v = 0; v < EXCP_THREADS / 64; ++v) {
        u32 mine = s_sum[v];
#pragma unroll
        for (u32 x = v + 1u; x < EXCP_THREADS / 64; ++x) if (s_run[x] == s_run[v]) { mine += s_sum[x]; s_sum[x] = 0u; }
        if (mine) atomicAdd(&part[s_run[v]], mine);
    }
}

// Exclusive scan of the per-tile counts of every tensor, a workgroup to a run of tiles (see k_decode_count): the first of every
// tensor, then those that begin at a multiple of SCAN_BLOCK.  The workgroup of a tensor's last run checks the total against the header
// and, where nothing can change the results after this, writes the record.
template <int WHICH>
__global__ __launch_bounds__(EXCP_THREADS) void k_decode_scan(Workspace w, u32 ntensors, u32 records) {
    __shared__ u32 s_wave[EXCP_THREADS / 64], s_before[EXCP_THREADS / 64], s_first[EXCP_THREADS / 64];
    const u32 tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    const u32 *begin = w.tile_begin, *part = w.dec_part + (WHICH == 0 ? 0u : w.dec_part_stride);
    u32 *table = WHICH == 0 ? w.dec_cnt_w : w.dec_cnt_o;
    const bool inner = blockIdx.x >= ntensors;             // not a tensor's first run
    const u32 s0 = inner ? (blockIdx.x - ntensors) * SCAN_BLOCK : begin[blockIdx.x];
    u32 t = blockIdx.x;
    if (inner) {                                           // the last tensor that begins before
        u32 c = 0;
        for (u32 i = tid; i < ntensors; i += EXCP_THREADS) c += begin[i] < s0;
        c = wave_sum_u32(c);
        if (lane == 0u) s_first[wave] = c;
        __syncthreads();
        c = (s_first[0] + s_first[1]) + (s_first[2] + s_first[3]);
        if (c == 0u) return;
        t = c - 1u;
    }
    const DDesc &D = w.ddesc[t];
    const u32 tb = begin[t], te = begin[t + 1u];
    if (inner && te <= s0) return;                         // (tensors without tiles apart, one begins here: its own workgroup takes the run)
    const u32 s1 = min(te, (s0 / SCAN_BLOCK + 1u) * SCAN_BLOCK);
    const bool last = s1 == te;
    if (WHICH == 1 && !wants_moments(D)) {                 // bitmap_o is not used for this one
        if (records && last && tid == 0) decode_record(w, t, D.n, w.dst[t]);
        return;
    }
    u32 v[SCAN_BLOCK / EXCP_THREADS], local = 0;
#pragma unroll
    for (u32 k = 0; k < SCAN_BLOCK / EXCP_THREADS; ++k) {
        const u32 i = s0 + tid * (SCAN_BLOCK / EXCP_THREADS) + k;
        v[k] = i < s1 ? table[i] : 0u;
        local += v[k];
    }
    u32 before = 0;                                        // in the runs before this one
    if (inner) {
        if (tid == 0) before = part[t];
        for (u32 b = tb / SCAN_BLOCK + 1u + tid; b < s0 / SCAN_BLOCK; b += EXCP_THREADS) before += part[ntensors + b];
    }
    before = wave_sum_u32(before);
    const u32 incl = wave_incl_scan_u32(local);
    if (lane == 63u) { s_before[wave] = before; s_wave[wave] = incl; }
    __syncthreads();
    const u32 carry = (s_before[0] + s_before[1]) + (s_before[2] + s_before[3]);
    u32 excl = carry + incl - local;
    for (u32 q = 0; q < wave; ++q) excl += s_wave[q];
#pragma unroll
    for (u32 k = 0; k < SCAN_BLOCK / EXCP_THREADS; ++k) {
        const u32 i = s0 + tid * (SCAN_BLOCK / EXCP_THREADS) + k;
        if (i < s1) table[i] = excl;
        excl += v[k];
    }
    if (!last || tid != 0) return;
    DState &S = w.dst[t];
    const u64 total = (u64)carry + ((s_wave[0] + s_wave[1]) + (s_wave[2] + s_wave[3]));
    if (WHICH == 0) { S.pop_w = total; if (S.status == 0 && total != S.n_w) S.status = -4; }
    else { S.pop_o = total; if (S.status == 0 && total != S.n_o) S.status = -4; }
    if (records) decode_record(w, t, D.n, S);
}

// Four consecutive floats at an address that is only known to be 4-byte aligned.
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));

#define DEC_CODE_WORDS 1032   // u32 words of one tile's codes: 4096 codes x 8 bits / 32 + slack
#define DEC_OBIT_WORDS 136    // u32 words of bitmap_o covering one tile's survivors: 4096 / 32 + slack

// Stage u32 words [first, first + count) of a blob section into LDS.
__device__ __forceinline__ void stage_words(u32 *dst, const EXCP_GLOBAL u32 *src, u32 count) {
    for (u32 i = threadIdx.x; i < count; i += EXCP_THREADS) dst[i] = src[i];
}

// 32 stream bits starting at bit p of a staged word array (p / 32 + 1 must be inside the array).
__device__ __forceinline__ u32 window32(const u32 *s, u32 p) {
    const u32 i = p >> 5;
    return __builtin_amdgcn_alignbit(s[i + 1], s[i], p & 31u);
}

// One tile (4096 elements) per workgroup iteration.  Each wave scans the tile's 64 bitmap words,
// the workgroup stages the tile's contiguous run of packed codes (and, for the moments, the run of
// bitmap_o bits of its survivors with their prefix counts) in LDS, then every lane reconstructs four
// consecutive elements: the codes of its survivors are consecutive fields of the staged stream, so
// one 32-bit window read per lane holds all of them.
//
// RAW: blobs written without quantisation hold fp32 values where the others hold codes; a lane reads
// its survivors' values straight from the blob (consecutive lanes, consecutive addresses).  Such
// blobs are skipped by the other instantiations, and this one skips everything else.
//
// WMODE: which weight storage this instantiation takes (blob flags bits 4-5): 0 = fp32 blobs only,
// 1 = blobs of 16-bit weights only (fp16 / bf16: widened exactly, the sum rounded to nearest even
// into the format, pruned positions keep their bits), 2 = both, decided per tensor.
template <bool MOMENTS, bool RAW, int WMODE>
__device__ __forceinline__ void decode_tiles(const Workspace &w, u32 ntensors, u32 ntiles) {
    __shared__ float s_book[RAW ? 1 : 3 * 256];
    __shared__ u32 s_tiles[EXCP_MAX_GROUP_TENSORS + 1];
    __shared__ u32 s_cw[RAW ? 2 : DEC_CODE_WORDS];
    __shared__ u32 s_cm[MOMENTS && !RAW ? DEC_CODE_WORDS : 2], s_cv[MOMENTS && !RAW ? DEC_CODE_WORDS : 2];
    __shared__ u32 s_ow[MOMENTS ? DEC_OBIT_WORDS : 1], s_oex[MOMENTS ? DEC_OBIT_WORDS : 1];
    const u32 tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    u32 cur_t = 0xffffffffu;
    load_tile_table(s_tiles, w.tile_begin, ntensors);
    for (u32 tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        const u32 owner = find_owner(s_tiles, ntensors, tile);
        const u32 t = w.cdesc ? w.cdesc[owner].first_desc + w.cdesc[owner].steps - 1u : owner;      // (of a chain: the last checkpoint)
        const DDesc &D = w.ddesc[t];
        const DState &S = w.dst[t];
        if (S.status != 0) continue;                       // same decision for the whole workgroup
        if ((S.nbits == EXCP_RAW_BITS) != RAW) continue;
        const u32 wt = WMODE == 0 ? 0u : excp_wtype(S.flags);
        if (WMODE == 0 && excp_wtype(S.flags) != 0u) continue;
        if (WMODE == 1 && wt == 0u) continue;
        const bool bf = wt == 2u;
        const u32 nbits = S.nbits, E = RAW ? 0u : 1u << (nbits & 15u), cmask = E - 1u;
        const u64 n = D.n;
        const u32 ltile = tile - s_tiles[owner], ctile = w.cdesc ? D.tile_begin + ltile : tile;      // (in the tensor; in the tables of counts)
        const u64 base = (u64)ltile * EXCP_TILE;
        const u32 rem = (n - base < (u64)EXCP_TILE) ? (u32)(n - base) : EXCP_TILE;   // elements of this tile
        const unsigned char *blob = D.blob;
        const bool has_w = D.W_out != nullptr;
        const bool has_m = MOMENTS && D.m_out != nullptr;
        const bool has_v = MOMENTS && D.v_out != nullptr;
        const bool moments = has_m || has_v;
        if (!has_w && !moments) continue;                  // nothing to write for this one

        // previous weights of the lane's 4 x 4 elements: issued first, consumed last
        float wp[4][4];
        us4 hp[4];                                         // 16-bit weights stay as they are until the sum
        if (has_w && WMODE != 0 && wt != 0u) {
            const EXCP_GLOBAL unsigned short *Hp = gptr((const unsigned short *)D.Wp) + base;
            const bool vec = ((uintptr_t)D.Wp & 7u) == 0u;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const u32 off = wave * 1024u + (u32)k * 256u + lane * 4u;
                if (vec && off + 4u <= rem) hp[k] = READ_ONCE(us4, (Hp + off));
                else {
#pragma unroll
                    for (int j = 0; j < 4; ++j) hp[k][j] = (off + (u32)j < rem) ? Hp[off + (u32)j] : (unsigned short)0;
                }
            }
        } else if (has_w) {
            const EXCP_GLOBAL float *Wp = gptr(D.Wp) + base;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const u32 off = wave * 1024u + (u32)k * 256u + lane * 4u;
                if (off + 4u <= rem) {
                    const f4u x = READ_ONCE(f4u, (Wp + off));
                    wp[k][0] = x.x; wp[k][1] = x.y; wp[k][2] = x.z; wp[k][3] = x.w;
                } else {
#pragma unroll
                    for (int j = 0; j < 4; ++j) wp[k][j] = (off + (u32)j < rem) ? Wp[off + (u32)j] : 0.f;
                }
            }
        }

        // survivors before each of the tile's 64 bitmap words (every wave computes all 64)
        u64 myword = 0;
        {
            const u64 wword = (u64)ltile * 64 + lane;
            const u32 bits_here = (lane * 64u < rem) ? min(64u, rem - lane * 64u) : 0u;
            if (bits_here) myword = gptr((const u64 *)(blob + S.off_bw))[wword];
            if (bits_here < 64u) myword &= (1ull << bits_here) - 1ull;
        }
        const u32 pc = __popcll(myword);
        u32 incl = wave_incl_scan_u32(pc);
        const u32 excl = incl - pc;
        const u32 cnt = __shfl(incl, 63, WAVE);            // survivors of this tile
        const u32 q_tile = w.dec_cnt_w[ctile];             // survivors before this tile
        const u64 wbit0 = (u64)q_tile * nbits;
        const u32 woff = (u32)(wbit0 & 31ull);
        u32 o_tile = 0, ocnt = 0, moff = 0, ooff = 0;
        const bool nw2m = MOMENTS && (S.flags & 8u) != 0u;    // M_o bits per element instead of per kept residual
        if (MOMENTS && moments) {
            o_tile = w.dec_cnt_o[ctile];
            const u32 o_next = (ltile + 1u < D.tile_count) ? w.dec_cnt_o[ctile + 1u] : (u32)S.pop_o;
            ocnt = o_next - o_tile;
            moff = (u32)(((u64)o_tile * nbits) & 31ull);
            ooff = nw2m ? 0u : q_tile & 31u;
        }

        __syncthreads();                                   // the previous tile's LDS readers are done
        if (!RAW && t != cur_t) {
            const EXCP_GLOBAL float *books = gptr((const float *)(blob + EXCP_HEADER));
            for (u32 i = tid; i < 3u * E; i += EXCP_THREADS) s_book[(i / E) * 256u + (i % E)] = books[i];
            cur_t = t;
        }
        if (!RAW) stage_words(s_cw, gptr((const u32 *)(blob + S.off_cw)) + (wbit0 >> 5), (woff + cnt * nbits + 31u) >> 5);
        if (MOMENTS && moments) {
            const u64 mbit0 = (u64)o_tile * nbits;
            const u32 mwords = (moff + ocnt * nbits + 31u) >> 5;
            if (!RAW) {
                stage_words(s_cm, gptr((const u32 *)(blob + S.off_cm)) + (mbit0 >> 5), mwords);
                stage_words(s_cv, gptr((const u32 *)(blob + S.off_cv)) + (mbit0 >> 5), mwords);
            }
            if (wave == 0) {
                // bitmap_o bits [q_tile, q_tile + cnt) as u32 words, with the count of set bits before each word
                const EXCP_GLOBAL u32 *bo = gptr((const u32 *)(blob + S.off_bo)) + (nw2m ? ltile * (EXCP_TILE / 32u) : q_tile >> 5);
                const u32 obits_total = nw2m ? rem : ooff + cnt;
                const u32 owords = (obits_total + 31u) >> 5;       // <= 129
                u32 carry = 0;
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    const u32 i = lane + 64u * (u32)c;
                    u32 word = (i < owords) ? bo[i] : 0u;
                    if (i == 0u) word &= ~((1u << ooff) - 1u);     // bits of earlier tiles' survivors
                    if (nw2m && i + 1u == owords && (obits_total & 31u)) word &= (1u << (obits_total & 31u)) - 1u;   // bits past the last element
                    const u32 opc = __popc(word);
                    u32 oincl = wave_incl_scan_u32(opc);
                    if (i < DEC_OBIT_WORDS) { s_ow[i] = word; s_oex[i] = carry + oincl - opc; }
                    carry += __shfl(oincl, 63, WAVE);
                }
            }
        }
        __syncthreads();

#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const u32 off = wave * 1024u + (u32)k * 256u + lane * 4u;   // first of the lane's 4 elements
            const u32 wq = wave * 16u + (u32)k * 4u + (lane >> 4);       // their bitmap word
            const u32 sub = (lane & 15u) * 4u;                           // their first bit in it
            const u32 wlo = __shfl((u32)myword, wq, WAVE), whi = __shfl((u32)(myword >> 32), wq, WAVE);
            const u32 wex = __shfl(excl, wq, WAVE);
            const u64 word = ((u64)whi << 32) | wlo;
            const u32 nib = (u32)(word >> sub) & 15u;
            const u32 r = wex + __popcll(word & ((1ull << sub) - 1ull));   // tile rank of the lane's first survivor
            u32 f = RAW ? 0u : window32(s_cw, woff + r * nbits);
            const EXCP_GLOBAL float *xw = gptr((const float *)(blob + S.off_cw)) + q_tile + r;   // RAW: the lane's first survivor
            if (has_w && WMODE != 0 && wt != 0u) {
                us4 o16;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const bool kept = (nib >> j) & 1u;
                    float c;
                    if (RAW) { c = kept ? *xw : 0.f; xw += kept; }
                    else c = s_book[f & cmask];
                    const u32 h = hp[k][j];
                    o16[j] = (unsigned short)(kept ? w16_narrow(w16_widen(h, bf) + c, bf) : h);
                    f = kept ? (f >> nbits) : f;
                }
                EXCP_GLOBAL unsigned short *Ho = gptr((unsigned short *)D.W_out) + base;
                if (((uintptr_t)D.W_out & 7u) == 0u && off + 4u <= rem) WRITE_ONCE(us4, (Ho + off), o16);
                else {
#pragma unroll
                    for (int j = 0; j < 4; ++j) if (off + (u32)j < rem) Ho[off + (u32)j] = o16[j];
                }
            } else if (has_w) {
                float out[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const bool kept = (nib >> j) & 1u;
                    float c;
                    if (RAW) { c = kept ? *xw : 0.f; xw += kept; }
                    else c = s_book[f & cmask];
                    out[j] = kept ? wp[k][j] + c : wp[k][j];
                    f = kept ? (f >> nbits) : f;
                }
                EXCP_GLOBAL float *Wo = gptr(D.W_out) + base;
                if (off + 4u <= rem) {
                    f4u y; y.x = out[0]; y.y = out[1]; y.z = out[2]; y.w = out[3];
                    WRITE_ONCE(f4u, (Wo + off), y);
                } else {
#pragma unroll
                    for (int j = 0; j < 4; ++j) if (off + (u32)j < rem) Wo[off + (u32)j] = out[j];
                }
            }
            if (MOMENTS && moments) {
                const u32 bpos = nw2m ? off : ooff + r;                   // the first survivor's (element's) bit in the staged bitmap_o
                const u32 bi = bpos >> 5, bsh = bpos & 31u;
                u32 obits = __builtin_amdgcn_alignbit(s_ow[bi + 1], s_ow[bi], bsh);
                const u32 orank = s_oex[bi] + __popc(s_ow[bi] & ((1u << bsh) - 1u));
                u32 fm = RAW ? 0u : window32(s_cm, moff + orank * nbits);
                u32 fv = RAW ? 0u : window32(s_cv, moff + orank * nbits);
                const EXCP_GLOBAL float *xm = gptr((const float *)(blob + S.off_cm)) + o_tile + orank;   // RAW
                const EXCP_GLOBAL float *xv = gptr((const float *)(blob + S.off_cv)) + o_tile + orank;
                float om[4], ov[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const bool kept = (nib >> j) & 1u;
                    const bool ko = (kept || nw2m) && (obits & 1u);
                    if (RAW) {
                        om[j] = ko ? *xm : 0.f; ov[j] = ko ? *xv : 0.f;
                        xm += ko; xv += ko;
                    } else {
                        om[j] = ko ? s_book[256u + (fm & cmask)] : 0.f;
                        ov[j] = ko ? s_book[512u + (fv & cmask)] : 0.f;
                    }
                    obits = (kept || nw2m) ? (obits >> 1) : obits;
                    fm = ko ? (fm >> nbits) : fm;
                    fv = ko ? (fv >> nbits) : fv;
                }
                if (off + 4u <= rem) {
                    f4u y;
                    if (has_m) { y.x = om[0]; y.y = om[1]; y.z = om[2]; y.w = om[3]; WRITE_ONCE(f4u, (gptr(D.m_out) + base + off), y); }
                    if (has_v) { y.x = ov[0]; y.y = ov[1]; y.z = ov[2]; y.w = ov[3]; WRITE_ONCE(f4u, (gptr(D.v_out) + base + off), y); }
                } else {
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        if (off + (u32)j < rem) {
                            if (has_m) gptr(D.m_out)[base + off + (u32)j] = om[j];
                            if (has_v) gptr(D.v_out)[base + off + (u32)j] = ov[j];
                        }
                    }
                }
            }
        }
    }
}

template <bool MOMENTS>
__global__ __launch_bounds__(EXCP_THREADS, MOMENTS ? 6 : 8) void k_decode_main(Workspace w, u32 ntensors, u32 ntiles) {
    if ((*w.dec_kinds & 1u) == 0u) return;                 // no blob of fp32 weights in this group
    decode_tiles<MOMENTS, false, 0>(w, ntensors, ntiles);
}
// The same for blobs of 16-bit weights (most batches hold none).
template <bool MOMENTS>
__global__ __launch_bounds__(EXCP_THREADS, MOMENTS ? 6 : 8) void k_decode_main16(Workspace w, u32 ntensors, u32 ntiles) {
    if ((*w.dec_kinds & 2u) == 0u) return;
    decode_tiles<MOMENTS, false, 1>(w, ntensors, ntiles);
}
// Blobs written without quantisation (most batches hold none).
template <bool MOMENTS>
__global__ __launch_bounds__(EXCP_THREADS) void k_decode_raw(Workspace w, u32 ntensors, u32 ntiles) {
    if ((*w.dec_kinds & 4u) == 0u) return;
    decode_tiles<MOMENTS, true, 2>(w, ntensors, ntiles);
}
// The codes themselves, as the per-element code tensors of Sec. 4.2: 0 where pruned; two codes per byte when nbits <= 4, the even
// element in the low four bits; one code per byte otherwise.
//
// It reads and writes 2 bytes an element, so what bounds it is the instructions between.  A wave has a tile to itself and takes it
// in four quarters, sixteen consecutive elements to a lane, without barriers.  Eight elements are a byte of the bitmap: their codes,
// at most eight consecutive fields of the stream, are spread over the bytes of two registers, and the bitmap byte looks up
// the byte selectors that put them in their elements' places (0 where pruned) -- twelve instructions for eight elements, where
// taking one code after the other from a window is five for each.  The M_o bits go from survivors to elements four at a time by
// a table too; their running count is then the moments' rank.  Everything of a tile that comes from memory is asked for as soon as
// its place is known: bitmap; codes of the weights and bitmap_o; codes of the moments.  (333 M elements of 4 bits, all three: a tile to
// a workgroup, four elements to a lane, one code after the other 545 us; now 188, 3.5 TB/s.  Stores past the caches 191, five or
// seven workgroups to a compute unit 187 and 183.)
constexpr u32 EXPORT_WAVES = EXCP_THREADS / 64, EXPORT_PER_CU = 12;
constexpr u32 EXPORT_CODE_WORDS = 260;       // of 1024 codes of 8 bits, one for the first bit's place, two for what a window reads beyond

// `split`: a tile to a workgroup, a quarter to each of its waves, up to four tiles a compute unit, where one tile after another in a
// wave is what is waited for; the waves then all work out all the ranks, which beyond that is work the others would wait for
// (5 tiles 7.9 -> 6.3 us, 35 tiles 9.9 -> 6.3 us).
__global__ __launch_bounds__(EXCP_THREADS, 6) void k_export_dense(Workspace w, u32 ntensors, u32 ntiles, u32 split) {
    __shared__ u64 s_pick[256];                            // per bitmap byte: selectors of the even elements, of the odd ones
    __shared__ unsigned char s_deposit[256];               // (four bits to place << 4 | four bits of bitmap): the bits in their places
    __shared__ u32 s_tiles[EXCP_MAX_GROUP_TENSORS + 1];
    __shared__ u32 s_code[EXPORT_WAVES][3][EXPORT_CODE_WORDS], s_bo[EXPORT_WAVES][DEC_OBIT_WORDS];
    const u32 tid = threadIdx.x, lane = tid & 63u;
    const u32 wave = (u32)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
    {
        static_assert(EXCP_THREADS == 256, "a thread makes an entry of either table");
        u32 pick[2] = {0u, 0u}, r = 0, place = 0, bits = tid >> 4;
#pragma unroll
        for (u32 j = 0; j < 8; ++j) {
            const bool kept = tid >> j & 1u;
            // code r of the eight is byte r / 2 of the register of the even ones (bytes 0 to 3) or odd ones (4 to 7); 12 gives zeros
            pick[j & 1u] |= (kept ? (r & 1u) * 4u + (r >> 1) : 12u) << (8u * (j >> 1));
            r += kept;
        }
#pragma unroll
        for (u32 j = 0; j < 4; ++j) if (tid >> j & 1u) { place |= (bits & 1u) << j; bits >>= 1; }
        s_pick[tid] = (u64)pick[1] << 32 | pick[0];
        s_deposit[tid] = (unsigned char)place;
    }
    load_tile_table(s_tiles, w.tile_begin, ntensors);
    u32 t = 0, first = 0, end = 0;                         // the tensor in hand, its first tile, one past its last
    const u32 q_lo = split ? wave : 0u, q_hi = split ? wave + 1u : 4u;               // the wave's quarters
    for (u32 tile = split ? blockIdx.x : blockIdx.x * EXPORT_WAVES + wave; tile < ntiles; tile += split ? gridDim.x : gridDim.x * EXPORT_WAVES) {
        if (tile >= end) {                                 // (a wave's tiles only go up)
            t = (u32)__builtin_amdgcn_readfirstlane((int)find_owner(s_tiles, ntensors, tile));
            first = (u32)__builtin_amdgcn_readfirstlane((int)s_tiles[t]);
            end = (u32)__builtin_amdgcn_readfirstlane((int)s_tiles[t + 1u]);
        }
        const EXCP_CONSTANT DDesc *D = (const EXCP_CONSTANT DDesc *)(uintptr_t)(w.ddesc + t);
        const EXCP_CONSTANT DState *S = (const EXCP_CONSTANT DState *)(uintptr_t)(w.dst + t);
        if (S->status != 0 || S->nbits > 8u) continue;
        unsigned char *const dst[3] = {D->cw, D->cm, D->cv};
        const bool moments = dst[1] != nullptr || dst[2] != nullptr;
        if (dst[0] == nullptr && !moments) continue;
        const u32 nbits = S->nbits, ltile = tile - first;
        const bool per_element = (S->flags & 8u) != 0u;    // M_o bits per element instead of per kept residual
        const u64 n = D->n, base = (u64)ltile * EXCP_TILE;
        const u32 rem = n - base < (u64)EXCP_TILE ? (u32)(n - base) : EXCP_TILE;
        const unsigned char *blob = D->blob;
        u32 *bo = s_bo[wave];
        const EXCP_CONSTANT u32 *count_w = (const EXCP_CONSTANT u32 *)(uintptr_t)w.dec_cnt_w, *count_o = (const EXCP_CONSTANT u32 *)(uintptr_t)w.dec_cnt_o;
        const u32 q_tile = count_w[tile];                  // survivors before the tile
        // sixteen bits of a bitmap with a bit per element: those of the lane's elements in quarter q
        auto bits_at = [&](u64 section, u32 q) {
            const u32 off = q * 1024u + lane * 16u, left = rem > off ? min(rem - off, 16u) : 0u;
            const u32 x = left ? (u32)gptr((const unsigned short *)(blob + section))[(u64)ltile * 256u + q * 64u + lane] : 0u;
            return x & ((1u << left) - 1u);
        };
        u32 keep[4], rank[4], at[5];                       // the lane's bitmap bits, survivors in front of them in the tile; those before every quarter
        u32 keep_o[4], rank_o[4], at_o[5];                 // the same of the moments
#pragma unroll
        for (u32 q = 0; q < 4; ++q) keep[q] = bits_at(S->off_bw, q);
        if (moments && per_element) {
#pragma unroll
            for (u32 q = 0; q < 4; ++q) keep_o[q] = bits_at(S->off_bo, q);
        }
        auto ranks = [&](const u32 (&bits)[4], u32 (&r)[4], u32 (&begin)[5]) {
            begin[0] = 0u;
#pragma unroll
            for (u32 q = 0; q < 4; ++q) {
                const u32 pc = (u32)__popc(bits[q]), incl = wave_incl_scan_u32(pc);
                r[q] = incl - pc + begin[q];
                begin[q + 1u] = begin[q] + last_lane_u32(incl);
            }
        };
        // a quarter's codes of one stream: where they begin, words, and the first 64 words, one to a lane (without any: any word of the blob)
        struct Codes { u32 off, words, word; const EXCP_GLOBAL u32 *from; };
        auto open = [&](u64 section, u64 before, u32 count) {
            Codes c;
            const u64 bit0 = before * nbits;
            c.off = (u32)(bit0 & 31ull);
            c.words = count ? (c.off + count * nbits + 31u) >> 5 : 0u;
            c.from = gptr((const u32 *)(c.words ? blob + section + (bit0 >> 5) * 4u : blob));
            c.word = c.from[lane < c.words ? lane : 0u];
            return c;
        };
        Codes cw[4], cm[4], cv[4];
        ranks(keep, rank, at);
        if (dst[0] != nullptr) {
#pragma unroll
            for (u32 q = 0; q < 4; ++q) if (q >= q_lo && q < q_hi) cw[q] = open(S->off_cw, (u64)q_tile + at[q], at[q + 1u] - at[q]);
        }
        if (moments) {
            if (!per_element) {
                // the survivors' M_o bits, then placed at their elements
                const u32 ooff = q_tile & 31u, words = at[4] ? (ooff + at[4] + 31u) >> 5 : 0u;      // <= 129
                const EXCP_GLOBAL u32 *from = gptr((const u32 *)(blob + S->off_bo)) + (q_tile >> 5);
                u32 x[3];
#pragma unroll
                for (u32 k = 0; k < 3; ++k) x[k] = lane + 64u * k < words ? from[lane + 64u * k] : 0u;
                wave_lds_fence();                          // (the tile before is done with them)
#pragma unroll
                for (u32 k = 0; k < 3; ++k) if (lane + 64u * k < DEC_OBIT_WORDS) bo[lane + 64u * k] = x[k];
                wave_lds_fence();
#pragma unroll
                for (u32 q = 0; q < 4; ++q) {
                    u32 bits = window32(bo, ooff + rank[q]), placed = 0;
#pragma unroll
                    for (u32 j = 0; j < 4; ++j) {
                        const u32 four = keep[q] >> (4u * j) & 15u;
                        placed |= (u32)s_deposit[(bits & 15u) << 4 | four] << (4u * j);
                        bits >>= __popc(four);
                    }
                    keep_o[q] = placed;
                }
            }
            ranks(keep_o, rank_o, at_o);
            const u64 o_tile = count_o[tile];
#pragma unroll
            for (u32 q = 0; q < 4; ++q) {
                const u32 count = at_o[q + 1u] - at_o[q];
                if (q < q_lo || q >= q_hi) continue;
                if (dst[1] != nullptr) cm[q] = open(S->off_cm, o_tile + at_o[q], count);
                if (dst[2] != nullptr) cv[q] = open(S->off_cv, o_tile + at_o[q], count);
            }
        }
        const u32 one = (1u << nbits) - 1u, two = (1u << 2u * nbits) - 1u;
#pragma unroll
        for (u32 q = 0; q < 4; ++q) {
            const u32 off = q * 1024u + lane * 16u;
            if (q < q_lo) continue;
            if (q >= q_hi || q * 1024u >= rem) break;
            const u32 left = rem > off ? min(rem - off, 16u) : 0u;
            wave_lds_fence();                              // (the quarter before is done with its codes)
#pragma unroll
            for (u32 k = 0; k < 3; ++k) {
                if (dst[k] == nullptr) continue;
                const Codes &c = k == 0u ? cw[q] : (k == 1u ? cm[q] : cv[q]);
                u32 *code = s_code[wave][k];
                code[lane] = c.word;
#pragma unroll 1
                for (u32 i = 64u + lane; i < c.words; i += 64u) code[i] = c.from[i];
            }
            wave_lds_fence();
#pragma unroll
            for (u32 k = 0; k < 3; ++k) {
                if (dst[k] == nullptr) continue;
                const Codes &c = k == 0u ? cw[q] : (k == 1u ? cm[q] : cv[q]);
                const u32 *code = s_code[wave][k];
                const u32 bits = k == 0u ? keep[q] : keep_o[q];
                const u32 r = k == 0u ? rank[q] - at[q] : rank_o[q] - at_o[q];
                u32 out[4];                                // the sixteen codes, two or one to a byte
#pragma unroll
                for (u32 h = 0; h < 2; ++h) {
                    const u32 eight = bits >> (8u * h) & 255u;
                    const u32 p = c.off + (r + (h ? (u32)__popc(bits & 255u) : 0u)) * nbits;
                    const u64 pick = s_pick[eight];
                    if (nbits <= 4u) {
                        u32 x = window32(code, p);
                        if (nbits < 4u) {                  // fields of two or three bits: half a byte apart
                            const u32 four = (1u << 4u * nbits) - 1u, pair = two * 0x00010001u;
                            x = (x & four) | (x << (16u - 4u * nbits) & four << 16);
                            x = (x & pair) | (x << (8u - 2u * nbits) & pair << 8);
                        }
                        const u32 low = one * 0x01010101u, even = x & low, odd = x >> nbits & low;
                        out[h] = __builtin_amdgcn_perm(odd, even, (u32)pick) | __builtin_amdgcn_perm(odd, even, (u32)(pick >> 32)) << 4;
                    } else {
                        u32 x[2];
#pragma unroll
                        for (u32 y = 0; y < 2; ++y) {      // four fields of five to eight bits, a byte apart
                            x[y] = window32(code, p + 4u * nbits * y);
                            x[y] = (x[y] & two) | (x[y] << (16u - 2u * nbits) & two << 16);
                            x[y] = (x[y] & one * 0x00010001u) | (x[y] << (8u - nbits) & (one * 0x00010001u) << 8);
                        }
                        const u32 even = __builtin_amdgcn_perm(x[1], x[0], 0x06040200u), odd = __builtin_amdgcn_perm(x[1], x[0], 0x07050301u);
                        const u32 e = __builtin_amdgcn_perm(odd, even, (u32)pick), o = __builtin_amdgcn_perm(odd, even, (u32)(pick >> 32));
                        out[2u * h] = __builtin_amdgcn_perm(o, e, 0x05010400u);
                        out[2u * h + 1u] = __builtin_amdgcn_perm(o, e, 0x07030602u);
                    }
                }
                typedef u32 u2 __attribute__((ext_vector_type(2)));
                typedef u32 u4 __attribute__((ext_vector_type(4)));
                if (nbits <= 4u) {
                    EXCP_GLOBAL unsigned char *to = gptr(dst[k]) + ((base + off) >> 1);
                    if (left == 16u) { u2 x; x.x = out[0]; x.y = out[1]; *(EXCP_GLOBAL u2 *)to = x; }
                    else for (u32 j = 0; j < (left + 1u) / 2u; ++j) to[j] = (unsigned char)(out[j >> 2 & 1u] >> (8u * (j & 3u)));
                } else {
                    EXCP_GLOBAL unsigned char *to = gptr(dst[k]) + base + off;
                    if (left == 16u) { u4 x; x.x = out[0]; x.y = out[1]; x.z = out[2]; x.w = out[3]; *(EXCP_GLOBAL u4 *)to = x; }
                    else for (u32 j = 0; j < left; ++j) to[j] = (unsigned char)(out[j >> 2 & 3u] >> (8u * (j & 3u)));
                }
            }
        }
    }
}

// Alg. 3: W_0 plus a chain of compressed checkpoints, oldest first, in ONE pass over the weights.
// A lane keeps its sixteen weights in registers and adds, checkpoint after checkpoint, the centre
// of every kept element (one fp32 addition per checkpoint, exactly what applying Alg. 2 again and
// again computes); W_0 is read once and the result written once, whatever the length of the chain.
//
// A checkpoint moves only 0.3 bytes per element, so from two checkpoints on the arithmetic of the rank and
// code look-ups bounds this kernel, not memory.  Each wave takes a quarter of a tile (1024 elements) for
// itself, with no barrier anywhere: bits and ranks go round the wave once per checkpoint, packed as
// "sixteen bits, survivors before them" (one exchange then gives a lane all it needs for four elements), and
// a code leaves its window by a bit-field extract whose width is 0 where the element is pruned.  While one
// checkpoint is worked on, the codes of the next and the bitmap word of the one after it are on their way.
// (A 410M-shaped checkpoint, eight steps of 4 bits: 2463 -> 1133 us in three launches, 1064 with the weights past the caches; the bytes alone take about 890.)
struct ChainBits {
    u32 pk;                                                // lane's 16-bit piece of the quarter's bitmap, survivors before it << 16
    u32 q, kept, nbits;                                    // survivors of the tensor before the quarter, in it (the same in every lane)
    u32 code; float centre;                                // the first 64 words of codes and of the codebook, one per lane
};
#define CHAIN_CODE_WORDS 260   // u32 words of 1024 codes of 8 bits, one for the first bit's place, one for the window's second half

// One wave's quarter of a tile through all checkpoints.
template <bool W16>
__device__ __forceinline__ void chain_quarter(const Workspace &w, const EXCP_CONSTANT CDesc *C, u32 tile, u32 wave, u32 wt, float *book, u32 *codes) {
    const bool bf = wt == 2u;
    const u32 steps = C->steps;
    u32 lane = threadIdx.x & 63u;
    asm volatile("" : "+v"(lane));                         // (keeps what follows from the lane out of the registers held over all tiles)
    const u32 sh4 = (lane & 3u) * 4u, below4 = (1u << sh4) - 1u;   // the lane's four bits in their piece
    const u32 ltile = tile - C->tile_begin;
    const u64 base = (u64)ltile * EXCP_TILE;
    const u32 rem = (C->n - base < (u64)EXCP_TILE) ? (u32)(C->n - base) : EXCP_TILE;
    if (wave * 1024u >= rem) return;
    const EXCP_CONSTANT DDesc *D0 = (const EXCP_CONSTANT DDesc *)(uintptr_t)(w.ddesc + C->first_desc);
    const EXCP_CONSTANT DState *S0 = (const EXCP_CONSTANT DState *)(uintptr_t)(w.dst + C->first_desc);
    const EXCP_CONSTANT u32 *counts = (const EXCP_CONSTANT u32 *)(uintptr_t)w.dec_cnt_w;
    const u32 bits_here = (lane * 64u < rem) ? min(64u, rem - lane * 64u) : 0u;
    const u32 my_word = min(lane, (rem - 1u) >> 6);
    const u32 from1 = lane & ~3u;                          // four times the lane / 4 of pk that the lane's elements of batch 0 belong to
    const u32 from4 = (wave * 16u + (lane >> 2)) * 4u;     // exchanges take lane numbers times four
    // the lane's word of the tile's bitmap (what lies past the last element is dropped in bits_of)
    auto load_word = [&](u32 step) { return gptr((const u64 *)(D0[step].blob + S0[step].off_bw))[(u64)ltile * 64u + my_word]; };
    auto bits_of = [&](u32 step, u64 word) {
        word &= bits_here < 64u ? (1ull << bits_here) - 1ull : ~0ull;
        const u32 pc = (u32)__popcll(word), excl = wave_incl_scan_u32(pc) - pc;
        const u32 q0 = (u32)__builtin_amdgcn_readlane((int)excl, (int)(wave * 16u));
        const u32 q1 = (u32)__builtin_amdgcn_readlane((int)(excl + pc), (int)(wave * 16u + 15u));
        // the lane's piece: quarter (lane & 3) of word wave * 16 + lane / 4
        const u32 lo = (u32)__builtin_amdgcn_ds_bpermute((int)from4, (int)(u32)word);
        const u32 hi = (u32)__builtin_amdgcn_ds_bpermute((int)from4, (int)(u32)(word >> 32));
        const u32 before = (u32)__builtin_amdgcn_ds_bpermute((int)from4, (int)excl) - q0;
        const u32 half = (lane & 2u) ? hi : lo, skip = (lane & 2u) ? (u32)__popc(lo) : 0u;
        const u32 piece = (lane & 1u) ? half >> 16 : half & 0xffffu, skip2 = (lane & 1u) ? (u32)__popc(half & 0xffffu) : 0u;
        ChainBits B;
        B.pk = piece | (before + skip + skip2) << 16;
        B.nbits = S0[step].nbits; B.q = counts[D0[step].tile_begin + ltile] + q0; B.kept = q1 - q0;
        const unsigned char *blob = D0[step].blob;
        const u64 bit0 = (u64)B.q * B.nbits;
        const u32 words = ((u32)(bit0 & 31ull) + B.kept * B.nbits + 31u) >> 5;
        // (no survivors: any word of the blob will do)
        const EXCP_GLOBAL u32 *cw = gptr((const u32 *)(words ? blob + S0[step].off_cw + (bit0 >> 5) * 4u : blob));
        B.code = cw[lane < words ? lane : 0u];
        B.centre = gptr((const float *)(blob + EXCP_HEADER))[min(lane, (1u << B.nbits) - 1u)];
        return B;
    };
    u64 word = load_word(0);
    float wp[4][4];
    if (!W16) {
        const EXCP_GLOBAL float *W0 = gptr(C->W0) + base;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const u32 off = wave * 1024u + (u32)k * 256u + lane * 4u;
            if (off + 4u <= rem) {
                const f4u x = READ_ONCE(f4u, (W0 + off));
                wp[k][0] = x.x; wp[k][1] = x.y; wp[k][2] = x.z; wp[k][3] = x.w;
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j) wp[k][j] = (off + (u32)j < rem) ? W0[off + (u32)j] : 0.f;
            }
        }
    } else {                                           // 16-bit weights: the registers hold the widened values
#pragma unroll
        for (int k = 0; k < 4; ++k) load_weights4(C->W0, base, wave * 1024u + (u32)k * 256u + lane * 4u, rem, wt, wp[k]);
    }
    ChainBits B = bits_of(0, word);
    wave_lds_fence();                                      // (loads in the order in which the loop waits for them)
    word = load_word(min(1u, steps - 1u));
    for (u32 step = 0; step < steps; ++step) {
        const u32 pk = B.pk, nbits = B.nbits;
        const u64 bit0 = (u64)B.q * nbits;
        const u32 woff = (u32)(bit0 & 31ull), words = (woff + B.kept * nbits + 31u) >> 5;
        codes[lane] = B.code;
        book[lane] = B.centre;
        if (words > 64u || nbits > 6u) {
            const EXCP_GLOBAL u32 *cw = gptr((const u32 *)(D0[step].blob + S0[step].off_cw)) + (bit0 >> 5);
            const EXCP_GLOBAL float *centres = gptr((const float *)(D0[step].blob + EXCP_HEADER));
#pragma unroll 1
            for (u32 i = 64u + lane; i < words; i += 64u) codes[i] = cw[i];
#pragma unroll 1
            for (u32 i = 64u + lane; i < (1u << nbits); i += 64u) book[i] = centres[i];
        }
        wave_lds_fence();
        // (past the last checkpoint the last one's bits are looked at again: no branch round a load)
        B = bits_of(min(step + 1u, steps - 1u), word);
        word = load_word(min(step + 2u, steps - 1u));
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const u32 p = (u32)__builtin_amdgcn_ds_bpermute((int)(from1 + (u32)k * 64u), (int)pk);
            const u32 r = (u32)__popc(p & below4) + (p >> 16);        // quarter rank of the lane's first survivor
            const u32 nib = p >> sh4;
            const u32 f = window32(codes, woff + r * nbits);
            u32 at = 0;                                               // first bit of the element's code in the window
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                u32 kept = (u32)__builtin_amdgcn_sbfe((int)nib, (u32)j, 1u);   // all ones or 0
                asm("" : "+v"(kept));                          // (a mask, not a comparison: one bit-field insert below)
                const u32 width = kept & nbits;
                float sum = wp[k][j] + book[__builtin_amdgcn_ubfe(f, at, width)];
                if (W16) sum = w16_widen(w16_narrow(sum, bf), bf);   // every checkpoint rounds into the storage format
                wp[k][j] = u2f((f2u(sum) & kept) | (f2u(wp[k][j]) & ~kept));
                at += width;
            }
        }
        // The wave's reads of these codes are done.  (It also keeps the loads for the next checkpoint above it:
        // without a fence the compiler moves them round the loop, to where they are waited for.)
        wave_lds_fence();
    }
    if (W16) {
        EXCP_GLOBAL unsigned short *Ho = gptr((unsigned short *)C->W_out) + base;
        const bool vec = ((uintptr_t)C->W_out & 7u) == 0u;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const u32 off = wave * 1024u + (u32)k * 256u + lane * 4u;
            us4 o16;
#pragma unroll
            for (int j = 0; j < 4; ++j) o16[j] = (unsigned short)w16_narrow(wp[k][j], bf);
            if (vec && off + 4u <= rem) WRITE_ONCE(us4, (Ho + off), o16);
            else {
#pragma unroll
                for (int j = 0; j < 4; ++j) if (off + (u32)j < rem) Ho[off + (u32)j] = o16[j];
            }
        }
        return;
    }
    EXCP_GLOBAL float *Wo = gptr(C->W_out) + base;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const u32 off = wave * 1024u + (u32)k * 256u + lane * 4u;
        if (off + 4u <= rem) {
            f4u y; y.x = wp[k][0]; y.y = wp[k][1]; y.z = wp[k][2]; y.w = wp[k][3];
            WRITE_ONCE(f4u, (Wo + off), y);
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) if (off + (u32)j < rem) Wo[off + (u32)j] = wp[k][j];
        }
    }
}

// W16: takes the chains of 16-bit weights, or else those of fp32 weights.
template <bool W16>
__global__ __launch_bounds__(EXCP_THREADS, W16 ? 6 : 8) void k_decode_chain(Workspace w, u32 ntensors, u32 ntiles) {
    __shared__ float s_book[EXCP_THREADS / 64][256];
    __shared__ u32 s_code[EXCP_THREADS / 64][CHAIN_CODE_WORDS];
    __shared__ u32 s_tiles[EXCP_MAX_GROUP_TENSORS + 1];
    const u32 wave = (u32)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    load_tile_table(s_tiles, w.chain_tile_begin, ntensors);
    u32 t = 0, end = 0, wt = 0;
    bool good = false;                                     // the tensor is wanted, every checkpoint of its chain parsed and counted fine
    for (u32 tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        if (tile >= end) {                                 // (a workgroup's tiles only go up)
            t = (u32)__builtin_amdgcn_readfirstlane((int)find_owner(s_tiles, ntensors, tile));
            end = (u32)__builtin_amdgcn_readfirstlane((int)s_tiles[t + 1u]);
            const EXCP_CONSTANT CDesc *Ct = (const EXCP_CONSTANT CDesc *)(uintptr_t)(w.cdesc + t);
            const EXCP_CONSTANT DState *S = (const EXCP_CONSTANT DState *)(uintptr_t)(w.dst + Ct->first_desc);
            wt = excp_wtype(S->flags);
            good = Ct->W_out != nullptr && (wt != 0u) == W16;       // ... and all store their weights alike
            for (u32 j = 0; j < Ct->steps; ++j) good = good && S[j].status == 0 && excp_wtype(S[j].flags) == wt;
        }
        if (!good) continue;
        const EXCP_CONSTANT CDesc *C = (const EXCP_CONSTANT CDesc *)(uintptr_t)(w.cdesc + t);
        chain_quarter<W16>(w, C, tile, wave, wt, s_book[wave], s_code[wave]);
    }
}

// Per tensor of a chain: status = the first checkpoint that failed, counts and size of the last one.
__global__ void k_chain_finish(Workspace w, u32 ntensors, u32 rec_base) {
    const u32 t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= ntensors) return;
    const CDesc &C = w.cdesc[t];
    int status = 0;
    for (u32 j = 0; j < C.steps && status == 0; ++j) {
        status = w.dst[C.first_desc + j].status;
        if (status == 0 && excp_wtype(w.dst[C.first_desc + j].flags) != excp_wtype(w.dst[C.first_desc].flags)) status = -4;
    }
    const DState &S = w.dst[C.first_desc + C.steps - 1u];
    HostRec &R = w.rec_dev[rec_base + t];
    R.n = C.n; R.n_w = S.n_w; R.n_o = S.n_o; R.blob_bytes = S.blob_bytes; R.nonfinite = 0;
    R.abs_sum = 0.0; R.obj[0] = R.obj[1] = R.obj[2] = 0.0;
    R.med = R.mean32 = R.t_w = R.r_o = 0.f;
    R.status = status; R.pad = 0;
}

__global__ void k_decode_finish(Workspace w, u32 ntensors) {
    const u32 t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t < ntensors) decode_record(w, t, w.ddesc[t].n, w.dst[t]);
}

// Export: header and codebooks of every well-formed blob, verbatim (one workgroup per tensor).
__global__ void k_export_head(Workspace w, u32 ntensors) {
    const u32 t = blockIdx.x;
    const DDesc &D = w.ddesc[t];
    const DState &S = w.dst[t];
    if (S.status != 0 || D.head == nullptr) return;
    const u32 words = (EXCP_HEADER + 12u * (1u << S.nbits)) / 4u;
    const EXCP_GLOBAL u32 *src = gptr((const u32 *)D.blob);
    EXCP_GLOBAL u32 *dst = gptr((u32 *)D.head);
    for (u32 i = threadIdx.x; i < words; i += blockDim.x) dst[i] = src[i];
}

// Reconstruction from the per-element code tensors: here `blob` holds only header and codebooks.
__global__ void k_dense_parse(Workspace w, u32 ntensors) {
    const u32 t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= ntensors) return;
    const DDesc &D = w.ddesc[t];
    DState &S = w.dst[t];
    S.status = 0; S.pop_w = 0; S.pop_o = 0;
    S.n_w = 0; S.n_o = 0; S.nbits = 4; S.blob_bytes = 0; S.flags = 0; S.pad = 0;
    if (D.blob_bytes < EXCP_HEADER) { S.status = -4; return; }
    const u32 *h = (const u32 *)D.blob;
    const u64 *h64 = (const u64 *)D.blob;
    const u32 nbits = h[2];
    bool ok = h[0] == EXCP_MAGIC && h[1] == EXCP_VERSION && nbits >= 2u && nbits <= 8u && h[3] < 64u && (h[3] & 0x30u) != 0x30u;
    ok = ok && h64[2] == D.n && D.blob_bytes >= EXCP_HEADER + 12ull * (1u << (nbits & 15u));
    ok = ok && (D.wtype == 3u || D.wtype == excp_wtype(h[3]));
    if (!ok) { S.status = -4; return; }
    S.n_w = h64[3]; S.n_o = h64[4]; S.nbits = nbits; S.blob_bytes = h64[8]; S.flags = h[3];
}

// Four consecutive elements per lane and step: one 16-bit (or 32-bit) load of codes per tensor, one 16-byte load of the previous
// weights, one 16-byte store per output, neighbours side by side.  Code 0 leaves the weight untouched (not "+ 0.0": a negative zero
// stays) and gives a zero moment.  A code beyond the codebook, or a set unused half of the last byte, marks the tensor as damaged.
// Memory bounds it if enough loads are on their way: those of a whole tile, up to sixteen a lane, come before its first store,
// because the compiler moves no load over a store.  (333 M elements with both moments, 5.84 GB: 1253 us with eight elements a lane
// and each load before its own store, 1522 with four elements in that order, 1120 with the loads first, 1099 = 5.3 TB/s with the
// stores past the caches as well.)
__global__ __launch_bounds__(EXCP_THREADS) void k_decode_dense(Workspace w, u32 ntensors, u32 ntiles) {
    __shared__ float s_book[3 * 256];
    __shared__ u32 s_tiles[EXCP_MAX_GROUP_TENSORS + 1];
    const u32 tid = threadIdx.x;
    u32 cur_t = 0xffffffffu;
    load_tile_table(s_tiles, w.tile_begin, ntensors);
    for (u32 tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        const u32 t = find_owner(s_tiles, ntensors, tile);
        const DDesc &D = w.ddesc[t];
        DState &S = w.dst[t];
        if (S.status != 0 && S.status != -40) continue;    // -40: damage found by another workgroup meanwhile
        const u32 nbits = S.nbits, E = 1u << nbits;
        const bool wide = nbits > 4u;
        const u32 wt = excp_wtype(S.flags);                // 16-bit weights: widen, add, round into the format
        const bool bf = wt == 2u;
        const u64 n = D.n;
        const u64 base = (u64)(tile - D.tile_begin) * EXCP_TILE;
        const u32 rem = (n - base < (u64)EXCP_TILE) ? (u32)(n - base) : EXCP_TILE;
        if (t != cur_t) {
            __syncthreads();
            const EXCP_GLOBAL float *books = gptr((const float *)(D.blob + EXCP_HEADER));
            for (u32 i = tid; i < 3u * E; i += EXCP_THREADS) s_book[(i / E) * 256u + (i % E)] = books[i];
            cur_t = t;
            __syncthreads();
        }
        // all loads of the tile first: behind a store the compiler keeps them where they stand
        const unsigned char *const src[3] = {D.W_out ? D.cw : nullptr, D.m_out ? D.cm : nullptr, D.v_out ? D.cv : nullptr};
        float *const dst[3] = {D.W_out, D.m_out, D.v_out};
        const bool whole = rem == EXCP_TILE, vec16 = wt != 0u && (((uintptr_t)D.Wp | (uintptr_t)D.W_out) & 7u) == 0u;
        u32 code[3][4];                                    // the four codes, a byte or half a byte each
        f4u wp[4];
        us4 hp[4];
        bool bad = false;
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            if (src[q] == nullptr) continue;               // (the same in the whole workgroup)
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const u32 off = (u32)k * 1024u + tid * 4u, left = whole ? 4u : min(4u, rem - min(rem, off));
                const EXCP_GLOBAL unsigned char *p = gptr(src[q]) + (wide ? base + off : (base + off) >> 1);
                u32 c4 = 0;
                if (left == 4u) {
                    c4 = wide ? *(const EXCP_GLOBAL u32 *)p : (u32)*(const EXCP_GLOBAL unsigned short *)p;
                } else {
                    const u32 bytes = wide ? left : (left + 1u) / 2u;
                    for (u32 j = 0; j < bytes; ++j) c4 |= (u32)p[j] << (8u * j);
                    if (!wide && (left & 1u) && (c4 >> (4u * left))) bad = true;      // the unused half of the last byte
                }
                code[q][k] = c4;
            }
        }
        if (src[0] != nullptr) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const u32 off = (u32)k * 1024u + tid * 4u, left = whole ? 4u : min(4u, rem - min(rem, off));
                if (wt != 0u) {
                    const EXCP_GLOBAL unsigned short *Hp = gptr((const unsigned short *)D.Wp) + base + off;
                    if (left == 4u && vec16) {
                        hp[k] = READ_ONCE(us4, Hp);
                    } else {
#pragma unroll
                        for (int j = 0; j < 4; ++j) hp[k][j] = ((u32)j < left) ? Hp[j] : (unsigned short)0;
                    }
                } else {
                    const EXCP_GLOBAL float *Wp = gptr(D.Wp) + base + off;
                    if (left == 4u) {
                        wp[k] = READ_ONCE(f4u, Wp);
                    } else {
#pragma unroll
                        for (int j = 0; j < 4; ++j) wp[k][j] = ((u32)j < left) ? Wp[j] : 0.f;
                    }
                }
            }
        }
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            if (src[q] == nullptr) continue;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const u32 off = (u32)k * 1024u + tid * 4u, left = whole ? 4u : min(4u, rem - min(rem, off));
                u32 c[4];
                float centre[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    c[j] = wide ? (code[q][k] >> (8 * j)) & 255u : (code[q][k] >> (4 * j)) & 15u;
                    if (c[j] >= E) bad = true;
                    centre[j] = s_book[(u32)q * 256u + (c[j] & (E - 1u))];
                }
                if (q == 0 && wt != 0u) {
                    EXCP_GLOBAL unsigned short *Ho = gptr((unsigned short *)D.W_out) + base + off;
                    us4 h = hp[k];
#pragma unroll
                    for (int j = 0; j < 4; ++j) if (c[j]) h[j] = (unsigned short)w16_narrow(w16_widen(h[j], bf) + centre[j], bf);
                    if (left == 4u && vec16) {
                        WRITE_ONCE(us4, Ho, h);
                    } else {
#pragma unroll
                        for (int j = 0; j < 4; ++j) if ((u32)j < left) Ho[j] = h[j];
                    }
                    continue;
                }
                f4u x;
                EXCP_GLOBAL float *out = gptr(dst[q]) + base + off;
#pragma unroll
                for (int j = 0; j < 4; ++j) x[j] = q == 0 ? (c[j] ? wp[k][j] + centre[j] : wp[k][j]) : (c[j] ? centre[j] : 0.f);
                if (left == 4u) {
                    WRITE_ONCE(f4u, out, x);
                } else {
#pragma unroll
                    for (int j = 0; j < 4; ++j) if ((u32)j < left) out[j] = x[j];
                }
            }
        }
        if (bad) S.status = -40;
    }
}

// -40 (damage seen while decoding) becomes the public "damaged blob" status.
__global__ void k_dense_status(Workspace w, u32 ntensors) {
    const u32 t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t < ntensors && w.dst[t].status == -40) w.dst[t].status = -4;
}

template <bool MOMENTS, bool W16>
__global__ __launch_bounds__(EXCP_THREADS) void k_decode_small(Workspace w, u32 ntensors, u32 ntiles) {
    decode_tiles<MOMENTS, false, W16 ? 1 : 0>(w, ntensors, ntiles);
    decode_tiles<MOMENTS, true, 2>(w, ntensors, ntiles);
}

}  // namespace

// Per-tile counts of a bitmap and their scan.
template <int WHICH>
static void launch_decode_counts(const Workspace &w, u32 ntensors, u32 ntiles, bool records, hipStream_t s) {
    if (ntiles) {
        const u32 blocks = std::min((ntiles + 31u) / 32u, excp_grid(w, 8));            // eight tiles to a wave at least
        hipLaunchKernelGGL(k_decode_count<WHICH>, dim3(blocks), dim3(EXCP_THREADS), (ntensors + 1u) * sizeof(u32), s, w, ntensors, ntiles);
    }
    hipLaunchKernelGGL(k_decode_scan<WHICH>, dim3(excp_scan_runs(ntensors, ntiles)), dim3(EXCP_THREADS), 0, s, w, ntensors, records ? 1u : 0u);
}
// Headers, counts and scans of a group whose largest tensor has `largest` tiles.  `single`: the description of its only tensor,
// not in the tables yet.  `records`: nothing can change the results after this, they go to the host.
void launch_decode_prep(const Workspace &w, u32 ntensors, u32 ntiles, u32 largest, bool allow_raw, bool moments, bool records, const DDesc *single, hipStream_t s) {
    if (!ntensors) return;
    if (excp_prep_small(largest)) {
        hipLaunchKernelGGL(k_decode_prep, dim3(ntensors), dim3(PREP_WAVES * 64), 0, s, w, allow_raw ? 1u : 0u, moments ? 1u : 0u, records ? 1u : 0u,
                           single ? *single : DDesc{}, single ? 1u : 0u);
        return;
    }
    hipLaunchKernelGGL(k_decode_parse, dim3((ntensors + PARSE_THREADS - 1u) / PARSE_THREADS), dim3(PARSE_THREADS), 0, s, w, ntensors, excp_scan_runs(ntensors, ntiles), allow_raw ? 1u : 0u,
                       single ? *single : DDesc{}, single ? 1u : 0u);
    launch_decode_counts<0>(w, ntensors, ntiles, records && !moments, s);
    if (moments) launch_decode_counts<1>(w, ntensors, ntiles, records, s);
}
// The main pass of a small group, of blobs written with and without quantisation in one launch: a launch that finds nothing to do
// is a tenth of such a call.
void launch_decode_small(const Workspace &w, u32 ntensors, u32 ntiles, bool moments, bool w16, hipStream_t s) {
    if (!ntiles) return;
    const dim3 grid(std::min(ntiles, excp_grid(w, 64))), block(EXCP_THREADS);
    if (moments && w16) hipLaunchKernelGGL((k_decode_small<true, true>), grid, block, 0, s, w, ntensors, ntiles);
    else if (moments) hipLaunchKernelGGL((k_decode_small<true, false>), grid, block, 0, s, w, ntensors, ntiles);
    else if (w16) hipLaunchKernelGGL((k_decode_small<false, true>), grid, block, 0, s, w, ntensors, ntiles);
    else hipLaunchKernelGGL((k_decode_small<false, false>), grid, block, 0, s, w, ntensors, ntiles);
}
// The main passes take a workgroup a tile: then those at work lie side by side.  (With 64 workgroups a compute unit, each of which
// goes on with the tile 16 384 further, as many regions are in hand as that makes rounds: weights of the 410M shape 662 instead of 650 us,
// 24 ragged tensors with their moments 709 instead of 682, the stored layout of 333 M elements 1112 instead of 1055; with runs of
// neighbouring tiles to a workgroup 723 and 770.  That every tile loads the table of tiles and the codebooks anew does not take it back:
// 1000 tensors of 200 000 elements with one-byte codes 448 instead of 404, with their moments 819 instead of 746, of 20 000 elements 125 either way.)
void launch_decode_main(const Workspace &w, u32 ntensors, u32 ntiles, bool moments, hipStream_t s) {
    if (!ntiles) return;
    if (moments) hipLaunchKernelGGL(k_decode_main<true>, dim3(ntiles), dim3(EXCP_THREADS), 0, s, w, ntensors, ntiles);
    else hipLaunchKernelGGL(k_decode_main<false>, dim3(ntiles), dim3(EXCP_THREADS), 0, s, w, ntensors, ntiles);
}
void launch_decode_main16(const Workspace &w, u32 ntensors, u32 ntiles, bool moments, hipStream_t s) {
    if (!ntiles) return;
    if (moments) hipLaunchKernelGGL(k_decode_main16<true>, dim3(ntiles), dim3(EXCP_THREADS), 0, s, w, ntensors, ntiles);
    else hipLaunchKernelGGL(k_decode_main16<false>, dim3(ntiles), dim3(EXCP_THREADS), 0, s, w, ntensors, ntiles);
}
void launch_decode_raw(const Workspace &w, u32 ntensors, u32 ntiles, bool moments, hipStream_t s) {
    if (!ntiles) return;
    u32 blocks = excp_grid(w, 32);
    if (blocks > ntiles) blocks = ntiles;
    if (moments) hipLaunchKernelGGL(k_decode_raw<true>, dim3(blocks), dim3(EXCP_THREADS), 0, s, w, ntensors, ntiles);
    else hipLaunchKernelGGL(k_decode_raw<false>, dim3(blocks), dim3(EXCP_THREADS), 0, s, w, ntensors, ntiles);
}
void launch_export_dense(const Workspace &w, u32 ntensors, u32 ntiles, hipStream_t s) {
    if (!ntensors) return;
    hipLaunchKernelGGL(k_export_head, dim3(ntensors), dim3(EXCP_THREADS), 0, s, w, ntensors);
    if (!ntiles) return;
    const bool split = ntiles <= excp_grid(w, 4);
    const u32 blocks = split ? ntiles : std::min((ntiles + EXPORT_WAVES - 1u) / EXPORT_WAVES, excp_grid(w, EXPORT_PER_CU));
    hipLaunchKernelGGL(k_export_dense, dim3(blocks), dim3(EXCP_THREADS), 0, s, w, ntensors, ntiles, split ? 1u : 0u);
}
void launch_dense_parse(const Workspace &w, u32 ntensors, hipStream_t s) {
    if (!ntensors) return;
    hipLaunchKernelGGL(k_dense_parse, dim3((ntensors + 255) / 256), dim3(256), 0, s, w, ntensors);
}
void launch_decode_dense(const Workspace &w, u32 ntensors, u32 ntiles, hipStream_t s) {
    if (!ntensors) return;
    if (ntiles) hipLaunchKernelGGL(k_decode_dense, dim3(ntiles), dim3(EXCP_THREADS), 0, s, w, ntensors, ntiles);
    hipLaunchKernelGGL(k_dense_status, dim3((ntensors + 255) / 256), dim3(256), 0, s, w, ntensors);
}
void launch_decode_finish(const Workspace &w, u32 ntensors, hipStream_t s) {
    if (!ntensors) return;
    hipLaunchKernelGGL(k_decode_finish, dim3((ntensors + 255) / 256), dim3(256), 0, s, w, ntensors);
}
void launch_decode_chain(const Workspace &w, u32 ntensors, u32 ntiles, bool w16, hipStream_t s) {
    if (!ntiles) return;
    u32 blocks = excp_grid(w, 64);
    if (blocks > ntiles) blocks = ntiles;
    if (w16) hipLaunchKernelGGL(k_decode_chain<true>, dim3(blocks), dim3(EXCP_THREADS), 0, s, w, ntensors, ntiles);
    else hipLaunchKernelGGL(k_decode_chain<false>, dim3(blocks), dim3(EXCP_THREADS), 0, s, w, ntensors, ntiles);
}
void launch_chain_finish(const Workspace &w, u32 ntensors, hipStream_t s) {
    if (!ntensors) return;
    hipLaunchKernelGGL(k_chain_finish, dim3((ntensors + 255) / 256), dim3(256), 0, s, w, ntensors, w.rec_base);
}

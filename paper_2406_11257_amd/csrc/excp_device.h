// Device-side tables shared by the ExCP kernels and their host orchestrator.
// One "group" of tensors is processed by every kernel at once: kernels walk a
// tile list (EXCP_TILE elements per tile, tiles of all tensors back to back)
// or a chunk list (EXCP_CHUNK survivors per chunk) and find their tensor from
// these tables, so no launch depends on a value that only the device knows.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <algorithm>

#define EXCP_TILE        4096u     // elements per tile of the full-tensor passes (256 threads x 16)
#define EXCP_CHUNK       8192u     // survivors per chunk of the survivor passes
#define EXCP_UNIT_SHIFT 17u        // log2 of the largest unit of the bucket counts, in positions of a stream (see excp_unit_shift)
#define EXCP_THREADS     256
#define EXCP_SMALL_ELEMS 8192u     // elements up to which a workgroup holds a tensor (k_small.hip)
#define EXCP_SAMPLE_PARTS 16u      // workgroups that draw a tensor's sample of residuals
#define EXCP_STATS_PER_CU 64u      // workgroups per compute unit of the statistics pass, at most (excp_stats_grid)
#define EXCP_ABSM_BINS   40        // u64 accumulators, 8 binary exponents apart, for the exact sum of |m|
#define EXCP_MAX_K       255
#define EXCP_KM_CELLS    4096u     // cells of the value -> bucket map (2048 per sign)
#define EXCP_KM_MAP_WORDS (4u + EXCP_KM_CELLS / 4u)
#define EXCP_HEADER      80u
#define EXCP_MAGIC       0x50435845u
#define EXCP_VERSION     1u

typedef unsigned long long u64;
typedef unsigned int u32;

// Host-filled description of one tensor of a compress group.
struct TDesc {
    const float *Wp, *W, *m, *v;
    u64 n;
    unsigned char *blob;
    u64 blob_cap;
    float *W_out;
    u64 elem_off;      // start of this tensor's survivor slots in the group workspace
    u64 cand_off;      // start and capacity of this tensor's median-candidate list
    u64 cand_cap;
    u32 cand_lists;    // a tensor's candidate list is cut into this many lists (1 .. 16), each with a counter of its
                       // own, so that thousands of workgroups do not queue at one address
    u32 turn;          // of the group's i-th entry: the tensor whose turn is i-th where the large ones go first
    u32 tile_begin;    // first tile of this tensor in the group's tile list
    u32 tile_count;
    u32 acc_slot;      // place of its streams' accumulators where many workgroups take a Lloyd iteration; EXCP_NO_SLOT:
                       // its streams are never taken that way
    u32 rec;           // its record among the group's, in the order of the call
};
#define EXCP_NO_SLOT 0xffffffffu

// What one workgroup of the statistics pass found out about a tensor: units of the exact sum of |m| (low and
// high 32-bit halves added up), keys below the median's bracket, non-finite values, keys equal to a one-value
// bracket, elements equal to the counted bracket values.
struct StatPart { u64 L, H; u32 clt, nf, cc, pad, atom[4]; };

// Device-written per-tensor state of a compress group.
struct TState {
    u64 absm[EXCP_ABSM_BINS];   // sum_g absm[g] * 2^(8g - 149) == exact sum of |m|
    u64 nonfinite;
    u64 n_w, n_o;
    u64 off_bo, off_cw, off_cm, off_cv, blob_bytes;
    double abs_sum;
    double obj[3];
    u32 br_lo, br_hi;           // median bracket (keys) from the sorted sample
    u32 med_state;              // 0 select among candidates pending, 1 median known, 2 full-tensor fallback
    u32 cand_count, cand_overflow, c_lt;   // keys inside / overflowing the list / below the bracket
    u32 sel_base, sel_width;    // radix select: key bits decided so far, number of undecided low bits
    u32 sel_rank;               // rank still to find among the undecided keys
    u32 med_bits;
    float mean32, t_w, r_o;
    int status;
    u32 absm_base;              // lowest bit position of the 24-position window used for the exact sum of |m|
    // tied data (16-bit weights): values inside the median bracket that the sample shows to be heavily
    // repeated are counted, not listed among the candidates
    u32 natoms, atom_key[4], atom_cnt[4];
    u32 lloyd_shared;           // many workgroups take each of the tensor's streams through a Lloyd iteration
    u32 pad2;
    StatPart part;              // of a tensor whose tiles all belong to one workgroup of the statistics pass
};

// One survivor stream (3 per tensor: residual, m, v) during codebook construction.
struct SegState {
    u64 len;
    u32 chunk_begin;            // first chunk of this stream in the group's chunk list
    u32 row_begin;              // first row of this stream in the table of bucket counts (a row per unit: GroupParams::unit_shift)
    u32 work;                   // what a Lloyd iteration is expected to cost, in values of cut buckets
    u32 crowded;                // a bucket holds far more than its share of the values
    u32 bin_lo, bin_hi;         // the bins of km_bsum that are not all zero lie in [bin_lo, bin_hi]
    u32 acc_lo, acc_hi;         // sums of any of the stream's values have no other bins than [acc_lo, acc_hi]
    // centres (K used) and cut keys (cut[k], 1 <= k < K: smallest key whose nearest centre has index >= k) by the
    // parity of the iteration that made them: iteration i reads those of i - 1 and writes its own
    float C[2][EXCP_MAX_K + 1];
    u32 cut[2][EXCP_MAX_K + 1];
};

// Host-filled description of one tensor of a decompress group.
struct DDesc {
    const float *Wp;
    const unsigned char *blob;
    u64 blob_bytes;
    u64 n;
    float *W_out, *m_out, *v_out;
    // per-element code tensors (two codes of 4 bits or fewer per byte, else one per byte): written by
    // the export of a blob, read by the reconstruction from that layout (then `blob` is the header
    // with the codebooks and `head` is unused)
    unsigned char *cw, *cm, *cv;
    unsigned char *head;        // export: receives header and codebooks (nullable)
    u32 tile_begin, tile_count;
    u32 wtype;                  // storage of the caller's weight arrays (0 fp32, 1 fp16, 2 bf16): the blob must
    u32 pad;                    // say the same; 3 = no weight arrays are involved
};

struct DState {
    u64 n_w, n_o, blob_bytes;
    u64 off_bw, off_bo, off_cw, off_cm, off_cv;
    u32 nbits;
    int status;
    u64 pop_w, pop_o;           // bitmap populations found while scanning
    u32 flags;                  // the blob's flags (bit 3: bitmap_o covers all elements)
    u32 pad;
};

// Host-filled description of one tensor of a chain reconstruction: its decode descriptors (one per
// compressed checkpoint, oldest first) are ddesc[first_desc .. first_desc + steps).
struct CDesc {
    const float *W0;
    float *W_out;
    u64 n;
    u32 first_desc, steps;
    u32 tile_begin, tile_count;     // in the group's list of tensor tiles
};

// Result record copied back to the host after a batch.
struct HostRec {
    u64 n, n_w, n_o, blob_bytes, nonfinite;
    double abs_sum, obj[3];
    float med, mean32, t_w, r_o;
    int status;
    int pad;
};

struct GroupParams {
    float alpha, beta;
    int nbits, K, iters;
    u32 flags;
    u32 ntensors, ntiles;
    u32 wide;                   // per-bucket kernels with sixteen waves: 1 = for the residual streams (16-bit weights: tied
                                // data), 2 = for all, one bucket per workgroup (a very large tensor in the group)
    u32 alone_work;             // SegState::work of a tensor's streams up to which one workgroup takes each of them through its
                                // Lloyd iterations
    u32 together;               // all of the group's tensors go the same way
    u32 slots;                  // tensors with an acc_slot
    u32 unit_shift;             // log2 of the positions of a stream whose bucket counts share a row
    u32 fine;                   // the first `fine` tensors in order of size may have cells inside their buckets (k_km_cells)
    u32 fine_size;              // ... by the workgroups of size 0, 1 or 2
    u32 fine_chunks;            // ... and the chunks of survivors up to which they do
    u64 largest;                // elements of the largest tensor
    u32 samples;                // values of a stream that its value -> bucket map is made from
};

#define EXCP_RAW_BITS    32u       // "code" width of a blob written without quantisation: fp32 values, no codebooks
// bytes of the three codebooks that follow the header
static __host__ __device__ inline u64 excp_books_bytes(u32 nbits) { return nbits >= EXCP_RAW_BITS ? 0ull : 12ull << nbits; }
static __host__ __device__ inline u64 excp_pad16(u64 b) { return (b + 15ull) & ~15ull; }
static __host__ __device__ inline u64 excp_words(u64 bits) { return (bits + 63ull) >> 6; }

// ---- launchers (defined next to their kernels) --------------------------------------------
struct Workspace {
    // group tables
    TDesc *desc; TState *st; SegState *seg; u32 *tile_begin;   // tile_begin has ntensors+1 entries
    // survivors
    float *xw, *xm, *xv;
    // median select
    u32 *sample;              // [tensor][8192] residual magnitudes of the sample
    u32 *sample_mmax;         // [tensor][EXCP_SAMPLE_PARTS] largest finite |m| pattern met by each part of the sample
    u32 *sel_ticket;          // [tensor] workgroups that have finished the pass of the select in hand (0 between passes)
    u32 *med_hist;            // [tensor][2048]
    u32 *cand;                // median candidates (keys inside the sample bracket), per tensor
    u32 *cand_ctr;            // [tensor][16][32] per list: [0] slots asked for, [1] end of the slots granted (128 B apart)
    StatPart *stat_part;      // [workgroup of the statistics pass][2] records of the tensors its tile range starts and ends in
    // mask pass
    u64 *tile_status;         // per 2048-element sub-tile: survivors << 32 | moment survivors
    u64 *mask_prefix;         // exclusive scan of tile_status within each tensor
    u64 *mask_part;           // [tensor][16] packed counts of each sixteenth of a tensor's sub-tiles
    u64 *mask_bo;             // [sub-tile][32] M_o bits of the sub-tile's survivors, local positions
    // survivor passes
    u32 *chunk_total;         // [1]
    u32 *seg_chunk_begin;     // [segments + 1] first chunk of every survivor stream
    u32 *scan_ticket;         // [1] tensors whose survivors have been counted (0 between launches)
    u32 *no_cells;            // [1] the group's survivors or a stream's buckets are too many or too large for cells (see k_km_scan)
    u32 *lloyd_shared;        // [1] TState::lloyd_shared of some tensor of the group
    u32 *seg_unit_begin;      // [segments + 1] first work unit of every survivor stream in a Lloyd iteration that many workgroups take
    float *pw, *pm, *pv;      // survivors partitioned into value-ordered buckets (same offsets as xw/xm/xv)
    u32 *km_split;            // [segment][EXCP_KM_MAP_WORDS] value -> bucket map: 4 parameters, then 4096 bucket bytes
    u32 *km_cnt;              // [row][256] bucket counts, then positions: a row per unit of a stream (GroupParams::unit_shift)
    u32 *km_begin;            // [segment][257] first position of every bucket
    u64 *km_bsum;             // [segment][EXCP_ABSM_BINS][257] exact signed sum of every bucket, then of all buckets before it
    u32 *km_min, *km_max;     // [segment][256] smallest / largest key of every bucket
    u32 *km_dom, *km_less;    // [segment][256] repetitions of every bucket's first value, values below it (sixteen-wave form only)
    u32 *km_mag;              // [segment][256] smallest non-zero magnitude (bit pattern) of every bucket
    u32 *km_fine;             // [segment][256] the cells inside every bucket (see k_km_cells); 0: none
    u32 *fine_begin;          // [which][fine_stride] first value of every cell, counted from its bucket's first
    u64 *fine_above;          // [which][fine_stride] exact sum of the bucket's values in higher cells
    u64 fine_stride;
    u64 *km_acc;              // [TDesc::acc_slot][stream][3][EXCP_ABSM_BINS + 1][K] per-centre exact sum and count, by iteration modulo 3
    double *part_obj;         // [chunk]
    // decode
    DDesc *ddesc; DState *dst;
    CDesc *cdesc; u32 *chain_tile_begin;   // chain reconstruction: tensors and their tile table
    u32 *dec_cnt_w, *dec_cnt_o;   // per tile counts -> exclusive bases
    u32 *dec_part;                // [which][dec_part_stride] sums of the counts by runs of tiles (see k_decode_count)
    u32 dec_part_stride;
    u32 *dec_kinds;               // [0] kinds of blob in the group being decoded: 1 fp32 weights, 2 16-bit weights, 4 unquantised; [1], [2] of its making (0 between launches)
    // results
    HostRec *rec_dev;         // (host memory, except in the static call)
    u32 rec_base;             // index of this group's first tensor in rec_dev
    int cus;                  // compute units of the device
};

// Grid of a persistent kernel: `per_cu` workgroups per compute unit (each kernel's figure was
// measured on its own).
static inline u32 excp_grid(const Workspace &w, u32 per_cu) { return (u32)w.cus * per_cu; }

// Lists that a tensor's median candidates are filed in, and the places they have together: a twelfth of the tensor and
// 4096, rounded down to a multiple of the lists, so that the tensors of a group never have more than excp_cand_words,
// which the workspace sets aside.
static inline u32 excp_cand_lists(u64 n, u64 list_elems) { return n / list_elems < 1 ? 1u : (n / list_elems > 16 ? 16u : (u32)(n / list_elems)); }
static inline u64 excp_cand_cap(u64 n, u32 lists) { return (n / 12 + 4096) / lists * lists; }
static inline u64 excp_cand_words(u64 group_elems, u32 group_tensors) { return group_elems / 12 + 4096ull * group_tensors; }
// The list that a workgroup of the statistics pass tries first: neighbours, which share a tensor, try different ones.  (With
// every fourth list for a start, those filled and the others were found by failing there: 3 M elements 28.6 -> 18.5 us
// for the pass, 16.8 M 41.2 -> 39.0 and 41.5 -> 37.4 for the select, whose waves share the lists out.)
static __host__ __device__ inline u32 excp_cand_first(u32 workgroup, u32 lists) { return workgroup % lists; }

// Workgroups of the statistics pass, each with a run of tiles: eight to a compute unit at least, and so many more, up to
// EXCP_STATS_PER_CU, that a run is about six tiles.  Short runs lie close together at any time, as memory likes it (8, 16, 32, 64 to
// a compute unit: 410M shape 854, 842, 832, 823 us, its weights in bf16 485, 477, 470, 461, four layers of the 7B shape 2314, 2300, 2310,
// 2245), but a run that ends asks for places in its tensor's candidate lists and leaves a record to add up (16.8 M elements 41, 43, 66,
// 125), so beyond eight to a compute unit the largest tensor has runs of 24 tiles at least (with k_stats_finish, one of 100 M elements 223, 227, 227,
// 228, 150 M 332, 336, 336, 337, 400 M 886, 871, 874, 883).
static inline u32 excp_stats_grid(u32 ntiles, u64 largest, u32 cus) {
    const u64 least = 8ull * cus, tiles = std::max<u64>((largest + EXCP_TILE - 1u) / EXCP_TILE, 1u);      // (of the largest)
    const u64 most = std::min<u64>((u64)EXCP_STATS_PER_CU * cus, std::max(least, tiles / 24u) * ntiles / tiles);
    return (u32)std::max(least, std::min<u64>(ntiles / 6u, most));
}

// Sub-tiles to a batch of the gather pass: as many as leave four batches to a compute unit, four at least, so that each of a
// workgroup's waves has one, and EXCP_GATHER_SUBS at most.  (With 32 always, a 16.8 M-element tensor was 256 workgroups of eight
// round trips each: 51 -> 29 us, and the 14M shape's small tensors 126 -> 35 us.)
#define EXCP_GATHER_SUBS 32u
static inline u32 excp_gather_subs(u32 ntiles, u32 cus) {
    const u32 subs = 2u * ntiles / (4u * cus) & ~3u;
    return subs < 4u ? 4u : (subs > EXCP_GATHER_SUBS ? EXCP_GATHER_SUBS : subs);
}
// Rows that the table of bucket counts has, and log2 of the positions that share a row in a group of `elems` elements:
// the scatter's workgroups begin at rows, so it is the smallest power of two that leaves one row to a compute unit
// when half the elements survive in the three streams together (a third of the weights, a tenth of the moments twice),
// between 2^14 (64 positions to a bucket: below that most of a workgroup's lines are partial ones) and 2^17, not less than a
// batch of the gather pass can span, and so much that the rows fit the table.
static inline u64 excp_count_rows(u64 group_elems, u32 group_tensors) { return 3 * (group_elems >> EXCP_UNIT_SHIFT) + 3ull * group_tensors + 4; }
static inline u32 excp_unit_shift(u64 elems, u32 tensors, u32 subs, u32 cus, u64 rows) {
    u32 s = 14;
    while (s < EXCP_UNIT_SHIFT && ((elems >> s) > 4ull * cus || (u64)subs * 2048u > (1ull << s) || 3 * (elems >> s) + 3ull * tensors > rows)) ++s;
    return s;
}

// Tiles whose counts a workgroup of the restores' scan takes, and the runs that the tiles of a group are cut into: the first of every
// tensor, and one for every multiple of that number.
#define EXCP_SCAN_TILES 1024u
static __host__ __device__ inline u32 excp_scan_runs(u32 tensors, u32 tiles) { return tensors + (tiles + EXCP_SCAN_TILES - 1u) / EXCP_SCAN_TILES; }

// A tensor's area in the arrays of survivors (whole lines: it begins on a multiple of 64 elements), and what a group's take.
static inline u64 excp_area_elems(u64 n) { return (n + 63) & ~63ull; }
static inline u64 excp_survivor_elems(u64 group_elems, u32 group_tensors) { return group_elems + 63ull * group_tensors; }

// Cells inside a bucket of 256 values or more: the largest power of two that leaves them 64 values each on average, 512
// at most.  A bucket's entries in the tables begin at (its tensor's elem_off >> 6) + 258 x tensor + (its first
// position >> 6) + its number, and are one more than its cells, so no two buckets' overlap.
#define EXCP_FINE_SHIFT 6u
static inline u64 excp_fine_words(u64 group_elems, u32 group_tensors) { return (group_elems >> EXCP_FINE_SHIFT) + 258ull * group_tensors + 1; }
static __host__ __device__ inline u64 excp_fine_at(u64 elem_off, u32 tensor, u32 position, u32 bucket) {
    return (elem_off >> EXCP_FINE_SHIFT) + 258ull * tensor + (position >> EXCP_FINE_SHIFT) + bucket;
}
static __host__ __device__ inline u32 excp_fine_cells_log2(u32 size) {
    u32 k = 0;
    while (k < 9u && (size >> (EXCP_FINE_SHIFT + 1u) >> k)) ++k;
    return k;
}
// A key (see key_of) without the gap between the largest negative and the smallest positive value of magnitude `mag` (bit
// pattern) or more.
static __host__ __device__ inline u32 excp_closed_key(u32 key, u32 mag) {
    const u32 a = 0x7fffffffu - mag, b = 0x80000000u + mag;          // keys of -mag and +mag (of -0 and +0 for mag = 0)
    return key <= a ? key : (key < b ? a + 1u : key - b + a + 2u);
}
// The cells of a bucket: 2^log2 equal ranges of the closed key between its extremes.  `gap`: the keys have the gap between
// them.  A zero lies inside it, on the far side of the other values, so this is so not only where there are both signs.
struct CellMap { u32 kmin, mag, k0, shift, flip; bool gap; };
static __host__ __device__ inline CellMap excp_cell_map(u32 kmin, u32 kmax, u32 mag, u32 log2) {
    CellMap M;
    M.kmin = kmin; M.mag = mag; M.k0 = excp_closed_key(kmin, mag);
    const u32 range = excp_closed_key(kmax, mag) - M.k0, bits = 32u - (u32)__builtin_clz(range | 1u);
    M.shift = bits > log2 ? bits - log2 : 0u;
    M.gap = kmin <= 0x80000000u && kmax >= 0x7fffffffu;
    M.flip = kmin < 0x80000000u ? 0xffffffffu : 0x80000000u;         // without the gap: from a value's bits to its key
    return M;
}
static __host__ __device__ inline u32 excp_cell_of_key(const CellMap &M, u32 key) { return (excp_closed_key(key, M.mag) - M.k0) >> M.shift; }
// (of a value by its bits; nearly every bucket has no gap, and there the plain difference of the keys is the same)
static __host__ __device__ inline u32 excp_cell_of_bits(const CellMap &M, u32 bits) {
    if (M.gap) return excp_cell_of_key(M, (bits & 0x80000000u) ? ~bits : bits | 0x80000000u);
    return ((bits ^ M.flip) - M.kmin) >> M.shift;
}
// Tensors whose buckets may be worth cells (2^17 is a power of two because the host lists the tensors by powers of two), and
// the largest ones whose buckets, a third of the values kept, nearly all fit a workgroup of k_km_cells in its three sizes.
// A group of more elements in all goes without cells, but for what excp_cells_group adds.  One tensor of more has buckets that do not fit
// (30 M elements, 4 bits, us a call 751, 798 if it sets out for cells, 45 M 942 / 998, 60 M 1120 / 1168).  Of many tensors cells cost 2 to 4 us
// a million elements, more than the 125 us that the iterations and initial centres gain (40 of 600 000: totals and cells 112 instead of 34 us,
// iterations 57 instead of 151; 80 of 3 M: 1081 and 149, 64 and 253).  A group of 16-bit weights, whose few distinct residuals are shared out in any
// case, has none.
static __host__ __device__ inline bool excp_fine_tensor(u64 n) { return n >= 1ull << 17; }
#define EXCP_FINE_SMALL (1ull << 21)
#define EXCP_FINE_MIDDLE (9ull << 21)
#define EXCP_FINE_LARGEST (25ull << 20)
static inline u32 excp_fine_size(u64 largest) { return largest <= EXCP_FINE_SMALL ? 0u : (largest <= EXCP_FINE_MIDDLE ? 1u : 2u); }
// Values that a bucket may have, by GroupParams::fine_size, and chunks of survivors that a group may: beyond either the
// group goes without cells (k_km_scan), which is what these sizes come to where more than a third is kept.  Where every element
// is (alpha = 0; beta = 0 with no check of the weights that drops any) that is known before the call, and the group does not
// set out for cells: `whole` of the three streams, and buckets a third above the average.  (Everything kept, 4 bits, us a
// call without cells / with what was made of them before: 2 M elements 488 / 532, 10 M 744 / 845, 3 x 8 M 1210 / 1384, 40 x 500 000
// 1191 / 1296; with cells that fit, 4 M 532 / 445, 10 x 500 000 585 / 547.)
static __host__ __device__ constexpr u32 excp_cells_most(u32 fine_size) { return fine_size == 0u ? 8192u : (fine_size == 1u ? 40960u : 53248u); }
#define EXCP_FINE_CHUNKS 4096u
static inline bool excp_fine_group(u64 elems, u64 largest, u32 whole) {
    return elems <= EXCP_FINE_LARGEST && (whole == 0u || (whole * elems <= (u64)EXCP_FINE_CHUNKS * EXCP_CHUNK &&
                                                          largest + largest / 3u <= 256ull * excp_cells_most(excp_fine_size(largest))));
}

// And groups beyond that line, as above of tensors whose buckets fit, for which the iterations and initial centres gain more than cells cost:
// 130 us with up to 63 centres, which 1.7 to 2.2 us a million elements are worth up to 54 M elements in tensors of 8 M, and 2.7 to 3.9
// up to 38 M in smaller ones, 4 M at least; 150 to 1100 us with more centres.  (us a call without and with, 4 bits: 2 x 14 M 700 / 618,
// 5 x 6 M 716 / 670, 4 x 10 M 840 / 783, 3 x 15 M 908 / 845, 2 x 25 M 957 / 929, but 10 x 4 M 864 / 873, 36 x 1 M 856 / 860, 3 x 20 M 1065 / 1084,
// 20 x 3 M 1107 / 1202; 6 bits: 6 x 10 M 1131 / 1094, 20 x 3 M 1196 / 1258; 7 bits: 20 x 3 M 1408 / 1351, 5 x 20 M 1769 / 1736, 48 x 2.5 M 2387 / 2442;
// 8 bits: 2 x 14 M 908 / 771, 36 x 1 M 1716 / 1130, 60 x 1 M 2581 / 1664, 5 x 20 M 2165 / 1838.)  Not where every element is kept.
#define EXCP_CELLS_FEW  (36ull << 20)
#define EXCP_CELLS_SOME (52ull << 20)
#define EXCP_CELLS_MANY (100ull << 20)
static inline bool excp_cells_group(u64 elems, u64 largest, u32 tensors, u32 K, u32 whole) {
    if (excp_fine_group(elems, largest, whole)) return true;
    if (whole != 0u || largest > EXCP_FINE_LARGEST) return false;
    if (K >= 127u) return elems <= EXCP_CELLS_MANY;
    return elems <= (elems >= (u64)tensors << 23 ? EXCP_CELLS_SOME : (elems >= (u64)tensors << 22 ? EXCP_CELLS_FEW : 0ull));
}
// Chunks of survivors up to which such a group keeps its cells: half the elements, and more of smaller groups.
static inline u32 excp_cells_chunks(u64 elems) { return elems <= EXCP_CELLS_SOME ? EXCP_FINE_CHUNKS : 2u * EXCP_FINE_CHUNKS; }

// Whether a group's small tensors (k_small.hip) take one launch, in which three workgroups a tensor, one to a stream, each read all of
// its inputs, and that of the residuals writes W_hat.  Nothing makes that one wait for the others, which may begin much later (they need most of
// a compute unit's LDS, and larger tensors may hold it), so W_hat must lie apart from everything that the launch reads: not over the
// previous or the current weights of its own tensor, nor of another.  Otherwise, and where there are more streams than compute units, two
// launches, the first of which reads all inputs before the second writes (a norm vector of 4096 elements 61 us a call, 57 in one).
#define EXCP_SMALL_ONCE 128u
static inline bool excp_small_once(const TDesc *d, u32 count, u32 cus, u32 weight_bytes) {
    if (3u * count > cus || count > EXCP_SMALL_ONCE) return false;
    struct Range { uintptr_t lo, hi; } out[EXCP_SMALL_ONCE];
    u32 outs = 0;
    uintptr_t lo = UINTPTR_MAX, hi = 0;                   // all outputs lie between
    for (u32 q = 0; q < count; ++q) {
        if (!d[q].W_out || !d[q].n) continue;
        const Range r{(uintptr_t)d[q].W_out, (uintptr_t)d[q].W_out + (uintptr_t)d[q].n * weight_bytes};
        lo = std::min(lo, r.lo); hi = std::max(hi, r.hi);
        out[outs++] = r;
    }
    bool sorted = false;
    for (u32 q = 0; q < count; ++q) {
        const void *in[4] = {d[q].Wp, d[q].W, d[q].m, d[q].v};
        for (u32 k = 0; k < 4u && d[q].n; ++k) {
            const uintptr_t a = (uintptr_t)in[k], b = a + (uintptr_t)d[q].n * (k < 2u ? weight_bytes : 4u);
            if (a >= hi || b <= lo) continue;
            if (!sorted) {                                // by their beginnings; `hi`: the furthest end up to here
                std::sort(out, out + outs, [](const Range &x, const Range &y) { return x.lo < y.lo; });
                for (u32 i = 1; i < outs; ++i) out[i].hi = std::max(out[i].hi, out[i - 1u].hi);
                sorted = true;
            }
            const Range *end = std::lower_bound(out, out + outs, b, [](const Range &x, uintptr_t y) { return x.lo < y; });
            if (end != out && end[-1].hi > a) return false;
        }
    }
    return true;
}

// Samples of a stream, from which its buckets are made: 32 to a bucket, whose sizes then differ by 18 %, or 64 and 12 % where
// cells are made and a bucket sixty per cent above the average of the largest tensor, a third of it kept, would fill more than three
// quarters of a workgroup (from 14.7 M elements on; of 25 M a few buckets did not fit otherwise).  More samples cost more to draw, and of
// a sign-like update they are more likely to meet one of the few strays, whose range then leaves all other values in two
// buckets: with 64 to a bucket whenever cells are made, such an update of 10 M elements took 4313 us instead of 1103 before there
// were cells, sixty tensors of 11 M in all 1576 instead of 1113; with 32, 1091 and 1160.)
#define EXCP_SAMPLES_FEW  8192u
#define EXCP_SAMPLES_MANY 16384u
static inline u32 excp_samples(bool cells, u64 largest) {
    return cells && largest / 480u > excp_cells_most(excp_fine_size(largest)) / 4u * 3u ? EXCP_SAMPLES_MANY : EXCP_SAMPLES_FEW;
}

// Tensors so small that one workgroup takes their streams through all Lloyd iterations whatever the values are
// (unless their group goes together and has others).
static inline bool excp_lloyd_small(u64 n, u32 K) { return n <= (K > 3u ? 1ull << 17 : 1ull << 22) && n * (K - 1u) <= (1ull << 24); }

// A work unit of a Lloyd iteration that many workgroups take, in SegState::work: `least`, or so much that the units of
// `streams` streams with `work` in all -- each has one that is not whole -- are at_once at most, or two a stream.  And
// the workgroups of a launch, at least as many as there can be units.
static __host__ __device__ inline u64 excp_lloyd_unit(u64 work, u32 streams, u32 at_once, u32 least) {
    const u32 spare = at_once - (streams < at_once / 2u ? streams : at_once / 2u), whole = spare > streams ? spare : streams;
    const u64 fit = work / whole + 1ull;
    return fit > least ? fit : least;
}
static inline u32 excp_lloyd_grid(u32 at_once, u32 slots) { return at_once + 6u * slots; }

void launch_zero_u32(u32 *p, u64 count, hipStream_t s);
void launch_copy_probe(const void *src, void *dst, u64 bytes, hipStream_t s);
void launch_stats(const Workspace &w, const GroupParams &g, int phase, const TDesc *single, hipStream_t s);
void launch_mask_compact(const Workspace &w, const GroupParams &g, int phase, hipStream_t s);
void launch_km_partition(const Workspace &w, const GroupParams &g, int phase, hipStream_t s);
void launch_km_cells(const Workspace &w, const GroupParams &g, hipStream_t s);
void launch_km_init(const Workspace &w, const GroupParams &g, hipStream_t s);
// A stream of the context's own beside the caller's, and the events that order the two.
struct SideStream { hipStream_t stream; hipEvent_t fork, join; };
void launch_km_iter(const Workspace &w, const GroupParams &g, hipStream_t s, const SideStream &side);
void launch_bitmap_o(const Workspace &w, const GroupParams &g, hipStream_t s);
void launch_assign_pack(const Workspace &w, const GroupParams &g, hipStream_t s);
void launch_small(const Workspace &w, const GroupParams &g, const TDesc *single, bool once, hipStream_t s);
void launch_finalize(const Workspace &w, const GroupParams &g, bool decode, hipStream_t s);
void launch_decode_prep(const Workspace &w, u32 ntensors, u32 ntiles, u32 largest, bool allow_raw, bool moments, bool records, const DDesc *single, hipStream_t s);
static inline bool excp_prep_small(u32 largest) { return largest <= 32u; }      // tiles of the largest tensor of a group that takes one launch
void launch_decode_small(const Workspace &w, u32 ntensors, u32 ntiles, bool moments, bool w16, hipStream_t s);
void launch_decode_main16(const Workspace &w, u32 ntensors, u32 ntiles, bool moments, hipStream_t s);
void launch_decode_raw(const Workspace &w, u32 ntensors, u32 ntiles, bool moments, hipStream_t s);
void launch_store_raw(const Workspace &w, const GroupParams &g, hipStream_t s);
void launch_decode_main(const Workspace &w, u32 ntensors, u32 ntiles, bool moments, hipStream_t s);
void launch_decode_finish(const Workspace &w, u32 ntensors, hipStream_t s);
void launch_export_dense(const Workspace &w, u32 ntensors, u32 ntiles, hipStream_t s);
void launch_dense_parse(const Workspace &w, u32 ntensors, hipStream_t s);
void launch_decode_dense(const Workspace &w, u32 ntensors, u32 ntiles, hipStream_t s);
void launch_decode_chain(const Workspace &w, u32 ntensors, u32 ntiles, bool w16, hipStream_t s);
void launch_chain_finish(const Workspace &w, u32 ntensors, hipStream_t s);

// Joint pruning masks (Sec. 3.2, Eq. "r_w" and Eq. "r_o") and the order-preserving compaction of
// the survivors.
//
// Pass A (k_mask_slots) reads W_prev, W_t, m and v once.  Work unit: a sub-tile of 2048 elements
// (half a 4096-element tile), owned by one wave, which writes the keep bitmap, the sub-tile's
// survivor counts, and the survivors themselves -- in index order, together with their M_o bits --
// into the sub-tile's own slot of a scratch area.  No wave waits for another: where a survivor
// finally goes depends on the counts of all earlier sub-tiles, and that is left to a scan
// (k_mask_scan over the sub-tile counts of every tensor) and to pass B (k_mask_gather), which copies
// every slot to its place in the dense survivor arrays; k_mask_bitmap_o then assembles bitmap_o from
// the sub-tiles' local bit streams.  The extra copy costs 8 bytes per survivor; it replaces a chained
// scan whose waits cost more than that.
#include <algorithm>

#include "excp_util.h"

namespace {

constexpr u32 SUB = 2048;          // elements per sub-tile
constexpr u32 QUARTER = 512;       // elements a wave holds at once
constexpr u32 GROUP = 256;         // elements decided together, four consecutive ones to a lane
constexpr u32 BO_WORDS = SUB / 64; // M_o words kept per sub-tile
constexpr u32 STAGE = QUARTER + 64; // survivors of a stream that wait in LDS for whole lines: less than a line, and a quarter's

// Four consecutive values at an address that is only known to be 4-byte aligned.
typedef float f4m __attribute__((ext_vector_type(4), aligned(4)));
typedef u32 u4m __attribute__((ext_vector_type(4), aligned(4)));

// The bits of one quarter as they arrive (weights as stored: fp32 bit patterns, or 16-bit values): element
// 256 h + 4 lane + j in [h][j].
template <bool W16> struct Regs {
    u32 w[2][W16 ? 2 : 4], p[2][W16 ? 2 : 4];
    float m[2][4], v[2][4];
};

// What a wave needs to know about the sub-tile it works on (all of it the same in every lane).
struct SubTile {
    u64 n, base;                   // elements of the tensor; first element of the sub-tile inside it
    float t_w, r_o;                // the tensor's thresholds
    float T_keep, T_drop;          // t_w^2 with the estimate's guard band on either side
    bool T_ok;                     // t_w^2 is a positive normal number: the estimate may be used at all
    EXCP_GLOBAL float *sw, *sm, *sv;   // the sub-tile's slot in the three survivor areas
};

// Loads of one quarter (512 elements starting at element `first` of the tensor) that lies wholly inside the tensor, sixteen
// bytes a lane (eight of 16-bit weights, whose arrays have to be 8-byte aligned for that).
template <bool W16>
__device__ __forceinline__ void load_quarter(Regs<W16> &R, const TDesc &D, u64 first, u32 lane) {
    const EXCP_GLOBAL float *gM = gptr(D.m) + first, *gV = gptr(D.v) + first;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const u32 off = (u32)h * GROUP + lane * 4u;
        if constexpr (W16) {
            const EXCP_GLOBAL unsigned short *hW = gptr((const unsigned short *)D.W) + first + off;
            const EXCP_GLOBAL unsigned short *hP = gptr((const unsigned short *)D.Wp) + first + off;
            typedef u32 u2 __attribute__((ext_vector_type(2)));
            const u2 a = __builtin_nontemporal_load((const EXCP_GLOBAL u2 *)hW), b = __builtin_nontemporal_load((const EXCP_GLOBAL u2 *)hP);
            R.w[h][0] = a.x; R.w[h][1] = a.y; R.p[h][0] = b.x; R.p[h][1] = b.y;
        } else {
            const u4m a = __builtin_nontemporal_load((const EXCP_GLOBAL u4m *)(gptr((const u32 *)D.W) + first + off)), b = __builtin_nontemporal_load((const EXCP_GLOBAL u4m *)(gptr((const u32 *)D.Wp) + first + off));
#pragma unroll
            for (int j = 0; j < 4; ++j) { R.w[h][j] = a[j]; R.p[h][j] = b[j]; }
        }
        const f4m m = __builtin_nontemporal_load((const EXCP_GLOBAL f4m *)(gM + off)), v = __builtin_nontemporal_load((const EXCP_GLOBAL f4m *)(gV + off));
#pragma unroll
        for (int j = 0; j < 4; ++j) { R.m[h][j] = m[j]; R.v[h][j] = v[j]; }
    }
}

// The same for 16-bit weights at any address.  (Two-byte loads and no second register set: bf16 tensors of 16.8 M elements at an
// odd offset take 54 us, 58 at an aligned one; 4e8 elements 1259.)
template <bool W16>
__device__ __forceinline__ void load_quarter_halves(Regs<W16> &R, const TDesc &D, u64 first, u32 lane) {
    if constexpr (W16) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const u64 at = first + (u32)h * GROUP + lane * 4u;
            const EXCP_GLOBAL unsigned short *hW = gptr((const unsigned short *)D.W) + at, *hP = gptr((const unsigned short *)D.Wp) + at;
#pragma unroll
            for (int j = 0; j < 2; ++j) { R.w[h][j] = (u32)hW[2 * j] | (u32)hW[2 * j + 1] << 16; R.p[h][j] = (u32)hP[2 * j] | (u32)hP[2 * j + 1] << 16; }
            const f4m m = *(const EXCP_GLOBAL f4m *)(gptr(D.m) + at), v = *(const EXCP_GLOBAL f4m *)(gptr(D.v) + at);
#pragma unroll
            for (int j = 0; j < 4; ++j) { R.m[h][j] = m[j]; R.v[h][j] = v[j]; }
        }
    }
}

// The same for a quarter of which only `rem` elements exist (a tensor's ragged end; rem may be 0).
template <bool W16>
__device__ __forceinline__ void load_quarter_ragged(Regs<W16> &R, const TDesc &D, u64 first, u32 rem, u32 lane) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        u32 w[4], p[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const u32 e = (u32)h * GROUP + lane * 4u + (u32)j;
            const bool ok = e < rem;
            const u64 idx = first + e;
            w[j] = ok ? (W16 ? (u32)((const unsigned short *)D.W)[idx] : ((const u32 *)D.W)[idx]) : 0u;
            p[j] = ok ? (W16 ? (u32)((const unsigned short *)D.Wp)[idx] : ((const u32 *)D.Wp)[idx]) : 0u;
            R.m[h][j] = ok ? D.m[idx] : 0.f;
            R.v[h][j] = ok ? D.v[idx] : 1.f;
        }
#pragma unroll
        for (int j = 0; j < (W16 ? 2 : 4); ++j) {
            R.w[h][j] = W16 ? w[2 * j & 3] | w[2 * j + 1 & 3] << 16 : w[j];
            R.p[h][j] = W16 ? p[2 * j & 3] | p[2 * j + 1 & 3] << 16 : p[j];
        }
    }
}

// OR over groups of eight lanes, in all of them: neighbours, pairs, then the two quads.
__device__ __forceinline__ u32 or_of_eight(u32 x) {
    x |= dpp_u32<0xb1, 0xf>(0u, x);           // quad_perm 1 0 3 2
    x |= dpp_u32<0x4e, 0xf>(0u, x);           // quad_perm 2 3 0 1
    x |= dpp_u32<0x141, 0xf>(0u, x);          // row_half_mirror
    return x;
}

// Survivors of one stream on their way from LDS to the sub-tile's slot: whole lines of 256 bytes as they fill up, past the
// caches like the loads.  What bounds this pass is memory: the 16 bytes an element that it reads would take 1218 us for 4e8 elements, the
// 2 bytes that it writes as much as 280 more.  (One element to a lane, survivors stored where they belong a batch at a time,
// everything through the caches: 1625 us; four to a lane and whole lines 1577; stores past the caches 1566; loads as well 1500, but
// 1800 with stores through them.)
struct Outlet { u32 held, done; };             // values waiting in LDS; values written (a multiple of 64)
__device__ __forceinline__ void drain(EXCP_GLOBAL float *slot, float *stage, Outlet &o, u32 lane) {
    wave_lds_fence();
    const u32 lines = o.held >> 6;
    if (lines) {                               // (the same in the whole wave)
        for (u32 k = 0; k < lines; ++k) __builtin_nontemporal_store(stage[k * 64u + lane], &slot[o.done + k * 64u + lane]);
        const float rest = stage[lines * 64u + lane];          // (less than a line is left; the lanes beyond it move what nobody reads)
        wave_lds_fence();
        stage[lane] = rest;
        o.done += lines * 64u; o.held &= 63u;
        wave_lds_fence();
    }
}

// Quarter r (0..3) of a sub-tile: decisions, bitmap words, survivors.  All lanes of the
// wave are active throughout: every decision is first a wave-wide bit mask (the ballot of one
// comparison), the masks are combined as 64-bit integers, and only the final masks become lane
// predicates again.  rem = elements of the quarter that exist (FULL: all 512).
// word: lane l keeps the 32-bit bitmap word of elements 256 (l & 7) + 32 (l >> 3) of the sub-tile (oword: of M_o where that has a
// bit per element).
template <bool NW2M, bool W16, bool FULL>
__device__ __forceinline__ void mask_quarter(const Regs<W16> &R, const SubTile &S, u32 r, u32 rem, u32 flags, u32 *my_bo, float *stage,
                                             u32 lane, Outlet &ow, Outlet &oo, u32 &nf_run, u32 &word, u32 &oword) {
    const bool bf = W16 && excp_wtype(flags) == 2u;
    float *st_w = stage, *st_m = stage + STAGE, *st_v = stage + 2u * STAGE;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        u64 bw[4], bo[4];
        float d[4];
        u32 nw = 0, no = 0;                               // the lane's four keep bits, M_o bits
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const u32 e = (u32)h * GROUP + lane * 4u + (u32)j;
            const u64 valid = FULL ? ~0ull : ballot64(e < rem);
            const float wv = W16 ? w16_widen(R.w[h][j / 2] >> (16 * (j & 1)) & 0xffffu, bf) : u2f(R.w[h][j]);
            const float pv = W16 ? w16_widen(R.p[h][j / 2] >> (16 * (j & 1)) & 0xffffu, bf) : u2f(R.p[h][j]);
            d[j] = wv - pv;                               // the residual
            const float ad = fabsf(d[j]), vv = R.v[h][j], mv = R.m[h][j];
            u64 keep;
            if (flags & 2u) {
                keep = ballot64(ad > S.t_w);              // ablation: the same scalar threshold for every element
            } else {
                // (d^2 may underflow where d^2 v does not: every factor and product must be a positive normal number)
                const float dd = ad * ad, x = dd * vv;
                const u64 b_keep = ballot64(x > S.T_keep), b_drop = ballot64(x < S.T_drop);
                const u64 b_trust = ballot64(__builtin_amdgcn_classf(vv, 0x100)) & ballot64(__builtin_amdgcn_classf(dd, 0x100)) &
                                    ballot64(__builtin_amdgcn_classf(x, 0x100));
                const u64 amb = S.T_ok ? (~(b_keep | b_drop) | ~b_trust) : ~0ull;
                keep = b_keep;
                if (amb & valid) {
                    // sqrtf and '/' are the correctly rounded forms (the build passes
                    // -fhip-fp32-correctly-rounded-divide-sqrt); __fsqrt_rn is NOT on this target
                    const u64 b_exact = ballot64(ad > S.t_w / sqrtf(vv));
                    keep = (b_keep & ~amb) | (b_exact & amb);
                }
            }
            bw[j] = keep & valid;
            nf_run += (u32)__popcll(ballot64((f2u(vv) & 0x7f800000u) == 0x7f800000u) & valid);
            bo[j] = ballot64(fabsf(mv) > S.r_o) & (NW2M ? valid : bw[j]);
            nw |= __builtin_amdgcn_inverse_ballot_w64(bw[j]) ? 1u << j : 0u;
            no |= __builtin_amdgcn_inverse_ballot_w64(bo[j]) ? 1u << j : 0u;
        }
        const u32 at = 2u * r + (u32)h;                   // which 256 elements of the sub-tile
        const u32 wd = or_of_eight(nw << (4u * (lane & 7u)));
        if ((lane & 7u) == at) word = wd;
        if (NW2M) { const u32 od = or_of_eight(no << (4u * (lane & 7u))); if ((lane & 7u) == at) oword = od; }
        // places among the group's survivors: both streams' counts in one scan
        const u32 c = (u32)__popc(nw) | (u32)__popc(no) << 16, incl = wave_incl_scan_u32(c), excl = incl - c, all = last_lane_u32(incl);
        const u32 rw = ow.held + (excl & 0xffffu), ro = oo.held + (excl >> 16);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const u32 kw = rw + (u32)__popc(nw & ((1u << j) - 1u)), ko = ro + (u32)__popc(no & ((1u << j) - 1u));
            if (__builtin_amdgcn_inverse_ballot_w64(bw[j])) st_w[kw] = d[j];
            if (__builtin_amdgcn_inverse_ballot_w64(bo[j])) { st_m[ko] = R.m[h][j]; st_v[ko] = R.v[h][j]; }
        }
        if (!NW2M && no) {
            // the lane's M_o bits in the order of its survivors, at their rank in the sub-tile
            u32 bits = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) bits |= (no >> j & 1u) << __popc(nw & ((1u << j) - 1u));
            const u32 rk = ow.done + rw, sh = rk & 31u;
            atomicOr(&my_bo[rk >> 5], bits << sh);
            if (sh > 28u && bits >> (32u - sh)) atomicOr(&my_bo[(rk >> 5) + 1u], bits >> (32u - sh));
        }
        ow.held += all & 0xffffu; oo.held += all >> 16;
    }
    drain(S.sw, st_w, ow, lane);
    Outlet ov = oo;
    drain(S.sm, st_m, oo, lane);
    drain(S.sv, st_v, ov, lane);
}

// Pass A.  A wave owns whole sub-tiles, neighbouring waves neighbouring ones, and walks each
// in four quarters of 512 elements, four consecutive elements to a lane.  (A wave goes on as many sub-tiles further as there are waves:
// those at work at a time lie together in all seven arrays, where a range of its own for every wave made as many regions.  410M shape
// 1535 -> 1462 us, its weights in bf16 1240 -> 1139, 7B shape, four layers, 4014 -> 3975, 30 M elements 119 -> 116.)  Nothing is shared between waves: no barrier after
// the tile table is loaded.  While one quarter is worked on the next is already on its way from memory (two register sets).
//
// Per element: the residual; the keep decision |d| > t_w / sqrt(v) with correctly rounded sqrt and
// divide -- taken from the estimate d^2 v against t_w^2 when that is not within 1e-5 of the boundary
// (the estimate's own error is below 3e-7) and from the exact expression otherwise, so it is always
// that of the exact expression; the M_o decision.  Survivors go to their rank in LDS and from there, as whole lines, to
// the sub-tile's slot; the M_o bits of kept residuals are ORed into the wave's own
// LDS words at the residuals' ranks.
//
// NW2M (Table "vit", no weights-to-momentum check): M_o(i) = |m_i| > r_o for every element, kept
// weight or not; the sub-tile's M_o words are then indexed by element.
// W16: the two weight arrays hold 16-bit values (fp16 or bf16 by the flags), widened as they are used.
template <bool NW2M, bool W16>
__global__ __launch_bounds__(EXCP_THREADS, 4) void k_mask_slots(Workspace w, GroupParams g) {
    __shared__ u32 s_bo[EXCP_THREADS / 64][SUB / 32 + 1];  // per wave: M_o bits of its sub-tile's kept residuals, by rank
    __shared__ float s_stage[EXCP_THREADS / 64][3 * STAGE];
    __shared__ u32 s_tiles[EXCP_MAX_GROUP_TENSORS + 1];
    const u32 lane = threadIdx.x & 63u;
    const u32 wave = (u32)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const u32 nsub = 2u * g.ntiles;
    load_tile_table(s_tiles, w.tile_begin, g.ntensors);
    const u32 nwaves = gridDim.x * (EXCP_THREADS / 64), wid = blockIdx.x * (EXCP_THREADS / 64) + wave;
    u32 *my_bo = s_bo[wave];
    float *stage = s_stage[wave];
    my_bo[lane] = 0u;
    if (lane == 0u) my_bo[SUB / 32] = 0u;
    u32 t = 0, first_sub = 0, end_sub = 0;                // the tensor in hand, its first sub-tile, one past its last
    Regs<W16> A, B;
    for (u32 sub = wid; sub < nsub; sub += nwaves) {
        if (sub >= end_sub) {                             // (looked up again only when a tensor's sub-tiles run out)
            t = (u32)__builtin_amdgcn_readfirstlane((int)find_owner(s_tiles, g.ntensors, sub >> 1));
            first_sub = (u32)__builtin_amdgcn_readfirstlane((int)(2u * s_tiles[t]));
            end_sub = (u32)__builtin_amdgcn_readfirstlane((int)(2u * s_tiles[t + 1u]));
        }
        // The tensor's description and thresholds are not written by this kernel: read as constant
        // memory they come through the scalar unit, which global memory that the kernel also
        // stores to may not.
        const EXCP_CONSTANT TDesc *Dc = (const EXCP_CONSTANT TDesc *)(uintptr_t)(w.desc + t);
        const EXCP_CONSTANT TState *St = (const EXCP_CONSTANT TState *)(uintptr_t)(w.st + t);
        TDesc D;
        D.Wp = Dc->Wp; D.W = Dc->W; D.m = Dc->m; D.v = Dc->v; D.n = Dc->n; D.blob = Dc->blob; D.elem_off = Dc->elem_off;
        SubTile S;
        S.n = D.n; S.base = (u64)(sub - first_sub) * SUB;
        S.t_w = St->t_w; S.r_o = St->r_o;
        const float T = S.t_w * S.t_w;
        S.T_keep = T * 1.00001f; S.T_drop = T * 0.99999f; S.T_ok = __builtin_amdgcn_classf(T, 0x100);
        const u64 slot = D.elem_off + S.base;
        S.sw = gptr(w.pw) + slot; S.sm = gptr(w.pm) + slot; S.sv = gptr(w.pv) + slot;
        Outlet ow = {0u, 0u}, oo = {0u, 0u};
        u32 nf_run = 0, word = 0, oword = 0;
        if (S.base + SUB <= S.n && (!W16 || (((uintptr_t)D.W | (uintptr_t)D.Wp) & 7u) == 0u)) {
            load_quarter<W16>(A, D, S.base, lane);
            load_quarter<W16>(B, D, S.base + QUARTER, lane);
            mask_quarter<NW2M, W16, true>(A, S, 0u, QUARTER, g.flags, my_bo, stage, lane, ow, oo, nf_run, word, oword);
            load_quarter<W16>(A, D, S.base + 2u * QUARTER, lane);
            mask_quarter<NW2M, W16, true>(B, S, 1u, QUARTER, g.flags, my_bo, stage, lane, ow, oo, nf_run, word, oword);
            load_quarter<W16>(B, D, S.base + 3u * QUARTER, lane);
            mask_quarter<NW2M, W16, true>(A, S, 2u, QUARTER, g.flags, my_bo, stage, lane, ow, oo, nf_run, word, oword);
            mask_quarter<NW2M, W16, true>(B, S, 3u, QUARTER, g.flags, my_bo, stage, lane, ow, oo, nf_run, word, oword);
        } else {
#pragma unroll 1
            for (u32 r = 0; r < 4u; ++r) {
                const u64 first = S.base + (u64)r * QUARTER;
                const u32 rem = S.n > first ? (S.n - first < (u64)QUARTER ? (u32)(S.n - first) : QUARTER) : 0u;
                if (W16 && rem == QUARTER) load_quarter_halves(A, D, first, lane);      // (arrays of 16-bit weights that are not 8-byte aligned)
                else load_quarter_ragged<W16>(A, D, first, rem, lane);
                mask_quarter<NW2M, W16, false>(A, S, r, rem, g.flags, my_bo, stage, lane, ow, oo, nf_run, word, oword);
            }
        }
        // the sub-tile is complete: what is left of the survivors, its bitmap words, its M_o words (by survivor rank), its counts
        if (lane < ow.held) S.sw[ow.done + lane] = stage[lane];
        if (lane < oo.held) { S.sm[oo.done + lane] = stage[STAGE + lane]; S.sv[oo.done + lane] = stage[2u * STAGE + lane]; }
        const u32 cw = ow.done + ow.held, co = oo.done + oo.held;
        const u32 mine = (lane & 7u) * 8u + (lane >> 3);  // 32-bit word of the sub-tile that this lane has
        const u64 nwords = excp_words(S.n), first_word = S.base >> 6;
        EXCP_GLOBAL u32 *bm = gptr((u32 *)(D.blob + EXCP_HEADER + excp_books_bytes((u32)g.nbits))) + 2u * first_word;
        // (words past the last element are zero: that is the section's 16-byte padding)
        if (first_word + (mine >> 1) < nwords + (nwords & 1ull)) bm[mine] = word;
        u64 *bo = w.mask_bo + (u64)sub * BO_WORDS;
        if (NW2M) {
            ((u32 *)bo)[mine] = oword;
        } else {
            wave_lds_fence();
            const u64 bits = (u64)my_bo[2u * (lane & 31u)] | ((u64)my_bo[2u * (lane & 31u) + 1u] << 32);
            if (lane < ((cw + 63u) >> 6)) bo[lane] = bits;
            wave_lds_fence();
            my_bo[lane] = 0u;
        }
        if (lane == 0u) {
            w.tile_status[sub] = ((u64)cw << 32) | (u64)co;
            if (nf_run) atomicAdd(&w.st[t].nonfinite, (u64)nf_run);
        }
        wave_lds_fence();
    }
}

// One wave copies floats in batches of N x 64; every load of a batch is issued before its stores so
// that a copy is not a chain of dependent round trips.
template <int N>
__device__ __forceinline__ void load_batch(float (&q)[N], const EXCP_GLOBAL float *src, u32 cnt, u32 b0, u32 lane) {
#pragma unroll
    for (int k = 0; k < N; ++k) {
        const u32 i = b0 + (u32)k * 64u + lane;
        q[k] = i < cnt ? src[i] : 0.f;
    }
}
template <int N>
__device__ __forceinline__ void store_batch(EXCP_GLOBAL float *dst, const float (&q)[N], u32 cnt, u32 b0, u32 lane) {
#pragma unroll
    for (int k = 0; k < N; ++k) {
        const u32 i = b0 + (u32)k * 64u + lane;
        if (i < cnt) dst[i] = q[k];
    }
}

// Exclusive scan of the sub-tile counts of every tensor; the totals are the tensor's n_w and n_o.
// Counts are packed (survivors << 32 | moment survivors).  A tensor's sub-tiles are cut into sixteen
// parts, one workgroup each, which begins from the sum of the parts before it: it adds their counts up itself, or, where those are
// more than MSCAN_DIRECT, their totals, which a launch before this one has made.  (16.8 M elements: 4.7 us and a launch less.)
constexpr u32 MSCAN_PARTS = 16, MSCAN_DIRECT = 1u << 14;

__device__ __forceinline__ void mscan_range(u32 nsub, u32 part, u32 &s0, u32 &s1) {
    const u32 per = ((nsub + MSCAN_PARTS - 1u) / MSCAN_PARTS + 3u) & ~3u;
    s0 = min(part * per, nsub);
    s1 = min(s0 + per, nsub);
}

__global__ __launch_bounds__(EXCP_THREADS) void k_mask_scan_parts(Workspace w, GroupParams g) {
    __shared__ u64 s_sum[EXCP_THREADS / 64];
    const u32 t = blockIdx.x / MSCAN_PARTS, part = blockIdx.x % MSCAN_PARTS, tid = threadIdx.x;
    const TDesc &D = w.desc[t];
    u32 s0, s1;
    mscan_range(2u * D.tile_count, part, s0, s1);
    const u64 *cnt = w.tile_status + 2ull * D.tile_begin;
    u64 local = 0;
    for (u32 i = s0 + tid; i < s1; i += EXCP_THREADS) local += cnt[i];
    local = wave_sum_u64(local);
    if ((tid & 63u) == 0u) s_sum[tid >> 6] = local;
    __syncthreads();
    if (tid == 0) w.mask_part[(u64)t * MSCAN_PARTS + part] = (s_sum[0] + s_sum[1]) + (s_sum[2] + s_sum[3]);
}

// After the masks: blob section offsets, capacity check, survivor stream lengths and the chunk
// list of the survivor passes.  One workgroup; tensors and streams are few.  The counts come from other workgroups of the launch:
// they are written and read past the caches that the compute dies do not share.
__device__ __forceinline__ u64 load_count(const u64 *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void layout(const Workspace &w, const GroupParams &g) {
    u32 *seg_chunk_begin = w.seg_chunk_begin;
    __shared__ u32 s_sum[2][EXCP_THREADS / 64];
    const u32 tid = threadIdx.x;
    const u32 nseg = 3u * g.ntensors;
    const u32 per = (nseg + EXCP_THREADS - 1) / EXCP_THREADS;
    u32 local[2] = {0u, 0u};                              // chunks, rows of the count table
    const u32 unit_chunks = (1u << g.unit_shift) / EXCP_CHUNK;
    for (u32 q = 0; q < per; ++q) {
        u32 sidx = tid * per + q;
        if (sidx >= nseg) break;
        u32 t = sidx / 3u, which = sidx % 3u;
        TState &S = w.st[t];
        const TDesc &D = w.desc[t];
        if (which == 0) {
            const u64 n = D.n, nw = load_count(&S.n_w), no = load_count(&S.n_o), nb = (u64)g.nbits;
            u64 off = EXCP_HEADER + excp_books_bytes((u32)g.nbits) + excp_pad16(8ull * excp_words(n));
            S.off_bo = off; off += excp_pad16(8ull * excp_words((g.flags & 8u) ? n : nw));
            S.off_cw = off; off += excp_pad16(8ull * excp_words(nw * nb));
            S.off_cm = off; off += excp_pad16(8ull * excp_words(no * nb));
            S.off_cv = off; off += excp_pad16(8ull * excp_words(no * nb));
            S.blob_bytes = off;
            int status = 0;
            if (off > D.blob_cap) status = -2;
            if (S.nonfinite) status = -3;
            S.status = status;
        }
    }
    for (u32 q = 0; q < per; ++q) {
        u32 sidx = tid * per + q;
        if (sidx >= nseg) break;
        u32 t = sidx / 3u, which = sidx % 3u;
        TState &S = w.st[t];
        // the status is recomputed here: (t, 1) and (t, 2) may belong to another thread than (t, 0)
        u64 len = load_count(which == 0 ? &S.n_w : &S.n_o);
        const TDesc &D = w.desc[t];
        {
            const u64 n = D.n, nw = load_count(&S.n_w), no = load_count(&S.n_o), nb = (u64)g.nbits;
            u64 off = EXCP_HEADER + excp_books_bytes((u32)g.nbits) + excp_pad16(8ull * excp_words(n));
            off += excp_pad16(8ull * excp_words((g.flags & 8u) ? n : nw)) + excp_pad16(8ull * excp_words(nw * nb)) +
                   2ull * excp_pad16(8ull * excp_words(no * nb));
            if (off > D.blob_cap || S.nonfinite) len = 0;
        }
        w.seg[sidx].len = len;
        const u32 chunks = (u32)((len + EXCP_CHUNK - 1) / EXCP_CHUNK);
        local[0] += chunks;
        local[1] += (chunks + unit_chunks - 1u) / unit_chunks;
    }
    u32 run[2], total[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        u32 incl = wave_incl_scan_u32(local[q]);
        if ((tid & 63u) == 63u) s_sum[q][tid >> 6] = incl;
        run[q] = incl - local[q];
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        total[q] = 0;
        for (u32 v = 0; v < EXCP_THREADS / 64; ++v) { if (v < (tid >> 6)) run[q] += s_sum[q][v]; total[q] += s_sum[q][v]; }
    }
    for (u32 q = 0; q < per; ++q) {
        u32 sidx = tid * per + q;
        if (sidx >= nseg) break;
        seg_chunk_begin[sidx] = run[0];
        w.seg[sidx].chunk_begin = run[0];
        w.seg[sidx].row_begin = run[1];
        const u32 chunks = (u32)((w.seg[sidx].len + EXCP_CHUNK - 1) / EXCP_CHUNK);
        run[0] += chunks;
        run[1] += (chunks + unit_chunks - 1u) / unit_chunks;
    }
    if (tid == EXCP_THREADS - 1) { seg_chunk_begin[nseg] = total[0]; *w.chunk_total = total[0]; *w.lloyd_shared = 0u; *w.no_cells = total[0] > g.fine_chunks ? 1u : 0u; }
}

// (The workgroup that finds a tensor's totals draws a ticket; the last one goes on with the layout.)
__global__ __launch_bounds__(EXCP_THREADS) void k_mask_scan(Workspace w, GroupParams g, u32 direct) {
    __shared__ u64 s_wave[EXCP_THREADS / 64], s_before[EXCP_THREADS / 64];
    __shared__ u32 s_ticket;
    const u32 t = blockIdx.x / MSCAN_PARTS, part = blockIdx.x % MSCAN_PARTS, tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    const TDesc &D = w.desc[t];
    const u32 nsub = 2u * D.tile_count;
    u32 s0, s1;
    mscan_range(nsub, part, s0, s1);
    const u64 *cnt = w.tile_status + 2ull * D.tile_begin;
    u64 carry = 0;
    if (direct) {
        for (u32 i = tid; i < s0; i += 8u * EXCP_THREADS) {
            u64 v[8];
#pragma unroll
            for (u32 q = 0; q < 8; ++q) v[q] = i + q * EXCP_THREADS < s0 ? cnt[i + q * EXCP_THREADS] : 0ull;
#pragma unroll
            for (u32 q = 0; q < 8; ++q) carry += v[q];
        }
    } else if (tid < part) {
        carry = w.mask_part[(u64)t * MSCAN_PARTS + tid];
    }
    carry = wave_sum_u64(carry);
    if (lane == 0u) s_before[wave] = carry;
    __syncthreads();
    carry = (s_before[0] + s_before[1]) + (s_before[2] + s_before[3]);
    for (u32 base = s0; base < s1; base += EXCP_THREADS * 4) {
        // four consecutive sub-tiles per thread
        u64 v[4], local = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            u32 i = base + tid * 4 + q;
            v[q] = (i < s1) ? cnt[i] : 0ull;
            local += v[q];
        }
        const u64 incl = wave_incl_scan_u64(local);
        if (lane == 63u) s_wave[wave] = incl;
        __syncthreads();
        u64 run = carry + incl - local;
        for (u32 q = 0; q < wave; ++q) run += s_wave[q];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            u32 i = base + tid * 4 + q;
            if (i < s1) w.mask_prefix[2ull * D.tile_begin + i] = run;
            run += v[q];
        }
        carry += (s_wave[0] + s_wave[1]) + (s_wave[2] + s_wave[3]);
        __syncthreads();
    }
    if (part == MSCAN_PARTS - 1u && tid == 0) {
        __hip_atomic_store(&w.st[t].n_w, carry >> 32, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&w.st[t].n_o, carry & 0xffffffffull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");        // (both have arrived before the ticket is drawn)
        s_ticket = atomicAdd(w.scan_ticket, 1u);
    }
    if (part != MSCAN_PARTS - 1u) return;
    __syncthreads();
    if (s_ticket != g.ntensors - 1u) return;
    if (tid == 0) *w.scan_ticket = 0u;
    layout(w, g);
}

// Pass B: one wave per sub-tile copies the slot to its place in the dense survivor arrays.  A workgroup takes a
// contiguous range of batches of up to 32 consecutive sub-tiles; a batch's counts, prefixes and tensor data are
// fetched once, side by side, into LDS, so that a wave's copies do not wait behind a chain of dependent
// look-ups.
// The same pass counts, for the value partition of the codebook stage, how many of the values it moves
// fall into each of the 256 value buckets (the map k_km_sample made from the slots): the values are in
// registers here, and a pass of its own would read them all again.  Counts are kept per unit of 2^14 to 2^17
// positions of a stream (excp_unit_shift), a row each; the scatter's workgroups begin only at such positions.  A workgroup adds up in LDS as long as its batches stay inside one tensor
// and one such unit per stream, and hands the sums over when that changes.
// A wave takes its sub-tiles of a batch one after the other (how many a batch has: excp_gather_subs).
constexpr u32 GATHER_SUBS = EXCP_GATHER_SUBS;

__global__ __launch_bounds__(EXCP_THREADS) void k_mask_gather(Workspace w, GroupParams g, u32 subs) {
    __shared__ u32 s_tiles[EXCP_MAX_GROUP_TENSORS + 1];
    __shared__ u32 s_tw[GATHER_SUBS], s_to[GATHER_SUBS], s_pw[GATHER_SUBS], s_po[GATHER_SUBS], s_t[GATHER_SUBS];
    __shared__ u64 s_slot[GATHER_SUBS], s_eoff[GATHER_SUBS];
    __shared__ u32 s_map[3][EXCP_KM_MAP_WORDS];
    __shared__ u32 s_hist[3][2][256];
    const u32 tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    const u32 nsub = 2u * g.ntiles;
    const bool counting = (g.flags & 4u) == 0u;          // (no codebooks without quantisation)
    load_tile_table(s_tiles, w.tile_begin, g.ntensors);
    const u32 nbatch = (nsub + subs - 1u) / subs;
    const u32 b_lo = (u32)(((u64)blockIdx.x * nbatch) / gridDim.x), b_hi = (u32)(((u64)(blockIdx.x + 1u) * nbatch) / gridDim.x);
    for (u32 i = tid; i < 3u * 2u * 256u; i += EXCP_THREADS) (&s_hist[0][0][0])[i] = 0;
    u32 cur_t = 0xffffffffu, cur_sc[3] = {0u, 0u, 0u};   // what the LDS counts belong to
    bool live[3] = {false, false, false};                // the stream has a place in the chunk list (its tensor did not fail)
    // hands the counts over: thread b adds bucket b of both units of the three streams
    auto flush = [&]() {
        __syncthreads();
        if (cur_t != 0xffffffffu) {
#pragma unroll
            for (u32 k = 0; k < 3; ++k) {
                if (!live[k]) continue;
                const u32 row0 = w.seg[3u * cur_t + k].row_begin + cur_sc[k];
#pragma unroll
                for (u32 u = 0; u < 2; ++u) {
                    const u32 h = s_hist[k][u][tid];
                    if (h) { atomicAdd(&w.km_cnt[(u64)(row0 + u) * 256u + tid], h); s_hist[k][u][tid] = 0; }
                }
            }
        }
        __syncthreads();
    };
    for (u32 batch = b_lo; batch < b_hi; ++batch) {
        const u32 sub0 = batch * subs;
        __syncthreads();
        if (tid < subs) {
            const u32 sub = sub0 + tid;
            u32 tw = 0, to = 0;
            if (sub < nsub) {
                const u64 c = w.tile_status[sub], pre = w.mask_prefix[sub];
                tw = (u32)(c >> 32); to = (u32)c;
                const u32 t = find_owner(s_tiles, g.ntensors, sub >> 1);
                const u64 eoff = w.desc[t].elem_off;
                s_pw[tid] = (u32)(pre >> 32); s_po[tid] = (u32)pre; s_t[tid] = t;
                s_eoff[tid] = eoff;
                s_slot[tid] = eoff + (u64)(sub - 2u * s_tiles[t]) * SUB;
            }
            s_tw[tid] = tw; s_to[tid] = to;
        }
        __syncthreads();
        const u32 nvalid = min(subs, nsub - sub0);
        const u32 t0 = s_t[0];
        const bool one_tensor = t0 == s_t[nvalid - 1u];
        if (counting) {
            if (one_tensor) {
                const u32 sc[3] = {s_pw[0] >> g.unit_shift, s_po[0] >> g.unit_shift, s_po[0] >> g.unit_shift};
                if (t0 != cur_t || sc[0] != cur_sc[0] || sc[1] != cur_sc[1]) {
                    flush();
                    if (t0 != cur_t) {
#pragma unroll
                        for (u32 k = 0; k < 3; ++k) {
                            live[k] = w.seg[3u * t0 + k].len != 0;
                            if (live[k])
                                for (u32 i = tid; i < EXCP_KM_MAP_WORDS; i += EXCP_THREADS) s_map[k][i] = w.km_split[(u64)(3u * t0 + k) * EXCP_KM_MAP_WORDS + i];
                        }
                    }
                    cur_t = t0; cur_sc[0] = sc[0]; cur_sc[1] = sc[1]; cur_sc[2] = sc[2];
                    __syncthreads();
                }
            } else if (cur_t != 0xffffffffu) {
                flush();
                cur_t = 0xffffffffu;
            }
        }
        const bool in_lds = counting && one_tensor;
        u32 par[3][4] = {};                              // the maps' four parameters, out of LDS once per batch
        if (in_lds) {
#pragma unroll
            for (u32 k = 0; k < 3; ++k)
                if (live[k]) { par[k][0] = s_map[k][0]; par[k][1] = s_map[k][1]; par[k][2] = s_map[k][2]; par[k][3] = s_map[k][3]; }
        }
        for (u32 j = wave; j < nvalid; j += 4) {
            const u32 tw = s_tw[j], to = s_to[j];
            if (tw == 0 && to == 0) continue;
            const u32 pw = s_pw[j], po = s_po[j];
            const u64 slot = s_slot[j], eoff = s_eoff[j];
            const EXCP_GLOBAL float *sw = gptr(w.pw) + slot, *sm = gptr(w.pm) + slot, *sv = gptr(w.pv) + slot;
            EXCP_GLOBAL float *xw = gptr(w.xw) + eoff + pw;
            EXCP_GLOBAL float *xm = gptr(w.xm) + eoff + po;
            EXCP_GLOBAL float *xv = gptr(w.xv) + eoff + po;
            // counts of a batch that holds the end of one tensor and the start of the next (small tensors) go
            // straight to the table, with that tensor's maps read where they are: what a stream needs for
            // that is fetched once per sub-tile
            const u32 tj = s_t[j];
            u32 g_row[3] = {0u, 0u, 0u}, g_par[3][4] = {};
            bool g_live[3] = {false, false, false};
            const EXCP_GLOBAL unsigned char *g_cells[3] = {nullptr, nullptr, nullptr};
            if (counting && !in_lds) {
#pragma unroll
                for (u32 k = 0; k < 3; ++k) {
                    const u32 sg = 3u * tj + k;
                    g_live[k] = w.seg[sg].len != 0;
                    g_row[k] = w.seg[sg].row_begin;
                    const u32 *mp = w.km_split + (u64)sg * EXCP_KM_MAP_WORDS;
                    if (g_live[k]) { g_par[k][0] = mp[0]; g_par[k][1] = mp[1]; g_par[k][2] = mp[2]; g_par[k][3] = mp[3]; }
                    g_cells[k] = gptr((const unsigned char *)(mp + 4));
                }
            }
            auto count = [&](u32 k, float x, u32 place) {
                if (in_lds) {
                    if (live[k]) atomicAdd(&s_hist[k][(place >> g.unit_shift) != cur_sc[k] ? 1u : 0u][((const unsigned char *)(s_map[k] + 4))[cell_of(x, par[k])]], 1u);
                } else if (g_live[k]) {
                    const u32 row = g_row[k] + (place >> g.unit_shift);
                    atomicAdd(&w.km_cnt[(u64)row * 256u + g_cells[k][cell_of(x, g_par[k])]], 1u);
                }
            };
            {
                // the first batch of all three runs in flight together (usually there is no second)
                float qw[12], qm[4], qv[4];
                load_batch<12>(qw, sw, tw, 0, lane); load_batch<4>(qm, sm, to, 0, lane); load_batch<4>(qv, sv, to, 0, lane);
                store_batch<12>(xw, qw, tw, 0, lane); store_batch<4>(xm, qm, to, 0, lane); store_batch<4>(xv, qv, to, 0, lane);
                if (counting) {
#pragma unroll
                    for (u32 k = 0; k < 12; ++k) { const u32 i = k * 64u + lane; if (i < tw) count(0, qw[k], pw + i); }
#pragma unroll
                    for (u32 k = 0; k < 4; ++k) { const u32 i = k * 64u + lane; if (i < to) { count(1, qm[k], po + i); count(2, qv[k], po + i); } }
                }
                for (u32 b0 = 768u; b0 < tw; b0 += 768u) {
                    load_batch<12>(qw, sw, tw, b0, lane); store_batch<12>(xw, qw, tw, b0, lane);
                    if (counting) {
#pragma unroll
                        for (u32 k = 0; k < 12; ++k) { const u32 i = b0 + k * 64u + lane; if (i < tw) count(0, qw[k], pw + i); }
                    }
                }
                for (u32 b0 = 256u; b0 < to; b0 += 256u) {
                    load_batch<4>(qm, sm, to, b0, lane); load_batch<4>(qv, sv, to, b0, lane);
                    store_batch<4>(xm, qm, to, b0, lane); store_batch<4>(xv, qv, to, b0, lane);
                    if (counting) {
#pragma unroll
                        for (u32 k = 0; k < 4; ++k) { const u32 i = b0 + k * 64u + lane; if (i < to) { count(1, qm[k], po + i); count(2, qv[k], po + i); } }
                    }
                }
            }
        }
    }
    if (counting) flush();
}

// bitmap_o (the M_o bits of the survivors, in survivor order) from the sub-tiles' local bit
// streams.  Output-centric: one lane builds one 64-bit word from the one to three sub-tiles whose
// survivors it covers, so the words are written whole, once, with no atomics; a wave takes 64
// consecutive words (4096 survivor positions) of one tensor.  The sub-tile that holds the wave's
// first position is found by a 64-way search over the tensor's scanned survivor counts.
__global__ __launch_bounds__(EXCP_THREADS) void k_mask_bitmap_o(Workspace w, GroupParams g) {
    __shared__ u32 s_tiles[EXCP_MAX_GROUP_TENSORS + 1];
    __shared__ u32 s_P[4][65], s_c[4][64];
    const u32 tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    load_tile_table(s_tiles, w.tile_begin, g.ntensors);
    for (u32 blk = blockIdx.x * 4 + wave; blk < g.ntiles; blk += gridDim.x * 4) {
        const u32 t = find_owner(s_tiles, g.ntensors, blk);
        const u32 b = blk - s_tiles[t];                     // the tensor's b-th run of 64 words
        const u32 n_w = (u32)w.st[t].n_w;
        const u32 nwo = (u32)excp_words(n_w), padded = nwo + (nwo & 1u);   // section length, zero-padded to 16 bytes
        if (64u * b >= padded) continue;
        const TDesc &D = w.desc[t];
        const u64 off_bo = EXCP_HEADER + excp_books_bytes((u32)g.nbits) + excp_pad16(8ull * excp_words(D.n));
        const u64 cap_words = (D.blob_cap > off_bo) ? (D.blob_cap - off_bo) >> 3 : 0ull;
        const u32 sb = 2u * s_tiles[t], se = 2u * s_tiles[t + 1];
        const u32 Q0 = 4096u * b;
        // last sub-tile whose first survivor position is <= Q0 (positions are non-decreasing)
        u32 lo = sb, hi = se;
        while (hi - lo > 1u) {
            const u32 span = hi - lo - 1u;                  // open choices lo + 1 .. hi - 1
            const bool act = span > 64u || lane < span;
            const u32 idx = span > 64u ? lo + 1u + (u32)(((u64)span * lane) >> 6) : lo + 1u + lane;
            const u32 P = act ? (u32)(w.mask_prefix[idx] >> 32) : 0xffffffffu;
            const u64 le = ballot64(act && P <= Q0);        // a run of ones from lane 0 up
            const u32 cnt = __popcll(le), nact = span > 64u ? 64u : span;
            const u32 up = __shfl(idx, cnt ? cnt - 1u : 0u, WAVE), dn = __shfl(idx, cnt < 64u ? cnt : 63u, WAVE);
            if (cnt < nact) hi = dn;
            if (cnt) lo = up;
        }
        const u32 s0 = lo;
        // the next 64 sub-tiles: first survivor position and survivor count, side by side in LDS
        {
            const u32 si = s0 + lane;
            const bool in = si < se;
            s_P[wave][lane] = in ? (u32)(w.mask_prefix[si] >> 32) : 0xffffffffu;
            s_c[wave][lane] = in ? (u32)(w.tile_status[si] >> 32) : 0u;
            if (lane == 0) s_P[wave][64] = 0xffffffffu;
        }
        const u32 widx = 64u * b + lane;
        if (widx >= padded) continue;
        u64 word = 0;
        if (widx < nwo) {
            const u32 Q = widx * 64u;                        // this word covers survivor positions [Q, Q + 64)
            u32 i = 0;                                       // last entry of the window with position <= Q
#pragma unroll
            for (u32 step = 32; step >= 1; step >>= 1) if (s_P[wave][i + step] <= Q) i += step;
            for (;; ++i) {
                const u32 cur = s0 + i;
                if (cur >= se) break;
                const u32 P = i < 64u ? s_P[wave][i] : (u32)(w.mask_prefix[cur] >> 32);
                if (P >= Q + 64u) break;
                const u32 c = i < 64u ? s_c[wave][i] : (u32)(w.tile_status[cur] >> 32);
                if (P + c <= Q) continue;                    // ends before this word (or is empty)
                const u32 a = max(Q, P), e = min(Q + 64u, P + c);      // overlap, in survivor positions
                const u32 la = a - P, len = e - a;           // first local bit, number of bits
                const u64 *loc = w.mask_bo + (u64)cur * BO_WORDS;
                const u32 k = la >> 6, sh = la & 63u;
                const u64 w0 = loc[k];
                const u64 w1 = ((k + 1u) * 64u < c) ? loc[k + 1u] : 0ull;
                u64 bits = sh ? ((w0 >> sh) | (w1 << (64u - sh))) : w0;
                if (len < 64u) bits &= (1ull << len) - 1ull;
                word |= bits << (a - Q);
            }
        }
        if (widx < cap_words) ((u64 *)(D.blob + off_bo))[widx] = word;
    }
}

// bitmap_o without the weights-to-momentum check: one bit per element, so the sub-tiles' words are
// already the section's words, 32 per sub-tile.
__global__ __launch_bounds__(EXCP_THREADS) void k_mask_bitmap_o_elems(Workspace w, GroupParams g) {
    __shared__ u32 s_tiles[EXCP_MAX_GROUP_TENSORS + 1];
    const u32 tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    load_tile_table(s_tiles, w.tile_begin, g.ntensors);
    for (u32 blk = blockIdx.x * 4 + wave; blk < g.ntiles; blk += gridDim.x * 4) {
        const u32 t = find_owner(s_tiles, g.ntensors, blk);
        const u32 b = blk - s_tiles[t];                     // the tensor's b-th tile = 64 words
        const TDesc &D = w.desc[t];
        const u64 nwo = excp_words(D.n), padded = nwo + (nwo & 1ull);
        const u64 widx = 64ull * b + lane;
        if (widx >= padded) continue;
        const u64 off_bo = EXCP_HEADER + excp_books_bytes((u32)g.nbits) + excp_pad16(8ull * nwo);
        const u64 cap_words = (D.blob_cap > off_bo) ? (D.blob_cap - off_bo) >> 3 : 0ull;
        const u64 word = widx < nwo ? w.mask_bo[(2ull * blk + (lane >> 5)) * BO_WORDS + (lane & 31u)] : 0ull;
        if (widx < cap_words) ((u64 *)(D.blob + off_bo))[widx] = word;
    }
}

}  // namespace

void launch_mask_compact(const Workspace &w, const GroupParams &g, int phase, hipStream_t s) {
    if (!g.ntiles && phase != 1) return;                   // (the scan also makes the layout, of empty tensors too)
    const u32 nsub = 2u * g.ntiles;
    if (phase == 0) {
        // A sub-tile to each wave, up to eighty workgroups a compute unit, which then take a few each: the fewer, the closer together
        // those lie that are at work (20, 40, 80, 160 workgroups: 410M shape 1454, 1441, 1419, 1442 us, bf16 weights 1195, 1129, 1097, 1105,
        // four layers of the 7B shape 3947, 3904, 3890, 3907; 30 M elements 116 with eight, 106 with a sub-tile to each wave).
        const dim3 grid(std::min(excp_grid(w, 80), (nsub + 3u) / 4u)), block(EXCP_THREADS);
        const bool nw2m = (g.flags & 8u) != 0, w16 = (g.flags & 0x30u) != 0;
        if (nw2m && w16) hipLaunchKernelGGL((k_mask_slots<true, true>), grid, block, 0, s, w, g);
        else if (nw2m) hipLaunchKernelGGL((k_mask_slots<true, false>), grid, block, 0, s, w, g);
        else if (w16) hipLaunchKernelGGL((k_mask_slots<false, true>), grid, block, 0, s, w, g);
        else hipLaunchKernelGGL((k_mask_slots<false, false>), grid, block, 0, s, w, g);
    } else if (phase == 1) {
        const bool direct = g.largest <= (u64)MSCAN_DIRECT * SUB;
        if (!direct) hipLaunchKernelGGL(k_mask_scan_parts, dim3(g.ntensors * MSCAN_PARTS), dim3(EXCP_THREADS), 0, s, w, g);
        hipLaunchKernelGGL(k_mask_scan, dim3(g.ntensors * MSCAN_PARTS), dim3(EXCP_THREADS), 0, s, w, g, direct ? 1u : 0u);
    } else {
        const u32 subs = excp_gather_subs(g.ntiles, (u32)w.cus);
        u32 grid = (nsub + subs - 1u) / subs;
        if (grid > excp_grid(w, 48)) grid = excp_grid(w, 48);
        hipLaunchKernelGGL(k_mask_gather, dim3(grid), dim3(EXCP_THREADS), 0, s, w, g, subs);
    }
}

// bitmap_o, any time after the scan (phase 1).
void launch_bitmap_o(const Workspace &w, const GroupParams &g, hipStream_t s) {
    if (!g.ntiles) return;
    const u32 grid = std::min((g.ntiles + 3u) / 4u, excp_grid(w, 16));
    if (g.flags & 8u) hipLaunchKernelGGL(k_mask_bitmap_o_elems, dim3(grid), dim3(EXCP_THREADS), 0, s, w, g);
    else hipLaunchKernelGGL(k_mask_bitmap_o, dim3(grid), dim3(EXCP_THREADS), 0, s, w, g);
}

// Full-tensor statistics for the pruning thresholds of Sec. 3.2:
//   * the lower median of |W_t - W_prev| per tensor (Eq. "r_w"), exactly, in ONE pass over the
//     tensor: two order statistics of a sample of 8192 residuals bracket the median between two
//     keys lo <= hi; the streaming pass counts the keys below lo and collects the few per cent of
//     keys inside the bracket; a radix-histogram select (LDS histograms, 11 bits per pass) over those
//     candidates then finds the order statistic.  The bracket can miss (probability about 2e-5 per
//     tensor, or adversarial data); the counts reveal that, and the tensor then takes the
//     always-correct fallback in the same three passes: a radix-histogram select over the whole
//     tensor (11 + 11 + 9 key bits);
//   * the exact sum of |m| per tensor (Eq. "r_o") by integer accumulation: every |m_i| is
//     mant * 2^(pos-149).  The sample fixes a window of 24 bit positions per tensor that holds
//     practically every value; inside it a value is a multiple of one unit below 2^48 units, so a
//     lane adds sixteen of them exactly in fp64, splits the sum into two 32-bit integers and keeps
//     those in 64-bit counters; values outside the window (rare) are filed one by one.  Everything
//     ends in per-tensor u64 bins 8 binary orders apart, so the sum is exact and does not depend on
//     the order of additions;
//   * non-finite detection on W_prev, W_t, m and the residual.
#include "excp_util.h"

#include <algorithm>

namespace {

constexpr u32 MED_SAMPLE = 8192;      // sample size (and the size up to which a tensor is simply sorted)
constexpr u32 MED_HALF_WIDTH = 192;   // bracket = sample ranks 4096 -+ 192 (about 4.2 sigma of the sample rank)
constexpr u32 CAND_STAGE = 2048;       // candidates a wave stages in LDS (it flushes when fewer than 1024 places are left)
constexpr u32 MED_THREADS = 1024;     // workgroup of the bracket kernel: one per tensor, so its own latency is the kernel's

enum { MED_PENDING = 0, MED_KNOWN = 1, MED_FALLBACK = 2 };

// The sample (all residual magnitudes of a tensor that is no larger): sixteen workgroups per tensor, because
// what it costs is the latency of 8192 loads from as many pages, and one compute unit overlaps few of those
// (16.8 M elements: 40 us of loads from one workgroup).
// The first kernel of a call also sets the tensor's state and candidate counters to zero, and where a call is about one tensor
// brings its description along as an argument and leaves it where the others look for it (no copy to wait for).
__global__ __launch_bounds__(EXCP_THREADS) void k_median_sample(Workspace w, GroupParams g, TDesc one, u32 single) {
    constexpr u32 PART = MED_SAMPLE / EXCP_SAMPLE_PARTS, PER = PART / EXCP_THREADS;
    __shared__ u32 s_mmax;
    const u32 t = blockIdx.x / EXCP_SAMPLE_PARTS, part = blockIdx.x % EXCP_SAMPLE_PARTS, tid = threadIdx.x;
    struct { const float *W, *Wp, *m; } D;
    u64 n;
    if (single) { D.W = one.W; D.Wp = one.Wp; D.m = one.m; n = one.n; }
    else { D.W = w.desc[t].W; D.Wp = w.desc[t].Wp; D.m = w.desc[t].m; n = w.desc[t].n; }
    if (part == 0u) {
        u32 *st = (u32 *)&w.st[t], *ctr = w.cand_ctr + (u64)t * 512u;
        for (u32 i = tid; i < sizeof(TState) / 4u; i += EXCP_THREADS) st[i] = 0u;
        for (u32 i = tid; i < 512u; i += EXCP_THREADS) ctr[i] = 0u;
        if (single && tid == 0) { w.desc[0] = one; w.tile_begin[0] = 0u; w.tile_begin[1] = one.tile_count; }
    }
    const u32 ns = n < MED_SAMPLE ? (u32)n : MED_SAMPLE;
    if (part * PART >= ns) return;
    if (tid == 0) s_mmax = 0;
    __syncthreads();
    const u32 wt = excp_wtype(g.flags);
    u32 mmax = 0;                                   // largest finite |m| pattern of the sample
#pragma unroll
    for (u32 q = 0; q < PER; ++q) {
        const u32 i = part * PART + q * EXCP_THREADS + tid;
        if (i < ns) {
            const u64 idx = n <= MED_SAMPLE ? (u64)i : ((u64)i * n) / MED_SAMPLE;
            const float wv = load_weight(D.W, idx, wt);
            w.sample[(u64)t * MED_SAMPLE + i] = f2u((g.flags & 1u) ? wv : wv - load_weight(D.Wp, idx, wt)) & 0x7fffffffu;   // flag: median of |W_t|
            if (q == 0) {                           // (half of them place the window of the exact sum well enough)
                const u32 mb = f2u(D.m[idx]) & 0x7fffffffu;
                if (mb < 0x7f800000u) mmax = max(mmax, mb);
            }
        }
    }
    mmax = wave_max_u32(mmax);
    if ((tid & 63u) == 0) atomicMax(&s_mmax, mmax);
    __syncthreads();
    if (tid == 0) w.sample_mmax[t * EXCP_SAMPLE_PARTS + part] = s_mmax;
}

// One workgroup per tensor: the two order statistics of the sample that bracket the median (the median itself of
// a small tensor), by a radix select over both ranks at once: 11 + 10 + 10 key bits, LDS histograms scanned by
// the whole workgroup.  (A full sort of the sample, 91 barrier rounds, took 58 us; this takes about 8.)
__global__ __launch_bounds__(MED_THREADS) void k_median_bracket(Workspace w, GroupParams g) {
    __shared__ u32 hist[2][2048];
    __shared__ u32 s_wave[MED_THREADS / 64];
    __shared__ u32 s_bin[2], s_rank[2], s_natoms, s_atom[64], s_acnt[64];
    constexpr u32 PER = MED_SAMPLE / MED_THREADS;
    const u32 t = blockIdx.x, tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    const TDesc &D = w.desc[t];
    TState &S = w.st[t];
    const u64 n = D.n;
    if (n == 0) { if (tid == 0) { S.med_bits = 0; S.med_state = MED_KNOWN; } return; }
    const u32 ns = n < MED_SAMPLE ? (u32)n : MED_SAMPLE;
    u32 key[PER];
#pragma unroll
    for (u32 j = 0; j < PER; ++j) {
        const u32 i = j * MED_THREADS + tid;
        key[j] = i < ns ? w.sample[(u64)t * MED_SAMPLE + i] : 0xffffffffu;      // (never a key: those have 31 bits)
    }
    const bool whole = n <= MED_SAMPLE;
    u32 pref[2] = {0u, 0u}, rank[2];
    rank[0] = whole ? (ns - 1u) >> 1 : MED_SAMPLE / 2 - MED_HALF_WIDTH;
    rank[1] = whole ? rank[0] : MED_SAMPLE / 2 + MED_HALF_WIDTH;
#pragma unroll
    for (u32 pass = 0; pass < 3; ++pass) {
        const u32 shift = pass == 0 ? 20u : (pass == 1 ? 10u : 0u), width = pass == 0 ? 11u : 10u;
#pragma unroll
        for (u32 i = tid; i < 2u * 2048u; i += MED_THREADS) (&hist[0][0])[i] = 0;
        __syncthreads();
        const bool apart = pref[0] != pref[1];           // else both ranks are looked for in the first histogram
#pragma unroll
        for (u32 j = 0; j < PER; ++j) {
            const u32 k = key[j], bin = (k >> shift) & ((1u << width) - 1u);
            if (k != 0xffffffffu) {
                const u32 up = pass == 0 ? 0u : k >> (shift + width);
                if (up == pref[0]) atomicAdd(&hist[0][bin], 1u);
                else if (apart && up == pref[1]) atomicAdd(&hist[1][bin], 1u);
            }
        }
        __syncthreads();
        // both histograms scanned together, 16 bits each (at most 8192 keys)
        const u32 *h1 = apart ? hist[1] : hist[0];
        const u32 c0 = hist[0][2u * tid] | (h1[2u * tid] << 16), c1 = hist[0][2u * tid + 1u] | (h1[2u * tid + 1u] << 16);
        u32 incl = wave_incl_scan_u32(c0 + c1);
        if (lane == 63u) s_wave[wave] = incl;
        __syncthreads();
        u32 before = incl - c0 - c1;
        for (u32 q = 0; q < wave; ++q) before += s_wave[q];
#pragma unroll
        for (u32 h = 0; h < 2; ++h) {
            const u32 lo = (before >> (16u * h)) & 0xffffu, n0 = (c0 >> (16u * h)) & 0xffffu, n1 = (c1 >> (16u * h)) & 0xffffu;
            if (rank[h] >= lo && rank[h] < lo + n0 + n1) {            // exactly one thread
                const bool second = rank[h] >= lo + n0;
                s_bin[h] = 2u * tid + (second ? 1u : 0u);
                s_rank[h] = rank[h] - lo - (second ? n0 : 0u);
            }
        }
        __syncthreads();
#pragma unroll
        for (u32 h = 0; h < 2; ++h) { pref[h] = (pref[h] << width) | s_bin[h]; rank[h] = s_rank[h]; }
    }
    const u32 klo = pref[0], khi = pref[1];
    // 16-bit weights: residuals are few distinct values.  Up to four values of the bracket that fill at least 32
    // places of the sample (0.4 % of the tensor) are counted during the streaming pass instead of being listed one
    // by one.  They are found by hashing the bracket's keys: a cell keeps one of its keys and counts that one
    // (a heavy value that loses its cell to another is listed like the rest: slower, no less exact).
    const bool atoms = (g.flags & 0x30u) && !whole && klo != khi;
    if (atoms) {                                         // the same in the whole workgroup
        u32 *rep = hist[0], *cnt = hist[1];
        auto cell = [](u32 k) { return (k * 2654435761u) >> 21; };
        for (u32 i = tid; i < 2048u; i += MED_THREADS) cnt[i] = 0;
        if (tid == 0) s_natoms = 0;
#pragma unroll
        for (u32 j = 0; j < PER; ++j) if (key[j] - klo <= khi - klo) rep[cell(key[j])] = key[j];
        __syncthreads();
#pragma unroll
        for (u32 j = 0; j < PER; ++j) if (key[j] - klo <= khi - klo && rep[cell(key[j])] == key[j]) atomicAdd(&cnt[cell(key[j])], 1u);
        __syncthreads();
        for (u32 i = tid; i < 2048u; i += MED_THREADS) {
            if (cnt[i] >= 32u) {
                const u32 at = atomicAdd(&s_natoms, 1u);
                if (at < 64u) { s_atom[at] = rep[i]; s_acnt[at] = cnt[i]; }
            }
        }
        __syncthreads();
    }
    if (tid == 0) {
        // window of the exact sum: its top sits 4 binary orders above the largest sampled |m|
        u32 mmax = 0;
        for (u32 q = 0; q < (ns + MED_SAMPLE / EXCP_SAMPLE_PARTS - 1u) / (MED_SAMPLE / EXCP_SAMPLE_PARTS); ++q)
            mmax = max(mmax, w.sample_mmax[t * EXCP_SAMPLE_PARTS + q]);
        const u32 e = mmax >> 23;
        const u32 pos = (e ? e : 1u) - 1u;
        S.absm_base = pos + 4u > 23u ? min(pos + 4u - 23u, 230u) : 0u;
        if (whole) {
            S.med_bits = klo;
            S.med_state = MED_KNOWN;
        } else {
            S.br_lo = klo;
            S.br_hi = khi;
            S.med_state = MED_PENDING;
            u32 na = 0;
            if (atoms) {                                 // the four most frequent
                const u32 have = min(s_natoms, 64u);
                for (; na < 4u; ++na) {
                    u32 best = 0;
                    for (u32 i = 1; i < have; ++i) if (s_acnt[i] > s_acnt[best]) best = i;
                    if (best >= have || s_acnt[best] == 0u) break;
                    S.atom_key[na] = s_atom[best];
                    s_acnt[best] = 0;
                }
            }
            S.natoms = na;
        }
    }
}

// Four consecutive floats at an address that is only known to be 4-byte aligned.
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));

// What one workgroup of the streaming pass found out about a tensor whose tiles it shares with other
// workgroups (StatPart in excp_device.h).  A workgroup takes a contiguous range of tiles, so it shares at
// most two tensors: the one its range starts in (record 0) and the one it ends in (record 1).  A tensor that
// lies inside one workgroup's range goes straight into its TState.  The records replace atomics on the
// tensor's state: thousands of waves queued at those few addresses (about 20 ns a turn, whatever the size of
// the tensor), which is what a 16.8 M-element tensor spent 300 of 361 us on.
__device__ __forceinline__ u32 stats_owner(u32 tile, u32 G, u32 ntiles) {      // workgroup whose range holds the tile
    return (u32)((((u64)tile + 1ull) * G + ntiles - 1ull) / ntiles) - 1u;
}
__device__ __forceinline__ u32 stats_lo(u32 b, u32 G, u32 ntiles) { return (u32)(((u64)b * ntiles) / G); }

// The streaming pass: exact sum of |m|, non-finite check, count of keys below the bracket and
// collection of the keys inside it.  Persistent workgroups over contiguous tile ranges; a lane
// takes four consecutive elements of each of four 256-element rows of its wave's quarter tile.
// Bound by memory: 12 bytes per element and nothing written but the candidates.
// W16: the weights are 16-bit (fp16 or bf16 by the flags), four to an 8-byte load where the arrays
// allow it; they are widened on arrival and everything after that is the fp32 code.
template <bool W16>
__global__ __launch_bounds__(EXCP_THREADS) void k_stats_stream(Workspace w, GroupParams g) {
    __shared__ u64 bins[EXCP_ABSM_BINS];
    __shared__ u32 l_cand[4][CAND_STAGE + 1];   // per wave: staged candidates, plus a spare slot
    __shared__ u64 s_L, s_H;
    __shared__ u32 s_nf, s_lt, s_cc, s_atom[4], s_wc[4], s_place;
    const u32 tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    const u32 G = gridDim.x, b = blockIdx.x;
    const u32 lo_tile = stats_lo(b, G, g.ntiles), hi_tile = stats_lo(b + 1u, G, g.ntiles);
    if (lo_tile >= hi_tile) return;
    if (tid < EXCP_ABSM_BINS) bins[tid] = 0;
    if (tid == 0) { s_nf = 0; s_lt = 0; s_cc = 0; s_L = 0; s_H = 0; }
    if (tid < 4) s_atom[tid] = 0;
    __syncthreads();

    // the tensor in hand (all of it the same in every lane), read again only when the tensor changes
    u32 t = 0, t_begin = 0, t_end = 0, B = 0, klo = 0, kspan = 0, natoms = 0, ak[4] = {0u, 0u, 0u, 0u};
    bool pending = false;
    u64 n = 0;
    const float *pW = nullptr, *pP = nullptr, *pM = nullptr;
    auto open_tensor = [&](u32 tile) {
        t = (u32)__builtin_amdgcn_readfirstlane((int)find_owner(w.tile_begin, g.ntensors, tile));
        t_begin = w.tile_begin[t]; t_end = w.tile_begin[t + 1];
        const TDesc &D = w.desc[t];
        const TState &S = w.st[t];
        n = D.n; pW = D.W; pP = D.Wp; pM = D.m;
        B = S.absm_base;               // window of the exact sum = bit positions [B, B + 24)
        pending = S.med_state == MED_PENDING;
        klo = S.br_lo; kspan = S.br_hi - klo;
        if (W16) {
            natoms = S.natoms;
#pragma unroll
            for (int q = 0; q < 4; ++q) ak[q] = S.atom_key[q];
        }
    };
    open_tensor(lo_tile);
    u32 nf = 0, clt = 0, cc = 0;   // clt, cc: the same in every lane of a wave
    u64 accL = 0, accH = 0;        // this lane's in-window units: sum of low / high 32-bit halves
    u32 acnt[4] = {0u, 0u, 0u, 0u};   // W16: elements equal to the tensor's counted bracket values (same in every lane)
    u32 wcount = 0;                // candidates this wave has staged in LDS (same in every lane)
    // Room for `cnt` candidates: one lane asks.  A tensor's list is cut into L lists with a counter each, so that
    // the workgroups do not queue at one address; one that finds its list full moves on to the next, so the lists
    // fail only when all of them are full.  Returns the place in the group's candidate array, 0xffffffff if none.
    // `turn`: what the list to begin with is chosen by.
    auto reserve = [&](u32 cnt, u32 turn) -> u32 {
        const TDesc &D = w.desc[t];
        const u32 L = D.cand_lists, cap = (u32)(D.cand_cap / L);
        u32 *ctr = w.cand_ctr + (u64)t * 512u;
        u32 j = excp_cand_first(turn, L);
        for (u32 attempt = 0; attempt < L; ++attempt, j = (j + 1u == L ? 0u : j + 1u)) {
            const u32 at = atomicAdd(&ctr[j * 32u], cnt);
            if ((u64)at + cnt <= cap) {
                atomicMax(&ctr[j * 32u + 1u], at + cnt);
                return j * cap + at;
            }
        }
        atomicOr(&w.st[t].cand_overflow, 1u);
        return 0xffffffffu;
    };
    auto flush_wave = [&]() {      // a wave's staging area is full: its candidates go to a list
        u32 at = 0;
        if (lane == 0) at = reserve(wcount, b + wave);
        at = __shfl(at, 0, WAVE);
        if (at != 0xffffffffu) {
            EXCP_GLOBAL u32 *dst = gptr(w.cand) + w.desc[t].cand_off + at;
            for (u32 i = lane; i < wcount; i += 64) dst[i] = l_cand[wave][i];
        }
        wcount = 0;
    };
    // the workgroup is done with the tensor in hand (called by all its threads)
    auto flush = [&]() {
        // the lanes' window sums: at positions B (L) and B + 32 (H)
        const u64 sumL = wave_sum_u64(accL), sumH = wave_sum_u64(accH);
        const u32 nfw = wave_sum_u32(nf);
        accL = 0; accH = 0;
        if (lane == 0) {
            atomicAdd(&s_L, sumL); atomicAdd(&s_H, sumH);
            if (clt) atomicAdd(&s_lt, clt);
            if (cc) atomicAdd(&s_cc, cc);
            if (nfw) atomicAdd(&s_nf, nfw);
            if (W16) {
#pragma unroll
                for (int q = 0; q < 4; ++q) if (acnt[q]) atomicAdd(&s_atom[q], acnt[q]);
            }
            s_wc[wave] = wcount;
        }
        nf = 0; clt = 0; cc = 0;
        acnt[0] = acnt[1] = acnt[2] = acnt[3] = 0u;
        __syncthreads();
        const u32 c0 = s_wc[0], c1 = s_wc[1], c2 = s_wc[2], total = c0 + c1 + c2 + s_wc[3];
        if (tid < EXCP_ABSM_BINS) {                       // (values outside the window: rare)
            const u64 c = bins[tid];
            if (c) { atomicAdd(&w.st[t].absm[tid], c); bins[tid] = 0; }
        }
        if (tid == 0) {
            s_place = total ? reserve(total, b) : 0xffffffffu;   // one reservation for the whole workgroup
            StatPart P;
            P.L = s_L; P.H = s_H; P.clt = s_lt; P.nf = s_nf; P.cc = s_cc; P.pad = 0;
#pragma unroll
            for (int q = 0; q < 4; ++q) { P.atom[q] = s_atom[q]; s_atom[q] = 0; }
            s_L = 0; s_H = 0; s_lt = 0; s_nf = 0; s_cc = 0;
            if (t_begin >= lo_tile && t_end <= hi_tile) w.st[t].part = P;      // nobody else holds tiles of it
            else w.stat_part[2u * b + (t_begin <= lo_tile ? 0u : 1u)] = P;
        }
        __syncthreads();
        const u32 at = s_place;
        if (at != 0xffffffffu) {
            const u32 mine = at + (wave > 0u ? c0 : 0u) + (wave > 1u ? c1 : 0u) + (wave > 2u ? c2 : 0u);
            EXCP_GLOBAL u32 *dst = gptr(w.cand) + w.desc[t].cand_off + mine;
            for (u32 i = lane; i < wcount; i += 64) dst[i] = l_cand[wave][i];
        }
        wcount = 0;
        __syncthreads();
    };

    for (u32 tile = lo_tile; tile < hi_tile; ++tile) {
        if (tile >= t_end) {
            flush();
            open_tensor(tile);
        }
        const u64 base = (u64)(tile - t_begin) * EXCP_TILE;
        const u32 rem = (n - base < (u64)EXCP_TILE) ? (u32)(n - base) : EXCP_TILE;

        u32 key[16], mb[16];
        u32 worst = 0;             // largest magnitude pattern seen: >= 0x7f800000 means Inf or NaN
        const bool of_weights = (g.flags & 1u) != 0;       // the median is that of |W_t|, not of the residual
        {
            const EXCP_GLOBAL float *gW = gptr(pW) + base, *gP = gptr(pP) + base, *gM = gptr(pM) + base;
            const u32 wt = W16 ? excp_wtype(g.flags) : 0u;
            const bool bf = wt == 2u;
            const EXCP_GLOBAL unsigned short *hW = gptr((const unsigned short *)pW) + base;
            const EXCP_GLOBAL unsigned short *hP = gptr((const unsigned short *)pP) + base;
            const bool vec16 = W16 && (((uintptr_t)pW | (uintptr_t)pP) & 7u) == 0u;   // 8-byte loads need 8-byte alignment
            if (rem == EXCP_TILE && (!W16 || vec16)) {
                f4u a[4], p[4], mm[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const u32 off = wave * 1024u + (u32)k * 256u + lane * 4u;
                    if (W16) {
                        const us4 ha = __builtin_nontemporal_load((const EXCP_GLOBAL us4 *)(hW + off));
                        const us4 hp = __builtin_nontemporal_load((const EXCP_GLOBAL us4 *)(hP + off));
#pragma unroll
                        for (int j = 0; j < 4; ++j) { a[k][j] = w16_widen(ha[j], bf); p[k][j] = w16_widen(hp[j], bf); }
                    } else {
                        a[k] = __builtin_nontemporal_load((const EXCP_GLOBAL f4u *)(gW + off));
                        p[k] = __builtin_nontemporal_load((const EXCP_GLOBAL f4u *)(gP + off));
                    }
                    mm[k] = __builtin_nontemporal_load((const EXCP_GLOBAL f4u *)(gM + off));
                }
#pragma unroll
                for (int k = 0; k < 4; ++k) {
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const float av = a[k][j], pv = p[k][j];
                        const u32 dk = f2u(av - pv) & 0x7fffffffu, wk = f2u(av) & 0x7fffffffu;
                        key[4 * k + j] = of_weights ? wk : dk;
                        mb[4 * k + j] = f2u(mm[k][j]) & 0x7fffffffu;
                        worst = max(max(worst, dk), max(mb[4 * k + j], max(wk, f2u(pv) & 0x7fffffffu)));
                    }
                }
            } else {
#pragma unroll
                for (int j = 0; j < 16; ++j) {
                    const u32 off = wave * 1024u + (u32)(j >> 2) * 256u + lane * 4u + (u32)(j & 3);
                    const bool ok = off < rem;
                    float av = 0.f, pv = 0.f;
                    if (ok) {
                        av = W16 ? w16_widen(hW[off], bf) : gW[off];
                        pv = W16 ? w16_widen(hP[off], bf) : gP[off];
                    }
                    const float mv = ok ? gM[off] : 0.f;
                    const u32 dk = f2u(av - pv) & 0x7fffffffu, wk = f2u(av) & 0x7fffffffu;
                    mb[j] = f2u(mv) & 0x7fffffffu;
                    worst = max(max(worst, dk), max(mb[j], max(wk, f2u(pv) & 0x7fffffffu)));
                    key[j] = ok ? (of_weights ? wk : dk) : 0xffffffffu;      // above every bracket, never a candidate
                }
            }
        }
        if (__any(worst >= 0x7f800000u)) {
            // rare: something is not finite; it is reported and keeps out of the sum
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                if (key[j] != 0xffffffffu && (key[j] & 0x7f800000u) == 0x7f800000u) nf += 1;
                if ((mb[j] & 0x7f800000u) == 0x7f800000u) { nf += 1; mb[j] = 0; }
            }
            if (nf == 0 && worst >= 0x7f800000u) nf = 1;
        }
        if (pending && kspan == 0u) {
            // a bracket of one value (heavily tied data, e.g. 16-bit weights that did not move): its number is
            // all that is needed
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                clt += __popcll(ballot64(key[j] < klo));
                cc += __popcll(ballot64(key[j] == klo));
            }
        } else if (pending) {
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                clt += __popcll(ballot64(key[j] < klo));
                bool cand = key[j] - klo <= kspan;            // klo <= key <= khi (a padded key wraps far above)
                if (W16 && natoms) {
                    const bool e0 = key[j] == ak[0], e1 = natoms > 1u && key[j] == ak[1];
                    const bool e2 = natoms > 2u && key[j] == ak[2], e3 = natoms > 3u && key[j] == ak[3];
                    acnt[0] += __popcll(ballot64(e0)); acnt[1] += __popcll(ballot64(e1));
                    acnt[2] += __popcll(ballot64(e2)); acnt[3] += __popcll(ballot64(e3));
                    cand = cand && !(e0 || e1 || e2 || e3);
                }
                const u64 bal = ballot64(cand);
                // branch-free: the others write to a spare slot past the end
                l_cand[wave][cand ? wcount + lanes_below(bal) : CAND_STAGE] = key[j];
                wcount += __popcll(bal);
            }
            if (wcount > CAND_STAGE - 1024u) flush_wave();    // room for another 1024 is kept
        }
        {
            // exact sum of |m|: in-window values are whole multiples of 2^(B-149) below 2^48 units,
            // so this lane's sixteen add exactly in fp64.
            const u32 thr_lo = B ? ((B + 1u) << 23) : 0u, span = ((B + 25u) << 23) - thr_lo;
            double dsum = 0.0;
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                const bool in = mb[j] - thr_lo < span;
                dsum += in ? (double)u2f(mb[j]) : 0.0;
                if (!in && mb[j]) {
                    const u32 e = mb[j] >> 23;
                    const u32 mant = (mb[j] & 0x7fffffu) | (e ? 0x800000u : 0u);
                    const u32 pos = (e ? e : 1u) - 1u;
                    atomicAdd(&bins[pos >> 3], (u64)mant << (pos & 7u));
                }
            }
            const double units = ldexp(dsum, 149 - (int)B);                // an integer below 2^52
            const u32 hi32 = (u32)(units * 2.3283064365386963e-10);     // floor(units / 2^32)
            const u32 lo32 = (u32)(units - (double)hi32 * 4294967296.0);
            accL += lo32;
            accH += hi32;
        }
    }
    flush();
}

// After the streaming pass, one workgroup per tensor: the workgroups' records are added up; the exact sum of
// |m| becomes the second threshold; and the bracket is checked: does it hold the median?  If so the select goes
// on inside the candidates (base key, number of undecided low bits, rank); if not the tensor falls back.
// `G` = workgroups of the streaming pass.
__global__ __launch_bounds__(EXCP_THREADS) void k_stats_finish(Workspace w, GroupParams g, u32 G) {
    __shared__ u64 bins[EXCP_ABSM_BINS];
    __shared__ u64 s_u64[3];
    __shared__ u32 s_u32[7];
    const u32 t = blockIdx.x, tid = threadIdx.x, lane = tid & 63u;
    TState &S = w.st[t];
    const TDesc &D = w.desc[t];
    const u64 n = D.n;
    if (n == 0) {
        if (tid == 0) { S.med_bits = 0; S.mean32 = 0.f; S.t_w = 0.f; S.r_o = 0.f; S.abs_sum = 0.0; }
        return;
    }
    if (tid < 3) s_u64[tid] = 0;
    if (tid < 7) s_u32[tid] = 0;
    if (tid < EXCP_ABSM_BINS) bins[tid] = S.absm[tid];
    __syncthreads();
    if (tid < D.cand_lists) atomicAdd(&s_u32[6], w.cand_ctr[(u64)t * 512u + tid * 32u + 1u]);      // listed candidates
    u64 L = 0, H = 0, nf = 0;
    u32 clt = 0, cc = 0, atom[4] = {0u, 0u, 0u, 0u};
    auto take = [&](const StatPart &P) {
        L += P.L; H += P.H; nf += P.nf; clt += P.clt; cc += P.cc;
#pragma unroll
        for (int q = 0; q < 4; ++q) atom[q] += P.atom[q];
    };
    const u32 tb = D.tile_begin, te = tb + D.tile_count;
    const u32 b0 = stats_owner(tb, G, g.ntiles), b1 = stats_owner(te - 1u, G, g.ntiles);
    if (b0 == b1) {
        if (tid == 0) take(S.part);
    } else {
        const u32 slot0 = tb <= stats_lo(b0, G, g.ntiles) ? 0u : 1u;       // (the others start inside the tensor)
        for (u32 b = b0 + tid; b <= b1; b += EXCP_THREADS)
            if (g.ntiles >= G || stats_lo(b, G, g.ntiles) < stats_lo(b + 1u, G, g.ntiles)) take(w.stat_part[2u * b + (b == b0 ? slot0 : 0u)]);
    }
    L = wave_sum_u64(L); H = wave_sum_u64(H); nf = wave_sum_u64(nf);
    clt = wave_sum_u32(clt); cc = wave_sum_u32(cc);
#pragma unroll
    for (int q = 0; q < 4; ++q) atom[q] = wave_sum_u32(atom[q]);
    if (lane == 0) {
        atomicAdd(&s_u64[0], L); atomicAdd(&s_u64[1], H); atomicAdd(&s_u64[2], nf);
        atomicAdd(&s_u32[0], clt); atomicAdd(&s_u32[1], cc);
#pragma unroll
        for (int q = 0; q < 4; ++q) atomicAdd(&s_u32[2 + q], atom[q]);
    }
    __syncthreads();
    if (tid != 0) return;
    L = s_u64[0]; H = s_u64[1];
    S.nonfinite += s_u64[2];
    {
        const u32 B = S.absm_base;
        const u64 lo64 = L + (H << 32), hi64 = (H >> 32) + (lo64 < L ? 1ull : 0ull);
        const u64 piece[3] = {lo64 & 0xffffffffull, lo64 >> 32, hi64};
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            const u32 p = B + 32u * (u32)q;
            if (piece[q]) bins[p >> 3] += piece[q] << (p & 7u);
        }
        const double sum = signed_bins_to_double(bins);
        const float mean32 = (float)(sum / (double)n);
        S.abs_sum = sum;
        S.mean32 = mean32;
        S.r_o = __fmul_rn(g.beta, mean32);
    }
    if (S.med_state == MED_PENDING) {
        const u64 r = (n - 1) >> 1;
        const u64 below = s_u32[0];
        S.c_lt = (u32)below;
        if (S.br_hi == S.br_lo) {              // one-value bracket: only counted, never listed
            const u64 cnt = s_u32[1];
            S.cand_count = (u32)cnt;
            if (r >= below && r < below + cnt) { S.med_bits = S.br_lo; S.med_state = MED_KNOWN; }
            else S.med_state = MED_FALLBACK;
        } else {
            const u64 cnt = s_u32[6];
            u64 counted = 0;                   // bracket values that were counted instead of listed
            S.cand_count = (u32)cnt;
#pragma unroll
            for (u32 q = 0; q < 4; ++q) { S.atom_cnt[q] = s_u32[2 + q]; if (q < S.natoms) counted += s_u32[2 + q]; }
            if (S.cand_overflow || r < below || r >= below + cnt + counted) {
                S.med_state = MED_FALLBACK;
            } else {
                S.sel_base = S.br_lo;
                S.sel_width = 32u - (u32)__clz((int)(S.br_hi - S.br_lo));
                S.sel_rank = (u32)(r - below);
            }
        }
    }
    S.t_w = __fmul_rn(g.alpha, u2f(S.med_bits));          // (final where the median is known by now)
}

// The exact median: three radix passes, each one launch for all tensors.  A tensor whose bracket held takes its
// candidates through the top (up to 11) undecided bits of the bracket's span per pass; one whose bracket
// missed takes all its keys through 11 + 11 + 9 key bits.  A workgroup does the share that belongs to
// SEL_TILES consecutive tiles of the group's tile list, tensor by tensor, and the last of a tensor's workgroups
// to finish resolves the pass: its counts are complete then, so no second launch is needed (this and one path for
// both kinds of tensor replace twelve launches by three).
// SEL_TILES: about 512 workgroups, with 32 tiles at least (fewer would leave a workgroup a few hundred candidates) and
// 256 at most (a workgroup's histogram goes to memory with up to 2048 atomics).
static u32 sel_tiles(u32 ntiles) { return std::min(std::max(ntiles / 512u, 32u), 256u); }

__global__ __launch_bounds__(EXCP_THREADS) void k_median_select(Workspace w, GroupParams g, u32 pass, u32 SEL_TILES) {
    __shared__ u32 s_tiles[EXCP_MAX_GROUP_TENSORS + 1];
    __shared__ u32 hist[2048];
    __shared__ u32 s_wave[EXCP_THREADS / 64], s_ticket, s_state[EXCP_THREADS];
    const u32 tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    const u32 lo = blockIdx.x * SEL_TILES, hi = min(lo + SEL_TILES, g.ntiles);
    for (u32 i = tid; i < 2048; i += EXCP_THREADS) hist[i] = 0;
    load_tile_table(s_tiles, w.tile_begin, g.ntensors);
    u32 t = find_owner(s_tiles, g.ntensors, lo);
    const u32 t0 = t;                                     // the states of the first 256 tensors, read side by side
    if (t0 + tid < g.ntensors) s_state[tid] = w.st[t0 + tid].med_state;
    __syncthreads();
    for (u32 a0 = lo; a0 < hi; ++t) {
        const u32 tb = s_tiles[t], te = s_tiles[t + 1];
        const u32 a1 = min(te, hi);                       // this workgroup's tiles of tensor t: [a0, a1)
        const u32 b0 = a0;
        a0 = a1;
        if (a1 <= b0) continue;
        TState &S = w.st[t];
        const u32 state = t - t0 < EXCP_THREADS ? s_state[t - t0] : S.med_state;
        if (state == MED_KNOWN) continue;                 // the same for the whole workgroup
        const TDesc &D = w.desc[t];
        const u32 base = S.sel_base, rank = S.sel_rank;
        const u32 cwidth = S.sel_width, cshift = cwidth > 11u ? cwidth - 11u : 0u;     // candidates
        const u32 fshift = pass == 0u ? 20u : (pass == 1u ? 9u : 0u);                  // all keys
        if (state == MED_PENDING) {
            const u64 limit = 1ull << cwidth;
            const u32 tc = te - tb;
            const u32 L = D.cand_lists, cap = (u32)(D.cand_cap / L);
            const u32 *ctr = w.cand_ctr + (u64)t * 512u;
            // the workgroup's share of every list; a wave takes every fourth list
            for (u32 j = L >= 4u ? wave : 0u; j < L; j += L >= 4u ? 4u : 1u) {
                const u32 cnt = ctr[j * 32u + 1u];
                const u32 i0 = (u32)(((u64)cnt * (b0 - tb)) / tc), i1 = (u32)(((u64)cnt * (a1 - tb)) / tc);
                const EXCP_GLOBAL u32 *c = gptr(w.cand) + D.cand_off + (u64)j * cap;
                const u32 first = L >= 4u ? lane : tid, step = L >= 4u ? 64u : EXCP_THREADS;
                for (u32 i = i0 + first; i < i1; i += 8u * step) {
                    u32 k[8];
#pragma unroll
                    for (u32 q = 0; q < 8; ++q) k[q] = i + q * step < i1 ? c[i + q * step] : base - 1u;
#pragma unroll
                    for (u32 q = 0; q < 8; ++q) {
                        const u32 rel = k[q] - base;      // keys below base wrap around and drop out
                        if ((u64)rel < limit) atomicAdd(&hist[rel >> cshift], 1u);
                    }
                }
            }
        } else {
            const u64 n = D.n;
            const u32 wt = excp_wtype(g.flags);
            const bool of_weights = (g.flags & 1u) != 0u;
            for (u32 tile = b0; tile < a1; ++tile) {
                const u64 first = (u64)(tile - tb) * EXCP_TILE;
                const u32 rem = (n - first < (u64)EXCP_TILE) ? (u32)(n - first) : EXCP_TILE;
                // (this path is taken for heavily tied data above all: see hist_add_tied)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const u32 off = wave * 1024u + (u32)q * 256u + lane * 4u;
                    float a[4], pv[4] = {0.f, 0.f, 0.f, 0.f};
                    load_weights4(D.W, first, off, rem, wt, a);
                    if (!of_weights) load_weights4(D.Wp, first, off, rem, wt, pv);
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const u32 k = f2u(a[j] - pv[j]) & 0x7fffffffu;
                        const bool act = off + (u32)j < rem && (pass == 0u || (k >> (pass == 1u ? 20u : 9u)) == base);
                        hist_add_tied(hist, (k >> fshift) & (pass == 2u ? 511u : 2047u), act);
                    }
                }
            }
        }
        __syncthreads();
        u32 *H = w.med_hist + (u64)t * 2048u;
        for (u32 i = tid; i < 2048; i += EXCP_THREADS) {
            const u32 v = hist[i];
            if (v) { atomicAdd(&H[i], v); hist[i] = 0; }
        }
        // The last of the tensor's workgroups sees everybody's counts: they are only ever touched by device-scope
        // atomics, which are done (vmcnt) before the ticket is drawn.  (A __threadfence here would write back the
        // whole L2 for every workgroup: 302 us a pass instead of 53 for 1.07e9 elements with 64 tiles to a workgroup.)
        const u32 parts = (te - 1u) / SEL_TILES - tb / SEL_TILES + 1u;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (tid == 0) s_ticket = parts == 1u ? 0u : atomicAdd(&w.sel_ticket[t], 1u);
        __syncthreads();
        if (s_ticket != parts - 1u) continue;
        u32 c[8], local = 0;
#pragma unroll
        for (int i = 0; i < 8; ++i) c[i] = __hip_atomic_load(&H[tid * 8 + i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (state == MED_PENDING) {
            // the counted bracket values join the listed candidates, each with its multiplicity
            for (u32 q = 0; q < S.natoms; ++q) {
                const u32 rel = S.atom_key[q] - base, bin = rel >> cshift;
#pragma unroll
                for (int i = 0; i < 8; ++i) if ((u64)rel < (1ull << cwidth) && bin == tid * 8u + (u32)i) c[i] += S.atom_cnt[q];
            }
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) { local += c[i]; H[tid * 8 + i] = 0; }
        u32 incl = wave_incl_scan_u32(local);
        if (lane == 63u) s_wave[wave] = incl;
        if (tid == 0) w.sel_ticket[t] = 0;
        __syncthreads();
        u32 before = incl - local;
        for (u32 q = 0; q < wave; ++q) before += s_wave[q];
        const u32 want = (state == MED_FALLBACK && pass == 0u) ? (u32)((D.n - 1ull) >> 1) : rank;
        if (want >= before && want < before + local) {            // exactly one thread
            u32 r = want - before;
            u32 i = 0;
#pragma unroll
            for (u32 q = 0; q < 7; ++q) if (i == q && r >= c[q]) { r -= c[q]; ++i; }
            const u32 bin = tid * 8u + i;
            u32 nb;
            bool done;
            if (state == MED_PENDING) {
                nb = base + (bin << cshift);
                done = cshift == 0u;
                S.sel_width = cshift;
            } else {
                nb = pass == 0u ? bin : (base << (pass == 2u ? 9u : 11u)) | bin;
                done = pass == 2u;
            }
            S.sel_base = nb;
            S.sel_rank = r;
            if (done) { S.med_bits = nb; S.med_state = MED_KNOWN; S.t_w = __fmul_rn(g.alpha, u2f(nb)); }
        }
        __syncthreads();
    }
}

__global__ void k_zero_u32(u32 *p, u64 count) {
    u64 i = (u64)blockIdx.x * blockDim.x + threadIdx.x;
    u64 stride = (u64)gridDim.x * blockDim.x;
    for (; i < count; i += stride) p[i] = 0u;
}

// Plain streaming copy of 16-byte words: a kernel whose HBM traffic is known exactly (bytes read =
// bytes written = the size), used to calibrate the profiler's byte counters.
__global__ __launch_bounds__(256) void k_copy_probe(const uint4 *__restrict__ src, uint4 *__restrict__ dst, u64 count) {
    u64 i = (u64)blockIdx.x * blockDim.x + threadIdx.x;
    const u64 stride = (u64)gridDim.x * blockDim.x;
    for (; i < count; i += stride) dst[i] = src[i];
}

}  // namespace

void launch_copy_probe(const void *src, void *dst, u64 bytes, hipStream_t s) {
    const u64 count = bytes / 16;
    if (!count) return;
    hipLaunchKernelGGL(k_copy_probe, dim3(8192), dim3(256), 0, s, (const uint4 *)src, (uint4 *)dst, count);
}

void launch_zero_u32(u32 *p, u64 count, hipStream_t s) {
    if (!count) return;
    u64 blocks = (count + 1023) / 1024;
    if (blocks > 2048) blocks = 2048;
    hipLaunchKernelGGL(k_zero_u32, dim3((u32)blocks), dim3(256), 0, s, p, count);
}

// phase 0: sample and bracket (`single`: the description of a call's only tensor, not in the tables yet), 1: streaming pass, 2: its records added up, bracket check, thresholds, and the
// passes that find the median
void launch_stats(const Workspace &w, const GroupParams &g, int phase, const TDesc *single, hipStream_t s) {
    if (!g.ntensors) return;
    const dim3 block(EXCP_THREADS);
    const dim3 stream_grid(excp_stats_grid(g.ntiles, g.largest, (u32)w.cus));
    switch (phase) {
        case 0:
            hipLaunchKernelGGL(k_median_sample, dim3(g.ntensors * EXCP_SAMPLE_PARTS), block, 0, s, w, g, single ? *single : TDesc{}, single ? 1u : 0u);
            hipLaunchKernelGGL(k_median_bracket, dim3(g.ntensors), dim3(MED_THREADS), 0, s, w, g);
            break;
        case 1:
            if (!g.ntiles) break;
            if (g.flags & 0x30u) hipLaunchKernelGGL(k_stats_stream<true>, stream_grid, block, 0, s, w, g);
            else hipLaunchKernelGGL(k_stats_stream<false>, stream_grid, block, 0, s, w, g);
            break;
        default:
            hipLaunchKernelGGL(k_stats_finish, dim3(g.ntensors), block, 0, s, w, g, stream_grid.x);
            if (!g.ntiles) break;
            for (u32 pass = 0; pass < 3u; ++pass)
                hipLaunchKernelGGL(k_median_select, dim3((g.ntiles + sel_tiles(g.ntiles) - 1u) / sel_tiles(g.ntiles)), block, 0, s, w, g, pass, sel_tiles(g.ntiles));
            break;
    }
}

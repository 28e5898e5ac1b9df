// Small device helpers shared by the ExCP kernels (wave64, gfx950).
#pragma once
#include "excp_device.h"

#define WAVE 64

__device__ __forceinline__ u32 f2u(float x) { return __float_as_uint(x); }
__device__ __forceinline__ float u2f(u32 x) { return __uint_as_float(x); }

__device__ __forceinline__ u64 ballot64(bool p) { return __builtin_amdgcn_ballot_w64(p); }
__device__ __forceinline__ u32 lane_id() { return threadIdx.x & 63u; }
// number of set bits of a wave-wide mask that belong to lanes below the calling one
__device__ __forceinline__ u32 lanes_below(unsigned long long m) {
    return __builtin_amdgcn_mbcnt_hi((u32)(m >> 32), __builtin_amdgcn_mbcnt_lo((u32)m, 0u));
}

__device__ __forceinline__ u64 shfl_xor_u64(u64 v, int m) {
    u32 lo = (u32)v, hi = (u32)(v >> 32);
    lo = __shfl_xor(lo, m, WAVE);
    hi = __shfl_xor(hi, m, WAVE);
    return ((u64)hi << 32) | lo;
}
// Sums, extremes and scans over a wave, by moves between registers: four shifts within rows of sixteen lanes, then
// a row's last lane into the rows above it.  (A shuffle is a trip through LDS, and six of them in a row are most of
// what a small reduction costs: the statistics pass over bf16 weights, which adds up its counters where candidates
// are listed, 754 -> 529 us for a 410M-shaped checkpoint.)  Every lane of the wave must be active; a reduction's result is in all lanes.
// FOLD(v, x): v joined with x; NEUTRAL: the bits that change nothing, where a lane has no partner.
template <int CTRL, int ROWS>
__device__ __forceinline__ u32 dpp_u32(u32 neutral, u32 v) { return (u32)__builtin_amdgcn_update_dpp((int)neutral, (int)v, CTRL, ROWS, 0xf, false); }
template <int CTRL, int ROWS>
__device__ __forceinline__ u64 dpp_u64(u64 v) { return (u64)dpp_u32<CTRL, ROWS>(0u, (u32)(v >> 32)) << 32 | dpp_u32<CTRL, ROWS>(0u, (u32)v); }
// the value of the lane above (the last lane: `v` itself), and of the lane below (the first: itself)
__device__ __forceinline__ u32 lane_above_u32(u32 v) { return dpp_u32<0x130, 0xf>(v, v); }
__device__ __forceinline__ u32 lane_below_u32(u32 v) { return dpp_u32<0x138, 0xf>(v, v); }
__device__ __forceinline__ float lane_above_f32(float v) { return u2f(lane_above_u32(f2u(v))); }
__device__ __forceinline__ float lane_below_f32(float v) { return u2f(lane_below_u32(f2u(v))); }
__device__ __forceinline__ __int128 lane_above_i128(__int128 v) {
    const unsigned __int128 x = (unsigned __int128)v;
    unsigned __int128 r = 0;
#pragma unroll
    for (int q = 3; q >= 0; --q) r = r << 32 | lane_above_u32((u32)(x >> (32 * q)));
    return (__int128)r;
}
#define EXCP_WAVE_SCAN(v, FOLD, MOVE)                                                                        \
    do {                                                                                                     \
        FOLD(v, MOVE(0x111, 0xf)); FOLD(v, MOVE(0x112, 0xf)); FOLD(v, MOVE(0x114, 0xf)); FOLD(v, MOVE(0x118, 0xf));   /* row_shr 1, 2, 4, 8 */ \
        FOLD(v, MOVE(0x142, 0xa)); FOLD(v, MOVE(0x143, 0xc));           /* row_bcast 15 into rows 1 and 3, 31 into rows 2 and 3 */            \
    } while (0)
#define EXCP_FOLD_ADD(v, x) (v += (x))
#define EXCP_FOLD_MAX(v, x) (v = max(v, (x)))
#define EXCP_FOLD_MIN(v, x) (v = min(v, (x)))
__device__ __forceinline__ u32 last_lane_u32(u32 v) { return (u32)__builtin_amdgcn_readlane((int)v, 63); }
__device__ __forceinline__ u64 last_lane_u64(u64 v) { return (u64)last_lane_u32((u32)(v >> 32)) << 32 | last_lane_u32((u32)v); }
// inclusive sum over the lanes up to the calling one
__device__ __forceinline__ u32 wave_incl_scan_u32(u32 v) {
#define EXCP_MOVE(CTRL, ROWS) dpp_u32<CTRL, ROWS>(0u, v)
    EXCP_WAVE_SCAN(v, EXCP_FOLD_ADD, EXCP_MOVE);
    return v;
}
__device__ __forceinline__ u32 wave_sum_u32(u32 v) { return last_lane_u32(wave_incl_scan_u32(v)); }
__device__ __forceinline__ u32 wave_max_u32(u32 v) { EXCP_WAVE_SCAN(v, EXCP_FOLD_MAX, EXCP_MOVE); return last_lane_u32(v); }
#undef EXCP_MOVE
__device__ __forceinline__ u32 wave_min_u32(u32 v) {
#define EXCP_MOVE(CTRL, ROWS) dpp_u32<CTRL, ROWS>(0xffffffffu, v)
    EXCP_WAVE_SCAN(v, EXCP_FOLD_MIN, EXCP_MOVE);
#undef EXCP_MOVE
    return last_lane_u32(v);
}
__device__ __forceinline__ u64 wave_incl_scan_u64(u64 v) {
#define EXCP_MOVE(CTRL, ROWS) dpp_u64<CTRL, ROWS>(v)
    EXCP_WAVE_SCAN(v, EXCP_FOLD_ADD, EXCP_MOVE);
#undef EXCP_MOVE
    return v;
}
__device__ __forceinline__ u64 wave_sum_u64(u64 v) { return last_lane_u64(wave_incl_scan_u64(v)); }
__device__ __forceinline__ double wave_sum_f64(double v) {
#define EXCP_MOVE(CTRL, ROWS) __longlong_as_double((long long)dpp_u64<CTRL, ROWS>((u64)__double_as_longlong(v)))
    EXCP_WAVE_SCAN(v, EXCP_FOLD_ADD, EXCP_MOVE);
#undef EXCP_MOVE
    return __longlong_as_double((long long)last_lane_u64((u64)__double_as_longlong(v)));
}
// LDS that only the calling wave uses: what it wrote before is what its lanes read after.
__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
__device__ __forceinline__ double shfl_xor_f64(double v, int m) {
    return __longlong_as_double((long long)shfl_xor_u64((u64)__double_as_longlong(v), m));
}

// Histogram increment in LDS for data that may be heavily tied (then most lanes of a wave hit the same
// bin, and plain atomics take turns): up to two groups of lanes that share a bin are added by one lane
// each, whoever is left adds for itself.  Every lane of the wave must call it.
__device__ __forceinline__ void hist_add_tied(u32 *hist, u32 bin, bool active) {
    u64 todo = ballot64(active);
#pragma unroll
    for (int round = 0; round < 2; ++round) {
        if (todo == 0ull) break;                            // the same in every lane
        const u32 leader = (u32)__ffsll((long long)todo) - 1u;
        const u32 lb = (u32)__shfl((int)bin, (int)leader, WAVE);
        const u64 same = ballot64(active && bin == lb) & todo;
        if (lane_id() == leader) atomicAdd(&hist[lb], (u32)__popcll(same));
        todo &= ~same;
    }
    if ((todo >> lane_id()) & 1ull) atomicAdd(&hist[bin], 1u);
}

// Largest t with begin[t] <= x (begin is non-decreasing, begin[0] == 0, count+1 entries,
// begin[count] > x).  Entries may repeat (empty items); the item found is never empty.
__device__ __forceinline__ u32 find_owner(const u32 *__restrict__ begin, u32 count, u32 x) {
    u32 lo = 0, hi = count;          // invariant: begin[lo] <= x < begin[hi]
    while (hi - lo > 1) {
        u32 mid = (lo + hi) >> 1;
        if (begin[mid] <= x) lo = mid; else hi = mid;
    }
    return lo;
}

// Pointers read from descriptor tables are generic to the compiler; these casts state that they
// point to global memory, which turns flat loads/stores into global ones with immediate offsets.
#define EXCP_GLOBAL __attribute__((address_space(1)))
#define EXCP_CONSTANT __attribute__((address_space(4)))      // global memory that the kernel at hand only reads
template <class T>
__device__ __forceinline__ const EXCP_GLOBAL T *gptr(const T *p) { return (const EXCP_GLOBAL T *)(uintptr_t)p; }
template <class T>
__device__ __forceinline__ EXCP_GLOBAL T *gptr(T *p) { return (EXCP_GLOBAL T *)(uintptr_t)p; }

// Weights stored in 16 bits (flags bits 4-5 of a compress call or a blob header: 1 = IEEE binary16,
// 2 = bfloat16).  Widening is exact; narrowing rounds to nearest even (a finite fp32 beyond the
// format's range becomes infinity, as IEEE conversion does).  All arithmetic stays fp32.
__device__ __forceinline__ u32 excp_wtype(u32 flags) { return (flags >> 4) & 3u; }
__device__ __forceinline__ float w16_widen(u32 h, bool bf) {
    const float half = (float)__builtin_bit_cast(_Float16, (unsigned short)h);
    return bf ? u2f(h << 16) : half;
}
__device__ __forceinline__ u32 w16_narrow(float x, bool bf) {
    const u32 b = f2u(x);
    const u32 bf_bits = (b + 0x7fffu + ((b >> 16) & 1u)) >> 16;       // never a NaN here: inputs are finite
    const u32 half_bits = (u32)__builtin_bit_cast(unsigned short, (_Float16)x);
    return bf ? bf_bits : half_bits;
}
typedef unsigned short us4 __attribute__((ext_vector_type(4), aligned(8)));
// One weight at index idx of an array whose element type is given by wt (0 = fp32).
__device__ __forceinline__ float load_weight(const float *p, u64 idx, u32 wt) {
    if (wt == 0u) return p[idx];
    return w16_widen(((const unsigned short *)p)[idx], wt == 2u);
}
__device__ __forceinline__ void store_weight(float *p, u64 idx, u32 wt, float x) {
    if (wt == 0u) p[idx] = x;
    else ((unsigned short *)p)[idx] = (unsigned short)w16_narrow(x, wt == 2u);
}

// Which decoder takes a blob: 1 = codes and fp32 weights, 2 = codes and 16-bit weights, 4 = written
// without quantisation (either weight storage).
__device__ __forceinline__ u32 blob_kind(u32 nbits, u32 flags) {
    return nbits == EXCP_RAW_BITS ? 4u : (excp_wtype(flags) != 0u ? 2u : 1u);
}

// Four consecutive weights of a tile: elements [off, off + 4) of the tile that starts at `tile0` (an
// element pointer into an array of type wt), of which `rem` exist; one 16-byte (fp32) or 8-byte
// (16-bit, if the array is 8-byte aligned) load where all four exist, else one by one; missing ones are 0.
typedef float f4w __attribute__((ext_vector_type(4), aligned(4)));
__device__ __forceinline__ void load_weights4(const float *arr, u64 tile0, u32 off, u32 rem, u32 wt, float (&out)[4]) {
    if (off + 4u <= rem && wt == 0u) {
        const f4w q = *(const EXCP_GLOBAL f4w *)(gptr(arr) + tile0 + off);
        out[0] = q.x; out[1] = q.y; out[2] = q.z; out[3] = q.w;
    } else if (off + 4u <= rem && ((uintptr_t)arr & 7u) == 0u) {
        const us4 q = *(const EXCP_GLOBAL us4 *)(gptr((const unsigned short *)arr) + tile0 + off);
#pragma unroll
        for (int j = 0; j < 4; ++j) out[j] = w16_widen(q[j], wt == 2u);
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) out[j] = (off + (u32)j < rem) ? load_weight(arr, tile0 + off + (u32)j, wt) : 0.f;
    }
}

// Copy of a tile table in LDS (the per-tile owner search then costs no global round trips).
#define EXCP_MAX_GROUP_TENSORS 1024
__device__ __forceinline__ void load_tile_table(u32 *dst, const u32 *__restrict__ src, u32 count) {
    for (u32 i = threadIdx.x; i <= count; i += blockDim.x) dst[i] = src[i];
    __syncthreads();
}

// ---- value -> bucket map of the codebook stage (built by k_km_sample)
constexpr u32 HALF_CELLS = EXCP_KM_CELLS / 2;

// Value -> cell, monotone in the value: negative values fill cells 2047 down to 0 as their
// magnitude grows, positive ones 2048 up to 4095.  map[0..3] = offset and shift of the negative
// side, offset and shift of the positive side; magnitudes beyond the sampled range clamp.
__device__ __forceinline__ u32 cell_of(float x, const u32 *map) {
    const u32 bits = f2u(x), a = bits & 0x7fffffffu;
    const bool neg = bits >> 31;
    const u32 amin = neg ? map[0] : map[2], sh = neg ? map[1] : map[3];
    const u32 c = min((max(a, amin) - amin) >> sh, HALF_CELLS - 1u);
    return neg ? (c ^ (HALF_CELLS - 1u)) : (c | HALF_CELLS);
}

// Order-preserving map of fp32 bit patterns to unsigned keys (and back).
__device__ __forceinline__ u32 key_of(float x) {
    u32 u = f2u(x);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float val_of(u32 k) {
    return u2f((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k);
}

// Position of a magnitude's lowest mantissa bit: value = mantissa * 2^(pos - 149).
__device__ __forceinline__ u32 bit_pos(u32 mag) { const u32 e = mag >> 23; return (e ? e : 1u) - 1u; }

// The nearest centre of x among centres in ascending order (Sec. 3.3 leaves the rule open; this is the
// rule the library fixes): a = last centre <= x, b = the next one; the two distances are evaluated in
// fp64 with one rounding each, b wins only if strictly nearer, and among centres of equal value the lowest
// index is taken.
// The nearest-centre rule is monotone in the value, so it is fully described by K - 1 cut keys:
// cut[k] = smallest key (order-preserving bit pattern) of a finite value whose nearest centre has
// index >= k, or 0xffffffff when no finite value reaches k; then "number of cut keys <= key(x)" IS
// nearest_centre(x), bit for bit.  With a = C[k-1] < b = C[k] a value in [a, b] reaches k exactly if
// |b - x| < |x - a| in the rule's arithmetic; smaller ones do not, larger ones do.  Where C[k-1] equals
// C[k] the lowest index of the run takes everything, so reaching k means reaching the first index after
// the run.  The border lies next to the midpoint: a bracket of five keys around it is probed first, and
// the bisection goes on from what the probes have proved.
//
// The cut key between two neighbours ca < cb.  (Strictly: of equal ones cut_key finds the end of the run first.)
__device__ __forceinline__ u32 cut_between(float ca, float cb) {
    const double a = (double)ca, b = (double)cb;
    auto reaches = [&](u32 key) { const double x = (double)val_of(key); return fabs(b - x) < fabs(x - a); };
    u32 lo = key_of(ca) + 1u, hi = key_of(cb);            // invariant: hi reaches, nothing below lo does
    if (lo > hi) lo = hi;
    const u32 mk = min(max(key_of((float)(0.5 * (a + b))), lo), hi);
    const u32 p_hi = hi - mk > 2u ? mk + 2u : hi, p_lo = mk - lo > 2u ? mk - 2u : lo;
    if (reaches(p_hi)) {
        hi = p_hi;
        if (p_lo < hi) { if (reaches(p_lo)) hi = p_lo; else lo = p_lo + 1u; }
    } else {
        lo = p_hi + 1u;
    }
    while (lo < hi) {
        const u32 mid = lo + ((hi - lo) >> 1);
        if (reaches(mid)) hi = mid; else lo = mid + 1u;
    }
    return hi;
}
// cut[k] of K centres in ascending order, equal ones among them.
__device__ __forceinline__ u32 cut_key(const float *C, u32 K, u32 k) {
    u32 j = k;
    while (j < K && !(C[j - 1u] < C[j])) ++j;
    return j < K ? cut_between(C[j - 1u], C[j]) : 0xffffffffu;
}
// All of them: threads 1..K-1 of the workgroup each find one; entries from K up to 255 are set to 0xffffffff.  C and cut are LDS
// arrays of 256 entries; the caller synchronises before and after.
__device__ __forceinline__ void compute_cut_keys(const float *C, int K, u32 *cut) {
    const u32 k = threadIdx.x;
    if (k == 0 || k > 255u) return;
    cut[k] = cut_key(C, (u32)K, k);
}

// Number of cut keys <= key, i.e. the index of the nearest centre.  kp2 = smallest power of two >= K.
__device__ __forceinline__ u32 centre_by_cuts(const u32 *cut, u32 kp2, u32 key) {
    u32 lo = 0;
    for (u32 step = kp2 >> 1; step >= 1; step >>= 1)
        if (cut[lo + step] <= key) lo += step;
    return lo;
}

// Signed bins (bin g has weight 2^(8g - 149)) -> the exact sum rounded once (to nearest, ties to even) to fp64.
// Everything stays in registers (fixed indices after unrolling): this runs once per centre and iteration on the
// critical path of a Lloyd iteration.  `stride`: distance between the bins of one sum; bins outside [g0, g1]
// (the same in the whole wave) are zero and not read.
__device__ __forceinline__ double signed_bins_to_double(const u64 *bins, u32 stride = 1u, u32 g0 = 0u, u32 g1 = EXCP_ABSM_BINS - 1u) {
    // eight bins make a word and what goes into the next one: Horner's scheme in 128 bits (|sum| < 2^121)
    u64 W[6] = {0, 0, 0, 0, 0, 0};
    long long carry = 0;
#pragma unroll
    for (u32 h = 0; h < EXCP_ABSM_BINS / 8u; ++h) {
        __int128 t = carry;
        if (8u * h <= g1 && 8u * h + 7u >= g0) {
            u64 b[8];
#pragma unroll
            for (u32 j = 0; j < 8; ++j) b[j] = 8u * h + j >= g0 && 8u * h + j <= g1 ? bins[(8u * h + j) * stride] : 0ull;
            __int128 v = (long long)b[7];
#pragma unroll
            for (int j = 6; j >= 0; --j) v = (v << 8) + (long long)b[j];
            t += v;
        }
        W[h] = (u64)t;
        carry = (long long)(t >> 64);
    }
    W[5] = (u64)carry;
    const bool neg = carry < 0;
    if (neg) {                                  // magnitude = two's complement negation of the 384 bits
        u64 c = 1;
#pragma unroll
        for (int i = 0; i < 6; ++i) { const u64 v = ~W[i] + c; c = (c && v == 0) ? 1ull : 0ull; W[i] = v; }
    }
    // the top non-zero word, the word below it, and whether anything lies below those
    u64 hi = 0, lo = 0, rest = 0; int wi = -1;
#pragma unroll
    for (int i = 5; i >= 0; --i) {
        if (wi < 0) { if (W[i]) { wi = i; hi = W[i]; } }
        else if (wi == i + 1) lo = W[i];
        else rest |= W[i];
    }
    if (wi < 0) return 0.0;
    const int top = 63 - __clzll((long long)hi), msb = 64 * wi + top;
    double mag;
    if (msb <= 52) {
        mag = ldexp((double)hi, -149);          // wi == 0: the value itself, exactly
    } else {
        // the 53 bits from msb down, out of hi:lo; sh = number of bits of hi:lo below them
        const int sh = top + 12;                // 64 + top - 52, in [12, 75]
        u64 mant, guard, sticky;
        if (sh < 64) {
            mant = (hi << (64 - sh)) | (lo >> sh);
            guard = (lo >> (sh - 1)) & 1ull;
            sticky = lo & ((1ull << (sh - 1)) - 1ull);
        } else if (sh == 64) {
            mant = hi; guard = lo >> 63; sticky = lo & 0x7fffffffffffffffull;
        } else {
            mant = hi >> (sh - 64);
            guard = (hi >> (sh - 65)) & 1ull;
            sticky = (hi & ((1ull << (sh - 65)) - 1ull)) | lo;
        }
        sticky |= rest;
        if (guard && (sticky || (mant & 1ull))) mant += 1;
        mag = ldexp((double)mant, msb - 52 - 149);
    }
    return neg ? -mag : mag;
}

// t * 2^(base - 149), rounded once (to nearest, ties to even).
__device__ __forceinline__ double i128_to_double(__int128 t, u32 base) {
    const bool neg = t < 0;
    const unsigned __int128 mag = neg ? (unsigned __int128)0 - (unsigned __int128)t : (unsigned __int128)t;
    const u64 hi = (u64)(mag >> 64), lo = (u64)mag;
    const int msb = hi ? 127 - __clzll((long long)hi) : 63 - __clzll((long long)(lo | 1ull));
    double m;
    if (msb <= 52) {
        m = ldexp((double)lo, (int)base - 149);
    } else {
        const int sh = msb - 52;                          // 1 .. 75
        u64 mant = (u64)(mag >> sh);
        const unsigned __int128 below = mag << (128 - sh);
        const u64 top = (u64)(below >> 64);
        if ((top >> 63) && ((top << 1) | (u64)below | (mant & 1ull))) ++mant;
        m = ldexp((double)mant, sh + (int)base - 149);
    }
    return neg ? -m : m;
}

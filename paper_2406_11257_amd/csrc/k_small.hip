// Tensors of at most EXCP_SMALL_ELEMS elements: Alg. 1 in one launch or two instead of some twenty-five, beside which a group's larger
// tensors go their way.  A call about such tensors moves a few hundred KB; what it costs is launches, and inside them chains of dependent steps
// with a wave or two at work.  Here a workgroup holds a whole tensor in registers (small_front: statistics, masks,
// compaction, header), and then one holds a whole survivor stream (small_codes: initial centres, Lloyd iterations,
// codes, and for the residuals W_hat), everything they look up in LDS.  Of few tensors a workgroup does both, for its stream.  (us a call, before and now: a norm vector of 4096
// elements 169 / 57 (in two launches 61), 1000 of them 1524 / 348, 8 bits 3814 / 477; 1000 tensors of 8192 elements, all kept, 1924 / 876; 8192
// residuals of a sign-like update, 337 / 141.)
//
// The definitions are those of the general kernels (k_stats, k_mask, k_kmeans) and so are the bytes: exact median, exact sums
// rounded once, thresholds in fp32 with correctly rounded sqrt and divide, exact sums per centre.
#include "excp_util.h"

namespace {

constexpr u32 SM = 1024, SM_WAVES = SM / 64, PER = EXCP_SMALL_ELEMS / SM;      // threads of a workgroup, elements of a thread
constexpr u32 BATCHES = EXCP_SMALL_ELEMS / 64;

// ---------------------------------------------------------------- statistics, masks, compaction, header
// Element (j * SM_WAVES + wave) * 64 + lane is the thread's j-th, so a ballot is a bitmap word.
struct SmallTensor {
    const float *W, *Wp, *m, *v;
    float *W_out;
    unsigned char *blob;
    u64 blob_cap, elem_off;
    u32 n, rec;
};
__device__ __forceinline__ SmallTensor small_tensor(const TDesc &D) {
    return {D.W, D.Wp, D.m, D.v, D.W_out, D.blob, D.blob_cap, D.elem_off, (u32)D.n, D.rec};
}
struct FrontShared {
    u32 hist[2048];
    u64 bins[EXCP_ABSM_BINS], L, H;
    u64 bw[BATCHES], bo[BATCHES];
    u32 at[BATCHES + 1], obits[EXCP_SMALL_ELEMS / 32];     // survivors before a batch (moment survivors << 16); M_o by rank
    u32 wave[SM_WAVES], pick[2], nf, med;
    float tw, ro, mean;
    double abs;
};
// What a thread knows of its elements afterwards: residuals, moments, and the two bitmaps' words of their batches.
struct FrontValues { float d[PER], m[PER], v[PER]; u64 bw[PER], bo[PER]; };
// Where the blob's sections are, and whether there is one.
struct SmallLayout { u64 off_bw, off_bo, off_cw, off_cm, off_cv, bytes; u32 n_w, n_o; int status; };
__device__ __forceinline__ SmallLayout small_layout(const FrontShared &F, const SmallTensor &D, const GroupParams &g) {
    SmallLayout s;
    const u64 nb = (u64)g.nbits;
    s.n_w = F.at[BATCHES] & 0xffffu; s.n_o = F.at[BATCHES] >> 16;
    s.off_bw = EXCP_HEADER + excp_books_bytes((u32)g.nbits);
    s.off_bo = s.off_bw + excp_pad16(8ull * excp_words(D.n));
    s.off_cw = s.off_bo + excp_pad16(8ull * excp_words(s.n_w));
    s.off_cm = s.off_cw + excp_pad16(8ull * excp_words(s.n_w * nb));
    s.off_cv = s.off_cm + excp_pad16(8ull * excp_words(s.n_o * nb));
    s.bytes = s.off_cv + excp_pad16(8ull * excp_words(s.n_o * nb));
    s.status = F.nf ? -3 : (s.bytes > D.blob_cap ? -2 : 0);
    return s;
}

__device__ __forceinline__ void small_front(const SmallTensor &D, const GroupParams &g, FrontShared &F, FrontValues &X) {
    const u32 tid = threadIdx.x, lane = tid & 63u, n = D.n;
    const u32 wave = (u32)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
    u32 *hist = F.hist, *s_at = F.at, *s_wave = F.wave, *s_pick = F.pick;
    u64 *bins = F.bins, *s_bw = F.bw, *s_bo = F.bo;
    float (&d)[PER] = X.d, (&mv)[PER] = X.m, (&vv)[PER] = X.v;
    u64 (&bw)[PER] = X.bw, (&bo)[PER] = X.bo;
    const u32 wt = excp_wtype(g.flags);
    u32 key[PER];
    {
        float a[PER], p[PER];
#pragma unroll
        for (u32 j = 0; j < PER; ++j) {
            const u32 e = (j * SM_WAVES + wave) * 64u + lane;
            const bool ok = e < n;
            a[j] = ok ? load_weight(D.W, e, wt) : 0.f; p[j] = ok ? load_weight(D.Wp, e, wt) : 0.f;
            mv[j] = ok ? D.m[e] : 0.f; vv[j] = ok ? D.v[e] : 1.f;
        }
#pragma unroll
        for (u32 j = 0; j < PER; ++j) {
            d[j] = a[j] - p[j];
            key[j] = (j * SM_WAVES + wave) * 64u + lane < n ? f2u(d[j]) & 0x7fffffffu : 0xffffffffu;      // (never a key: those have 31 bits)
        }
    }
    // what is not finite (a residual is not where a weight is not); the window of the exact sum of |m|: the 24 positions below the largest
    u32 nf = 0, mmax = 0;
#pragma unroll
    for (u32 j = 0; j < PER; ++j) {
        if (key[j] != 0xffffffffu) nf += (key[j] & 0x7f800000u) == 0x7f800000u;
        nf += (f2u(vv[j]) & 0x7f800000u) == 0x7f800000u;
        const u32 mb = f2u(mv[j]) & 0x7fffffffu;
        if (mb >= 0x7f800000u) ++nf; else mmax = max(mmax, mb);
    }
    for (u32 i = tid; i < 2048u; i += SM) hist[i] = 0;
    if (tid < EXCP_SMALL_ELEMS / 32u) F.obits[tid] = 0;
    if (tid < EXCP_ABSM_BINS) bins[tid] = 0;
    if (tid == 0) { F.L = 0; F.H = 0; F.nf = 0; s_pick[0] = 0; }
    mmax = wave_max_u32(mmax);
    if (lane == 0u) s_wave[wave] = mmax;
    __syncthreads();
#pragma unroll
    for (u32 q = 0; q < SM_WAVES; ++q) mmax = max(mmax, s_wave[q]);
    {
        const u32 e = mmax >> 23, pos = (e ? e : 1u) - 1u, B = pos > 23u ? pos - 23u : 0u;
        const u32 thr_lo = B ? ((B + 1u) << 23) : 0u, span = ((B + 25u) << 23) - thr_lo;
        double dsum = 0.0;                                 // eight values below 2^48 units: exact
#pragma unroll
        for (u32 j = 0; j < PER; ++j) {
            const u32 mb = f2u(mv[j]) & 0x7fffffffu;
            const bool in = mb - thr_lo < span && mb < 0x7f800000u;
            dsum += in ? (double)u2f(mb) : 0.0;
            if (!in && mb && mb < 0x7f800000u) {
                const u32 ee = mb >> 23, mant = (mb & 0x7fffffu) | (ee ? 0x800000u : 0u), pp = (ee ? ee : 1u) - 1u;
                atomicAdd(&bins[pp >> 3], (u64)mant << (pp & 7u));
            }
        }
        const double units = ldexp(dsum, 149 - (int)B);
        const u32 hi32 = (u32)(units * 2.3283064365386963e-10), lo32 = (u32)(units - (double)hi32 * 4294967296.0);
        const u64 L = wave_sum_u64(lo32), H = wave_sum_u64(hi32);
        nf = wave_sum_u32(nf);
        if (lane == 0u) { atomicAdd(&F.L, L); atomicAdd(&F.H, H); if (nf) atomicAdd(&F.nf, nf); }
        // the lower median of |d|: 11 + 10 + 10 key bits
        u32 prefix = 0, rank = n ? (n - 1u) >> 1 : 0u;
#pragma unroll
        for (u32 pass = 0; pass < 3u; ++pass) {
            const u32 shift = pass == 0u ? 20u : (pass == 1u ? 10u : 0u), width = pass == 0u ? 11u : 10u;
            if (pass) { __syncthreads(); for (u32 i = tid; i < 2048u; i += SM) hist[i] = 0; __syncthreads(); }
#pragma unroll
            for (u32 j = 0; j < PER; ++j) {
                const bool in = key[j] != 0xffffffffu && (pass == 0u || key[j] >> (shift + width) == prefix);
                const u32 bin = (key[j] >> shift) & ((1u << width) - 1u);
                if (wt) hist_add_tied(hist, bin, in); else if (in) atomicAdd(&hist[bin], 1u);
            }
            __syncthreads();
            const u32 c0 = hist[2u * tid], c1 = hist[2u * tid + 1u], incl = wave_incl_scan_u32(c0 + c1);
            if (lane == 63u) s_wave[wave] = incl;
            __syncthreads();
            u32 before = incl - c0 - c1;
            for (u32 q = 0; q < wave; ++q) before += s_wave[q];
            if (rank >= before && rank < before + c0 + c1) {               // exactly one thread
                const bool second = rank >= before + c0;
                s_pick[0] = 2u * tid + (second ? 1u : 0u); s_pick[1] = rank - before - (second ? c0 : 0u);
            }
            __syncthreads();
            prefix = (prefix << width) | s_pick[0]; rank = s_pick[1];
        }
        if (tid == 0) {
            const u64 lo64 = F.L + (F.H << 32), hi64 = (F.H >> 32) + (lo64 < F.L ? 1ull : 0ull);
            const u64 piece[3] = {lo64 & 0xffffffffull, lo64 >> 32, hi64};
#pragma unroll
            for (u32 q = 0; q < 3u; ++q) { const u32 p = B + 32u * q; if (piece[q]) bins[p >> 3] += piece[q] << (p & 7u); }
            const double sum = n ? signed_bins_to_double(bins) : 0.0;
            F.abs = sum;
            F.mean = n ? (float)(sum / (double)n) : 0.f;
            F.ro = __fmul_rn(g.beta, F.mean);
            F.tw = n ? __fmul_rn(g.alpha, u2f(prefix)) : 0.f;
            F.med = n ? prefix : 0u;
        }
    }
    __syncthreads();
    const float t_w = F.tw, r_o = F.ro;
    const float T = t_w * t_w, T_keep = T * 1.00001f, T_drop = T * 0.99999f;
    const bool T_ok = __builtin_amdgcn_classf(T, 0x100);
#pragma unroll
    for (u32 j = 0; j < PER; ++j) {
        const u32 b = j * SM_WAVES + wave, left = n > b * 64u ? n - b * 64u : 0u;
        const u64 valid = left >= 64u ? ~0ull : ((1ull << left) - 1ull);
        const float ad = fabsf(d[j]);
        u64 keep;
        if (g.flags & 2u) {
            keep = ballot64(ad > t_w);
        } else {                                          // the estimate where it is clear, the exact expression elsewhere (see k_mask_slots)
            const float dd = ad * ad, x = dd * vv[j];
            const u64 b_keep = ballot64(x > T_keep), b_drop = ballot64(x < T_drop);
            const u64 b_trust = ballot64(__builtin_amdgcn_classf(vv[j], 0x100)) & ballot64(__builtin_amdgcn_classf(dd, 0x100)) & ballot64(__builtin_amdgcn_classf(x, 0x100));
            const u64 amb = T_ok ? (~(b_keep | b_drop) | ~b_trust) : ~0ull;
            keep = b_keep;
            if (amb & valid) keep = (b_keep & ~amb) | (ballot64(ad > t_w / sqrtf(vv[j])) & amb);
        }
        bw[j] = keep & valid;
        bo[j] = ballot64(fabsf(mv[j]) > r_o) & bw[j];
        if (lane == 0u) { s_bw[b] = bw[j]; s_bo[b] = bo[j]; }
    }
    __syncthreads();
    if (tid < BATCHES) {
        const u32 c = (u32)__popcll(s_bw[tid]) | (u32)__popcll(s_bo[tid]) << 16, incl = wave_incl_scan_u32(c);
        s_at[tid] = incl - c;
        if (lane == 63u) s_wave[wave] = incl;
    }
    __syncthreads();
    if (tid >= 64u && tid < BATCHES) {
        u32 before = 0;
        for (u32 q = 0; q < wave; ++q) before += s_wave[q];
        s_at[tid] += before;
    }
    if (tid == 0) { u32 all = 0; for (u32 q = 0; q < BATCHES / 64u; ++q) all += s_wave[q]; s_at[BATCHES] = all; }
    __syncthreads();
}

// The bitmaps, the header and the record.  (The record's objectives are written by the workgroups that know them.)
__device__ __forceinline__ void small_outputs(const Workspace &w, const SmallTensor &D, const GroupParams &g, const SmallLayout &s, FrontShared &F, const FrontValues &X) {
    const u32 tid = threadIdx.x;
    const u32 wave = (u32)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
#pragma unroll
    for (u32 j = 0; j < PER; ++j) {
        if (__builtin_amdgcn_inverse_ballot_w64(X.bo[j])) {
            const u32 rk = (F.at[j * SM_WAVES + wave] & 0xffffu) + lanes_below(X.bw[j]);
            atomicOr(&F.obits[rk >> 5], 1u << (rk & 31u));
        }
    }
    {
        const u32 nwords = (u32)excp_words(D.n), padded = nwords + (nwords & 1u);
        if (tid < padded) ((u64 *)(D.blob + s.off_bw))[tid] = tid < BATCHES ? F.bw[tid] : 0ull;      // (padded <= BATCHES: it is even)
    }
    __syncthreads();
    {
        const u32 nwo = (u32)excp_words(s.n_w), padded = nwo + (nwo & 1u);
        const u64 cap_words = D.blob_cap > s.off_bo ? (D.blob_cap - s.off_bo) >> 3 : 0ull;
        if (tid < padded && tid < cap_words) ((u64 *)(D.blob + s.off_bo))[tid] = (u64)F.obits[2u * tid] | (u64)F.obits[2u * tid + 1u] << 32;
    }
    if (tid != 0) return;
    u32 *h = (u32 *)D.blob;
    u64 *h64 = (u64 *)D.blob;
    float *hf = (float *)D.blob;
    const float r_o = D.n ? F.ro : 0.f;
    h[0] = EXCP_MAGIC; h[1] = EXCP_VERSION; h[2] = (u32)g.nbits; h[3] = g.flags;
    h64[2] = D.n; h64[3] = s.n_w; h64[4] = s.n_o;
    hf[10] = g.alpha; hf[11] = g.beta; hf[12] = u2f(F.med); hf[13] = F.mean;
    hf[14] = F.tw; hf[15] = r_o;
    h64[8] = s.bytes;
    h[18] = (u32)g.iters; h[19] = 0u;
    HostRec &R = w.rec_dev[w.rec_base + D.rec];
    R.n = D.n; R.n_w = s.n_w; R.n_o = s.n_o; R.blob_bytes = s.bytes; R.nonfinite = F.nf; R.abs_sum = F.abs;
    R.med = u2f(F.med); R.mean32 = F.mean; R.t_w = F.tw; R.r_o = r_o; R.status = s.status; R.pad = 0;
}

// A stream's survivors to their places in `to`.
__device__ __forceinline__ void small_compact(const FrontShared &F, const u64 (&words)[PER], const float (&x)[PER], u32 shift, float *to) {
    const u32 wave = (u32)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
#pragma unroll
    for (u32 j = 0; j < PER; ++j)
        if (__builtin_amdgcn_inverse_ballot_w64(words[j])) to[(F.at[j * SM_WAVES + wave] >> shift & 0xffffu) + lanes_below(words[j])] = x[j];
}

// `single`: the only tensor's description comes as an argument and is left where k_small_codes looks for it.
__global__ __launch_bounds__(SM) void k_small_front(Workspace w, GroupParams g, TDesc one, u32 single) {
    __shared__ FrontShared F;
    const u32 t = blockIdx.x;
    if (single && threadIdx.x == 0) w.desc[0] = one;
    const SmallTensor D = single ? small_tensor(one) : small_tensor(w.desc[t]);
    FrontValues X;
    small_front(D, g, F, X);
    const SmallLayout s = small_layout(F, D, g);
    small_compact(F, X.bw, X.d, 0u, w.xw + D.elem_off);
    small_compact(F, X.bo, X.m, 16u, w.xm + D.elem_off);
    small_compact(F, X.bo, X.v, 16u, w.xv + D.elem_off);
    small_outputs(w, D, g, s, F, X);
    if (threadIdx.x != 0) return;
    TState &S = w.st[t];
    S.off_bo = s.off_bo; S.off_cw = s.off_cw; S.off_cm = s.off_cm; S.off_cv = s.off_cv;
    S.n_w = s.n_w; S.n_o = s.n_o; S.blob_bytes = s.bytes; S.status = s.status;
}

// ---------------------------------------------------------------- codebook, codes, W_hat
constexpr u32 CELLS = 4096, CELLS_PER = CELLS / SM;
constexpr u32 HALF_BITS = 42, WIDE_SPAN = 60;             // a value is lo + hi 2^42 units; 8192 halves add up below 2^55
constexpr u32 CROWD = 48;                                 // values of a cell that one lane reads; with more the stream is sorted, and a cell is two values
struct CellSum { u64 lo, hi; };                           // while the sums are taken; then one integer of 128 bits

struct SmallShared {
    __int128 before[CELLS + 1u];                          // sum of the cells before, in units of the stream's lowest bit position
    u32 sorted[EXCP_SMALL_ELEMS];                         // the values' keys by cell
    u32 begin[CELLS + 1u];
    u32 pack[EXCP_SMALL_ELEMS / 4u + 2u];                 // the packed codes
    float C[EXCP_MAX_K + 1u], fresh[EXCP_MAX_K + 1u];
    u32 cut[EXCP_MAX_K + 1u];
    __int128 above[EXCP_MAX_K + 2u];                      // per border: sum and number of the values from its cut key up
    u32 n_above[EXCP_MAX_K + 2u];
    u64 bits[BATCHES];                                    // keep bitmap, survivors before each of its words
    u32 at[BATCHES];
    u64 wave_lo[SM_WAVES], wave_hi[SM_WAVES];
    double wave_obj[SM_WAVES];
    u32 wave_cnt[SM_WAVES], ext[4], disorder, most;
};

// Signed value in two halves.
__device__ __forceinline__ CellSum halves(u32 bits, u32 pos_lo) {
    const u32 mb = bits & 0x7fffffffu, e = mb >> 23;
    const u64 mant = mb ? (u64)((mb & 0x7fffffu) | (e ? 0x800000u : 0u)) : 0ull;
    const u32 s = mb ? bit_pos(mb) - pos_lo : 0u;         // <= WIDE_SPAN
    u64 lo, hi;
    if (s >= HALF_BITS) { lo = 0; hi = mant << (s - HALF_BITS); }
    else { lo = (mant << s) & ((1ull << HALF_BITS) - 1ull); hi = s + 24u > HALF_BITS ? mant >> (HALF_BITS - s) : 0ull; }
    if (bits >> 31) { lo = (u64)0 - lo; hi = (u64)0 - hi; }
    return {lo, hi};
}
__device__ __forceinline__ __int128 joined(u64 lo, u64 hi) { return (__int128)((unsigned __int128)(__int128)(long long)lo + ((unsigned __int128)(__int128)(long long)hi << HALF_BITS)); }

// Ascending order of the first len entries (bitonic; the places up to the next power of two are filled).  A wave has 512
// neighbouring places, so up to that distance it is alone with them.
__device__ __forceinline__ void sort_keys(u32 *a, u32 len) {
    const u32 tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    u32 n = 512u;
    while (n < len) n <<= 1;
    for (u32 i = len + tid; i < n; i += SM) a[i] = 0xffffffffu;
    __syncthreads();
    for (u32 k = 2u; k <= n; k <<= 1) {
        for (u32 j = k >> 1; j >= 1u; j >>= 1) {
#pragma unroll
            for (u32 q = 0; q < PER / 2u; ++q) {
                const u32 pair = wave * 256u + q * 64u + lane, lo = ((pair & ~(j - 1u)) << 1) | (pair & (j - 1u)), hi = lo | j;
                if (lo < n) {
                    const u32 x = a[lo], y = a[hi];
                    if ((x > y) == ((lo & k) == 0u)) { a[lo] = y; a[hi] = x; }
                }
            }
            // (the next step's distance is j / 2, or k after the last)
            if (j > 256u || (j == 1u && k >= 512u)) __syncthreads(); else wave_lds_fence();
        }
    }
    __syncthreads();
}

// One stream of `len` values, of which the thread holds every SM-th: centres, codes into `out`, and of the residuals (which = 0) W_hat by the
// keep bitmap at `keep`.  `x`: the stream's place in the survivors' area, `there`: it has been written.
template <bool ONE_WAVE>                                  // up to 63 centres: one wave's work
__device__ __forceinline__ void small_codes(const Workspace &w, const GroupParams &g, SmallShared &A, const SmallTensor &D, u32 which, bool good, u32 len,
                                            const float (&v)[PER], float *x, bool there, u64 *out, const u64 *keep) {
    const u32 tid = threadIdx.x, lane = tid & 63u;
    const u32 wave = (u32)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
    const u32 K = (u32)g.K, nbits = (u32)g.nbits, E = 1u << nbits;
    u32 kp2 = 1; while (kp2 < K) kp2 <<= 1;
    for (u32 i = tid; i < EXCP_SMALL_ELEMS / 4u + 2u; i += SM) A.pack[i] = 0;
    if (tid <= EXCP_MAX_K) { A.cut[tid] = 0xffffffffu; A.C[tid] = 0.f; }
    double obj = 0.0;
    if (len) {                                            // (the same in the whole workgroup)
        if (tid < 4) A.ext[tid] = tid == 1u || tid == 3u ? 0u : 0xffffffffu;
        if (tid == 0) { A.disorder = 0u; A.most = 0u; }
        for (u32 i = tid; i < CELLS; i += SM) { A.begin[i] = 0; ((CellSum *)A.before)[i] = {0ull, 0ull}; }
        __syncthreads();
        u32 kmin = 0xffffffffu, kmax = 0u, mag = 0xffffffffu, top = 0u;          // mag: smallest magnitude less one (zero wraps to the largest)
#pragma unroll
        for (u32 j = 0; j < PER; ++j) {
            if (j * SM + tid >= len) continue;
            const u32 k = key_of(v[j]), mb = f2u(v[j]) & 0x7fffffffu;
            kmin = min(kmin, k); kmax = max(kmax, k); mag = min(mag, mb - 1u); top = max(top, mb);
        }
        kmin = wave_min_u32(kmin); kmax = wave_max_u32(kmax); mag = wave_min_u32(mag); top = wave_max_u32(top);
        if (lane == 0u) { atomicMin(&A.ext[0], kmin); atomicMax(&A.ext[1], kmax); atomicMin(&A.ext[2], mag); atomicMax(&A.ext[3], top); }
        __syncthreads();
        kmin = A.ext[0]; kmax = A.ext[1]; mag = A.ext[2] + 1u; top = A.ext[3];   // (mag 0: nothing but zeros)
        const u32 base = bit_pos(mag), span = bit_pos(top) - base;
        const bool wide = span > WIDE_SPAN;               // more binary orders than 128 bits hold: sums in bins instead
        // the values by cell: equal ranges of the key
        const u32 k0 = excp_closed_key(kmin, mag), range = excp_closed_key(kmax, mag) - k0, rbits = 32u - (u32)__clz((int)(range | 1u));
        const u32 shift = rbits > 12u ? rbits - 12u : 0u;
        u32 cell[PER];                                    // cell << 16 | arrival
#pragma unroll
        for (u32 j = 0; j < PER; ++j) {
            cell[j] = 0;
            if (j * SM + tid >= len) continue;
            const u32 c = (excp_closed_key(key_of(v[j]), mag) - k0) >> shift;
            cell[j] = c << 16 | atomicAdd(&A.begin[c], 1u);
            if (!wide) {
                const CellSum q = halves(f2u(v[j]), base);
                CellSum *s = (CellSum *)A.before + c;
                if (q.lo) atomicAdd(&s->lo, q.lo);
                if (q.hi) atomicAdd(&s->hi, q.hi);
            }
        }
        __syncthreads();
        // exclusive scans over the cells: numbers into `begin`, sums into `before`
        auto scan_cells = [&]() {
            u32 c[CELLS_PER], cs = 0, most = 0;
            u64 lo[CELLS_PER], hi[CELLS_PER], los = 0, his = 0;
#pragma unroll
            for (u32 q = 0; q < CELLS_PER; ++q) {
                const CellSum s = ((const CellSum *)A.before)[tid * CELLS_PER + q];
                c[q] = A.begin[tid * CELLS_PER + q]; lo[q] = s.lo; hi[q] = s.hi;
                cs += c[q]; los += lo[q]; his += hi[q]; most = max(most, c[q]);
            }
            const u32 ci = wave_incl_scan_u32(cs);
            const u64 li = wave_incl_scan_u64(los), hii = wave_incl_scan_u64(his);
            most = wave_max_u32(most);
            if (lane == 63u) { A.wave_cnt[wave] = ci; A.wave_lo[wave] = li; A.wave_hi[wave] = hii; atomicMax(&A.most, most); }
            __syncthreads();
            u32 cr = ci - cs;
            u64 lr = li - los, hr = hii - his;
            for (u32 q = 0; q < wave; ++q) { cr += A.wave_cnt[q]; lr += A.wave_lo[q]; hr += A.wave_hi[q]; }
#pragma unroll
            for (u32 q = 0; q < CELLS_PER; ++q) {
                A.begin[tid * CELLS_PER + q] = cr; A.before[tid * CELLS_PER + q] = joined(lr, hr);
                cr += c[q]; lr += lo[q]; hr += hi[q];
            }
            if (tid == SM - 1u) { A.begin[CELLS] = cr; A.before[CELLS] = joined(lr, hr); }
            __syncthreads();
        };
        scan_cells();
#pragma unroll
        for (u32 j = 0; j < PER; ++j) if (j * SM + tid < len) A.sorted[A.begin[cell[j] >> 16] + (cell[j] & 0xffffu)] = key_of(v[j]);
        const bool ties = A.most > CROWD;                 // (ties, or values bunched beside a few far away)
        __syncthreads();
        if (ties) {
            sort_keys(A.sorted, len);
            for (u32 c = tid; c < CELLS; c += SM) {       // a cell is two places now
                CellSum s = {0ull, 0ull};
#pragma unroll
                for (u32 q = 0; q < 2u; ++q)
                    if (2u * c + q < len && !wide) { const CellSum h = halves(f2u(val_of(A.sorted[2u * c + q])), base); s.lo += h.lo; s.hi += h.hi; }
                ((CellSum *)A.before)[c] = s;
                A.begin[c] = 2u * c < len ? min(len - 2u * c, 2u) : 0u;
            }
            __syncthreads();
            scan_cells();
        }
        // the cell that a key of the stream's range belongs to: no smaller value lies in a higher one, no larger one in a lower
        auto cell_of_key = [&](u32 key) -> u32 {
            if (!ties) return (excp_closed_key(key, mag) - k0) >> shift;
            u32 p = 0;                                    // number of values below the key (the key is not above all of them)
#pragma unroll
            for (u32 step = EXCP_SMALL_ELEMS / 2u; step >= 1u; step >>= 1) if (p + step <= len && A.sorted[p + step - 1u] < key) p += step;
            return p >> 1;
        };
        // Initial centres: rank ((2k + 1) len) / (2K).  Sixteen lanes take one: its cell by bisection, and in the cell each lane
        // counts, for its share of the values, those before them in the order.
        for (u32 k = tid >> 4; k < K; k += SM / 16u) {
            const u32 r = (u32)(((u64)(2u * k + 1u) * len) / (2ull * K));
            if (ties) { if ((tid & 15u) == 0u) A.C[k] = val_of(A.sorted[r]); continue; }
            u32 c = 0;                                    // last cell with begin <= r: it holds rank r
#pragma unroll
            for (u32 step = CELLS / 2u; step >= 1u; step >>= 1) if (A.begin[c + step] <= r) c += step;
            const u32 b0 = A.begin[c], b1 = A.begin[c + 1u];
            for (u32 i = b0 + (tid & 15u); i < b1; i += 16u) {
                const u32 mine = A.sorted[i];
                u32 less = 0;
                for (u32 q = b0; q < b1; ++q) { const u32 o = A.sorted[q]; less += (o < mine || (o == mine && q < i)) ? 1u : 0u; }
                if (less == r - b0) A.C[k] = val_of(mine);
            }
        }
        __syncthreads();
        const bool centre = tid < K;
        // the ascending order of the centres after an update (stable; nothing moves unless a run of equal centres was torn apart)
        auto put_back = [&](float c, bool unsorted) {
            if (!centre) return;
            u32 rank = tid;
            if (unsorted) {
                rank = 0;
#pragma unroll 1
                for (u32 j = 0; j < K; ++j) { const float cj = A.fresh[j]; rank += (cj < c || (cj == c && j < tid)) ? 1u : 0u; }
            }
            A.C[rank] = c;
        };
        // The sum and number of the values from a cut key up: those of the higher cells, and the cell's own one by one.
        auto above_cut = [&](u32 cut, __int128 &sum, u32 &cnt) {
            sum = 0; cnt = 0;
            if (cut > kmax) return;
            if (cut <= kmin) { sum = A.before[CELLS]; cnt = len; return; }
            const u32 c = cell_of_key(cut), b0 = A.begin[c], b1 = A.begin[c + 1u];
            u64 lo = 0, hi = 0;
            sum = A.before[CELLS] - A.before[c + 1u]; cnt = len - b1;
            for (u32 q = b0; q < b1; q += 4u) {
                u32 key[4];
#pragma unroll
                for (u32 e = 0; e < 4u; ++e) key[e] = A.sorted[min(q + e, b1 - 1u)];
#pragma unroll
                for (u32 e = 0; e < 4u; ++e)
                    if (q + e < b1 && key[e] >= cut) { const CellSum h = halves(f2u(val_of(key[e])), base); lo += h.lo; hi += h.hi; ++cnt; }
            }
            sum += joined(lo, hi);
        };
        if (!wide && ONE_WAVE) {
            // A lane a centre, and what neighbours tell each other goes through registers: what bounds an iteration is its chain of
            // dependent steps, and a trip through LDS is as long as thirty instructions.
            if (wave == 0u) {
                float own = A.C[min(tid, K - 1u)];
                for (u32 i = 0;; ++i) {
                    const float below = lane_below_f32(own);
                    u32 cut = 0;
                    if (__all(!centre || tid == 0u || below < own)) {
                        if (centre && tid) cut = cut_between(below, own);
                    } else {                               // equal centres: the lowest of a run takes everything
                        if (centre) A.C[tid] = own;
                        wave_lds_fence();
                        if (centre && tid) cut = cut_key(A.C, K, tid);
                        wave_lds_fence();
                    }
                    if (i == (u32)g.iters) {
                        if (centre) A.C[tid] = own;
                        if (centre && tid) A.cut[tid] = cut;
                        break;
                    }
                    __int128 sum = tid == 0u ? A.before[CELLS] : (__int128)0;
                    u32 cnt = tid == 0u ? len : 0u;
                    if (centre && tid) above_cut(cut, sum, cnt);
                    const __int128 next = lane_above_i128(sum);            // (of lane K: nothing)
                    const u32 m = cnt - lane_above_u32(cnt);
                    float c = own;
                    if (centre && m) c = (float)(i128_to_double(sum - next, base) / (double)m);
                    const float above = lane_above_f32(c);
                    if (__any(tid + 1u < K && !(c <= above))) {
                        if (centre) A.fresh[tid] = c;
                        wave_lds_fence();
                        put_back(c, true);
                        wave_lds_fence();
                        c = A.C[min(tid, K - 1u)];
                    }
                    own = c;
                }
            }
        } else if (!wide) {
            if (tid == 0) { A.above[K] = 0; A.n_above[K] = 0; A.above[0] = A.before[CELLS]; A.n_above[0] = len; }
            for (u32 i = 0;; ++i) {
                u32 cut = 0;
                if (centre && tid) { cut = cut_key(A.C, K, tid); A.cut[tid] = cut; }
                if (i == (u32)g.iters) break;
                if (wave * 64u >= K) { __syncthreads(); __syncthreads(); __syncthreads(); __syncthreads(); continue; }
                if (centre && tid) {
                    __int128 sum;
                    u32 cnt;
                    above_cut(cut, sum, cnt);
                    A.above[tid] = sum; A.n_above[tid] = cnt;
                }
                __syncthreads();
                float c = 0.f;
                if (centre) {
                    const u32 m = A.n_above[tid] - A.n_above[tid + 1u];
                    c = m ? (float)(i128_to_double(A.above[tid] - A.above[tid + 1u], base) / (double)m) : A.C[tid];
                    A.fresh[tid] = c;
                }
                __syncthreads();
                if (tid + 1u < K && !(c <= A.fresh[tid + 1u])) A.disorder = 1u;
                __syncthreads();
                put_back(c, A.disorder != 0u);
                __syncthreads();
                if (tid == 0) A.disorder = 0u;
            }
        } else {
            // sixty binary orders and more: every value goes to its centre's bins in every iteration
            if (!there) {
#pragma unroll
                for (u32 j = 0; j < PER; ++j) if (j * SM + tid < len) x[j * SM + tid] = v[j];      // (read back below by the same workgroup)
            }
            u64 *acc = (u64 *)A.before;                   // [bin][K], and [K] numbers: runs on into `sorted`, which is done with
            static_assert(sizeof(A.before) + sizeof(A.sorted) >= (EXCP_ABSM_BINS + 1u) * EXCP_MAX_K * sizeof(u64), "bins of all centres");
            for (u32 i = 0;; ++i) {
                if (centre && tid) A.cut[tid] = cut_key(A.C, K, tid);
                for (u32 q = tid; q < (EXCP_ABSM_BINS + 1u) * K; q += SM) acc[q] = 0;
                __syncthreads();
                if (i == (u32)g.iters) break;
#pragma unroll 1
                for (u32 j = tid; j < len; j += SM) {
                    const u32 bits = f2u(x[j]), mb = bits & 0x7fffffffu, e = mb >> 23, c = centre_by_cuts(A.cut, kp2, key_of(u2f(bits))), pb = bit_pos(mb);
                    const u64 m = mb ? (u64)((mb & 0x7fffffu) | (e ? 0x800000u : 0u)) << (pb & 7u) : 0ull;
                    if (m) atomicAdd(&acc[(pb >> 3) * K + c], (bits >> 31) ? (u64)0 - m : m);
                    atomicAdd(&acc[EXCP_ABSM_BINS * K + c], 1ull);
                }
                __syncthreads();
                float c = 0.f;
                if (centre) {
                    const u64 m = acc[EXCP_ABSM_BINS * K + tid];
                    c = m ? (float)(signed_bins_to_double(acc + tid, K) / (double)m) : A.C[tid];
                    A.fresh[tid] = c;
                }
                __syncthreads();
                if (tid + 1u < K && !(c <= A.fresh[tid + 1u])) A.disorder = 1u;
                __syncthreads();
                put_back(c, A.disorder != 0u);
                __syncthreads();
                if (tid == 0) A.disorder = 0u;
            }
        }
        __syncthreads();
        // codes, packed in index order
#pragma unroll
        for (u32 j = 0; j < PER; ++j) {
            const u32 i = j * SM + tid;
            if (i >= len) continue;
            const u32 pick = centre_by_cuts(A.cut, kp2, key_of(v[j]));
            const double e = (double)v[j] - (double)A.C[pick];
            obj += e * e;
            const u32 field = pick + 1u, bitpos = i * nbits, wi = bitpos >> 5, sh = bitpos & 31u;
            atomicOr(&A.pack[wi], field << sh);
            if (sh && (field >> (32u - sh))) atomicOr(&A.pack[wi + 1u], field >> (32u - sh));
        }
#pragma unroll
        for (int mm = 32; mm >= 1; mm >>= 1) obj += shfl_xor_f64(obj, mm);
        if (lane == 0u) A.wave_obj[wave] = obj;
        __syncthreads();
        const u32 nwords = (u32)excp_words((u64)len * nbits), padded = nwords + (nwords & 1u);
        for (u32 i = tid; i < padded; i += SM) out[i] = i < nwords ? (u64)A.pack[2u * i] | (u64)A.pack[2u * i + 1u] << 32 : 0ull;
        obj = 0.0;
        if (tid == 0) for (u32 q = 0; q < SM_WAVES; ++q) obj += A.wave_obj[q];
    }
    if (tid == 0) w.rec_dev[w.rec_base + D.rec].obj[which] = obj;
    float *books = (float *)(D.blob + EXCP_HEADER) + which * E;
    if (tid < E) books[tid] = tid && len ? A.C[tid - 1u] : 0.f;
    if (which != 0u || !good || D.W_out == nullptr) return;
    // W_hat: the previous weights, plus the centre where the residual was kept
    const u32 n = D.n, wt = excp_wtype(g.flags);
    __syncthreads();
    if (tid < BATCHES) {
        A.bits[tid] = tid < excp_words(n) ? keep[tid] : 0ull;
        const u32 c = (u32)__popcll(A.bits[tid]), incl = wave_incl_scan_u32(c);
        A.at[tid] = incl - c;
        if (lane == 63u) A.wave_cnt[wave] = incl;
    }
    __syncthreads();
#pragma unroll
    for (u32 j = 0; j < PER; ++j) {
        const u32 b = j * SM_WAVES + wave, e = b * 64u + lane;
        if (e >= n) continue;
        const u64 word = A.bits[b];
        const bool kept = (word >> lane) & 1ull;
        u32 rank = A.at[b] + lanes_below(word);
        for (u32 q = 0; q < b / 64u; ++q) rank += A.wave_cnt[q];
        float c = 0.f;
        if (kept) {
            const u32 bit = rank * nbits, i = bit >> 5;
            c = A.C[(__builtin_amdgcn_alignbit(A.pack[i + 1u], A.pack[i], bit & 31u) & (E - 1u)) - 1u];
        }
        if (wt == 0u) {
            const float p = D.Wp[e];
            D.W_out[e] = kept ? p + c : p;
        } else {
            const u32 p = ((const unsigned short *)D.Wp)[e];
            ((unsigned short *)D.W_out)[e] = (unsigned short)(kept ? w16_narrow(w16_widen(p, wt == 2u) + c, wt == 2u) : p);
        }
    }
}

template <bool ONE_WAVE>
__global__ __launch_bounds__(SM) void k_small_codes(Workspace w, GroupParams g) {
    __shared__ SmallShared A;
    const u32 t = blockIdx.x / 3u, which = blockIdx.x % 3u, tid = threadIdx.x;
    const SmallTensor D = small_tensor(w.desc[t]);
    const TState &T = w.st[t];
    const bool good = T.status == 0;
    const u32 len = good ? (u32)(which == 0u ? T.n_w : T.n_o) : 0u;
    float *x = (which == 0u ? w.xw : (which == 1u ? w.xm : w.xv)) + D.elem_off;
    float v[PER];
#pragma unroll
    for (u32 j = 0; j < PER; ++j) v[j] = j * SM + tid < len ? x[j * SM + tid] : 0.f;
    small_codes<ONE_WAVE>(w, g, A, D, which, good, len, v, x, true, (u64 *)(D.blob + (which == 0u ? T.off_cw : (which == 1u ? T.off_cm : T.off_cv))),
                          (const u64 *)(D.blob + EXCP_HEADER + excp_books_bytes((u32)g.nbits)));
}

// Both in one launch, where there are no more streams than compute units: a workgroup a stream, each of which finds out about the
// whole tensor for itself.  The three of a tensor run in any order, so nothing that one writes is read by another: sections of the blob are each
// its own, and W_hat lies apart from all inputs (excp_small_once sees to it).  (A norm vector of 4096 elements: 14.7 and 28.1 us with what lies between them in two launches, 42 in one, 39
// with the iterations' exchange through registers; the call 60.9 -> 57.0.)
template <bool ONE_WAVE>
__global__ __launch_bounds__(SM) void k_small_whole(Workspace w, GroupParams g, TDesc one, u32 single) {
    __shared__ FrontShared F;
    __shared__ SmallShared A;
    const u32 t = blockIdx.x / 3u, which = blockIdx.x % 3u, tid = threadIdx.x;
    const SmallTensor D = single ? small_tensor(one) : small_tensor(w.desc[t]);
    float v[PER];
    bool good;
    u32 len;
    u64 at;
    {
        FrontValues X;
        small_front(D, g, F, X);
        const SmallLayout s = small_layout(F, D, g);
        good = s.status == 0;
        len = good ? (which == 0u ? s.n_w : s.n_o) : 0u;
        at = which == 0u ? s.off_cw : (which == 1u ? s.off_cm : s.off_cv);
        float *to = (float *)A.sorted;
        if (which == 0u) small_compact(F, X.bw, X.d, 0u, to);
        else if (which == 1u) small_compact(F, X.bo, X.m, 16u, to);
        else small_compact(F, X.bo, X.v, 16u, to);
        if (which == 0u) small_outputs(w, D, g, s, F, X);
        __syncthreads();
#pragma unroll
        for (u32 j = 0; j < PER; ++j) v[j] = j * SM + tid < len ? to[j * SM + tid] : 0.f;
    }
    small_codes<ONE_WAVE>(w, g, A, D, which, good, len, v, (which == 0u ? w.xw : (which == 1u ? w.xm : w.xv)) + D.elem_off, false, (u64 *)(D.blob + at), F.bw);
}

}  // namespace

void launch_small(const Workspace &w, const GroupParams &g, const TDesc *single, bool once, hipStream_t s) {
    const bool few = g.K <= 63;
    if (once) {
        if (few) hipLaunchKernelGGL(k_small_whole<true>, dim3(3u * g.ntensors), dim3(SM), 0, s, w, g, single ? *single : TDesc{}, single ? 1u : 0u);
        else hipLaunchKernelGGL(k_small_whole<false>, dim3(3u * g.ntensors), dim3(SM), 0, s, w, g, single ? *single : TDesc{}, single ? 1u : 0u);
        return;
    }
    hipLaunchKernelGGL(k_small_front, dim3(g.ntensors), dim3(SM), 0, s, w, g, single ? *single : TDesc{}, single ? 1u : 0u);
    if (few) hipLaunchKernelGGL(k_small_codes<true>, dim3(3u * g.ntensors), dim3(SM), 0, s, w, g);
    else hipLaunchKernelGGL(k_small_codes<false>, dim3(3u * g.ntensors), dim3(SM), 0, s, w, g);
}

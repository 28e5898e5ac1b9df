// Tables that groups of tensors share: rows of bucket counts, and the cells inside buckets; and the cell of a value.  Compiled
// and run by tests/test_host_tables.py with the rules of excp_device.h; needs no GPU.
#include <math.h>
#include <stdio.h>

#include <algorithm>
#include <vector>

#include "../paper_2406_11257_amd/csrc/excp_device.h"

static int fails = 0;
static const u32 GROUP = 1024;                            // tensors that a group takes
#define CHECK(c, ...) do { if (!(c)) { printf("FAIL line %d: %s: ", __LINE__, #c); printf(__VA_ARGS__); printf("\n"); ++fails; } } while (0)

int main() {
    u64 seed = 1;
    auto random = [&]() { seed = seed * 6364136223846793005ull + 1442695040888963407ull; return (u32)(seed >> 33); };
    // Every group that a context takes has rows enough, whatever survives, and no batch of the gather pass spans three units.
    for (u32 cus : {64u, 256u, 304u})
        for (u64 G : {4096ull, 100000ull, 16777216ull, 25165843ull, 405334016ull, 3400000000ull})
            for (u32 tensors : {1u, 2u, 76u, 292u, 1024u})
                for (u64 elems : {(u64)tensors, G / 7 + tensors, G}) {
                    if (elems > G) continue;
                    const u32 ntiles = (u32)(elems / EXCP_TILE + tensors), subs = excp_gather_subs(ntiles, cus);
                    const u64 have = excp_count_rows(G, GROUP);
                    const u32 s = excp_unit_shift(elems, tensors, subs, cus, have);
                    u64 need = 0;                                     // tensors of one element each but the last
                    need += 3ull * (tensors - 1) + 3 * ((elems - (tensors - 1) + (1ull << s) - 1) >> s);
                    CHECK(need <= have, "%llu rows of %llu: %llu elements, %u tensors, 2^%u", need, have, elems, tensors, s);
                    CHECK(s >= 14 && s <= EXCP_UNIT_SHIFT && (u64)subs * 2048 <= 1ull << s && subs >= 4 && subs % 4 == 0, "2^%u, %u sub-tiles", s, subs);
                }
    // A group that is known to keep whole streams sets out for cells only if they are not too many and buckets a third above the
    // average fit; a single tensor without a known share, up to the largest of the rule.
    for (u64 n : {131072ull, 1500000ull, 1700000ull, 2097152ull, 2097153ull, 7000000ull, 8000000ull, 16777216ull, 26214400ull, 26214401ull})
        for (u32 count : {1u, 3u, 40u})
            for (u32 whole = 0; whole <= 3; ++whole) {
                const bool fits = n / 256 * 4 / 3 <= excp_cells_most(excp_fine_size(n)), want = n * count <= 26214400ull && (!whole || (fits && whole * n * count <= 33554432ull));
                CHECK(excp_fine_group(n * count, n, whole) == want, "%u tensors of %llu elements, %u whole streams", count, n, whole);
            }
    // The groups whose blobs test_gpu_cells_many.py compares set out for cells, and do not with a tensor beside them that is too large.
    struct Sizes { std::vector<u64> n; u32 nbits; };
    for (const Sizes &x : {Sizes{{13500001, 14600003}, 4}, Sizes{{9000001, 8500077, 11000000, 9999999}, 3}, Sizes{std::vector<u64>(5, 6000005), 6},
                           Sizes{std::vector<u64>(12, 3000401), 8}, Sizes{{131071, 131073, 20000001, 25ull << 20}, 7}}) {
        u64 elems = 0, largest = 0;
        for (u64 n : x.n) { elems += n; largest = std::max(largest, n); }
        const u32 count = (u32)x.n.size(), K = (1u << x.nbits) - 1u;
        CHECK(elems > EXCP_FINE_LARGEST && excp_cells_group(elems, largest, count, K, 0) && !excp_cells_group(elems, largest, count, K, 3), "%u tensors, %llu elements", count, elems);
        CHECK(!excp_cells_group(elems + 28000003, 28000003, count + 1, K, 0), "%u tensors and a larger one", count);
        CHECK(elems / 2 <= (u64)excp_cells_chunks(elems) * EXCP_CHUNK, "half of %llu elements", elems);
    }
    // A third of the largest tensor kept, its buckets fit the workgroups also where they are four deviations above the average.
    for (u64 n = 131072; n <= EXCP_FINE_LARGEST; n += n / 50) {
        const u32 samples = excp_samples(true, n);
        const double largest = (double)n / 3 / 256 * (1 + 4 / sqrt(samples / 256.0));
        CHECK(largest <= excp_cells_most(excp_fine_size(n)) && excp_samples(false, n) == EXCP_SAMPLES_FEW && samples <= EXCP_SAMPLES_MANY, "%llu elements, %u samples: %g", n, samples, largest);
    }
    // No two buckets' entries in the cell tables overlap, and none lies outside; nor does a tensor's survivor area.  Areas begin on
    // multiples of 64 elements, for which a context of G elements has 63 a tensor more.
    for (u32 shape = 0; shape < 44; ++shape) {
        const bool many = shape >= 40;                    // as many tensors as a group takes, all of odd length
        const u32 tensors = many ? GROUP : (shape % 4 == 0 ? 1u : 1u + random() % 90u);
        std::vector<u64> n(tensors);
        u64 G = 0;
        for (auto &x : n) { x = many ? 1u + 64u * (random() % (shape == 43 ? 3u : 300u)) : 1 + random() % (shape % 3 == 0 ? 300u : 400000u); G += x; }
        const u64 area = excp_survivor_elems(G, GROUP), words = excp_fine_words(area, GROUP);
        u64 elem_off = 0, end = 0;
        for (u32 t = 0; t < tensors; ++t) {
            CHECK(elem_off % 64 == 0 && elem_off + n[t] <= area, "tensor %u at %llu + %llu of %llu", t, elem_off, n[t], area);
            const u32 len = shape % 2 ? (u32)n[t] : (u32)(n[t] / 3);
            std::vector<u32> cut{0u, len};
            for (u32 b = 1; b < 256; ++b) cut.push_back(shape % 5 == 0 ? len : random() % (len + 1));
            std::sort(cut.begin(), cut.end());
            for (u32 b = 0; b < 256; ++b) {
                const u32 size = cut[b + 1] - cut[b];
                if (size < 256) continue;
                const u32 lg = excp_fine_cells_log2(size);
                const u64 at = excp_fine_at(elem_off, t, cut[b], b);
                CHECK(at >= end && at + (1u << lg) + 1 <= words, "tensor %u bucket %u at %llu, the last ended at %llu of %llu", t, b, at, end, words);
                CHECK(lg >= 1 && lg <= 9 && (size >> lg) >= 64 && (lg == 9 || (size >> lg) < 128), "%u values in 2^%u cells", size, lg);
                end = at + (1u << lg) + 1;
            }
            elem_off += excp_area_elems(n[t]);
        }
    }
    // The cell that a value is filed in is the one that a border of the same key is looked up in, inside the table, and higher for
    // higher values: buckets of one sign, of both, with zeros of either sign beside them, of nothing but zeros.
    for (u32 shape = 0; shape < 600; ++shape) {
        std::vector<u32> bits;                            // of the bucket's values
        const u32 low = shape % 7 == 0 ? random() % 1000u : (1u + random() % 230u) << 23 | (random() & 0x7fffffu), orders = 1u + random() % 10u;
        const u32 signs = shape % 3, zeros = shape / 3 % 4, count = shape % 11 == 0 ? 0u : 300u;      // signs: +, -, both; zeros: none, +0, -0, both
        for (u32 i = 0; i < count; ++i) bits.push_back((low + random() % (orders << 23)) | (signs == 1 || (signs == 2 && i % 2) ? 0x80000000u : 0u));
        if (zeros & 1u) bits.push_back(0u);
        if (zeros & 2u) bits.push_back(0x80000000u);
        if (bits.empty()) continue;
        auto key = [](u32 b) { return b >> 31 ? ~b : b | 0x80000000u; };
        std::sort(bits.begin(), bits.end(), [&](u32 a, u32 b) { return key(a) < key(b); });
        const u32 kmin = key(bits.front()), kmax = key(bits.back());
        u32 mag = 0;
        for (u32 b : bits) if (b & 0x7fffffffu) mag = mag ? std::min(mag, b & 0x7fffffffu) : b & 0x7fffffffu;
        if (kmin >= kmax) continue;
        // places on a line without the gap: magnitudes count from the smallest one, zero lies between the signs
        auto place = [&](u32 b) -> long long {
            const long long a = (long long)(b & 0x7fffffffu) - mag + 1;
            return (b & 0x7fffffffu) || !mag ? (b >> 31 ? -a : a) : 0;
        };
        for (u32 lg = 1; lg <= 9; ++lg) {
            const CellMap M = excp_cell_map(kmin, kmax, mag, lg);
            const unsigned long long range = (unsigned long long)(place(bits.back()) - place(bits.front()));
            u32 shift = 0, last = 0;
            while (range >> shift >> lg) ++shift;
            CHECK(M.shift == shift, "shape %u, 2^%u cells: shift %u, not %u", shape, lg, M.shift, shift);
            for (u32 b : bits) {
                const u32 in = excp_cell_of_bits(M, b), want = (u32)((unsigned long long)(place(b) - place(bits.front())) >> shift);
                CHECK(in == want && in < 1u << lg && in >= last && excp_cell_of_key(M, key(b)) == want, "shape %u, value %08x: cell %u of 2^%u, not %u", shape, b, in, lg, want);
                last = in;
            }
        }
    }
    if (fails) return 1;
    printf("ok\n");
    return 0;
}

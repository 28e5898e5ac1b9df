// Tables that groups of tensors share: rows of bucket counts, and the cells inside buckets.  Compiled and run by
// tests/test_host_tables.py with the rules of excp_device.h; needs no GPU.
#include <stdio.h>

#include <algorithm>
#include <vector>

#include "../paper_2406_11257_amd/csrc/excp_device.h"

static int fails = 0;
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
                    const u64 have = excp_count_rows(G, 1024);
                    const u32 s = excp_unit_shift(elems, tensors, subs, cus, have);
                    u64 need = 0;                                     // tensors of one element each but the last
                    need += 3ull * (tensors - 1) + 3 * ((elems - (tensors - 1) + (1ull << s) - 1) >> s);
                    CHECK(need <= have, "%llu rows of %llu: %llu elements, %u tensors, 2^%u", need, have, elems, tensors, s);
                    CHECK(s >= 14 && s <= EXCP_UNIT_SHIFT && (u64)subs * 2048 <= 1ull << s && subs >= 4 && subs % 4 == 0, "2^%u, %u sub-tiles", s, subs);
                }
    // No two buckets' entries in the cell tables overlap, and none lies outside.
    for (u32 shape = 0; shape < 40; ++shape) {
        const u32 tensors = shape % 4 == 0 ? 1u : 1u + random() % 90u;
        std::vector<u64> n(tensors);
        u64 G = 0;
        for (auto &x : n) { x = 1 + random() % (shape % 3 == 0 ? 300u : 400000u); G += x; }
        const u64 words = excp_fine_words(G, 1024);
        u64 elem_off = 0, end = 0;
        for (u32 t = 0; t < tensors; ++t) {
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
            elem_off += n[t];
        }
    }
    if (fails) return 1;
    printf("ok\n");
    return 0;
}

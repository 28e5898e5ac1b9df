// What is handed out of a context's workspace, against what is allocated, and how evenly.  Compiled and run by
// tests/test_host_sizes.py with the rules of excp_device.h; needs no GPU.
#include <stdio.h>

#include "../paper_2406_11257_amd/csrc/excp_device.h"

static int fails = 0;
#define CHECK(c, ...) do { if (!(c)) { printf("FAIL line %d: %s: ", __LINE__, #c); printf(__VA_ARGS__); printf("\n"); ++fails; } } while (0)

int main() {
    // Median candidates: groups as full as they get, in a context of exactly their size, at the list length the library
    // begins with and at ones a caller may set.
    for (u64 per : {1ull << 20, 1ull << 26, 65536ull, 1000ull, 1ull})
        for (u64 n0 : {1ull, 4096ull, 100000ull, 1048572ull, 2097152ull, 2097156ull, 4194304ull, 8388608ull})
            for (u64 step : {0ull, 1ull, 11ull}) {
                u64 elems = 0, used = 0;
                for (u32 q = 0; q < 1024; ++q) {
                    const u64 n = n0 + step * (q % 12);
                    const u32 lists = excp_cand_lists(n, per);
                    const u64 cap = excp_cand_cap(n, lists);
                    CHECK(lists >= 1 && lists <= 16 && cap % lists == 0 && cap / lists > 0, "%u lists of %llu", lists, cap);
                    elems += n; used += cap;
                }
                CHECK(used <= excp_cand_words(elems, 1024), "%llu of %llu (n %llu, %llu to a list)", used, excp_cand_words(elems, 1024), n0, per);
            }
    // The lists that consecutive workgroups try first: every list by as many of them.
    for (u32 lists = 1; lists <= 16; ++lists) {
        u32 first[16] = {0}, least = ~0u, most = 0;
        for (u32 b = 100; b < 100 + 64 * lists; ++b) ++first[excp_cand_first(b, lists)];
        for (u32 j = 0; j < lists; ++j) { least = first[j] < least ? first[j] : least; most = first[j] > most ? first[j] : most; }
        CHECK(least == 64 && most == 64, "%u lists: %u to %u", lists, least, most);
    }
    // The runs of the statistics pass: within the records that the workspace has, and of the largest tensor no more than it gains from.
    for (u32 cus : {80u, 256u, 304u})
        for (u64 largest : {1ull, 9000ull, 16777216ull, 100000000ull, 400000000ull, 2147479552ull})
            for (u64 others : {0ull, 1ull, 9000ull, 16777216ull, 1000000000ull, 20000000000ull}) {
                const u32 tiles = (u32)((largest + EXCP_TILE - 1) / EXCP_TILE), all = tiles + (u32)(others / EXCP_TILE);
                const u64 runs = excp_stats_grid(all, largest, cus);
                CHECK(runs >= 8u * cus && runs <= EXCP_STATS_PER_CU * cus, "%llu runs", runs);
                CHECK(runs * tiles / all <= (tiles / 24u > 8u * cus ? tiles / 24u : 8u * cus), "%llu runs, %u of %u tiles", runs, tiles, all);
                if (others >= 16u * largest && all / 6u >= EXCP_STATS_PER_CU * cus) CHECK(runs == EXCP_STATS_PER_CU * cus, "%llu runs", runs);
            }
    // The units of a Lloyd iteration: never more than the launch has workgroups, and one round of them for few streams.
    u64 seed = 1;
    auto random = [&]() { seed = seed * 6364136223846793005ull + 1442695040888963407ull; return (u32)(seed >> 33); };
    for (u32 at_once : {256u, 512u, 304u})
        for (u32 least : {4096u, 8192u})
            for (u32 slots : {1u, 2u, 40u, 85u, 86u, 171u, 341u, 1024u})
                for (u32 shape = 0; shape < 12; ++shape) {
                    static u32 x[3072];
                    u64 work = 0, units = 0;
                    u32 streams = 0;
                    for (u32 s = 0; s < 3 * slots; ++s) {
                        const u32 r = random();
                        x[s] = shape == 0 ? 1u : shape == 1 ? 0xffffffffu : shape == 2 ? (s ? 0u : 0xffffffffu) : shape == 3 ? least + 1u : shape == 4 ? (s ? 1u : 0xffffffffu)
                               : shape == 5 ? s % 3u == 0u ? 24577u : 0u : r >> (r % 31u);
                        work += x[s]; streams += x[s] != 0;
                    }
                    if (!streams) continue;
                    const u64 unit = excp_lloyd_unit(work, streams, at_once, least);
                    for (u32 s = 0; s < 3 * slots; ++s) units += (x[s] + unit - 1) / unit;
                    CHECK(unit >= least && units >= streams && units <= excp_lloyd_grid(at_once, slots), "%llu units, %u slots, shape %u", units, slots, shape);
                    CHECK(units <= (2 * streams <= at_once ? at_once : 2u * streams), "%llu units, %u streams, %u at once", units, streams, at_once);
                }
    // Small tensors in one launch: only where no W_hat lies over anything that the launch reads, by an interval test of every pair.
    u32 both[2] = {0, 0};
    for (u32 weight_bytes : {2u, 4u})
        for (u32 shape = 0; shape < 4000; ++shape) {
            static TDesc d[90];
            const u32 count = shape % 3u == 0u ? 1u : 1u + random() % 88u, cus = random() % 8u ? 256u : 80u;
            const u32 mode = shape / 3u % 5u;             // apart, in place, over W_t, in place for one, anywhere
            const uintptr_t base = 1ull << 40, step = 8192 * 4;
            for (u32 q = 0; q < count; ++q) {
                TDesc &D = d[q];
                D = TDesc{};
                D.n = random() % 16u ? 1u + random() % 8192u : 0u;
                auto place = [&](u32 i) { return (float *)(base + (5u * q + i) * step); };        // (arrays of all kinds side by side)
                D.Wp = place(0); D.W = place(1); D.m = place(2); D.v = place(3); D.W_out = place(4);
                if (mode == 1u || (mode == 3u && q == count / 2u)) D.W_out = (float *)D.Wp;
                if (mode == 2u) D.W_out = (float *)D.W;
                if (mode == 4u) D.W_out = (float *)(base + random() % (5u * count * step) / 2u * 2u);
                if (random() % 4u == 0u) D.W_out = nullptr;
            }
            bool apart = true;
            for (u32 q = 0; q < count; ++q)
                for (u32 r = 0; r < count && d[q].W_out; ++r) {
                    const void *in[4] = {d[r].Wp, d[r].W, d[r].m, d[r].v};
                    for (u32 k = 0; k < 4u; ++k) {
                        const uintptr_t a = (uintptr_t)d[q].W_out, b = (uintptr_t)in[k];
                        if (d[q].n && d[r].n && a < b + d[r].n * (k < 2u ? weight_bytes : 4u) && b < a + d[q].n * weight_bytes) apart = false;
                    }
                }
            const bool once = excp_small_once(d, count, cus, weight_bytes);
            CHECK(once == (apart && 3u * count <= cus), "%u tensors, mode %u, %u compute units", count, mode, cus);
            ++both[once];
        }
    CHECK(both[0] > 1000 && both[1] > 1000, "%u in two launches, %u in one", both[0], both[1]);
    if (fails) return 1;
    printf("ok\n");
    return 0;
}

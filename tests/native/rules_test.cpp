// Host checks of the rules that choose launch shapes and kernels
// (paper_1810_11966_amd/csrc/trig_rules.hpp).  Built with g++ by
// tests/test_rules.py and run on the CPU.
#include <cstdio>
#include <initializer_list>

#include "trig_rules.hpp"

using namespace trig_rules;

static long failures = 0;
#define CHECK(c)                                                     \
    do {                                                             \
        if (!(c)) {                                                  \
            if (failures < 20) std::printf("FAIL %s:%d: %s\n", __FILE__, __LINE__, #c); \
            ++failures;                                              \
        }                                                            \
    } while (0)

static const int kCus = 256;

// Every shape is one that a kernel exists for, and given values stay.
static void test_shapes() {
    for (int n : {1, 3, 100, 1000, 4096, 4097, 8000, 25000, 100000, 1000000, 20000000})
        for (int hits : {0, 1, 9, 45, 54, 90, 109, 270, 360, 450, 3000}) {
            const long long all = (long long)n * hits;
            if (all > 2000000000ll) continue;
            for (bool stealing : {false, true}) {
                const BlockShape s = choose_block_shape(0, 0, 0, stealing, n, (int)all, kCus);
                CHECK(s.hb == 2048 || s.hb == 4096);
                CHECK(s.nw == 4 && s.eb >= 1 && s.eb <= kMaxEvents);
                // a block of average events fits, if it has more than one event per wave
                CHECK(s.eb <= 4 || s.eb * (double)hits <= s.hb);
                for (int hb : {1024, 2048, 4096})
                    for (int nw : {1, 2, 4})
                        for (int eb : {1, 7, 128}) {
                            const BlockShape g = choose_block_shape(hb, nw, eb, stealing, n, (int)all, kCus);
                            CHECK(g.hb == hb && g.nw == nw && g.eb == eb);
                        }
                const BlockShape h = choose_block_shape(1024, 0, 0, stealing, n, (int)all, kCus);
                CHECK(h.hb == 1024 && h.nw == 2 && h.eb <= kMaxEvents);
            }
        }
}

// Small batches: without stealing their blocks are spread over the CUs; with
// stealing there are no more of them than CUs (its claims pass one counter).
static void test_small_batches() {
    const auto blocks = [](const BlockShape& s, int n) { return (n + s.eb - 1) / s.eb; };
    for (int n : {1000, 4000, 8000, 16000})
        for (int hits : {9, 24, 45}) {
            const BlockShape p = choose_block_shape(0, 0, 0, false, n, n * hits, kCus);
            const BlockShape s = choose_block_shape(0, 0, 0, true, n, n * hits, kCus);
            CHECK(blocks(p, n) >= n / 8 || blocks(p, n) > 4 * kCus);
            CHECK(blocks(s, n) <= kCus || s.eb * (double)hits > 0.5 * s.hb);
        }
    // (4,000 events of 15 hits per layer: a block per CU)
    CHECK(choose_block_shape(0, 0, 0, true, 4000, 4000 * 45, kCus).eb == 16);
    // few large events in all: blocks that hold four with room to spare
    CHECK(choose_block_shape(0, 0, 0, false, 600, 600 * 450, kCus).hb == 4096);
    CHECK(choose_block_shape(0, 0, 0, false, 100000, 100000 * 450, kCus).hb == 2048);
    // stealing: 4096 where they fill the CUs
    CHECK(choose_block_shape(0, 0, 0, true, 100000, 100000 * 75, kCus).hb == 4096);
    CHECK(choose_block_shape(0, 0, 0, true, 8000, 8000 * 75, kCus).hb == 2048);
    CHECK(choose_block_shape(0, 0, 0, true, 40000, 40000 * 420, kCus).hb == 4096);
    // not quite full while a CU has few of them: heavy events may lie together
    CHECK(choose_block_shape(0, 0, 0, true, 300000, 300000 * 44, kCus).eb == 48);
    CHECK(choose_block_shape(0, 0, 0, true, 1000000, 1000000 * 90, kCus).eb == 40);
    // or where events are few and large, four or eight at a time
    for (int n : {300, 1900, 4000, 20000})
        for (int hits : {300, 450}) {
            const BlockShape s = choose_block_shape(0, 0, 0, true, n, n * hits, kCus);
            CHECK(s.hb == 4096 && s.nw == 4 && s.eb == (n <= 4096 || hits > 307 ? 4 : 8));
        }
    CHECK(choose_block_shape(0, 0, 0, true, 100000, 100000 * 600, kCus).hb == 4096);
}

// Per-hit z: a wave per event for arrays off a 16-byte boundary, small batches
// and large events.
static void test_blocks_z() {
    for (bool window : {false, true}) {
        CHECK(!blocks_z(false, window, 1000000, 1000000 * 24));
        CHECK(blocks_z(true, window, 1000000, 1000000 * 24));
        CHECK(blocks_z(true, window, 1000000, 1000000 * 90));
        CHECK(!blocks_z(true, window, 3000, 3000 * 90));
        CHECK(!blocks_z(true, window, 100000, 100000 * 300));
    }
    CHECK(blocks_z(true, false, 20000, 20000 * 180) && !blocks_z(true, false, 10000, 10000 * 180));
    CHECK(blocks_z(true, true, 80000, 80000 * 90) && !blocks_z(true, true, 40000, 40000 * 90));
}

// Station filter: no workgroup sums more totals than it is worth, and one or
// two events per wave always go with the sums.
static void test_filter_shape() {
    for (int n : {1, 6143, 6144, 6145, 8192, 8193, 12288, 12289, 16384, 32768, 32769, 49152, 49153, 2000000000})
        for (int64_t hits : {0, 10, 999, 1000, 5000}) {
            const FilterShape f = filter_shape(n, hits * n);
            const int64_t blocks = (n + (int64_t)f.per * 4 - 1) / ((int64_t)f.per * 4);
            CHECK(f.per == (n <= (hits >= 1000 ? 8192 : 6144) ? 1 : n <= 12288 || (hits >= 1000 && n <= 32768) ? 2 : 4));
            CHECK(f.self ? blocks <= 4096 : f.per == 4 && n > 49152);
        }
    CHECK(filter_shape(0, 0).per == 1);
}

int main() {
    test_shapes();
    test_filter_shape();
    test_blocks_z();
    test_small_batches();
    if (failures) {
        std::printf("%ld checks failed\n", failures);
        return 1;
    }
    std::printf("all checks passed\n");
    return 0;
}

// Host checks of the batched form's prefilter bound and of the binned form's
// cells (paper_1810_11966_amd/csrc/trig_bounds.hpp: direct_bounds, direct_pre,
// cell_scale).  Built with g++ -ffp-contract=off by tests/test_prefilter.py and run on the
// CPU (x86-64 SSE binary32 arithmetic, round to nearest even, subnormals
// kept).
//
// Pairs (c0, c1) built to pass the pair test or to sit on its edge, at
// coordinate scales from subnormal to the largest binary32 and layer
// positions whose ratio spans the bound's range and more: every pair that
// passes has a score within direct_pre for M = max(|c0|, |c1|), in both
// orientations.
//
// Keys and intervals up to the ends of binary32: the cells of the interval's
// ends enclose the cell of every key inside it.
#include <algorithm>
#include <cfloat>
#include <cmath>
#include <cstdio>
#include <random>

#include "trig_bounds.hpp"

using namespace trig_host;

static long failures = 0;
#define CHECK(c)                                                     \
    do {                                                             \
        if (!(c)) {                                                  \
            if (failures < 20) std::printf("FAIL %s:%d: %s\n", __FILE__, __LINE__, #c); \
            ++failures;                                              \
        }                                                            \
    } while (0)

// The scan's score of one plane with layer `lane` (0 or 1) in the lanes.
static float score(const DirectBounds& d, int orientation, float c0, float c1) {
    const float cB = orientation ? c1 : c0, cL = orientation ? c0 : c1;
    volatile float p = d.k[orientation] * cL;
    volatile float s = cB + p;
    return std::fabs((float)s);
}

static long passes = 0, infinite = 0;  // pairs; infinite ones of their two bounds each

static void check_pair(const DirectBounds& d, float pre, float c0, float c1) {
    const float M = std::max(std::fabs(c0), std::fabs(c1));
    ++passes;
    for (int o = 0; o < 2; ++o) {
        const float s = score(d, o, c0, c1), bound = direct_pre(pre, d.scale[o], d.slack[o], M);
        infinite += std::isinf(bound);
        // the kernel takes the event on unless every score is above the bound
        CHECK(s <= bound);
    }
}

static void test_direct_bounds() {
    std::mt19937_64 rng(4711);
    std::uniform_real_distribution<double> U(-1.0, 1.0);
    const double zs[] = {400.0, 410.0, 465.54053, 409.91873, 1.0, 3.0, 1e-3, 1e-10, 1e10, 1e17, 1e18, 1e19, 1e-18, 3e38, 1e-38};
    const double scales[] = {1e-44, 1e-38, 1e-20, 1.0, 200.0, 1e6, 1e20, 1e30, 1e37, 1e38, 3.4e38};
    for (double z0 : zs)
        for (double z1 : zs) {
            const float f0 = (float)z0, f1 = (float)z1;
            const DirectBounds dw = direct_bounds(1.0 / (double)f0, -1.0 / (double)f1);
            const Basis K = basis(f0, f1, 420.0f);
            const DirectBounds db = direct_bounds(K.U0, K.U1);
            for (double scale : scales)
                for (int it = 0; it < 400; ++it) {
                    // one line through the vertex, its larger hit near `scale`
                    const double m = scale / std::max(z0, z1) * (it % 3 ? 1.0 + 0.02 * U(rng) : U(rng));
                    const double off = it % 2 ? 0.0 : scale * 1e-6 * U(rng);
                    const auto clip = [](double v) { return (float)std::max(-(double)FLT_MAX, std::min((double)FLT_MAX, v)); };
                    const float c0 = clip(m * z0), c1 = clip(m * z1 + off);
                    // window test: the smallest windows that the pair passes, and wide ones
                    volatile float s0 = c0 / f0, s1 = c1 / f1;
                    volatile float dv = s1 - s0;
                    const float diff = std::fabs((float)dv);
                    for (float w : {std::nextafter(diff, INFINITY), 2.0f * diff, 1.0f, FLT_MAX})
                        if (diff < w && std::isfinite(w)) check_pair(dw, w, c0, c1);
                    // basis form: |a| <= beta
                    volatile float p0 = K.U0 * c0, p1 = K.U1 * c1;
                    volatile float av = p0 + p1;
                    const float a = std::fabs((float)av);
                    for (float b : {a, 2.0f * a, 0.25f, 1e19f})
                        if (a <= b && std::isfinite(b)) check_pair(db, b, c0, c1);
                }
        }
    // The pair of FLT_MAX whose scaled product overflows.
    const DirectBounds d = direct_bounds(1.0 / (double)465.54053f, -1.0 / (double)409.91873f);
    check_pair(d, 0.005f, FLT_MAX, 2.9962613e38f);
    // The bound prunes at ordinary coordinates: close to the pair test's own.
    const DirectBounds n = direct_bounds(1.0 / 400.0, -1.0 / 410.0);
    for (int o = 0; o < 2; ++o)
        CHECK(direct_pre(0.005f, n.scale[o], n.slack[o], 400.0f) < 1.001f * 0.005f * (o ? 410.0f : 400.0f));
    std::printf("direct bounds: %ld passing pairs, %ld infinite bounds\n", passes, infinite);
    CHECK(2 * passes - infinite > 1000000);
}

// The kernel's cell of a value (its conversion truncates and saturates, NaN
// and negative values give 0).
static uint32_t cell(float v, float scale) {
    volatile float p = v * scale;
    volatile float t = p + 128.0f;
    if (!((float)t > 0.0f)) return 0;
    return (float)t >= 256.0f ? 255u : (uint32_t)(float)t;
}

static void test_cells() {
    std::mt19937_64 rng(99);
    std::uniform_real_distribution<double> U(-1.0, 1.0);
    const double Ks[] = {0.0, 1e-45, 1e-40, 1.2e-38, 1e-20, 0.45, 300.0, 1e20, 8e37, 9e37, 1.7e38, 3.4e38, INFINITY};
    const float big = FLT_MAX, inf = INFINITY;
    long checked = 0;
    for (double Kd : Ks) {
        const float K = (float)Kd;
        // the reciprocal as it is, and flushed to 0 or overflowing
        for (float rcp : {1.0f / K, 0.0f, inf}) {
            const float scale = cell_scale(K, rcp, 256.0f);
            CHECK(std::isfinite(scale) && scale > 0.0f);
            for (int it = 0; it < 3000; ++it) {
                const float key = it % 9 ? (float)std::max(-(double)big, std::min((double)big, Kd * U(rng))) : 0.0f;
                const float radius[] = {0.0f, 1e-45f, 1e-38f, (float)(std::min(Kd, 1e37) * std::fabs(U(rng))), 3e38f, big, inf};
                for (float r : radius)
                    for (float mid : {key, (float)(key * (1.0 + 1e-3 * U(rng))), 0.0f, big, -big, (float)(3e38 * U(rng))}) {
                        volatile float lo = mid - r, hi = mid + r;
                        if (!(std::isfinite(key) && (float)lo <= key && key <= (float)hi)) continue;
                        ++checked;
                        CHECK(cell((float)lo, scale) <= cell(key, scale) && cell(key, scale) <= cell((float)hi, scale));
                    }
            }
        }
    }
    // keys spread over the cells
    const float s = cell_scale(200.0f, 1.0f / 200.0f, 256.0f);
    CHECK(cell(-200.0f, s) == 0 && cell(-100.0f, s) == 64 && cell(0.0f, s) == 128 && cell(199.0f, s) == 255);
    std::printf("cells: %ld keys in intervals\n", checked);
    CHECK(checked > 100000);
}

int main() {
    test_direct_bounds();
    test_cells();
    if (failures) {
        std::printf("%ld checks failed\n", failures);
        return 1;
    }
    std::printf("all checks passed\n");
    return 0;
}

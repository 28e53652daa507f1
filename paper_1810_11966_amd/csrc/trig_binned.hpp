// Slope-cell binned selection (the binned form) for high-multiplicity events.
//
// The count is the brute-force one (paper Sec. 3.2 steps 1-3) in the binary32
// contract of include/trig.h.  Instead of scanning every (i, j) pair, each
// layer-1 hit is put into a cell by a key that is proportional to its slope
// x/z, and each layer-0 hit looks only at the cells that can hold a partner:
//
//   MSD tests: a triplet passes only if |a| <= A in both planes and
//     |b| <= B in the x-z plane (see the batched form; MSD_BASIS: A = B = beta,
//     MSD: A = a0 + a1 M and B = b0 + b1 M with M the event's largest layer-1
//     |x|, |y|), a = f32(u + v) with u = f32(U0 x_i), v = f32(U1 x_j).  As
//     binary32 rounding is monotone and A_up >= next float above A,
//     |f32(u + v)| <= A implies -A_up < u + v < A_up in real numbers,
//     so v lies in (-u - A_up, -u + A_up).  The layer-1 key is v.  In
//     the same way b = f32(p + w_k) with p = f32(V0 x_i + V1 x_j) and
//     w_k = f32(V2 x_k) needs w_k in (-p - B_up, -p + B_up); the
//     layer-2 key is w_k.
//   window test: |f32(s_j - s_i)| < W implies |s_j - s_i| < W (W is a binary32
//     value), so s_j lies in (s_i - W, s_i + W); the same for s_k.  Here the
//     layer-2 condition depends on i alone, so an i's count is the product of
//     its numbers of layer-1 and layer-2 partners.
//
// The interval ends are rounded outwards (by at least one binary32 step
// past the rounded end point), and the cell of a key is a non-decreasing
// function of the key, so the cells from cell(lower end) to cell(upper end)
// contain every key in the interval whatever the cell width.  Every
// candidate then gets the full binary32 test, so the count is exact; a hit
// whose key is not finite can never pass (its a or b is infinite or NaN) and
// is left out.
//
// The pairs that pass their test are listed, and only an event with such a
// pair reads its layer 2 (wave_event_binned): a few pairs are completed
// against all of it, more look their partners up in layer-2 cells.  Events
// whose bounds let too many pairs through for the list have both layers in
// cells and list none.
//
// One wave per event.  Cells are built in LDS with a counting sort (histogram
// of the cell indices, exclusive scan, scatter); events with more than
// kBinCap hits in layer 1 or 2 take the batched form's pair-pruned path from
// HBM instead.
#pragma once

#include "trig_block.hpp"
#include "trig_device.hpp"

namespace trig {

constexpr int kBinCap = 256;            // layer-1 / layer-2 hits per event in LDS
constexpr int kBinRounds = kBinCap / kWave;

// f moved outwards by d = f32(f32(|f| 2^-22) + 2^-126), at least one binary32
// step for any finite f (a step is at most 2^-23 |f| for normal f and 2^-149
// below), so that the result lies beyond every real number that rounds to f
// (those lie within 2^-24 |f| + 2^-150 of it): the rounding of the sum and
// of the final subtraction stay far below the slack d leaves.  Infinities
// stay infinite (+inf - inf is NaN, which the cell function maps to cell 0:
// still a superset).  Three vector instructions, no branch.
__device__ __forceinline__ float widen_down(float f) {
    return f - (__builtin_fabsf(f) * 0x1p-22f + 0x1p-126f);
}
__device__ __forceinline__ float widen_up(float f) {
    return f + (__builtin_fabsf(f) * 0x1p-22f + 0x1p-126f);
}


// Surviving pairs of an event that its list holds (wave_event_binned).
constexpr int kBinPairs = 128;

// LDS of one wave: cell ends and the two payload floats per hit, in cell
// order: first the layer-1 cells in a1/b1 and the surviving pairs (x_i, y_i,
// x_j, y_j), then the layer-2 cells in a1/b1 with the pairs or, where both
// layers are needed in cells, layer 1 in a2/b2.  Float arrays first (16-byte
// aligned: the fallback path reuses a1/b1 as its layer-0 buffers).  A cell end
// is at most kBinCap = 256, so the ends are 16-bit, two cells per 32-bit word
// (cell t in the half t & 1 of word t >> 1): 5 KB per wave, eight workgroups
// per CU.
struct BinLds {
    float a1[kBinCap], b1[kBinCap];
    union {
        float4 pairs[kBinPairs];
        struct {
            float a2[kBinCap], b2[kBinCap];
        };
    };
    // Cell ends of a1/b1 and of a2/b2 (kBinCap / 2 words each); or, while pairs
    // are listed, the layer-1 cells' starts (starts()), and the number of
    // surviving pairs in the last word.
    uint32_t ends[kBinCap];
    __device__ __forceinline__ uint32_t* end1() { return ends; }
    __device__ __forceinline__ uint32_t* end2() { return ends + kBinCap / 2; }
    __device__ __forceinline__ const uint32_t* end1() const { return ends; }
    __device__ __forceinline__ const uint32_t* end2() const { return ends + kBinCap / 2; }
    __device__ __forceinline__ uint16_t* starts() { return reinterpret_cast<uint16_t*>(ends); }
    __device__ __forceinline__ uint32_t* n_pairs() { return ends + kBinCap - 1; }
};
static_assert(kBinCap < 65536, "cell ends fit in 16 bits");

// Cell t's 16-bit entry of a packed end array.
__device__ __forceinline__ int cell_end(const uint32_t* end, int t) {
    return (int)reinterpret_cast<const uint16_t*>(end)[t];
}

// Cells over [kmin, kmax] of one layer.  cell(v) is non-decreasing in v
// (binary32 subtraction, multiplication and floor are monotone, the clamps
// too, and fmaxf maps a NaN to cell 0, as for every v when inv_w is 0).
struct Bins {
    float kmin, kmax, inv_w;
    int n_cells;
    __device__ __forceinline__ int cell(float v) const {
        const float t = __builtin_floorf((v - kmin) * inv_w);
        return (int)__builtin_fminf(__builtin_fmaxf(t, 0.0f), (float)(n_cells - 1));
    }
    // Index range [first, last) of the hits in cells cell(lo) .. cell(hi).
    __device__ __forceinline__ void range(const uint32_t* end, float lo, float hi, int& first, int& last) const {
        const int cl = cell(lo), ch = cell(hi);
        first = cl > 0 ? cell_end(end, cl - 1) : 0;
        last = cell_end(end, ch);
    }
};

// The hits [o, o + n) (1 <= n <= kBinCap) of one layer in registers, hit
// r kWave + lane in round r; the loads are issued together and unguarded
// (indices clamped to the layer), so that several layers can be in flight.
struct LayerRegs {
    float x[kBinRounds], y[kBinRounds];
    __device__ __forceinline__ void load(const float* __restrict__ xs, const float* __restrict__ ys, int o, int n) {
        // (byte offsets from a scalar base: one vector instruction per round)
        const char* bx = reinterpret_cast<const char*>(xs + o);
        const char* by = reinterpret_cast<const char*>(ys + o);
        const uint32_t lane4 = 4u * lane_id(), last = 4u * (uint32_t)(n - 1);
#pragma unroll
        for (int r = 0; r < kBinRounds; ++r) {
            x[r] = y[r] = 0.0f;
            if (r * kWave < n) {  // wave-uniform: rounds past the layer are skipped
                const uint32_t t = min(lane4 + 4u * kWave * r, last);
                x[r] = *reinterpret_cast<const float*>(bx + t);
                y[r] = *reinterpret_cast<const float*>(by + t);
            }
        }
    }
};

// Counting sort of the n hits of one layer (held in h, n <= NR kWave) into
// cells of the key K::key, storing K::payload in cell order.  Whole wave.
template <class K, int NR>
__device__ Bins build_bins_r(const Consts& c, const LayerRegs& h, int n, uint32_t* end, float* pa, float* pb) {
    const int lane = (int)lane_id();
    float key[NR];
    float2 pay[NR];
    float lo = __builtin_inff(), hi = -__builtin_inff();
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        const int t = r * kWave + lane;
        key[r] = __builtin_nanf("");
        if (t < n) {
            key[r] = K::key(c, h.x[r], h.y[r]);
            pay[r] = K::payload(c, h.x[r], h.y[r]);
        }
        if (__builtin_isfinite(key[r])) {
            lo = __builtin_fminf(lo, key[r]);
            hi = __builtin_fmaxf(hi, key[r]);
        } else {
            key[r] = __builtin_nanf("");  // left out below
        }
    }
    Bins b;
    b.kmin = wave_min_f(lo);
    b.kmax = wave_max_f(hi);
    int nc = 64;
    while (nc < n) nc <<= 1;  // power of two >= n, at most kBinCap
    b.n_cells = uniform_i(nc);
    const float width = b.kmax - b.kmin;
    // Any non-negative scale keeps cell() monotone; the hardware reciprocal
    // is enough to spread the keys over the cells.
    b.inv_w = (width > 0.0f && width < __builtin_inff()) ? __builtin_amdgcn_rcpf(width) * (float)b.n_cells : 0.0f;
    for (int t = lane; t < b.n_cells / 2; t += kWave) end[t] = 0u;
    wave_lds_sync();
    // Histogram: cell t counts in the half t & 1 of word t >> 1 (a half
    // never exceeds kBinCap, so no carry reaches the other half).
    int cell[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        cell[r] = -1;
        if (!__builtin_isnan(key[r])) {
            cell[r] = b.cell(key[r]);
            atomicAdd(&end[cell[r] >> 1], 1u << (16 * (cell[r] & 1)));
        }
    }
    wave_lds_sync();
    // Exclusive scan of the cell sizes: lane L owns cells [L*per, L*per + per)
    // (per = 1, 2 or 4), read and written with one access per lane
    // (consecutive lanes, consecutive addresses: no bank conflicts).
    static_assert(kBinCap <= 4 * kWave, "at most four cells per lane");
    const int per = b.n_cells / kWave;  // n_cells is a multiple of 64
    int4 sz = make_int4(0, 0, 0, 0);
    if (per == 4) {
        const uint2 v = reinterpret_cast<const uint2*>(end)[lane];
        sz = make_int4((int)(v.x & 0xFFFFu), (int)(v.x >> 16), (int)(v.y & 0xFFFFu), (int)(v.y >> 16));
    } else if (per == 2) {
        const uint32_t v = end[lane];
        sz = make_int4((int)(v & 0xFFFFu), (int)(v >> 16), 0, 0);
    } else {
        sz.x = cell_end(end, lane);
    }
    const int local = (sz.x + sz.y) + (sz.z + sz.w);
    const int s0 = wave_inclusive_sum(local) - local;  // starts of the lane's cells
    const int4 st = make_int4(s0, s0 + sz.x, s0 + sz.x + sz.y, s0 + sz.x + sz.y + sz.z);
    if (per == 4)
        reinterpret_cast<uint2*>(end)[lane] =
            make_uint2((uint32_t)st.x | ((uint32_t)st.y << 16), (uint32_t)st.z | ((uint32_t)st.w << 16));
    else if (per == 2)
        end[lane] = (uint32_t)st.x | ((uint32_t)st.y << 16);
    else
        reinterpret_cast<uint16_t*>(end)[lane] = (uint16_t)st.x;
    wave_lds_sync();
    // Scatter; afterwards cell t's entry is the end of cell t.
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        if (cell[r] >= 0) {
            const int sh = 16 * (cell[r] & 1);
            const int pos = (int)((atomicAdd(&end[cell[r] >> 1], 1u << sh) >> sh) & 0xFFFFu);
            pa[pos] = pay[r].x;
            pb[pos] = pay[r].y;
        }
    }
    wave_lds_sync();
    return b;
}

// build_bins_r with the fewest rounds that hold the layer (1, 2 or 4 times
// kWave hits; n <= kBinCap).
template <class K>
__device__ __forceinline__ Bins build_bins(const Consts& c, const LayerRegs& h, int n, uint32_t* end, float* pa,
                                           float* pb) {
    static_assert(kBinRounds == 4, "round counts 1, 2 and 4");
    if (n <= kWave) return build_bins_r<K, 1>(c, h, n, end, pa, pb);
    if (n <= 2 * kWave) return build_bins_r<K, 2>(c, h, n, end, pa, pb);
    return build_bins_r<K, 4>(c, h, n, end, pa, pb);
}

// A surviving pair (whole lanes of a divergent loop): the first kBinPairs of
// the event are kept, all are counted.
__device__ __forceinline__ void push_pair(BinLds& L, float4 p) {
    const uint32_t at = atomicAdd(L.n_pairs(), 1u);
    if (at < (uint32_t)kBinPairs) L.pairs[at] = p;
}

// Bounds of one event: pair test |a_x| <= bx, |a_y| <= by (window: strict,
// with the windows), and the half-widths r1, r2 of the layer-1 and layer-2
// key intervals, each at least the next binary32 value above its bound.
struct BinBounds {
    float bx, by, r1, r2;
};

// ---------------------------------------------------------------- MSD ---

// TRIG_TEST_MSD_BASIS.
struct MsdBasisBin {
    using Prune = MsdBasisPrune;
    static constexpr int kFewPairs = 4;
    static constexpr bool kMag = false;
    __device__ static __forceinline__ BinBounds bounds(const Consts& c, float) {
        return BinBounds{c.beta_x, c.beta_y, c.bin_r, c.bin_r};
    }
    struct Key1 {  // layer 1: key U1 x, payload (x, y)
        __device__ static __forceinline__ float key(const Consts& c, float x, float) { return c.U1 * x; }
        __device__ static __forceinline__ float2 payload(const Consts&, float x, float y) {
            return make_float2(x, y);
        }
    };
    struct Key2 {  // layer 2: key V2 x, payload (V2 x, V2 y)
        __device__ static __forceinline__ float key(const Consts& c, float x, float) { return c.V2 * x; }
        __device__ static __forceinline__ float2 payload(const Consts& c, float x, float y) {
            return make_float2(c.V2 * x, c.V2 * y);
        }
    };
    // Largest layer-1 |key| for hits within |x| <= M.
    __device__ static __forceinline__ float key_max(const Consts& c, float M) { return __builtin_fabsf(c.U1) * M; }
    // A layer-0 hit's side of the pair test, the centre of its key interval,
    // the test's score (at most bx + by for a pair that passes) and the test.
    __device__ static __forceinline__ float2 side(const Consts& c, float x, float y) {
        return make_float2(c.U0 * x, c.U0 * y);
    }
    __device__ static __forceinline__ float centre(float2 u) { return -u.x; }
    __device__ static __forceinline__ float2 diff(const Consts& c, float2 u, float xj, float yj) {
        return make_float2(u.x + c.U1 * xj, u.y + c.U1 * yj);
    }
    __device__ static __forceinline__ bool pair(const BinBounds& bb, float2 a) {
        return __builtin_fabsf(a.x) <= bb.bx && __builtin_fabsf(a.y) <= bb.by;
    }
    // What the event's list holds of a pair that passed.
    __device__ static __forceinline__ float4 entry(float xi, float yi, float2, float xj, float yj) {
        return make_float4(xi, yi, xj, yj);
    }
    // Lanes whose layer-2 hit (x, y) makes a passing triplet with the pair.
    __device__ static __forceinline__ uint64_t complete(const Consts& c, float4 p, float x, float y) {
        const MsdBasisTest::Pair pr = MsdBasisTest::pair(c, p.x, p.y, p.z, p.w);
        const float h[2] = {c.V2 * x, c.V2 * y};
        return MsdBasisTest::pass(c, pr, h);
    }
    // Passing triplets of a pair, from the layer-2 cells (in a1/b1).
    __device__ static uint32_t count_cells(const Consts& c, const BinBounds& bb, float xi, float yi, float xj, float yj,
                                           const Bins& b2, const BinLds& L) {
        const float ax = c.U0 * xi + c.U1 * xj;
        const float ay = c.U0 * yi + c.U1 * yj;
        const float ax2 = ax * ax, ay2 = ay * ay;
        const float bx0 = c.V0 * xi + c.V1 * xj;
        const float by0 = c.V0 * yi + c.V1 * yj;
        if (!__builtin_isfinite(bx0)) return 0;
        const float lo2 = widen_down(-bx0 - bb.r2), hi2 = widen_up(-bx0 + bb.r2);
        if (hi2 < b2.kmin || lo2 > b2.kmax) return 0;
        int k0, k1;
        b2.range(L.end1(), lo2, hi2, k0, k1);
        uint32_t cnt = 0;
        for (int k = k0; k < k1; ++k) {
            const float bx = bx0 + L.a1[k];
            const float qx = ax2 + bx * bx;
            const float by = by0 + L.b1[k];
            const float qy = ay2 + by * by;
            cnt += (uint32_t)((qx <= c.qmax_x) & (qy <= c.qmax_y));
        }
        return cnt;
    }
    __device__ static uint32_t count_pair(const Consts& c, const BinBounds& bb, float4 p, const Bins& b2,
                                          const BinLds& L) {
        return count_cells(c, bb, p.x, p.y, p.z, p.w, b2, L);
    }
    // Passing triplets with layer-0 hit (xi, yi), from the cells of both layers
    // (layer 1 in a2/b2).
    __device__ static uint32_t count_i(const Consts& c, const BinBounds& bb, float xi, float yi, const Bins& b1,
                                       const Bins& b2, const BinLds& L) {
        const float ux = c.U0 * xi;
        const float r = bb.r1;
        if (!__builtin_isfinite(ux)) return 0;
        const float lo = widen_down(-ux - r), hi = widen_up(-ux + r);
        if (hi < b1.kmin || lo > b1.kmax) return 0;
        int j0, j1;
        b1.range(L.end2(), lo, hi, j0, j1);
        uint32_t cnt = 0;
        for (int j = j0; j < j1; ++j) {
            const float xj = L.a2[j], yj = L.b2[j];
            const float ax = c.U0 * xi + c.U1 * xj;
            const float ay = c.U0 * yi + c.U1 * yj;
            if (!(__builtin_fabsf(ax) <= bb.bx && __builtin_fabsf(ay) <= bb.by)) continue;
            cnt += count_cells(c, bb, xi, yi, xj, yj, b2, L);
        }
        return cnt;
    }
};

// TRIG_TEST_MSD: cells and pair test from the written-out fit's bounds
// (a0 + a1 M, b0 + b1 M), candidates completed with the fit written out.
// A pair whose b partial is infinite has no passing triplet: with
// M = |x_j| (finite for a hit in a cell) the bound on |b| is finite.
struct MsdFitBin {
    using Prune = MsdFitPrune;
    static constexpr int kFewPairs = 4;
    static constexpr bool kMag = true;
    __device__ static __forceinline__ BinBounds bounds(const Consts& c, float M) {
        // 1 + 2^-20: fl(A (1 + 2^-20)) >= A (1 + 2^-23), above the next
        // binary32 value after any A >= 2^-126 (the bounds are normal)
        constexpr float kUp = 1.00000095367431640625f;
        const float bx = c.fit_a0x + c.fit_a1x * M;
        const float by = c.fit_a0y + c.fit_a1y * M;
        const float B = c.fit_b0x + c.fit_b1x * M;
        return BinBounds{bx, by, bx * kUp, B * kUp};
    }
    struct Key1 {  // layer 1: key U1 x, payload (x, y)
        __device__ static __forceinline__ float key(const Consts& c, float x, float) { return c.U1 * x; }
        __device__ static __forceinline__ float2 payload(const Consts&, float x, float y) {
            return make_float2(x, y);
        }
    };
    struct Key2 {  // layer 2: key V2 x, payload (x, y)
        __device__ static __forceinline__ float key(const Consts& c, float x, float) { return c.V2 * x; }
        __device__ static __forceinline__ float2 payload(const Consts&, float x, float y) {
            return make_float2(x, y);
        }
    };
    __device__ static __forceinline__ float key_max(const Consts& c, float M) { return MsdBasisBin::key_max(c, M); }
    __device__ static __forceinline__ float2 side(const Consts& c, float x, float y) {
        return MsdBasisBin::side(c, x, y);
    }
    __device__ static __forceinline__ float centre(float2 u) { return MsdBasisBin::centre(u); }
    __device__ static __forceinline__ float2 diff(const Consts& c, float2 u, float xj, float yj) {
        return MsdBasisBin::diff(c, u, xj, yj);
    }
    __device__ static __forceinline__ bool pair(const BinBounds& bb, float2 a) { return MsdBasisBin::pair(bb, a); }
    __device__ static __forceinline__ float4 entry(float xi, float yi, float2, float xj, float yj) {
        return make_float4(xi, yi, xj, yj);
    }
    __device__ static __forceinline__ uint64_t complete(const Consts& c, float4 p, float x, float y) {
        const MsdFitTest::Pair pr = MsdFitTest::pair(c, p.x, p.y, p.z, p.w);
        const float h[4] = {x, y, x * c.z2, y * c.z2};
        return MsdFitTest::pass(c, pr, h);
    }
    __device__ static uint32_t count_cells(const Consts& c, const BinBounds& bb, float xi, float yi, float xj, float yj,
                                           const Bins& b2, const BinLds& L) {
        const float bx0 = c.V0 * xi + c.V1 * xj;
        if (!__builtin_isfinite(bx0)) return 0;
        const float lo2 = widen_down(-bx0 - bb.r2), hi2 = widen_up(-bx0 + bb.r2);
        if (hi2 < b2.kmin || lo2 > b2.kmax) return 0;
        int k0, k1;
        b2.range(L.end1(), lo2, hi2, k0, k1);
        const float sx01 = xi * c.z0 + xj * c.z1;
        const float sy01 = yi * c.z0 + yj * c.z1;
        uint32_t cnt = 0;
        for (int k = k0; k < k1; ++k) {
            const float xk = L.a1[k], yk = L.b1[k];
            const float qx = MsdFitTest::plane_q(c, xi, xj, sx01, xk, xk * c.z2);
            const float qy = MsdFitTest::plane_q(c, yi, yj, sy01, yk, yk * c.z2);
            cnt += (uint32_t)((qx <= c.qmax_x) & (qy <= c.qmax_y));
        }
        return cnt;
    }
    __device__ static uint32_t count_pair(const Consts& c, const BinBounds& bb, float4 p, const Bins& b2,
                                          const BinLds& L) {
        return count_cells(c, bb, p.x, p.y, p.z, p.w, b2, L);
    }
    __device__ static uint32_t count_i(const Consts& c, const BinBounds& bb, float xi, float yi, const Bins& b1,
                                       const Bins& b2, const BinLds& L) {
        const float ux = c.U0 * xi;
        if (!__builtin_isfinite(ux)) return 0;  // x_i not finite: the fit fails
        const float lo = widen_down(-ux - bb.r1), hi = widen_up(-ux + bb.r1);
        if (hi < b1.kmin || lo > b1.kmax) return 0;
        int j0, j1;
        b1.range(L.end2(), lo, hi, j0, j1);
        uint32_t cnt = 0;
        for (int j = j0; j < j1; ++j) {
            const float xj = L.a2[j], yj = L.b2[j];
            const float ax = c.U0 * xi + c.U1 * xj;
            const float ay = c.U0 * yi + c.U1 * yj;
            if (!(__builtin_fabsf(ax) <= bb.bx && __builtin_fabsf(ay) <= bb.by)) continue;
            cnt += count_cells(c, bb, xi, yi, xj, yj, b2, L);
        }
        return cnt;
    }
};

// ------------------------------------------------------------- window ---

struct WindowBin {
    using Prune = WindowPrune;
    static constexpr int kFewPairs = 6;
    static constexpr bool kMag = false;
    __device__ static __forceinline__ BinBounds bounds(const Consts& c, float) {
        return BinBounds{c.win_x, c.win_y, c.bin_r, c.bin_r};
    }
    struct Key1 {  // layer 1: slopes (x / z1, y / z1), key the x slope
        __device__ static __forceinline__ float key(const Consts& c, float x, float) { return x / c.z1; }
        __device__ static __forceinline__ float2 payload(const Consts& c, float x, float y) {
            return make_float2(x / c.z1, y / c.z1);
        }
    };
    struct Key2 {
        __device__ static __forceinline__ float key(const Consts& c, float x, float) { return x / c.z2; }
        __device__ static __forceinline__ float2 payload(const Consts& c, float x, float y) {
            return make_float2(x / c.z2, y / c.z2);
        }
    };
    __device__ static __forceinline__ float key_max(const Consts& c, float M) { return M / c.z1; }
    __device__ static __forceinline__ float2 side(const Consts& c, float x, float y) {
        return make_float2(x / c.z0, y / c.z0);
    }
    __device__ static __forceinline__ float centre(float2 u) { return u.x; }
    __device__ static __forceinline__ float2 diff(const Consts&, float2 u, float sxj, float syj) {
        return make_float2(sxj - u.x, syj - u.y);
    }
    __device__ static __forceinline__ bool pair(const BinBounds& bb, float2 d) {
        return __builtin_fabsf(d.x) < bb.bx && __builtin_fabsf(d.y) < bb.by;
    }
    // (the layer-1 window is tested by pair(); layer 2 needs s_i only)
    __device__ static __forceinline__ float4 entry(float, float, float2 u, float, float) {
        return make_float4(u.x, u.y, 0.0f, 0.0f);
    }
    __device__ static __forceinline__ uint64_t complete(const Consts& c, float4 p, float x, float y) {
        return lanes(__builtin_fabsf(x / c.z2 - p.x) < c.win_x) & lanes(__builtin_fabsf(y / c.z2 - p.y) < c.win_y);
    }
    // Layer-2 partners of a layer-0 hit with slopes (sxi, syi).
    __device__ static uint32_t count_cells(const Consts& c, const BinBounds& bb, float sxi, float syi, const Bins& b2,
                                           const BinLds& L) {
        if (!__builtin_isfinite(sxi)) return 0;
        const float lo = widen_down(sxi - bb.r2), hi = widen_up(sxi + bb.r2);
        if (hi < b2.kmin || lo > b2.kmax) return 0;
        int k0, k1;
        b2.range(L.end1(), lo, hi, k0, k1);
        uint32_t nk = 0;
        for (int k = k0; k < k1; ++k)
            nk += (uint32_t)((__builtin_fabsf(L.a1[k] - sxi) < c.win_x) & (__builtin_fabsf(L.b1[k] - syi) < c.win_y));
        return nk;
    }
    __device__ static uint32_t count_pair(const Consts& c, const BinBounds& bb, float4 p, const Bins& b2,
                                          const BinLds& L) {
        return count_cells(c, bb, p.x, p.y, b2, L);
    }
    __device__ static uint32_t count_i(const Consts& c, const BinBounds& bb, float xi, float yi, const Bins& b1,
                                       const Bins& b2, const BinLds& L) {
        const float sxi = xi / c.z0, syi = yi / c.z0;
        if (!__builtin_isfinite(sxi)) return 0;
        const float lo = widen_down(sxi - bb.r1), hi = widen_up(sxi + bb.r1);
        uint32_t nj = 0;
        if (!(hi < b1.kmin || lo > b1.kmax)) {
            int j0, j1;
            b1.range(L.end2(), lo, hi, j0, j1);
            for (int j = j0; j < j1; ++j)
                nj += (uint32_t)((__builtin_fabsf(L.a2[j] - sxi) < c.win_x) &
                                 (__builtin_fabsf(L.b2[j] - syi) < c.win_y));
        }
        return nj == 0 ? 0u : nj * count_cells(c, bb, sxi, syi, b2, L);
    }
};

// Passing triplets of one event with 1 <= n0 and 1 <= n1, n2 <= kBinCap,
// hits straight from HBM (x, y absolute arrays).  Whole wave; the same count
// on every lane.
//
// Layer 2 is read only for events with a pair that can pass: an event of 200
// hits per layer in the default cuts has 0.16 such pairs on average, so most
// events neither read nor sort a third of their hits.  A few pairs are
// completed one by one, lanes over layer 2 (at most kFewPairs, which cost about
// what putting layer 2 into cells does); with more, up to kBinPairs, layer 2 goes into cells and each
// lane looks a pair's partners up there.  An event whose list overflows, or
// whose bounds let half of that through (P = bx by / K^2 of its pairs, for
// hits spread over +-M), has both layers in cells and each lane follows a
// layer-0 hit through both, so that its work stays in proportion to its hits.
// Whole calls, us, with every layer in cells / the pairs of a longer list one by
// one / so: 20,000 events of 30 hits per layer each on a track, MSD 24.5, 35.4,
// 15.3, window 15.0, 25.2, 15.5; 100,000 of 200 with windows 3 and 10 times the
// default 325, 419, 309 and 1035, 1396, 1050.
// 100,000 events of 200 hits per layer, whole call: 0.156 ms with layer 2
// sorted for every event, 0.122 ms without (1M mixture events, mean 80 per
// layer: 0.783 and 0.559 ms).
//
// The layer-1 cells are kBinCap = 256 equal intervals of [-K, K], K = key_max(M)
// (rounding is monotone, so every key of a finite hit lies in it; others
// land in some cell and fail the pair test): one wave-wide maximum gives
// both the cells and the bounds.  A cell's count and its hits' ranks come
// from one pass of LDS additions of 4 (bytes), on words that the sorted
// hits overwrite later.  What bounds it is the vector unit: with three
// wave-wide reductions, two passes of additions on packed counts and one
// candidate per step the kernel issued 682 vector instructions per event of
// 200 hits per layer, 89 of its 122 us; the same call takes 0.103 ms now (1M
// mixture events 0.559 -> 0.483 ms).
__device__ __forceinline__ uint32_t bin_cell(float key, float inv) {
    // saturating and truncating: negative values and NaN give 0; non-decreasing
    // in key for the scales that cell_scale gives
    uint32_t t;
    asm("v_cvt_u32_f32 %0, %1" : "=v"(t) : "v"(key * inv + 0.5f * (float)kBinCap));
    return min(t, (uint32_t)(kBinCap - 1));
}

template <class B>
__device__ uint32_t wave_event_binned(const Consts& c, const float* __restrict__ x, const float* __restrict__ y,
                                      int o0, int n0, int o1, int n1, int o2, int n2, BinLds& L) {
    // The loads of layer 1 and of layer 0's first four rounds in flight at
    // once (one HBM latency).  Indices are clamped to the layers (n0, n1, n2
    // >= 1).
    const int lane = (int)lane_id();
    LayerRegs h1, h0;
    h1.load(x, y, o1, n1);
    h0.load(x, y, o0, min(n0, kBinCap));
    // M: the largest layer-1 |x|, |y| (rounds past the layer hold 0).  A hit
    // with a coordinate that is not finite passes no test and does not count.
    uint32_t m = 0u;
#pragma unroll
    for (int r = 0; r < kBinRounds; ++r) m = max(m, max(abs_bits(h1.x[r]), abs_bits(h1.y[r])));
    m = wave_max_u(m);
    if (m >= 0x7f800000u) {
        m = 0u;
#pragma unroll
        for (int r = 0; r < kBinRounds; ++r) {
            const uint32_t b = max(abs_bits(h1.x[r]), abs_bits(h1.y[r]));
            m = max(m, b < 0x7f800000u ? b : 0u);
        }
        m = wave_max_u(m);
    }
    const float M = __builtin_bit_cast(float, m);
    const BinBounds bb = B::bounds(c, M);
    const float K = B::key_max(c, M);
    // (the hardware reciprocal is enough to spread the keys over the cells)
    const float inv = trig_host::cell_scale(K, __builtin_amdgcn_rcpf(K), (float)kBinCap);
    const float share = __builtin_amdgcn_rcpf(K);
    int n_pairs = kBinPairs + 1;
    if (!((float)n0 * (float)n1 * (bb.bx * share) * (bb.by * share) > 0.5f * (float)kBinPairs)) {
        uint32_t* hist = reinterpret_cast<uint32_t*>(L.a1);
        static_assert(kBinCap == 4 * kWave, "four cells per lane");
        reinterpret_cast<uint4*>(hist)[lane] = make_uint4(0u, 0u, 0u, 0u);
        if (lane == 0) *L.n_pairs() = 0u;
        wave_lds_sync();
        uint32_t cell[kBinRounds], rank[kBinRounds];  // rank: 4 bytes per hit of the cell before this one
#pragma unroll
        for (int r = 0; r < kBinRounds; ++r) {
            cell[r] = rank[r] = 0u;
            if (r * kWave < n1) {
                cell[r] = bin_cell(B::Key1::key(c, h1.x[r], h1.y[r]), inv);
                if (r * kWave + lane < n1) rank[r] = atomicAdd(&hist[cell[r]], 4u);
            }
        }
        wave_lds_sync();
        {
            // exclusive scan: starts()[t] the first byte of cell t's hits
            const uint4 v = reinterpret_cast<const uint4*>(hist)[lane];
            const uint32_t own = (v.x + v.y) + (v.z + v.w);
            const uint32_t s0 = (uint32_t)wave_inclusive_sum((int)own) - own;
            const uint32_t s1 = s0 + v.x, s2 = s1 + v.y, s3 = s2 + v.z;
            reinterpret_cast<uint2*>(L.ends)[lane] = make_uint2(s0 | (s1 << 16), s2 | (s3 << 16));
            if (lane == 0) L.starts()[kBinCap] = (uint16_t)(4 * n1);
        }
        wave_lds_sync();
        char* pa = reinterpret_cast<char*>(L.a1);
        char* pb = reinterpret_cast<char*>(L.b1);
#pragma unroll
        for (int r = 0; r < kBinRounds; ++r)
            if (r * kWave + lane < n1) {
                const uint32_t at = L.starts()[cell[r]] + rank[r];
                const float2 p = B::Key1::payload(c, h1.x[r], h1.y[r]);
                *reinterpret_cast<float*>(pa + at) = p.x;
                *reinterpret_cast<float*>(pb + at) = p.y;
            }
        wave_lds_sync();
        // Layer-0 hit (xi, yi): its cells' hits, two per step.  The interval's ends
        // are moved outwards by |centre| 2^-21 and r1 2^-20 + 2^-126, more than the
        // rounding of the two sums.
        const float r1 = bb.r1 * 1.00000095367431640625f + 0x1p-126f, pre = bb.bx + bb.by;
        auto scan = [&](float xi, float yi) {
            const float2 u = B::side(c, xi, yi);
            const float mid = B::centre(u), w = __builtin_fabsf(mid) * 0x1p-21f + r1;
            uint32_t j = L.starts()[bin_cell(mid - w, inv)];
            const uint32_t end = L.starts()[bin_cell(mid + w, inv) + 1];
            for (; j < end; j += 8u) {
                // (the second hit may lie past the cells: it fails the pair test, as
                // every hit outside the interval does, or is not looked at)
                const float x0 = *reinterpret_cast<const float*>(pa + j), x1 = *reinterpret_cast<const float*>(pa + j + 4);
                const float y0 = *reinterpret_cast<const float*>(pb + j), y1 = *reinterpret_cast<const float*>(pb + j + 4);
                const float2 a0 = B::diff(c, u, x0, y0), a1 = B::diff(c, u, x1, y1);
                const float s0 = __builtin_fabsf(a0.x) + __builtin_fabsf(a0.y);
                const float s1 = __builtin_fabsf(a1.x) + __builtin_fabsf(a1.y);
                if (__builtin_fminf(s0, s1) <= pre) {
                    if (B::pair(bb, a0)) push_pair(L, B::entry(xi, yi, u, x0, y0));
                    if (j + 4u < end && B::pair(bb, a1)) push_pair(L, B::entry(xi, yi, u, x1, y1));
                }
            }
        };
#pragma unroll
        for (int r = 0; r < kBinRounds; ++r)
            if (r * kWave + lane < n0) scan(h0.x[r], h0.y[r]);
        for (int i = kBinCap + lane; i < n0; i += kWave) scan(x[o0 + i], y[o0 + i]);
        wave_lds_sync();
        n_pairs = uniform_i((int)*L.n_pairs());
    }
    uint32_t cnt = 0;
    if (n_pairs > 0) {
        LayerRegs h2;
        h2.load(x, y, o2, n2);
        if (n_pairs <= B::kFewPairs) {
            for (int p = 0; p < n_pairs; ++p) {
                const float4 pr = L.pairs[p];
#pragma unroll
                for (int r = 0; r < kBinRounds; ++r)
                    if (r * kWave < n2)
                        cnt += (uint32_t)__builtin_popcountll(lanes(r * kWave + lane < n2) &
                                                              B::complete(c, pr, h2.x[r], h2.y[r]));
                if (cnt >= (uint32_t)c.count_cap) break;  // the result is capped there
            }
        } else {
            wave_lds_sync();  // the layer-2 cells overwrite layer 1's
            const Bins b2 = build_bins<typename B::Key2>(c, h2, n2, L.end1(), L.a1, L.b1);
            if (n_pairs <= kBinPairs) {
                for (int p = lane; p < n_pairs; p += kWave) cnt += B::count_pair(c, bb, L.pairs[p], b2, L);
            } else {
                LayerRegs g1;
                g1.load(x, y, o1, n1);
                const Bins b1 = build_bins<typename B::Key1>(c, g1, n1, L.end2(), L.a2, L.b2);
                for (int i0 = 0; i0 < n0; i0 += kWave) {
                    if (i0 + lane < n0) cnt += B::count_i(c, bb, x[o0 + i0 + lane], y[o0 + i0 + lane], b1, b2, L);
                    // decision only: stop once the (capped) result is known
                    if (c.count_cap != INT32_MAX && i0 + kWave < n0 && wave_sum_u(cnt) >= (uint32_t)c.count_cap) break;
                }
            }
            cnt = wave_sum_u(cnt);
        }
    }
    wave_lds_sync();  // the next event rebuilds the cells
    return cnt;
}

}  // namespace trig

// Device-side building blocks of the trigger-station triplet selection:
// per-plane test policies, per-event CSR loading and the wave-level triplet
// loop shared by the plain and the persistent kernels.
//
// Method: paper Sec. 3.2 "Algorithm" - all one-hit-per-layer triplets (step
// 1), straight-line fit through the vertex in x-z and y-z and a cut on its
// mean square deviation per degree of freedom (step 2), event selected with at
// least two passing triplets (step 3).  The binary32 operation order is the
// one fixed in include/trig.h; this file must be compiled with
// -ffp-contract=off and without flushing fp32 subnormals.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace trig {

constexpr int kWave = 64;

// Everything a kernel needs from the parameters, derived on the host
// (csrc/trig_bounds.hpp holds the derivations).
struct Consts {
    // Orthonormal basis of the plane orthogonal to (z0, z1, z2): the
    // TRIG_TEST_MSD_BASIS evaluation, and the partial sums a, b that the
    // pruned and binned forms of both MSD tests look at
    float U0, U1, V0, V1, V2;
    // TRIG_TEST_MSD (the fit written out): layer positions and w = 1 / sum z^2
    float z0, z1, z2, w;
    // MSD tests: largest binary32 Q with f32(Q / ndf) <= msd_max, per plane
    float qmax_x, qmax_y;
    // TRIG_TEST_MSD_BASIS pair bound: largest binary32 b >= 0 with
    // f32(b * b) <= qmax, per plane
    float beta_x, beta_y;
    // Per-hit z, pruned form: a triplet that passes a plane has
    // |f32(s_j - s_i)| <= (a0 + a1 M) / zmin for the hits' slopes s = c / z
    // (M >= |c_i|, |c_j|, zmin <= z_i, z_j), per plane
    float zs_a0x, zs_a1x, zs_a0y, zs_a1y;
    // TRIG_TEST_MSD: a triplet that passes a plane has |a| <= a0 + a1 M and
    // |b| <= b0 + b1 M (device evaluation order, M >= |c1| the plane's
    // layer-1 coordinate), per plane
    float fit_a0x, fit_a1x, fit_a0y, fit_a1y, fit_b0x, fit_b1x, fit_b0y, fit_b1y;
    // Prefilters: (|u| <= bx and |v| <= by) implies |u| + |v| <= bx + by and
    // max(|u|, |v|) <= max(bx, by), in binary32 too.  MSD_BASIS: the sum of
    // the betas; window: the sum of the windows and the larger window.
    float pre_msd, pre_win_sum, pre_win;
    // TRIG_TEST_SLOPE_WINDOW
    float win_x, win_y;
    // Batched form's prefilter on staged coordinates, by the layer in the
    // lanes (index 0: layer 1, index 1: layer 0): trig_host::DirectBounds
    float dir_k[2], dir_scale[2], dir_slack[2];
    // Binned form, MSD_BASIS and window: half-width of the key interval
    // around a hit's centre (MSD_BASIS: the binary32 value above beta_x;
    // window: win_x).
    float bin_r;
    // accept iff count >= min_triplets (two-particle mode: the candidates,
    // count >= 2)
    int32_t min_triplets;
    // counts are written as min(count, count_cap) (INT32_MAX unless the
    // caller asked for the decision only); an event's search may stop once
    // its count reaches the cap
    int32_t count_cap;
    int32_t n_hits;
};

// The count an event's result holds (errors, negative, unchanged).
__device__ __forceinline__ int32_t capped(int32_t cnt, const Consts& c) {
    return cnt < c.count_cap ? cnt : c.count_cap;
}

__device__ __forceinline__ int uniform_i(int v) { return __builtin_amdgcn_readfirstlane(v); }
// cond ? a : b for wave-uniform operands, on the scalar unit (a compare
// and a scalar select; the compiler would otherwise select per lane).
__device__ __forceinline__ float select_uniform(int cond, float a, float b) {
    const int c = uniform_i(cond);
    const int ia = uniform_i(__builtin_bit_cast(int, a)), ib = uniform_i(__builtin_bit_cast(int, b));
    int r;
    asm("s_cmp_lg_u32 %1, 0\n\ts_cselect_b32 %0, %2, %3" : "=s"(r) : "s"(c), "s"(ia), "s"(ib) : "scc");
    return __builtin_bit_cast(float, r);
}

__device__ __forceinline__ unsigned lane_id() { return threadIdx.x & (kWave - 1); }

// Order this wave's LDS writes before its later LDS reads, and its reads
// before later writes, across lanes of the wave.  The LDS performs one
// wave's operations in issue order, so nothing has to drain (no s_waitcnt:
// the LDS counter only orders LDS against other memory and other waves);
// only the compiler must be kept from moving memory operations across.
// Global loads in flight, such as the next block's prefetch, keep flying.
__device__ __forceinline__ void wave_lds_sync() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_wave_barrier();
    asm volatile("" ::: "memory");
}

__device__ __forceinline__ bool wave_any(bool pred) { return __builtin_amdgcn_ballot_w64(pred) != 0ull; }

// Cross-lane steps on the vector unit (DPP, gfx9 controls) for whole-wave
// code (all 64 lanes active).  dpp_i<C, ROWS>(old, v): lanes of the rows of 16
// in the mask ROWS take v from the lane that control C names; other lanes,
// and lanes whose source lies outside their row, keep `old`.
constexpr int kDppQuadXor1 = 0xB1;     // quad_perm [1, 0, 3, 2]
constexpr int kDppQuadXor2 = 0x4E;     // quad_perm [2, 3, 0, 1]
constexpr int kDppRowShr = 0x110;      // row_shr:n = kDppRowShr + n
constexpr int kDppRowMirror = 0x140;   // lane i of a row takes lane 15 - i
constexpr int kDppHalfMirror = 0x141;  // lane i of a half row takes lane 7 - i
constexpr int kDppBcast15 = 0x142;     // with rows 0xA: rows 1, 3 take lane 15 of the row before
constexpr int kDppBcast31 = 0x143;     // with rows 0xC: rows 2, 3 take lane 31

template <int C, int ROWS = 0xF>
__device__ __forceinline__ int dpp_i(int old, int v) {
    return __builtin_amdgcn_update_dpp(old, v, C, ROWS, 0xF, false);
}
template <int C, int ROWS = 0xF>
__device__ __forceinline__ float dpp_f(float old, float v) {
    return __builtin_bit_cast(float, dpp_i<C, ROWS>(__builtin_bit_cast(int, old), __builtin_bit_cast(int, v)));
}

// Wave-wide min, max and sum (result in every lane's return value, taken
// from lane 63): butterflies within quads, mirrors within rows of 16 (every
// lane then holds its row's result), then the row broadcasts carry rows 0-2
// into row 3.  fminf/fmaxf drop NaN as the scalar functions do.
__device__ __forceinline__ float wave_min_f(float v) {
    v = __builtin_fminf(v, dpp_f<kDppQuadXor1>(v, v));
    v = __builtin_fminf(v, dpp_f<kDppQuadXor2>(v, v));
    v = __builtin_fminf(v, dpp_f<kDppHalfMirror>(v, v));
    v = __builtin_fminf(v, dpp_f<kDppRowMirror>(v, v));
    v = __builtin_fminf(v, dpp_f<kDppBcast15, 0xA>(v, v));
    v = __builtin_fminf(v, dpp_f<kDppBcast31, 0xC>(v, v));
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 63));
}
__device__ __forceinline__ float wave_max_f(float v) {
    v = __builtin_fmaxf(v, dpp_f<kDppQuadXor1>(v, v));
    v = __builtin_fmaxf(v, dpp_f<kDppQuadXor2>(v, v));
    v = __builtin_fmaxf(v, dpp_f<kDppHalfMirror>(v, v));
    v = __builtin_fmaxf(v, dpp_f<kDppRowMirror>(v, v));
    v = __builtin_fmaxf(v, dpp_f<kDppBcast15, 0xA>(v, v));
    v = __builtin_fmaxf(v, dpp_f<kDppBcast31, 0xC>(v, v));
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 63));
}
__device__ __forceinline__ uint32_t wave_max_u(uint32_t v) {
    v = max(v, (uint32_t)dpp_i<kDppQuadXor1>(0, (int)v));
    v = max(v, (uint32_t)dpp_i<kDppQuadXor2>(0, (int)v));
    v = max(v, (uint32_t)dpp_i<kDppHalfMirror>(0, (int)v));
    v = max(v, (uint32_t)dpp_i<kDppRowMirror>(0, (int)v));
    v = max(v, (uint32_t)dpp_i<kDppBcast15, 0xA>(0, (int)v));
    v = max(v, (uint32_t)dpp_i<kDppBcast31, 0xC>(0, (int)v));
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}
__device__ __forceinline__ uint32_t wave_sum_u(uint32_t v) {
    int x = (int)v;
    x += dpp_i<kDppQuadXor1>(0, x);
    x += dpp_i<kDppQuadXor2>(0, x);
    x += dpp_i<kDppHalfMirror>(0, x);
    x += dpp_i<kDppRowMirror>(0, x);
    x += dpp_i<kDppBcast15, 0xA>(0, x);
    x += dpp_i<kDppBcast31, 0xC>(0, x);
    return (uint32_t)__builtin_amdgcn_readlane(x, 63);
}
// Inclusive prefix sum over the lanes: shifts by 1, 2, 4, 8 within rows
// (lanes without a source add 0), then the row broadcasts add the totals of
// the rows before.
__device__ __forceinline__ int wave_inclusive_sum(int x) {
    x += dpp_i<kDppRowShr + 1>(0, x);
    x += dpp_i<kDppRowShr + 2>(0, x);
    x += dpp_i<kDppRowShr + 4>(0, x);
    x += dpp_i<kDppRowShr + 8>(0, x);
    x += dpp_i<kDppBcast15, 0xA>(0, x);
    x += dpp_i<kDppBcast31, 0xC>(0, x);
    return x;
}

// Lane mask of a single comparison.  Combining two comparisons with a scalar
// AND of their masks (rather than a ballot of `a & b`) keeps each predicate a
// plain vector compare writing scalar registers.
__device__ __forceinline__ uint64_t lanes(bool cmp) { return __builtin_amdgcn_ballot_w64(cmp); }

// ----------------------------------------------------------------------------
// Test policies.  HF = floats of a layer-2 hit that pass() reads (stage());
// Pair = the part of the test that depends on (i, j) only; pass() completes it
// with hit k and returns the mask of lanes whose triplet passes.
//
// Rejecting test of the every-triplet loops (wave_count): pre_pair(i, j) and
// pre_k(k) give one value per plane, and a triplet that passes has
// |pre_pair + pre_k| <= a bound in each plane, one binary32 sum each.
//   MSD tests: the partial sum b = f32(p + w) of the basis form, p = f32(
//     f32(V0 c_i) + f32(V1 c_j)), w = f32(V2 c_k).  Basis form: Q =
//     f32(f32(a^2) + f32(b^2)) >= f32(b^2), so |b| <= beta.  Fit written out:
//     |b| <= b0 + b1 M (csrc/trig_bounds.hpp).
//   window: s_k - s_i (as s_k + (-s_i), the same binary32 value) is the
//     test's own quantity; a pair outside the layer-1 window gives NaN.
//   per-hit z, MSD: s_k - s_i, |.| <= (a0 + a1 M) / zmin.
// kLoose, kNear, kShare: where the rejecting test does not pay, see wave_count;
// kMinHits: layer-2 hits from which on it does.  kPreTests: pre_pair and pre_k
// are all that the test itself needs (pre_pass).  kTile: small events by
// wave_count_tile, with bound().
// Invalid pairs and padding are NaN, which fails every comparison.
// ----------------------------------------------------------------------------

// TRIG_TEST_MSD_BASIS: Q = a^2 + b^2 in the basis (u, v).
struct MsdBasisTest {
    static constexpr int HF = 2;
    static constexpr float kLoose = 12.0f;
    static constexpr int kNear = 8, kShare = 3, kMinHits = 1;
    static constexpr bool kPreTests = false;
    static constexpr bool kZ = false;  // layer positions from the parameters
    static constexpr bool kTile = true;
    struct Pair {
        float ax2, bx0, ay2, by0;
    };
    // The rejecting test's bound (m: the lane's largest |layer-1 coordinate|).
    __device__ static __forceinline__ float bound(const Consts& c, float) { return c.pre_msd; }
    __device__ static __forceinline__ void stage(const Consts& c, float x, float y, float* h) {
        h[0] = c.V2 * x;
        h[1] = c.V2 * y;
    }
    __device__ static __forceinline__ float2 pre_k(const Consts& c, float x, float y) {
        return make_float2(c.V2 * x, c.V2 * y);
    }
    __device__ static __forceinline__ float2 pre_pair(const Consts& c, float xi, float yi, float xj, float yj) {
        return make_float2(c.V0 * xi + c.V1 * xj, c.V0 * yi + c.V1 * yj);
    }
    __device__ static __forceinline__ Pair pair(const Consts& c, float xi, float yi, float xj,
                                                float yj) {
        Pair p;
        const float ax = c.U0 * xi + c.U1 * xj;
        const float ay = c.U0 * yi + c.U1 * yj;
        p.ax2 = ax * ax;
        p.ay2 = ay * ay;
        p.bx0 = c.V0 * xi + c.V1 * xj;
        p.by0 = c.V0 * yi + c.V1 * yj;
        return p;
    }
    __device__ static __forceinline__ Pair invalid() {
        const float n = __builtin_nanf("");
        return Pair{n, n, n, n};
    }
    __device__ static __forceinline__ uint64_t pass(const Consts& c, const Pair& p, const float* h) {
        const float bx = p.bx0 + h[0];
        const float qx = p.ax2 + bx * bx;
        const float by = p.by0 + h[1];
        const float qy = p.ay2 + by * by;
        return lanes(qx <= c.qmax_x) & lanes(qy <= c.qmax_y);
    }
};

// TRIG_TEST_MSD: the fit through the vertex written out (slope, residuals,
// their sum of squares), the paper's definition of the test.
struct MsdFitTest {
    static constexpr int HF = 4;
    static constexpr float kLoose = 12.0f;
    static constexpr int kNear = 8, kShare = 3, kMinHits = 1;
    static constexpr bool kPreTests = false;
    static constexpr bool kZ = false;  // layer positions from the parameters
    static constexpr bool kTile = true;
    struct Pair {
        float xi, xj, sx01, yi, yj, sy01;
    };
    __device__ static __forceinline__ float bound(const Consts& c, float m) { return of_max(c, wave_max_f(m)); }
    __device__ static __forceinline__ float of_max(const Consts& c, float M) {
        return (c.fit_b0x + c.fit_b1x * M) + (c.fit_b0y + c.fit_b1y * M);
    }
    __device__ static __forceinline__ void stage(const Consts& c, float x, float y, float* h) {
        h[0] = x;
        h[1] = y;
        h[2] = x * c.z2;
        h[3] = y * c.z2;
    }
    __device__ static __forceinline__ float2 pre_k(const Consts& c, float x, float y) {
        return MsdBasisTest::pre_k(c, x, y);
    }
    __device__ static __forceinline__ float2 pre_pair(const Consts& c, float xi, float yi, float xj, float yj) {
        return MsdBasisTest::pre_pair(c, xi, yi, xj, yj);
    }
    __device__ static __forceinline__ Pair pair(const Consts& c, float xi, float yi, float xj,
                                                float yj) {
        Pair p;
        p.xi = xi; p.xj = xj; p.yi = yi; p.yj = yj;
        p.sx01 = xi * c.z0 + xj * c.z1;
        p.sy01 = yi * c.z0 + yj * c.z1;
        return p;
    }
    __device__ static __forceinline__ Pair invalid() {
        const float n = __builtin_nanf("");
        return Pair{n, n, n, n, n, n};
    }
    __device__ static __forceinline__ float plane_q(const Consts& c, float ci, float cj, float s01,
                                                    float ck, float pk) {
        const float m = (s01 + pk) * c.w;
        const float r0 = ci - m * c.z0;
        const float r1 = cj - m * c.z1;
        const float r2 = ck - m * c.z2;
        return (r0 * r0 + r1 * r1) + r2 * r2;
    }
    __device__ static __forceinline__ uint64_t pass(const Consts& c, const Pair& p, const float* h) {
        const float qx = plane_q(c, p.xi, p.xj, p.sx01, h[0], h[2]);
        const float qy = plane_q(c, p.yi, p.yj, p.sy01, h[1], h[3]);
        return lanes(qx <= c.qmax_x) & lanes(qy <= c.qmax_y);
    }
};

struct WindowTest {
    static constexpr int HF = 2;
    static constexpr float kLoose = 3.0f;
    static constexpr int kNear = 16, kShare = 3, kMinHits = 5;
    static constexpr bool kPreTests = true, kTile = false;
    static constexpr bool kZ = false;  // layer positions from the parameters
    struct Pair {
        float sxi, syi;  // NaN when the layer-1 window already fails
    };
    __device__ static __forceinline__ void stage(const Consts& c, float x, float y, float* h) {
        h[0] = x / c.z2;
        h[1] = y / c.z2;
    }
    __device__ static __forceinline__ uint64_t pre_pass(const Consts& c, float2 p, float wx, float wy) {
        return lanes(__builtin_fabsf(p.x + wx) < c.win_x) & lanes(__builtin_fabsf(p.y + wy) < c.win_y);
    }
    __device__ static __forceinline__ float2 pre_k(const Consts& c, float x, float y) {
        return make_float2(x / c.z2, y / c.z2);
    }
    __device__ static __forceinline__ float2 pre_pair(const Consts& c, float xi, float yi, float xj, float yj) {
        const Pair p = pair(c, xi, yi, xj, yj);
        return make_float2(-p.sxi, -p.syi);
    }
    __device__ static __forceinline__ Pair pair(const Consts& c, float xi, float yi, float xj,
                                                float yj) {
        const float sxi = xi / c.z0, syi = yi / c.z0;
        const float sxj = xj / c.z1, syj = yj / c.z1;
        const bool ok = (__builtin_fabsf(sxj - sxi) < c.win_x) & (__builtin_fabsf(syj - syi) < c.win_y);
        const float n = __builtin_nanf("");
        return Pair{ok ? sxi : n, ok ? syi : n};
    }
    __device__ static __forceinline__ Pair invalid() {
        const float n = __builtin_nanf("");
        return Pair{n, n};
    }
    __device__ static __forceinline__ uint64_t pass(const Consts& c, const Pair& p, const float* h) {
        return lanes(__builtin_fabsf(h[0] - p.sxi) < c.win_x) & lanes(__builtin_fabsf(h[1] - p.syi) < c.win_y);
    }
};

// Per-hit z (trig_hits.z): the fit written out with each hit's own z, its
// Szz and reciprocal per triplet (one binary32 division shared by both
// planes):  Szz = (zi*zi + zj*zj) + zk*zk,  w = 1 / Szz,
// m = ((ci*zi + cj*zj) + ck*zk) * w,  r_l = c_l - m*z_l.
struct MsdZTest {
    static constexpr int HF = 6;
    static constexpr float kLoose = 6.0f;
    static constexpr int kNear = 8, kShare = 3, kMinHits = 1;
    static constexpr bool kPreTests = false, kTile = false;
    static constexpr bool kZ = true;
    struct Pair {
        float xi, xj, sx01, yi, yj, sy01, zi, zj, szz01;
    };
    __device__ static __forceinline__ void stage(const Consts&, float x, float y, float z, float* h) {
        h[0] = x;
        h[1] = y;
        h[2] = z;
        h[3] = x * z;
        h[4] = y * z;
        h[5] = z * z;
    }
    __device__ static __forceinline__ float2 pre_k(const Consts&, float x, float y, float z) {
        return make_float2(x / z, y / z);
    }
    __device__ static __forceinline__ float2 pre_pair(const Consts&, float xi, float yi, float zi, float, float,
                                                      float) {
        return make_float2(-(xi / zi), -(yi / zi));
    }
    __device__ static __forceinline__ Pair pair(const Consts&, float xi, float yi, float zi, float xj, float yj,
                                                float zj) {
        Pair p;
        p.xi = xi; p.xj = xj; p.yi = yi; p.yj = yj; p.zi = zi; p.zj = zj;
        p.sx01 = xi * zi + xj * zj;
        p.sy01 = yi * zi + yj * zj;
        p.szz01 = zi * zi + zj * zj;
        return p;
    }
    __device__ static __forceinline__ Pair invalid() {
        const float n = __builtin_nanf("");
        return Pair{n, n, n, n, n, n, n, n, n};
    }
    __device__ static __forceinline__ float plane_q(float ci, float cj, float s01, float ck, float pk, float zi,
                                                    float zj, float zk, float w) {
        const float m = (s01 + pk) * w;
        const float r0 = ci - m * zi;
        const float r1 = cj - m * zj;
        const float r2 = ck - m * zk;
        return (r0 * r0 + r1 * r1) + r2 * r2;
    }
    __device__ static __forceinline__ uint64_t pass(const Consts& c, const Pair& p, const float* h) {
        const float w = 1.0f / (p.szz01 + h[5]);
        const float qx = plane_q(p.xi, p.xj, p.sx01, h[0], h[3], p.zi, p.zj, h[2], w);
        const float qy = plane_q(p.yi, p.yj, p.sy01, h[1], h[4], p.zi, p.zj, h[2], w);
        return lanes(qx <= c.qmax_x) & lanes(qy <= c.qmax_y);
    }
};

// Per-hit z, window test: slopes c / z with each hit's own z.
struct WindowZTest {
    static constexpr int HF = 2;
    static constexpr float kLoose = 3.0f;
    static constexpr int kNear = 16, kShare = 3, kMinHits = 5;
    static constexpr bool kPreTests = true, kTile = false;
    static constexpr bool kZ = true;
    struct Pair {
        float sxi, syi;  // NaN when the layer-1 window already fails
    };
    __device__ static __forceinline__ void stage(const Consts&, float x, float y, float z, float* h) {
        h[0] = x / z;
        h[1] = y / z;
    }
    __device__ static __forceinline__ uint64_t pre_pass(const Consts& c, float2 p, float wx, float wy) {
        return lanes(__builtin_fabsf(p.x + wx) < c.win_x) & lanes(__builtin_fabsf(p.y + wy) < c.win_y);
    }
    __device__ static __forceinline__ float2 pre_k(const Consts&, float x, float y, float z) {
        return make_float2(x / z, y / z);
    }
    __device__ static __forceinline__ float2 pre_pair(const Consts& c, float xi, float yi, float zi, float xj,
                                                      float yj, float zj) {
        const Pair p = pair(c, xi, yi, zi, xj, yj, zj);
        return make_float2(-p.sxi, -p.syi);
    }
    __device__ static __forceinline__ Pair pair(const Consts& c, float xi, float yi, float zi, float xj, float yj,
                                                float zj) {
        const float sxi = xi / zi, syi = yi / zi;
        const float sxj = xj / zj, syj = yj / zj;
        const bool ok = (__builtin_fabsf(sxj - sxi) < c.win_x) & (__builtin_fabsf(syj - syi) < c.win_y);
        const float n = __builtin_nanf("");
        return Pair{ok ? sxi : n, ok ? syi : n};
    }
    __device__ static __forceinline__ Pair invalid() {
        const float n = __builtin_nanf("");
        return Pair{n, n};
    }
    __device__ static __forceinline__ uint64_t pass(const Consts& c, const Pair& p, const float* h) {
        return lanes(__builtin_fabsf(h[0] - p.sxi) < c.win_x) & lanes(__builtin_fabsf(h[1] - p.syi) < c.win_y);
    }
};

// ----------------------------------------------------------------------------
// Events
// ----------------------------------------------------------------------------

struct EventRange {
    int o0, o1, o2;
    int n0, n1, n2;
};

// Reads and checks the CSR range of event e (wave-uniform).  Returns 0, or
// the per-event error count (-1 malformed, -2 count not representable).
__device__ __forceinline__ int load_event(const int32_t* __restrict__ off, int e, int n_hits,
                                          EventRange& ev) {
    const int64_t b = 3 * (int64_t)e;
    const int a0 = uniform_i(off[b]), a1 = uniform_i(off[b + 1]);
    const int a2 = uniform_i(off[b + 2]), a3 = uniform_i(off[b + 3]);
    if (!(0 <= a0 && a0 <= a1 && a1 <= a2 && a2 <= a3 && a3 <= n_hits)) return -1;
    ev.o0 = a0; ev.o1 = a1; ev.o2 = a2;
    ev.n0 = a1 - a0; ev.n1 = a2 - a1; ev.n2 = a3 - a2;
    // (n0 n1 < 2^62, and with n0 n1 <= INT32_MAX the product with n2 too)
    const int64_t n01 = (int64_t)ev.n0 * ev.n1;
    if (ev.n2 > 0 && (n01 > (int64_t)INT32_MAX || n01 * ev.n2 > (int64_t)INT32_MAX)) return -2;
    return 0;
}

__device__ __forceinline__ uint32_t pair_tiles(const EventRange& ev) {
    const uint64_t np = (uint64_t)ev.n0 * (uint64_t)ev.n1;
    return (ev.n2 == 0) ? 0u : (uint32_t)((np + kWave - 1) / kWave);
}

// Rejecting-test bound (see the test policies): a triplet passes only if the
// magnitudes of the two planes' sums add up to at most `bound`; valid = false:
// no bound holds (per-hit z outside (0, inf) in layers 0 or 2) and every
// triplet takes the full test.
struct PreBound {
    float bound;
    bool valid;
};

// One step of 64 pairs for a lane's pair (i, j).
struct PairStep {
    uint32_t n1, dq, dr;
    __device__ __forceinline__ explicit PairStep(uint32_t n) : n1(n), dq(kWave / n), dr(kWave % n) {}
    __device__ __forceinline__ void operator()(uint32_t& i, uint32_t& j) const {
        j += dr;
        i += dq;
        if (j >= n1) {
            j -= n1;
            ++i;
        }
    }
};

// The pair part of the full test for the lane's pair (i, j).
template <class T>
__device__ __forceinline__ typename T::Pair pair_of(const float* __restrict__ x, const float* __restrict__ y,
                                                    const float* __restrict__ z, const EventRange& ev, const Consts& c,
                                                    uint32_t i, uint32_t j) {
    typename T::Pair pr = T::invalid();
    if (i < (uint32_t)ev.n0) {
        if constexpr (T::kZ)
            pr = T::pair(c, x[ev.o0 + i], y[ev.o0 + i], z[ev.o0 + i], x[ev.o1 + j], y[ev.o1 + j], z[ev.o1 + j]);
        else
            pr = T::pair(c, x[ev.o0 + i], y[ev.o0 + i], x[ev.o1 + j], y[ev.o1 + j]);
    }
    return pr;
}

// pre_k of the layer-2 hits [k0, k0 + nk) into wx and wy, NaN up to a whole
// group of four.  Returns |pre_k| (both planes' sum) of the lane's first hit.
template <class T>
__device__ __forceinline__ float stage_pre(const float* __restrict__ x, const float* __restrict__ y,
                                           const float* __restrict__ z, const EventRange& ev, const Consts& c, int k0,
                                           int nk, float* __restrict__ wx, float* __restrict__ wy) {
    const int lane = (int)lane_id(), nk_pad = (nk + 3) & ~3;
    const float nan = __builtin_nanf("");
    float own = __builtin_inff();
    for (int t = lane; t < nk_pad; t += kWave) {
        const int k = ev.o2 + k0 + min(t, nk - 1);
        float2 w;
        if constexpr (T::kZ)
            w = T::pre_k(c, x[k], y[k], z[k]);
        else
            w = T::pre_k(c, x[k], y[k]);
        wx[t] = t < nk ? w.x : nan;
        wy[t] = t < nk ? w.y : nan;
        if (t < kWave) own = __builtin_fabsf(w.x) + __builtin_fabsf(w.y);
    }
    return own;
}

// The full test of every triplet of pair tiles [t_begin, t_end) (see
// wave_count), the hits' part of it staged in the wave's LF floats of LDS;
// staged: the first chunk's pre_k is there (tests of two values per hit only).
template <class T, int LF>
__device__ __forceinline__ uint32_t wave_count_full(const float* __restrict__ x, const float* __restrict__ y,
                                                    const float* __restrict__ z, const EventRange& ev,
                                                    uint32_t t_begin, uint32_t t_end, const Consts& c,
                                                    float* __restrict__ lds, bool staged) {
    constexpr bool kPlanes = T::HF == 2;  // the values are pre_k, kept as wave_count_pre does
    constexpr int KCH = LF / T::HF & ~3;  // hits per chunk
    static_assert(KCH > 0, "room for one group of four hits");
    const uint32_t stop = (uint32_t)c.count_cap;  // enough: the result is capped there
    const unsigned lane = lane_id();
    const PairStep step((uint32_t)ev.n1);
    uint32_t cnt = 0;
    for (int k0 = 0; k0 < ev.n2; k0 += KCH) {
        const int nk = min(KCH, ev.n2 - k0);
        const int nk_pad = (nk + 3) & ~3;
        if constexpr (kPlanes) {
            if (!(staged && k0 == 0)) stage_pre<T>(x, y, z, ev, c, k0, nk, lds, lds + KCH);
        } else {
            for (int t = (int)lane; t < nk_pad; t += kWave) {
                float* h = lds + t * T::HF;
                if (t < nk) {
                    if constexpr (T::kZ)
                        T::stage(c, x[ev.o2 + k0 + t], y[ev.o2 + k0 + t], z[ev.o2 + k0 + t], h);
                    else
                        T::stage(c, x[ev.o2 + k0 + t], y[ev.o2 + k0 + t], h);
                } else {
#pragma unroll
                    for (int f = 0; f < T::HF; ++f) h[f] = __builtin_nanf("");
                }
            }
        }
        wave_lds_sync();
        const uint32_t p0 = t_begin * (uint32_t)kWave + lane;
        uint32_t i = p0 / step.n1, j = p0 - (p0 / step.n1) * step.n1;
        for (uint32_t t = t_begin; t < t_end; ++t) {
            const typename T::Pair pr = pair_of<T>(x, y, z, ev, c, i, j);
            // nk_pad is a multiple of 4: four layer-2 hits per iteration
            for (int k = 0; k < nk_pad; k += 4) {
                uint64_t m[4];
                if constexpr (kPlanes) {
                    const float4 vx = *reinterpret_cast<const float4*>(lds + k);
                    const float4 vy = *reinterpret_cast<const float4*>(lds + KCH + k);
                    const float h[8] = {vx.x, vy.x, vx.y, vy.y, vx.z, vy.z, vx.w, vy.w};
#pragma unroll
                    for (int u = 0; u < 4; ++u) m[u] = T::pass(c, pr, h + 2 * u);
                } else {
#pragma unroll
                    for (int u = 0; u < 4; ++u) m[u] = T::pass(c, pr, lds + (k + u) * T::HF);
                }
                cnt += (uint32_t)(__builtin_popcountll(m[0]) + __builtin_popcountll(m[1]) +
                                  __builtin_popcountll(m[2]) + __builtin_popcountll(m[3]));
            }
            step(i, j);
            if (cnt >= stop) break;  // wave-uniform
        }
        wave_lds_sync();
        if (cnt >= stop) break;
    }
    return cnt;
}

// The same with the rejecting test before the full one (see wave_count); false
// where it does not pay (cnt is then not the count; the first chunk is staged
// if the event has one only).
template <class T, int LF>
__device__ __forceinline__ bool wave_count_pre(const float* __restrict__ x, const float* __restrict__ y,
                                               const float* __restrict__ z, const EventRange& ev, uint32_t t_begin,
                                               uint32_t t_end, const Consts& c, float bound, float* __restrict__ lds,
                                               uint32_t& cnt) {
    constexpr int KCH = LF / 2;  // hits per chunk
    static_assert(KCH % 4 == 0, "chunk must hold whole float4 groups");
    const uint32_t stop = (uint32_t)c.count_cap;  // enough: the result is capped there
    float* wx = lds;
    float* wy = lds + KCH;
    const unsigned lane = lane_id();
    const uint32_t n0 = (uint32_t)ev.n0;
    const PairStep step((uint32_t)ev.n1);
    const float nan = __builtin_nanf("");
    cnt = 0;
    int32_t budget = T::kNear;  // of groups (a tile and four hits) taken on
    for (int k0 = 0; k0 < ev.n2; k0 += KCH) {
        const int nk = min(KCH, ev.n2 - k0);
        const int nk_pad = (nk + 3) & ~3;
        const float own = stage_pre<T>(x, y, z, ev, c, k0, nk, wx, wy);
        wave_lds_sync();
        // (MsdFitTest: by its bound and M, before anything is staged)
        const bool check = T::HF == 2 || (T::kZ && t_end - t_begin > 4u);
        if (check && k0 == 0 &&
            2 * __builtin_popcountll(lanes((int)lane < nk && own <= bound * T::kLoose)) >= min(nk, kWave))
            return false;
        const uint32_t p0 = t_begin * (uint32_t)kWave + lane;
        uint32_t i = p0 / step.n1, j = p0 - (p0 / step.n1) * step.n1;  // the lane's pair of tile t
        uint32_t t = t_begin;
        auto tiles = [&](auto np) {
            constexpr int NP = decltype(np)::value;
            float2 p[NP];
            uint32_t in = i, jn = j;
#pragma unroll
            for (int q = 0; q < NP; ++q) {
                const bool v = in < n0;
                const int hi = ev.o0 + (int)min(in, n0 - 1), hj = ev.o1 + (int)jn;
                if constexpr (T::kZ)
                    p[q] = T::pre_pair(c, x[hi], y[hi], z[hi], x[hj], y[hj], z[hj]);
                else
                    p[q] = T::pre_pair(c, x[hi], y[hi], x[hj], y[hj]);
                p[q].x = v ? p[q].x : nan;
                p[q].y = v ? p[q].y : nan;
                step(in, jn);
            }
            // nk_pad is a multiple of 4: four layer-2 hits per iteration
            for (int k = 0; k < nk_pad; k += 4) {
                const float4 vx = *reinterpret_cast<const float4*>(wx + k);
                const float4 vy = *reinterpret_cast<const float4*>(wy + k);
                // the smallest sum over q's four triplets and `from`
                auto fold = [&](int q, float from) {
                    const float s0 = __builtin_fabsf(p[q].x + vx.x) + __builtin_fabsf(p[q].y + vy.x);
                    const float s1 = __builtin_fabsf(p[q].x + vx.y) + __builtin_fabsf(p[q].y + vy.y);
                    const float s2 = __builtin_fabsf(p[q].x + vx.z) + __builtin_fabsf(p[q].y + vy.z);
                    const float s3 = __builtin_fabsf(p[q].x + vx.w) + __builtin_fabsf(p[q].y + vy.w);
                    const float m = __builtin_fminf(__builtin_fminf(from, s0), s1);
                    return __builtin_fminf(__builtin_fminf(m, s2), s3);
                };
                float m = nan;  // fmin drops NaN; all NaN stays NaN and fails
#pragma unroll
                for (int q = 0; q < NP; ++q) m = fold(q, m);
                if (!wave_any(m <= bound)) continue;
                if constexpr (T::kPreTests) {
#pragma unroll
                    for (int q = 0; q < NP; ++q)
                        cnt += (uint32_t)(__builtin_popcountll(T::pre_pass(c, p[q], vx.x, vy.x)) +
                                          __builtin_popcountll(T::pre_pass(c, p[q], vx.y, vy.y)) +
                                          __builtin_popcountll(T::pre_pass(c, p[q], vx.z, vy.z)) +
                                          __builtin_popcountll(T::pre_pass(c, p[q], vx.w, vy.w)));
                    budget -= NP;
                } else {
                    uint32_t near = 1u;  // the tiles to take on
                    if constexpr (NP > 1) {
                        near = 0u;
#pragma unroll
                        for (int q = 0; q < NP; ++q) near |= wave_any(fold(q, nan) <= bound) ? 1u << q : 0u;
                    }
                    budget -= __builtin_popcount(near);
                    uint32_t pi = i, pj = j;
#pragma unroll 1
                    for (; near; near >>= 1, step(pi, pj)) {
                        if (!(near & 1u)) continue;
                        const typename T::Pair pr = pair_of<T>(x, y, z, ev, c, pi, pj);
#pragma unroll 1
                        for (int kk = k; kk < min(k + 4, nk); ++kk) {
                            float h[T::HF];
                            const int h2 = ev.o2 + k0 + kk;
                            if constexpr (T::HF == 2) {
                                h[0] = wx[kk];
                                h[1] = wy[kk];
                            } else if constexpr (T::kZ) {
                                T::stage(c, x[h2], y[h2], z[h2], h);
                            } else {
                                T::stage(c, x[h2], y[h2], h);
                            }
                            cnt += (uint32_t)__builtin_popcountll(T::pass(c, pr, h));
                        }
                    }
                }
            }
            budget += (int32_t)(NP * nk_pad) >> T::kShare;  // its share of the tiles' groups
            i = in;
            j = jn;
            t += NP;
        };
        // wave-uniform control flow
        while (t + 4 <= t_end && cnt < stop && budget >= 0) tiles(std::integral_constant<int, 4>{});
        if (t + 2 <= t_end && cnt < stop && budget >= 0) tiles(std::integral_constant<int, 2>{});
        if (t < t_end && cnt < stop && budget >= 0) tiles(std::integral_constant<int, 1>{});
        wave_lds_sync();
        if (cnt >= stop) return true;
        if (t < t_end) return false;  // out of budget
    }
    return true;
}

// Passing triplets of a small event, one tile of pairs and at most kTileHits
// layer-2 hits (T::kTile tests): lane p holds pair p and layer-2 hit p, all in
// one round trip and without LDS; the layer-2 values reach the lanes through
// scalar registers.  Bound by instructions and that round trip: 450,000 events
// of 4 hits per layer, whole call, MSD 147 us by wave_count, 97 here, basis form
// 137 and 91; of 6 hits 157 and 120, 146 and 111.  At more layer-2 hits the two
// meet (9 hits, of which some events still are one tile: 180 and 171).
constexpr int kTileHits = 16;

__device__ __forceinline__ bool one_tile(const EventRange& ev) {
    return (uint64_t)ev.n0 * (uint64_t)ev.n1 <= (uint64_t)kWave && ev.n2 <= kTileHits;
}

// (n0, n1, n2 > 0)
template <class T>
__device__ __forceinline__ uint32_t wave_count_tile(const float* __restrict__ x, const float* __restrict__ y,
                                                    const EventRange& ev, const Consts& c) {
    const int lane = (int)lane_id();
    // lane / n1: the quotient's distance from a whole number, 0.5 / n1, is far
    // above its error
    const int i = (int)(((float)lane + 0.5f) * __builtin_amdgcn_rcpf((float)ev.n1)), j = lane - i * ev.n1;
    const bool v = i < ev.n0;
    const int hi = ev.o0 + min(i, ev.n0 - 1), hj = ev.o1 + j, hk = ev.o2 + min(lane, ev.n2 - 1);
    const float xi = x[hi], yi = y[hi], xj = x[hj], yj = y[hj], xk = x[hk], yk = y[hk];
    const float2 p = T::pre_pair(c, xi, yi, xj, yj), w = T::pre_k(c, xk, yk);
    const float bound = T::bound(c, __builtin_fmaxf(__builtin_fabsf(xj), __builtin_fabsf(yj)));
    auto of_hit = [](float f, int k) {
        return __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(f), k));
    };
    float m = __builtin_nanf("");  // fmin drops NaN; all NaN fails
    for (int k = 0; k < ev.n2; ++k)
        m = __builtin_fminf(m, __builtin_fabsf(p.x + of_hit(w.x, k)) + __builtin_fabsf(p.y + of_hit(w.y, k)));
    if (!wave_any(v && m <= bound) && bound < __builtin_inff()) return 0u;
    const typename T::Pair pr = v ? T::pair(c, xi, yi, xj, yj) : T::invalid();
    float own[T::HF];
    T::stage(c, xk, yk, own);
    uint32_t cnt = 0;
#pragma unroll 2
    for (int k = 0; k < ev.n2; ++k) {
        float h[T::HF];
#pragma unroll
        for (int f = 0; f < T::HF; ++f) h[f] = of_hit(own[f], k);
        cnt += (uint32_t)__builtin_popcountll(T::pass(c, pr, h));
    }
    return cnt;
}

// Passing triplets of one event over pair tiles [t_begin, t_end); each tile
// is 64 consecutive (i, j) pairs in row-major order (pair p -> i = p / n1,
// j = p % n1), one pair per lane, looping over every layer-2 hit staged in
// this wave's LF floats of LDS (16-byte aligned).  Called by a whole wave with
// uniform arguments; returns the same count on every lane.
//
// Every triplet gets the rejecting test of the policy (three sums and half a
// min3 on the vector unit: 8 SIMD cycles against 60 of the written-out fit),
// on the sum of the two planes' magnitudes, folded over four layer-2 hits and
// the lane's NP pairs before one vote; only a tile and group of four hits in
// which some triplet is within the bound is evaluated in full.  (A sum takes 2
// SIMD cycles for 64 lanes, a max or min 4: the sum of the magnitudes instead
// of the larger one saves 2 of 10 and lets twice as many of the few close
// triplets through.)  NP pairs per lane share one 16-byte LDS read per plane
// and four layer-2 hits: with one pair per lane those reads (all lanes at one
// address, still 1 KB each on a 128 B/clock LDS) take longer than the sums.
// Bound by the vector unit.  100,000 events of 30 hits per layer, whole call:
// 1.335 ms with the full test per triplet, 0.246 ms now (2.7e9 triplets; 0.14 ms
// at 8 SIMD cycles per 64 of them and 2.4 GHz).
//
// The rejecting test pays while few groups are taken on.  So an event goes to
// the staged full test (wave_count_full) at once if no bound holds or if kLoose
// times the bound reaches at least half of its layer-2 hits' |pre_k| (of the
// first 64; MsdFitTest: about |V2| M): with sums spread evenly over +-S, median
// 3/4 S, the share of groups (256 triplets) with one within B is 128 (B / S)^2
// (MSD; 0.5 at 1/16), 12 / 2 (B / S)^2 per-hit z at 30 hits per layer, and for
// the window tests, whose pairs have passed the layer-1 window, 512 (B / 2
// S)^4.  Events of another kind (many tracks) go there, from the start again,
// once more than kNear groups and a share of 2^(2 - kShare) of them were taken
// on.  20,000 events of 30 hits per layer, cuts 1, 10 and 100 times the default
// in cm, us: MSD 58, 129, 329 (always the full test: 326), basis form 56, 101,
// 126 (124), window 81, 87, 116 (115); each hit on a track: MSD 130 (280),
// window 81 (94).
template <class T, int LF>
__device__ uint32_t wave_count(const float* __restrict__ x, const float* __restrict__ y,
                               const float* __restrict__ z, const EventRange& ev, uint32_t t_begin,
                               uint32_t t_end, const Consts& c, const PreBound& pb, float* __restrict__ lds) {
    uint32_t cnt;
    const bool pre = pb.valid && (T::kMinHits <= 1 || ev.n2 >= T::kMinHits);  // (n2 > 0)
    if (pre && wave_count_pre<T, LF>(x, y, z, ev, t_begin, t_end, c, pb.bound, lds, cnt)) return cnt;
    return wave_count_full<T, LF>(x, y, z, ev, t_begin, t_end, c, lds, pre && ev.n2 <= LF / 2);
}

}  // namespace trig

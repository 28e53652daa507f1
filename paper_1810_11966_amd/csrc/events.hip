// Event building from a time-ordered hit stream (include/trig_events.h):
// time-gap clustering, the reading this library takes of the paper's outlook
// on free-streaming data (Sec. 8), which gives no algorithm.
//
// Partition: a workgroup of 4 waves owns kEbHits consecutive hits; wave w
// takes the kEbRounds * 128 hits from (4 b + w) * kEbWaveHits on, 128 per
// round, lane L on hits 128 r + 2 L and the one after it (one 16-byte load).
// An odd hit's predecessor is the lane's even one, an even hit's the odd hit
// of the lane below (a wave shift), lane 0's the previous round's last (or,
// for a wave's first round, one scalar load).  The count kernel writes each
// round's two ballots of event starts, of its even and of its odd hits, to a
// bit mask in the workspace (one bit per hit), the wave's count and the
// workgroup's total; the scan turns the totals into positions (streams of at
// most kEbSelfPrefix workgroups: each sums the totals before its own); the
// scatter kernel gives each of a wave's rounds (one lane per round) its first
// position by a wave scan of the masks' popcounts and writes the hit index of
// every set bit.
//
// Bound by reading the times.  100 million hits, the whole call: 159 us with
// one 8-byte load per lane and round and shuffles through the LDS, 144 us
// (5.6 TB/s) now.  The non-temporal loads of long streams matter: with the
// default policy the same kernel took 160, 166, 162, 156 us with 16, 8, 4, 2
// rounds in flight, against 152, 147, 144 for 8, 4, 2 so.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "scan_i64.hpp"
#include "trig.h"
#include "trig_device.hpp"
#include "trig_events.h"

namespace {

constexpr int kEbWaves = 4;
constexpr int kEbThreads = kEbWaves * trig::kWave;
constexpr int kEbRounds = 32;  // rounds of 128 hits per wave (lane r holds round r's masks)
static_assert(kEbRounds <= trig::kWave, "one lane per round's masks");
constexpr int64_t kEbRoundHits = 2 * trig::kWave;
constexpr int64_t kEbWaveHits = kEbRounds * kEbRoundHits;
constexpr int64_t kEbHits = kEbWaveHits * kEbWaves;  // hits per workgroup
constexpr int64_t kEbMaxHits = (int64_t)1 << 40;

// Does hit h (time tc, predecessor's time tp) start an event: h == 0, or a
// later time by more than gap (the exact difference: for tc > tp the
// unsigned difference of the two int64 values is the true one).
__device__ __forceinline__ bool starts(int64_t h, int64_t tc, int64_t tp, uint64_t gap) {
    return h == 0 || (tc > tp && (uint64_t)tc - (uint64_t)tp > gap);
}

// The previous lane's int64 value (lane 0 gets `first`): a shift over the
// whole wave on the vector unit.
__device__ __forceinline__ int64_t from_lane_below(int64_t v, int64_t first) {
    constexpr int kWaveShr1 = 0x138;
    const int lo = __builtin_amdgcn_update_dpp((int)(uint32_t)first, (int)(uint32_t)v, kWaveShr1, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp((int)(uint32_t)((uint64_t)first >> 32),
                                               (int)(uint32_t)((uint64_t)v >> 32), kWaveShr1, 0xF, 0xF, false);
    return (int64_t)(((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo);
}

typedef int64_t i64x2 __attribute__((ext_vector_type(2)));

// Streams beyond this many hits (320 MiB of times) do not fit the 256 MiB
// last-level cache: their loads are non-temporal with two rounds in flight;
// shorter ones keep the default policy, which finds what an earlier kernel
// wrote there, with eight.  Whole calls, long form against short: 60 million
// hits 89 against 102 us, 50 million 74 and 85, 40 million 66 and 65, 30 million
// 47.4 and 46.9, 20 million 32.4 and 34.7, 8 million 24 and 20.
constexpr int64_t kEbLongHits = (int64_t)40 << 20;

// VEC: t is 16-byte aligned.  LONG: see kEbLongHits.
template <bool VEC, bool LONG>
__global__ __launch_bounds__(kEbThreads) void k_eb_count(const int64_t* __restrict__ t, int64_t n, uint64_t gap,
                                                         uint64_t* __restrict__ masks, int32_t* __restrict__ wcount,
                                                         int64_t* __restrict__ partials, uint32_t* status) {
    __shared__ int32_t wave_total[kEbWaves];
    const int w = trig::uniform_i((int)(threadIdx.x / trig::kWave));
    const int lane = (int)trig::lane_id();
    const int64_t gw = (int64_t)blockIdx.x * kEbWaves + w;
    const int64_t h0 = gw * kEbWaveHits;
    // the hit before the wave's first (scalar load)
    int64_t carry = (h0 > 0 && h0 - 1 < n) ? t[h0 - 1] : 0;
    uint64_t even = 0u, odd = 0u;  // lane r: round r's masks
    int32_t cnt = 0;
    bool bad = false;
    constexpr int kBatch = LONG ? 2 : 8;  // rounds whose loads are in flight together
#pragma unroll 1
    for (int r0 = 0; r0 < kEbRounds; r0 += kBatch) {
        const int64_t b0 = h0 + r0 * kEbRoundHits;
        if (b0 >= n) break;  // wave-uniform
        const bool full = b0 + kBatch * kEbRoundHits <= n;  // wave-uniform
        i64x2 tv[kBatch];
        if (VEC && full) {
#pragma unroll
            for (int k = 0; k < kBatch; ++k) {
                const auto* p = reinterpret_cast<const i64x2*>(t + b0 + k * kEbRoundHits + 2 * lane);
                tv[k] = LONG ? __builtin_nontemporal_load(p) : *p;
            }
        } else if (full) {
#pragma unroll
            for (int k = 0; k < kBatch; ++k) {
                const int64_t* p = t + b0 + k * kEbRoundHits + 2 * lane;
                tv[k].x = LONG ? __builtin_nontemporal_load(p) : p[0];
                tv[k].y = LONG ? __builtin_nontemporal_load(p + 1) : p[1];
            }
        } else {
#pragma unroll
            for (int k = 0; k < kBatch; ++k) {
                const int64_t h = b0 + k * kEbRoundHits + 2 * lane;
                tv[k].x = h < n ? t[h] : 0;
                tv[k].y = h + 1 < n ? t[h + 1] : 0;
            }
        }
#pragma unroll
        for (int k = 0; k < kBatch; ++k) {
            const int64_t h = b0 + k * kEbRoundHits + 2 * lane;
            const bool v0 = full || h < n, v1 = full || h + 1 < n;
            const int64_t tp = from_lane_below(tv[k].y, carry);
            bad |= (v0 && h > 0 && tv[k].x < tp) || (v1 && tv[k].y < tv[k].x);
            const uint64_t m0 = trig::lanes(v0 && starts(h, tv[k].x, tp, gap));
            const uint64_t m1 = trig::lanes(v1 && starts(h + 1, tv[k].y, tv[k].x, gap));
            cnt += (int32_t)(__builtin_popcountll(m0) + __builtin_popcountll(m1));
            even = lane == r0 + k ? m0 : even;
            odd = lane == r0 + k ? m1 : odd;
            const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)tv[k].y, 63);
            const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)tv[k].y >> 32), 63);
            carry = (int64_t)(((uint64_t)hi << 32) | lo);
        }
    }
    if (lane < kEbRounds) {
        masks[gw * 2 * kEbRounds + 2 * lane] = even;
        masks[gw * 2 * kEbRounds + 2 * lane + 1] = odd;
    }
    if (trig::wave_any(bad) && lane == 0 && status) atomicOr(status, TRIG_EVENTS_UNSORTED);
    if (lane == 0) {
        wcount[gw] = cnt;
        wave_total[w] = cnt;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        int64_t s = 0;
        for (int k = 0; k < kEbWaves; ++k) s += wave_total[k];
        partials[blockIdx.x] = s;
    }
}

// Streams of at most this many workgroups (25 million hits): each wave sums
// the totals of the workgroups before its own (at most 12 KB from L2) instead
// of a scan kernel.  Whole calls with the sums and with the scan: 8 million
// hits 17.3 and 19.6 us, 20 million 33.6 and 34.7, 24 million 38.0 and 38.4, 30
// million 47.5 and 46.9.
constexpr int kEbSelfPrefix = 1536;

__global__ __launch_bounds__(kEbThreads) void k_eb_scatter(int64_t n, const uint64_t* __restrict__ masks,
                                                           const int32_t* __restrict__ wcount,
                                                           const int64_t* __restrict__ partials, int n_blocks,
                                                           int64_t* __restrict__ out, int64_t cap,
                                                           int64_t* __restrict__ out_n, uint32_t* status) {
    const int w = trig::uniform_i((int)(threadIdx.x / trig::kWave));
    const int lane = (int)trig::lane_id();
    const int64_t gw = (int64_t)blockIdx.x * kEbWaves + w;
    const int64_t h0 = gw * kEbWaveHits;
    const uint64_t even = lane < kEbRounds ? masks[gw * 2 * kEbRounds + 2 * lane] : 0u;
    const uint64_t odd = lane < kEbRounds ? masks[gw * 2 * kEbRounds + 2 * lane + 1] : 0u;
    const bool self = n_blocks <= kEbSelfPrefix;
    const int64_t first = self ? wave_prefix_i64(partials, (int)blockIdx.x) : partials[blockIdx.x];
    int64_t base = first;
    for (int k = 0; k < w; ++k) base += wcount[(int64_t)blockIdx.x * kEbWaves + k];
    const int pc = __builtin_popcountll(even) + __builtin_popcountll(odd);
    int64_t pos = base + (trig::wave_inclusive_sum(pc) - pc);
    for (uint64_t bits = even | odd; bits; bits &= bits - 1u) {  // event starts are sparse
        const int i = __builtin_ctzll(bits);
        const int64_t h = h0 + kEbRoundHits * lane + 2 * i;
        if ((even >> i) & 1u) {
            if (pos < cap) out[pos] = h;
            ++pos;
        }
        if ((odd >> i) & 1u) {
            if (pos < cap) out[pos] = h + 1;
            ++pos;
        }
    }
    if ((int)blockIdx.x == n_blocks - 1 && threadIdx.x == 0) {
        const int64_t e = self ? first + partials[blockIdx.x] : partials[n_blocks];
        if (e < cap) out[e] = n;
        if (e + 1 > cap && status) atomicOr(status, TRIG_EVENTS_CAPACITY);
        *out_n = e;
    }
}

__global__ void k_eb_empty(int64_t* out, int64_t* out_n) {
    out[0] = 0;
    *out_n = 0;
}

size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }

int64_t eb_blocks(int64_t n) { return (n + kEbHits - 1) / kEbHits; }

}  // namespace

extern "C" {

size_t trig_build_events_workspace_bytes(int64_t n_hits) {
    if (n_hits < 0 || n_hits > kEbMaxHits) return 0;
    const int64_t nb = std::max<int64_t>(1, eb_blocks(n_hits));
    return align256(sizeof(uint64_t) * (size_t)(nb * kEbWaves * 2 * kEbRounds)) +
           align256(sizeof(int32_t) * (size_t)(nb * kEbWaves)) + align256(sizeof(int64_t) * (size_t)(nb + 1));
}

int trig_build_events(const int64_t* t, int64_t n_hits, int64_t gap, int64_t* out_offsets, int64_t out_capacity,
                      int64_t* out_n_events, uint32_t* out_status, void* workspace, size_t workspace_bytes,
                      void* stream) {
    if (n_hits < 0 || n_hits > kEbMaxHits || gap < 0 || out_capacity < 1 || !out_offsets || !out_n_events)
        return TRIG_EINVAL;
    if (n_hits > 0 && !t) return TRIG_EINVAL;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    if (n_hits == 0) {
        hipLaunchKernelGGL(k_eb_empty, dim3(1), dim3(1), 0, s, out_offsets, out_n_events);
        return hipGetLastError() == hipSuccess ? TRIG_OK : TRIG_EHIP;
    }
    const size_t need = trig_build_events_workspace_bytes(n_hits);
    if (!workspace || workspace_bytes < need || (reinterpret_cast<uintptr_t>(workspace) & 255)) return TRIG_EINVAL;
    const int64_t nb = eb_blocks(n_hits);  // <= 2^40 / 16384 = 2^26
    char* ws = static_cast<char*>(workspace);
    auto* masks = reinterpret_cast<uint64_t*>(ws);
    const size_t mask_bytes = align256(sizeof(uint64_t) * (size_t)(nb * kEbWaves * 2 * kEbRounds));
    auto* wcount = reinterpret_cast<int32_t*>(ws + mask_bytes);
    auto* partials = reinterpret_cast<int64_t*>(ws + mask_bytes + align256(sizeof(int32_t) * (size_t)(nb * kEbWaves)));
    const bool vec = (reinterpret_cast<uintptr_t>(t) & 15) == 0;
    const bool big = n_hits > kEbLongHits;
    const auto kern = vec ? (big ? k_eb_count<true, true> : k_eb_count<true, false>)
                          : (big ? k_eb_count<false, true> : k_eb_count<false, false>);
    hipLaunchKernelGGL(kern, dim3((unsigned)nb), dim3(kEbThreads), 0, s, t, n_hits,
                       (uint64_t)gap, masks, wcount, partials, out_status);
    if (hipGetLastError() != hipSuccess) return TRIG_EHIP;
    if (nb > kEbSelfPrefix) {
        hipLaunchKernelGGL(k_scan_i64, dim3(1), dim3(kScanThreads), 0, s, partials, nb);
        if (hipGetLastError() != hipSuccess) return TRIG_EHIP;
    }
    hipLaunchKernelGGL(k_eb_scatter, dim3((unsigned)nb), dim3(kEbThreads), 0, s, n_hits, masks, wcount, partials,
                       (int)nb, out_offsets, out_capacity, out_n_events, out_status);
    return hipGetLastError() == hipSuccess ? TRIG_OK : TRIG_EHIP;
}

}  // extern "C"

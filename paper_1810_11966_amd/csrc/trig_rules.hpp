// Rules that choose a launch shape or a kernel from the sizes of a batch.
// Plain C++ (no HIP): the library's host code and a CPU test (g++) compile the
// same file.  `cus`: compute units of the device.
#pragma once

#include <algorithm>
#include <cmath>
#include <cstdint>

namespace trig_rules {

constexpr int kMaxEvents = 128;       // events per block, at most
constexpr int kRuleHits = 2048;       // batched form: hit capacity of a block, its waves
constexpr int kRuleWaves = 4;
constexpr double kRuleFill = 0.92;    // and hits per block over the capacity
constexpr int kLargeHits = 4096;      // the larger capacity

// Hits per event of a batch, at least one.
inline double mean_hits(int n_events, int n_hits) {
    return std::max(n_events > 0 ? (double)n_hits / n_events : 1.0, 1.0);
}

// Events per block that fill `fill` of an hb-hit block at the batch's mean
// event size, in whole rounds over nw waves.
inline int events_for_fill(double fill, int hb, int nw, int n_events, int n_hits) {
    int eb = (int)std::max(1.0, std::min((double)kMaxEvents, std::floor(fill * hb / mean_hits(n_events, n_hits))));
    if (nw > 0 && eb >= nw) eb -= eb % nw;
    return eb;
}

// The same, but no more than spread the batch over `blocks` blocks per compute
// unit, and at least one event per wave.
inline int spread_events(int eb, int nw, int n_events, int cus, int blocks) {
    const int64_t waves = std::max(nw, 1), per = (int64_t)cus * blocks;
    const int64_t spread = ((n_events + per - 1) / per + waves - 1) / waves * waves;
    return (int)std::min<int64_t>(eb, std::max(waves, spread));
}

// Shape of the batched form: LDS hit capacity (hb), waves per workgroup (nw)
// and events per block (eb).  Given values (> 0) are used as they are.
//
// Default without stealing: kRuleHits hits and kRuleWaves waves, eight
// workgroups on a CU (seven with more than 52 events in a block), at every
// multiplicity, filled to kRuleFill of the capacity by events of the batch's
// mean size (a block that overflows is split into sub-blocks by the kernel).
// Whole calls, MSD, this shape against 1024 hits and 2 waves and 4096 and 4:
// a million events of 15 hits per layer 120, 140, - us; 60,000 of 100 hits 84,
// 90, 104; 30,000 of 200 hits 156, 257, 207; 5,000 of 450 hits 290, 221, 301
// (the binned form's field); only at 300 hits with the window test was 4096
// faster (364 against 354).  300,000 events of 30 hits take 63.6 us at a fill of
// 0.92 and 67.3 at 0.85 (20 and 16 events per block).
// Batches whose blocks run all at once take smaller ones, kSmallBlocks per CU:
// the time is a block's own (1,000 events of 15 hits per layer: 7.7 us at 18
// events per block, 5.4 us at one or two per wave; 25,000 uneven events of 54
// hits, window test, 14.0 us at four blocks per CU, 10.7 at eight).  If all run
// at once with kLargeHits too (four per CU) and four events would as often as
// not overflow kRuleHits, they take that (600 uneven events of 450 hits: 56.6 us
// with 2048, 35.3 with 4096).
//
// Default with stealing: its claims pass one counter and its registers leave
// five workgroups on a CU (three with kLargeHits), so fewer, larger blocks are
// better: one per CU in small batches (4,000 events of 15 hits per layer: 16.5 us,
// at four per CU 40.8), and kLargeHits where they still give every CU one
// (100,000 events of 25 hits per layer: 62 against 90 us; 8,000: 24.5 against
// 23.3) or four events come near kRuleHits (50,000 of 200 hits: 357 against
// 398; 40,000 of 140 hits, window test, 236 against 224, but uneven events of
// 200 hits 375 against 398).  Those hold kStealEvents, or 0.6 of what fits,
// while a CU has fewer than kStealParts blocks: stealing is for batches whose heavy events lie
// together, in blocks that are cut up (300,000 events, the first 2 % of 240
// hits per layer and the rest of 10: 84 events per block 966 us, 48 of them 589,
// 2048 hits and 40 events 666; even events lose less, 100,000 of 25 hits 78 for
// 62; a million of 30 would take 309 for 278, 50,000 of 100 at four 187 for 130).  A claim of many large events
// holds its workgroup for long, so batches of few and large events take
// kLargeHits and four of them at a time, or eight where there are more and they
// fit (events of 100 to 150 hits per layer, four, eight and twelve at a time:
// 4,000 uneven ones 64, 71 and 98 us, 20,000 116, 119 and 137; 6,000 even ones of
// 100 hits, MSD 61, 57 and 57, window 61, 62 and 69; 1,900 of 200 hits 65, 104
// and, with 2048, 89).
struct BlockShape {
    int hb, nw, eb;
};
constexpr int kSmallBlocks = 8, kStealBlocks = 1, kStealParts = 40, kStealEvents = 28;

inline BlockShape choose_block_shape(int hb, int nw, int eb, bool stealing, int n_events, int n_hits, int cus) {
    const double mean = mean_hits(n_events, n_hits);
    if (hb <= 0) {
        hb = kRuleHits;
        const double four = mean * kRuleWaves, waves = (double)kRuleWaves * cus;  // hits of four events
        const bool choose = nw <= 0 && eb <= 0;
        if (!stealing) {
            if (choose && four > 0.6 * kRuleHits && n_events <= 4 * waves) {
                hb = kLargeHits;
                eb = kRuleWaves;
            }
        } else if (choose && four > 0.4 * kRuleHits && n_events <= (four > 0.55 * kRuleHits ? 20 : 8) * waves) {
            hb = kLargeHits;
            eb = n_events <= (four > 0.55 * kRuleHits ? 4 : 2) * waves || 2.0 * four > 0.6 * kLargeHits ? kRuleWaves
                                                                                                     : 2 * kRuleWaves;
        } else if (n_hits >= (double)cus * kRuleFill * kLargeHits || four > 0.75 * kRuleHits) {
            hb = kLargeHits;
        }
    }
    if (nw <= 0) nw = std::min(kRuleWaves, hb / 512);
    if (eb <= 0) {
        eb = spread_events(events_for_fill(kRuleFill, hb, nw, n_events, n_hits), nw, n_events, cus,
                           stealing ? kStealBlocks : kSmallBlocks);
        if (stealing && hb == kLargeHits) {
            const int most = n_events / (kStealParts * cus) / nw * nw;
            const int part = events_for_fill(0.6 * kRuleFill, hb, nw, n_events, n_hits);
            eb = std::min(eb, std::max({part, most, kStealEvents}));
        }
    }
    return {hb, nw, eb};
}

// Per-hit z: whether blocks of events staged in LDS (k_block_z: kZHits hits,
// kZWaves waves) are faster than a wave per event from HBM (k_event_z).  They
// need 16-byte aligned arrays (without, nothing is staged: 100,000 events of 70
// hits per layer 127 us for 122) and at least kMinZEvents events of the mean
// size, two per wave.  A block's barrier and its longest wave show while the
// events' own waves would run all at once (8,192 events): in whole calls, blocks
// against waves, 10,000 events of 8 hits per layer take 6.4 and 7.1 us (MSD), of
// 60 hits 16.8 and 14.9, 20,000 20.5 and 23.5.  With the window test more events
// have close pairs, and their completion from HBM is spread less evenly: 20,000
// of 8 hits 8.0 and 9.0, of 30 hits 17.7 and 13.0, 80,000 33.9 and 37.3, of 60
// hits 83.9 and 75.4.
constexpr int kZHits = 2048, kZWaves = 4;
constexpr int kMinZEvents = 8;

inline bool blocks_z(bool aligned, bool window, int n_events, int n_hits) {
    const double mean = mean_hits(n_events, n_hits);
    if (!aligned || mean * kMinZEvents > kRuleFill * kZHits) return false;
    if (window) return mean <= 120.0 && n_events >= std::max(8192.0, 720.0 * mean);
    return n_events >= std::max(8192.0, 90.0 * mean);
}

// Station filter: events per wave (of kFilterWaves per workgroup, 1, 2 or
// kFilterMaxPer) and whether the scatter's workgroups sum the totals before
// their own (self) instead of a scan kernel between the two.
//
// Fewer events per wave keep more loads in flight while the GPU is not full;
// more workgroups cost prologues and longer sums.  Whole calls at one, two and
// four per wave with the sums, events of 194 hits: 4,000 events 11.0, 11.3 and
// 14.7 us, 6,000 13.4, 12.9 and 16.7, 10,000 18.6, 16.0 and 18.8, 13,000 23.4,
// 20.9 and 20.8, 20,000 32.7, 26.2 and 25.3.  Of large events (kFilterLarge
// hits) a wave has more to read, and fewer are the better for longer: 8,000
// events of 5,004 hits 23.1, 21.6 and 25.4, in random station order 42.5, 44.1
// and 48.6, 16,000 36.7, 32.3 and 33.9, 32,000 of 1,260 hits in random order
// 93.7, 91.2 and 96.7.  The scan and its gap take 5 us: with it
// 4,000 events take 13.3 us, 32,000 36.0 against 34.1 with the sums, 50,000
// 50.1 and 49.8, 80,000 in random order 86.2 and 89.5.
constexpr int kFilterWaves = 4, kFilterMaxPer = 4;
constexpr int kFilterOne = 6144, kFilterTwo = 12288;  // at most this many events: one, two per wave
constexpr int kFilterLarge = 1000, kFilterLargeOne = 8192, kFilterLargeTwo = 32768;
constexpr int kFilterSelf = 49152;  // and at most this many: the sums

struct FilterShape {
    int per;    // events per wave
    bool self;  // (one or two per wave always)
};

inline FilterShape filter_shape(int n_events, int64_t n_hits) {
    const bool large = n_events > 0 && n_hits / n_events >= kFilterLarge;
    const int per = n_events <= (large ? kFilterLargeOne : kFilterOne)   ? 1
                    : n_events <= (large ? kFilterLargeTwo : kFilterTwo) ? 2
                                                                         : kFilterMaxPer;
    return {per, n_events <= kFilterSelf};
}

}  // namespace trig_rules

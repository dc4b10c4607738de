// Rules of the host runtime that need no GPU: the library's own bin table, and which
// launches a call takes.
#pragma once

#include <stdint.h>

#include <algorithm>
#include <cmath>

namespace ph {

// One bin of the FP32 sweep: reads up to max_m bases in groups of P lanes x
// K rows.  A table line may add a haplotype-length split "n_split P2 K2":
// pairs of that read range whose haplotype has at least n_split bases go to
// a second bin of P2 x K2 (a table entry that follows its parent, with the
// same max_m, so that the read-length map never selects it).
struct TuneEntry {
    int max_m, P, K;
    int n_split = 0, P2 = 0, K2 = 0;
};

// The library's own bin table, shortest reads first: 16 lanes x K rows
// (K = 1..16) up to 255 bases, then 64 lanes x K rows (K = 5..16).  Written
// into a fixed array (the allocation-free forward uses it too); returns the
// number of entries.
inline int builtin_table(TuneEntry *t)
{
    int n = 0;
    for (int K = 1; K <= 16; ++K) t[n++] = {16 * K - 1, 16, K};
    for (int K = 5; K <= 16; ++K) t[n++] = {64 * K - 1, 64, K};
    return n;
}

// its entry for reads of m bases (1 to 1,023)
inline int builtin_entry(int m) { return m < 256 ? m >> 4 : 12 + (m >> 6); }

// Which way a call goes: one launch of one-pair tiles (k_one), or the binned
// launches.  Both are priced by their tiles, in ns: a step of K rows takes a SIMD
// 19 + 13 K clocks where the GPU is full (step_ns, of the whole GPU; measured with
// 150,000 pairs of 10 to 250 bases), a tile alone 2 ns per vector instruction, about
// 5.5 K + 10 of them per step (tile_ns).
//
// One-pair tiles take 64 lanes each and 130 steps beside their columns; half of the
// longest tile adds to their sum.  Binned tiles pad fewer rows and lanes, but their
// launches take 55 us and 9 more for every further bin (without a plan 45 us, 9 per
// bin, 4.9 ns a pair, beyond 15,000 pairs 1.5, 6 a batch), single pairs 2.5 ns beside
// their steps (0.6 in 4 lanes, 1.3 in 8), and every bin's kernel ends with its longest
// tile: a plan's bins on side streams in turn, otherwise one after the other; the
// tiles' sum and those ends overlap in part.  13 to 16 rows in 16 lanes run at 2 waves
// per SIMD.  Some of the 1,001 shapes that this was fitted to (1 to 60 reads and 1 to
// 20 haplotypes a region), us, binned / one-pair, and the way taken where it is the
// longer one:
//   10 x 300 bases: 4,500 pairs 62 / 47, 15,000 79 / 113
//   60 x 300: 15,000 130 / 111, 45,000 227 / 302; 60 x 4,000: 4,500 388 / 362, 15,000
//   653 / 995; 60 x 150, two haplotypes: 24,800 133 / 109 (binned)
//   150 x 300: 15,000 204 / 181, 45,000 352 / 500; 150 x 1,000: 4,500 205 / 177,
//   15,000 384 / 470
//   100-150 x 1,010, four bins: 12,000 376 / 328; 60-250 x 350, 14 bins: 60,000 738 /
//   804 (one-pair); 50-250 x 1,000: 15,000 782 / 453, 150,000 3,298 / 4,079
//   without a plan: 10 x 1,000, 4,500 118 / 99, 15,000 200 / 272; 100 x 1,000, 4,500
//   183 / 126, 15,000 306 / 351; 50-250 x 1,000, 45,000 2,090 / 1,311
// 23 of the choices take 5 to 14% longer than the other way, one 22%.
//
// Pairs with reads of more than 255 bases hold 50 KB of tables each, three a
// CU: 768 of them run at once, and what is beyond that waits for a second
// round, of twice the binned sweeps' length (haplotypes of 350 bases, us,
// binned / one-pair: 300 bases, 512 pairs 96 / 48, 1,024 101 / 87, 4,096
// 143 / 235; 500 bases, all redone in FP64, 187 / 120, 215 / 223, 421 / 637;
// 1,000 bases 523 / 429, 855 / 847, 2,336 / 2,520).
constexpr double kOneNs = 12e3, kBinnedNs = 55e3, kNextBinNs = 9e3, kSingleNs = 0.16;
constexpr double kFreeNs = 45e3, kFreePairNs = 4.9, kFreeFurtherNs = 1.5, kFreeBatchNs = 6;  // without a plan
constexpr int64_t kFreeFurther = 15000;
constexpr int64_t kOneSteps = 130, kBinnedSteps = 60;  // beside the columns of a tile
constexpr int64_t kOneLongPairs = 768;
// a launch counts its threads in 32 bits: 2^26 workgroups are refused, more of them
// start the rest of the division only
constexpr int64_t kOneMaxPairs = ((int64_t)1 << 26) - 1;
constexpr double kStepNs = 0.0081, kRowNs = 0.00557;
inline double step_ns(int K) { return kStepNs + kRowNs * K; }
inline double tile_ns(int64_t cols, int P, int K) { return 2.0 * (double)(cols + P + 2) * (5.5 * K + 10); }
// the sum of a bin's tiles, which take that many steps
inline double bin_ns(double steps, int P, int K) { return steps * step_ns(K) * (P == 16 && K > 12 ? 1.2 : 1.0); }
// ns is no more than the binned launches take, their tiles' sum and their ends overlapping
inline bool within_binned(double ns, double launches, double sum, double ends)
{
    const double left = ns - launches;
    if (left <= std::max(sum, ends)) return true;
    return left <= sum + ends && left <= std::pow(std::pow(sum, 1.6) + std::pow(ends, 1.6), 1 / 1.6);
}

// Time of the one-pair launch (infinite: too many pairs of long reads, or more than a
// launch holds): the steps of all tiles, and times their rows per lane; the longest
// haplotype and read.
inline double one_pair_ns(int64_t pairs, double steps, double row_steps, int64_t n_max, int m_max, int64_t long_pairs)
{
    if (pairs > kOneMaxPairs || long_pairs > kOneLongPairs) return INFINITY;
    return kOneNs + kStepNs * steps + kRowNs * row_steps + 0.5 * tile_ns(n_max, 64, (m_max + 64) >> 6);
}

// Adjoint configuration of reads of m bases (up to 319): 32 lanes x K <= 5 rows, then
// 64 x K; wide: 64 lanes x K, but for reads that 32 lanes hold with one row each, whose
// steps would be no shorter and more (160 to 2,000 pairs of 20-31 bases: 4 to 33% longer).
inline bool adj_config(int m, bool wide, int &P, int &K)
{
    if (m + 1 <= 32 * (wide ? 1 : 5)) {
        P = 32;
        K = (m + 1 + 31) / 32;
    } else if (m + 1 <= 64 * 5) {
        P = 64;
        K = (m + 1 + 63) / 64;
        if (!wide) K = std::max(3, K);
    } else {
        return false;
    }
    return true;
}

// Calls of no more pairs than that may take 64 lanes for each: every tile is under
// way at once and shorter.
constexpr int64_t kAdjWidePairs = 2048;
// 1,024 tiles have a SIMD each; a wave that shares its SIMD with another of its length
// takes 1.58 times as long.
constexpr int64_t kAdjAlone = 1024;
constexpr double kAdjShared = 0.58;
// instructions of a tile's step
inline int adj_step(int K) { return 40 * K + 25; }

// Whether a plan takes 64 lanes for each pair.  K: the rows per lane of its only
// configuration of 32 lanes, or 0 where its reads take several or 64 lanes; n1, n1025:
// its longest haplotype and the 1,025th of its pairs' (0: no more than 1,024 pairs).
// With several configurations the lengths of the tiles even out (us, 32 and 64 lanes /
// 64 lanes: reads of 60-300 x 200-600 bases, 1,200 pairs 336 / 360, 1,800 457 / 407,
// 2,300 461 / 425, 4,000 747 / 754; 50-150 x 400-600, 800 315 / 244, 2,040 330 / 301,
// 3,000 371 / 399).  With one, a tile of 64 lanes is shorter but shares its SIMD
// beyond 1,024 pairs (32 / 64 lanes: 60 x 300, 800 pairs 111 / 102, 1,500 117 / 133;
// 100 x 1,000, 800 420 / 297, 1,500 429 / 401, 4,000 687 / 697; 150 x 2,000, 800 939 /
// 674, 1,500 971 / 1,010; 150 x 200-600, 1,500 319 / 296, 2,300 367 / 390).
inline bool adj_wide(int64_t pairs, int K, int64_t n1, int64_t n1025)
{
    if (pairs > kAdjWidePairs) return false;
    if (K == 0) return true;
    const double narrow = (double)(n1 + 33) * adj_step(K);
    double wide = (double)(n1 + 65) * adj_step((K + 1) / 2);
    if (pairs > kAdjAlone) wide += kAdjShared * (double)(n1025 + 65) * adj_step((K + 1) / 2);
    return wide < narrow;
}

// Adjoint tiles by their steps: up to 1,280, where the LDS of 8 workgroups fits a CU,
// and twice that again and again.  Groups share a launch or are launched apart,
// whichever takes less time by adj_launch_time: a launch's LDS and checkpoint slices
// are its longest tile's, which leaves fewer workgroups for the shorter ones, while
// launches apart each end with their longest tile.  (Reads of 50-300 x 1,300-2,000 bases
// and one pair of 100 x 20,000, ms, together / apart: 3,600 pairs 7.3 / 9.0, 27,000
// 30.0 / 19.3; 150 x 1,000-3,000, 3,600 pairs 2.0 / 2.4; 50-300 x 2,000-10,000, 600
// pairs 2.6 / 4.7, 27,000 51 / 45.)
constexpr int kAdjGroups = 6;
inline int adj_group(int steps)
{
    int g = 0;
    while (g < kAdjGroups - 1 && steps > 1280 << g) ++g;
    return g;
}
// Time of a launch (2 ns) with that many workgroups resident: 1,024 SIMDs run a wave
// each at its own rate, two at 1 / 1.58 of it, and one and a half on average gain as much
// as two; a launch costs 5 us beside that.
inline double adj_launch_time(double longest, double total, int64_t grid)
{
    const double waves = (double)grid / kAdjAlone;
    const double rate = waves <= 1 ? waves : std::min(1 + 0.54 * (waves - 1), 1.27);
    return 2500 + std::max(longest * (waves > 1 ? 1 + kAdjShared : 1), total / (kAdjAlone * rate));
}

}  // namespace ph

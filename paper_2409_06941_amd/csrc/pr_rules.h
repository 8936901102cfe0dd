// The sizes of the partition-centric layout, and the rules that choose among its kernels.  Host code only.
// (The times beside the rules are of the sweeps as they were when each line was drawn, both sides by the same kernels.  The present
// ones - a branch-free gather loop, side-by-side searches in the scatter sweep - take 9 to 23 % less, and were measured again with either
// side of gather_alone and of scatter_alone forced: 138 graphs, 8 to 20 edges a vertex, 8000 to 150 000 edges a unit, 16 to 256 units.
//   scatter_alone: within 3 % of the faster side on 130, 5 % on 136; at worst 7.3 (uniform 3.2 x 10^6 / 2.6 x 10^7), where the other side
//     of the rule elsewhere costs up to 38 % (uniform 2.4 x 10^6 / 1.9 x 10^7 on 128 units 64.6 -> 88.8).
//   gather_alone: within 3 % on 109; the others are all on the side of two workgroups, on up to 64 units from 48 000 to 100 000 edges a
//     unit: one would take us an iteration 22.9 -> 19.6 (skewed 153 600 / 3.1 x 10^6 on 64 units), 25.6 -> 23.4 (201 600 / 4.0 x 10^6), 32.1 -> 29.9
//     (320 000 / 6.4 x 10^6), 21.9 -> 18.7 (76 800 / 1.5 x 10^6 on 32), 23.8 -> 21.2 (50 400 / 1.0 x 10^6 on 16), uniform ones of 48 000 and 63 000
//     a unit 3 to 11 % less; at 100 000 uniform ones take 5 to 10 % more with one, at 150 000 all but a few do.  On 256 units: uniform 2.0 x 10^6 /
//     1.6 x 10^7 51.6 -> 48.9.  So that line could lie higher on few units by now; the kernels before them are what it is drawn for.
// kMergeBalance 20, 29, 40 with the present kernels: 2^18 / 2^22 22.3, 20.3, 21.0.)
#ifndef FR_PR_RULES_H
#define FR_PR_RULES_H

#include <cmath>
#include <cstdint>

constexpr uint32_t kRowsSmall = 8192, kRowsLarge = 16384;   // destination rows per range (8 B each in LDS)
constexpr uint32_t kSrcSmall = 16384, kSrcLarge = 32768;    // source vertices per scatter partition (4 B each in LDS)
constexpr int64_t kLargeRowsFrom = int64_t(1) << 22;        // vertex counts from which the large sizes are used
constexpr int64_t kLargeSrcFrom = int64_t(1) << 24;

// Does the scatter sweep deal groups of four messages in runs to the wavefronts (else groups of eight round-robin)?
// Groups of four store in longer pieces and search for their bin twice as often.  The small kernel: where a launch hands out
// tiles (uniform graph of 2^23 vertices / 2^28 edges on 64 units 1640 -> 1442 us an iteration; one round of tiles is bound by latency:
// 10^6 / 10^7 30.4 -> 31.4).  The large kernel, one workgroup a unit: where there are enough units for the stores to bind, and
// long bins.  us an iteration, eight -> four, uniform graphs / skewed ones:
//   2^24 / 2^28: 64 units 1815 -> 1968 / 912 -> 910, 128 1142 -> 1105 / 534 -> 519, 256 816 -> 752 / 367 -> 349
//   2^24 / 2^26: 64 units 634 -> 693 / 326 -> 337, 128 387 -> 388 / 203 -> 200, 256 294 -> 285 / 133 -> 129
//   (large partitions asked for: 3 x 10^6 / 6 x 10^7, 8192 rows a range, 256 units 83.0 -> 85.7; 64 units 177 -> 187)
constexpr uint32_t kRunsFromUnits = 128;
inline bool scatter_in_runs(uint32_t src_per_part, int64_t V, uint32_t cus, bool hands_out)
{
    return src_per_part == kSrcSmall ? hands_out : V >= kLargeSrcFrom && cus >= kRunsFromUnits;
}

// The small kernels fit twice on a compute unit, but a sweep of a small graph is faster with one workgroup each: with
// more, some units hold two and take twice as long as the others, and every piece of a merged range is one more row of
// partial sums to write and to add up.  Gather: while there are two units or more per range (else light ranges share
// workgroups badly: 10^6 vertices / 10^7 edges on 64 units 50.5 -> 58.0 us an iteration) and a unit's share of the weight
// (two an edge, and some for repeated ones) is at most kGatherAloneShare per unit, or that of 64 units on fewer.  (On few units each
// has more bandwidth to itself and needs two workgroups to use it; but a sweep that makes fewer than two tiles of the least
// size a unit leaves some units with two and some with one.)  us an iteration, two a unit -> one, at these thousands of edges a unit:
//   16 units: 31 22.2 -> 19.6, 63 26.9 -> 28.8, 125 37.6 -> 42.9   32: 16 23.4 -> 18.6, 31 24.8 -> 21.3, 63 28.6 -> 29.3
//   64: 31 26.8 -> 21.8, 66 35.6 -> 39.4   128: 33 28.4 -> 23.2, 78 39.1 -> 38.4   256: 39 34.9 -> 30.8, 63 43.5 -> 37.0, 148 59.8 -> 56.2
constexpr uint64_t kGatherAloneShare = 1600;
inline bool gather_alone(uint32_t rows_per_part, uint32_t Qe, uint64_t total, uint32_t cus)
{
    return rows_per_part == kRowsLarge || (2 * Qe <= cus && total <= (uint64_t)cus * (cus < 64 ? 64 : cus) * kGatherAloneShare);
}

// Gather pieces weigh at least kLeastGather (two an edge, some for repeated ones), or kMergeBalance x the root of the heaviest
// range's weight: a row of a range cut into n pieces costs the scatter sweep n loads, a piece costs the gather sweep its own
// weight, and the sum of both is least where the pieces weigh as the root of the range (2^18 vertices / 2^22 edges: 162 pieces 22.8 us
// an iteration, 256 24.9, 313 28.9).  (2^14 vertices / 2^18 edges: 12 + 8 tiles of at least 65536 and of 16384 messages 18.6 us, 23 + 51 tiles
// 16.2, 45 + 95 tiles 16.6; a piece's fixed weight counts against a step's budget, so the gather sweep stays coarser.)
// Where two workgroups share a unit and the sweep makes more tiles than there are units, light ranges would be cut in two for
// nothing: pieces weigh kLeastGatherOfTwo there.  us an iteration, uniform graphs, 49152 -> 65536: 1.6 x 10^6 / 6.1 x 10^6 (315 -> 260
// tiles) 37.6 -> 35.6, 2.5 x 10^6 / 8.5 x 10^6 (449 -> 378) 46.7 -> 43.6, on 64 units 600 000 / 1.8 x 10^6 (100 -> 86) 32.4 -> 31.4, on 128
// 1.2 x 10^6 / 3.6 x 10^6 (199 -> 170) 36.4 -> 34.8.  Likewise with the large ranges, whose rows of partial sums are twice as long (skewed
// 4.3 x 10^6 / 3 x 10^6 29.8 -> 29.4, 9 x 10^6 / 6.3 x 10^6 35.2 -> 35.8).  Partial sums count against the memory of the run that allocates
// nothing: 3 x 10^6 / 9 x 10^6 took 54.2 MB of its 64 and takes 50.0.
constexpr uint64_t kLeastGather = 49152, kLeastGatherOfTwo = 65536, kMergeBalance = 29;
inline uint64_t least_gather_weight(uint32_t rows_per_part, uint64_t heaviest)
{
    const uint64_t least = rows_per_part == kRowsLarge ? kLeastGatherOfTwo : kLeastGather, balance = (uint64_t)((double)kMergeBalance * std::sqrt((double)heaviest));
    return balance > least ? balance : least;
}

// Scatter: up to kScatterAloneShare (messages and values read) a unit per unit, or kScatterAloneLeast a unit on fewer than 171;
// beyond it one workgroup cannot keep a unit's share of the bandwidth busy.  us an iteration, two a unit -> one, at these
// thousands a unit:
//   16 units: 9 18.1 -> 16.8, 22 27.5 -> 27.0, 53 64.8 -> 67.0, 84 40.0 -> 41.0   32: 9 18.6 -> 17.4, 22 24.8 -> 23.8, 72 116.7 -> 123.0
//   64: 13 21.2 -> 19.6, 25 23.6 -> 22.0 and 30.5 -> 31.1, 44 69.8 -> 76.2, 72 35.6 -> 37.0
//   128: 13 25.1 -> 23.2, 27 39.4 -> 38.0, 58 47.8 -> 57.5, 98 48.0 -> 50.0   256: 17 33.5 -> 32.1, 29 39.6 -> 37.5, 49 41.8 -> 40.4, 72 55.5 -> 63.0
constexpr uint64_t kScatterAloneShare = 192, kScatterAloneLeast = 32768;
inline bool scatter_alone(uint32_t src_per_part, uint64_t all, uint32_t cus)
{
    const uint64_t share = cus * kScatterAloneShare > kScatterAloneLeast ? cus * kScatterAloneShare : kScatterAloneLeast;
    return src_per_part == kSrcLarge || all <= cus * share;
}

// Scatter pieces weigh at least kMinTileMessages, or kPieceBalance x the root of the sweep's weight (as pieces of a range do); a
// sweep of up to kOneTileMessages is one tile: what a second one saves in stores it costs in start-up and in dangling sums.
// us an iteration, tiles of at least 4096 -> one tile: 4096 vertices / 16 384 edges (weight 8200) 15.3 -> 14.7, 5000 / 20 000
// (10 000) 15.9 -> 15.2; 10 000 / 40 000 (26 000) 15.9 -> 17.0 with three tiles and 17.6 with two.
constexpr uint64_t kMinTileMessages = 4096, kOneTileMessages = 16384, kPieceBalance = 6;
inline uint64_t least_scatter_weight(uint64_t all)
{
    if (all <= kOneTileMessages) return all ? all : 1;
    const uint64_t balance = (uint64_t)((double)kPieceBalance * std::sqrt((double)all));
    return balance > kMinTileMessages ? balance : kMinTileMessages;
}

#endif

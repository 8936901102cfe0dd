// The sizes of the partition-centric layout, and the rules that choose among its kernels.  Host code only.
#ifndef FR_PR_RULES_H
#define FR_PR_RULES_H

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

#endif

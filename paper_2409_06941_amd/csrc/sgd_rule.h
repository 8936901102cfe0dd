// Whether a Graph SGD task's ratings are worked on in rounds (k_sgd) or one after the other (k_sgd_chain).  Host code only.
#ifndef FR_SGD_RULE_H
#define FR_SGD_RULE_H

#include <algorithm>
#include <cstdint>

constexpr uint32_t kSgdBatch = 128;                 // ratings of a cell that are worked on out of LDS at a time
constexpr uint64_t kSgdLongCell = 2 * kSgdBatch;    // mean ratings of a cell up to which cells may be worked on in rounds

// What a stratum of B cells takes either way, in us: the longest chain of one cell (`chain`: the mean over the strata of
// their largest cell) and the work of all cells on `cus` compute units, the longer of them in full and the other, which mostly
// runs beside it, by half.  In rounds a cell is a workgroup with a record, rows and LDS of its own even if it has one rating: few
// ratings a cell and few units are what they are worse at.  Measured, ms an iteration, one after the other -> rounds:
//   1024 x 1024 cells, F = 64, 256 units: 0.02 ratings a cell 2.4 -> 4.0, 1 (chain 6.6) 4.2 -> 4.8, 2 (10.4) 5.4 -> 5.3, 4 8.2 -> 6.2
//   the same on 32 units, 1.7 ratings a cell: F = 64 7.3 -> 22.3, F = 16 6.4 -> 12.0; 256 x 256 cells of 27 6.0 -> 3.3
//   512 x 512 cells of 61, F = 64: 256 units 25.3 -> 8.5, 24 31.1 -> 27.9, 16 34.8 -> 38.9, 8 56.4 -> 72.5; F = 16, 8 units 29.6 -> 20.4
inline bool sgd_rounds_pay(uint64_t ratings, uint32_t B, uint64_t chain_ratings, int F, uint32_t cus)
{
    const double cells = (double)B * B;
    if (B == 0 || cus == 0 || (double)ratings > (double)kSgdLongCell * cells) return false;
    const double mean = (double)ratings / cells, chain = (double)chain_ratings / B, cells_per_unit = (double)B / cus;
    auto together = [](double a, double b) { return std::max(a, b) + 0.5 * std::min(a, b); };
    const double rounds = together(2.8 + 0.008 * F + (0.06 + 0.0004 * F) * chain,
                                   (0.2 + 0.0047 * F + mean * F * (0.00018 + 0.0000036 * F)) * cells_per_unit);
    const double in_a_row = together(2.0 + 0.33 * chain, 0.00035 * F * mean * cells_per_unit);
    return rounds < in_a_row;
}

#endif

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
// (with kernels whose rounds waited at every third one.  The present ones, 196 points of 16 to 1024 blocks, 8 to 256 units, F = 16 and 64:
// the line lies where it did - 512 blocks of 61, F = 64: 256 units 22.8 -> 7.1, 24 28.6 -> 25.7, 16 32.5 -> 36, 8 54 -> 68 - and on its
// wrong side are 1024 blocks of 3.9 on 128 units, F = 64, 7.7 -> 8.4, and 128 of 3.8 on 24 units, F = 64, 0.68 -> 0.74.)
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

// Whether a launch of `n` cells of a stratum reads ahead, with the wavefronts that have no rounds to work through, what the next
// stratum's cells begin with (k_sgd).  It takes the wait for the programs out of the next launch where those come from memory
// (many ratings a stratum) and the rounds are long enough to cover the reads (ratings a cell: the workgroup waits for them before it
// ends); where a unit has cell after cell to work on, the reads stand in the way of its other cells and are forgotten before they
// are of use.  Time of an iteration with it over without it, F = 16, 32, 64, whole strata:
//   up to 2 cells a unit: 128 blocks of 17 ratings a cell 1.06 1.02 1.02, of 25 0.98 0.99 0.99; 256 of 8 1.08 1.04 1.02, of 17 0.96 0.97 0.98;
//     384 of 13 1.05 1.02 1.04; 512 of 8 (F = 16, 64) 1.01 1.00, of 17 0.98 0.94 0.99, of 61 (16, 64) 0.89 0.96
//   3: 256 of 17 1.01 0.99 1.00, of 25 0.95 0.97 0.99; 384 of 13 1.07 1.05 1.06, of 25 0.96 0.97 0.99; 512 of 17 1.01 0.97 1.02
//   4: 128 of 34 1.01 1.02 1.03, of 102 0.95 0.99 0.99; 256 of 33 0.97 1.00 1.02, of 48 0.96 1.00 1.01; 384 of 25 1.00 1.01 1.02, of 50 0.94 0.97
//     0.98; 512 of 25 0.96 0.98 1.00; 1024 of 15 (16, 64) 0.96 1.01, of 25 0.92 0.98
//   5 to 16: 256 of 31 on 32 units 1.18 (16), 1.03 (64); 512 of 8 on 32 units 1.49 (16); 512 of 49 on 96 0.95 1.02 1.01; 512 of 61 on 24 1.09 1.09
//   below 128 blocks: 32 1.04 (64)
// Launches of 3 cells 1.02 to 1.07, of 20 0.95 to 1.02, of 52 0.90 to 0.98 where whole strata gain; of 100 of the 512 of 61 on 64 units, where
// whole strata do not, 0.91 and 0.97.
inline bool sgd_reads_ahead(uint64_t ratings, uint32_t B, uint32_t n, uint32_t cus)
{
    if (B < 128 || n < 32 || (uint64_t)n > 4ull * cus) return false;
    const double stratum = (double)ratings / B, mean = stratum / B;
    if (n <= 2 * cus) return mean >= 16 && stratum >= 3072;
    return mean >= 24 && stratum >= (n <= 3 * cus ? 6144 : 12288);
}

// Whether eight workgroups of a launch of `n` cells are to share a unit (64 registers a lane) rather than seven (72), with 16
// factors: the eighth has work from eight cells a unit on.
inline bool sgd_eight_cells_a_unit(uint32_t n, uint32_t cus) { return (uint64_t)n > 7ull * cus; }

#endif

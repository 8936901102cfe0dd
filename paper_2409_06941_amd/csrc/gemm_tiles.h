// The tiles of the bf16 GEMM kernels and the choice among them.  Host code only.
#ifndef FR_GEMM_TILES_H
#define FR_GEMM_TILES_H

#include <algorithm>
#include <cmath>

constexpr int BK = 64;                         // K of a k-tile: 128 bytes of a row
constexpr int kShortM = 256, kShortN = 128;    // tile of k_gemm_bf16_nt_short

// Tiles and what they were measured to take, in us: `start` to begin and end a workgroup, and per k-tile `alone` with few
// workgroups on the chip, `full` with one on every compute unit (shared L2, lower clock), and `more` for every further one per
// compute unit.  Where one workgroup fills a compute unit (side_by_side 1) a part of a round costs a round; others overlap.
// 2048 x 4096 x 4096, for instance, takes 75 us in 128 tiles of 256 x 256, 55 in 256 of 128 x 256 and 58 in 512 of
// 128 x 128; 512 x 768 x 1024 from operands that are in no L2 takes 22.9 us in 6 tiles of 256 x 256, 8.1 in 96 of 64 x 64 and 6.6
// if four parts of K are worked on side by side as well (with K = 512: 15.3, 4.0 and 5.1).
struct GemmTile { int bm, bn, side_by_side; float start, alone, full, more; };
constexpr GemmTile kTiles[] = {
    {256, 256, 1, 8.5f, 0.97f, 1.39f, 1.39f}, {128, 256, 1, 5.7f, 0.57f, 0.80f, 0.80f}, {128, 128, 2, 5.1f, 0.33f, 0.46f, 0.43f},
    {64, 128, 2, 2.7f, 0.24f, 0.35f, 0.28f}, {64, 64, 4, 2.6f, 0.22f, 0.30f, 0.28f},
    {64, 64, 1, 3.9f, 0.134f, 0.20f, 0.20f},                       // kSplit 4
    {kShortM, kShortN, 2, 4.8f, 1.0f, 1.1f, 1.0f},                 // k_gemm_bf16_nt_short
};

inline float gemm_estimate(const GemmTile& T, int M, int N, int K, int cus)
{
    const float u = (float)((double)(M / T.bm) * (double)(N / T.bn) / cus), nk = (float)(K / BK), rounds = std::floor(u), rest = u - rounds;
    if (T.side_by_side == 1)
        return (rounds + (rest > 0.0f ? 1.0f : 0.0f)) * T.start + nk * (rounds * T.full + (rest > 0.0f ? T.alone + (T.full - T.alone) * rest : 0.0f));
    // (the compute units with one workgroup more than the others set the time, though less than if all had as many)
    const float v = u <= 1.0f ? u : 0.35f * u + 0.65f * std::ceil(u);
    return T.start * std::max(1.0f, v / T.side_by_side) + nk * (v <= 1.0f ? T.alone + (T.full - T.alone) * v : T.full + (v - 1.0f) * T.more);
}

// The ring kernels' loads reach eight rows from one address with a 32-bit offset: rows of up to 2^28 bytes.  A longer K takes
// k_gemm_bf16_nt_short, whose addresses have 64 bits.
constexpr int kRingMostK = 1 << 27;
constexpr int kGemmTiles = (int)(sizeof(kTiles) / sizeof(kTiles[0]));

// The tile (its place in kTiles) that takes least on `cus` compute units: those the stream may use.  (For all 256, on a stream of
// 64: 256 x 16384 x 16384 532 us where the tile for 64 takes 302, 512 x 11008 x 64 14.9 and 9.6; both 434 and 9.6 with tiles of 256 x 128
// throughout.)
inline int gemm_choose(int M, int N, int K, int cus)
{
    if (K > kRingMostK) return kGemmTiles - 1;
    int best = 0;
    float least = gemm_estimate(kTiles[0], M, N, K, cus);
    for (int k = 1; k < kGemmTiles; ++k) {
        const float us = gemm_estimate(kTiles[k], M, N, K, cus);
        if (us < least) { least = us; best = k; }
    }
    return best;
}

#endif

// The PageRank side task: pull-based power iteration, fp32 ranks, for gfx950.
//
// The paper's graph-analytics side task (Section 6.1.4) with one iteration = one pass over the graph
// (Section 6.2), written as a step-wise task for the iterative interface (Section 4.2): work is cut into tiles
// that are fixed at init, a step is a run of consecutive tiles of one segment, and every tile computes the same
// bits whichever launch carries it, so pausing and resuming at any tile boundary cannot change the result.
//
// The pull pass runs on the partition-centric layout of pr_layout.h (vertices renumbered by in-degree).  One run =
//     V0, S_0 G_0, S_1 G_1, ..., S_{K-1} G_{K-1}, F
//   V0   vertex pass (tile = row range): dangling partials of r_0 = 1/V
//   S_k  scatter     (tile = source interval): contrib_k of the interval goes into LDS - r_0 / outdeg for k = 0,
//                    read back for rows of direct ranges, made on the spot for rows of merged ranges (partial
//                    sums of G_{k-1} added in tile order, then the vertex-pass arithmetic) and of empty ranges
//                    (r = base) - then one message per (range, source) is written
//   G_k  gather      (tile = run of edges of one range): id stream + messages -> 64-bit fixed-point sums in LDS;
//                    direct range: fused, the next vertex pass for its rows,
//                    r_{k+1} = base_k + d * sum, contrib_{k+1} = r_{k+1} / outdeg, dangling partials;
//                    merged range: the sums are stored as one row of fp32 partial sums
//   F    finish      (tile = merged or empty range): after the last iteration, r_K of their rows
// base_k = (1 - d)/V + d * D_k / V, D_k = fixed-order sum of the dangling partials of r_k.
// In the last iteration G writes r_K to ranks_out (through perm) instead of contrib; F does the same.
// No floating-point atomics anywhere: float sums have a fixed order, the LDS atomics add integers.

#include <algorithm>
#include <cmath>
#include <cstring>
#include <mutex>
#include <new>
#include <type_traits>

#include "freeride_device.h"
#include "pr_layout.h"

namespace {

constexpr int kBlock = 512;                     // threads per workgroup of the first vertex pass
constexpr int kGatherBlock = 1024;              // threads per workgroup of the gather sweep
constexpr int kGatherWaves = kGatherBlock / 64;
constexpr int kScatterBlock = 1024;             // threads per workgroup of the scatter sweep
constexpr int kScatterWaves = kScatterBlock / 64;
// row sums are kept as 64-bit fixed point with scale 2^62: contrib sums are <= 1, so they fit
constexpr float kFixInv = 1.0f / 4611686018427387904.0f;
// messages are contrib * 2^30: see to_fixed
constexpr float kMsgScale = 1073741824.0f;

// ---- fixed-order reductions ----
// (by moves between lanes of the vector unit: inside rows of 16 lanes, then row 0 into row 1 and row 2 into row 3, then the
// lower half into the upper; six exchanges through the LDS unit take some 0.2 us)
template <int kCtrl, int kRows>
__device__ __forceinline__ int from_lane(int x)
{
    return __builtin_amdgcn_update_dpp(0, x, kCtrl, kRows, 0xf, false);      // 0 in lanes without a source
}

__device__ __forceinline__ float wave_sum(float x)
{
    auto add = [&](int moved) { x += __int_as_float(moved); };
    add(from_lane<0x111, 0xf>(__float_as_int(x)));       // row_shr 1, 2, 4, 8
    add(from_lane<0x112, 0xf>(__float_as_int(x)));
    add(from_lane<0x114, 0xf>(__float_as_int(x)));
    add(from_lane<0x118, 0xf>(__float_as_int(x)));
    add(from_lane<0x142, 0xa>(__float_as_int(x)));       // row_bcast 15 into rows 1 and 3
    add(from_lane<0x143, 0xc>(__float_as_int(x)));       // row_bcast 31 into rows 2 and 3
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 63));
}

// Inclusive prefix sums over the lanes.
__device__ __forceinline__ uint32_t wave_scan(uint32_t x)
{
    x += (uint32_t)from_lane<0x111, 0xf>((int)x);
    x += (uint32_t)from_lane<0x112, 0xf>((int)x);
    x += (uint32_t)from_lane<0x114, 0xf>((int)x);
    x += (uint32_t)from_lane<0x118, 0xf>((int)x);
    x += (uint32_t)from_lane<0x142, 0xa>((int)x);
    x += (uint32_t)from_lane<0x143, 0xc>((int)x);
    return x;
}

// Sum of a per-thread value over the workgroup, same association for a given blockDim.  All threads call.
__device__ __forceinline__ float block_sum(float x, float* lds /* one float per wavefront */)
{
    x = wave_sum(x);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    __syncthreads();
    if (lane == 0) lds[w] = x;
    __syncthreads();
    float s = 0.0f;
    const int nw = (int)(blockDim.x >> 6);
    for (int i = 0; i < nw; ++i) s += lds[i];
    return s;
}

// D = sum of dpart[0 .. n), n >= 1, in one order whatever the kernel: strand i (of kStrands) is the sum of the elements i,
// i + kStrands, i + 2 kStrands, ... in turn, the strands of a group of 64 are joined by the balanced tree over consecutive lanes
// that wave_sum makes (pairs, fours, eights, rows of 16, halves), the groups one after the other.  A workgroup of the sweeps has a thread for every strand, so that up to 1024 partials are one load a thread, asked
// for before the tile's record; the sum is put together behind the next barrier.  (Every wavefront for itself, as it was
// before, the compiler waited for every fourth element a lane and for each of the last three in front of the tile's first
// load: 10^6 vertices / 10^7 edges 32.0 -> 31.4 us an iteration, 2^22 / 2^26 77.0 -> 76.2.)
constexpr uint32_t kStrands = 1024;
__device__ __forceinline__ float dangling_strand(const float* __restrict__ dpart, uint32_t n, uint32_t i)
{
    float s = dpart[i < n ? i : n - 1];
    s = i < n ? s : 0.0f;
    for (uint32_t j = i + kStrands; j < n; j += 4 * kStrands) {
        float x[4];
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k) x[k] = dpart[j + k * kStrands < n ? j + k * kStrands : n - 1];
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k) s += j + k * kStrands < n ? x[k] : 0.0f;
    }
    return s;
}

// The wavefront's strands (64 consecutive ones) go to their group's word; after a barrier the groups are added up.
__device__ __forceinline__ void dangling_group(float strand, uint32_t first, float* groups)
{
    const float s = wave_sum(strand);
    if ((threadIdx.x & 63) == 0) groups[first / 64] = s;
}

__device__ __forceinline__ float dangling_total(const float* groups)
{
    float D = 0.0f;
#pragma unroll
    for (uint32_t g = 0; g < kStrands / 64; ++g) D += groups[g];
    return D;
}

struct DevArgs {
    int64_t V, E;
    uint32_t M, Q, Qe, n_gather, n_pieces, n_scatter, n_spieces, n_finish, n_dpart;
    uint32_t rows_per_part, rows_shift;           // rows per range and its log2
    uint32_t void_slot;                           // scatter piece whose slot of dangling partials takes the void pieces' mass (kNoVoid: none)
    float n_void_dangling;                        // rows of void pieces in ranges without in-edges: each holds the base value
    float damping;
    const uint16_t* ids16;
    const uint16_t* src16;
    const uint32_t* mbase;
    const uint64_t* starts;
    const uint2* bins;
    const float* inv_out;
    const int32_t* perm;
    const RangeInfo* range_info;
    const GatherPiece* gather_pieces;
    const GatherTile* gather_tiles;
    const ScatterPiece* scatter_pieces;
    const ScatterTile* scatter_tiles;
    const uint32_t* finish_ranges;
    float* msg;
    float* contrib;
    float* dpart;                 // [2][n_dpart]
    float* partials;              // [n_partials][rows_per_part]
    float* ranks_out;
    uint32_t* sched;              // [2] tiles handed out beyond a launch's first round; workgroups that have left
};

// What a step's kernels need to ask the device gate (Section 4.5's check, made by the GPU when the kernel starts).
struct GateArg {
    fr_gate* gate;                // NULL: no gate
    uint32_t slot, need_ticks;    // need_ticks: the whole step's modelled duration
    uint32_t tile_ticks;          // the modelled duration of the step's heaviest tile run alone
};

// Sum of a merged row's partial sums p_0 .. p_{nt-1}.  The order is fixed: sixteen leaves, leaf g = p_g + p_{g+16} +
// ... in rising order, joined by a balanced tree over g.  kLanes lanes (a power of two up to 16, consecutive in
// the wavefront, all active) share the row: lane `sub` owns the leaves sub * 16 / kLanes onwards, joins them, and
// the lanes' results are joined by butterfly exchanges, which is the same tree.  Every lane gets the sum.
template <int kLanes>
__device__ __forceinline__ float merged_sum(const DevArgs& A, RangeInfo info, uint32_t local, uint32_t sub)
{
    constexpr int kLeaves = 16 / kLanes;
    const uint32_t nt = info.cls_tiles >> 2;
    const float* p = A.partials + ((size_t)info.partial0 << A.rows_shift) + local;
    float s[kLeaves];
#pragma unroll
    for (int k = 0; k < kLeaves; ++k) s[k] = 0.0f;
    // kDeep rounds of 16 at a time, then half as many, then what is left of one: sixteen loads or more are issued before the
    // first is used (a round at a time, the 90 partial sums of a row of the heaviest range of 2^26 edges were six latencies
    // one after the other).  The last round has two, four, eight or sixteen leaves: most merged ranges have two or three
    // pieces, and sixteen loads a row instead of three made the scatter sweep of 2^24 / 2^28 7 us longer.
    constexpr uint32_t kDeep = kLeaves >= 16 ? 1 : kLeaves >= 8 ? 2 : 4;
    uint32_t t0 = 0;
    auto rounds = [&](auto count) {
        constexpr uint32_t R = decltype(count)::value;
        float x[R][kLeaves];
#pragma unroll
        for (uint32_t j = 0; j < R; ++j)
#pragma unroll
            for (int k = 0; k < kLeaves; ++k) {
                const uint32_t t = t0 + 16 * j + sub * kLeaves + k;
                x[j][k] = p[(size_t)(j + 1 < R || t < nt ? t : nt - 1) << A.rows_shift];
            }
#pragma unroll
        for (uint32_t j = 0; j < R; ++j)
#pragma unroll
            for (int k = 0; k < kLeaves; ++k) s[k] += j + 1 < R || t0 + 16 * j + sub * kLeaves + k < nt ? x[j][k] : 0.0f;
        t0 += 16 * R;
    };
    while (t0 + 16 * (kDeep > 1 ? kDeep - 1 : 1) < nt) rounds(std::integral_constant<uint32_t, kDeep>{});
    if constexpr (kDeep >= 4)
        while (t0 + 16 < nt) rounds(std::integral_constant<uint32_t, 2>{});
    auto rest = [&](auto count) {                // nt - t0 <= count: leaves 0 .. count - 1
        constexpr int C = decltype(count)::value < kLeaves ? decltype(count)::value : kLeaves;
        float x[C];
#pragma unroll
        for (int k = 0; k < C; ++k) {
            const uint32_t t = t0 + sub * kLeaves + k;
            x[k] = p[(size_t)(t < nt ? t : nt - 1) << A.rows_shift];
        }
#pragma unroll
        for (int k = 0; k < C; ++k) s[k] += t0 + sub * kLeaves + k < nt ? x[k] : 0.0f;
    };
    const uint32_t left = t0 < nt ? nt - t0 : 0;
    if (left > 8) rest(std::integral_constant<int, 16>{});
    else if (left > 4) rest(std::integral_constant<int, 8>{});
    else if (left > 2) rest(std::integral_constant<int, 4>{});
    else if (left) rest(std::integral_constant<int, 2>{});
#pragma unroll
    for (int w = 1; w < kLeaves; w <<= 1)
#pragma unroll
        for (int k = 0; k + w < kLeaves; k += 2 * w) s[k] += s[k + w];
    float r = s[0];
#pragma unroll
    for (int off = 1; off < kLanes; off <<= 1) r += __shfl_xor(r, off, 64);
    return r;
}

// Rows [i0, i1) of a scatter tile's slice, all in one merged range: r = base + d * (sum of the row's partial sums),
// contrib = r / outdeg.  kLanes lanes work on a row.  Returns this thread's share of the dangling mass.
template <int kLanes, int kThreads>
__device__ __forceinline__ float fill_merged(const DevArgs& A, RangeInfo info, uint32_t u0, uint32_t i0, uint32_t i1, float base, float* slice)
{
    const uint32_t sub = threadIdx.x % kLanes;
    float dangling = 0.0f;
    for (uint32_t ib = i0; ib < i1; ib += kThreads / kLanes) {       // uniform trip count: the lanes exchange values
        const uint32_t i = ib + threadIdx.x / kLanes;
        if (i >= i1) continue;                                       // (all lanes of a row leave together)
        const uint32_t u = u0 + i;
        const float inv = A.inv_out[u];
        const float r = fmaf(A.damping, merged_sum<kLanes>(A, info, u & (A.rows_per_part - 1), sub), base);
        if (sub == 0) {
            slice[i] = r * inv * kMsgScale;
            dangling += (inv == 0.0f ? r : 0.0f);
        }
    }
    return dangling;
}

// contrib of the sources [u0, u0 + n) of a scatter tile for an iteration after the first, into `slice`; returns
// this thread's share of the dangling mass among the rows finished here.  The sources lie in a handful of ranges.
// kOneKind (the large slice): where these are all of one kind and not merged - nearly all pieces of the sources with
// few messages - every row needs one value from one array (its contrib, finished by the range's gather tile, or
// 1/outdeg if the rows have no in-edges), and the slice is read in rounds of kFillRound rows per thread whose loads
// are all issued before the first is used, whatever the ranges' boundaries: two memory latencies for 32768 sources
// (walked range by range, a round per range, it was three or four, and 24 us of a piece's 33 with four rows a round).
// Otherwise the tile is walked range by range, so that each loop has one kind of row.
// `first_info`: what range_info holds for the range of u0.
template <int kThreads, int kFillRound, bool kOneKind>
__device__ __forceinline__ float fill_slice(const DevArgs& A, uint32_t u0, uint32_t n, float base, float* slice, RangeInfo first_info)
{
    if constexpr (kOneKind) {
        const uint32_t q0 = u0 >> A.rows_shift, q_last = (u0 + n - 1) >> A.rows_shift;
        const uint32_t cls0 = first_info.cls_tiles & 3u;
        bool same = cls0 != kRangeMerged;
        for (uint32_t q = q0 + 1; q <= q_last; ++q) same = same && (A.range_info[q].cls_tiles & 3u) == cls0;
        if (same) {
            const float* __restrict__ from = (cls0 == kRangeDirect ? A.contrib : A.inv_out) + u0;
            float dangling = 0.0f;
            for (uint32_t ib = threadIdx.x; ib < n; ib += kFillRound * kThreads) {
                float v[kFillRound];
#pragma unroll
                for (int k = 0; k < kFillRound; ++k) {
                    const uint32_t i = ib + k * kThreads;
                    v[k] = i < n ? from[i] : 1.0f;
                }
                if (cls0 == kRangeDirect) {
#pragma unroll
                    for (int k = 0; k < kFillRound; ++k) {
                        const uint32_t i = ib + k * kThreads;
                        if (i < n) slice[i] = v[k] * kMsgScale;
                    }
                } else {
#pragma unroll
                    for (int k = 0; k < kFillRound; ++k) {
                        const uint32_t i = ib + k * kThreads;
                        if (i < n) slice[i] = base * v[k] * kMsgScale;
                        dangling += (v[k] == 0.0f ? base : 0.0f);
                    }
                }
            }
            return dangling;
        }
    }
    float dangling = 0.0f;
    for (uint32_t i0 = 0; i0 < n;) {
        const uint32_t q = (u0 + i0) >> A.rows_shift;
        const uint32_t range_end = ((q + 1) << A.rows_shift) - u0;
        const uint32_t i1 = range_end < n ? range_end : n;
        const RangeInfo info = i0 == 0 ? first_info : A.range_info[q];
        const uint32_t cls = info.cls_tiles & 3u;
        if (cls == kRangeDirect || cls == kRangeEmpty) {
            // one value per row: contrib, finished by the range's gather tile, or 1/outdeg of a row without in-edges.
            // All loads of a round are issued before the first is used: a round is kFillRound rows per thread, and a
            // range's share of the slice is no more than that at 1024 threads, so the slice costs one memory latency.
            const float* __restrict__ from = cls == kRangeDirect ? A.contrib : A.inv_out;
            for (uint32_t ib = i0 + threadIdx.x; ib < i1; ib += kFillRound * kThreads) {
                float v[kFillRound];
#pragma unroll
                for (int k = 0; k < kFillRound; ++k) {
                    const uint32_t i = ib + k * kThreads;
                    v[k] = i < i1 ? from[u0 + i] : 1.0f;
                }
                if (cls == kRangeDirect) {
#pragma unroll
                    for (int k = 0; k < kFillRound; ++k) {
                        const uint32_t i = ib + k * kThreads;
                        if (i < i1) slice[i] = v[k] * kMsgScale;
                    }
                } else {
#pragma unroll
                    for (int k = 0; k < kFillRound; ++k) {
                        const uint32_t i = ib + k * kThreads;
                        if (i < i1) slice[i] = base * v[k] * kMsgScale;
                        dangling += (v[k] == 0.0f ? base : 0.0f);
                    }
                }
            }
        } else {
            // few rows (sources with many messages; their rows are the ones with many partial sums): several lanes a row
            const uint32_t len = i1 - i0;
            if (len * 16 <= kThreads) dangling += fill_merged<16, kThreads>(A, info, u0, i0, i1, base, slice);
            else if (len * 4 <= kThreads) dangling += fill_merged<4, kThreads>(A, info, u0, i0, i1, base, slice);
            else if (len * 2 <= kThreads) dangling += fill_merged<2, kThreads>(A, info, u0, i0, i1, base, slice);
            else dangling += fill_merged<1, kThreads>(A, info, u0, i0, i1, base, slice);
        }
        i0 = i1;
    }
    return dangling;
}

// ---- V0 ----
__global__ __launch_bounds__(kBlock) void k_vertex0(DevArgs A, GateArg G, uint32_t tile0, int final_pass)
{
    __shared__ float red[8];
    if (!fr_gate_admit(G.gate, G.slot, G.need_ticks)) return;
    const uint32_t q = tile0 + blockIdx.x;
    const int64_t v0 = (int64_t)q << A.rows_shift;
    const float r0 = 1.0f / (float)A.V;
    float dangling = 0.0f;
    for (uint32_t i = threadIdx.x; i < A.rows_per_part; i += kBlock) {
        const int64_t v = v0 + i;
        if (v >= A.V) break;
        if (final_pass) A.ranks_out[v] = r0;              // every vertex gets the same value: no need for perm
        else dangling += (A.inv_out[v] == 0.0f ? r0 : 0.0f);
    }
    if (!final_pass) {
        const float total = block_sum(dangling, red);
        if (threadIdx.x == 0) A.dpart[q] = total;
        if (q == 0)
            for (uint32_t i = A.Q + threadIdx.x; i < A.n_dpart; i += kBlock) A.dpart[i] = 0.0f;
    }
    fr_gate_done(G.gate, G.slot);
}

// Workgroups are handed to the 8 XCDs round-robin (workgroup b runs on XCD b % 8), and every XCD has an L2 of its
// own.  This map gives every XCD runs of kTileRun consecutive tiles, the runs dealt round-robin: neighbouring tiles
// write neighbouring messages (and share the lines at the seams) through one L2, while the heaviest tiles, which
// come first and read the most partial sums, are spread over all XCDs (in one contiguous block per XCD they were
// measured to take twice as long to fill their slices).  It is a bijection on [0, n) for any n.
constexpr uint32_t kTileRun = 4;
__device__ __forceinline__ uint32_t xcd_runs(uint32_t b, uint32_t n)
{
    constexpr uint32_t kXcds = 8;
    const uint32_t full = n / (kXcds * kTileRun) * (kXcds * kTileRun);
    if (b >= full) return b;
    return ((b / kXcds / kTileRun) * kXcds + b % kXcds) * kTileRun + (b / kXcds) % kTileRun;
}

// ---- hand-out of a launch's tiles ----
// A launch covers the tiles tile0 .. tile0 + n - 1 of one segment with g <= n workgroups.  Workgroup b starts on
// the b-th of them (the first g dealt by first_round).  If n > g, it asks towards the end of every tile for the next
// tile nobody has taken: tile g + (value of a counter that every asker bumps); the answer is looked at once the
// tile in hand is done, so most of the atomic's round trip is covered (asked at the start of a tile, the answer
// stood in the way of the tile's first loads, which the hardware hands back in order: with all workgroups of
// a launch asking at once that was 10 to 20 us).  The last workgroup to leave puts the two words back to zero for
// the next launch (launches of one task run one after the other on one stream).  Which workgroup takes which tile has
// no bearing on what the tile computes.  Thread 0 only.
constexpr uint32_t kHandOutStopped = 1u << 30;      // set in the counter: every later asker is sent home
constexpr uint32_t kAskLater = 0xffffffffu;

__device__ __forceinline__ uint32_t ask_next_tile(uint32_t* sched)
{
    return gridDim.x + atomicAdd(&sched[0], 1u);        // (at or beyond the launch's tile count: nothing left)
}

// With the device gate: the time left in the bubble is no longer enough for another tile.  The hand-out stops - the
// tiles taken so far, which form the head of the launch's tile list, are finished by their workgroups - and the
// first workgroup to find this out records how many tiles that is.  Returns a tile number beyond the launch.
__device__ __forceinline__ uint32_t stop_hand_out(uint32_t* sched, const GateArg& G, uint32_t n_tiles)
{
    const uint32_t before = atomicOr(&sched[0], kHandOutStopped);
    if (!(before & kHandOutStopped)) {
        const uint32_t taken = gridDim.x + before < n_tiles ? gridDim.x + before : n_tiles;
        if (taken < n_tiles) fr_gate_stop_short(G.gate, G.slot, taken);
    }
    return n_tiles;
}

// The question for the next tile, put late in a tile (ahead_ticks: what of the tile is still to come): asked only
// if the gate leaves time for the rest of this tile and another one, else put off to the tile's end.
__device__ __forceinline__ uint32_t ask_if_time(uint32_t* sched, const GateArg& G)
{
    return fr_gate_may_take(G.gate, G.tile_ticks, G.tile_ticks) ? ask_next_tile(sched) : kAskLater;
}

// At a tile's end: the answer, asking now if that was put off and stopping the hand-out if time has run out.
__device__ __forceinline__ uint32_t settle_next_tile(uint32_t asked, uint32_t* sched, const GateArg& G, uint32_t n_tiles)
{
    if (asked != kAskLater) return asked;
    return fr_gate_may_take(G.gate, 0u, G.tile_ticks) ? ask_next_tile(sched) : stop_hand_out(sched, G, n_tiles);
}

__device__ __forceinline__ void leave_launch(uint32_t* sched)
{
    // (this thread's own asks have returned: their values were used)
    if (atomicAdd(&sched[1], 1u) == gridDim.x - 1) {
        __hip_atomic_store(&sched[0], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&sched[1], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// The two words start at zero (and every launch leaves them so).
__global__ void k_clear_sched(uint32_t* sched)
{
    if (threadIdx.x < 2) sched[threadIdx.x] = 0u;
}

// ---- S_k ----
// One workgroup per scatter tile at a time: contrib of its sources sits in LDS, and for every range j the messages of bin
// (tile, j) - a contiguous run [x, y) of message numbers - are written.  The unit of work is a GROUP of four or eight
// consecutive message numbers, aligned to as many: one 8- or 16-byte load brings the sources, LDS reads their contrib,
// one or two 16-byte stores write the messages (groups cut by the ends of a bin store element by element).
// The groups of all bins of a batch are numbered consecutively (prefix sums in LDS) and dealt to the threads, so bins of
// any length keep all lanes busy; a thread finds a group's bin by binary search, and the loads of the groups a thread has
// in flight are issued before the first is used.
// Groups of four are dealt to the wavefronts in runs of up to kAhead * 64 lane by lane (a wavefront's store is 1 KB in one
// piece, and the next 64 groups are mostly in the same bin), groups of eight round-robin; which: scatter_in_runs.
constexpr uint32_t kDescBatch = 1024;       // bins per batch

// Exclusive prefix sums of one value per thread over the workgroup, in two halves with a barrier between them: the first
// leaves every wavefront's total in wave_tot; the second returns the sum of the values of the threads before this one, and
// the sum of all.
__device__ __forceinline__ uint32_t scan_in_wave(uint32_t value, uint32_t* wave_tot)
{
    const uint32_t incl = wave_scan(value);
    if ((threadIdx.x & 63) == 63) wave_tot[threadIdx.x >> 6] = incl;
    return incl - value;
}
__device__ __forceinline__ uint32_t scan_over_waves(uint32_t before_in_wave, const uint32_t* wave_tot, uint32_t* all)
{
    static_assert(kScatterWaves == 16, "the totals are one row of lanes");
    const uint32_t lane = threadIdx.x & 63, wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint32_t incl = wave_scan(lane < kScatterWaves ? wave_tot[lane] : 0u);
    *all = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
    return before_in_wave + (wave ? (uint32_t)__builtin_amdgcn_readlane((int)incl, (int)wave - 1) : 0u);
}

struct GroupRef {
    uint32_t m0;      // first message number of the group (a multiple of its size)
    uint32_t bin;     // its bin in the batch
};

// Group numbers k[0 .. n) of the batch: the bin of one is the last whose first group number is <= k.  The n searches go side by
// side, a fixed number of steps each (one after the other, four searches among a thousand bins were forty reads of the LDS
// in a row).  step0: the largest power of two below the number of bins; gpre holds the number of all groups behind its end.
template <int kSearches>
__device__ __forceinline__ void find_bins(const uint32_t (&k)[kSearches], const uint32_t* gpre, uint32_t step0, uint32_t (&bin)[kSearches])
{
#pragma unroll
    for (int a = 0; a < kSearches; ++a) bin[a] = 0;
    for (uint32_t step = step0; step; step >>= 1) {
#pragma unroll
        for (int a = 0; a < kSearches; ++a) {
            const uint32_t at = bin[a] + step;
            bin[a] = gpre[at] <= k[a] ? at : bin[a];
        }
    }
}

__device__ __forceinline__ uint32_t find_bin(uint32_t k, const uint32_t* gpre, uint32_t lo, uint32_t hi)
{
    while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) >> 1;
        if (gpre[mid] <= k) lo = mid;
        else hi = mid;
    }
    return lo;
}

// The bin of a group 64 numbers on from one in bin `lo`: mostly the same, else within 64 bins unless there are empty ones.
__device__ __forceinline__ uint32_t next_bin(uint32_t k, const uint32_t* gpre, uint32_t lo, uint32_t nb)
{
    if (k < gpre[lo + 1]) return lo;
    const uint32_t near = lo + 65 < nb ? lo + 65 : nb;
    return find_bin(k, gpre, lo + 1, gpre[near] > k ? near : nb);
}

template <uint32_t kGroup>
struct GroupSources { uint32_t w[kGroup / 2]; };      // two 16-bit sources a word

template <uint32_t kGroup>
__device__ __forceinline__ GroupSources<kGroup> load_group(const uint16_t* __restrict__ src16, uint32_t m0)
{
    if constexpr (kGroup == 4) {
        const uint2 r = reinterpret_cast<const uint2*>(src16)[m0 / 4];
        return {{r.x, r.y}};
    } else {
        const uint4 r = reinterpret_cast<const uint4*>(src16)[m0 / 8];
        return {{r.x, r.y, r.z, r.w}};
    }
}

template <uint32_t kGroup>
__device__ __forceinline__ void emit_group(const GroupRef& ref, const uint2* desc, const GroupSources<kGroup>& raw, const float* slice, uint32_t n,
                                           float* __restrict__ msg)
{
    struct { uint32_t m0, x, y; } g = {ref.m0, desc[ref.bin].x, desc[ref.bin].y};
    float val[kGroup];
#pragma unroll
    for (int e = 0; e < (int)kGroup; ++e) {
        const uint32_t src = (e & 1) ? (raw.w[e >> 1] >> 16) : (raw.w[e >> 1] & 0xffffu);
        val[e] = src < n ? slice[src] : 0.0f;
    }
    if (g.m0 >= g.x && g.m0 + kGroup <= g.y) {
        float4* out = reinterpret_cast<float4*>(msg + g.m0);
#pragma unroll
        for (int e = 0; e < (int)kGroup; e += 4) out[e / 4] = make_float4(val[e], val[e + 1], val[e + 2], val[e + 3]);
    } else {
#pragma unroll
        for (int e = 0; e < (int)kGroup; ++e)
            if (g.m0 + e >= g.x && g.m0 + e < g.y) msg[g.m0 + e] = val[e];
    }
}

// `parity` names the set of dangling partials that belongs to the iteration just finished (ignored when first).
// (two workgroups of the small size share a CU: 8 wavefronts per SIMD, hence at most 64 registers per lane)
// kPacked: some tile has more than one piece (kept apart: the loop over pieces costs the small size registers it
// does not have).
// kRuns: groups of four in runs (see above).
// kDynamic: the launch has more tiles than workgroups (else a workgroup's one tile is all it does, and the code of
// the hand-out, which costs registers too, is left out).
template <uint32_t kSrcPerPart, bool kPacked, bool kDynamic, bool kRuns>
__global__ __launch_bounds__(kScatterBlock) __attribute__((amdgpu_waves_per_eu(kSrcPerPart == kSrcSmall ? 8 : 4, kSrcPerPart == kSrcSmall ? 8 : 4)))
void k_scatter(DevArgs A, GateArg G, uint32_t tile0, uint32_t n_tiles, int parity, int first, const ScatterTile* __restrict__ tiles)
{
    __shared__ __align__(16) float slice[kSrcPerPart];
    __shared__ uint2 desc[kDescBatch];
    __shared__ uint32_t gpre[kScatterBlock + 1];          // groups before each bin of the batch; [kScatterBlock] = all
    __shared__ uint32_t wave_tot[kScatterWaves];
    __shared__ float red[kScatterWaves];
    __shared__ float groups[kStrands / 64];
    __shared__ uint32_t next_local;
    static_assert(kDescBatch <= kScatterBlock, "one bin per thread");
    static_assert(kScatterBlock == kStrands, "a thread per strand");
    if (!fr_gate_admit(G.gate, G.slot, kDynamic ? G.tile_ticks : G.need_ticks)) return;
    const uint32_t Qe = A.Qe;
    float strand = 0.0f, base = 0.0f;
    if (!first) strand = dangling_strand(A.dpart + (size_t)parity * A.n_dpart, A.n_dpart, threadIdx.x);
    bool summed = first;                          // base is known
    auto base_value = [&] { return (1.0f - A.damping) / (float)A.V + A.damping * dangling_total(groups) / (float)A.V; };
    // Where a workgroup does one tile of the small size the groups are numbered while the slice's values are not there yet, and
    // the dangling partials put together behind the same barrier.  (The large size asks for its slice, 128 KB, first: 2^24 / 2^28
    // 116.8 -> 113.6 us a sweep; and where tiles are handed out there are no registers for it.  With packed tiles it takes registers, too,
    // eleven spilled instead of seven, and is about as fast: fourteen graphs of 10^6 to 4 x 10^6 vertices and 0.3 to 2 edges a vertex, on 24
    // units up to 2.5 % less an iteration with it, on 64 up to 1.6 % more.)
    constexpr bool kNumberFirst = kSrcPerPart == kSrcSmall && !kDynamic;
    if constexpr (!kNumberFirst)
        if (!first) {
            dangling_group(strand, threadIdx.x & ~63u, groups);
            __syncthreads();
            base = base_value();
        }
    constexpr uint32_t kGroup = kRuns ? 4 : 8;
    // rows a thread reads per round while the slice is filled (the small size has 64 registers per lane)
    constexpr int kFillRound = kSrcPerPart == kSrcSmall ? 4 : 16;
    uint32_t asked = kAskLater;          // thread 0: the answer to its question for the next tile
    bool last_piece = false;
    auto do_piece = [&](uint32_t t, ScatterPiece T, RangeInfo first_info) {
        // the first batch of bin descriptors is asked for now and used after the slice is filled
        uint2 d_first = make_uint2(0, 0);
        if (threadIdx.x < Qe) d_first = A.bins[(uint64_t)t * Qe + threadIdx.x];
        uint32_t total = 0, step0 = 0;            // groups of the batch; for the search among its bins
        // the groups of a batch of bins are numbered (`then`: what is ready for the same barrier)
        auto number_groups = [&](uint2 d, uint32_t nb, auto then) {
            if (d.y > A.M) d.y = A.M;
            if (d.x > d.y) d.x = d.y;
            const uint32_t mine = threadIdx.x < nb && d.y > d.x ? (d.y - 1) / kGroup - d.x / kGroup + 1 : 0;
            const uint32_t before = scan_in_wave(mine, wave_tot);
            then();
            __syncthreads();
            gpre[threadIdx.x] = scan_over_waves(before, wave_tot, &total);
            if (threadIdx.x == 0) gpre[kScatterBlock] = total;
            desc[threadIdx.x] = d;
            if constexpr (!kRuns) step0 = nb > 1 ? 1u << (31 - __builtin_clz(nb - 1)) : 0u;
        };
        if constexpr (kNumberFirst) {
            number_groups(d_first, Qe < kDescBatch ? Qe : kDescBatch, [&] { if (!summed) dangling_group(strand, threadIdx.x & ~63u, groups); });
            if (!summed) base = base_value();
            summed = true;
        }
        const uint32_t u0 = T.u0;
        const uint32_t n = T.u1 - T.u0 < kSrcPerPart ? T.u1 - T.u0 : kSrcPerPart;
        if (first) {
            const float r0 = 1.0f / (float)A.V;
            for (uint32_t ib = threadIdx.x; ib < n; ib += kFillRound * kScatterBlock) {
                float v[kFillRound];
#pragma unroll
                for (int k = 0; k < kFillRound; ++k) {
                    const uint32_t i = ib + k * kScatterBlock;
                    v[k] = i < n ? A.inv_out[u0 + i] : 0.0f;
                }
#pragma unroll
                for (int k = 0; k < kFillRound; ++k) {
                    const uint32_t i = ib + k * kScatterBlock;
                    if (i < n) slice[i] = r0 * v[k] * kMsgScale;
                }
            }
        } else {
            const float mass = wave_sum(fill_slice<kScatterBlock, kFillRound, kSrcPerPart == kSrcLarge>(A, u0, n, base, slice, first_info));
            if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = mass;
        }
        for (uint32_t qb = 0; qb == 0 || qb < Qe; qb += kDescBatch) {       // (once where there are no bins at all)
            const uint32_t nb = Qe - qb < kDescBatch ? Qe - qb : kDescBatch;
            if (!kNumberFirst || qb) {
                __syncthreads();                                 // previous batch consumed
                uint2 d = d_first;
                if (qb) d = threadIdx.x < nb ? A.bins[(uint64_t)t * Qe + qb + threadIdx.x] : make_uint2(0, 0);
                number_groups(d, nb, [] {});
            }
            __syncthreads();                                     // slice filled, groups numbered
            if (qb == 0 && !first && threadIdx.x == 0) {
                float mass = 0.0f;
#pragma unroll
                for (int w = 0; w < kScatterWaves; ++w) mass += red[w];
                A.dpart[(size_t)(parity ^ 1) * A.n_dpart + A.n_pieces + t] = mass;
            }
            // the question for the next tile goes out with the tile's last groups: put earlier, a workgroup on a
            // heavy tile would book its next tile hundreds of microseconds before it is free to start it
            auto ask_with_last = [&](bool last_groups) {
                if constexpr (kDynamic)
                    if (threadIdx.x == 0 && last_piece && qb + kDescBatch >= Qe && last_groups) asked = ask_if_time(A.sched, G);
            };
            auto group_at = [&](uint32_t k, uint32_t bin) { return GroupRef{(desc[bin].x / kGroup + (k - gpre[bin])) * kGroup, bin}; };
            if constexpr (!kRuns) {
                constexpr uint32_t kAhead = 4;                   // groups a thread has in flight
                for (uint32_t k0 = threadIdx.x; k0 < total; k0 += kAhead * kScatterBlock) {
                    ask_with_last(k0 + kAhead * kScatterBlock >= total);
                    uint32_t number[kAhead], bin[kAhead];
                    GroupRef ref[kAhead];
                    GroupSources<kGroup> raw[kAhead];
#pragma unroll
                    for (uint32_t a = 0; a < kAhead; ++a) number[a] = k0 + a * kScatterBlock < total ? k0 + a * kScatterBlock : k0;
                    find_bins(number, gpre, step0, bin);
#pragma unroll
                    for (uint32_t a = 0; a < kAhead; ++a) {      // (behind the last group: one that is there)
                        ref[a] = group_at(number[a], bin[a]);
                        raw[a] = load_group<kGroup>(A.src16, ref[a].m0);
                    }
#pragma unroll
                    for (uint32_t a = 0; a < kAhead; ++a)
                        if (k0 + a * kScatterBlock < total) emit_group<kGroup>(ref[a], desc, raw[a], slice, n, A.msg);
                }
            } else {
                // (runs are shorter where all wavefronts get some then)
                constexpr uint32_t kAhead = 4;
                const uint32_t ahead = total >= kAhead * kScatterBlock ? kAhead : (total + kScatterBlock - 1) / kScatterBlock;
                for (uint32_t k0 = (threadIdx.x / 64) * (ahead * 64) + threadIdx.x % 64; k0 < total; k0 += ahead * kScatterBlock) {
                    ask_with_last(k0 + ahead * kScatterBlock >= total);
                    GroupRef ref[kAhead];
                    GroupSources<kGroup> raw[kAhead];
                    uint32_t bin = 0;
#pragma unroll
                    for (uint32_t a = 0; a < kAhead; ++a) {
                        const uint32_t k = k0 + a * 64;
                        ref[a] = GroupRef{0, 0};
                        raw[a] = GroupSources<kGroup>{};
                        if (a < ahead && k < total) {
                            bin = a == 0 ? find_bin(k, gpre, 0, nb) : next_bin(k, gpre, bin, nb);
                            ref[a] = group_at(k, bin);
                            raw[a] = load_group<kGroup>(A.src16, ref[a].m0);
                        }
                    }
#pragma unroll
                    for (uint32_t a = 0; a < kAhead; ++a)
                        if (a < ahead && k0 + a * 64 < total) emit_group<kGroup>(ref[a], desc, raw[a], slice, n, A.msg);
                }
            }
        }
    };
    uint32_t local = xcd_runs(blockIdx.x, gridDim.x);
    do {
        asked = kAskLater;
        const uint4* rec = reinterpret_cast<const uint4*>(tiles + (tile0 + (uint32_t)__builtin_amdgcn_readfirstlane((int)local)));
        const uint4 span = rec[0];                               // x, y: the tile's pieces, worked on one after the other;
        const uint4 span_info = rec[1];                          // z, w: the sources of the first; then their range
        if constexpr (!kPacked) {
            last_piece = true;
            do_piece(span.x, ScatterPiece{span.z, span.w}, RangeInfo{span_info.x, span_info.y});
            __syncthreads();                                     // the piece is done with slice and desc
        } else {
            for (uint32_t t = span.x; t < span.y; ++t) {
                last_piece = t + 1 == span.y;
                if (t == span.x) {
                    do_piece(t, ScatterPiece{span.z, span.w}, RangeInfo{span_info.x, span_info.y});
                } else {
                    const ScatterPiece T = A.scatter_pieces[t];
                    do_piece(t, T, first ? RangeInfo{kRangeEmpty, 0} : A.range_info[T.u0 >> A.rows_shift]);
                }
                __syncthreads();                                 // the piece is done with slice and desc
            }
        }
        if (tile0 + local == 0 && !first && A.void_slot != kNoVoid && threadIdx.x == 0)       // (once per sweep)
            A.dpart[(size_t)(parity ^ 1) * A.n_dpart + A.n_pieces + A.void_slot] = base * A.n_void_dangling;
        if constexpr (kDynamic) {
            if (threadIdx.x == 0) next_local = settle_next_tile(asked, A.sched, G, n_tiles);
            __syncthreads();
            local = next_local;
        }
    } while (kDynamic && local < n_tiles);
    if constexpr (kDynamic)
        if (threadIdx.x == 0) leave_launch(A.sched);
    fr_gate_done(G.gate, G.slot);
}

// ---- G_k ----

// floor(x * 2^62) for 0 <= x <= 1, exactly, from t = x * 2^30 (the scatter sweep writes its messages scaled so: a
// power of two, hence exact, and one multiplication less per edge here): the integer part of t is the high word,
// its fraction times 2^32 (exact again, then truncated) the low word.
__device__ __forceinline__ unsigned long long to_fixed(float t)
{
    const uint32_t hi = (uint32_t)t;
    const uint32_t lo = (uint32_t)(__builtin_amdgcn_fractf(t) * 4294967296.0f);
    return ((unsigned long long)hi << 32) | lo;
}

__device__ __forceinline__ unsigned long long* acc_at(unsigned long long* acc, uint32_t byte_offset)
{
    return reinterpret_cast<unsigned long long*>(reinterpret_cast<char*>(acc) + byte_offset);
}

__device__ __forceinline__ uint32_t id_of(const uint4& raw, int j)
{
    const uint32_t w = (j >> 1) == 0 ? raw.x : (j >> 1) == 1 ? raw.y : (j >> 1) == 2 ? raw.z : raw.w;
    return (j & 1) ? (w >> 16) : (w & 0xffffu);
}

// One workgroup per gather tile; it takes the tile's pieces one after the other, the accumulators of the piece's
// range (one u64 per row) in LDS.  Per step a wavefront takes one chunk of 512 ids (8 per lane).  The chunks that lie wholly
// inside the piece go through a pipeline without a branch in it, so that the compiler can count what is in flight:
//   A  the chunk's start bits (through the scalar unit) are asked for two steps before its messages, its ids one;
//   B  the start bits tell every id which message it belongs to, and the messages are requested (64 consecutive ids per load,
//      so the addresses are all but contiguous): eight loads, one base address for the chunk and 32-bit offsets from it;
//   C  the chunk of the step before (messages now here): each id adds its message, as a 64-bit fixed-point integer, to its
//      row's accumulator with an LDS atomic.  An id is the byte offset of its row's accumulator divided by 8 / kIdScale, so
//      any 16-bit value stays inside `acc` (the sink slot is its end).
// Behind a wavefront's last chunk that one is asked for again: loads that nothing uses instead of conditions.  (With loads
// under conditions, and checked and unchecked chunks in one loop, as it was before, the compiler waited for a chunk's messages
// in the step that asked for them, and the small kernel for every start record as soon as it was requested.  us an iteration:
// 2^14 vertices / 2^18 edges 17.2 -> 15.0, 10^6 / 10^7 31.4 -> 26.3, 2^22 / 2^26 76.2 -> 74.1, 2^24 / 2^28 343 -> 339.  What
// bounds it on the large graphs is the memory's rate, on the small ones the chain record - ids - messages.)
// The first and last chunk of a piece that is not cut on multiples of 512 go through a path with a check per id, before the
// others, in the wavefronts that have fewest of those.
// (two workgroups of the small size share a CU: 8 wavefronts per SIMD, hence at most 64 registers per lane)
template <uint32_t kRowsPerPart, bool kDynamic>
__global__ __launch_bounds__(kGatherBlock) __attribute__((amdgpu_waves_per_eu(kRowsPerPart == kRowsSmall ? 8 : 4, kRowsPerPart == kRowsSmall ? 8 : 4)))
void k_gather(DevArgs A, GateArg G, uint32_t tile0, uint32_t n_tiles, int parity, int final_pass, const uint64_t* __restrict__ starts,
              const uint32_t* __restrict__ mbase, const GatherTile* __restrict__ tiles, const GatherPiece* __restrict__ pieces)
{
    constexpr uint32_t kAccSlots = kRowsPerPart;
    constexpr uint32_t kIdScale = id_scale_for(kRowsPerPart);
    static_assert(65535u * (8 / kIdScale) + 8 <= (kAccSlots + 1) * 8, "any id addresses a slot of acc");
    __shared__ __align__(16) unsigned long long acc[kAccSlots + 2];      // + the sink slot, and one to make pairs
    __shared__ float red[kGatherWaves];
    __shared__ float groups[kStrands / 64];
    __shared__ uint32_t next_local;
    static_assert(kGatherBlock == kStrands, "a thread per strand");
    if (!fr_gate_admit(G.gate, G.slot, kDynamic ? G.tile_ticks : G.need_ticks)) return;
    const float strand = dangling_strand(A.dpart + (size_t)parity * A.n_dpart, A.n_dpart, threadIdx.x);
    float* dnext = A.dpart + (size_t)(parity ^ 1) * A.n_dpart;
    const uint32_t lane = threadIdx.x & 63, wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    uint32_t local = blockIdx.x;
    do {
    const GatherTile* tile = tiles + (tile0 + (uint32_t)__builtin_amdgcn_readfirstlane((int)local));
    const uint32_t p0 = tile->p0, p1 = tile->p1;                 // the tile's pieces, worked on one after the other;
    GatherPiece T = tile->first;                                 // with a copy of the first (saves a dependent load)
    uint32_t asked = 0;
    for (uint32_t t = p0; t < p1; ++t) {
    const GatherPiece T_next = pieces[t + 1 < p1 ? t + 1 : t];
    for (uint32_t i = threadIdx.x; i < kAccSlots / 2 + 1; i += kGatherBlock) reinterpret_cast<ulonglong2*>(acc)[i] = make_ulonglong2(0ull, 0ull);
    __syncthreads();

    const uint32_t e0 = T.e0, e1 = T.e1 < (uint64_t)A.E ? T.e1 : (uint32_t)A.E;
    const uint4* ids4 = reinterpret_cast<const uint4*>(A.ids16);
    // a chunk's start bits (row j: bit l - 1 says that position l begins a message, bit 63 that position 0 does) and the number
    // of messages begun before it; the same in all lanes of a wavefront, hence in scalar registers
    struct Starts { uint64_t bits[8]; uint32_t mb; };
    auto ask_starts = [&](Starts& S, uint32_t c) {
        const uint64_t* rec = starts + (uint64_t)c * kStartWords;
#pragma unroll
        for (int j = 0; j < 8; ++j) S.bits[j] = rec[j];
        S.mb = mbase[c];
    };
    // The message of the id in lane l (position 64 j + l) is the message of the row's first id plus the messages begun at
    // positions 1 .. l, which is what mbcnt counts in the row's word: as a distance from message mb - 1, in bytes
    auto distances = [&](uint32_t (&at)[8], const Starts& S) {
        uint32_t before = 0;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const uint32_t begun = __builtin_amdgcn_mbcnt_hi((uint32_t)(S.bits[j] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)S.bits[j], 0u));
            at[j] = (begun << 2) + ((before + (uint32_t)(S.bits[j] >> 63)) << 2);
            before += (uint32_t)__popcll(S.bits[j]);
        }
    };
    const uint32_t f0 = (e0 + kIdChunk - 1) / kIdChunk, f1 = e1 / kIdChunk;      // chunks wholly inside: [f0, f1)
    const uint32_t n_full = f1 > f0 ? f1 - f0 : 0;
    if (e1 > e0) {
        const uint32_t ca = e0 / kIdChunk, cb = e1 / kIdChunk;
        const bool has_a = e0 % kIdChunk != 0, has_b = e1 % kIdChunk != 0 && !(has_a && ca == cb);
        const bool do_a = has_a && wave == n_full % kGatherWaves, do_b = has_b && wave == (n_full + 1) % kGatherWaves;
        if (do_a || do_b) {
            const uint32_t c = do_a ? ca : cb;
            const uint4 raw = ids4[(uint64_t)c * (kIdChunk / 8) + lane];
            Starts S;
            ask_starts(S, c);
            uint32_t at[8];
            distances(at, S);
            uint32_t ok = 0;
            float val[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const uint32_t mi = S.mb - 1u + at[j] / 4, e = c * kIdChunk + lane + 64 * j;
                const bool good = e >= e0 && e < e1 && id_of(raw, j) < kAccSlots * kIdScale && mi < A.M;   // (mi wraps if no message precedes)
                ok |= (good ? 1u : 0u) << j;
                val[j] = A.msg[good ? mi : 0u];
            }
#pragma unroll
            for (int j = 0; j < 8; ++j)
                if ((ok >> j) & 1u) atomicAdd(acc_at(acc, id_of(raw, j) * (8 / kIdScale)), to_fixed(val[j]));
        }
    }
    if (wave < n_full) {
        uint32_t c = f0 + wave;
        const uint32_t last = c + (n_full - 1 - wave) / kGatherWaves * kGatherWaves;       // this wavefront's last chunk
        uint4 raw[2];
        Starts S[2];
        float val[2][8];
        auto ahead = [&](uint32_t steps) { return c + steps * kGatherWaves < last ? c + steps * kGatherWaves : last; };
        auto ask_ids = [&](uint4& r, uint32_t at) { r = ids4[(uint64_t)at * (kIdChunk / 8) + lane]; };
        auto ask_messages = [&](float (&v)[8], const Starts& of) {
            // (message mb - 1 is not touched by a chunk that begins a message at its first position: not below the array)
            const char* near = reinterpret_cast<const char*>(A.msg) + ((uint64_t)of.mb << 2) - 4;
            uint32_t at[8];
            distances(at, of);
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = *reinterpret_cast<const float*>(near + at[j]);
        };
        auto add = [&](const uint4& r, const float (&v)[8]) {
#pragma unroll
            for (int j = 0; j < 8; ++j) atomicAdd(acc_at(acc, id_of(r, j) * (8 / kIdScale)), to_fixed(v[j]));
        };
        // one step, on a chunk whose messages were asked for in the step before
        auto step = [&](int k) {
            ask_messages(val[k ^ 1], S[k ^ 1]);                  // of the next chunk
            ask_starts(S[k ^ 1], ahead(3));
            __builtin_amdgcn_sched_barrier(0);
            add(raw[k], val[k]);
            __builtin_amdgcn_sched_barrier(0);
            ask_ids(raw[k], ahead(2));
            c += kGatherWaves;
        };
        ask_starts(S[0], c);
        ask_ids(raw[0], c);
        ask_ids(raw[1], ahead(1));
        ask_messages(val[0], S[0]);
        ask_starts(S[1], ahead(1));
        ask_starts(S[0], ahead(2));
        const uint32_t steps = (last - c) / kGatherWaves + 1;
        for (uint32_t i = 0; i < steps / 2; ++i) {               // (one basic block: else requests sink to where they are used)
            step(0);
            step(1);
        }
        if (steps & 1) add(raw[0], val[0]);
    }
    if (t == p0) dangling_group(strand, threadIdx.x & ~63u, groups);
    const uint32_t q = T.range;
    const int64_t v0 = (int64_t)q * kRowsPerPart;
    const uint32_t nrows = (uint32_t)(A.V - v0 < (int64_t)kRowsPerPart ? A.V - v0 : (int64_t)kRowsPerPart);
    __syncthreads();
    if constexpr (kDynamic)
        if (t + 1 == p1 && threadIdx.x == 0) asked = ask_if_time(A.sched, G);   // covered by the row pass below

    if (T.partial != kNoPartial) {
        // merged range: the sums go out as one row of partial sums; the next scatter sweep (or F) finishes the rows
        float2* out = reinterpret_cast<float2*>(A.partials + (size_t)T.partial * kRowsPerPart);
#pragma unroll 4
        for (uint32_t i = threadIdx.x; i < kRowsPerPart / 2; i += kGatherBlock) {
            const ulonglong2 two = reinterpret_cast<const ulonglong2*>(acc)[i];
            out[i] = make_float2((float)two.x * kFixInv, (float)two.y * kFixInv);
        }
        if (threadIdx.x == 0 && !final_pass) dnext[t] = 0.0f;
    } else {
    // direct range: fused vertex pass for its rows
    const float base = (1.0f - A.damping) / (float)A.V + A.damping * dangling_total(groups) / (float)A.V;
    float dangling = 0.0f;
    constexpr int kRowsPerThread = (kRowsPerPart + kGatherBlock - 1) / kGatherBlock;
    if (final_pass) {
#pragma unroll
        for (int k = 0; k < kRowsPerThread; ++k) {
            const uint32_t i = threadIdx.x + kGatherBlock * k;
            if (i < nrows) A.ranks_out[A.perm[v0 + i]] = fmaf(A.damping, (float)acc[i] * kFixInv, base);
        }
    } else {
        float inv[kRowsPerThread];
#pragma unroll
        for (int k = 0; k < kRowsPerThread; ++k) {
            const uint32_t i = threadIdx.x + kGatherBlock * k;
            inv[k] = A.inv_out[v0 + (i < nrows ? i : nrows - 1)];
        }
#pragma unroll
        for (int k = 0; k < kRowsPerThread; ++k) {
            const uint32_t i = threadIdx.x + kGatherBlock * k;
            if (i >= nrows) continue;
            const float r = fmaf(A.damping, (float)acc[i] * kFixInv, base);
            A.contrib[v0 + i] = r * inv[k];
            dangling += (inv[k] == 0.0f ? r : 0.0f);
        }
        const float total = block_sum(dangling, red);
        if (threadIdx.x == 0) dnext[t] = total;
    }
    }
    if (tile0 == 0 && blockIdx.x == 0 && local == 0 && t == p0 && !final_pass)   // slots no gather piece writes: the scatter tiles of the next
        for (uint32_t i = A.n_pieces + threadIdx.x; i < A.n_dpart; i += kGatherBlock) dnext[i] = 0.0f;   // sweep fill theirs in, void pieces have none
    __syncthreads();                                             // the piece is done with acc
    T = T_next;
    }       // pieces
    if constexpr (kDynamic) {
        if (threadIdx.x == 0) next_local = settle_next_tile(asked, A.sched, G, n_tiles);
        __syncthreads();
        local = next_local;
    }
    } while (kDynamic && local < n_tiles);       // tiles
    if constexpr (kDynamic)
        if (threadIdx.x == 0) leave_launch(A.sched);
    fr_gate_done(G.gate, G.slot);
}

// ---- F ----
// After the last iteration: r_K of kFinishRows rows of one merged range (partial sums of G_{K-1}) or of one empty
// range (the base value) goes to ranks_out.
constexpr uint32_t kFinishRows = 2048;
__global__ __launch_bounds__(kBlock) void k_finish(DevArgs A, GateArg G, uint32_t tile0, int parity)
{
    __shared__ float groups[kStrands / 64];
    if (!fr_gate_admit(G.gate, G.slot, G.need_ticks)) return;
    const uint32_t t = tile0 + blockIdx.x;
    for (uint32_t i = threadIdx.x; i < kStrands; i += kBlock)
        dangling_group(dangling_strand(A.dpart + (size_t)parity * A.n_dpart, A.n_dpart, i), i & ~63u, groups);
    __syncthreads();
    const float base = (1.0f - A.damping) / (float)A.V + A.damping * dangling_total(groups) / (float)A.V;
    const uint32_t per_range = A.rows_per_part / kFinishRows;
    if (t / per_range < A.n_finish) {
        const uint32_t q = A.finish_ranges[t / per_range];
        const RangeInfo info = A.range_info[q];
        const bool merged = (info.cls_tiles & 3u) == kRangeMerged;
        const int64_t v0 = (int64_t)q << A.rows_shift;
        for (uint32_t k = threadIdx.x; k < kFinishRows; k += kBlock) {
            const uint32_t i = (t % per_range) * kFinishRows + k;
            const int64_t v = v0 + i;
            if (v >= A.V) break;
            A.ranks_out[A.perm[v]] = merged ? fmaf(A.damping, merged_sum<1>(A, info, i, 0), base) : base;
        }
    }
    fr_gate_done(G.gate, G.slot);
}

uint32_t ceil_div_u64(uint64_t a, uint64_t b) { return (uint32_t)((a + b - 1) / b); }

uint64_t ceil_fs_to_ns(unsigned __int128 fs)
{
    const uint64_t ns = (uint64_t)((fs + 999999) / 1000000);
    return ns ? ns : 1;
}

struct PrTask {
    fr_pagerank_desc d{};
    PrLayout L;
    std::vector<uint64_t> prefix[4];      // cumulative modelled tile costs per segment kind (after init)
    uint64_t footprint_after = 0, footprint_peak = 0;
    float *msg = nullptr, *contrib = nullptr, *dpart = nullptr, *partials = nullptr;
    uint32_t* sched = nullptr;
    uint32_t n_dpart = 0;
    DevArgs args{};
    bool inited = false;
    bool registered = false;
    fr_alloc own;                         // used by the standalone run only
    int hip_error = 0;
    uint32_t run = 0, seg = 0, tile = 0;  // cursor

    // V0, then S_k G_k for k < K, then F (no S, G, F at all when K = 0)
    uint32_t n_segments() const { return d.iterations == 0 ? 1u : 2u + 2u * (uint32_t)d.iterations; }
    int kind_of(uint32_t g) const
    {
        if (g == 0) return FR_PR_SEG_VERTEX;
        if (g + 1 == n_segments()) return FR_PR_SEG_FINISH;
        return ((g - 1) & 1u) ? FR_PR_SEG_GATHER : FR_PR_SEG_SCATTER;
    }
    uint32_t tiles_of(int kind) const
    {
        switch (kind) {
        case FR_PR_SEG_VERTEX: return L.Q;
        case FR_PR_SEG_SCATTER: return L.n_scatter;
        case FR_PR_SEG_GATHER: return L.n_gather;
        default: return std::max<uint32_t>(1, L.n_finish * (L.rows_per_part / kFinishRows));
        }
    }
    uint64_t rows_of_q(uint32_t q) const
    {
        return std::min<uint64_t>(L.rows_per_part, (uint64_t)L.V - (uint64_t)q * L.rows_per_part);
    }
};

void build_cost_tables(PrTask* p)
{
    const PrLayout& L = p->L;
    const uint64_t pe = p->d.fs_per_edge, pm = p->d.fs_per_message, pv = p->d.fs_per_vertex;
    auto& v = p->prefix[FR_PR_SEG_VERTEX];
    v.assign(L.Q + 1, 0);
    for (uint32_t q = 0; q < L.Q; ++q) v[q + 1] = v[q] + ceil_fs_to_ns((unsigned __int128)p->rows_of_q(q) * pv);
    auto& s = p->prefix[FR_PR_SEG_SCATTER];
    s.assign(L.n_scatter + 1, 0);
    for (uint32_t i = 0; i < L.n_scatter; ++i) {
        s[i + 1] = s[i] + ceil_fs_to_ns((unsigned __int128)(L.st_msgs[i] + L.st_rows[i]) * pm);   // a value read costs about a message
    }
    auto& g = p->prefix[FR_PR_SEG_GATHER];
    const uint32_t ng = p->tiles_of(FR_PR_SEG_GATHER);
    g.assign(ng + 1, 0);
    for (uint32_t t = 0; t < ng; ++t) {
        g[t + 1] = g[t] + ceil_fs_to_ns((unsigned __int128)L.gt_weight[t] * pe / 2);
    }
    auto& h = p->prefix[FR_PR_SEG_FINISH];
    const uint32_t nf = p->tiles_of(FR_PR_SEG_FINISH);
    h.assign(nf + 1, 0);
    for (uint32_t t = 0; t < nf; ++t) h[t + 1] = h[t] + std::max<uint64_t>(1, p->d.finish_tile_ns);
}

// `with`: the kernel arguments to use instead of the task's own (the run that works in the static scratch array).
int pr_launch(PrTask* p, uint32_t g, uint32_t tile0, uint32_t tile1, hipStream_t stream, GateArg G = GateArg{nullptr, 0, 0, 0},
              const DevArgs* with = nullptr)
{
    const DevArgs& args = with ? *with : p->args;
    const int kind = p->kind_of(g);
    if (tile1 <= tile0 || tile1 > p->tiles_of(kind)) return FR_ERR_ARG;
    const uint32_t n = tile1 - tile0;
    const uint32_t K = (uint32_t)p->d.iterations;
    if (kind == FR_PR_SEG_VERTEX) {
        hipLaunchKernelGGL(k_vertex0, dim3(n), dim3(kBlock), 0, stream, args, G, tile0, K == 0 ? 1 : 0);
    } else if (kind == FR_PR_SEG_FINISH) {
        // after G_{K-1}: the dangling partials of r_{K-1} sit in set (K-1) & 1
        hipLaunchKernelGGL(k_finish, dim3(n), dim3(kBlock), 0, stream, args, G, tile0, (int)((K - 1) & 1u));
    } else {
        const uint32_t k = (g - 1) / 2;
        if (kind == FR_PR_SEG_SCATTER) {    // S_k finishes rows of r_k with D_{k-1}: set (k-1) & 1
            const int parity = (int)((k + 1) & 1u), first = k == 0 ? 1 : 0;
            const uint32_t grid = std::min(n, p->L.scatter_slots);
            const bool packed = p->L.scatter_packed, dynamic = n > grid;
            auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3(grid), dim3(kScatterBlock), 0, stream, args, G, tile0, n, parity, first, args.scatter_tiles); };
            const bool runs = scatter_in_runs(p->L.src_per_part, p->d.n_vertices, p->L.cus, dynamic);
            auto go_as = [&](auto packs) {
                constexpr bool kPacked = decltype(packs)::value;
                if (p->L.src_per_part == kSrcSmall) { if (runs) go(k_scatter<kSrcSmall, kPacked, true, true>); else go(k_scatter<kSrcSmall, kPacked, false, false>); }
                else if (runs) { if (dynamic) go(k_scatter<kSrcLarge, kPacked, true, true>); else go(k_scatter<kSrcLarge, kPacked, false, true>); }
                else { if (dynamic) go(k_scatter<kSrcLarge, kPacked, true, false>); else go(k_scatter<kSrcLarge, kPacked, false, false>); }
            };
            if (packed) go_as(std::true_type{});
            else go_as(std::false_type{});
        } else {
            const int parity = (int)(k & 1u), final_pass = (k + 1 == K) ? 1 : 0;
            const uint32_t grid = std::min(n, p->L.gather_slots);
            const bool dynamic = n > grid;
            auto go = [&](auto kernel) {
                hipLaunchKernelGGL(kernel, dim3(grid), dim3(kGatherBlock), 0, stream, args, G, tile0, n, parity, final_pass, args.starts, args.mbase, args.gather_tiles, args.gather_pieces);
            };
            if (p->L.rows_per_part == kRowsLarge) { if (dynamic) go(k_gather<kRowsLarge, true>); else go(k_gather<kRowsLarge, false>); }
            else { if (dynamic) go(k_gather<kRowsSmall, true>); else go(k_gather<kRowsSmall, false>); }
        }
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) { p->hip_error = (int)e; return FR_ERR_HIP; }
    return FR_OK;
}

int pr_init(void* user, fr_alloc* a, void* stream_v)
{
    PrTask* p = static_cast<PrTask*>(user);
    hipStream_t stream = (hipStream_t)stream_v;
    if (a->host_only) return FR_ERR_ARG;      // this task needs a GPU
    const int64_t V = p->d.n_vertices, E = p->d.n_edges;
    // caller-provided buffers count against the task's limit: row_ptr, col, out_degree, ranks_out
    const uint64_t caller = 4ull * (uint64_t)(V + 1) + 4ull * (uint64_t)E + 4ull * (uint64_t)V + 4ull * (uint64_t)V;
    if (fr_alloc_charge(a, caller) != FR_OK) return FR_ERR_OOM;
    int rc = pr_build_layout(&p->L, V, E, p->d.row_ptr, p->d.col, p->d.out_degree, p->d.rows_per_partition,
                             p->d.sources_per_partition, fr_stream_cus(stream), a, stream, &p->hip_error);
    if (rc != FR_OK) return rc;
    PrLayout& L = p->L;
    // dangling partials: one slot per range (V0), or one per gather piece followed by one per scatter piece
    p->n_dpart = std::max(L.Q, L.n_pieces + L.n_spieces);
    Carve work;
    work.add(&p->msg, L.M); work.add(&p->contrib, (uint64_t)V); work.add(&p->dpart, 2ull * p->n_dpart);
    work.add(&p->partials, (uint64_t)L.n_partials * L.rows_per_part); work.add(&p->sched, 2);
    if (!work.keep_apart(a)) return a->hip_error ? FR_ERR_HIP : FR_ERR_OOM;
    hipLaunchKernelGGL(k_clear_sched, dim3(1), dim3(64), 0, stream, p->sched);
    if (hipStreamSynchronize(stream) != hipSuccess) return FR_ERR_HIP;
    DevArgs& A = p->args;
    A.V = V; A.E = E; A.M = (uint32_t)L.M; A.Q = L.Q; A.Qe = L.Qe;
    A.n_gather = L.n_gather; A.n_pieces = L.n_pieces; A.n_scatter = L.n_scatter; A.n_spieces = L.n_spieces;
    A.n_finish = L.n_finish;
    A.n_dpart = p->n_dpart; A.damping = p->d.damping;
    A.rows_per_part = L.rows_per_part;
    A.rows_shift = L.rows_per_part == kRowsLarge ? 14 : 13;
    A.void_slot = L.void_slot; A.n_void_dangling = (float)L.n_void_dangling;
    A.ids16 = L.ids16; A.src16 = L.src16; A.mbase = L.mbase; A.starts = L.starts; A.bins = L.bins;
    A.inv_out = L.inv_out; A.perm = L.perm; A.range_info = L.range_info;
    A.gather_pieces = L.gather_pieces; A.gather_tiles = L.gather_tiles;
    A.scatter_pieces = L.scatter_pieces; A.scatter_tiles = L.scatter_tiles; A.finish_ranges = L.finish_ranges;
    A.msg = p->msg; A.contrib = p->contrib; A.dpart = p->dpart; A.partials = p->partials; A.ranks_out = p->d.ranks_out;
    A.sched = p->sched;
    build_cost_tables(p);
    p->footprint_after = fr_alloc_used(a);
    p->footprint_peak = fr_alloc_peak(a);
    p->run = 0; p->seg = 0; p->tile = 0;
    p->inited = true;
    return FR_OK;
}

int pr_create(void* user)
{
    static_cast<PrTask*>(user)->registered = true;
    return FR_OK;
}

int pr_plan(void* user, uint64_t budget_ns, uint64_t launch_cost_ns, fr_step* out)
{
    PrTask* p = static_cast<PrTask*>(user);
    std::memset(out, 0, sizeof(*out));
    out->run = p->run; out->segment = p->seg; out->tile0 = p->tile; out->tile1 = p->tile;
    if (!p->inited) return FR_ERR_STATE;
    out->cost_class = (uint32_t)p->kind_of(p->seg);
    if (p->d.max_runs > 0 && p->run >= (uint32_t)p->d.max_runs) { out->finished = 1; return FR_OK; }
    const int kind = p->kind_of(p->seg);
    const std::vector<uint64_t>& pre = p->prefix[kind];
    const uint64_t floor_ns = p->d.min_step_ns[kind];
    if (floor_ns > budget_ns || launch_cost_ns > budget_ns - floor_ns) return FR_OK;     // even the shortest step is too long
    uint32_t n = 0;
    int rc = fr_chunk_fit(pre.data(), p->tiles_of(kind), p->tile, budget_ns, launch_cost_ns, &n);
    if (rc != FR_OK) return rc;
    if (n == 0) return FR_OK;
    // A launch of more tiles than workgroups runs in rounds, each workgroup taking a next tile when it is done with
    // one; the summed tile costs are what whole rounds take.  A step that does not reach the segment's end is
    // therefore cut to whole rounds (the tiles are in order of falling weight, so the light ones that close the
    // segment's last round smoothly are at its end): a round and a few tiles would take two rounds' time.
    const uint32_t slots = kind == FR_PR_SEG_SCATTER ? p->L.scatter_slots : kind == FR_PR_SEG_GATHER ? p->L.gather_slots : 0;
    if (slots && n > slots && p->tile + n < p->tiles_of(kind)) n = n / slots * slots;
    uint64_t cost = std::max(pre[p->tile + n] - pre[p->tile], floor_ns);
    if (slots && n <= slots) {
        // A step of up to a round: its tiles run side by side on part of the slots.  One tile alone takes the floor,
        // a full round the sum of its tiles' costs (each a share of a round), and in between the time was measured
        // to grow linearly with the number of tiles: the sum plus the floor's share of the slots left empty.
        // (a sweep of fewer tiles than slots is full with all of them)
        const uint32_t full = std::min(slots, p->tiles_of(kind));
        auto part = [&](uint32_t k) {
            return std::max(floor_ns, pre[p->tile + k] - pre[p->tile] + floor_ns * (full - k) / full);
        };
        const uint64_t room = budget_ns - launch_cost_ns;            // (launch_cost_ns <= budget_ns - floor_ns, above)
        while (n > 0 && part(n) > room) --n;
        if (n == 0) return FR_OK;
        cost = part(n);
    }
    out->tile1 = p->tile + n;
    out->modelled_ns = cost;
    if (slots && n > slots) {
        // the step's kernel hands its tiles out and can stop between them: what its heaviest tile - the first, they
        // are in order of falling weight - takes a workgroup, i.e. the slot's whole time for it (a tile's cost is its
        // share of a round of `slots` tiles side by side) and a quarter more.  (Not the floor of the segment, which is
        // the heaviest tile of the whole sweep run alone: the steps near a bubble's end are made of the light tiles.)
        const uint64_t heaviest = std::max<uint64_t>(10000, (pre[p->tile + 1] - pre[p->tile]) * slots * 5 / 4);
        out->gate_tile = (uint32_t)std::min<uint64_t>(heaviest, 4000000000ull);
    }
    if (kind == FR_PR_SEG_GATHER) {
        uint64_t edges = 0;
        for (uint32_t t = p->tile; t < p->tile + n && t < p->L.n_gather; ++t) edges += p->L.gt_edges[t];
        out->work_units = edges;
    }
    out->completes_run = (p->seg + 1 == p->n_segments() && out->tile1 == p->tiles_of(kind)) ? 1 : 0;
    return FR_OK;
}

int pr_run(void* user, void* stream, const fr_step* st)
{
    PrTask* p = static_cast<PrTask*>(user);
    if (!p->inited || st->run != p->run || st->segment != p->seg || st->tile0 != p->tile) return FR_ERR_STATE;
    int rc = pr_launch(p, p->seg, st->tile0, st->tile1, (hipStream_t)stream,
                       GateArg{static_cast<fr_gate*>(st->gate), st->gate_slot, st->gate_need_ticks, st->gate_tile});
    if (rc != FR_OK) return rc;
    p->tile = st->tile1;
    if (p->tile == p->tiles_of(p->kind_of(p->seg))) {
        p->tile = 0;
        if (++p->seg == p->n_segments()) { p->seg = 0; p->run++; }
    }
    return FR_OK;
}

// The device gate cut `first` off after `tiles_done` of its tiles, and every step after it did nothing: the cursor goes
// back to the first tile not done.  (A tile done twice computes the same values again: tiles only read what earlier
// segments wrote.)
int pr_rewind(void* user, const fr_step* first, uint32_t tiles_done, uint64_t* work_done)
{
    PrTask* p = static_cast<PrTask*>(user);
    if (!p->inited || !first || !work_done || first->segment >= p->n_segments()) return FR_ERR_ARG;
    const int kind = p->kind_of(first->segment);
    if (first->tile0 >= p->tiles_of(kind) || first->tile1 > p->tiles_of(kind) || tiles_done > first->tile1 - first->tile0) return FR_ERR_ARG;
    p->run = first->run; p->seg = first->segment; p->tile = first->tile0 + tiles_done;
    uint64_t edges = 0;
    if (kind == FR_PR_SEG_GATHER)
        for (uint32_t t = first->tile0; t < first->tile0 + tiles_done && t < p->L.n_gather; ++t) edges += p->L.gt_edges[t];
    *work_done = edges;
    if (p->tile == p->tiles_of(kind)) {            // (a step is only cut off before its last tile; kept for safety)
        p->tile = 0;
        if (++p->seg == p->n_segments()) { p->seg = 0; p->run++; }
    }
    return FR_OK;
}

int pr_stop(void* user)
{
    PrTask* p = static_cast<PrTask*>(user);
    p->inited = false;        // the runtime's allocator frees the device blocks
    p->registered = false;
    return FR_OK;
}

// ---- working memory of fr_pagerank_run_standalone_noalloc: messages, contributions, dangling partials and partial
// sums of one run live in this array instead of in memory taken from an allocator.  Every GPU the library is loaded
// on holds its own copy at its own address; host code never uses the array's name as an address, only the pointer
// hipGetSymbolAddress gave for the device at hand.
constexpr size_t kStaticScratchBytes = (size_t)64 << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
unsigned char* g_scratch_ptr[kMaxDevices] = {};

size_t round256(size_t n) { return (n + 255) / 256 * 256; }

}  // namespace

extern "C" {

int fr_pagerank_make(const fr_pagerank_desc* d, fr_task_ops* ops_out, void** user_out, fr_task_profile* prof_out)
{
    if (!d || !ops_out || !user_out || !prof_out) return FR_ERR_ARG;
    if (d->n_vertices < 1 || d->n_vertices > 0x7fffffffLL || d->n_edges < 0 || d->n_edges > 0x7fffffffLL) return FR_ERR_ARG;
    if (!d->row_ptr || !d->out_degree || !d->ranks_out || (d->n_edges > 0 && !d->col)) return FR_ERR_ARG;
    if (d->iterations < 0 || d->iterations > 100000 || d->max_runs < 0) return FR_ERR_ARG;
    if (!(d->damping >= 0.0f && d->damping <= 1.0f)) return FR_ERR_ARG;
    PrTask* p = new (std::nothrow) PrTask();
    if (!p) return FR_ERR_ARG;
    p->d = *d;
    if (!p->d.fs_per_edge) p->d.fs_per_edge = 2000;
    if (!p->d.fs_per_message) p->d.fs_per_message = 2000;
    if (!p->d.fs_per_vertex) p->d.fs_per_vertex = 4000;
    if (!p->d.finish_tile_ns) p->d.finish_tile_ns = 2000;
    ops_out->create = pr_create;
    ops_out->init = pr_init;
    ops_out->plan_step = pr_plan;
    ops_out->run_step = pr_run;
    ops_out->stop = pr_stop;
    ops_out->rewind = pr_rewind;
    prof_out->mem_limit_bytes = d->mem_limit_bytes;
    prof_out->min_step_ns = 1;
    *user_out = p;
    return FR_OK;
}

int fr_pagerank_destroy(void* user)
{
    PrTask* p = static_cast<PrTask*>(user);
    if (!p) return FR_ERR_ARG;
    if (p->registered) return FR_ERR_STATE;
    if (p->inited) fr_alloc_hand_back(&p->own);
    delete p;
    return FR_OK;
}

int fr_pagerank_info(void* user, fr_pagerank_info_t* out)
{
    PrTask* p = static_cast<PrTask*>(user);
    if (!p || !out) return FR_ERR_ARG;
    if (p->prefix[0].empty()) return FR_ERR_STATE;       // known once InitSideTask has run
    std::memset(out, 0, sizeof(*out));
    out->messages = p->L.M;
    out->ranges = p->L.Q;
    out->nonempty_ranges = p->L.Qe;
    out->merged_ranges = p->L.n_merged;
    out->partial_rows = p->L.n_partials;
    out->gather_tiles = p->L.n_gather;
    out->scatter_tiles = p->L.n_scatter;
    out->rows_per_partition = p->L.rows_per_part;
    out->sources_per_partition = p->L.src_per_part;
    out->bytes_resident = p->footprint_after;
    out->bytes_peak = p->footprint_peak;
    out->scatter_slots = p->L.scatter_slots;
    out->gather_slots = p->L.gather_slots;
    return FR_OK;
}

int fr_pagerank_tiles(void* user, int32_t seg_kind, uint32_t* n_out)
{
    PrTask* p = static_cast<PrTask*>(user);
    if (!p || !n_out || seg_kind < 0 || seg_kind > 3) return FR_ERR_ARG;
    if (p->prefix[0].empty()) return FR_ERR_STATE;
    *n_out = p->tiles_of(seg_kind);
    return FR_OK;
}

int fr_pagerank_tile_costs(void* user, int32_t seg_kind, uint32_t* costs, size_t cap, size_t* n_out)
{
    PrTask* p = static_cast<PrTask*>(user);
    if (!p || !n_out || seg_kind < 0 || seg_kind > 3 || (!costs && cap)) return FR_ERR_ARG;
    if (p->prefix[0].empty()) return FR_ERR_STATE;
    const std::vector<uint64_t>& pre = p->prefix[seg_kind];
    const size_t n = pre.size() - 1;
    for (size_t t = 0; t < std::min(n, cap); ++t) costs[t] = (uint32_t)std::min<uint64_t>(pre[t + 1] - pre[t], 0xffffffffu);
    *n_out = n;
    return FR_OK;
}

int fr_pagerank_tile_work(void* user, int32_t seg_kind, uint64_t* work, size_t cap, size_t* n_out)
{
    PrTask* p = static_cast<PrTask*>(user);
    if (!p || !n_out || seg_kind < 0 || seg_kind > 3 || (!work && cap)) return FR_ERR_ARG;
    if (p->prefix[0].empty()) return FR_ERR_STATE;
    const size_t n = p->tiles_of(seg_kind);
    for (size_t t = 0; t < std::min(n, cap); ++t) {
        if (seg_kind == FR_PR_SEG_GATHER) work[t] = t < p->L.n_gather ? p->L.gt_edges[t] : 0;
        else if (seg_kind == FR_PR_SEG_SCATTER) work[t] = p->L.st_msgs[t];
        else if (seg_kind == FR_PR_SEG_VERTEX) work[t] = p->rows_of_q((uint32_t)t);
        else work[t] = 0;
    }
    *n_out = n;
    return FR_OK;
}

int fr_pagerank_tile_weights(void* user, int32_t seg_kind, uint64_t* weights, size_t cap, size_t* n_out)
{
    PrTask* p = static_cast<PrTask*>(user);
    if (!p || !n_out || seg_kind < 0 || seg_kind > 3 || (!weights && cap)) return FR_ERR_ARG;
    if (p->prefix[0].empty()) return FR_ERR_STATE;
    const size_t n = p->tiles_of(seg_kind);
    for (size_t t = 0; t < std::min(n, cap); ++t) {
        if (seg_kind == FR_PR_SEG_GATHER) weights[t] = p->L.gt_weight[t];
        else if (seg_kind == FR_PR_SEG_SCATTER) weights[t] = p->L.st_rows[t];
        else if (seg_kind == FR_PR_SEG_VERTEX) weights[t] = p->rows_of_q((uint32_t)t);
        else weights[t] = 0;
    }
    *n_out = n;
    return FR_OK;
}

int fr_pagerank_run_standalone(void* user, int32_t device_id, void* stream_v, uint32_t max_tiles, uint64_t* phase_ns)
{
    PrTask* p = static_cast<PrTask*>(user);
    if (!p || device_id < 0) return FR_ERR_ARG;
    if (p->registered) return FR_ERR_STATE;
    hipStream_t stream = (hipStream_t)stream_v;
    FR_HIP_TRY(hipSetDevice(device_id), p->hip_error);
    if (!p->inited) {
        fr_alloc_reset(&p->own, p->d.mem_limit_bytes, false, device_id);
        p->own.pooled = true;
        int rc = pr_init(p, &p->own, stream_v);
        if (rc != FR_OK) {
            const bool oom = p->own.oom;
            fr_alloc_release(&p->own);
            p->inited = false;
            return oom ? FR_ERR_OOM : rc;
        }
    }
    hipEvent_t ev[2] = {nullptr, nullptr};
    float ms_sum[4] = {0.f, 0.f, 0.f, 0.f};
    if (phase_ns) {
        FR_HIP_TRY(hipEventCreate(&ev[0]), p->hip_error);
        FR_HIP_TRY(hipEventCreate(&ev[1]), p->hip_error);
    }
    int rc = FR_OK;
    for (uint32_t g = 0; g < p->n_segments() && rc == FR_OK; ++g) {
        const int kind = p->kind_of(g);
        const uint32_t nt = p->tiles_of(kind);
        const uint32_t step = max_tiles ? max_tiles : nt;
        if (phase_ns) (void)hipEventRecord(ev[0], stream);
        for (uint32_t t0 = 0; t0 < nt && rc == FR_OK; t0 += step) rc = pr_launch(p, g, t0, std::min(nt, t0 + step), stream);
        if (phase_ns) {
            (void)hipEventRecord(ev[1], stream);
            (void)hipEventSynchronize(ev[1]);
            float ms = 0.f;
            if (hipEventElapsedTime(&ms, ev[0], ev[1]) == hipSuccess) ms_sum[kind] += ms;
        }
    }
    hipError_t e = hipStreamSynchronize(stream);
    if (phase_ns) {
        for (int k = 0; k < 4; ++k) phase_ns[k] = (uint64_t)((double)ms_sum[k] * 1.0e6 + 0.5);
        (void)hipEventDestroy(ev[0]);
        (void)hipEventDestroy(ev[1]);
    }
    if (rc != FR_OK) return rc;
    if (e != hipSuccess) { p->hip_error = (int)e; return FR_ERR_HIP; }
    return FR_OK;
}

int fr_pagerank_run_standalone_noalloc(void* user, int32_t device_id, void* stream_v, uint32_t max_tiles)
{
    PrTask* p = static_cast<PrTask*>(user);
    if (!p || device_id < 0 || device_id >= kMaxDevices) return FR_ERR_ARG;
    if (p->registered || !p->inited) return FR_ERR_STATE;        // the layout must exist already: nothing is built here
    hipStream_t stream = (hipStream_t)stream_v;
    FR_HIP_TRY(hipSetDevice(device_id), p->hip_error);
    unsigned char* base = nullptr;
    {
        std::lock_guard<std::mutex> lock(g_scratch_mu);
        if (!g_scratch_ptr[device_id]) {
            void* sym = nullptr;
            FR_HIP_TRY(hipGetSymbolAddress(&sym, HIP_SYMBOL(scratch)), p->hip_error);
            g_scratch_ptr[device_id] = static_cast<unsigned char*>(sym);
        }
        base = g_scratch_ptr[device_id];
    }
    const PrLayout& L = p->L;
    const size_t b_msg = round256((size_t)std::max<uint64_t>(L.M, 1) * 4), b_contrib = round256((size_t)L.V * 4),
                 b_dpart = round256((size_t)2 * p->n_dpart * 4),
                 b_partials = round256((size_t)std::max<uint64_t>((uint64_t)L.n_partials * L.rows_per_part, 1) * 4);
    constexpr size_t b_sched = 256;
    if (b_msg + b_contrib + b_dpart + b_partials + b_sched > kStaticScratchBytes) return FR_ERR_ARG;   // too large for the array
    DevArgs A = p->args;
    A.msg = reinterpret_cast<float*>(base);
    A.contrib = reinterpret_cast<float*>(base + b_msg);
    A.dpart = reinterpret_cast<float*>(base + b_msg + b_contrib);
    A.partials = reinterpret_cast<float*>(base + b_msg + b_contrib + b_dpart);
    A.sched = reinterpret_cast<uint32_t*>(base + b_msg + b_contrib + b_dpart + b_partials);
    hipLaunchKernelGGL(k_clear_sched, dim3(1), dim3(64), 0, stream, A.sched);     // the hand-out words must start at zero
    int rc = FR_OK;
    for (uint32_t g = 0; g < p->n_segments() && rc == FR_OK; ++g) {
        const uint32_t nt = p->tiles_of(p->kind_of(g));
        const uint32_t step = max_tiles ? max_tiles : nt;
        for (uint32_t t0 = 0; t0 < nt && rc == FR_OK; t0 += step)
            rc = pr_launch(p, g, t0, std::min(nt, t0 + step), stream, GateArg{nullptr, 0, 0, 0}, &A);
    }
    hipError_t e = hipStreamSynchronize(stream);
    if (rc != FR_OK) return rc;
    if (e != hipSuccess) { p->hip_error = (int)e; return FR_ERR_HIP; }
    return FR_OK;
}

}  // extern "C"

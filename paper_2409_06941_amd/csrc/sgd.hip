// Graph SGD side task: stochastic gradient descent for matrix factorization over a rating graph, the second graph
// workload the paper harvests bubbles with (Section 6.1.4; Section 6.2: one iteration = one pass over the graph).
//
// The paper names the method only, so the arithmetic is the textbook one (Koren, Bell, Volinsky 2009): for every
// rating r_ui, one after the other,
//     e = r_ui - <p_u, q_i>,   p_u += gamma (e q_i - lambda p_u),   q_i += gamma (e p_u - lambda q_i)
// and the order of the updates is a stratified one (Gemulla et al. 2011), which a GPU can follow without races and
// without depending on timing: users and items are cut into B blocks of consecutive ids holding about E / B ratings
// each (block k begins at the first id with ceil(k E / B) or more ratings before it); the ratings of user block a
// and item block b are cell (a, b); an iteration is B strata, stratum s = the cells (a, (a + s) mod B), which share
// no user and no item and therefore run side by side; inside a cell the ratings are taken by user, then by item,
// one after the other.  Every rounding of an update is fixed (see k_sgd), so the factors do not depend on how the
// cells are grouped into launches, and an fp32 CPU implementation of the same steps gives the same bits.
//
// One run = K iterations = K * B segments (a segment is a stratum; a step is a run of consecutive cells of one
// stratum; tile = cell).  The factors carry over from run to run: the task keeps training.
//
// Layout, built once in InitSideTask (see k_sgd): the ratings are sorted by cell; a cell is cut into BATCHES of at most
// kBatch ratings, and every batch becomes a small program: the rows of P and Q it touches, and its ratings dealt to
// rounds in which several of them are worked on side by side.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <new>
#include <vector>

#include <rocprim/rocprim.hpp>

#include "common.h"
#include "freeride_device.h"
#include "sgd_rule.h"

namespace {

constexpr int kSgdBlock = 256;
constexpr uint32_t kBatch = kSgdBatch;
constexpr uint32_t kMaxRounds = 2 * kBatch;      // a rating is at most two rounds behind the last one before it
constexpr int kAhead = 2;                        // long cells: ratings whose rows are in flight ahead of the one being worked on (>= 2)
constexpr uint64_t kMostBytes = 128;              // per rating that the rounds' layout may take for good (see k_sgd_chain)
constexpr uint32_t kMaxBlocks = 1024;
constexpr int64_t kMaxIds = (1ll << 27) - 1024;
constexpr uint32_t kNoBatch = 0xffffffffu;
constexpr int kMaxLds = (kMaxRounds + 3) * 2 * 16 + (2 * kBatch + 1) * 256;      // of a batch of 64 factors: 74 KB

// A batch: a record of `stride` 16-byte words, the head and then the ids of its rows (users, then items with kItemRow set,
// then kNoRow), so that the rows can be asked for after one load; the rounds' entries are elsewhere, packed.
// Head: first entry (rounds | high bits << 16), rounds, the next batch of the same cell.
struct BatchHead { uint32_t first, rounds, rows, next; };     // rows = users | items << 16
static_assert(sizeof(BatchHead) == 16, "read as one 16-byte word");
constexpr uint32_t kItemRow = 0x80000000u, kNoRow = 0xffffffffu;

// What one slot does in one round: bits of the rating, byte offsets of the two rows in LDS (multiples of 64); the sign bit
// of an offset: the row is the one the slot has just updated, still in its registers.
struct SlotEntry { uint32_t rating, p, q, pad; };
static_assert(sizeof(SlotEntry) == 16, "read as one 16-byte word");

struct SgdArgs {
    const uint4* records;        // the first batch of cell s * B + a at that index, then the further batches of long cells
    const uint4* entries;
    float* P;
    float* Q;
    uint32_t layout;             // 16-byte words of a record | blocks << 16 (in a word of its own the launch's arguments would end in
                                 // another cache line, 0.2 us a launch)
    float gamma, gl;             // gl = gamma * lambda, rounded once
};

// (arguments of its own: in one struct with those above they lie behind a cache line's end, and a launch takes 0.15 us more)
struct ChainArgs {
    const uint64_t* keys;        // user << 32 | item and rating in the order of the cells, and the cells' starts
    const float* rating;
    const uint32_t* cell_ptr;
    float* P;
    float* Q;
    float gamma, gl;
};

struct GateArg {
    fr_gate* gate;
    uint32_t slot, need_ticks;
};

// Lanes that share a rating: F / lanes factors in each.
constexpr int lanes_for(int F) { return F == 64 ? 32 : 16; }

// The update of a rating, with every rounding fixed:
//     t_l = p_l * q_l;  in rounds w = 1, 2, 4, .., F/2: t_l = t_l + t_(l xor w)   (all end with the same sum)
//     e = r - t;  ge = gamma * e;  p_l' = fma(ge, q_l, fma(-gl, p_l, p_l));  q_l' = fma(ge, p_l, fma(-gl, q_l, q_l))
// (The product p_l * q_l has to be kept from being folded into the first addition of the tree as a fused
// multiply-add: the rounded-operation intrinsics are plain operators to the compiler, so the product passes
// through an empty asm statement, which hides where it came from.)
__device__ __forceinline__ float rounded_product(float x, float y)
{
    float t = x * y;
    asm("" : "+v"(t));
    return t;
}

// The tree sum over the lanes of a rating.  Inside a row of 16 lanes by DPP moves: quad permutations for lanes xor 1 and
// 2; for xor 4 and 8 the half-row and row mirrors, which pair every lane with a lane of the other half - not lane l xor 4
// itself, but by then all lanes of a quad (of a half-row) hold the same value, so the sums are the same numbers.  Two rows
// are joined by swapping the odd rows of one copy with the even rows of another.
template <int kCtrl>
__device__ __forceinline__ float add_dpp(float t)
{
    const int moved = __builtin_amdgcn_mov_dpp(__float_as_int(t), kCtrl, 0xf, 0xf, true);      // (every lane has a source lane: folds into the addition)
    return __fadd_rn(t, __int_as_float(moved));
}

template <int kLanes>
__device__ __forceinline__ float lane_sum(float t)
{
    t = add_dpp<0xB1>(t);        // quad_perm [1, 0, 3, 2]
    t = add_dpp<0x4E>(t);        // quad_perm [2, 3, 0, 1]
    t = add_dpp<0x141>(t);       // row_half_mirror
    t = add_dpp<0x140>(t);       // row_mirror
    if constexpr (kLanes == 32) {
        const auto rows = __builtin_amdgcn_permlane16_swap((unsigned)__float_as_int(t), (unsigned)__float_as_int(t), false, false);
        t = __fadd_rn(__int_as_float((int)rows[0]), __int_as_float((int)rows[1]));
    }
    return t;
}

// kN consecutive floats of a row in LDS
typedef __attribute__((address_space(3))) char* LdsBytes;
typedef uint32_t Entry3 __attribute__((ext_vector_type(3)));      // an entry's words in use
template <int kN> struct Piece { float v[kN]; };
template <int kN>
__device__ __forceinline__ Piece<kN> lds_read(LdsBytes at)
{
    typedef float Vec __attribute__((ext_vector_type(kN)));
    const Vec w = *reinterpret_cast<const __attribute__((address_space(3))) Vec*>(at);
    Piece<kN> x;
#pragma unroll
    for (int k = 0; k < kN; ++k) x.v[k] = w[k];
    return x;
}
template <int kN>
__device__ __forceinline__ void lds_write(LdsBytes at, const Piece<kN>& x)
{
    typedef float Vec __attribute__((ext_vector_type(kN)));
    Vec w;
#pragma unroll
    for (int k = 0; k < kN; ++k) w[k] = x.v[k];
    *reinterpret_cast<__attribute__((address_space(3))) Vec*>(at) = w;
}

// (rows of the caller's matrices are read and written 16 bytes at a time; their addresses are multiples of 4)
typedef float float4_any __attribute__((ext_vector_type(4), aligned(4)));

// One workgroup per cell.  Updates of one cell that share neither user nor item do not touch each other, and any order of
// updates that keeps the order of those that do gives the same bits; what is serial is only the longest chain of updates
// linked by a common user or item.  So a batch of the cell's ratings is worked on in rounds of 64 / lanes_for(F) ratings
// side by side in one wavefront, laid out once by k_sgd_schedule.  All four wavefronts bring the batch's rows to LDS, the
// first one works through the rounds, all four write the rows back.
// What bounds it: the longest chain of a stratum (16.1 M ratings, 512 x 512 cells, 64 factors: 85 updates, where its largest
// cell has 109 ratings and a mean cell 61), at 81 ns a round with 64 factors, 73 with 32, 55 with 16 (a cell that is one chain of
// n ratings takes 2.5 us + n rounds): one wavefront's instructions, some forty, and the latency of the sum's dependent moves.
// Hence 32 lanes with two factors each (90.7 rounds) and not 16 with four (87.5 rounds of half as many instructions again),
// rows fetched from LDS a round ahead, before the stores of the round that is being computed, and the row of a chain handed on
// in registers; and twelve rounds without a branch (six with 32 factors, where twelve are no better): at a loop's head the
// wavefront waits for everything it has asked the LDS for, which every third round took 102, 89 and 75 ns a round.  A stratum
// takes 13 us there, of which the rounds are some 7.5; the rest is fetching and storing 42 000 rows (21 MB) and the
// launch.  An iteration of 512 strata takes 6.5 to 7.3 ms (7.6 to 8.3 with branches between the rounds and nothing read ahead); one rating after
// the other straight from memory, as k_sgd_chain does it, it took 21.9 ms (16 factors, 300 000 ratings in 64 x 64 cells: 0.40, 0.45
// and 1.9 ms).
template <int F, int kLanes>
__device__ __forceinline__ void run_rounds(LdsBytes entries, uint32_t rounds, float gamma, float gl)
{
    constexpr int kN = F / kLanes, kSlots = 64 / kLanes;
    constexpr uint32_t kUnroll = F == 32 ? 6 : 12;
    const uint32_t lane = threadIdx.x & 63, at = (lane % kLanes) * (kN * 4);
    const LdsBytes mine = entries + (lane / kLanes) * sizeof(SlotEntry);
    struct Turn { float rating; uint32_t p, q; };         // p, q: as in the entry, and addresses once the rows are asked for
    auto turn = [&](uint32_t r) {
        const Entry3 w = *reinterpret_cast<const __attribute__((address_space(3))) Entry3*>(mine + r * (kSlots * sizeof(SlotEntry)));
        return Turn{__uint_as_float(w.x), w.y, w.z};
    };
    auto address = [&](uint32_t offset) { return (offset & 0x7fffffc0u) | at; };
    auto row = [&](uint32_t address) { return reinterpret_cast<LdsBytes>(address); };
    Turn A = turn(0), B = turn(1), C = turn(2);
    A.p = address(A.p); A.q = address(A.q);
    Piece<kN> p = lds_read<kN>(row(A.p)), q = lds_read<kN>(row(A.q));
    // one round: `now` with p and q in hand, the rows of `next` asked for; then the entry of three rounds on
    auto step = [&](Turn& now, Turn& next, uint32_t r) {
        const bool keep_p = (int32_t)next.p < 0, keep_q = (int32_t)next.q < 0;
        next.p = address(next.p); next.q = address(next.q);
        const Piece<kN> pn = lds_read<kN>(row(next.p)), qn = lds_read<kN>(row(next.q));
        float t[kN];
#pragma unroll
        for (int k = 0; k < kN; ++k) t[k] = rounded_product(p.v[k], q.v[k]);
#pragma unroll
        for (int w = 1; w < kN; w <<= 1)
#pragma unroll
            for (int k = 0; k + w < kN; k += 2 * w) t[k] = __fadd_rn(t[k], t[k + w]);
        const float dot = lane_sum<kLanes>(t[0]);
        const float ge = __fmul_rn(gamma, __fsub_rn(now.rating, dot));
        Piece<kN> p2, q2;
#pragma unroll
        for (int k = 0; k < kN; ++k) {
            p2.v[k] = __fmaf_rn(ge, q.v[k], __fmaf_rn(-gl, p.v[k], p.v[k]));
            q2.v[k] = __fmaf_rn(ge, p.v[k], __fmaf_rn(-gl, q.v[k], q.v[k]));
        }
        lds_write<kN>(row(now.p), p2);
        lds_write<kN>(row(now.q), q2);
        now = turn(r + 3);
#pragma unroll
        for (int k = 0; k < kN; ++k) {
            p.v[k] = keep_p ? p2.v[k] : pn.v[k];
            q.v[k] = keep_q ? q2.v[k] : qn.v[k];
        }
    };
    // (three more entries are there to be read)
    uint32_t r = 0;
    for (; r + kUnroll <= rounds; r += kUnroll) {         // one basic block: at a loop's head the wavefront waits for all of the LDS
#pragma unroll
        for (uint32_t k = 0; k < kUnroll; k += 3) {
            step(A, B, r + k);
            step(B, C, r + k + 1);
            step(C, A, r + k + 2);
        }
    }
    while (r < rounds) {
        step(A, B, r);
        if (++r == rounds) break;
        step(B, C, r);
        if (++r == rounds) break;
        step(C, A, r);
        ++r;
    }
}

// kAhead: the next stratum's programs are read ahead (a kernel of its own: its registers, 64 -> 72 with 16 factors, cost 10 to 19 %
// where eight small cells share a unit).  kCells: workgroups that are to fit on a unit.  With 16 factors eight have 64 registers
// a lane, two fewer than the rounds take without waits between their dependent moves (a wait a round, 1.8 % of an iteration of 20 011 x
// 5003 ids and 300 000 ratings), seven have 72; with 32 and 64 factors the rounds take more than either.
template <int F, bool kAhead, int kCells>
__global__ __launch_bounds__(kSgdBlock) __attribute__((amdgpu_waves_per_eu(1, kCells))) void k_sgd(SgdArgs A, GateArg G, uint32_t cell0)
{
    // the rows begin at LDS address 0 (the kernel has no other LDS): an entry's offset is an address
    extern __shared__ __align__(16) char lds[];
    if (!fr_gate_admit(G.gate, G.slot, G.need_ticks)) return;
    constexpr uint32_t kSlots = 64 / lanes_for(F), kWords = F / 4;      // 16-byte words of a row
    constexpr int kDepth = F / 8 + 2;                                   // words in flight per thread: 160 rows or more at once
    const uint32_t stride = A.layout & 0xffffu, blocks = A.layout >> 16;
    uint32_t b = cell0 + blockIdx.x;
    do {
        const uint4* record = A.records + (uint64_t)b * stride;
        const uint32_t* ids = reinterpret_cast<const uint32_t*>(record + 1);
        const uint4 head = record[0];
        const uint32_t most = (stride - 1) * 4 * kWords;              // words of the rows there can be
        uint32_t id[kDepth];
        auto ask_ids = [&](uint32_t i0) {
#pragma unroll
            for (int k = 0; k < kDepth; ++k) {
                const uint32_t i = i0 + k * kSgdBlock;
                id[k] = i < most ? ids[i / kWords] : kNoRow;
            }
        };
        auto global_row = [&](uint32_t x) { return (x & kItemRow ? A.Q : A.P) + (size_t)(x & ~kItemRow) * F; };
        ask_ids(threadIdx.x);
        const BatchHead H{head.x, head.y & 0xffffu, head.z, head.w};
        const uint64_t first = (uint64_t)(head.y >> 16) << 32 | head.x;
        const uint32_t n_rows = (H.rows & 0xffffu) + (H.rows >> 16), n_words = n_rows * kWords;
        const uint32_t n_entries = H.rounds ? (H.rounds + 3) * kSlots : 0;
        float4* rows = reinterpret_cast<float4*>(lds);                  // the rows, one for idle slots, the entries
        uint4* entries = reinterpret_cast<uint4*>(lds + (n_rows + 1) * (F * 4));
        for (uint32_t i0 = threadIdx.x;;) {
            float4_any v[kDepth];
#pragma unroll
            for (int k = 0; k < kDepth; ++k)
                if (id[k] != kNoRow) v[k] = *reinterpret_cast<const float4_any*>(global_row(id[k]) + ((i0 + k * kSgdBlock) % kWords) * 4);
            if (i0 < kSgdBlock)
                for (uint32_t i = threadIdx.x; i < n_entries; i += kSgdBlock) entries[i] = A.entries[first + i];
#pragma unroll
            for (int k = 0; k < kDepth; ++k)
                if (id[k] != kNoRow) rows[i0 + k * kSgdBlock] = make_float4(v[k].x, v[k].y, v[k].z, v[k].w);
            i0 += kDepth * kSgdBlock;
            if (i0 - threadIdx.x >= n_words) break;
            ask_ids(i0);
        }
        __syncthreads();
        if (threadIdx.x < 64) {
            if (H.rounds) {                                             // (a cell without ratings has no entries to read)
                const LdsBytes at = reinterpret_cast<LdsBytes>((uint32_t)((n_rows + 1) * (F * 4)));
                run_rounds<F, lanes_for(F)>(at, H.rounds, A.gamma, A.gl);
            }
        } else if (kAhead && b < blocks * blocks) {                     // (not for a cell's further batches)
            // meanwhile the other wavefronts read what the next stratum's cell of this user block begins with - its record, its
            // entries and its rows of P, which no other workgroup writes - so that the launch of that stratum finds them in the
            // L2 (whole strata: the workgroup of this number runs on the same compute die again) or in the cache behind it.
            // Where it pays: sgd_reads_ahead.
            const uint32_t after = b + blocks < blocks * blocks ? b + blocks : b + blocks - blocks * blocks;
            const uint4* soon = A.records + (uint64_t)after * stride;
            const uint32_t* soon_ids = reinterpret_cast<const uint32_t*>(soon + 1);
            const uint4 soon_head = soon[0];
            const uint32_t rounds = soon_head.y & 0xffffu, entry_words = rounds ? (rounds + 3) * kSlots : 0, words = (soon_head.z & 0xffffu) * kWords;
            const uint64_t entry0 = (uint64_t)(soon_head.y >> 16) << 32 | soon_head.x;
            uint32_t read = 0;
            for (uint32_t i = threadIdx.x - 64; i < stride; i += kSgdBlock - 64) read ^= soon[i].x;
            for (uint32_t i = threadIdx.x - 64; i < entry_words; i += kSgdBlock - 64) read ^= A.entries[entry0 + i].x;
            for (uint32_t i = threadIdx.x - 64; i < words; i += kSgdBlock - 64) {
                const uint32_t id = soon_ids[i / kWords];
                if (!(id & kItemRow)) read ^= __float_as_uint(A.P[(size_t)id * F + (i % kWords) * 4]);
            }
            asm volatile("" :: "v"(read));                              // (the values are of no use, but the loads are to be made)
        }
        __syncthreads();
        for (uint32_t i0 = threadIdx.x; i0 < n_words; i0 += kDepth * kSgdBlock) {
            if (n_words > kDepth * kSgdBlock) ask_ids(i0);              // (else they are still here)
#pragma unroll
            for (int k = 0; k < kDepth; ++k) {
                const uint32_t i = i0 + k * kSgdBlock;
                if (id[k] == kNoRow) continue;
                const float4 x = rows[i];
                float4_any y;
                y.x = x.x; y.y = x.y; y.z = x.z; y.w = x.w;
                *reinterpret_cast<float4_any*>(global_row(id[k]) + (i % kWords) * 4) = y;
            }
        }
        b = H.next;
        if (b != kNoBatch) __syncthreads();                             // the next batch may read what this one wrote
    } while (b != kNoBatch);
    fr_gate_done(G.gate, G.slot);
}

// Cells of more than kSgdLongCell ratings on average - a caller that asks for fewer blocks than the library would make, or more
// than 2^28 ratings -, cells of a few ratings and many cells on few compute units (sgd_rounds_pay), cells whose layout in rounds
// would take more than kMostBytes per rating, and tasks whose limit has no room for that layout are worked on by a group of F lanes per cell, lane l holding dimension l, its ratings one after the
// other, straight from the matrices.  (12 bytes per rating where the rounds' layout takes 29 on the benchmark's ratings: memory
// is what a side task is given least of.  A batch's record has the stride of the batch with most rows, so many cells with few
// ratings and one with 128 in 256 rows cost 1040 bytes each: 1024 x 1024 cells of a million ratings 750 MB.  The blocks the
// library makes by itself leave 25 to 50 bytes per rating.  It is the slower of the two: 0.23 us per rating of a cell where a batch of 128 takes
// some 10 us in rounds.)  What a rating costs is the latency of fetching its rows.  The loop therefore looks two ratings
// ahead (and three for the keys): while rating x - 2 is being worked
// on, the rows of rating x are requested, unless they are held in registers by then (same user / same item as
// rating x - 1) or could still be written before they are used: q of rating x may be requested early only if its
// item differs from those of ratings x - 2 and x - 1; if it is the item of rating x - 2, the request waits until
// that rating's row has been stored (a wavefront's own store and later load of one address stay in order).  Users
// ascend inside a cell, so a row of P asked for early is never written in between.
// The sum over F lanes: rows of 16 as in lane_sum; rows are joined through readlane: row sums R_0 .. R_3, (R_0 + R_1) and
// (R_2 + R_3), then their sum - the same tree.  (readlane ignores the execution mask; a group only uses its own
// rows, whose lanes are all active together.)
template <int F>
__device__ __forceinline__ float chain_sum(float t)
{
    t = lane_sum<16>(t);
    if constexpr (F == 16) return t;
    const float r0 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(t), 0));
    const float r1 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(t), 16));
    const float r2 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(t), 32));
    const float r3 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(t), 48));
    const float lo = __fadd_rn(r0, r1), hi = __fadd_rn(r2, r3);
    if constexpr (F == 32) return (threadIdx.x & 32) ? hi : lo;
    return __fadd_rn(lo, hi);
}

template <int F>
__global__ __launch_bounds__(kSgdBlock) void k_sgd_chain(ChainArgs A, GateArg G, uint32_t cell0, uint32_t n_cells)
{
    if (!fr_gate_admit(G.gate, G.slot, G.need_ticks)) return;
    const uint32_t g = (blockIdx.x * kSgdBlock + threadIdx.x) / F, l = threadIdx.x % F;
    if (g < n_cells) {
        uint32_t e = A.cell_ptr[cell0 + g];
        const uint32_t e1 = A.cell_ptr[cell0 + g + 1];
        if (e < e1) {
            const float* __restrict__ rating = A.rating;
            const uint64_t* __restrict__ keys = A.keys;
            // Slot k holds rating e + k: slot 0 is being worked on, the rows of slots 1 .. kAhead have been asked
            // for, slot kAhead + 1 holds a key only.  Every iteration issues the same loads and stores whether
            // their values are needed or not (behind the cell's end: those of its last rating again), so that the
            // compiler can count what is in flight and waits only for the oldest request, not for all of them.
            uint32_t us[kAhead + 2], is[kAhead + 2];
            float rs[kAhead + 2], ps[kAhead + 1], qs[kAhead + 1];
            bool late[kAhead + 1] = {};
#pragma unroll
            for (int k = 0; k < kAhead + 2; ++k) {
                const uint32_t ek = e + k < e1 ? e + k : e1 - 1;
                const uint64_t key = keys[ek];
                us[k] = (uint32_t)(key >> 32); is[k] = (uint32_t)key; rs[k] = rating[ek];
            }
#pragma unroll
            for (int k = 0; k < kAhead; ++k) {
                ps[k] = A.P[(size_t)us[k] * F + l];
                qs[k] = A.Q[(size_t)is[k] * F + l];
                bool clash = false;
#pragma unroll
                for (int j = 0; j + 1 < k; ++j) clash |= is[k] == is[j];
                late[k] = k >= 2 && is[k] != is[k - 1] && clash;
            }
            for (;;) {
                // the rows of slot kAhead.  q may be used as it arrives if no rating before it in flight writes it:
                // not the one just before it (then the registers are handed on) and none of the others (then the
                // row is asked for again once they have stored theirs: late)
                ps[kAhead] = A.P[(size_t)us[kAhead] * F + l];
                qs[kAhead] = A.Q[(size_t)is[kAhead] * F + l];
                {
                    bool clash = false;
#pragma unroll
                    for (int j = 0; j + 1 < kAhead; ++j) clash |= is[kAhead] == is[j];
                    late[kAhead] = is[kAhead] != is[kAhead - 1] && clash;
                }
                const uint32_t en = e + kAhead + 2 < e1 ? e + kAhead + 2 : e1 - 1;
                const uint64_t keyn = keys[en];
                const float rn = rating[en];
                const float p = ps[0], q = qs[0];
                const float t = chain_sum<F>(rounded_product(p, q));
                const float ge = __fmul_rn(A.gamma, __fsub_rn(rs[0], t));
                const float p2 = __fmaf_rn(ge, q, __fmaf_rn(-A.gl, p, p));
                const float q2 = __fmaf_rn(ge, p, __fmaf_rn(-A.gl, q, q));
                A.P[(size_t)us[0] * F + l] = p2;
                A.Q[(size_t)is[0] * F + l] = q2;
                if (e + 1 >= e1) break;
                if (us[1] == us[0]) ps[1] = p2;          // the same user / item again: its row is in registers
                if (is[1] == is[0]) qs[1] = q2;
                // every rating before slot 1 has stored its row by now: a late row can be asked for
                const float again = A.Q[(size_t)is[2] * F + l];
                if (late[2]) qs[2] = again;
#pragma unroll
                for (int k = 0; k < kAhead; ++k) { ps[k] = ps[k + 1]; qs[k] = qs[k + 1]; }
#pragma unroll
                for (int k = 1; k < kAhead; ++k) late[k] = k == 1 ? false : late[k + 1];
#pragma unroll
                for (int k = 0; k < kAhead + 1; ++k) { us[k] = us[k + 1]; is[k] = is[k + 1]; rs[k] = rs[k + 1]; }
                us[kAhead + 1] = (uint32_t)(keyn >> 32); is[kAhead + 1] = (uint32_t)keyn; rs[kAhead + 1] = rn;
                ++e;
            }
        }
    }
    fr_gate_done(G.gate, G.slot);
}

// ---- set-up kernels ----
__global__ void k_sgd_set(int32_t* p, int32_t v) { *p = v; }

__global__ __launch_bounds__(256) void k_sgd_validate(int64_t U, int64_t I, int64_t E, const int32_t* __restrict__ row_ptr,
                                                      const int32_t* __restrict__ item, int32_t* bad)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; u <= U; u += stride) {
        const int32_t a = row_ptr[u];
        if (a < 0 || a > E || (u == 0 && a != 0) || (u == U && a != E) || (u < U && row_ptr[u + 1] < a)) *bad = 1;
    }
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < E; e += stride)
        if (item[e] < 0 || item[e] >= I) *bad = 1;
}

// The block of id x: the last k below B with starts[k] <= x (empty blocks share their start with the next one).
__device__ __forceinline__ uint32_t block_of(const uint32_t* __restrict__ starts, uint32_t B, uint32_t x)
{
    uint32_t lo = 0, hi = B - 1;
    while (lo < hi) {
        const uint32_t mid = (lo + hi + 1) / 2;
        if (starts[mid] <= x) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

__global__ __launch_bounds__(256) void k_sgd_zero(uint32_t* p, uint64_t n)
{
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0u;
}

__global__ __launch_bounds__(256) void k_sgd_count_items(int64_t E, const int32_t* __restrict__ item, uint32_t* count)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e < E) atomicAdd(&count[item[e]], 1u);
}

// starts[k], k = 0 .. B: block k begins at the first id x with before[x] >= ceil(k E / B); before[x] = ratings of the
// ids below x (n + 1 entries, int32 or uint32: the values are below 2^31 either way).
__global__ __launch_bounds__(256) void k_sgd_starts(uint32_t n, const uint32_t* __restrict__ before, int64_t E, uint32_t B,
                                                    uint32_t* __restrict__ starts)
{
    const uint32_t k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k > B) return;
    if (k == 0 || k == B) { starts[k] = k == 0 ? 0u : n; return; }
    const uint64_t want = ((uint64_t)k * (uint64_t)E + B - 1) / B;
    uint32_t lo = 0, hi = n;                    // first x with before[x] >= want (before[n] = E >= want)
    while (lo < hi) {
        const uint32_t mid = lo + (hi - lo) / 2;
        if ((uint64_t)before[mid] < want) lo = mid + 1;
        else hi = mid;
    }
    starts[k] = lo;
}

// cell and user of rating e; the user is found by bisection of row_ptr.  Also checks that items ascend inside a row.
__global__ __launch_bounds__(256) void k_sgd_keys(int64_t U, int64_t E, const int32_t* __restrict__ row_ptr,
                                                  const int32_t* __restrict__ item, uint32_t B,
                                                  const uint32_t* __restrict__ ustart, const uint32_t* __restrict__ istart,
                                                  uint32_t* __restrict__ cell, uint32_t* __restrict__ index, uint32_t* __restrict__ user,
                                                  int32_t* bad)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= E) return;
    int64_t lo = 0, hi = U;                     // the last u with row_ptr[u] <= e
    while (hi - lo > 1) {
        const int64_t mid = (lo + hi) / 2;
        if (row_ptr[mid] <= e) lo = mid;
        else hi = mid;
    }
    const uint32_t u = (uint32_t)lo, i = (uint32_t)item[e];
    if (e > row_ptr[u] && item[e - 1] >= item[e]) *bad = 1;
    const uint32_t a = block_of(ustart, B, u), b = block_of(istart, B, i);
    const uint32_t s = (b + B - a) % B;
    cell[e] = s * B + a;
    index[e] = (uint32_t)e;
    user[e] = u;
}

__global__ __launch_bounds__(256) void k_sgd_cells(int64_t E, uint32_t B, const uint32_t* __restrict__ cell, uint32_t* __restrict__ cell_ptr)
{
    const uint32_t c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c > B * B) return;
    int64_t lo = 0, hi = E;                     // first rating whose cell is c or a later one
    while (lo < hi) {
        const int64_t mid = (lo + hi) / 2;
        if (cell[mid] < c) lo = mid + 1;
        else hi = mid;
    }
    cell_ptr[c] = (uint32_t)lo;
}

// long cells: key and rating of every place in the order of the cells
__global__ __launch_bounds__(256) void k_sgd_stream(int64_t E, const uint32_t* __restrict__ index, const uint32_t* __restrict__ user,
                                                    const int32_t* __restrict__ item, const float* __restrict__ rating,
                                                    uint64_t* __restrict__ keys, float* __restrict__ sorted)
{
    const int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (x >= E) return;
    const uint32_t e = index[x];
    keys[x] = (uint64_t)user[e] << 32 | (uint32_t)item[e];
    sorted[x] = rating[e];
}

// A batch of a cell beyond its first: the cell and the batch's first rating.
struct MoreBatch { uint32_t cell, first; };

struct BatchSpan { uint32_t first, n, next; };

// Ratings of batch b: the first kBatch of cell b, or for b >= B * B those of more[b - B * B]; and the cell's next batch.
__device__ __forceinline__ BatchSpan span_of(uint32_t b, uint32_t n_cells, const uint32_t* __restrict__ cell_ptr,
                                             const MoreBatch* __restrict__ more, uint32_t n_more)
{
    uint32_t cell = b, k = 0;                   // k: the first entry of `more` behind this batch
    BatchSpan S;
    if (b < n_cells) {
        S.first = cell_ptr[b];
        uint32_t lo = 0, hi = n_more;
        while (lo < hi) {
            const uint32_t mid = (lo + hi) / 2;
            if (more[mid].cell < b) lo = mid + 1;
            else hi = mid;
        }
        k = lo;
    } else {
        k = b - n_cells;
        cell = more[k].cell;
        S.first = more[k].first;
        ++k;
    }
    const uint32_t left = cell_ptr[cell + 1] - S.first;
    S.n = left < kBatch ? left : kBatch;
    S.next = k < n_more && more[k].cell == cell ? n_cells + k : kNoBatch;
    return S;
}

// The place of a rating in its batch: row of its user and of its item (among the batch's users and items), slot and
// round (round * slots + slot), and whether a row is handed on in registers.
constexpr uint32_t kPlaceItem = 7, kPlacePos = 14, kPlaceKeepP = 30, kPlaceKeepQ = 31;
static_assert(kBatch <= 128 && kMaxRounds * 4 <= 65536, "fields of a place");

// One wavefront per batch lays its ratings out in rounds: in their order, each in the first round that leaves the
// results as they are.  While a round is computed the rows of the next one have already been read, so a rating has to
// be two rounds behind the ratings before it that share its user or its item - or one round behind the later of
// the two in that one's slot, where the row is still in registers.  (With a look at which ratings have the longest chains
// behind them a mean batch takes 10 % fewer rounds and the longest ones, which set a stratum's time, 2 %.)
__global__ __launch_bounds__(64) void k_sgd_schedule(uint32_t n_cells, uint32_t n_more, uint32_t slots, const uint32_t* __restrict__ cell_ptr,
                                                     const MoreBatch* __restrict__ more, const uint32_t* __restrict__ index,
                                                     const uint32_t* __restrict__ user, const int32_t* __restrict__ item,
                                                     uint32_t* __restrict__ place, uint64_t* __restrict__ size, uint4* __restrict__ heads)
{
    __shared__ int32_t us[kBatch], is[kBatch];
    __shared__ int16_t before_item[kBatch], round_of[kBatch];
    __shared__ uint8_t slot_of[kBatch];
    __shared__ uint32_t taken[kMaxRounds + 64];           // bit s: slot s of the round is taken
    const uint32_t b = blockIdx.x, lane = threadIdx.x;
    const BatchSpan S = span_of(b, n_cells, cell_ptr, more, n_more);
    constexpr int kPer = kBatch / 64;
    for (uint32_t r = lane; r < kMaxRounds + 64; r += 64) taken[r] = 0u;
    for (int k = 0; k < kPer; ++k) {
        const uint32_t x = lane + 64 * k;
        if (x < S.n) {
            const uint32_t e = index[S.first + x];
            us[x] = (int32_t)user[e]; is[x] = item[e];
        }
    }
    __syncthreads();
    // rows: users ascend, so a new one begins where it differs from the one before; items in order of first appearance
    uint32_t urow[kPer], irow[kPer];
    int32_t first_same[kPer], last_same[kPer];
    uint32_t n_users = 0, n_items = 0;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const uint32_t x = lane + 64 * k;
        first_same[k] = last_same[k] = -1;
        const bool fresh = x < S.n && (x == 0 || us[x] != us[x - 1]);
        const uint64_t m = __ballot(fresh);
        urow[k] = n_users + __popcll(m & (~0ull >> (63 - lane))) - 1u;
        n_users += __popcll(m);
    }
    for (uint32_t y = 0; y < S.n; ++y) {
        const int32_t iy = is[y];
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const uint32_t x = lane + 64 * k;
            if (x < S.n && y < x && is[x] == iy) {
                last_same[k] = (int32_t)y;
                if (first_same[k] < 0) first_same[k] = (int32_t)y;
            }
        }
    }
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const uint32_t x = lane + 64 * k;
        const uint64_t m = __ballot(x < S.n && first_same[k] < 0);
        irow[k] = n_items + __popcll(m & (~0ull >> (63 - lane))) - 1u;
        n_items += __popcll(m);
        if (x < S.n) {
            before_item[x] = (int16_t)last_same[k];
            round_of[x] = (int16_t)irow[k];               // (for the moment: the row of an item's first rating)
        }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kPer; ++k)
        if (lane + 64 * k < S.n && first_same[k] >= 0) irow[k] = (uint32_t)round_of[first_same[k]];
    __syncthreads();
    const uint32_t all = (1u << slots) - 1u;
    uint32_t rounds = 0;
    for (uint32_t x = 0; x < S.n; ++x) {                  // (the same in all lanes)
        const int32_t pu = x > 0 && us[x] == us[x - 1] ? (int32_t)x - 1 : -1, pi = before_item[x];
        const int32_t ru = pu >= 0 ? round_of[pu] : -2, ri = pi >= 0 ? round_of[pi] : -2;
        const int32_t late = ru > ri ? ru : ri, early = ru > ri ? ri : ru;
        uint32_t round = 0, slot = 0;
        bool placed = false;
        if (late >= 0 && early < late) {
            slot = slot_of[ru > ri ? pu : pi];
            round = (uint32_t)late + 1;
            placed = !((taken[round] >> slot) & 1u);
        }
        for (uint32_t r0 = (uint32_t)(late + 2); !placed; r0 += 64) {      // (a round no rating is in yet comes within 64 of kMaxRounds)
            const uint64_t room = __ballot(taken[r0 + lane < kMaxRounds + 64 ? r0 + lane : kMaxRounds + 63] != all);
            if (!room) continue;
            round = r0 + (uint32_t)__ffsll((unsigned long long)room) - 1u;
            slot = (uint32_t)__ffs((int)~taken[round]) - 1u;
            placed = true;
        }
        __syncthreads();
        if (lane == 0) {
            taken[round] |= 1u << slot;
            round_of[x] = (int16_t)round;
            slot_of[x] = (uint8_t)slot;
        }
        if (round + 1 > rounds) rounds = round + 1;
        __syncthreads();
    }
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const uint32_t x = lane + 64 * k;
        if (x >= S.n) continue;
        const int32_t r = round_of[x], pi = last_same[k];
        const uint32_t keep_p = x > 0 && us[x] == us[x - 1] && round_of[x - 1] == r - 1 ? 1u : 0u;
        const uint32_t keep_q = pi >= 0 && round_of[pi] == r - 1 ? 1u : 0u;
        place[S.first + x] = urow[k] | irow[k] << kPlaceItem | ((uint32_t)r * slots + slot_of[x]) << kPlacePos | keep_p << kPlaceKeepP | keep_q << kPlaceKeepQ;
    }
    if (lane == 0) {
        heads[b] = make_uint4(0u, rounds, n_users | n_items << 16, S.next);
        size[b] = rounds ? (rounds + 3) * slots : 0u;
    }
}

// Writes a batch's record and its entries (`before`: entries of the batches before it).  Slots without a rating work on a
// row of their own behind the batch's rows, which nobody reads.
__global__ __launch_bounds__(64) void k_sgd_program(uint32_t n_cells, uint32_t n_more, uint32_t slots, uint32_t row_bytes, uint32_t stride,
                                                    const uint32_t* __restrict__ cell_ptr, const MoreBatch* __restrict__ more,
                                                    const uint32_t* __restrict__ index, const uint32_t* __restrict__ user,
                                                    const int32_t* __restrict__ item, const float* __restrict__ rating,
                                                    const uint32_t* __restrict__ place, const uint64_t* __restrict__ before,
                                                    const uint4* __restrict__ heads, uint4* __restrict__ records, uint4* __restrict__ all_entries)
{
    const uint32_t b = blockIdx.x, lane = threadIdx.x;
    const BatchSpan S = span_of(b, n_cells, cell_ptr, more, n_more);
    const uint4 H = heads[b];
    const uint32_t users = H.z & 0xffffu, n_rows = users + (H.z >> 16), n_entries = H.y ? (H.y + 3) * slots : 0u;
    const uint64_t at = before[b];
    uint4* entries = all_entries + at;
    uint32_t* ids = reinterpret_cast<uint32_t*>(records + (uint64_t)b * stride + 1);
    for (uint32_t i = n_rows + lane; i < (stride - 1) * 4; i += 64) ids[i] = kNoRow;
    for (uint32_t i = lane; i < n_entries; i += 64) entries[i] = make_uint4(0u, n_rows * row_bytes, n_rows * row_bytes, 0u);
    __syncthreads();
    for (uint32_t x = lane; x < S.n; x += 64) {
        const uint32_t e = index[S.first + x], w = place[S.first + x];
        const uint32_t ul = w & 127u, il = (w >> kPlaceItem) & 127u, pos = (w >> kPlacePos) & 0xffffu;
        entries[pos] = make_uint4(__float_as_uint(rating[e]), ul * row_bytes | ((w >> kPlaceKeepP) & 1u) << 31,
                                  (users + il) * row_bytes | (w >> kPlaceKeepQ) << 31, 0u);
        ids[ul] = user[e];                                // (every rating of a row writes the same id)
        ids[users + il] = (uint32_t)item[e] | kItemRow;
    }
    if (lane == 0) records[(uint64_t)b * stride] = make_uint4((uint32_t)at, H.y | (uint32_t)(at >> 32) << 16, H.z, H.w);
}

uint64_t ceil_fs_to_ns(unsigned __int128 fs)
{
    const uint64_t ns = (uint64_t)((fs + 999999) / 1000000);
    return ns ? ns : 1;
}

struct SgdTask {
    fr_sgd_desc d{};
    uint32_t B = 0;
    uint32_t *ustart = nullptr, *istart = nullptr;      // device, B + 1 entries each
    std::vector<uint32_t> ustart_host, istart_host;
    std::vector<uint32_t> cells;          // first rating of cell s * B + a, in the order of the cells; B * B + 1 entries
    uint32_t lds_bytes = 0;               // LDS of a workgroup: the largest batch's entries and rows
    std::vector<uint64_t> prefix;         // cumulative modelled cost of the cells, in the order of cell_ptr
    uint32_t max_cell = 0;
    uint64_t chain_ratings = 0;           // sum over the strata of their largest cell
    uint64_t footprint_after = 0, footprint_peak = 0;
    SgdArgs args{};
    ChainArgs chain{};                    // keys: NULL if the ratings are worked on in rounds
    uint32_t cus = 1;                     // compute units of the stream the task was set up on
    bool inited = false, registered = false;
    fr_alloc own;                         // used by the standalone run only
    int hip_error = 0;
    uint32_t run = 0, seg = 0, tile = 0;  // cursor

    uint32_t n_segments() const { return (uint32_t)d.iterations * B; }
};

int sgd_launch(SgdTask* p, uint32_t seg, uint32_t tile0, uint32_t tile1, hipStream_t stream, GateArg G = GateArg{nullptr, 0, 0})
{
    if (tile1 <= tile0 || tile1 > p->B || seg >= p->n_segments()) return FR_ERR_ARG;
    const uint32_t s = seg % p->B, n = tile1 - tile0, cell0 = s * p->B + tile0;
    const int F = p->d.factors;
    const bool reads_ahead = sgd_reads_ahead((uint64_t)p->d.n_ratings, p->B, n, p->cus);
    auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3(n), dim3(kSgdBlock), p->lds_bytes, stream, p->args, G, cell0); };
    auto go_chain = [&](auto kernel) {
        const unsigned grid = (unsigned)(((uint64_t)n * F + kSgdBlock - 1) / kSgdBlock);
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(kSgdBlock), 0, stream, p->chain, G, cell0, n);
    };
    if (p->chain.keys) {
        if (F == 64) go_chain(k_sgd_chain<64>);
        else if (F == 32) go_chain(k_sgd_chain<32>);
        else go_chain(k_sgd_chain<16>);
    } else if (F == 64) go(reads_ahead ? k_sgd<64, true, 8> : k_sgd<64, false, 8>);
    else if (F == 32) go(reads_ahead ? k_sgd<32, true, 8> : k_sgd<32, false, 8>);
    else if (sgd_eight_cells_a_unit(n, p->cus)) go(k_sgd<16, false, 8>);           // (too many to read ahead)
    else go(reads_ahead ? k_sgd<16, true, 7> : k_sgd<16, false, 7>);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) { p->hip_error = (int)e; return FR_ERR_HIP; }
    return FR_OK;
}

#define SGD_HIP(expr) do { hipError_t e__ = (expr); if (e__ != hipSuccess) { p->hip_error = (int)e__; return FR_ERR_HIP; } } while (0)
#define SGD_NEED(ptr) do { if (!(ptr)) return a->hip_error ? FR_ERR_HIP : FR_ERR_OOM; } while (0)

// The cells' programs: laid out once to learn their sizes, then written.  FR_ERR_OOM also where they take more than kMostBytes
// per rating.
int sgd_lay_out_rounds(SgdTask* p, fr_alloc* a, hipStream_t stream, const uint32_t* cell_ptr, const uint32_t* index, const uint32_t* user_of)
{
    const uint64_t n = (uint64_t)std::max<int64_t>(1, p->d.n_ratings);
    const uint32_t n_cells = p->B * p->B;
    const int F = p->d.factors;
    std::vector<MoreBatch> more;
    std::vector<uint4> heads_host;
    struct Wait { hipStream_t stream; ~Wait() { (void)hipStreamSynchronize(stream); } } wait{stream};      // (an early return may leave work)
    for (uint32_t c = 0; c < n_cells; ++c) {
        if (p->cells[c + 1] < p->cells[c]) return FR_ERR_ARG;
        for (uint32_t e = p->cells[c]; p->cells[c + 1] - e > kBatch;) {
            e += kBatch;
            more.push_back(MoreBatch{c, e});
        }
    }
    const uint32_t n_more = (uint32_t)more.size(), n_batches = n_cells + n_more;
    const uint32_t slots = 64u / (uint32_t)lanes_for(F), row_bytes = (uint32_t)F * 4;
    uint4* heads = static_cast<uint4*>(fr_alloc_device(a, (uint64_t)n_batches * sizeof(uint4)));
    MoreBatch* more_dev = static_cast<MoreBatch*>(fr_alloc_device(a, std::max<uint64_t>(1, n_more) * sizeof(MoreBatch)));
    uint32_t* place = static_cast<uint32_t*>(fr_alloc_device(a, n * 4));
    uint64_t* size = static_cast<uint64_t*>(fr_alloc_device(a, ((uint64_t)n_batches + 1) * 8));
    uint64_t* before = static_cast<uint64_t*>(fr_alloc_device(a, ((uint64_t)n_batches + 1) * 8));
    SGD_NEED(heads); SGD_NEED(more_dev); SGD_NEED(place); SGD_NEED(size); SGD_NEED(before);
    if (n_more) SGD_HIP(hipMemcpyAsync(more_dev, more.data(), (size_t)n_more * sizeof(MoreBatch), hipMemcpyHostToDevice, stream));
    hipLaunchKernelGGL(k_sgd_zero, dim3(1), dim3(256), 0, stream, reinterpret_cast<uint32_t*>(size + n_batches), (uint64_t)2);
    hipLaunchKernelGGL(k_sgd_schedule, dim3(n_batches), dim3(64), 0, stream, n_cells, n_more, slots, cell_ptr, more_dev, index, user_of,
                       p->d.item, place, size, heads);
    {
        size_t bytes = 0;
        SGD_HIP(rocprim::exclusive_scan(nullptr, bytes, size, before, (uint64_t)0, (size_t)n_batches + 1, rocprim::plus<uint64_t>(), stream));
        void* tmp = fr_alloc_device(a, bytes ? bytes : 1);
        SGD_NEED(tmp);
        SGD_HIP(rocprim::exclusive_scan(tmp, bytes, size, before, (uint64_t)0, (size_t)n_batches + 1, rocprim::plus<uint64_t>(), stream));
        SGD_HIP(hipStreamSynchronize(stream));
        (void)fr_alloc_free(a, tmp);
    }
    uint64_t total = 0;
    heads_host.resize(n_batches);
    SGD_HIP(hipMemcpyAsync(&total, before + n_batches, 8, hipMemcpyDeviceToHost, stream));
    SGD_HIP(hipMemcpyAsync(heads_host.data(), heads, (size_t)n_batches * sizeof(uint4), hipMemcpyDeviceToHost, stream));
    SGD_HIP(hipStreamSynchronize(stream));
    p->lds_bytes = 0;
    uint32_t most_rows = 1;
    for (const uint4& h : heads_host) {
        const uint32_t rows = (h.z & 0xffffu) + (h.z >> 16);
        most_rows = std::max(most_rows, rows);
        if (h.y) p->lds_bytes = std::max<uint32_t>(p->lds_bytes, (h.y + 3) * slots * (uint32_t)sizeof(SlotEntry) + (rows + 1) * row_bytes);
    }
    const uint32_t stride = 1 + (most_rows + 3) / 4;
    if (((uint64_t)n_batches * stride + total) * sizeof(uint4) > kMostBytes * n) return FR_ERR_OOM;
    uint4* records = static_cast<uint4*>(fr_alloc_device(a, (uint64_t)n_batches * stride * sizeof(uint4)));
    uint4* entries = static_cast<uint4*>(fr_alloc_device(a, std::max<uint64_t>(1, total) * sizeof(uint4)));
    SGD_NEED(records); SGD_NEED(entries);
    hipLaunchKernelGGL(k_sgd_program, dim3(n_batches), dim3(64), 0, stream, n_cells, n_more, slots, row_bytes, stride, cell_ptr, more_dev, index,
                       user_of, p->d.item, p->d.rating, place, before, heads, records, entries);
    SGD_HIP(hipStreamSynchronize(stream));
    (void)fr_alloc_free(a, before); (void)fr_alloc_free(a, size); (void)fr_alloc_free(a, place); (void)fr_alloc_free(a, more_dev);
    (void)fr_alloc_free(a, heads);
    if (F == 64)
        for (auto kernel : {k_sgd<64, false, 8>, k_sgd<64, true, 8>})
            SGD_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLds));
    p->args.records = records; p->args.entries = entries; p->args.layout = stride | p->B << 16;
    return FR_OK;
}

// Ratings in the order of the cells, for k_sgd_chain.
int sgd_lay_out_chain(SgdTask* p, fr_alloc* a, hipStream_t stream, const uint32_t* cell_ptr, const uint32_t* index, const uint32_t* user_of)
{
    const int64_t E = p->d.n_ratings;
    const uint64_t n = (uint64_t)std::max<int64_t>(1, E);
    uint64_t* keys = static_cast<uint64_t*>(fr_alloc_device(a, n * 8));
    float* sorted = static_cast<float*>(fr_alloc_device(a, n * 4));
    SGD_NEED(keys); SGD_NEED(sorted);
    if (E > 0)
        hipLaunchKernelGGL(k_sgd_stream, dim3((unsigned)((E + 255) / 256)), dim3(256), 0, stream, E, index, user_of, p->d.item, p->d.rating, keys, sorted);
    SGD_HIP(hipStreamSynchronize(stream));
    p->chain.keys = keys; p->chain.rating = sorted; p->chain.cell_ptr = cell_ptr;
    return FR_OK;
}

int sgd_init(void* user, fr_alloc* a, void* stream_v)
{
    SgdTask* p = static_cast<SgdTask*>(user);
    hipStream_t stream = (hipStream_t)stream_v;
    if (a->host_only) return FR_ERR_ARG;      // this task needs a GPU
    const int64_t U = p->d.n_users, I = p->d.n_items, E = p->d.n_ratings;
    const int F = p->d.factors;
    // caller-provided buffers count against the task's limit
    const uint64_t caller = 4ull * (uint64_t)(U + 1) + 8ull * (uint64_t)E + 4ull * (uint64_t)F * (uint64_t)(U + I);
    if (fr_alloc_charge(a, caller) != FR_OK) return FR_ERR_OOM;
    const uint32_t B = p->B;

    int32_t* bad = static_cast<int32_t*>(fr_alloc_device(a, sizeof(int32_t)));
    SGD_NEED(bad);
    hipLaunchKernelGGL(k_sgd_set, dim3(1), dim3(1), 0, stream, bad, 0);
    const unsigned vgrid = (unsigned)std::min<int64_t>((std::max<int64_t>(U + 1, E) + 255) / 256, 65536);
    hipLaunchKernelGGL(k_sgd_validate, dim3(vgrid), dim3(256), 0, stream, U, I, E, p->d.row_ptr, p->d.item, bad);
    int32_t bad_host = 0;
    SGD_HIP(hipMemcpyAsync(&bad_host, bad, sizeof(int32_t), hipMemcpyDeviceToHost, stream));
    SGD_HIP(hipStreamSynchronize(stream));
    if (bad_host) return FR_ERR_ARG;          // (indices are only trusted from here on)

    // ---- blocks of about E / B ratings
    p->ustart = static_cast<uint32_t*>(fr_alloc_device(a, ((uint64_t)B + 1) * 4));
    p->istart = static_cast<uint32_t*>(fr_alloc_device(a, ((uint64_t)B + 1) * 4));
    SGD_NEED(p->ustart); SGD_NEED(p->istart);
    {
        uint32_t* count = static_cast<uint32_t*>(fr_alloc_device(a, ((uint64_t)I + 1) * 4));
        uint32_t* before = static_cast<uint32_t*>(fr_alloc_device(a, ((uint64_t)I + 1) * 4));
        SGD_NEED(count); SGD_NEED(before);
        hipLaunchKernelGGL(k_sgd_zero, dim3((unsigned)((I + 1 + 255) / 256)), dim3(256), 0, stream, count, (uint64_t)I + 1);
        if (E > 0) hipLaunchKernelGGL(k_sgd_count_items, dim3((unsigned)((E + 255) / 256)), dim3(256), 0, stream, E, p->d.item, count);
        size_t bytes = 0;
        SGD_HIP(rocprim::exclusive_scan(nullptr, bytes, count, before, 0u, (size_t)I + 1, rocprim::plus<uint32_t>(), stream));
        void* tmp = fr_alloc_device(a, bytes ? bytes : 1);
        SGD_NEED(tmp);
        SGD_HIP(rocprim::exclusive_scan(tmp, bytes, count, before, 0u, (size_t)I + 1, rocprim::plus<uint32_t>(), stream));
        hipLaunchKernelGGL(k_sgd_starts, dim3((B + 1 + 255) / 256), dim3(256), 0, stream, (uint32_t)I, before, E, B, p->istart);
        hipLaunchKernelGGL(k_sgd_starts, dim3((B + 1 + 255) / 256), dim3(256), 0, stream, (uint32_t)U,
                           reinterpret_cast<const uint32_t*>(p->d.row_ptr), E, B, p->ustart);
        p->ustart_host.assign((size_t)B + 1, 0); p->istart_host.assign((size_t)B + 1, 0);
        SGD_HIP(hipMemcpyAsync(p->ustart_host.data(), p->ustart, ((size_t)B + 1) * 4, hipMemcpyDeviceToHost, stream));
        SGD_HIP(hipMemcpyAsync(p->istart_host.data(), p->istart, ((size_t)B + 1) * 4, hipMemcpyDeviceToHost, stream));
        SGD_HIP(hipStreamSynchronize(stream));
        (void)fr_alloc_free(a, tmp); (void)fr_alloc_free(a, before); (void)fr_alloc_free(a, count);
    }

    // ---- ratings in the order of the cells: the caller's order is by user and item already, and the sort is stable
    const uint64_t n = (uint64_t)(E ? E : 1);
    const uint32_t n_cells = B * B;
    uint32_t* cell_a = static_cast<uint32_t*>(fr_alloc_device(a, n * 4));
    uint32_t* cell_b = static_cast<uint32_t*>(fr_alloc_device(a, n * 4));
    uint32_t* index_a = static_cast<uint32_t*>(fr_alloc_device(a, n * 4));
    uint32_t* index_b = static_cast<uint32_t*>(fr_alloc_device(a, n * 4));
    uint32_t* user_of = static_cast<uint32_t*>(fr_alloc_device(a, n * 4));
    uint32_t* cell_ptr = static_cast<uint32_t*>(fr_alloc_device(a, ((uint64_t)n_cells + 1) * 4));
    SGD_NEED(cell_a); SGD_NEED(cell_b); SGD_NEED(index_a); SGD_NEED(index_b); SGD_NEED(user_of); SGD_NEED(cell_ptr);
    uint32_t *cell = cell_a, *index = index_a;
    if (E > 0) {
        hipLaunchKernelGGL(k_sgd_keys, dim3((unsigned)((E + 255) / 256)), dim3(256), 0, stream, U, E, p->d.row_ptr, p->d.item, B,
                           p->ustart, p->istart, cell_a, index_a, user_of, bad);
        SGD_HIP(hipMemcpyAsync(&bad_host, bad, sizeof(int32_t), hipMemcpyDeviceToHost, stream));
        SGD_HIP(hipStreamSynchronize(stream));
        if (bad_host) return FR_ERR_ARG;      // items of a row not ascending / not distinct
        unsigned end_bit = 1;
        while (end_bit < 32 && (1ull << end_bit) < (uint64_t)n_cells) ++end_bit;
        rocprim::double_buffer<uint32_t> keys(cell_a, cell_b), values(index_a, index_b);
        size_t bytes = 0;
        SGD_HIP(rocprim::radix_sort_pairs(nullptr, bytes, keys, values, (size_t)E, 0u, end_bit, stream));
        void* tmp = fr_alloc_device(a, bytes ? bytes : 1);
        SGD_NEED(tmp);
        SGD_HIP(rocprim::radix_sort_pairs(tmp, bytes, keys, values, (size_t)E, 0u, end_bit, stream));
        SGD_HIP(hipStreamSynchronize(stream));
        (void)fr_alloc_free(a, tmp);
        cell = keys.current(); index = values.current();
    }
    (void)fr_alloc_free(a, bad);
    hipLaunchKernelGGL(k_sgd_cells, dim3((n_cells + 1 + 255) / 256), dim3(256), 0, stream, E, B, cell, cell_ptr);
    p->cells.assign((size_t)n_cells + 1, 0);
    SGD_HIP(hipMemcpyAsync(p->cells.data(), cell_ptr, p->cells.size() * 4, hipMemcpyDeviceToHost, stream));
    SGD_HIP(hipStreamSynchronize(stream));
    (void)fr_alloc_free(a, cell_a); (void)fr_alloc_free(a, cell_b);
    (void)fr_alloc_free(a, index == index_a ? index_b : index_a);
    if (p->cells[0] != 0 || p->cells[n_cells] != (uint32_t)E) return FR_ERR_ARG;

    p->prefix.assign((size_t)B * B + 1, 0);
    p->max_cell = 0;
    p->chain_ratings = 0;
    uint32_t stratum_max = 0;
    for (size_t c = 0; c < (size_t)B * B; ++c) {
        if (p->cells[c + 1] < p->cells[c]) return FR_ERR_ARG;
        const uint32_t len = p->cells[c + 1] - p->cells[c];
        p->max_cell = std::max(p->max_cell, len);
        stratum_max = std::max(stratum_max, len);
        if ((c + 1) % B == 0) { p->chain_ratings += stratum_max; stratum_max = 0; }
        p->prefix[c + 1] = p->prefix[c] + ceil_fs_to_ns((unsigned __int128)len * p->d.fs_per_rating);
    }
    p->args = SgdArgs{};
    p->chain = ChainArgs{};
    // Rounds, or where they do not pay, or the rounds' layout is out of proportion to the ratings or has no room in the task's
    // limit (or on the device), one rating after the other: that needs no more memory than the sort before it did.
    p->cus = fr_stream_cus(stream);
    bool rounds = sgd_rounds_pay((uint64_t)E, B, p->chain_ratings, F, p->cus);
    if (rounds) {
        const size_t mark = fr_alloc_mark(a);
        int rc = sgd_lay_out_rounds(p, a, stream, cell_ptr, index, user_of);
        if (rc == FR_ERR_OOM || (rc != FR_OK && a->oom)) {
            fr_alloc_back_to(a, mark);
            p->lds_bytes = 0;
            rounds = false;
        } else if (rc != FR_OK) {
            return rc;
        }
    }
    if (rounds) {
        (void)fr_alloc_free(a, cell_ptr);
    } else {
        int rc = sgd_lay_out_chain(p, a, stream, cell_ptr, index, user_of);
        if (rc != FR_OK) return rc;
    }
    (void)fr_alloc_free(a, user_of); (void)fr_alloc_free(a, index);
    auto shared = [&](auto& A) { A.P = p->d.P; A.Q = p->d.Q; A.gamma = p->d.gamma; A.gl = p->d.gamma * p->d.lambda; };
    shared(p->args);
    shared(p->chain);
    p->footprint_after = fr_alloc_used(a);
    p->footprint_peak = fr_alloc_peak(a);
    p->run = 0; p->seg = 0; p->tile = 0;
    p->inited = true;
    return FR_OK;
}

int sgd_create(void* user)
{
    static_cast<SgdTask*>(user)->registered = true;
    return FR_OK;
}

int sgd_plan(void* user, uint64_t budget_ns, uint64_t launch_cost_ns, fr_step* out)
{
    SgdTask* p = static_cast<SgdTask*>(user);
    std::memset(out, 0, sizeof(*out));
    out->run = p->run; out->segment = p->seg; out->tile0 = p->tile; out->tile1 = p->tile;
    if (!p->inited) return FR_ERR_STATE;
    if (p->d.max_runs > 0 && p->run >= (uint32_t)p->d.max_runs) { out->finished = 1; return FR_OK; }
    const uint64_t floor_ns = p->d.min_step_ns;
    if (floor_ns > budget_ns || launch_cost_ns > budget_ns - floor_ns) return FR_OK;     // even the shortest step is too long
    const uint64_t* pre = p->prefix.data() + (size_t)(p->seg % p->B) * p->B;             // this stratum's cells
    uint32_t n = 0;
    int rc = fr_chunk_fit(pre, p->B, p->tile, budget_ns, launch_cost_ns, &n);
    if (rc != FR_OK) return rc;
    if (n == 0) return FR_OK;
    const uint32_t c0 = (p->seg % p->B) * p->B;
    uint64_t cost = std::max(pre[p->tile + n] - pre[p->tile], floor_ns);
    if (p->d.fs_per_chain_rating) {
        uint32_t longest = 0;
        for (uint32_t t = p->tile; t < p->tile + n; ++t) longest = std::max(longest, p->cells[c0 + t + 1] - p->cells[c0 + t]);
        cost = std::max(cost, ceil_fs_to_ns((unsigned __int128)longest * p->d.fs_per_chain_rating));
        if (cost > budget_ns || launch_cost_ns > budget_ns - cost) return FR_OK;     // the chain does not fit
    }
    out->tile1 = p->tile + n;
    out->modelled_ns = cost;
    out->work_units = p->cells[c0 + out->tile1] - p->cells[c0 + p->tile];
    out->completes_run = (p->seg + 1 == p->n_segments() && out->tile1 == p->B) ? 1 : 0;
    return FR_OK;
}

int sgd_run(void* user, void* stream, const fr_step* st)
{
    SgdTask* p = static_cast<SgdTask*>(user);
    if (!p->inited || st->run != p->run || st->segment != p->seg || st->tile0 != p->tile) return FR_ERR_STATE;
    int rc = sgd_launch(p, p->seg, st->tile0, st->tile1, (hipStream_t)stream,
                        GateArg{static_cast<fr_gate*>(st->gate), st->gate_slot, st->gate_need_ticks});
    if (rc != FR_OK) return rc;
    p->tile = st->tile1;
    if (p->tile == p->B) {
        p->tile = 0;
        if (++p->seg == p->n_segments()) { p->seg = 0; p->run++; }
    }
    return FR_OK;
}

// (this task's steps are all or nothing - plan_step leaves gate_tile at 0 and the kernel never stops between cells,
// whose updates are made in place and must not be made twice - so tiles_done is always 0)
int sgd_rewind(void* user, const fr_step* first, uint32_t tiles_done, uint64_t* work_done)
{
    SgdTask* p = static_cast<SgdTask*>(user);
    if (!p->inited || !first || !work_done || tiles_done != 0 || first->segment >= p->n_segments() || first->tile0 >= p->B) return FR_ERR_ARG;
    p->run = first->run; p->seg = first->segment; p->tile = first->tile0;
    *work_done = 0;
    return FR_OK;
}

int sgd_stop(void* user)
{
    SgdTask* p = static_cast<SgdTask*>(user);
    p->inited = false;        // the runtime's allocator frees the device blocks
    p->registered = false;
    return FR_OK;
}

}  // namespace

extern "C" {

int fr_sgd_make(const fr_sgd_desc* d, fr_task_ops* ops_out, void** user_out, fr_task_profile* prof_out)
{
    if (!d || !ops_out || !user_out || !prof_out) return FR_ERR_ARG;
    if (d->n_users < 1 || d->n_users >= kMaxIds || d->n_items < 1 || d->n_items >= kMaxIds) return FR_ERR_ARG;
    if (d->n_ratings < 0 || d->n_ratings > 0x7fffffffLL) return FR_ERR_ARG;
    if (!d->row_ptr || !d->P || !d->Q || (d->n_ratings > 0 && (!d->item || !d->rating))) return FR_ERR_ARG;
    if (d->factors != 16 && d->factors != 32 && d->factors != 64) return FR_ERR_ARG;
    if (d->blocks < 0 || d->blocks > (int32_t)kMaxBlocks) return FR_ERR_ARG;
    if (d->iterations < 1 || d->iterations > 100000 || d->max_runs < 0) return FR_ERR_ARG;
    if (!(d->gamma >= 0.0f) || !(d->lambda >= 0.0f)) return FR_ERR_ARG;
    SgdTask* p = new (std::nothrow) SgdTask();
    if (!p) return FR_ERR_ARG;
    p->d = *d;
    // blocks: as many as there are cells to run side by side, but cells of a few dozen ratings at least
    uint32_t B = (uint32_t)d->blocks;
    if (B == 0) {
        B = kMaxBlocks;
        while (B > 1 && (uint64_t)d->n_ratings / ((uint64_t)B * B) < 32) B /= 2;
    }
    B = (uint32_t)std::min<int64_t>(B, std::min(d->n_users, d->n_items));
    if ((uint64_t)p->d.iterations * B > 0xffffffffull) { delete p; return FR_ERR_ARG; }
    p->B = B;
    if (!p->d.fs_per_rating) p->d.fs_per_rating = 1000000;
    ops_out->create = sgd_create;
    ops_out->init = sgd_init;
    ops_out->plan_step = sgd_plan;
    ops_out->run_step = sgd_run;
    ops_out->stop = sgd_stop;
    ops_out->rewind = sgd_rewind;
    prof_out->mem_limit_bytes = d->mem_limit_bytes;
    prof_out->min_step_ns = d->min_step_ns ? d->min_step_ns : 1;
    *user_out = p;
    return FR_OK;
}

int fr_sgd_destroy(void* user)
{
    SgdTask* p = static_cast<SgdTask*>(user);
    if (!p) return FR_ERR_ARG;
    if (p->registered) return FR_ERR_STATE;
    if (p->inited) {
        (void)hipDeviceSynchronize();
        fr_alloc_release(&p->own);
    }
    delete p;
    return FR_OK;
}

int fr_sgd_info(void* user, fr_sgd_info_t* out)
{
    SgdTask* p = static_cast<SgdTask*>(user);
    if (!p || !out) return FR_ERR_ARG;
    if (p->prefix.empty()) return FR_ERR_STATE;          // known once InitSideTask has run
    std::memset(out, 0, sizeof(*out));
    out->blocks = p->B;
    out->largest_cell = p->max_cell;
    out->chain_ratings = p->chain_ratings;
    out->bytes_resident = p->footprint_after;
    out->bytes_peak = p->footprint_peak;
    return FR_OK;
}

int fr_sgd_block_starts(void* user, int32_t items, uint32_t* starts_host, size_t cap, size_t* n_out)
{
    SgdTask* p = static_cast<SgdTask*>(user);
    if (!p || !n_out || (!starts_host && cap)) return FR_ERR_ARG;
    if (p->prefix.empty()) return FR_ERR_STATE;
    const std::vector<uint32_t>& v = items ? p->istart_host : p->ustart_host;
    for (size_t k = 0; k < std::min(v.size(), cap); ++k) starts_host[k] = v[k];
    *n_out = v.size();
    return FR_OK;
}

int fr_sgd_cell_sizes(void* user, uint32_t stratum, uint32_t* sizes_host, size_t cap, size_t* n_out)
{
    SgdTask* p = static_cast<SgdTask*>(user);
    if (!p || !n_out || (!sizes_host && cap)) return FR_ERR_ARG;
    if (p->prefix.empty()) return FR_ERR_STATE;
    if (stratum >= p->B) return FR_ERR_ARG;
    for (size_t a = 0; a < std::min<size_t>(p->B, cap); ++a)
        sizes_host[a] = p->cells[(size_t)stratum * p->B + a + 1] - p->cells[(size_t)stratum * p->B + a];
    *n_out = p->B;
    return FR_OK;
}

int fr_sgd_run_standalone(void* user, int32_t device_id, void* stream_v, uint32_t max_cells, uint64_t* ns_out)
{
    SgdTask* p = static_cast<SgdTask*>(user);
    if (!p || device_id < 0) return FR_ERR_ARG;
    if (p->registered) return FR_ERR_STATE;
    hipStream_t stream = (hipStream_t)stream_v;
    FR_HIP_TRY(hipSetDevice(device_id), p->hip_error);
    if (!p->inited) {
        fr_alloc_reset(&p->own, p->d.mem_limit_bytes, false, device_id);
        int rc = sgd_init(p, &p->own, stream_v);
        if (rc != FR_OK) {
            const bool oom = p->own.oom;
            fr_alloc_release(&p->own);
            p->inited = false;
            return oom ? FR_ERR_OOM : rc;
        }
    }
    hipEvent_t ev[2] = {nullptr, nullptr};
    if (ns_out) {
        FR_HIP_TRY(hipEventCreate(&ev[0]), p->hip_error);
        FR_HIP_TRY(hipEventCreate(&ev[1]), p->hip_error);
        (void)hipEventRecord(ev[0], stream);
    }
    int rc = FR_OK;
    const uint32_t step = max_cells ? max_cells : p->B;
    for (uint32_t g = 0; g < p->n_segments() && rc == FR_OK; ++g)
        for (uint32_t t0 = 0; t0 < p->B && rc == FR_OK; t0 += step) rc = sgd_launch(p, g, t0, std::min(p->B, t0 + step), stream);
    if (ns_out) (void)hipEventRecord(ev[1], stream);
    hipError_t e = hipStreamSynchronize(stream);
    if (ns_out) {
        float ms = 0.f;
        *ns_out = hipEventElapsedTime(&ms, ev[0], ev[1]) == hipSuccess ? (uint64_t)((double)ms * 1.0e6 + 0.5) : 0;
        (void)hipEventDestroy(ev[0]);
        (void)hipEventDestroy(ev[1]);
    }
    if (rc != FR_OK) return rc;
    if (e != hipSuccess) { p->hip_error = (int)e; return FR_ERR_HIP; }
    return FR_OK;
}

}  // extern "C"

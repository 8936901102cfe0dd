// Builds the partition-centric layout (pr_layout.h) of the PageRank side task on the GPU, once, in InitSideTask
// (Section 4.1 of the paper: the transition that loads the task's context into GPU memory).
//
// Pipeline: check the CSR -> order the vertices by in-degree (radix sorts; perm and its inverse) -> one 64-bit key
// per edge (range, source, local row) in new ids, made in the order of the new rows -> stable radix sort by (range,
// source) -> one pass over the sorted keys: message starts, messages per chunk and per source -> scans -> scatter tiles
// (host) -> id stream, message sources, edge offsets of the ranges -> gather tiles and range classes (host) -> message
// range of every (scatter tile, range).  rocPRIM supplies the device-wide sorts and scans; they run once per task and
// are not part of any iteration.

#include <cstring>

#include <rocprim/rocprim.hpp>

#include <algorithm>
#include <cmath>

#include "pr_layout.h"

namespace {

constexpr int kBlk = 256;

inline unsigned blocks_for(uint64_t n) { return (unsigned)((n + kBlk - 1) / kBlk); }

__global__ void k_set_i32(int32_t* p, int32_t value) { *p = value; }

// Structure check of the caller's CSR so that no later kernel can index out of bounds.
__global__ __launch_bounds__(kBlk) void k_validate(int64_t V, int64_t E, const int32_t* __restrict__ row_ptr,
                                                   const int32_t* __restrict__ col, int32_t* __restrict__ bad)
{
    const int64_t i = (int64_t)blockIdx.x * kBlk + threadIdx.x;
    const int64_t stride = (int64_t)gridDim.x * kBlk;
    int err = 0;
    if (i == 0 && (row_ptr[0] != 0 || (int64_t)row_ptr[V] != E)) err = 1;
    for (int64_t v = i; v < V; v += stride) {
        const int32_t a = row_ptr[v], b = row_ptr[v + 1];
        if (a > b || a < 0 || (int64_t)b > E) err = 1;
    }
    for (int64_t e = i; e < E; e += stride) {
        const int32_t c = col[e];
        if (c < 0 || (int64_t)c >= V) err = 1;
    }
    if (err) *bad = 1;
}

// Vertex order: larger in-degree first, ties by the caller's id - except among the vertices without in-edges, which
// are ordered by falling out-degree first.  Those vertices have no row sums to gather, so their order is free as far
// as the gather sweep goes, and for the scatter sweep it lines up the ones without out-edges, which send no message,
// in one run at the very end that no scatter piece has to load.  (Breaking all ties by out-degree gives a few more
// such runs and made the gather sweep 2 to 6 % slower on R-MAT graphs: rows of like out-degree are like in whom
// they are pointed to by, and the ids of a wavefront's 64 edges then fall on fewer accumulators.)
// Two stable sorts of keys (top - degree) << 32 | id by their upper half, made in the order of the ids; `top` is 2^bits - 1
// with as many bits as a degree can have, so that a graph of 2^26 edges takes four passes of eight bits per sort (all 64
// bits: eight).  The vertices without in-edges, which end the second order, are then put in the order of the first.
__global__ __launch_bounds__(kBlk) void k_vertex_keys_out(int64_t V, uint32_t top, const int32_t* __restrict__ outdeg, uint64_t* __restrict__ keys)
{
    const int64_t v = (int64_t)blockIdx.x * kBlk + threadIdx.x;
    if (v >= V) return;
    const int32_t d = outdeg[v];
    keys[v] = ((uint64_t)(top - ((uint32_t)(d < 0 ? 0 : d) < top ? (uint32_t)(d < 0 ? 0 : d) : top)) << 32) | (uint64_t)(uint32_t)v;
}

__global__ __launch_bounds__(kBlk) void k_vertex_keys_in(int64_t V, uint32_t top, const int32_t* __restrict__ row_ptr, uint64_t* __restrict__ keys)
{
    const int64_t v = (int64_t)blockIdx.x * kBlk + threadIdx.x;
    if (v >= V) return;
    keys[v] = ((uint64_t)(top - (uint32_t)(row_ptr[v + 1] - row_ptr[v])) << 32) | (uint64_t)(uint32_t)v;
}

// A vertex without in-edges?  (its key of the first order)
struct NoInEdges {
    const int32_t* row_ptr;
    __host__ __device__ bool operator()(uint64_t key) const
    {
        const uint32_t v = (uint32_t)key;
        return row_ptr[v + 1] == row_ptr[v];
    }
};

// perm[new] = old, inv[old] = new, inv_out[new] = 1/outdeg (0 for dangling vertices), indeg[new].  `sorted` is the second
// order, `no_in` the vertices without in-edges in the first order (n_no_in[0] of them): they are the last of the order.
__global__ __launch_bounds__(kBlk) void k_perm(int64_t V, const uint64_t* __restrict__ sorted, const uint64_t* __restrict__ no_in,
                                               const uint32_t* __restrict__ n_no_in, const int32_t* __restrict__ row_ptr,
                                               const int32_t* __restrict__ outdeg, int32_t* __restrict__ perm, int32_t* __restrict__ inv,
                                               float* __restrict__ inv_out, uint32_t* __restrict__ indeg)
{
    const int64_t n = (int64_t)blockIdx.x * kBlk + threadIdx.x;
    if (n > V) return;
    if (n == V) { indeg[n] = 0; return; }
    const int64_t with_in = V - (int64_t)*n_no_in;
    uint32_t old = (uint32_t)(n < with_in ? sorted[n] : no_in[n - with_in]);
    if ((int64_t)old >= V) old = 0;                    // cannot happen: the keys hold 0 .. V-1
    perm[n] = (int32_t)old;
    inv[old] = (int32_t)n;
    const int32_t d = outdeg[old];
    inv_out[n] = d > 0 ? 1.0f / (float)d : 0.0f;
    indeg[n] = (uint32_t)(row_ptr[old + 1] - row_ptr[old]);
}

// Last index n of [0, V) with first[n] <= p, for first[0] <= p < first[V] (first: rising).  A wavefront looks together,
// 64 places at a time: four loads one after the other for 2^24 entries instead of 24.
__device__ __forceinline__ uint32_t wave_find(const uint32_t* __restrict__ first, uint32_t V, uint32_t p)
{
    const uint32_t lane = threadIdx.x & 63;
    uint64_t lo = 0, hi = V;                           // first[lo] <= p < first[hi]
    while (hi - lo > 1) {
        const uint64_t step = (hi - lo + 63) / 64;
        const uint64_t at = lo + (lane + 1) * step;
        const uint32_t n = (uint32_t)__popcll(__ballot(at < hi && first[at] <= p));
        lo += n * step;
        hi = lo + step < hi ? lo + step : hi;
    }
    return (uint32_t)lo;
}

// One key per edge, range << (kKeyLocalBits + src_bits) | source << kKeyLocalBits | local row, in the order of the new
// rows (`first`: edges before each), so that a stable sort by range and source leaves the rows of a source in order:
// 30 of 64 bits to sort for 2^22 vertices, four passes.  A workgroup makes kKeyRun keys; the rows with edges come first
// in the new order, so these lie in kKeyRun rows at most, whose starts are held in LDS.  Bound by the look-ups of inv[].
// (2^26 edges: keys and sort 5.1 ms with a search of row_ptr per edge and all 54 bits of a key sorted.)
constexpr uint32_t kKeyRun = 2048;
__global__ __launch_bounds__(kBlk) void k_keys(uint32_t V, uint32_t E, const uint32_t* __restrict__ first, const int32_t* __restrict__ row_ptr,
                                               const int32_t* __restrict__ perm, const int32_t* __restrict__ col, const int32_t* __restrict__ inv,
                                               uint32_t rows_per_part, uint32_t src_bits, uint64_t* __restrict__ keys)
{
    __shared__ uint32_t row_first[kKeyRun + 1];        // edges before the run's rows, new order
    __shared__ uint32_t row_old[kKeyRun];              // where their edges are in the caller's order
    __shared__ uint32_t ends[2];
    const uint32_t p0 = blockIdx.x * kKeyRun, p1 = E - p0 < kKeyRun ? E : p0 + kKeyRun;
    if (threadIdx.x < 128) {
        const uint32_t n = wave_find(first, V, threadIdx.x < 64 ? p0 : p1 - 1);
        if ((threadIdx.x & 63) == 0) ends[threadIdx.x >> 6] = n;
    }
    __syncthreads();
    const uint32_t n0 = ends[0], rows = ends[1] - n0 + 1 < kKeyRun ? ends[1] - n0 + 1 : kKeyRun;
    for (uint32_t i = threadIdx.x; i < rows; i += kBlk) {
        row_first[i] = first[n0 + i];
        row_old[i] = (uint32_t)row_ptr[perm[n0 + i]];
    }
    __syncthreads();
    constexpr int kEach = kKeyRun / kBlk;
    uint32_t n[kEach], c[kEach];
#pragma unroll
    for (int k = 0; k < kEach; ++k) {
        const uint32_t p = p0 + k * kBlk + threadIdx.x;
        n[k] = 0; c[k] = 0;
        if (p >= p1) continue;
        uint32_t lo = 0, hi = rows;                    // row_first[lo] <= p
        while (hi - lo > 1) {
            const uint32_t mid = (lo + hi) >> 1;
            if (row_first[mid] <= p) lo = mid;
            else hi = mid;
        }
        n[k] = n0 + lo;
        c[k] = (uint32_t)col[row_old[lo] + (p - row_first[lo])];
    }
#pragma unroll
    for (int k = 0; k < kEach; ++k) c[k] = (uint32_t)inv[c[k]];
#pragma unroll
    for (int k = 0; k < kEach; ++k) {
        const uint32_t p = p0 + k * kBlk + threadIdx.x;
        if (p < p1)
            keys[p] = ((uint64_t)(n[k] / rows_per_part) << (kKeyLocalBits + src_bits)) | ((uint64_t)c[k] << kKeyLocalBits) | (n[k] % rows_per_part);
    }
}

// ---- the sorted keys, a chunk of kIdChunk edges per wavefront: lane l holds the edges at positions 64 j + l (row j)
constexpr int kChunkRows = (int)(kIdChunk / 64);
constexpr uint32_t kChunksPerBlock = kBlk / 64;

struct ChunkKeys {
    uint64_t key[kChunkRows];        // 0 beyond the last edge
    uint64_t begins[kChunkRows];     // per row: which edges are the first of their (range, source) group, i.e. begin a message
    uint64_t repeats[kChunkRows];    // which repeat their predecessor (same range, source and row: a multi-edge)
};

__device__ __forceinline__ void read_chunk(ChunkKeys& K, uint32_t c, uint32_t E, const uint64_t* __restrict__ keys)
{
    const uint32_t lane = threadIdx.x & 63;
    const uint64_t e0 = (uint64_t)c * kIdChunk;
#pragma unroll
    for (int j = 0; j < kChunkRows; ++j) K.key[j] = e0 + 64 * j + lane < E ? keys[e0 + 64 * j + lane] : 0ull;
    uint64_t before = e0 ? keys[e0 - 1] : ~0ull;       // (no key has all bits set)
#pragma unroll
    for (int j = 0; j < kChunkRows; ++j) {
        const uint64_t k = K.key[j];
        uint64_t prev = __shfl_up(k, 1, 64);
        if (lane == 0) prev = before;
        before = __shfl(k, 63, 64);
        const bool held = e0 + 64 * j + lane < E;
        K.begins[j] = __ballot(held && (k >> kKeyLocalBits) != (prev >> kKeyLocalBits));
        K.repeats[j] = __ballot(held && k == prev);
    }
}

// One pass over the keys: message-start records, messages and repeated edges per chunk, messages per source (cnt, zero
// before; integer atomics).  A chunk's record, kStartWords 64-bit words: word j for row j (stream positions 64 j ..
// 64 j + 63 of the chunk), bit l - 1 set if position l begins a message, bit 63 if position 0 does.  The message of position l
// of row j is then: mbase[c] - 1 + (set bits of the words before j) + (bit 63 of word j) + (set bits below l in word j).
// Repeated edges, adjacent in the stream, hit one accumulator
// from neighbouring lanes, which the LDS serialises; the tile cutter counts them.  Bound by the atomics: 2^26 edges 0.3 ms
// (a pass each for records, numbering, repeats and counts, the records 64 keys a thread: 1.9 ms).
__global__ __launch_bounds__(kBlk) void k_chunk_facts(uint32_t E, int64_t V, uint32_t n_chunks, uint32_t src_mask, const uint64_t* __restrict__ keys,
                                                      uint64_t* __restrict__ starts, uint32_t* __restrict__ messages, uint32_t* __restrict__ rep,
                                                      uint32_t* __restrict__ cnt)
{
    const uint32_t c = blockIdx.x * kChunksPerBlock + threadIdx.x / 64, lane = threadIdx.x & 63;
    if (c > n_chunks) return;
    if (c == n_chunks) {                               // (the scan's last element)
        if (lane == 0) messages[c] = 0;
        return;
    }
    ChunkKeys K;
    read_chunk(K, c, E, keys);
    uint64_t* rec = starts + (uint64_t)c * kStartWords;
    uint32_t begun = 0, repeated = 0;
    uint64_t word = 0;
#pragma unroll
    for (int j = 0; j < kChunkRows; ++j) {
        if (lane == (uint32_t)j) word = K.begins[j] >> 1 | K.begins[j] << 63;
        begun += (uint32_t)__popcll(K.begins[j]);
        repeated += (uint32_t)__popcll(K.repeats[j]);
        if ((K.begins[j] >> lane) & 1u) {
            const uint32_t u = (uint32_t)(K.key[j] >> kKeyLocalBits) & src_mask;
            if ((int64_t)u < V) atomicAdd(&cnt[u], 1u);
        }
    }
    if (lane < (uint32_t)kChunkRows) rec[lane] = word;
    if (lane == 0) { messages[c] = begun; rep[c] = repeated; }
}

// Scatter tile that holds source u: the t with ubound[t] <= u < ubound[t + 1].
__device__ __forceinline__ uint32_t tile_of_source(const uint32_t* __restrict__ ubound, uint32_t n_tiles, uint32_t u)
{
    uint32_t lo = 0, hi = n_tiles;             // first index in [0, n_tiles] whose bound exceeds u
    while (lo < hi) {
        const uint32_t mid = (lo + hi) >> 1;
        if (ubound[mid] > u) hi = mid;
        else lo = mid + 1;
    }
    return lo ? lo - 1 : 0;
}

// What the host needs of the messages per source to cut the scatter sweep: which sources send any (a bit each), and the
// messages before every kFineSources-th source of all beyond the first kHeadSources (cum: before every source).  With
// falling in-degree the sources of very many messages are among the first, whose messages the host gets one by one.
// (2^22 vertices: the whole array is a 16 MB copy to memory the host has to touch first, and a walk over it.)
constexpr uint64_t kHeadSources = 1u << 18, kFineSources = 16;
__global__ __launch_bounds__(kBlk) void k_source_facts(uint64_t V, const uint32_t* __restrict__ cnt, const uint32_t* __restrict__ cum,
                                                       uint64_t* __restrict__ sends, uint32_t* __restrict__ fine, uint32_t* __restrict__ all)
{
    const uint64_t u = (uint64_t)blockIdx.x * kBlk + threadIdx.x;
    const uint64_t any = __ballot(u < V && cnt[u] != 0);
    if ((threadIdx.x & 63) == 0 && u < V) sends[u / 64] = any;
    if (u >= V) return;
    if (u >= kHeadSources && u % kFineSources == 0) fine[(u - kHeadSources) / kFineSources] = cum[u];
    if (u == V - 1) *all = cum[u] + cnt[u];
}

__global__ __launch_bounds__(kBlk) void k_zero_u32(uint64_t n, uint32_t* p)
{
    const uint64_t i = (uint64_t)blockIdx.x * kBlk + threadIdx.x;
    if (i < n) p[i] = 0u;
}

// Id stream and message sources.  Inside every chunk of kIdChunk ids the stream is stored transposed: stream position
// 64 j + l sits at slot 8 l + j, so that one 16-byte access is a lane's ids 64 apart and, for a fixed j, the 64 lanes of
// a wavefront hold 64 consecutive ids of the stream.
__global__ __launch_bounds__(kBlk) void k_emit(uint32_t E, uint32_t n_chunks, uint32_t M, uint32_t src_mask, const uint64_t* __restrict__ keys,
                                               const uint32_t* __restrict__ mbase, const uint32_t* __restrict__ ubound, uint32_t n_tiles,
                                               uint32_t id_scale, uint16_t* __restrict__ ids16, uint16_t* __restrict__ src16)
{
    const uint32_t c = blockIdx.x * kChunksPerBlock + threadIdx.x / 64, lane = threadIdx.x & 63;
    if (c >= n_chunks) return;
    ChunkKeys K;
    read_chunk(K, c, E, keys);
    uint32_t m0 = mbase[c];
    uint32_t id[kChunkRows];
#pragma unroll
    for (int j = 0; j < kChunkRows; ++j) {
        id[j] = ((uint32_t)K.key[j] & kLocalMask) * id_scale;
        if ((K.begins[j] >> lane) & 1u) {
            const uint32_t m = m0 + (uint32_t)__popcll(K.begins[j] & ((1ull << lane) - 1));
            const uint32_t u = (uint32_t)(K.key[j] >> kKeyLocalBits) & src_mask;
            if (m < M) src16[m] = (uint16_t)(u - ubound[tile_of_source(ubound, n_tiles, u)]);
        }
        m0 += (uint32_t)__popcll(K.begins[j]);
    }
    static_assert(kChunkRows == 8, "one 16-byte store a lane");
    reinterpret_cast<uint4*>(ids16)[(uint64_t)c * 64 + lane] = make_uint4(id[0] | id[1] << 16, id[2] | id[3] << 16, id[4] | id[5] << 16, id[6] | id[7] << 16);
}

__device__ __forceinline__ int64_t lower_bound_key(const uint64_t* __restrict__ keys, int64_t E, uint64_t target)
{
    int64_t lo = 0, hi = E;
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (keys[mid] < target) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

__global__ __launch_bounds__(kBlk) void k_eoff(uint32_t Q, int64_t E, uint32_t src_bits, const uint64_t* __restrict__ keys, uint32_t* __restrict__ eoff)
{
    const uint32_t q = blockIdx.x * kBlk + threadIdx.x;
    if (q > Q) return;
    eoff[q] = (uint32_t)lower_bound_key(keys, E, (uint64_t)q << (kKeyLocalBits + src_bits));
}

// Message of edge e, from its chunk's record.
__device__ __forceinline__ uint32_t message_of(uint32_t e, const uint64_t* __restrict__ starts, const uint32_t* __restrict__ mbase)
{
    const uint32_t c = e / kIdChunk, j = e % kIdChunk / 64, l = e % 64;
    const uint64_t* rec = starts + (uint64_t)c * kStartWords;
    uint32_t m = mbase[c] - 1;
    for (uint32_t i = 0; i < j; ++i) m += (uint32_t)__popcll(rec[i]);
    return m + (uint32_t)(rec[j] >> 63) + (uint32_t)__popcll(rec[j] & ((1ull << l) - 1));
}

// bins[t * Qe + j] = message range of the edges of range j whose source lies in scatter tile t.
// The first edge of a bin always begins a message, so its message is the first of the bin.
__global__ __launch_bounds__(kBlk) void k_bins(uint32_t n_tiles, uint32_t Qe, int64_t E, uint32_t M, uint32_t src_bits, const uint32_t* __restrict__ ubound,
                                               const uint64_t* __restrict__ keys, const uint64_t* __restrict__ starts,
                                               const uint32_t* __restrict__ mbase, uint2* __restrict__ bins)
{
    const uint64_t idx = (uint64_t)blockIdx.x * kBlk + threadIdx.x;
    if (idx >= (uint64_t)n_tiles * Qe) return;
    const uint64_t t = idx / Qe, j = idx % Qe;
    const uint64_t base = j << (kKeyLocalBits + src_bits);
    const int64_t lo = lower_bound_key(keys, E, base + ((uint64_t)ubound[t] << kKeyLocalBits));
    const int64_t hi = lower_bound_key(keys, E, base + ((uint64_t)ubound[t + 1] << kKeyLocalBits));
    uint2 r;
    r.x = lo < E ? message_of((uint32_t)lo, starts, mbase) : M;
    r.y = hi < E ? message_of((uint32_t)hi, starts, mbase) : M;
    if (r.y < r.x) r.y = r.x;
    bins[idx] = r;
}

struct Scratch {
    fr_alloc* a;
    hipStream_t stream;
    std::vector<void*> held;
    template <typename T>
    T* take(uint64_t count)
    {
        void* p = fr_alloc_scratch(a, (size_t)(count ? count : 1) * sizeof(T));
        if (p) held.push_back(p);
        return static_cast<T*>(p);
    }
    void drop(void* p)
    {
        for (size_t i = 0; i < held.size(); ++i)
            if (held[i] == p) { (void)fr_alloc_free(a, p); held.erase(held.begin() + (long)i); return; }
    }
    ~Scratch()
    {
        if (!held.empty()) (void)hipStreamSynchronize(stream);       // (an early return may leave work that uses them)
        for (void* p : held) (void)fr_alloc_free(a, p);
    }
};

}  // namespace

#define PREP_HIP(expr)                                             \
    do {                                                           \
        hipError_t e__ = (expr);                                   \
        if (e__ != hipSuccess) { *hip_error = (int)e__; return FR_ERR_HIP; } \
    } while (0)
#define PREP_NEED(ptr)                                             \
    do {                                                           \
        if (!(ptr)) { if (a->hip_error) *hip_error = a->hip_error; return a->hip_error ? FR_ERR_HIP : FR_ERR_OOM; } \
    } while (0)

int pr_build_layout(PrLayout* L, int64_t V, int64_t E, const int32_t* row_ptr, const int32_t* col,
                    const int32_t* out_degree, uint32_t rows_per_part, uint32_t src_per_part, uint32_t cus, fr_alloc* a,
                    hipStream_t stream, int* hip_error)
{
    if (!cus) cus = kDefaultCus;
    if (!rows_per_part) rows_per_part = V >= kLargeRowsFrom ? kRowsLarge : kRowsSmall;
    if (!src_per_part) src_per_part = V >= kLargeSrcFrom ? kSrcLarge : kSrcSmall;
    if ((rows_per_part != kRowsSmall && rows_per_part != kRowsLarge) || (src_per_part != kSrcSmall && src_per_part != kSrcLarge))
        return FR_ERR_ARG;
    L->V = V; L->E = E;
    L->rows_per_part = rows_per_part; L->src_per_part = src_per_part;
    L->Q = (uint32_t)((V + rows_per_part - 1) / rows_per_part);
    L->n_chunks = (uint32_t)((E + kIdChunk - 1) / kIdChunk);
    const int64_t padded = (int64_t)std::max<uint32_t>(L->n_chunks, 1) * kIdChunk;
    const uint32_t Q = L->Q;
    if ((uint64_t)Q >= (1ull << (63 - kKeyLocalBits - kKeySrcBits))) return FR_ERR_ARG;
    uint32_t src_bits = 1;                             // (so that ubound = V as a key's source does not reach the range, V <= 2^src_bits
    while (src_bits < (uint32_t)kKeySrcBits && (1ll << src_bits) <= V) ++src_bits;         // is not enough)
    const uint32_t src_mask = (uint32_t)((1ull << src_bits) - 1);

    Scratch tmp{a, stream, {}};

    // ---- refuse a malformed CSR before anything indexes with it
    int32_t* bad = tmp.take<int32_t>(1);
    PREP_NEED(bad);
    hipLaunchKernelGGL(k_set_i32, dim3(1), dim3(1), 0, stream, bad, 0);
    const unsigned vgrid = std::min<unsigned>(blocks_for((uint64_t)std::max<int64_t>(V, E)), 65536u);
    hipLaunchKernelGGL(k_validate, dim3(vgrid), dim3(kBlk), 0, stream, V, E, row_ptr, col, bad);
    int32_t bad_host = 0;
    PREP_HIP(hipMemcpyAsync(&bad_host, bad, sizeof(int32_t), hipMemcpyDeviceToHost, stream));
    PREP_HIP(hipStreamSynchronize(stream));
    if (bad_host) return FR_ERR_ARG;

    // ---- vertices in order of falling in-degree; those without in-edges by falling out-degree
    // The keys' two buffers are taken first; while the second is unused, what is needed to order the vertices and to make
    // the keys lies in it, if it has room (E of about 4 V; else it has blocks of its own, given back as soon as they are done with).
    {
        Carve kept;
        kept.add(&L->perm, (uint64_t)V); kept.add(&L->inv_out, (uint64_t)V);
        if (!kept.keep_apart(a)) PREP_NEED((void*)nullptr);
    }
    int32_t* inv = nullptr;
    uint64_t* keys_a = nullptr;
    uint64_t* keys_b = nullptr;
    uint32_t* first = nullptr;                         // edges before each row, new order (V + 1)
    void* vertex_block = nullptr;
    {
        uint32_t degree_bits = 1;                      // an in-degree has at most these; a larger out-degree (the caller's array
        while ((1ll << degree_bits) <= E && degree_bits < 31) ++degree_bits;      // is not held against the edges) counts as 2^bits - 1
        const uint32_t top = (uint32_t)((1ull << degree_bits) - 1);
        uint64_t *by_out = nullptr, *vk_a = nullptr, *vk_b = nullptr;
        uint8_t* t = nullptr;
        size_t sort_bytes = 0, select_bytes = 0, scan_bytes = 0;
        uint32_t* n_no_in = reinterpret_cast<uint32_t*>(bad);        // (its check is done)
        const NoInEdges no_in_edges{row_ptr};
        {
            rocprim::double_buffer<uint64_t> probe(vk_a, vk_b);
            PREP_HIP(rocprim::radix_sort_keys(nullptr, sort_bytes, probe, (size_t)V, 32u, 32u + degree_bits, stream));
        }
        PREP_HIP(rocprim::select(nullptr, select_bytes, vk_a, by_out, n_no_in, (size_t)V, no_in_edges, stream));
        PREP_HIP(rocprim::exclusive_scan(nullptr, scan_bytes, first, first, 0u, (size_t)V + 1, rocprim::plus<uint32_t>(), stream));
        Carve longer, parts;                           // what the keys are made from, and what is only needed for the order
        longer.add(&inv, (uint64_t)V); longer.add(&by_out, (uint64_t)V);
        parts.add(&vk_a, (uint64_t)V); parts.add(&vk_b, (uint64_t)V);
        // (the selection and the scan work in a key buffer that is free at the time; too few vertices for that: in `t`)
        auto in_t = [&](size_t bytes) -> size_t { return bytes > (size_t)V * 8 ? bytes : 0; };
        parts.add(&t, std::max(sort_bytes, std::max(in_t(select_bytes), in_t(scan_bytes))));
        void* order_block = nullptr;
        if (longer.bytes + parts.bytes <= (uint64_t)E * 8) {
            keys_a = tmp.take<uint64_t>((uint64_t)E);
            keys_b = tmp.take<uint64_t>((uint64_t)E);
            PREP_NEED(keys_a); PREP_NEED(keys_b);
            longer.place(keys_b);
            parts.place(reinterpret_cast<char*>(keys_b) + longer.bytes);
        } else {
            vertex_block = tmp.take<uint8_t>(longer.bytes);
            order_block = tmp.take<uint8_t>(parts.bytes);
            PREP_NEED(vertex_block); PREP_NEED(order_block);
            longer.place(vertex_block);
            parts.place(order_block);
        }
        rocprim::double_buffer<uint64_t> order(vk_a, vk_b);
        hipLaunchKernelGGL(k_vertex_keys_out, dim3(blocks_for((uint64_t)V)), dim3(kBlk), 0, stream, V, top, out_degree, vk_a);
        PREP_HIP(rocprim::radix_sort_keys(t, sort_bytes, order, (size_t)V, 32u, 32u + degree_bits, stream));
        PREP_HIP(rocprim::select(in_t(select_bytes) ? (void*)t : (void*)order.alternate(), select_bytes, order.current(), by_out, n_no_in, (size_t)V, no_in_edges, stream));
        order = rocprim::double_buffer<uint64_t>(vk_a, vk_b);
        hipLaunchKernelGGL(k_vertex_keys_in, dim3(blocks_for((uint64_t)V)), dim3(kBlk), 0, stream, V, top, row_ptr, vk_a);
        PREP_HIP(rocprim::radix_sort_keys(t, sort_bytes, order, (size_t)V, 32u, 32u + degree_bits, stream));
        uint32_t* indeg = reinterpret_cast<uint32_t*>(order.alternate());          // V + 1 words where 2 V have room
        hipLaunchKernelGGL(k_perm, dim3(blocks_for((uint64_t)V + 1)), dim3(kBlk), 0, stream, V, order.current(), by_out, n_no_in, row_ptr, out_degree, L->perm, inv, L->inv_out, indeg);
        first = reinterpret_cast<uint32_t*>(by_out);
        PREP_HIP(rocprim::exclusive_scan(in_t(scan_bytes) ? (void*)t : (void*)order.current(), scan_bytes, indeg, first, 0u, (size_t)V + 1, rocprim::plus<uint32_t>(), stream));
        if (order_block) {
            PREP_HIP(hipStreamSynchronize(stream));
            tmp.drop(order_block);
        }
    }

    // ---- sort the edges by (range, source, local row); set-up scratch is returned as soon as it is done with
    uint64_t* keys = nullptr;
    uint32_t M = 0;
    if (E > 0) {
        if (!keys_a) keys_a = tmp.take<uint64_t>((uint64_t)E);
        PREP_NEED(keys_a);
        hipLaunchKernelGGL(k_keys, dim3((unsigned)((E + kKeyRun - 1) / kKeyRun)), dim3(kBlk), 0, stream, (uint32_t)V, (uint32_t)E, first, row_ptr, L->perm, col, inv,
                           rows_per_part, src_bits, keys_a);
        if (!keys_b) {
            PREP_HIP(hipStreamSynchronize(stream));
            tmp.drop(vertex_block);
            keys_b = tmp.take<uint64_t>((uint64_t)E);
            PREP_NEED(keys_b);
        }
        unsigned end_bit = kKeyLocalBits + src_bits;
        while (end_bit < 63 && (1ull << (end_bit - kKeyLocalBits - src_bits)) < (uint64_t)Q) ++end_bit;
        rocprim::double_buffer<uint64_t> db(keys_a, keys_b);
        size_t bytes = 0;
        PREP_HIP(rocprim::radix_sort_keys(nullptr, bytes, db, (size_t)E, (unsigned)kKeyLocalBits, end_bit, stream));
        void* t = tmp.take<uint8_t>(bytes);
        PREP_NEED(t);
        PREP_HIP(rocprim::radix_sort_keys(t, bytes, db, (size_t)E, (unsigned)kKeyLocalBits, end_bit, stream));
        PREP_HIP(hipStreamSynchronize(stream));
        keys = db.current();
        tmp.drop(t);
        tmp.drop(keys == keys_a ? keys_b : keys_a);
    } else {
        PREP_HIP(hipStreamSynchronize(stream));
        tmp.drop(vertex_block);
    }

    // ---- scatter pieces: source intervals of about equal numbers of messages
    // (`cum`: messages before each of the first kHeadSources sources, then before every kFineSources-th; `sends`: a bit a source)
    const uint64_t n_head = std::min<uint64_t>((uint64_t)V, kHeadSources), n_fine = ((uint64_t)V - n_head + kFineSources - 1) / kFineSources;
    const uint64_t n_words = ((uint64_t)V + 63) / 64;
    const uint32_t *cum_head = nullptr, *cum_fine = nullptr, *rep_host = nullptr;
    const uint64_t* sends = nullptr;
    std::vector<uint64_t> facts;                       // the four of them, as they come from the device in one copy
    std::vector<uint32_t> mbase_host((size_t)L->n_chunks + 1, 0u);
    {
        Carve kept;
        kept.add(&L->starts, (uint64_t)padded / kIdChunk * kStartWords); kept.add(&L->mbase, (uint64_t)L->n_chunks + 1);
        if (!kept.keep(a)) PREP_NEED((void*)nullptr);
    }
    if (E > 0) {
        uint32_t *cnt = nullptr, *cum_dev = nullptr, *messages = nullptr, *rep = nullptr, *fine = nullptr;
        uint64_t* sends_dev = nullptr;
        uint8_t* t = nullptr;
        size_t bytes = 0, bytes_m = 0;
        PREP_HIP(rocprim::exclusive_scan(nullptr, bytes, cnt, cum_dev, 0u, (size_t)V, rocprim::plus<uint32_t>(), stream));
        PREP_HIP(rocprim::exclusive_scan(nullptr, bytes_m, messages, L->mbase, 0u, (size_t)L->n_chunks + 1, rocprim::plus<uint32_t>(), stream));
        Carve parts;
        // (rep's last entry: the messages of all sources; the host takes everything up to the head of cum in one copy)
        parts.add(&fine, n_fine); parts.add(&sends_dev, n_words); parts.add(&rep, (uint64_t)L->n_chunks + 1);
        const uint64_t fact_bytes = parts.bytes + n_head * 4;
        parts.add(&cum_dev, (uint64_t)V); parts.add(&cnt, (uint64_t)V); parts.add(&messages, (uint64_t)L->n_chunks + 1); parts.add(&t, std::max(bytes, bytes_m));
        char* block = static_cast<char*>(static_cast<void*>(tmp.take<uint8_t>(parts.bytes)));
        PREP_NEED(block);
        parts.place(block);
        hipLaunchKernelGGL(k_zero_u32, dim3(blocks_for((uint64_t)V)), dim3(kBlk), 0, stream, (uint64_t)V, cnt);
        hipLaunchKernelGGL(k_chunk_facts, dim3(L->n_chunks / kChunksPerBlock + 1), dim3(kBlk), 0, stream, (uint32_t)E, V, L->n_chunks, src_mask, keys, L->starts,
                           messages, rep, cnt);
        PREP_HIP(rocprim::exclusive_scan(t, bytes_m, messages, L->mbase, 0u, (size_t)L->n_chunks + 1, rocprim::plus<uint32_t>(), stream));
        PREP_HIP(rocprim::exclusive_scan(t, bytes, cnt, cum_dev, 0u, (size_t)V, rocprim::plus<uint32_t>(), stream));
        hipLaunchKernelGGL(k_source_facts, dim3(blocks_for((uint64_t)V)), dim3(kBlk), 0, stream, (uint64_t)V, cnt, cum_dev, sends_dev, fine, rep + L->n_chunks);
        facts.resize(fact_bytes / 8 + 1);                 // (while the device works)
        PREP_HIP(hipMemcpyAsync(facts.data(), block, fact_bytes, hipMemcpyDeviceToHost, stream));
        PREP_HIP(hipMemcpyAsync(mbase_host.data(), L->mbase, ((size_t)L->n_chunks + 1) * 4, hipMemcpyDeviceToHost, stream));
        PREP_HIP(hipStreamSynchronize(stream));
        auto on_host = [&](const void* p) { return static_cast<const void*>(reinterpret_cast<const char*>(facts.data()) + (static_cast<const char*>(p) - block)); };
        cum_head = static_cast<const uint32_t*>(on_host(cum_dev));
        cum_fine = static_cast<const uint32_t*>(on_host(fine));
        sends = static_cast<const uint64_t*>(on_host(sends_dev));
        rep_host = static_cast<const uint32_t*>(on_host(rep));
        const uint32_t sum = rep_host[L->n_chunks];
        tmp.drop(block);
        M = mbase_host[L->n_chunks];
        if (sum != M) return FR_ERR_ARG;
    } else {
        facts.assign((n_head + n_fine) / 2 + 1 + n_words, 0ull);       // no messages, and no source that sends any
        sends = facts.data();
        cum_head = reinterpret_cast<const uint32_t*>(facts.data() + n_words);
        cum_fine = cum_head + n_head;
        PREP_HIP(hipMemcpyAsync(L->mbase, mbase_host.data(), 4, hipMemcpyHostToDevice, stream));
    }
    // messages of the sources before u: any u up to kHeadSources, beyond it a multiple of kFineSources or V
    auto messages_before = [&](uint64_t u) -> uint64_t {
        if (u >= (uint64_t)V) return M;
        return u < n_head ? cum_head[u] : cum_fine[(u - n_head) / kFineSources];
    };
    L->M = M;

    // ---- the arrays that stay
    {
        Carve kept;
        kept.add(&L->ids16, (uint64_t)padded); kept.add(&L->src16, ((uint64_t)M + 15) / 8 * 8);     // (read eight at a time)
        if (!kept.keep(a)) PREP_NEED((void*)nullptr);
    }
    uint32_t* eoff = tmp.take<uint32_t>((uint64_t)Q + 1);
    PREP_NEED(eoff);
    hipLaunchKernelGGL(k_eoff, dim3(blocks_for((uint64_t)Q + 1)), dim3(kBlk), 0, stream, Q, E, src_bits, keys, eoff);
    std::vector<uint32_t> eoff_host((size_t)Q + 1);
    PREP_HIP(hipMemcpyAsync(eoff_host.data(), eoff, ((size_t)Q + 1) * 4, hipMemcpyDeviceToHost, stream));
    PREP_HIP(hipStreamSynchronize(stream));
    if (eoff_host[0] != 0 || eoff_host[Q] != (uint32_t)E) return FR_ERR_ARG;

    // ---- gather tiles and range classes.  Rows are in order of falling in-degree, so the ranges with edges come first.
    uint32_t Qe = 0;
    for (uint32_t j = 0; j < Q; ++j)
        if (eoff_host[j + 1] > eoff_host[j]) Qe = j + 1;
    if (Qe == 0) Qe = 1;          // a graph without edges: range 0 still gets a (direct) gather tile
    L->Qe = Qe;
    // weight of the stream up to every chunk boundary: an edge counts 1, a message kGatherMessageWeight more, a
    // repeated edge kGatherRepeatWeight more (measured on single tiles: 0.09 ns, 0.18 ns and 0.28 ns a piece)
    std::vector<uint64_t> wcum((size_t)L->n_chunks + 1, 0);
    if (E > 0) {
        for (uint32_t c = 0; c < L->n_chunks; ++c) {
            const uint64_t edges = std::min<uint64_t>(kIdChunk, (uint64_t)E - (uint64_t)c * kIdChunk);
            wcum[c + 1] = wcum[c] + kGatherEdgeWeight * edges + kGatherMessageWeight * (uint64_t)(mbase_host[c + 1] - mbase_host[c]) +
                          kGatherRepeatWeight * (uint64_t)rep_host[c];
        }
    }
    auto weight_at = [&](uint64_t e) -> uint64_t {          // weight of the edges before e (linear inside a chunk)
        const uint64_t c = e / kIdChunk;
        if (c >= L->n_chunks) return wcum[L->n_chunks];
        const uint64_t held = std::min<uint64_t>(kIdChunk, (uint64_t)E - c * kIdChunk);      // the last chunk may be short
        return wcum[c] + (wcum[c + 1] - wcum[c]) * std::min(e - c * kIdChunk, held) / held;
    };
    L->gp.clear(); L->gt.clear(); L->gt_weight.clear(); L->gt_edges.clear();
    L->ri.assign(Q, RangeInfo{kRangeEmpty, 0}); L->fin.clear();
    {
        // A piece costs its weight plus a fixed part (kTileFixedWeight: the chain of dependent loads at its start and
        // the row pass at its end).  Ranges are cut into pieces of at most `body` weight; pieces are then grouped, in
        // order, into tiles of at most body + kTileFixedWeight.  A launch has no more workgroups than run side by
        // side (`slots`), each of which takes the next tile when it is done with one.  Where a slot's share of the
        // sweep is long against what a tile costs to start and to end (kGatherFineShare), heavy ranges are cut for
        // two pieces per slot and every piece is a tile of its own, so that the many light tiles at the end fill
        // the gaps the heavy ones leave; below that there are no more tiles than slots, light pieces share tiles, and
        // `body` is the smallest (to 2 %) that achieves it (least_gather_weight, kLeastGatherOfTwo).
        std::vector<uint64_t> w(Qe);
        uint64_t total = 0, heaviest = 0;
        for (uint32_t j = 0; j < Qe; ++j) {
            w[j] = weight_at(eoff_host[j + 1]) - weight_at(eoff_host[j]);
            total += w[j];
            heaviest = std::max(heaviest, w[j]);
        }
        const bool alone = gather_alone(rows_per_part, Qe, total, cus);                // one workgroup a unit
        const uint64_t slots = (uint64_t)cus * (alone ? 1 : 2);
        const uint64_t share = (total + slots - 1) / slots;
        const uint64_t fine = share >= kGatherFineShare ? 2 : 1;
        const uint64_t least = least_gather_weight(rows_per_part, heaviest);
        std::vector<GatherPiece> pieces;
        std::vector<uint64_t> piece_w;
        std::vector<uint2> tiles;
        uint64_t body = std::max<uint64_t>(least, (total + slots * fine - 1) / (slots * fine));
        for (int round = 0; round < 400; ++round) {
            pieces.clear(); piece_w.clear(); tiles.clear();
            L->ri.assign(Q, RangeInfo{kRangeEmpty, 0});
            L->fin.clear();
            L->n_merged = 0; L->n_partials = 0;
            for (uint32_t j = 0; j < Qe; ++j) {
                const uint64_t e0 = eoff_host[j], e1 = eoff_host[j + 1];
                const uint64_t nt = std::max<uint64_t>(1, (w[j] + body - 1) / body);
                std::vector<uint64_t> cuts;                      // chunk boundaries strictly inside (e0, e1)
                const uint64_t w0 = weight_at(e0);
                for (uint64_t i = 1; i < nt; ++i) {
                    const uint64_t want = w0 + w[j] * i / nt;
                    const uint64_t c = (uint64_t)(std::lower_bound(wcum.begin(), wcum.end(), want) - wcum.begin());
                    const uint64_t cut = c * kIdChunk;
                    if (cut > (cuts.empty() ? e0 : cuts.back()) && cut < e1) cuts.push_back(cut);
                }
                if (cuts.empty()) {
                    pieces.push_back(GatherPiece{j, (uint32_t)e0, (uint32_t)e1, kNoPartial});
                    piece_w.push_back(w[j] + kTileFixedWeight);
                    L->ri[j] = RangeInfo{kRangeDirect | (1u << 2), 0};
                    continue;
                }
                L->ri[j] = RangeInfo{kRangeMerged | ((uint32_t)(cuts.size() + 1) << 2), L->n_partials};
                L->fin.push_back(j);
                L->n_merged++;
                cuts.push_back(e1);
                uint64_t lo = e0;
                for (uint64_t hi : cuts) {
                    pieces.push_back(GatherPiece{j, (uint32_t)lo, (uint32_t)hi, L->n_partials++});
                    piece_w.push_back(weight_at(hi) - weight_at(lo) + kTileFixedWeight);
                    lo = hi;
                }
            }
            uint64_t in_tile = 0;
            uint32_t first = 0;
            for (uint32_t i = 0; i < pieces.size(); ++i) {
                if (i > first && (fine > 1 || in_tile + piece_w[i] > body + kTileFixedWeight)) {
                    tiles.push_back(make_uint2(first, i));
                    first = i; in_tile = 0;
                }
                in_tile += piece_w[i];
            }
            tiles.push_back(make_uint2(first, (uint32_t)pieces.size()));
            if (fine > 1) break;
            if (!alone && tiles.size() > cus && body < kLeastGatherOfTwo) { body = kLeastGatherOfTwo; continue; }      // some units have two
            if (tiles.size() <= slots) break;
            body += body / 50 + 1;
        }
        for (uint32_t j = Qe; j < Q; ++j) L->fin.push_back(j);
        L->gp = pieces;
        L->gt.clear();
        for (const uint2& t : tiles) L->gt.push_back(GatherTile{t.x, t.y, pieces[t.x], {0, 0}});
        for (const uint2& t : tiles) {
            uint64_t wsum = 0, esum = 0;
            for (uint32_t i = t.x; i < t.y; ++i) { wsum += piece_w[i]; esum += (uint64_t)pieces[i].e1 - pieces[i].e0; }
            L->gt_weight.push_back(wsum);
            L->gt_edges.push_back(esum);
        }
    }
    L->cus = cus;
    L->gather_slots = cus * (rows_per_part == kRowsSmall ? 2u : 1u);
    L->scatter_slots = cus * (src_per_part == kSrcSmall ? 2u : 1u);
    L->n_pieces = (uint32_t)L->gp.size();
    L->n_gather = (uint32_t)L->gt.size();
    L->n_finish = (uint32_t)L->fin.size();

    // ---- scatter pieces and tiles.  A piece is an interval of at most src_per_part sources and at most `target`
    // weight, where a message weighs kScatterMessageWeight and a source kScatterRowWeight times the values read to
    // finish it (its contrib or 1/outdeg, and the partial sums of a row of a merged range); the pieces of the sources
    // with few messages are as wide as allowed and light whatever the target.  A tile is a run of consecutive pieces
    // whose costs (weight + kScatterFixedWeight a piece, for the chain of dependent loads at its start) add up to at
    // most target + kScatterFixedWeight.  A launch has no more workgroups than run side by side (`slots`), each of
    // which takes the next tile when it is done with one; with `fine` tiles per slot the light tiles at the end fill
    // the gaps the heavy ones leave, which pays where a slot's share of the sweep is long: from kScatterFineShare on
    // the pieces are cut for two per slot and each is a tile of its own.  Below that the target is the smallest one
    // (to 2 %) that leaves no more tiles than slots.
    std::vector<uint32_t> ubound;
    std::vector<uint8_t> piece_void;
    std::vector<uint2> stiles;
    {
        std::vector<uint64_t> per_row(Q), rows_before((size_t)Q + 1, 0);
        for (uint32_t j = 0; j < Q; ++j) {
            per_row[j] = 1 + ((L->ri[j].cls_tiles & 3u) == kRangeMerged ? (L->ri[j].cls_tiles >> 2) : 0u);
            const uint64_t lo = (uint64_t)j * rows_per_part, hi = std::min<uint64_t>((uint64_t)V, lo + rows_per_part);
            rows_before[j + 1] = rows_before[j] + (hi - lo) * per_row[j];
        }
        // Runs of kVoidMin or more consecutive sources that send no message (vertices without out-edges: the order by
        // in-degree, then out-degree, lines them up at the end of every class of equal in-degree) become VOID pieces,
        // which no tile holds: nothing of them is loaded.  Not in merged ranges, whose rows the scatter sweep
        // finishes.  Their dangling mass is not lost: in a range with in-edges the gather tile counts it, and in a
        // range without, every such row holds the base value, so the sweep adds base x their number in one go.
        std::vector<std::pair<uint64_t, uint64_t>> voids;
        std::vector<uint64_t> void_rows_before_void;        // rows in the void runs before each of them
        {
            uint64_t first_voidable = std::min<uint64_t>((uint64_t)V, src_per_part);      // (the first piece always exists)
            for (uint32_t j = 0; j < Q; ++j)
                if ((L->ri[j].cls_tiles & 3u) == kRangeMerged) first_voidable = std::max(first_voidable, std::min<uint64_t>((uint64_t)V, ((uint64_t)j + 1) * rows_per_part));
            // (by words of 64 sources; beyond kHeadSources a run is cut to multiples of kFineSources)
            uint64_t run_start = first_voidable, rows = 0;
            auto end_run = [&](uint64_t lo, uint64_t hi) {
                if (lo >= kHeadSources) lo = (lo + kFineSources - 1) / kFineSources * kFineSources;
                if (hi > kHeadSources && hi < (uint64_t)V) hi = hi / kFineSources * kFineSources;
                if (hi < lo + kVoidMin) return;
                voids.push_back({lo, hi}); void_rows_before_void.push_back(rows);
                rows += hi - lo;
            };
            for (uint64_t k = first_voidable / 64; k < n_words; ++k) {
                uint64_t w = sends[k];
                if (k == first_voidable / 64) w &= ~0ull << (first_voidable % 64);
                if (!w) continue;
                end_run(run_start, k * 64 + (uint64_t)__builtin_ctzll(w));
                run_start = k * 64 + 64 - (uint64_t)__builtin_clzll(w);      // (shorter runs inside the word do not count)
            }
            end_run(run_start, (uint64_t)V);
            void_rows_before_void.push_back(rows);
        }
        auto void_rows_before = [&](uint64_t u) -> uint64_t {        // rows of void runs among the sources before u
            if (voids.empty() || u <= voids[0].first) return 0;
            const size_t k = (size_t)(std::upper_bound(voids.begin(), voids.end(), std::pair<uint64_t, uint64_t>(u, ~(uint64_t)0)) - voids.begin());   // runs starting at or before u
            if (k == 0) return 0;
            return void_rows_before_void[k - 1] + std::min(u, voids[k - 1].second) - voids[k - 1].first;
        };
        // (asked for some 20 times a piece and cut: with a division and a search among the void runs each time most of the 1.7 ms
        // that the device waited for the host's cuts on 2^22 vertices / 2^26 edges)
        const int row_bits = rows_per_part == kRowsLarge ? 14 : 13;
        auto weight_before = [&](uint64_t u) -> uint64_t {
            const uint64_t j = std::min<uint64_t>(u >> row_bits, Q);
            const uint64_t rows = rows_before[j] + (j < Q ? (u - (j << row_bits)) * per_row[j] : 0);
            return kScatterMessageWeight * messages_before(u) + kScatterRowWeight * (rows - void_rows_before(u));
        };
        auto cut = [&](uint64_t target) {
            ubound.clear(); piece_void.clear();
            uint64_t u = 0;
            size_t vi = 0;
            while (u < (uint64_t)V) {
                if (vi < voids.size() && u == voids[vi].first) {
                    ubound.push_back((uint32_t)u); piece_void.push_back(1);
                    u = voids[vi++].second;
                    continue;
                }
                uint64_t limit = std::min<uint64_t>((uint64_t)V, u + src_per_part);
                if (vi < voids.size()) limit = std::min(limit, voids[vi].first);
                if (limit > kHeadSources && limit < (uint64_t)V) limit = limit / kFineSources * kFineSources;
                const uint64_t want = weight_before(u) + target;
                uint64_t lo = u + 1, hi = limit;             // the first end in (u, limit] that reaches `want`, else limit
                if (hi > kHeadSources) {                     // (beyond the head: the first multiple of kFineSources that does)
                    const uint64_t from = std::max(kHeadSources, u);
                    if (u < kHeadSources && weight_before(kHeadSources) >= want) {
                        hi = kHeadSources;
                    } else {
                        uint64_t a_lo = from / kFineSources + 1, a_hi = (limit + kFineSources - 1) / kFineSources;      // (u is a multiple there)
                        while (a_lo < a_hi) {
                            const uint64_t mid = (a_lo + a_hi) / 2;
                            if (weight_before(mid * kFineSources) >= want) a_hi = mid;
                            else a_lo = mid + 1;
                        }
                        lo = hi = std::min(limit, a_lo * kFineSources);
                    }
                }
                while (lo < hi) {
                    const uint64_t mid = (lo + hi) / 2;
                    if (weight_before(mid) >= want) hi = mid;
                    else lo = mid + 1;
                }
                ubound.push_back((uint32_t)u); piece_void.push_back(0);
                u = lo;
            }
            ubound.push_back((uint32_t)V);
        };
        auto live_pieces = [&]() { size_t n = 0; for (uint8_t v : piece_void) n += v ? 0 : 1; return n; };
        auto pack = [&](uint64_t limit) {                    // (limit 0: a tile per piece); void pieces are in no tile
            stiles.clear();
            const uint32_t n = (uint32_t)ubound.size() - 1;
            uint64_t in_tile = 0;
            uint32_t first = 0;
            bool open = false;
            for (uint32_t i = 0; i < n; ++i) {
                if (piece_void[i]) {
                    if (open) stiles.push_back(make_uint2(first, i));
                    open = false;
                    continue;
                }
                const uint64_t c = weight_before(ubound[i + 1]) - weight_before(ubound[i]) + kScatterFixedWeight;
                if (open && in_tile + c > limit) {
                    stiles.push_back(make_uint2(first, i));
                    open = false;
                }
                if (!open) { first = i; in_tile = 0; open = true; }
                in_tile += c;
            }
            if (open) stiles.push_back(make_uint2(first, n));
        };
        const uint64_t all = weight_before((uint64_t)V);
        const uint64_t least = least_scatter_weight(all);
        const bool alone = scatter_alone(src_per_part, all, cus);                      // one workgroup a unit
        const uint64_t slots = (uint64_t)cus * (alone ? 1 : 2);
        const uint64_t share = (all + slots - 1) / slots;
        const uint64_t fine = share >= kScatterFineShare ? 2 : 1;
        const uint64_t start = std::max<uint64_t>(least, (all + slots * fine - 1) / (slots * fine));
        bool done = false;
        if (fine > 1) {
            cut(start);
            pack(0);
            done = true;
        } else if (src_per_part == kSrcSmall) {
            // the small kernel is faster without the loop over pieces: a tile per piece, if a target up to one
            // compute unit's share of the weight leaves few enough pieces
            const uint64_t most = std::max<uint64_t>(least, (all + cus - 1) / cus);
            std::vector<uint64_t> targets;                   // (a larger target never leaves more pieces: bisection finds the first that fits)
            for (uint64_t target = start;; target = std::min(most, target + target / 50 + 1)) {
                targets.push_back(target);
                if (target >= most) break;
            }
            size_t lo = 0, hi = targets.size();
            while (lo < hi) {
                const size_t mid = (lo + hi) / 2;
                cut(targets[mid]);
                if (live_pieces() <= slots) hi = mid;
                else lo = mid + 1;
            }
            if (lo < targets.size()) { cut(targets[lo]); pack(0); done = true; }
        }
        if (!done)
            for (uint64_t target = start;; target += target / 50 + 1) {
                cut(target);
                pack(target + kScatterFixedWeight);
                if (stiles.size() <= slots) break;
            }
    }
    L->n_spieces = (uint32_t)ubound.size() - 1;
    // the void pieces' rows in ranges without in-edges (all dangling: no message means no out-edge), and the slot of
    // the dangling partials that takes base x their number
    L->void_slot = kNoVoid; L->n_void_dangling = 0;
    {
        const uint64_t first_empty_row = std::min<uint64_t>((uint64_t)V, (uint64_t)Qe * rows_per_part);
        for (uint32_t i = 0; i < L->n_spieces; ++i) {
            if (!piece_void[i]) continue;
            if (L->void_slot == kNoVoid) L->void_slot = i;
            const uint64_t u0 = std::max<uint64_t>(ubound[i], first_empty_row), u1 = ubound[i + 1];
            if (u1 > u0) L->n_void_dangling += u1 - u0;
        }
    }
    uint32_t* ubound_dev = tmp.take<uint32_t>(ubound.size());
    PREP_NEED(ubound_dev);
    PREP_HIP(hipMemcpyAsync(ubound_dev, ubound.data(), ubound.size() * 4, hipMemcpyHostToDevice, stream));
    if (E > 0)
        hipLaunchKernelGGL(k_emit, dim3((L->n_chunks + kChunksPerBlock - 1) / kChunksPerBlock), dim3(kBlk), 0, stream, (uint32_t)E, L->n_chunks, M, src_mask, keys,
                           L->mbase, ubound_dev, L->n_spieces, id_scale_for(rows_per_part), L->ids16, L->src16);

    // ---- what the cost model needs of every scatter tile
    L->sp.clear(); L->st.clear(); L->st_msgs.clear(); L->st_rows.clear();
    {
        std::vector<uint64_t> msgs(L->n_spieces), rows(L->n_spieces);
        for (uint32_t t = 0; t < L->n_spieces; ++t) {
            const uint64_t u0 = ubound[t], u1 = ubound[t + 1];
            uint64_t partials = 0;
            for (uint64_t j = u0 / rows_per_part; j < Q && j * rows_per_part < u1; ++j) {
                if ((L->ri[j].cls_tiles & 3u) != kRangeMerged) continue;
                const uint64_t lo = std::max<uint64_t>(u0, j * rows_per_part), hi = std::min<uint64_t>(u1, (j + 1) * (uint64_t)rows_per_part);
                partials += (hi - lo) * (L->ri[j].cls_tiles >> 2);
            }
            L->sp.push_back(ScatterPiece{(uint32_t)u0, (uint32_t)u1});
            msgs[t] = messages_before(u1) - messages_before(u0);
            rows[t] = (u1 - u0) + partials;
        }
        for (const uint2& t : stiles) {
            L->st.push_back(ScatterTile{t.x, t.y, L->sp[t.x].u0, L->sp[t.x].u1, L->ri[L->sp[t.x].u0 / rows_per_part], {0, 0}});
            uint64_t m = 0, r = 0;
            for (uint32_t i = t.x; i < t.y; ++i) { m += msgs[i]; r += rows[i]; }
            L->st_msgs.push_back(m);
            L->st_rows.push_back(r);
        }
    }
    L->n_scatter = (uint32_t)L->st.size();
    L->scatter_packed = false;
    for (const ScatterTile& t : L->st) L->scatter_packed = L->scatter_packed || t.p1 - t.p0 > 1;

    Carve tables;                                      // uploaded together
    tables.add(&L->range_info, (uint64_t)Q); tables.add(&L->gather_pieces, (uint64_t)L->n_pieces); tables.add(&L->gather_tiles, (uint64_t)L->n_gather);
    tables.add(&L->scatter_pieces, (uint64_t)L->n_spieces); tables.add(&L->scatter_tiles, (uint64_t)L->n_scatter); tables.add(&L->finish_ranges, (uint64_t)L->n_finish);
    const uint64_t table_bytes = tables.bytes;
    tables.add(&L->bins, (uint64_t)L->n_spieces * Qe);
    if (!tables.keep(a)) PREP_NEED((void*)nullptr);
    std::vector<char> packed(table_bytes, 0);
    {
        const char* base = reinterpret_cast<const char*>(L->range_info);
        auto put = [&](const void* where, const void* from, size_t bytes) {
            if (bytes) std::memcpy(packed.data() + (static_cast<const char*>(where) - base), from, bytes);
        };
        put(L->range_info, L->ri.data(), (size_t)Q * sizeof(RangeInfo));
        put(L->gather_pieces, L->gp.data(), (size_t)L->n_pieces * sizeof(GatherPiece));
        put(L->gather_tiles, L->gt.data(), (size_t)L->n_gather * sizeof(GatherTile));
        put(L->scatter_pieces, L->sp.data(), (size_t)L->n_spieces * sizeof(ScatterPiece));
        put(L->scatter_tiles, L->st.data(), (size_t)L->n_scatter * sizeof(ScatterTile));
        put(L->finish_ranges, L->fin.data(), (size_t)L->n_finish * 4);
    }
    if (Qe)
        hipLaunchKernelGGL(k_bins, dim3(blocks_for((uint64_t)L->n_spieces * Qe)), dim3(kBlk), 0, stream, L->n_spieces, Qe, E, M, src_bits, ubound_dev,
                           keys, L->starts, L->mbase, L->bins);
    PREP_HIP(hipGetLastError());
    PREP_HIP(hipMemcpyAsync(L->range_info, packed.data(), table_bytes, hipMemcpyHostToDevice, stream));
    PREP_HIP(hipStreamSynchronize(stream));       // the host vectors and `tmp` go away after this
    return FR_OK;     // `tmp` returns the scratch blocks to the allocator
}

// Internal declarations shared by the library's translation units (not part of the C ABI).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <vector>

#include "freeride.h"

// Accounting allocator handed to a task's init() (memory limit, Section 4.5 of the paper).
struct fr_alloc {
    uint64_t limit = 0;
    uint64_t used = 0;
    bool oom = false;
    bool host_only = false;
    int device = 0;
    int hip_error = 0;
    uint64_t peak = 0;
    bool pooled = false;                 // set-up scratch may come from, and go back to, the pool of kept blocks ...
    int series = -1;                     // ... if the set-up follows another one (-1: not asked yet)
    struct Block { void* ptr; uint64_t bytes; uint64_t room; bool kept; };      // room: the size of a block of a pool (0: not one); kept: of the layouts'
    std::vector<Block> blocks;
};

void fr_alloc_reset(fr_alloc* a, uint64_t limit, bool host_only, int device);
void fr_alloc_release(fr_alloc* a);   // frees every block handed out
void fr_alloc_hand_back(fr_alloc* a); // the same at the end of a task: waits for its device, and blocks of the layouts' pool go back to it
// Memory a task holds until it ends (else as fr_alloc_scratch).
void* fr_alloc_kept(fr_alloc* a, size_t bytes);
bool fr_alloc_pools(const fr_alloc* a);      // does it get blocks of the pools?  (known once it has been asked for memory)
// Memory a task needs while it is set up, and counts only that long.  Given back with fr_alloc_free, by a caller that has
// waited for the work that used it.
void* fr_alloc_scratch(fr_alloc* a, size_t bytes);

// A set-up that has a smaller layout to fall back on: fr_alloc_mark before it takes memory for the larger one; if memory runs
// out, fr_alloc_back_to (the stream has been waited for) frees what was handed out since and forgets that it ran out.
size_t fr_alloc_mark(const fr_alloc* a);
void fr_alloc_back_to(fr_alloc* a, size_t mark);

// Several arrays in one block of the allocator, each on a 256-byte boundary: what they count as is what they would as
// blocks of their own, at the price of one allocation (10 to 300 us each, and as much to give back).
struct Carve {
    uint64_t bytes = 0;
    struct Part { void** where; uint64_t at; };
    std::vector<Part> parts;
    template <typename T>
    void add(T** out, uint64_t count)
    {
        parts.push_back({reinterpret_cast<void**>(out), bytes});
        bytes += ((count ? count : 1) * sizeof(T) + 255) / 256 * 256;
    }
    void place(void* base)
    {
        for (const Part& x : parts) *x.where = static_cast<char*>(base) + x.at;
    }
    bool keep(fr_alloc* a)
    {
        void* base = fr_alloc_kept(a, (size_t)bytes);
        if (base) place(base);
        return base != nullptr;
    }
    // One block of a pool, else one each: the driver makes a small block in a few microseconds, and one of some megabytes in 300.
    bool keep_apart(fr_alloc* a)
    {
        if (fr_alloc_pools(a)) return keep(a);
        for (size_t i = 0; i < parts.size(); ++i) {
            void* p = fr_alloc_kept(a, (size_t)((i + 1 < parts.size() ? parts[i + 1].at : bytes) - parts[i].at));
            if (!p) return false;
            *parts[i].where = p;
        }
        return true;
    }
};

// Compute units that `stream` may use: those of its mask, if it has one, else all of the current device's.
uint32_t fr_stream_cus(hipStream_t stream);

// Stage-load kernels (gemm.hip).
int fr_busywait_launch(uint64_t ns, int wall_clock_khz, hipStream_t stream);
int fr_alufill_launch(uint64_t ns, int wall_clock_khz, uint32_t workgroups, hipStream_t stream);

#define FR_HIP_TRY(expr, errslot)                      \
    do {                                               \
        hipError_t e__ = (expr);                       \
        if (e__ != hipSuccess) {                       \
            (errslot) = (int)e__;                      \
            return FR_ERR_HIP;                         \
        }                                              \
    } while (0)

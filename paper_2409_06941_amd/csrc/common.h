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
    struct Block { void* ptr; uint64_t bytes; uint64_t room; };      // room: the size of a block of the pool (0: not one)
    std::vector<Block> blocks;
};

void fr_alloc_reset(fr_alloc* a, uint64_t limit, bool host_only, int device);
void fr_alloc_release(fr_alloc* a);   // frees every block handed out
// Memory a task needs while it is set up, and counts only that long.  Given back with fr_alloc_free, by a caller that has
// waited for the work that used it.
void* fr_alloc_scratch(fr_alloc* a, size_t bytes);

// A set-up that has a smaller layout to fall back on: fr_alloc_mark before it takes memory for the larger one; if memory runs
// out, fr_alloc_back_to (the stream has been waited for) frees what was handed out since and forgets that it ran out.
size_t fr_alloc_mark(const fr_alloc* a);
void fr_alloc_back_to(fr_alloc* a, size_t mark);

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

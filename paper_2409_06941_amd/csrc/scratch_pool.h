// Blocks of device memory kept between set-ups (see runtime.cpp for what they are kept for).  `Mem` is where they come from:
//   free(p), now_ns(), keep_at_most(device): bytes that may be kept on a device, and, for take_back, wait(device): is that device
//   done with all it was given?
#ifndef FR_SCRATCH_POOL_H
#define FR_SCRATCH_POOL_H

#include <cstddef>
#include <cstdint>
#include <mutex>

// The largest block that may serve a request of `bytes`: a task without a limit of its own (one beyond the device's `total`) may
// be handed up to a quarter more than it asked for; one with a limit gets the size that is booked against it, so that the limit
// holds for what is in use as well.
inline uint64_t most_room(uint64_t limit, uint64_t total, uint64_t bytes) { return total && limit >= total ? bytes + bytes / 4 : bytes; }

// Blocks of a device that each of the library's pools keeps.  A set-up has a handful of scratch blocks and a task holds five: with
// eight, graphs of two sizes in turn were enough to have each find the other's, and to free those in its own time.  ms for set-up, one
// iteration and destruction, eight blocks (and those of the scratch alone) -> 64, in turn: 2^14 vertices / 2^18 edges, 2^18 / 2^22, 2^20 / 2^24,
// 2^22 / 2^26: 2.58 (1.40) -> 0.45, 2.22 (1.82) -> 0.99, 2.88 (5.2) -> 1.92, 6.70 (9.6) -> 5.40; 2^14 / 2^18 and 2^22 / 2^26: 1.61 (1.40) -> 0.45, 5.75
// (8.2) -> 5.37; nineteen sizes from 16 000 to 2 065 395 vertices, mean 2.42 (2.78) -> 1.12 (32 blocks 1.98, 128 1.10).  What bounds the
// memory is its bytes.
constexpr size_t kKeptBlocks = 64;

template <class Mem, size_t kMostBlocks = 8>
class ScratchPool {
public:
    static constexpr size_t kBlocks = kMostBlocks;          // of a device
    static constexpr uint64_t kKeepNs = 5000000000ull;

    // A set-up begins on `device`: does it follow another one within kKeepNs?  (Only then is anything worth keeping for the next.)
    bool begins(int device)
    {
        if (device < 0 || device >= (int)(sizeof(last_) / sizeof(last_[0]))) return false;
        std::lock_guard<std::mutex> lk(mu_);
        const uint64_t now = Mem::now_ns(), last = last_[device];
        last_[device] = now ? now : 1;
        return last != 0 && now - last <= kKeepNs;
    }

    // A kept block of `bytes` to `most` bytes, the smallest there is; NULL if there is none.
    void* take(int device, uint64_t bytes, uint64_t most, uint64_t* room)
    {
        trim(false);
        std::lock_guard<std::mutex> lk(mu_);
        size_t best = n_;
        for (size_t i = 0; i < n_; ++i) {
            const Block& b = kept_[i];
            if (b.device != device || b.room < bytes || b.room > most) continue;
            if (best == n_ || b.room < kept_[best].room) best = i;
        }
        if (best == n_) return nullptr;
        *room = kept_[best].room;
        return remove(best);
    }

    void give(int device, void* ptr, uint64_t room)
    {
        trim(false);
        const uint64_t most = Mem::keep_at_most(device);
        Freed freed;
        std::lock_guard<std::mutex> lk(mu_);
        if (room > most) { freed.add(ptr); return; }
        for (;;) {
            uint64_t held = 0;
            size_t blocks = 0, oldest = n_;
            for (size_t i = n_; i-- > 0;)
                if (kept_[i].device == device) { held += kept_[i].room; ++blocks; oldest = i; }
            if (n_ < kAll && (!blocks || (blocks < kBlocks && held + room <= most))) break;
            freed.add(remove(oldest < n_ ? oldest : 0));
        }
        kept_[n_++] = {device, ptr, room, Mem::now_ns()};
    }

    // A task has ended: its blocks marked `kept` go to the pool (and their ptr to NULL), once their device is done with them -
    // theirs, which need not be the calling thread's current one.  Nothing is taken where that cannot be said.
    template <class Blocks>
    void take_back(int device, Blocks& blocks)
    {
        if (!Mem::wait(device)) return;
        for (auto& b : blocks) {
            if (!b.kept || !b.room) continue;
            give(device, b.ptr, b.room);
            b.ptr = nullptr;
        }
    }

    // Gives back what has been kept for longer than kKeepNs, or all of it; bytes given back.
    uint64_t trim(bool all)
    {
        Freed freed;
        std::lock_guard<std::mutex> lk(mu_);
        uint64_t bytes = 0;
        while (n_ && (all || Mem::now_ns() - kept_[0].since > kKeepNs)) { bytes += kept_[0].room; freed.add(remove(0)); }
        return bytes;
    }

private:
    static constexpr size_t kAll = 8 * kBlocks;             // of all devices

    struct Block { int device; void* ptr; uint64_t room, since; };

    // What left the pool under the lock, freed after it: giving memory back waits for the device.
    struct Freed {
        void* p[kAll + 1];
        size_t n = 0;
        void add(void* ptr) { p[n++] = ptr; }
        ~Freed() { for (size_t i = 0; i < n; ++i) Mem::free(p[i]); }
    };

    void* remove(size_t i)
    {
        void* p = kept_[i].ptr;
        for (--n_; i < n_; ++i) kept_[i] = kept_[i + 1];
        return p;
    }

    std::mutex mu_;
    Block kept_[kAll];                      // oldest first
    size_t n_ = 0;
    uint64_t last_[64] = {};                // when the last set-up of a device began; 0: there was none
};

#endif

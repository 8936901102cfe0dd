// Blocks of device memory kept between set-ups (see runtime.cpp for what they are kept for).  `Mem` is where they come from:
//   free(p), now_ns(), and keep_at_most(device): bytes that may be kept on a device.
#ifndef FR_SCRATCH_POOL_H
#define FR_SCRATCH_POOL_H

#include <cstddef>
#include <cstdint>
#include <mutex>
#include <vector>

// The largest block that may serve a request of `bytes`: a task without a limit of its own (one beyond the device's `total`) may
// be handed up to a quarter more than it asked for; one with a limit gets the size that is booked against it, so that the limit
// holds for what is in use as well.
inline uint64_t most_room(uint64_t limit, uint64_t total, uint64_t bytes) { return total && limit >= total ? bytes + bytes / 4 : bytes; }

template <class Mem>
class ScratchPool {
public:
    static constexpr size_t kBlocks = 8;                    // of a device
    static constexpr uint64_t kKeepNs = 5000000000ull;

    // A kept block of `bytes` to `most` bytes, the smallest there is; NULL if there is none.
    void* take(int device, uint64_t bytes, uint64_t most, uint64_t* room)
    {
        trim(false);
        std::lock_guard<std::mutex> lk(mu_);
        size_t best = kept_.size();
        for (size_t i = 0; i < kept_.size(); ++i) {
            const Block& b = kept_[i];
            if (b.device != device || b.room < bytes || b.room > most) continue;
            if (best == kept_.size() || b.room < kept_[best].room) best = i;
        }
        if (best == kept_.size()) return nullptr;
        void* p = kept_[best].ptr;
        *room = kept_[best].room;
        kept_.erase(kept_.begin() + (long)best);
        return p;
    }

    void give(int device, void* ptr, uint64_t room)
    {
        trim(false);
        const uint64_t most = Mem::keep_at_most(device);
        std::lock_guard<std::mutex> lk(mu_);
        if (room > most) { Mem::free(ptr); return; }
        for (;;) {
            uint64_t held = 0;
            size_t blocks = 0, oldest = kept_.size();
            for (size_t i = kept_.size(); i-- > 0;)
                if (kept_[i].device == device) { held += kept_[i].room; ++blocks; oldest = i; }
            if (!blocks || (blocks < kBlocks && held + room <= most)) break;
            free_locked(oldest);
        }
        kept_.push_back({device, ptr, room, Mem::now_ns()});
    }

    void trim(bool all)
    {
        std::lock_guard<std::mutex> lk(mu_);
        while (!kept_.empty() && (all || Mem::now_ns() - kept_.front().since > kKeepNs)) free_locked(0);
    }

private:
    struct Block { int device; void* ptr; uint64_t room, since; };

    void free_locked(size_t i)
    {
        Mem::free(kept_[i].ptr);
        kept_.erase(kept_.begin() + (long)i);
    }

    std::mutex mu_;
    std::vector<Block> kept_;               // oldest first
};

#endif

// idle_pool.h -- device buffers of freed jobs, kept for the next ones.
// Host code without HIP calls (the buffers are freed through a function pointer).
#pragma once
#include <cstddef>
#include <mutex>
#include <vector>

namespace fsmmc {

// One per device, shared by its contexts without an HBM budget, at most `cap` bytes: a
// buffer that does not fit beside the others takes the place of the oldest.  The last
// of those contexts to close gives everything back.  Nothing on the device may use a buffer given to the pool.
class IdlePool {
public:
    IdlePool(size_t cap, void (*free)(void*)) : cap_(cap), free_(free) {}

    void open()
    {
        std::lock_guard<std::mutex> lk(mu_);
        ++users_;
    }
    void close()
    {
        std::lock_guard<std::mutex> lk(mu_);
        if (--users_ == 0) drop(0);
    }

    // A buffer of at least `bytes` and at most a quarter more, or NULL.
    void* take(size_t bytes, size_t* got)
    {
        std::lock_guard<std::mutex> lk(mu_);
        for (size_t i = 0; i < idle_.size(); ++i) {
            const Idle b = idle_[i];
            if (b.bytes < bytes || b.bytes > bytes + bytes / 4) continue;
            idle_.erase(idle_.begin() + i);
            held_ -= b.bytes;
            *got = b.bytes;
            return b.p;
        }
        return nullptr;
    }

    // False: not kept, the caller frees it.
    bool give(void* p, size_t bytes)
    {
        std::lock_guard<std::mutex> lk(mu_);
        if (users_ == 0 || bytes > cap_) return false;
        drop(cap_ - bytes);
        idle_.push_back({p, bytes});
        held_ += bytes;
        return true;
    }

    void release()
    {
        std::lock_guard<std::mutex> lk(mu_);
        drop(0);
    }

private:
    struct Idle {
        void* p;
        size_t bytes;
    };

    // The oldest buffers go until at most `most` bytes are held.
    void drop(size_t most)
    {
        size_t n = 0;
        for (; held_ > most; ++n) {
            held_ -= idle_[n].bytes;
            free_(idle_[n].p);
        }
        idle_.erase(idle_.begin(), idle_.begin() + n);
    }

    const size_t cap_;
    void (*const free_)(void*);
    std::mutex mu_;
    std::vector<Idle> idle_;  // oldest first
    size_t held_ = 0;
    int users_ = 0;
};

}  // namespace fsmmc

// Page-locked host buffers that threads hold and give back, free of any device
// call (Mem makes and frees the memory), so that the CPU test suite can compile
// and check it on its own.
#pragma once

#include <algorithm>
#include <cstddef>
#include <mutex>
#include <vector>

namespace mcubes {
namespace host {

struct HostBuffer {
    char *host = nullptr;
    size_t cap = 0;
};

// Buffers that no thread holds.  One that a thread gives up when it ends serves
// a later thread; one that is too small is freed before a larger one is
// made, so there are never more than threads have held at one time.  Mem:
// static char *make(size_t bytes) (null: no memory) and static bool free(char *).
template <typename Mem>
class BufferPool {
  public:
    // Never destroyed: threads that outlive the process's static objects may
    // still give buffers back.
    static BufferPool &get() {
        static BufferPool *pool = new BufferPool;
        return *pool;
    }

    // A buffer of at least bytes: the smallest free one that holds them, or a
    // new one, in place of the largest free one if there is any.  False without
    // memory.
    bool take(size_t bytes, HostBuffer *out) {
        HostBuffer old;
        {
            std::lock_guard<std::mutex> lock(mu_);
            if (!free_.empty()) {
                auto best = free_.begin();
                for (auto it = free_.begin(); it != free_.end(); ++it) {
                    const bool fits = it->cap >= bytes, best_fits = best->cap >= bytes;
                    if (fits != best_fits ? fits : fits ? it->cap < best->cap : it->cap > best->cap) best = it;
                }
                old = *best;
                free_.erase(best);
            }
        }
        if (old.cap >= bytes && old.host) {
            *out = old;
            return true;
        }
        if (old.host && !Mem::free(old.host)) return false;
        const size_t want = std::max(bytes, kLeast);
        char *p = Mem::make(want);
        if (!p) return false;
        out->host = p;
        out->cap = want;
        return true;
    }

    // (called as threads end: where the list cannot grow, the buffer is lost
    // rather than the process)
    void give(const HostBuffer &b) noexcept {
        if (!b.host) return;
        try {
            std::lock_guard<std::mutex> lock(mu_);
            free_.push_back(b);
        } catch (...) {
        }
    }

    static constexpr size_t kLeast = size_t(1) << 16;

  private:
    std::mutex mu_;
    std::vector<HostBuffer> free_;
};

// The calling thread's buffer (a thread_local object), grown on demand and
// given back when the thread ends.
template <typename Mem>
class HeldBuffer {
  public:
    ~HeldBuffer() { BufferPool<Mem>::get().give(buf_); }
    // The buffer with room for bytes, or null without memory; what it held is
    // lost where it had to grow.
    char *reserve(size_t bytes) {
        if (bytes > buf_.cap) {
            BufferPool<Mem>::get().give(buf_);
            buf_ = HostBuffer{};
            if (!BufferPool<Mem>::get().take(bytes, &buf_)) return nullptr;
        }
        return buf_.host;
    }

  private:
    HostBuffer buf_;
};

}  // namespace host
}  // namespace mcubes

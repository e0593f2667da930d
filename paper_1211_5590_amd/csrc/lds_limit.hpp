// What has been allowed so far of dynamic LDS beyond 64 KB, per kernel and device: the limit belongs to a
// kernel on a device, so a second GPU of the process needs its own.  Safe with several threads.
#pragma once
#include <stddef.h>
#include <stdint.h>

#include <mutex>

namespace rnn {

class LdsRecord {
  public:
    bool covers(const void* fn, int dev, size_t bytes) {
        std::lock_guard<std::mutex> lock(mu_);
        const Entry* e = find(fn, dev);
        return e && e->fn == fn && e->bytes >= bytes;
    }
    // a full table forgets nothing and takes nothing new: the limit is then set again for each launch
    void allowed(const void* fn, int dev, size_t bytes) {
        std::lock_guard<std::mutex> lock(mu_);
        Entry* e = find(fn, dev);
        if (!e) return;
        if (e->fn != fn) *e = Entry{fn, dev, 0};
        if (bytes > e->bytes) e->bytes = bytes;
    }

  private:
    struct Entry { const void* fn; int dev; size_t bytes; };
    static constexpr unsigned N = 1024;
    // the entry of (fn, dev), or the free one where it belongs, or null
    Entry* find(const void* fn, int dev) {
        const uintptr_t h = (reinterpret_cast<uintptr_t>(fn) >> 4) * 0x9e3779b1u + (unsigned)dev * 0x85ebca6bu;
        for (unsigned i = 0; i < N; ++i) {
            Entry& e = table_[(h + i) % N];
            if (!e.fn || (e.fn == fn && e.dev == dev)) return &e;
        }
        return nullptr;
    }
    std::mutex mu_;
    Entry table_[N] = {};
};

}  // namespace rnn

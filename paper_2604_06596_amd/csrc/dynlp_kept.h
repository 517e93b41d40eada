// Memory that waits for the next context or call of the process.
//
// A context takes some forty arrays and gives them back when it is destroyed.  hipMalloc and hipFree cost 5 to 20 us each for
// small arrays, about 7 ms together for a graph of 3M vertices, and much more once a process has handed out all of the device's
// memory before: what is given back then has to be cleared before it is handed out again (50M vertices, 20 GB: 40 to 1,750 ms).
// Arrays of destroyed contexts without an allocator of their own therefore wait here, and arrays that live within one call; what a
// living context has no use for any more does not.
//   bounded     so many bytes per device and kind of memory as the caller of give() says, and kMostBlocks; what does not fit goes back
//               to the runtime at once
//   given back  when the runtime has none left (all of it, see take), and what has waited for too long (release_older)
//   streams     the caller of give() has made sure that nothing on the device uses the block any more
//   threads     one lock; calls of the runtime are made outside it
//   exceptions  none: arrays come back in destructors and behind C entries
// Measured: 3M vertices create 0.66 / 0.20 ms, destroy 5.2 / 0.01; 400,000 with 100 sweeps, whole 10.1 / 8.9 ms; 50M 188 / 179 ms,
// and 880 / 181 ms where the memory had been in use before.
//
// Runtime: void* allocate(bool pinned, size_t) (NULL: no memory), void release(bool pinned, void*), Clock::time_point now().
#pragma once

#include <stddef.h>

#include <chrono>
#include <mutex>

namespace dynlp {

template <class Runtime>
class KeptMemory {
   public:
    using Clock = std::chrono::steady_clock;
    static constexpr int kMostBlocks = 1024;  // (each allocation looks through all of them)

    explicit KeptMemory(Runtime r = Runtime()) : runtime(r) {}

    // Device memory of the current device, which is `device`, or pinned memory: a block that waits, of at least `bytes` and not much
    // more, or one of the runtime's; where that has none, it gets all that waits back first.  NULL: no memory.  *got: the block's size.
    void* take(int device, bool pinned, size_t bytes, size_t* got) {
        *got = bytes;
        {
            std::lock_guard<std::mutex> hold(lock);
            int best = -1;
            for (int i = 0; i < count; ++i) {
                const Block& b = block[i];
                if (b.device != device || b.pinned != pinned || b.bytes < bytes || b.bytes > bytes + bytes / 8 + 4096) continue;
                if (best < 0 || b.bytes < block[best].bytes) best = i;
            }
            if (best >= 0) {
                void* const p = block[best].p;
                *got = block[best].bytes;
                for (int i = best + 1; i < count; ++i) block[i - 1] = block[i];
                --count;
                return p;
            }
        }
        void* p = runtime.allocate(pinned, bytes);
        if (!p && release_older(0.f) > 0) p = runtime.allocate(pinned, bytes);
        return p;
    }

    // Keeps the block, or gives it back to the runtime where more than `most` bytes of the device's and its kind would wait.
    void give(int device, bool pinned, void* p, size_t bytes, size_t most) {
        bool kept = false;
        {
            std::lock_guard<std::mutex> hold(lock);
            size_t held = 0;
            for (int i = 0; i < count; ++i)
                if (block[i].device == device && block[i].pinned == pinned) held += block[i].bytes;
            if (count < kMostBlocks && held <= most && bytes <= most - held) {
                block[count++] = Block{p, bytes, device, pinned, runtime.now()};
                kept = true;
            }
        }
        if (!kept) runtime.release(pinned, p);
    }

    // Gives back what has waited for `ms` or more; how many bytes.
    size_t release_older(float ms) {
        size_t bytes = 0;
        for (;;) {
            Block old[32];
            int n = 0;
            {
                std::lock_guard<std::mutex> hold(lock);
                if (count == 0) break;
                const Clock::time_point now = runtime.now();
                // (oldest first)
                while (n < count && n < 32 && std::chrono::duration<float, std::milli>(now - block[n].since).count() >= ms) {
                    old[n] = block[n];
                    ++n;
                }
                for (int i = n; i < count; ++i) block[i - n] = block[i];
                count -= n;
            }
            for (int i = 0; i < n; ++i) {
                runtime.release(old[i].pinned, old[i].p);
                bytes += old[i].bytes;
            }
            if (n < 32) break;
        }
        return bytes;
    }

   private:
    struct Block {
        void* p;
        size_t bytes;
        int device;
        bool pinned;
        Clock::time_point since;
    };
    Runtime runtime;
    std::mutex lock;
    Block block[kMostBlocks];  // the first `count`, oldest first
    int count = 0;
};

}  // namespace dynlp

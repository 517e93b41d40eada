// The list of memory that waits between contexts (csrc/dynlp_kept.h, the code the library runs), on the host, with a runtime and a
// clock of its own.  Prints "ok" or the line that is not met.
#include <cstdio>
#include <cstdlib>
#include <map>
#include <thread>
#include <vector>

#include "dynlp_kept.h"

using namespace dynlp;

namespace {

struct World {
    std::mutex lock;
    std::map<void*, size_t> out[2];  // what the runtime has handed out
    size_t room = (size_t)1 << 40, used = 0;
    int allocations = 0, releases = 0;
    double ms = 0.0;
} w;

struct Runtime {
    void* allocate(bool pinned, size_t bytes) {
        std::lock_guard<std::mutex> hold(w.lock);
        if (bytes > w.room - w.used) return nullptr;
        void* const p = std::malloc(1);
        w.out[pinned][p] = bytes;
        w.used += bytes;
        ++w.allocations;
        return p;
    }
    void release(bool pinned, void* p) {
        std::lock_guard<std::mutex> hold(w.lock);
        if (!w.out[pinned].count(p)) {
            std::printf("a block that was not handed out, or of the other kind, is released\n");
            std::exit(1);
        }
        w.used -= w.out[pinned][p];
        w.out[pinned].erase(p);
        std::free(p);
        ++w.releases;
    }
    std::chrono::steady_clock::time_point now() {
        return std::chrono::steady_clock::time_point(std::chrono::microseconds((long long)(w.ms * 1000.0)));
    }
};

KeptMemory<Runtime> g_kept;  // (large)

#define CHECK(x)                                              \
    do {                                                      \
        if (!(x)) {                                           \
            std::printf("line %d: %s\n", __LINE__, #x);       \
            std::exit(1);                                     \
        }                                                     \
    } while (0)

constexpr size_t MB = (size_t)1 << 20, kAny = (size_t)1 << 50;
size_t got;

void* fresh(size_t bytes, bool pinned = false, int device = 0) { return g_kept.take(device, pinned, bytes, &got); }

void sizes_kinds_and_devices() {
    void* const p = fresh(10 * MB);
    CHECK(p && got == 10 * MB);
    g_kept.give(0, false, p, got, kAny);
    const int before = w.allocations;
    void* q = fresh(10 * MB, true);  // of the other kind
    CHECK(q != p);
    g_kept.give(0, true, q, got, 0);
    q = fresh(10 * MB, false, 1);  // of another device
    CHECK(q != p);
    g_kept.give(1, false, q, got, 0);
    q = fresh(10 * MB + 1);  // too small
    CHECK(q != p);
    g_kept.give(0, false, q, got, 0);
    q = fresh(8 * MB);  // much too large: an eighth and a page more at most
    CHECK(q != p);
    g_kept.give(0, false, q, got, 0);
    CHECK(w.allocations == before + 4);
    q = fresh(9 * MB);
    CHECK(q == p && got == 10 * MB && w.allocations == before + 4);
    void* const r = fresh(9 * MB + 100);
    g_kept.give(0, false, q, 10 * MB, kAny);
    g_kept.give(0, false, r, 9 * MB + 100, kAny);
    CHECK(fresh(9 * MB) == r && got == 9 * MB + 100);  // the smallest that is large enough
    CHECK(fresh(9 * MB) == q);
    g_kept.give(0, false, q, 10 * MB, 0);
    g_kept.give(0, false, r, 9 * MB + 100, 0);
    CHECK(w.used == 0);
}

void bounds() {
    std::vector<void*> p;
    for (int i = 0; i < 6; ++i) p.push_back(fresh(2 * MB));
    for (int i = 0; i < 6; ++i) g_kept.give(0, false, p[(size_t)i], 2 * MB, 7 * MB);
    CHECK(w.used == 6 * MB);  // three of them; what does not fit went back at once
    void* const q = fresh(1 * MB);
    g_kept.give(0, false, q, 1 * MB, 7 * MB);
    CHECK(w.used == 7 * MB);
    // another kind and another device have bounds of their own
    void* const r = fresh(5 * MB, true);
    g_kept.give(0, true, r, 5 * MB, 7 * MB);
    void* const s = fresh(5 * MB, false, 3);
    g_kept.give(3, false, s, 5 * MB, 7 * MB);
    CHECK(w.used == 17 * MB);
    // a smaller bound than what waits already
    void* const t = fresh(4096);
    g_kept.give(0, false, t, 4096, 1 * MB);
    CHECK(w.used == 17 * MB);
    CHECK(g_kept.release_older(0.f) == 17 * MB && w.used == 0 && g_kept.release_older(0.f) == 0);
    // and so many blocks
    p.clear();
    for (int i = 0; i < KeptMemory<Runtime>::kMostBlocks + 40; ++i) p.push_back(fresh(256));
    for (void* x : p) g_kept.give(0, false, x, 256, kAny);
    CHECK(w.used == 256u * KeptMemory<Runtime>::kMostBlocks);
    CHECK(g_kept.release_older(0.f) == 256u * KeptMemory<Runtime>::kMostBlocks && w.used == 0);
}

void age() {
    void* const p = fresh(2 * MB);
    void* const q = fresh(3 * MB);
    void* const r = fresh(9 * MB);
    g_kept.give(0, false, p, 2 * MB, kAny);
    w.ms += 6000.0;
    g_kept.give(0, false, q, 3 * MB, kAny);
    g_kept.give(0, false, r, 9 * MB, kAny);
    CHECK(g_kept.release_older(10000.f) == 0);
    w.ms += 5000.0;
    CHECK(fresh(9 * MB) == r);
    g_kept.give(0, false, r, 9 * MB, kAny);  // (waits anew)
    CHECK(g_kept.release_older(10000.f) == 2 * MB && w.used == 12 * MB);
    w.ms += 5000.0;
    CHECK(g_kept.release_older(10000.f) == 3 * MB && w.used == 9 * MB);
    w.ms += 5000.0;
    CHECK(g_kept.release_older(10000.f) == 9 * MB && w.used == 0);
}

void no_memory_left() {
    void* const p = fresh(40 * MB);
    void* const q = fresh(50 * MB, true);
    g_kept.give(0, false, p, 40 * MB, kAny);
    g_kept.give(0, true, q, 50 * MB, kAny);
    w.room = 100 * MB;
    void* const r = fresh(70 * MB);  // not without what waits
    CHECK(r && w.used == 70 * MB);
    const int releases = w.releases;
    CHECK(!fresh(70 * MB) && w.releases == releases);
    g_kept.give(0, false, r, 70 * MB, kAny);
    CHECK(fresh(90 * MB, true) && w.used == 90 * MB);  // pinned memory likewise
    w.room = (size_t)1 << 40;
}

void threads() {
    std::vector<std::thread> all;
    for (int k = 0; k < 4; ++k)
        all.emplace_back([k] {
            for (int i = 0; i < 20000; ++i) {
                size_t n = 0;
                void* const p = g_kept.take(0, false, (size_t)(1 + (i * 7 + k) % 50) * 4096, &n);
                if (!p) std::exit(1);
                g_kept.give(0, false, p, n, MB);
                if (i % 97 == 0) (void)g_kept.release_older(0.f);
            }
        });
    for (std::thread& t : all) t.join();
    (void)g_kept.release_older(0.f);
    CHECK(w.out[0].empty());
}

}  // namespace

int main() {
    sizes_kinds_and_devices();
    bounds();
    age();
    threads();
    no_memory_left();
    std::printf("ok\n");
    return 0;
}

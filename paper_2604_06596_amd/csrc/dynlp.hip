// libdynlp: host side of the DynLP library (context, memory, launch sequencing, C ABI).
// Every step of the path runs in the kernels of dynlp_kernels.h; there is no CPU fallback.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <chrono>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <limits>
#include <mutex>
#include <new>
#include <string>
#include <thread>
#include <type_traits>
#include <unordered_map>
#include <unordered_set>
#include <vector>

#include "dynlp.h"
#include "dynlp_kernels.h"
#include "dynlp_conjugate.h"
#include "dynlp_frontier.h"
#include "dynlp_components.h"
#include "dynlp_binned.h"
#include "dynlp_insert.h"
#include "dynlp_kept.h"
#include "dynlp_packed.h"
#include "dynlp_small.h"
#include "dynlp_xcd.h"

using namespace dynlp;

namespace {

thread_local std::string g_create_error;

inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }
inline int64_t round_up(int64_t a, int64_t b) { return ceil_div(a, b) * b; }

int padded_classes(int C) {
    if (C <= 1) return 1;
    if (C <= 2) return 2;
    if (C <= 4) return 4;
    if (C <= 8) return 8;
    if (C <= 16) return 16;
    if (C <= 32) return 32;
    return 64;
}

const char* validation_message(int code) {
    switch (code) {
        case kErrRowPtr: return "row_ptr must start at 0, be non-decreasing and end at the entry count (row index %lld)";
        case kErrColRange: return "neighbour id out of range (entry %lld)";
        case kErrSelfLoop: return "self loop (item %lld)";
        case kErrWeight: return "weight must be finite and > 0 (item %lld)";
        case kErrSeedVertex: return "seed vertex out of range (seed %lld)";
        case kErrSeedClass: return "seed class out of range (seed %lld)";
        case kErrSeedConflict: return "one vertex listed with two different classes (seed %lld)";
        case kErrEndpoint: return "edge endpoint out of range (edge %lld)";
        case kErrRelabel: return "vertex is already a seed of another class (seed %lld)";
        case kErrDeleted: return "deleted vertex out of range (item %lld)";
        default: return "validation error %lld";
    }
}

using Clock = std::chrono::steady_clock;
inline float ms_since(Clock::time_point t0) {
    return std::chrono::duration<float, std::milli>(Clock::now() - t0).count();
}

}  // namespace

// Staging area of dynlp_get_labels_static: device memory that exists without any allocation call.  Every GPU
// the library runs on holds its own copy, at its own address, until the process ends.  In host code the name
// `scratch` is only a handle for hipGetSymbolAddress; kernels and copies take the resolved per-device address.
constexpr size_t kStaticScratchBytes = DYNLP_STATIC_SCRATCH_BYTES;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices] = {};        // device address of `scratch` on each device, once resolved
hipError_t g_scratch_err[kMaxDevices] = {};   // what the resolution returned there

// Resolve the address of `scratch` on `device` (which must be the current device).  Once per device.
void resolve_static_scratch(int device) {
    if (device < 0 || device >= kMaxDevices) return;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (g_scratch_ptr[device]) return;
    void* ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    g_scratch_err[device] = e;
    if (e == hipSuccess) g_scratch_ptr[device] = ptr;
    else (void)hipGetLastError();
}

// Calls of this process at work on a device, and when two of them last were at the same time.
struct CallsAtWork {
    std::atomic<int> now{0};
    std::atomic<Clock::rep> together{Clock::time_point::min().time_since_epoch().count()};
};
CallsAtWork g_at_work[kMaxDevices];
constexpr float kTogetherMs = 100.f;

class AtWork {
    CallsAtWork* on;

   public:
    explicit AtWork(int device) : on(device >= 0 && device < kMaxDevices ? &g_at_work[device] : nullptr) {
        if (on && on->now.fetch_add(1) > 0) on->together = Clock::now().time_since_epoch().count();
    }
    ~AtWork() {
        if (on && on->now.fetch_sub(1) > 1) on->together = Clock::now().time_since_epoch().count();
    }
    AtWork(const AtWork&) = delete;
    AtWork& operator=(const AtWork&) = delete;
};

// Whether other contexts have work for the device, as far as that can be told: a program that makes its calls one after the other
// has one at a time, whatever contexts it holds.
bool others_at_work(int device) {
    if (device < 0 || device >= kMaxDevices) return true;
    if (g_at_work[device].now > 1) return true;
    const Clock::rep then = g_at_work[device].together;
    return then > (Clock::now() - std::chrono::microseconds((int64_t)(kTogetherMs * 1000.f))).time_since_epoch().count();
}

}  // namespace

struct dynlp_ctx {
    int device = 0;
    hipStream_t stream = nullptr;
    bool dev_ptrs = false;
    float slack = 1.25f;
    bool time_kernels = false;
    int group_lanes = 0;
    std::unordered_map<void*, size_t> live;  // every device array handed out by dev_alloc and not yet freed, and its bytes:
                                             // whatever an error path left behind goes back when the context is destroyed
    bool idle = false;  // nothing of this context is running or will be launched: its arrays may go to another one at once
    void* (*alloc_fn)(size_t, void*) = nullptr;
    void (*dealloc_fn)(void*, void*) = nullptr;
    void* alloc_user = nullptr;
    int num_cu = 256;

    int C = 0, CP = 0;
    int Cs = 0, coff = 0;  // stored columns and the class of stored column 0 (binary scalar layout: 1, 1)
    int64_t n = 0, n_cap = 0, flag_cap = 0;
    int64_t entries = 0;  // directed CSR entries stored
    RowMeta* meta = nullptr;
    Edge* pool = nullptr;
    int64_t pool_cap = 0, pool_tail = 0;
    float* F = nullptr;   // current labels, n_cap x CP
    float* F2 = nullptr;  // second buffer: ping-pong partner (static) / staging by queue position (dynamic)
    int32_t* seed_class = nullptr;
    uint8_t* flag = nullptr;
    int32_t* queue[3] = {nullptr, nullptr, nullptr};  // frontier storage: two parities + the list of all
                                                      // updatable vertices (see dynlp_frontier.h)
    int32_t* add_cnt = nullptr;
    float* deg = nullptr;
    unsigned int* moved[3] = {nullptr, nullptr, nullptr};  // 1 bit per vertex: "moved by > tol" of ping-pong rounds;
    int64_t moved_words = 0;                                // round t of a stretch reads t-1's, sets t's, clears t+1's

    int32_t* touched = nullptr;
    int64_t* reloc_off = nullptr;
    int32_t* he_rank = nullptr;  // per half-edge of the batch: its place among the entries appended to its row (or NULL)
    int64_t he_rank_cap = 0;
    int64_t touched_cap = 0;
    int32_t *b_eu = nullptr, *b_ev = nullptr, *b_sv = nullptr, *b_sc = nullptr;
    float* b_ew = nullptr;
    int64_t b_edge_cap = 0, b_seed_cap = 0;
    int32_t* b_del = nullptr;
    int64_t b_del_cap = 0;
    // small calls with host arrays: pinned memory that all inputs are gathered in for one copy (to d_io), and that the label
    // kernel writes to over the bus
    unsigned char *h_io = nullptr, *d_io = nullptr;
    int64_t h_io_cap = 0, d_io_cap = 0;

    // pipelined ingest of host-resident batches (see ingest_edges)
    int64_t ingest_chunk = 0;            // edges per chunk
    hipStream_t copy_stream = nullptr;   // default priority, used only for the batch's host-to-device copies
    hipEvent_t ingest_ev[2] = {nullptr, nullptr};
    void* bounce[2] = {nullptr, nullptr};  // pinned staging for callers whose arrays are pageable, 12 bytes per chunk edge
    int64_t bounce_edges = 0;
    int ingest_chunks_last = 0, ingest_pinned_last = 0;  // what the last batch's ingest did (inspection)

    RoundCtr* ring = nullptr;  // kRing round slots + the start slot
    BatchCtr* bc = nullptr;
    RoundCtr* h_slot = nullptr;  // pinned, kRing slots
    unsigned int h_slot_start_long = 0;  // long rows among the updatable vertices of the running static solve
    struct HostStart {
        RoundCtr start;
        BatchCtr bc;
    }* h_start = nullptr;        // pinned: the start slot and the batch counters, which lie behind it on the device too
    BatchCtr* h_bc = nullptr;    // (in h_start)
    unsigned int* h_flag = nullptr;  // pinned: number of the last k_to_host that has arrived
    unsigned int h_sent = 0;         // ... that was launched
    void* h_fixed = nullptr;         // the one pinned allocation that h_slot, h_start, h_flag and h_xcd lie in
    size_t h_fixed_bytes = 0;
    // rounds of small graphs on one XCD (dynlp_xcd.h)
    XcdCtl* xcd = nullptr;
    XcdResult* h_xcd = nullptr;      // pinned
    unsigned int xcd_launches = 0;   // numbers them
    int xcd_groups = 0;              // dynlp_set_shared_rounds, and launches asked for since
    int64_t xcd_from = 0, xcd_asked = 0;

    int update_mode = DYNLP_UPDATE_SYNCHRONOUS;
    bool final_check = false;  // dynlp_set_final_check
    // several rounds per launch (k_rounds_persistent)
    int persist = 0;                  // option: 1 = whenever a stretch allows it, 0 / -1 = never
    unsigned int persist_spin = 1u << 20;  // polls a workgroup waits at the grid barrier before it gives up
    unsigned int* persist_ctl = nullptr;   // device: the words of the grid barrier (kBarWords; [1] = "given up")
    bool persist_failed = false;      // a launch was refused or a barrier was given up: ordinary launches from then on
    int persist_launches_last = 0, persist_aborts_last = 0;  // of the last batch (inspection)
    // binned rounds for scalar labels (dynlp_binned.h)
    int binned = 0;                 // option: 0 = automatic, -1 = never, 8..15 = always, with this many bin bits
    bool pb_built = false;          // the arrays below describe the graph as it stands
    int pb_bits = 0, pb_bins = 0;
    // per stored entry, rows in vertex order
    unsigned int* pb_src = nullptr;    // its row
    unsigned int* pb_sp = nullptr;     // row as an offset from pb_row0 of its chunk << 16 | pb_lpos: what the scatter pass reads
    unsigned int* pb_row0 = nullptr;   // per chunk: the row of its first entry; [chunk capacity]: "an offset needs > 16 bits"
    bool pb_packed_ok = false;
    unsigned short* pb_lpos = nullptr;  // its position in its chunk once sorted by slot
    float* pb_tmp = nullptr;           // build scratch: the entries' weights in stream order
    // per slot
    unsigned short* pb_dst = nullptr;
    float* pb_wn = nullptr;
    unsigned int* pb_val = nullptr;
    int64_t pb_ent_cap = 0;
    int pb_chunks = 0;
    // per vertex
    int32_t* pb_len = nullptr;
    unsigned int* pb_upd = nullptr;
    unsigned int* pb_first = nullptr;  // (+1) first entry of the row in the stream
    unsigned int* pb_block = nullptr;  // per kBlock vertices: scan scratch
    int64_t pb_vcap = 0;
    unsigned int* pb_bin = nullptr;  // bin_count | bin_off (+1), kPbMaxBins + 1 each
    unsigned int* pb_table = nullptr;  // entries per (chunk, bin) during the build
    int64_t pb_table_cap = 0;
    // in-place mode: the vertices are cut into pb_parts ranges of whole bins that are updated one after the other
    // within a round (range i: bins [pb_part_bin[i], pb_part_bin[i+1]), its rows' entries lie in chunks
    // [pb_part_chunk[i][0], pb_part_chunk[i][1]))
    int pb_parts = 1;
    int pb_part_bin[kPbMaxParts + 1] = {};
    int pb_part_chunk[kPbMaxParts][2] = {};
    // packed rounds for label rows (dynlp_packed.h)
    bool pk_built = false;  // the arrays below describe the graph as it stands
    int pk_rows = 0, pk_parts = 0, pk_bits = 0;  // vertices per part, parts, bits of a neighbour id in an entry
    PkEntry* pk_ent = nullptr;
    int64_t pk_ent_cap = 0;
    int32_t* pk_len = nullptr;
    int64_t pk_vcap = 0;
    float* pk_deg = nullptr;         // degrees the weights are divided by
    unsigned int* pk_tab = nullptr;  // per part its first entry, and all entries; most entries and rows of a part, the
                                     // longest row; per part its first row / 32, and the last; build scratch
    int64_t pk_tab_cap = 0;
    // conjugate rounds (dynlp_conjugate.h)
    float *cg_z = nullptr, *cg_p = nullptr;
    int64_t cg_cap = 0;             // floats in each
    int cg_idle = 0;                // calls in a row that had no use for them
    CgSlot* cg_ring = nullptr;      // kCgRing slots
    CgSlot* h_cg = nullptr;         // pinned, kChain slots
    // label initialisation of inserted vertices (dynlp_components.h)
    int init_mode = DYNLP_INIT_UNIFORM;
    float tau = 0.f;
    int32_t *cc_par = nullptr, *cc_dense = nullptr, *cc_comp = nullptr;
    unsigned int* cc_block = nullptr;
    int64_t cc_vcap = 0;
    int2* cc_kept = nullptr;
    int64_t cc_ecap = 0;
    double* cc_W = nullptr;
    int64_t cc_wcap = 0;
    InitCtr* cc_ctr = nullptr;  // device
    InitCtr* h_cc = nullptr;    // pinned
    hipEvent_t init_ev[2] = {nullptr, nullptr};
    dynlp_init_info last_init = {};  // of the last dynlp_apply_batch; vertices == 0: nothing to report

    float tol = 1e-4f;
    int32_t max_iter = 100000;
    std::vector<dynlp_round_info> log;  // one entry per round of the last solve / batch
    std::vector<hipEvent_t> events;   // pairs: events[2k], events[2k+1] bracket the k-th timed launch
    size_t events_used = 0;               // 2 x the number of timed spans
    size_t events_next = 0;               // events handed out (a span that directly follows another shares its event)
    std::vector<int> ev_first, ev_last;   // event indices of span k
    bool ev_adjacent = false;             // set by a caller: nothing was queued since the previous span was closed
    std::vector<int> ev_round, ev_count;  // rounds [ev_round[k], ev_round[k] + ev_count[k]) ran inside the k-th launch;
                                          // ev_round[k] < 0: the launch found nothing to do (queued past the end)
    int clock_khz = 0;  // of wall_clock64
    std::string err;
    bool poisoned = false;
};

namespace {

struct Fail {
    dynlp_status st;
};

#define HIPCHK(ctx, expr)                                                                              \
    do {                                                                                               \
        hipError_t _e = (expr);                                                                        \
        if (_e != hipSuccess) {                                                                        \
            (ctx)->err = std::string("HIP error: ") + hipGetErrorString(_e) + " in " #expr;            \
            (ctx)->poisoned = true;                                                                    \
            throw Fail{_e == hipErrorOutOfMemory ? DYNLP_ERR_OOM : DYNLP_ERR_DEVICE};                   \
        }                                                                                              \
    } while (0)

// ---- memory between contexts (dynlp_kept.h) --------------------------------------------------------
struct HipMemory {
    void* allocate(bool pinned, size_t bytes) {
        void* p = nullptr;
        if ((pinned ? hipHostMalloc(&p, bytes, hipHostMallocDefault) : hipMalloc(&p, bytes)) == hipSuccess) return p;
        (void)hipGetLastError();
        return nullptr;
    }
    void release(bool pinned, void* p) { (void)(pinned ? hipHostFree(p) : hipFree(p)); }
    std::chrono::steady_clock::time_point now() { return std::chrono::steady_clock::now(); }
};
KeptMemory<HipMemory> g_kept;
constexpr float kKeepMs = 10000.f;  // looked at by each create, destroy, solve and batch
constexpr size_t kKeepPinned = (size_t)16 << 20;

// Bytes of device memory that may wait: an eighth of the device's.
size_t kept_device_bytes(int device) {
    static std::atomic<size_t> known[kMaxDevices];
    const bool listed = device >= 0 && device < kMaxDevices;
    if (listed && known[device] > 0) return known[device];
    size_t free_bytes = 0, total = 0;
    if (hipMemGetInfo(&free_bytes, &total) != hipSuccess) {  // (of the current device, which is the context's)
        (void)hipGetLastError();
        return 0;
    }
    if (listed) known[device] = total / 8;
    return total / 8;
}

// NULL when the allocator has no memory left (nothing else changes).
void* dev_try_alloc(dynlp_ctx* c, size_t bytes) {
    if (bytes == 0) bytes = 256;
    void* const p = c->alloc_fn ? c->alloc_fn(bytes, c->alloc_user) : g_kept.take(c->device, false, bytes, &bytes);
    if (p) c->live.emplace(p, bytes);
    return p;
}

// Pinned memory, kept between contexts likewise.  *got: its size, at least `bytes`; pinned_free needs it.
void* pinned_try_alloc(dynlp_ctx* c, size_t bytes, size_t* got) { return g_kept.take(c->device, true, bytes, got); }

// As pinned_try_alloc, for an array that a call cannot do without.
void* pinned_alloc(dynlp_ctx* c, size_t bytes, size_t* got) {
    void* const p = pinned_try_alloc(c, bytes, got);
    if (!p) {
        c->err = "allocation of " + std::to_string(bytes) + " bytes of pinned memory failed";
        c->poisoned = true;
        throw Fail{DYNLP_ERR_OOM};
    }
    return p;
}

void pinned_free(dynlp_ctx* c, void* p, size_t bytes) {  // (nothing of the context is running)
    if (p) g_kept.give(c->device, true, p, bytes, kKeepPinned);
}

void free_binned(dynlp_ctx* c);
void free_packed(dynlp_ctx* c);
void free_conjugate(dynlp_ctx* c);

// As dev_try_alloc, for an array that a call cannot do without: the arrays of the binned, packed and conjugate rounds, which
// only save time and are laid out again by the next solve or batch that wants them, give way to it.  (Called outside of
// rounds.)
void* dev_alloc_or_reclaim(dynlp_ctx* c, size_t bytes) {
    void* p = dev_try_alloc(c, bytes);
    // (an allocator of the context's own may stand on the same device)
    if (!p && c->alloc_fn && g_kept.release_older(0.f) > 0) p = dev_try_alloc(c, bytes);
    if (p || (!c->pk_ent && !c->pb_src && !c->cg_z)) return p;
    (void)hipStreamSynchronize(c->stream);
    free_packed(c);
    free_binned(c);
    free_conjugate(c);
    return dev_try_alloc(c, bytes);
}

void* dev_alloc(dynlp_ctx* c, size_t bytes) {
    void* p = dev_alloc_or_reclaim(c, bytes);
    if (!p) {
        c->err = "device allocation of " + std::to_string(bytes) + " bytes failed";
        c->poisoned = true;
        throw Fail{DYNLP_ERR_OOM};
    }
    return p;
}

// Ends the life of an array; 0: it is none that dev_try_alloc handed out and that has not been freed yet, or its allocator has it
// back; else its bytes.
size_t dev_forget(dynlp_ctx* c, void* p) {
    const auto it = p ? c->live.find(p) : c->live.end();
    if (it == c->live.end()) return 0;
    const size_t bytes = it->second;
    c->live.erase(it);
    if (!c->dealloc_fn) return bytes;
    c->dealloc_fn(p, c->alloc_user);
    return 0;
}

// The memory goes back to the device; where the context is being destroyed, it may wait for the next one.
void dev_free(dynlp_ctx* c, void* p) {
    if (const size_t bytes = dev_forget(c, p)) g_kept.give(c->device, false, p, bytes, c->idle ? kept_device_bytes(c->device) : 0);
}

// An array that lives within a call and that the next such call takes again (2^28 half-edges of a batch: 2.5 GB): waits likewise.
void scratch_free(dynlp_ctx* c, void* p) {
    const size_t bytes = dev_forget(c, p);
    if (!bytes) return;
    const bool dry = hipStreamSynchronize(c->stream) == hipSuccess && (!c->copy_stream || hipStreamSynchronize(c->copy_stream) == hipSuccess);
    g_kept.give(c->device, false, p, bytes, dry ? kept_device_bytes(c->device) : 0);
    (void)g_kept.release_older(kKeepMs);
}

template <typename T>
T* dev_alloc_n(dynlp_ctx* c, int64_t count) {
    return static_cast<T*>(dev_alloc(c, (size_t)std::max<int64_t>(count, 1) * sizeof(T)));
}

// Temporary device array of a call that does not change the context: when the allocator has no memory the call
// ends with DYNLP_ERR_OOM and the context stays usable (nothing in it has changed); freed on scope exit.
struct SoftOom {};
template <typename T>
struct Temp {
    dynlp_ctx* c;
    T* ptr = nullptr;
    Temp(dynlp_ctx* ctx, int64_t count) : c(ctx) {
        ptr = static_cast<T*>(dev_alloc_or_reclaim(c, (size_t)std::max<int64_t>(count, 1) * sizeof(T)));
        if (!ptr) {
            c->err = "device allocation of " + std::to_string((size_t)std::max<int64_t>(count, 1) * sizeof(T)) +
                     " bytes failed (the context is unchanged)";
            throw SoftOom{};
        }
    }
    ~Temp() { dev_free(c, ptr); }
    Temp(const Temp&) = delete;
    Temp& operator=(const Temp&) = delete;
    T* release() {
        T* p = ptr;
        ptr = nullptr;
        return p;
    }
};

inline unsigned int grid_for(int64_t items) { return (unsigned int)std::max<int64_t>(1, ceil_div(items, kBlock)); }

// A device array argument: either the caller's device pointer, or a temporary device copy of the
// caller's host array (freed by the destructor).
template <typename T>
struct DevIn {
    dynlp_ctx* c;
    const T* ptr = nullptr;
    T* owned = nullptr;
    DevIn(dynlp_ctx* ctx, const T* src, int64_t count) : c(ctx) {
        if (count <= 0 || !src) return;
        if (c->dev_ptrs) {
            ptr = src;
        } else {
            owned = dev_alloc_n<T>(c, count);
            HIPCHK(c, hipMemcpyAsync(owned, src, (size_t)count * sizeof(T), hipMemcpyHostToDevice, c->stream));
            ptr = owned;
        }
    }
    ~DevIn() {
        if (owned) {
            (void)hipStreamSynchronize(c->stream);
            scratch_free(c, owned);
        }
    }
};

void read_bc(dynlp_ctx* c) {
    HIPCHK(c, hipMemcpyAsync(c->h_bc, c->bc, sizeof(BatchCtr), hipMemcpyDeviceToHost, c->stream));
    HIPCHK(c, hipStreamSynchronize(c->stream));
}

void write_bc(dynlp_ctx* c) {
    HIPCHK(c, hipMemcpyAsync(c->bc, c->h_bc, sizeof(BatchCtr), hipMemcpyHostToDevice, c->stream));
    HIPCHK(c, hipStreamSynchronize(c->stream));
}

// How long the counters are polled for before the runtime waits for the stream.  After kPollAloneMs (more than a chain of
// short rounds takes, so that the few microseconds between looks do not show) the thread offers its core to others every 64 polls:
// programs with more contexts than cores have use for it.
constexpr float kPollMs = 20.f, kPollAloneMs = 0.2f;

// Waits for a kernel that ends by setting the flag (k_to_host, k_xcd_rounds), the last work of the stream.
void wait_for_flag(dynlp_ctx* c, unsigned int value) {
    // the flag comes with the last work of the stream, so the wait ends when that does; an error of the device, after which
    // the flag may never come, shows in the state of the stream
    auto arrived = [&]() { return __atomic_load_n(c->h_flag, __ATOMIC_ACQUIRE) == value; };
    const auto t0 = Clock::now();
    for (unsigned int polls = 0; !arrived(); ++polls) {
        if (polls % 64 != 63) {
            __builtin_ia32_pause();
            continue;
        }
        const float waited = ms_since(t0);
        if (waited < kPollMs) {
            if (waited > kPollAloneMs) std::this_thread::yield();
            continue;
        }
        // (not a chain of rounds of a graph that waits show on: let the runtime wait)
        HIPCHK(c, hipStreamSynchronize(c->stream));
        if (!arrived()) {
            c->err = "internal error: the counters did not arrive";
            c->poisoned = true;
            throw Fail{DYNLP_ERR_DEVICE};
        }
    }
}

// Device records (whole multiples of 16 bytes, in up to two runs) to pinned host memory; waits for them, and with that for
// everything the stream holds.
void read_to_host(dynlp_ctx* c, void* to, const void* a, size_t bytes_a, const void* b = nullptr, size_t bytes_b = 0) {
    const unsigned int value = ++c->h_sent;
    hipLaunchKernelGGL(k_to_host, dim3(1), dim3(kBlock), 0, c->stream, static_cast<const uint4*>(a), (unsigned int)(bytes_a / 16),
                       static_cast<const uint4*>(b), (unsigned int)(bytes_b / 16), static_cast<uint4*>(to), c->h_flag, value);
    HIPCHK(c, hipGetLastError());
    wait_for_flag(c, value);
}

std::string format_validation(int code, long long index) {
    char buf[256];
    std::snprintf(buf, sizeof buf, validation_message(code), index);
    return buf;
}

// ---- vertex-indexed arrays --------------------------------------------------------------------
void alloc_vertex_arrays(dynlp_ctx* c, int64_t new_cap) {
    const int64_t old_n = c->n;
    const int64_t flag_cap = round_up(new_cap, 4 * kFlagsPerBlock) + 4 * kFlagsPerBlock;
    RowMeta* meta = dev_alloc_n<RowMeta>(c, new_cap);
    float* F = dev_alloc_n<float>(c, new_cap * c->CP);
    float* F2 = dev_alloc_n<float>(c, new_cap * c->CP);
    int32_t* sc = dev_alloc_n<int32_t>(c, new_cap);
    uint8_t* flag = dev_alloc_n<uint8_t>(c, flag_cap);
    int32_t* q0 = dev_alloc_n<int32_t>(c, new_cap);
    int32_t* q1 = dev_alloc_n<int32_t>(c, new_cap);
    int32_t* q2 = dev_alloc_n<int32_t>(c, new_cap);
    int32_t* add = dev_alloc_n<int32_t>(c, new_cap);
    float* deg = dev_alloc_n<float>(c, new_cap);
    const int64_t moved_words = (new_cap + 31) / 32 + 64;
    unsigned int* mv0 = dev_alloc_n<unsigned int>(c, moved_words);
    unsigned int* mv1 = dev_alloc_n<unsigned int>(c, moved_words);
    unsigned int* mv2 = dev_alloc_n<unsigned int>(c, moved_words);
    HIPCHK(c, hipMemsetAsync(flag, 0, (size_t)flag_cap, c->stream));
    HIPCHK(c, hipMemsetAsync(add, 0, (size_t)new_cap * sizeof(int32_t), c->stream));
    if (old_n > 0 && c->meta) {
        HIPCHK(c, hipMemcpyAsync(meta, c->meta, (size_t)old_n * sizeof(RowMeta), hipMemcpyDeviceToDevice, c->stream));
        HIPCHK(c, hipMemcpyAsync(F, c->F, (size_t)old_n * c->CP * sizeof(float), hipMemcpyDeviceToDevice, c->stream));
        HIPCHK(c, hipMemcpyAsync(sc, c->seed_class, (size_t)old_n * sizeof(int32_t), hipMemcpyDeviceToDevice, c->stream));
        HIPCHK(c, hipMemcpyAsync(deg, c->deg, (size_t)old_n * sizeof(float), hipMemcpyDeviceToDevice, c->stream));
    }
    HIPCHK(c, hipStreamSynchronize(c->stream));
    dev_free(c, c->meta);
    dev_free(c, c->F);
    dev_free(c, c->F2);
    dev_free(c, c->seed_class);
    dev_free(c, c->flag);
    dev_free(c, c->queue[0]);
    dev_free(c, c->queue[1]);
    dev_free(c, c->queue[2]);
    dev_free(c, c->add_cnt);
    dev_free(c, c->deg);
    dev_free(c, c->moved[0]);
    dev_free(c, c->moved[1]);
    dev_free(c, c->moved[2]);
    c->moved[0] = mv0;
    c->moved[1] = mv1;
    c->moved[2] = mv2;
    c->moved_words = moved_words;
    c->meta = meta;
    c->F = F;
    c->F2 = F2;
    c->seed_class = sc;
    c->flag = flag;
    c->queue[0] = q0;
    c->queue[1] = q1;
    c->queue[2] = q2;
    c->add_cnt = add;
    c->deg = deg;
    c->n_cap = new_cap;
    c->flag_cap = flag_cap;
}

// must: no memory is the end of the context; else the pool stays as it is and the result is false.
bool grow_pool(dynlp_ctx* c, int64_t min_cap, bool must = true) {
    int64_t new_cap = std::max<int64_t>(min_cap, c->pool_cap + c->pool_cap / 2);
    new_cap = round_up(new_cap, kRowAlign);
    Edge* p = must ? dev_alloc_n<Edge>(c, new_cap) : static_cast<Edge*>(dev_alloc_or_reclaim(c, (size_t)new_cap * sizeof(Edge)));
    if (!p) return false;
    if (c->pool && c->pool_tail > 0)
        HIPCHK(c, hipMemcpyAsync(p, c->pool, (size_t)c->pool_tail * sizeof(Edge), hipMemcpyDeviceToDevice, c->stream));
    HIPCHK(c, hipStreamSynchronize(c->stream));
    dev_free(c, c->pool);
    c->pool = p;
    c->pool_cap = new_cap;
    return true;
}

// Pinned memory for `bytes` of a small call with host arrays; false: too large a call, or no memory (nothing is lost but time).
// Up to kIoBytes: beyond, the copies themselves take longer than what they cost to start.
constexpr int64_t kIoBytes = (int64_t)1 << 20;
constexpr int64_t kIoOutBytes = (int64_t)128 << 10;  // of labels, for contexts with an allocator of their own

bool ensure_pinned(dynlp_ctx* c, int64_t bytes) {
    if (bytes > kIoBytes) return false;
    if (bytes <= c->h_io_cap) return true;
    pinned_free(c, c->h_io, (size_t)c->h_io_cap);  // (no copy from or to it is under way: every call ends with a wait)
    c->h_io_cap = 0;
    size_t got = 0;
    const int64_t cap = std::min<int64_t>(kIoBytes, round_up(std::max<int64_t>(bytes + bytes / 2, 64 << 10), 4096));
    c->h_io = static_cast<unsigned char*>(pinned_try_alloc(c, (size_t)cap, &got));
    if (!c->h_io) return false;
    c->h_io_cap = (int64_t)got;
    return true;
}

void ensure_batch_scratch(dynlp_ctx* c, int64_t nd, int64_t m, int64_t s) {
    // (with deletions any vertex may lose an entry)
    const int64_t need_t = nd > 0 ? c->n_cap : std::max<int64_t>(1, std::min<int64_t>(2 * m, c->n_cap));
    if (need_t > c->touched_cap) {
        dev_free(c, c->touched);
        dev_free(c, c->reloc_off);
        c->touched = nullptr;
        c->reloc_off = nullptr;
        const int64_t cap = nd > 0 ? need_t : need_t + need_t / 2;
        c->touched_cap = 0;
        c->touched = dev_alloc_n<int32_t>(c, cap);
        c->reloc_off = dev_alloc_n<int64_t>(c, cap);
        c->touched_cap = cap;
    }
    if (!c->dev_ptrs) {
        if (nd > c->b_del_cap) {
            dev_free(c, c->b_del);
            c->b_del = nullptr;
            c->b_del_cap = 0;
            c->b_del = dev_alloc_n<int32_t>(c, nd + nd / 2);
            c->b_del_cap = nd + nd / 2;
        }
        if (m > c->b_edge_cap) {
            dev_free(c, c->b_eu);
            dev_free(c, c->b_ev);
            dev_free(c, c->b_ew);
            c->b_eu = c->b_ev = nullptr;
            c->b_ew = nullptr;
            const int64_t cap = m + m / 2;
            c->b_eu = dev_alloc_n<int32_t>(c, cap);
            c->b_ev = dev_alloc_n<int32_t>(c, cap);
            c->b_ew = dev_alloc_n<float>(c, cap);
            c->b_edge_cap = cap;
        }
        if (s > c->b_seed_cap) {
            dev_free(c, c->b_sv);
            dev_free(c, c->b_sc);
            c->b_sv = c->b_sc = nullptr;
            const int64_t cap = s + s / 2;
            c->b_sv = dev_alloc_n<int32_t>(c, cap);
            c->b_sc = dev_alloc_n<int32_t>(c, cap);
            c->b_seed_cap = cap;
        }
    }
}

// ---- pipelined ingest of a host-resident batch --------------------------------------------------------------
// The paper overlaps the transfer of a batch with the Step-1 kernels that only need what has already arrived.
// Here the graph lives on the device and only the batch's edge list crosses PCIe; for a batch of more than one
// chunk the list is sent chunk by chunk on a second stream while the main stream validates and counts the
// chunks that have landed (k_validate_edges, k_count_halfedges: the part of Step 1 that needs nothing but the
// chunk).  Caller arrays in pinned memory are sent as they are; pageable arrays go through two pinned staging
// buffers filled by a few host threads, so that filling chunk i+1 overlaps the transfer of chunk i.
constexpr int kIngestThreads = 6;

bool host_pointer_is_pinned(const void* p) {
    hipPointerAttribute_t a;
    if (hipPointerGetAttributes(&a, p) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    return a.type == hipMemoryTypeHost;
}

void parallel_copy(void* dst, const void* src, size_t bytes) {
    if (bytes < ((size_t)4 << 20)) {
        std::memcpy(dst, src, bytes);
        return;
    }
    std::thread workers[kIngestThreads];
    const size_t slice = round_up((int64_t)ceil_div((int64_t)bytes, kIngestThreads), 4096);
    int started = 0;
    for (int t = 0; t < kIngestThreads; ++t) {
        const size_t lo = std::min(bytes, slice * t), hi = std::min(bytes, slice * (t + 1));
        if (hi <= lo) break;
        workers[t] = std::thread([=] { std::memcpy(static_cast<char*>(dst) + lo, static_cast<const char*>(src) + lo, hi - lo); });
        ++started;
    }
    for (int t = 0; t < started; ++t) workers[t].join();
}

// Copies eu / ev / ew (host) into c->b_eu / b_ev / b_ew and, per chunk, launches validation and counting on the
// main stream.  bc must have been reset on the main stream before the call.
void ingest_edges(dynlp_ctx* c, int64_t m, int64_t n_total, const int32_t* eu, const int32_t* ev, const float* ew, int32_t* touched) {
    const int64_t chunk = c->ingest_chunk;
    if (!c->copy_stream) {
        HIPCHK(c, hipStreamCreateWithFlags(&c->copy_stream, hipStreamNonBlocking));
        for (hipEvent_t& e : c->ingest_ev) HIPCHK(c, hipEventCreateWithFlags(&e, hipEventDisableTiming));
    }
    const bool pinned = host_pointer_is_pinned(eu) && host_pointer_is_pinned(ev) && host_pointer_is_pinned(ew);
    if (!pinned && c->bounce_edges < chunk) {
        for (void*& b : c->bounce) {
            if (b) (void)hipHostFree(b);
            b = nullptr;
        }
        c->bounce_edges = 0;
        size_t got = 0;
        for (void*& b : c->bounce) b = pinned_alloc(c, (size_t)chunk * 12, &got);
        c->bounce_edges = chunk;
    }
    // the copies must not start before earlier work on the main stream that still reads the device buffers is done
    // (there is none: the previous call ended with a synchronisation), nor before bc has been reset
    HIPCHK(c, hipEventRecord(c->ingest_ev[0], c->stream));
    HIPCHK(c, hipStreamWaitEvent(c->copy_stream, c->ingest_ev[0], 0));
    int chunks = 0;
    bool slot_used[2] = {false, false};
    for (int64_t off = 0; off < m; off += chunk, ++chunks) {
        const int64_t mc = std::min(chunk, m - off);
        const int slot = chunks & 1;
        const int32_t *s_eu = eu + off, *s_ev = ev + off;
        const float* s_ew = ew + off;
        if (!pinned) {
            if (slot_used[slot]) HIPCHK(c, hipEventSynchronize(c->ingest_ev[slot]));  // its last transfer has left the buffer
            char* b = static_cast<char*>(c->bounce[slot]);
            parallel_copy(b, s_eu, (size_t)mc * 4);
            parallel_copy(b + (size_t)chunk * 4, s_ev, (size_t)mc * 4);
            parallel_copy(b + (size_t)chunk * 8, s_ew, (size_t)mc * 4);
            s_eu = reinterpret_cast<const int32_t*>(b);
            s_ev = reinterpret_cast<const int32_t*>(b + (size_t)chunk * 4);
            s_ew = reinterpret_cast<const float*>(b + (size_t)chunk * 8);
        }
        HIPCHK(c, hipMemcpyAsync(c->b_eu + off, s_eu, (size_t)mc * 4, hipMemcpyHostToDevice, c->copy_stream));
        HIPCHK(c, hipMemcpyAsync(c->b_ev + off, s_ev, (size_t)mc * 4, hipMemcpyHostToDevice, c->copy_stream));
        HIPCHK(c, hipMemcpyAsync(c->b_ew + off, s_ew, (size_t)mc * 4, hipMemcpyHostToDevice, c->copy_stream));
        HIPCHK(c, hipEventRecord(c->ingest_ev[slot], c->copy_stream));
        slot_used[slot] = true;
        HIPCHK(c, hipStreamWaitEvent(c->stream, c->ingest_ev[slot], 0));
        hipLaunchKernelGGL(k_validate_edges, dim3(grid_for(mc)), dim3(kBlock), 0, c->stream, mc, n_total, c->b_eu + off,
                           c->b_ev + off, c->b_ew + off, c->bc, off);
        hipLaunchKernelGGL(k_count_halfedges, dim3(grid_for(ceil_div(2 * mc, kAppendItems))), dim3(kBlock), 0, c->stream, mc,
                           n_total, c->b_eu + off, c->b_ev + off, c->add_cnt, touched, c->bc,
                           c->he_rank ? c->he_rank + off : nullptr, c->he_rank ? c->he_rank + m + off : nullptr,
                           grid_for(ceil_div(2 * mc, kAppendItems)), (int64_t)0, (const int32_t*)nullptr, (int32_t*)nullptr);
        HIPCHK(c, hipGetLastError());
    }
    c->ingest_chunks_last = chunks;
    c->ingest_pinned_last = pinned ? 1 : 0;
}

// ---- frontier launches ---------------------------------------------------------------------------
int lanes_per_neighbour(int CP) { return CP >= 4 ? CP / 4 : 1; }

// mean row length up to which narrow rows get 4 lanes, and from which rows get more than 16
constexpr unsigned int kGroupLen4 = 8, kGroupLen32 = 96;

int choose_group(const dynlp_ctx* c, double avg_len) {
    const int lpn = lanes_per_neighbour(c->CP);
    if (c->group_lanes) return std::max(c->group_lanes, lpn);
    // Measured on MI355X (1M-vertex graph, mean row length 20, C = 4 .. 50): 16 lanes per row is the
    // fastest or within 2% of it for every padded class count; wider groups only pay off when the
    // typical row fills several 16-entry chunks.
    int g = 16;
    // rows of a few entries with one to four label columns (50M vertices of degree 5, one column: 6.2 / 6.3 / 6.5 ms
    // per round over all rows with 4 / 8 / 16 lanes): narrow groups leave fewer lanes idle
    if (avg_len < (double)kGroupLen4 && c->CP <= 4) g = 4;
    if (avg_len >= (double)kGroupLen32) g = 32;
    if (avg_len >= 384.0) g = 64;
    return std::max(g, lpn);
}

// One propagation round's frontier lives in the array of one parity: short rows from the front,
// long rows from the back.  Its size is only on the device (the previous round's counter slot).
struct Frontier {
    int32_t* front = nullptr;
    int32_t* back = nullptr;
    unsigned int ns = 0, nl = 0;  // only meaningful for lists whose size the host has read
    unsigned int size() const { return ns + nl; }
};

Frontier frontier_of(dynlp_ctx* c, int parity, unsigned int ns = 0, unsigned int nl = 0) {
    Frontier f;
    f.front = c->queue[parity];
    f.back = c->queue[parity] + (c->n_cap - 1);
    f.ns = ns;
    f.nl = nl;
    return f;
}

struct UpdateArgs {
    const RoundCtr* prev;  // slot that holds the size of the frontier to work on
    int static_stop;       // 0: frontier round; 1: static sweep; 2: static sweep that checks prev's stop rule
    const float* F_in;
    float* F_out;
    unsigned int* moved;  // "moved by > tol" bitmap of this round (ping-pong rounds), NULL otherwise
    float tol;
    RoundCtr* ctr;
    RoundCtr* ctr_zero;
    int64_t rows_bound;  // upper bounds of the frontier size and of its long rows (they size the grid)
    int64_t long_bound;
    int by_vertex = 0;  // flag-marking rounds only: kRowByVertex (write row u of F_out instead of staging by position), kRowLazy
};

template <int CP, int G, bool STAGED>
void launch_update_inst(dynlp_ctx* c, const Frontier& f, const UpdateArgs& a) {
    constexpr int GPB = kBlock / G;
    const int64_t cap = (int64_t)c->num_cu * 32;
    const unsigned int short_blocks = (unsigned int)std::max<int64_t>(1, std::min<int64_t>(ceil_div(a.rows_bound, GPB), cap));
    const unsigned int long_max = (unsigned int)std::min<int64_t>(a.long_bound, cap / 2);
    unsigned int stop_bits;
    std::memcpy(&stop_bits, &a.tol, sizeof stop_bits);
    hipLaunchKernelGGL((k_row_update<CP, G, STAGED>), dim3(short_blocks + long_max), dim3(kBlock), 0, c->stream, a.prev,
                       a.static_stop, stop_bits, long_max, f.front, f.back, c->meta, c->pool, a.F_in, a.F_out, a.by_vertex, c->flag, a.moved, a.tol,
                       a.ctr, a.ctr_zero);
}

template <int CP, bool STAGED>
void launch_update_cp(dynlp_ctx* c, int G, const Frontier& f, const UpdateArgs& a) {
    constexpr int LPN = CP >= 4 ? CP / 4 : 1;
#define DYNLP_CASE(GV)                                              \
    case GV:                                                        \
        if constexpr (GV >= LPN) {                                  \
            launch_update_inst<CP, GV, STAGED>(c, f, a);            \
            return;                                                 \
        }                                                           \
        break;
    switch (G) {
        DYNLP_CASE(4)
        DYNLP_CASE(8)
        DYNLP_CASE(16)
        DYNLP_CASE(32)
        DYNLP_CASE(64)
        default: break;
    }
#undef DYNLP_CASE
    launch_update_inst<CP, 64, STAGED>(c, f, a);
}

// With kernel timing on, two events bracket every row-update launch; `round` / `count` say which rounds it runs.
// A launch that directly follows the previous timed launch (c->ev_adjacent, set by the caller for this one call)
// takes that launch's closing event as its opening one: an event record costs a few microseconds on the stream,
// which shows once a round takes 40 of them.
hipEvent_t open_timed_span(dynlp_ctx* c, int round, int count) {
    const bool adjacent = c->ev_adjacent && c->events_used > 0;
    c->ev_adjacent = false;
    if (!c->time_kernels) return nullptr;
    while (c->events.size() < c->events_next + 2) {
        hipEvent_t e;
        HIPCHK(c, hipEventCreate(&e));
        c->events.push_back(e);
    }
    const size_t k = c->events_used / 2;
    if (c->ev_round.size() <= k) {
        c->ev_round.resize(k + 1);
        c->ev_count.resize(k + 1);
        c->ev_first.resize(k + 1);
        c->ev_last.resize(k + 1);
    }
    c->ev_round[k] = round;
    c->ev_count[k] = count;
    c->events_used += 2;
    if (adjacent) {
        c->ev_first[k] = c->ev_last[k - 1];
    } else {
        c->ev_first[k] = (int)c->events_next;
        HIPCHK(c, hipEventRecord(c->events[c->events_next++], c->stream));
    }
    c->ev_last[k] = (int)c->events_next;
    return c->events[c->events_next++];
}

void close_timed_span(dynlp_ctx* c, hipEvent_t e1) {
    if (e1) HIPCHK(c, hipEventRecord(e1, c->stream));
}

void reset_timed_spans(dynlp_ctx* c) {
    c->events_used = 0;
    c->events_next = 0;
    c->ev_adjacent = false;
}

// After a chain has been read back: launches of rounds >= first_unexecuted did nothing.
void trim_timed_spans(dynlp_ctx* c, size_t first_pair, int first_unexecuted) {
    for (size_t k = first_pair; k < c->events_used / 2; ++k) {
        if (c->ev_round[k] >= first_unexecuted) c->ev_round[k] = -1;
        else c->ev_count[k] = std::min(c->ev_count[k], first_unexecuted - c->ev_round[k]);
    }
}

// Row update of one frontier: one launch (long rows and short rows share the grid).  With kernel
// timing on, two events per round bracket it.
template <bool STAGED>
void launch_update(dynlp_ctx* c, int G, const Frontier& f, const UpdateArgs& a, int round) {
    hipEvent_t e1 = open_timed_span(c, round, 1);
    switch (c->CP) {
        case 1: launch_update_cp<1, STAGED>(c, G, f, a); break;
        case 2: launch_update_cp<2, STAGED>(c, G, f, a); break;
        case 4: launch_update_cp<4, STAGED>(c, G, f, a); break;
        case 8: launch_update_cp<8, STAGED>(c, G, f, a); break;
        case 16: launch_update_cp<16, STAGED>(c, G, f, a); break;
        case 32: launch_update_cp<32, STAGED>(c, G, f, a); break;
        default: launch_update_cp<64, STAGED>(c, G, f, a); break;
    }
    HIPCHK(c, hipGetLastError());
    close_timed_span(c, e1);
}

// A ping-pong round that evaluates V_aff membership itself (k_row_update_pull): `universe` lists every
// updatable vertex, moved_prev / moved_cur / moved_clear are the bitmaps of the previous, this and the next round.
struct PullRoundArgs {
    const RoundCtr* prev;
    const float* F_in;
    float* F_out;
    const unsigned int* moved_prev;
    unsigned int* moved_cur;
    unsigned int* moved_clear;
    float tol;
    RoundCtr* ctr;
    RoundCtr* ctr_zero;
    int flags = 0;       // kRoundAll, kRoundForce
    float omega = 1.f;   // relaxation of a round over all rows
};

template <int CP, int G>
void launch_update_pull_inst(dynlp_ctx* c, const Frontier& universe, const PullRoundArgs& a) {
    constexpr int GPB = kBlock / G;
    const int64_t cap = (int64_t)c->num_cu * 32;
    const unsigned int short_blocks =
        (unsigned int)std::max<int64_t>(1, std::min<int64_t>(ceil_div((int64_t)universe.ns, GPB), cap));
    const unsigned int long_max = (unsigned int)std::min<int64_t>((int64_t)universe.nl, cap / 2);
    auto kernel = a.flags & kRoundAll ? k_row_update_pull<CP, G, true> : k_row_update_pull<CP, G, false>;
    hipLaunchKernelGGL(kernel, dim3(short_blocks + long_max), dim3(kBlock), 0, c->stream, a.prev, long_max,
                       universe.front, universe.back, universe.ns, universe.nl, c->meta, c->pool, a.F_in, a.F_out,
                       a.moved_prev, a.moved_cur, a.moved_clear, (unsigned int)c->moved_words, a.tol, a.flags, a.omega, a.ctr,
                       a.ctr_zero);
}

template <int CP>
void launch_update_pull_cp(dynlp_ctx* c, int G, const Frontier& universe, const PullRoundArgs& a) {
    constexpr int LPN = CP >= 4 ? CP / 4 : 1;
#define DYNLP_CASE(GV)                                              \
    case GV:                                                        \
        if constexpr (GV >= LPN) {                                  \
            launch_update_pull_inst<CP, GV>(c, universe, a);        \
            return;                                                 \
        }                                                           \
        break;
    switch (G) {
        DYNLP_CASE(4)
        DYNLP_CASE(8)
        DYNLP_CASE(16)
        DYNLP_CASE(32)
        DYNLP_CASE(64)
        default: break;
    }
#undef DYNLP_CASE
    launch_update_pull_inst<CP, 64>(c, universe, a);
}

void launch_update_pull(dynlp_ctx* c, int G, const Frontier& universe, const PullRoundArgs& a, int round) {
    hipEvent_t e1 = open_timed_span(c, round, 1);
    switch (c->CP) {
        case 1: launch_update_pull_cp<1>(c, G, universe, a); break;
        case 2: launch_update_pull_cp<2>(c, G, universe, a); break;
        case 4: launch_update_pull_cp<4>(c, G, universe, a); break;
        case 8: launch_update_pull_cp<8>(c, G, universe, a); break;
        case 16: launch_update_pull_cp<16>(c, G, universe, a); break;
        case 32: launch_update_pull_cp<32>(c, G, universe, a); break;
        default: launch_update_pull_cp<64>(c, G, universe, a); break;
    }
    HIPCHK(c, hipGetLastError());
    close_timed_span(c, e1);
}

// Rounds queued per host round trip.
constexpr int kChain = 8;
static_assert(kChain <= kXcdChain, "k_xcd_rounds keeps the counters of a chain");
// A batch of more half-edges than one per kInOrderShare vertices lists the rows it touches by a pass over all vertices.
constexpr int64_t kInOrderShare = 8;
// Such a batch sorts what a row receives with 8 lanes instead of 16 where it holds fewer half-edges than this per vertex and
// the chip is full either way (20,000 rows: 11 us with 16 lanes, 14 with 8).
constexpr int64_t kSortLanes8 = 8, kSortRows8 = 131072;
constexpr int64_t kPlanItems = (int64_t)2 << 20;  // touched rows from which the plan takes several per thread (k_plan_reserve)
// Batches whose steps share launches of one workgroup each (dynlp_small.h).  Deleted rows are taken 64 at a time, those of more
// than 128 entries one after the other; how many entries they have only the mean tells.
bool small_batch(const dynlp_ctx* c, int64_t nd, int64_t k, int64_t m, int64_t s) {
    constexpr int64_t kDeleted = 128, kDeletedEntries = 2048, kSeeds = 1024, kNewLabels = 16384;
    return 2 * m <= kSmallHalfEdges && nd <= kDeleted && nd * c->entries <= kDeletedEntries * std::max<int64_t>(1, c->n) && s <= kSeeds &&
           k * c->CP <= kNewLabels;
}

// Rounds in a row that repeat themselves exactly before the rows are averaged (see dynlp_apply_update).
constexpr int kSameRounds = 16;

// Optional (the insertion falls back to a second atomic per half-edge without it).
void ensure_ranks(dynlp_ctx* c, int64_t m) {
    if (2 * m <= c->he_rank_cap) return;
    dev_free(c, c->he_rank);
    c->he_rank_cap = 0;
    c->he_rank = static_cast<int32_t*>(dev_try_alloc(c, (size_t)(3 * m) * sizeof(int32_t)));
    if (c->he_rank) c->he_rank_cap = 3 * m;
}

// ---- insertion through bins (dynlp_insert.h) --------------------------------------------------------------------
// Scratch of one batch: freed where the call has waited for the insertion.
struct BinnedInsert {
    dynlp_ctx* c;
    bool on = false;
    int bits = 0, nbins = 0, chunks = 0;
    unsigned short* row = nullptr;
    int32_t* col = nullptr;
    float* w = nullptr;
    unsigned int *table = nullptr, *bins = nullptr;  // bins: counts, offsets, first slices
    explicit BinnedInsert(dynlp_ctx* ctx) : c(ctx) {}
    BinnedInsert(const BinnedInsert&) = delete;
    BinnedInsert& operator=(const BinnedInsert&) = delete;
    ~BinnedInsert() {
        if (row) (void)hipStreamSynchronize(c->stream);  // (a call that ends early)
        release();
    }
    void release() {
        void* const all[] = {row, col, w, table, bins};
        for (void* p : all) scratch_free(c, p);
        row = nullptr;
        col = nullptr;
        w = nullptr;
        table = bins = nullptr;
    }
    // From so many half-edges on (insertion in us, atomics / bins, 4 half-edges per row and 1 per row: 2^19 105 / 123 and 133 / 143,
    // 2^20 169 / 152 and 235 / 217, 2^21 301 / 238 and 349 / 282, 2^22 629 / 448 and 739 / 597; a quarter per row: 2^20 307 / 308,
    // 2^22 1052 / 934).
    static constexpr int64_t kMinHalfEdges = (int64_t)1 << 21;
    // Whether m edges into n rows go this way (no memory for it: no).
    void choose(int64_t m, int64_t n) {
        bits = kHbMaxBits;
        while (bits > 11 && ceil_div(n, (int64_t)1 << bits) < 2 * c->num_cu) --bits;
        if (2 * m < kMinHalfEdges || ceil_div(n, (int64_t)1 << bits) > kPbMaxBins) return;
        nbins = (int)ceil_div(n, (int64_t)1 << bits);
        chunks = (int)ceil_div(2 * m, kHbChunk);
        row = static_cast<unsigned short*>(dev_try_alloc(c, (size_t)(2 * m) * sizeof(unsigned short)));
        col = row ? static_cast<int32_t*>(dev_try_alloc(c, (size_t)(2 * m) * sizeof(int32_t))) : nullptr;
        w = col ? static_cast<float*>(dev_try_alloc(c, (size_t)(2 * m) * sizeof(float))) : nullptr;
        table = w ? static_cast<unsigned int*>(dev_try_alloc(c, ((size_t)chunks + 1 + kPbSegs) * nbins * sizeof(unsigned int))) : nullptr;
        bins = table ? static_cast<unsigned int*>(dev_try_alloc(c, (3 * (size_t)nbins + 2) * sizeof(unsigned int))) : nullptr;
        on = bins != nullptr;
        if (!on) release();
    }
    unsigned int* offsets() const { return bins + nbins; }
    unsigned int* slices() const { return bins + 2 * nbins + 1; }
    unsigned int most_slices(int64_t m) const { return (unsigned int)(nbins + ceil_div(2 * m, kHbSlice)); }
    void launch_count(int64_t m, int64_t n, const int32_t* eu, const int32_t* ev, const float* ew) {
        hipLaunchKernelGGL(k_hb_count, dim3(chunks), dim3(kHbThreads), 0, c->stream, m, n, bits, nbins, eu, ev, table);
        unsigned int* const seg = table + ((size_t)chunks + 1) * nbins;
        const dim3 columns(grid_for(nbins), kPbSegs);
        hipLaunchKernelGGL(k_pb_seg_sums, columns, dim3(kBlock), 0, c->stream, nbins, chunks, table, seg);
        hipLaunchKernelGGL(k_pb_seg_scan, dim3(grid_for(nbins)), dim3(kBlock), 0, c->stream, nbins, chunks, seg, table, bins);
        hipLaunchKernelGGL(k_pb_chunk_bases, columns, dim3(kBlock), 0, c->stream, nbins, chunks, seg, table);
        hipLaunchKernelGGL(k_pb_offsets, dim3(1), dim3(kBlock), 0, c->stream, nbins, bins, offsets());
        hipLaunchKernelGGL(k_hb_slices, dim3(1), dim3(kBlock), 0, c->stream, nbins, bins, slices());
        int lg = 2;  // lanes per run: about as many as it has half-edges
        while (lg < 10 && ((int64_t)nbins << lg) < kHbChunk) ++lg;
        hipLaunchKernelGGL(k_hb_place, dim3(8 * (unsigned int)ceil_div(chunks, 8)), dim3(kHbThreads), 0, c->stream, m, n, bits, nbins, lg, eu,
                           ev, ew, table, offsets(), row, col, w);
        hipLaunchKernelGGL(k_hb_rows, dim3(most_slices(m)), dim3(kHbThreads), 0, c->stream, n, bits, nbins, offsets(), slices(), row, c->add_cnt);
    }
    void launch_write(int64_t m, int64_t n, const BatchGate& gate) {
        HIPCHK(c, hipFuncSetAttribute(reinterpret_cast<const void*>(&k_hb_write), hipFuncAttributeMaxDynamicSharedMemorySize, 8 << kHbMaxBits));
        hipLaunchKernelGGL(k_hb_write, dim3(most_slices(m)), dim3(kHbThreads), 8u << bits, c->stream, n, bits, nbins, offsets(), slices(), row,
                           col, w, c->meta, c->pool, gate);
    }
};

// ---- many rounds over a small V_aff in one launch (k_tail_rounds) -----------------------------------------------
// One CU gathers about 0.4 rows per clock and looks up every neighbour it marks; the launches of an ordinary round take
// 12 to 14 us whatever their size.  Measured per round: 3,000 vertices with one label column, up to 886 rows and 6,000
// entries, 15 -> 8 us (whole batch 534 -> 436 us); 24,000 vertices with 5 columns, rounds of 4,000 to 8,000 entries, 12 ->
// 16 us: the limits depend on the columns.  A launch pays when it runs several rounds, so a V_aff that is about to outgrow
// the limits (every row may bring its neighbours) is left to ordinary rounds.
constexpr int kTailRounds = 32;

void tail_limits(const dynlp_ctx* c, unsigned int* rows, unsigned int* entries) {
    *rows = c->CP <= 2 ? 1024 : c->CP <= 16 ? 512 : 256;
    *entries = c->CP <= 2 ? 8192 : c->CP <= 16 ? 3072 : 1536;
}

bool tail_rounds_pay(const dynlp_ctx* c, unsigned int known, unsigned int before, double avg_len) {
    unsigned int rows, entries;
    tail_limits(c, &rows, &entries);
    if (known > rows || (double)known * avg_len > (double)entries) return false;
    return before >= known || (double)known * avg_len <= (double)rows;
}

// LDS that a launch with the labels on the CU may ask for: what one workgroup can have, less the kernel's own arrays.
constexpr unsigned int kTailLds = 120 << 10;

template <int CP, int G>
void launch_tail_inst(dynlp_ctx* c, const TailArgs& a) {
    const unsigned int lds = c->n < 65536 ? tail_resident_bytes((unsigned int)c->n, CP, a.max_rows) : 0xffffffffu;
    bool resident = lds <= kTailLds && c->pool_cap < ((int64_t)1 << 32);
    if (resident) {
        // always the same value: the attribute belongs to the kernel, not to this context
        resident = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_tail_rounds<CP, G, true>), hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)kTailLds) == hipSuccess;
        if (!resident) (void)hipGetLastError();
    }
    if (resident) hipLaunchKernelGGL((k_tail_rounds<CP, G, true>), dim3(1), dim3(kTailThreads), lds, c->stream, a);
    else hipLaunchKernelGGL((k_tail_rounds<CP, G, false>), dim3(1), dim3(kTailThreads), 0, c->stream, a);
}

template <int CP>
void launch_tail_cp(dynlp_ctx* c, int G, const TailArgs& a) {
    if constexpr (CP <= 4) {
        if (G == 4) {
            launch_tail_inst<CP, 4>(c, a);
            return;
        }
    }
    launch_tail_inst<CP, 16>(c, a);
}

// Rounds [round, round + count) at most; the list of the first one is that of parity `cur`.  chain_off: rounds of the
// running chain of kChain that came before; same_run, sig: the batch's run of rounds that repeat themselves so far.
void launch_tail(dynlp_ctx* c, int G, int cur, int round, int count, int by_vertex, int chain_off, int same_run,
                 const unsigned int (&sig)[3]) {
    TailArgs a{};
    a.chain = kChain;
    a.chain_off = chain_off;
    a.len_lo = G == 4 || c->CP > 4 ? 0u : kGroupLen4;
    a.len_hi = G == 4 ? kGroupLen4 : kGroupLen32;
    a.same_run = same_run;
    a.same_max = kSameRounds;
    for (int i = 0; i < 3; ++i) a.sig[i] = sig[i];
    a.ring = c->ring;
    a.t0 = round;
    a.rounds = count;
    for (int i = 0; i < 2; ++i) {
        const Frontier f = frontier_of(c, cur ^ i);
        a.front[i] = f.front;
        a.back[i] = f.back;
    }
    a.meta = c->meta;
    a.pool = c->pool;
    a.seed_class = c->seed_class;
    a.F = c->F;
    a.staged = c->F2;
    a.by_vertex = by_vertex;
    a.flag = c->flag;
    a.tol = c->tol;
    a.n = (unsigned int)c->n;
    tail_limits(c, &a.max_rows, &a.max_entries);
    hipEvent_t e1 = open_timed_span(c, round, count);
    switch (c->CP) {
        case 1: launch_tail_cp<1>(c, G, a); break;
        case 2: launch_tail_cp<2>(c, G, a); break;
        case 4: launch_tail_cp<4>(c, G, a); break;
        case 8: launch_tail_cp<8>(c, G, a); break;
        case 16: launch_tail_cp<16>(c, G, a); break;
        case 32: launch_tail_cp<32>(c, G, a); break;
        default: launch_tail_cp<64>(c, G, a); break;
    }
    HIPCHK(c, hipGetLastError());
    close_timed_span(c, e1);
}

// ---- rounds of small graphs on one XCD (k_xcd_rounds) -----------------------------------------------------------
// One XCD has an eighth of the chip's CUs, so a round over all rows costs it more than the whole chip from some size on, which
// the launches it saves make up for.  Whole calls, ms, ordinary launches / one XCD (planted blocks, 3 and 14 classes, tol =
// 1e-6):
//                          24,000 entries           80,000               160,000              280,000              400,000
//   batches, synchronous   6.11/3.01  6.14/3.19     6.13/3.56  6.59/4.21  6.59/4.52  7.25/5.38  7.36/6.34  7.48/6.83  6.88/7.20  8.02/8.53
//   batches, in place      6.11/2.74  6.64/2.84     6.38/3.17  6.65/3.78  6.30/3.64  7.56/4.03  6.80/5.48  7.53/5.14  7.38/5.84  7.91/6.36
// (in place it also needs fewer rounds there: fewer rows are updated at the same time.)  Cold starts, 4 and 12 classes, whose
// sweeps are one launch each: synchronous 16,000 entries 5.60/2.86 5.90/3.39, 96,000 6.38/5.08 6.80/6.00, 192,000 5.92/6.18
// 6.89/7.57; in place 192,000 5.95/5.42 6.96/6.75, 200,000 7.37/5.85 8.56/7.00, 400,000 7.22/9.31 8.28/9.03.  At tol = 1e-4,
// 8 to 25 rounds: 0.34/0.22 at 42,000 entries, 0.47/0.34 at 160,000, 0.36/0.31 at 280,000.
// More than 16 columns (a row is two lines of the L2 or four) are left to ordinary launches, because kernels for them are not built:
// with two more of them 24 and 50 classes took, at 25,000 / 81,000 / 162,000 / 287,000 / 406,000 entries, synchronous 8.2/3.8 6.6/4.8
// 7.2/6.1 5.5/7.5 10.4/13.9 and 7.7/4.4 7.6/6.9 5.0/8.5 10.2/18.7 13.0/28.3, in place 7.6/3.4 6.7/3.9 7.1/4.1 9.8/5.8 10.0/6.5 and
// 7.4/3.8 7.6/4.6 8.8/6.0 10.4/9.8 12.0/14.7 (batches, tol = 1e-6).
int64_t xcd_max_entries(const dynlp_ctx* c, bool sweeps) {
    const bool in_place = c->update_mode == DYNLP_UPDATE_IN_PLACE;
    return sweeps ? (in_place ? 256000 : 128000) : (in_place ? 440000 : 300000);
}

bool xcd_rounds_pay(const dynlp_ctx* c, const Frontier& universe, int G, bool sweeps) {
    if (c->group_lanes != 0 || c->persist > 0 || (c->CP == 1 && c->binned > 0) || c->CP > 16 || G > 16) return false;
    if (universe.nl != 0 || universe.size() == 0 || c->n > kXcdMaxRows || c->entries > xcd_max_entries(c, sweeps)) return false;
    // room for an eighth more than a workgroup's even share of the entries (the kernel has the last word)
    const int64_t rows = c->n / kXcdGroups + 32, head = c->n / 8 + 64 + 7 * rows;
    return head + c->entries / kXcdGroups * 9 / 8 * (int64_t)sizeof(Edge) <= (int64_t)kXcdLds;
}

// Rounds of one launch at most (whole chains), from round `it` of a call on.
// A launch holds all registers of its XCD's CUs, and every other launch has workgroups for that XCD: those wait for its end, and
// with them all that their stream holds (a kernel of another process or library too).  While other calls of this process are at work
// launches are therefore short, and shorter still in a call that goes on for long.  us for a call (medians), of threads with a context
// and a stream each; N = one vertex into 3,001, T = 37 into 20,011, K = 100 into 2,000 with 230 rounds, S = 30,000 into 300,007:
//                                            K       N        K+K          N+N        T+T        K+N         T+K+N             S+N
//   a launch for each round                  2,400   215      2,550 2,830  265 265    488 488    2,520  211  662 2,910  330    2,690 320
//   240 rounds at once, whatever others do   1,130   139      2,230 2,280  161 161    383 384    1,157 1,107                   2,843 251
//   16 rounds at once                        1,130   139      1,660 1,670  167 172    396 396    1,520  375  440 1,740  380    2,850 258
//   16, from round 32 on 8 (here)            1,130   139      1,910 2,010  170 172    390 390    1,810  242  400 2,160  330    2,790 270
//   16, from round 32 on launches for each   1,140   140      2,450 2,790  168 174    393 393    2,370  134  328 4,270  287    2,840 260
constexpr int kXcdTogether = 32, kXcdTogetherFirst = 16, kXcdTogetherThen = 8;
static_assert(kXcdTogetherFirst % kChain == 0 && kXcdTogetherThen % kChain == 0 && kXcdRounds % kChain == 0, "whole chains");
int xcd_rounds_at_once(const dynlp_ctx* c, int it) {
    return !others_at_work(c->device) ? kXcdRounds : it < kXcdTogether ? kXcdTogetherFirst : kXcdTogetherThen;
}

// (A number is taken by a launch that takes place and by no other: each launch clears the list of the next number.)
unsigned int next_xcd_launch(dynlp_ctx* c) {
    if (c->xcd_launches == kXcdLaunches) {  // (the words of an exchange are told apart by the launch's number)
        HIPCHK(c, hipMemsetAsync(c->xcd, 0, sizeof(XcdCtl), c->stream));
        c->xcd_launches = 0u;
    }
    return ++c->xcd_launches;
}

template <int CP, int G>
void launch_xcd_inst(dynlp_ctx* c, XcdArgs& a, bool refuse) {
    const void* kernel = reinterpret_cast<const void*>(&k_xcd_rounds<CP, G>);
    // (always the same value: the attribute belongs to the kernel, not to this context)
    if (refuse || hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kXcdLds) != hipSuccess) {
        (void)hipGetLastError();
        c->h_xcd->rounds = 0;
        *c->h_flag = a.value;  // nothing was launched: refused
        return;
    }
    a.launch = next_xcd_launch(c);
    hipLaunchKernelGGL((k_xcd_rounds<CP, G>), dim3(8 * a.want), dim3(kXcdThreads), kXcdLds, c->stream, a);
}

// Rounds [round, round + count) at most, from the list of parity `cur` (all_rows: over every updatable row); waits for them.
// What they did is in c->h_xcd then; 0 rounds: they have to be launched one by one.
void run_xcd(dynlp_ctx* c, int G, int cur, int round, int count, float* F_in, float* F_out, bool all_rows, bool lazy, float tol,
             int chain_off, int same_run, const unsigned int (&sig)[3]) {
    XcdArgs a{};
    a.ctl = c->xcd;
    a.result = c->h_xcd;
    a.flag = c->h_flag;
    a.value = ++c->h_sent;
    const int limit = c->xcd_asked++ >= c->xcd_from ? c->xcd_groups : 0;
    const bool refuse = limit < 0;
    a.want = (unsigned int)std::max<int64_t>(1, std::min<int64_t>(limit > 0 ? limit : kXcdGroups, ceil_div(c->n, 64)));
    a.ring = c->ring;
    a.t0 = round;
    a.rounds = count;
    for (int i = 0; i < 2; ++i) a.front[i] = frontier_of(c, cur ^ i).front;
    a.meta = c->meta;
    a.pool = c->pool;
    a.seed_class = c->seed_class;
    a.F[0] = F_in;
    a.F[1] = F_out;
    a.n = (unsigned int)c->n;
    a.all_rows = all_rows ? 1 : 0;
    a.lazy = lazy ? 1 : 0;
    a.tol = tol;
    a.chain = kChain;
    a.chain_off = chain_off;
    a.len_lo = G == 4 || c->CP > 4 ? 0u : kGroupLen4;
    a.len_hi = G == 4 ? kGroupLen4 : kGroupLen32;
    a.same_run = same_run;
    a.same_max = kSameRounds;
    for (int i = 0; i < 3; ++i) a.sig[i] = sig[i];
    hipEvent_t e1 = open_timed_span(c, round, count);
    switch (c->CP) {
        case 1: G == 4 ? launch_xcd_inst<1, 4>(c, a, refuse) : launch_xcd_inst<1, 16>(c, a, refuse); break;
        case 2: G == 4 ? launch_xcd_inst<2, 4>(c, a, refuse) : launch_xcd_inst<2, 16>(c, a, refuse); break;
        case 4: G == 4 ? launch_xcd_inst<4, 4>(c, a, refuse) : launch_xcd_inst<4, 16>(c, a, refuse); break;
        case 8: launch_xcd_inst<8, 16>(c, a, refuse); break;
        default: launch_xcd_inst<16, 16>(c, a, refuse); break;
    }
    HIPCHK(c, hipGetLastError());
    close_timed_span(c, e1);
    wait_for_flag(c, a.value);
}

// A round of such a launch as the round log has it.
RoundCtr xcd_round(const XcdPart& p) {
    RoundCtr r{};
    r.executed = 1u;
    r.rows_short = p.rows;
    r.resid_bits = p.resid_bits;
    r.changed = p.changed;
    r.edges = p.entries;
    return r;
}

// ---- several rounds per launch (k_rounds_persistent) ------------------------------------------------------------
// Whether a stretch of rounds that evaluate V_aff themselves should run many rounds per launch.  Off unless asked
// for: measured on MI355X on a 100,000-vertex kNN graph (10 classes, 2M stored entries) a round inside such a
// launch takes 68 us against 52-58 us as a launch of its own - the label rows that cross the barrier must be
// read past the per-XCD L2s, and a workgroup runs its share of a round's rows one after the other - so that the
// fewer rounds an in-place batch then needs (370 against 500: fewer rows in flight at once) only tie the batch at
// 26 ms, and a synchronous batch loses (46 against 38 ms).
constexpr int kPersistRounds = 32;  // rounds per launch; the ring of counter slots holds kRing = 64

bool persistent_rounds_pay(const dynlp_ctx* c, const Frontier& universe) {
    (void)universe;
    return c->persist > 0 && !c->persist_failed;
}

template <int CP, int G>
bool launch_persistent_inst(dynlp_ctx* c, const Frontier& universe, PersistArgs& a) {
    constexpr int GPB = kBlock / G;
    static int per_cu_cache[64] = {};  // by device ordinal
    int& per_cu = per_cu_cache[c->device & 63];
    if (per_cu == 0) {
        int v = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&v, k_rounds_persistent<CP, G>, kBlock, 0) != hipSuccess || v < 1) {
            (void)hipGetLastError();
            return false;
        }
        per_cu = v;
    }
    const int64_t resident = std::min<int64_t>((int64_t)c->num_cu * per_cu, (int64_t)kBarGroup * kBarMaxGroups);
    const int64_t want = std::max<int64_t>(1, ceil_div((int64_t)universe.ns, GPB)) + std::min<int64_t>(universe.nl, resident / 2);
    const unsigned int grid = (unsigned int)std::min<int64_t>(want, resident);
    a.long_blocks_max = (unsigned int)std::min<int64_t>((int64_t)universe.nl, std::max<int64_t>(grid / 2, universe.ns ? 0 : grid));
    if (a.long_blocks_max >= grid && universe.ns > 0) a.long_blocks_max = grid - 1;
    a.ngroups = (unsigned int)ceil_div((int64_t)grid, (int64_t)kBarGroup);
    // an ordinary launch of a grid that fits the device all at once (a cooperative launch costs milliseconds here);
    // should the grid not be resident as a whole for any reason, the bounded wait at the barrier ends the launch
    hipLaunchKernelGGL((k_rounds_persistent<CP, G>), dim3(grid), dim3(kBlock), 0, c->stream, a);
    if (hipGetLastError() != hipSuccess) return false;
    return true;
}

template <int CP>
bool launch_persistent_cp(dynlp_ctx* c, int G, const Frontier& universe, PersistArgs& a) {
    constexpr int LPN = CP >= 4 ? CP / 4 : 1;
#define DYNLP_CASE(GV)                                                  \
    case GV:                                                            \
        if constexpr (GV >= LPN) return launch_persistent_inst<CP, GV>(c, universe, a); \
        break;
    switch (G) {
        DYNLP_CASE(4)
        DYNLP_CASE(8)
        DYNLP_CASE(16)
        DYNLP_CASE(32)
        DYNLP_CASE(64)
        default: break;
    }
#undef DYNLP_CASE
    return launch_persistent_inst<CP, 64>(c, universe, a);
}

// Rounds [round, round + count) of a stretch in one launch.  False: the launch was refused (nothing was queued);
// the caller queues ordinary rounds instead.
bool launch_persistent(dynlp_ctx* c, int G, const Frontier& universe, PersistArgs& a, int round) {
    HIPCHK(c, hipMemsetAsync(c->persist_ctl, 0, kBarWords * sizeof(unsigned int), c->stream));
    hipEvent_t e1 = open_timed_span(c, round, a.rounds);
    bool ok;
    switch (c->CP) {
        case 1: ok = launch_persistent_cp<1>(c, G, universe, a); break;
        case 2: ok = launch_persistent_cp<2>(c, G, universe, a); break;
        case 4: ok = launch_persistent_cp<4>(c, G, universe, a); break;
        case 8: ok = launch_persistent_cp<8>(c, G, universe, a); break;
        case 16: ok = launch_persistent_cp<16>(c, G, universe, a); break;
        case 32: ok = launch_persistent_cp<32>(c, G, universe, a); break;
        default: ok = launch_persistent_cp<64>(c, G, universe, a); break;
    }
    close_timed_span(c, e1);
    if (!ok && c->time_kernels) c->ev_round[c->events_used / 2 - 1] = -1;
    return ok;
}

// ---- binned rounds (dynlp_binned.h) -----------------------------------------------------------------
// Whether a stretch of rounds over nearly all vertices should run as scatter + gather passes: one label column,
// and either forced by the option or labels well beyond one XCD's L2 (4 MB = 1M labels), so that the ordinary
// round's gathers miss it.  Measured on MI355X, binary labels, one round over all rows, binned against ordinary
// (and whole batches, in-place mode): 50M vertices of degree 5: 1.64 against 6.2 ms (957 against 1,463 ms); 10M
// vertices of mean degree 38: 2.26 against 6.2 ms (1,095 against 1,510 ms); 5M of degree 5: 0.18 against 0.64 ms
// (105 against 164 ms); 2M of degree 5: 0.10 against 0.28 ms (77 against 101 ms); 1M of mean degree 20 (4 MB of
// labels): 0.29 against 0.24 ms, and whole batches twice as slow because the binned rounds are Jacobi rounds
// also in in-place mode.
bool binned_rounds_pay(const dynlp_ctx* c, const Frontier& universe) {
    if (c->CP != 1 || c->binned < 0) return false;
    if (ceil_div(c->n, (int64_t)1 << (c->binned > 0 ? c->binned : kPbMaxBinBits)) > kPbMaxBins) return false;
    if (c->entries >= ((int64_t)1 << 32) - 2 * kPbChunk) return false;  // slots and stream positions are 32-bit
    if (c->binned > 0) return true;
    return universe.size() >= (2u << 20);
}

// Free every array of the binned rounds.
void free_binned(dynlp_ctx* c) {
    void* all[] = {c->pb_src, c->pb_sp, c->pb_row0, c->pb_lpos, c->pb_tmp, c->pb_dst, c->pb_wn, c->pb_val,
                   c->pb_len, c->pb_upd, c->pb_first, c->pb_block, c->pb_bin, c->pb_table};
    for (void* q : all) dev_free(c, q);
    c->pb_src = c->pb_val = c->pb_upd = c->pb_first = c->pb_block = c->pb_bin = c->pb_table = c->pb_row0 = c->pb_sp = nullptr;
    c->pb_lpos = c->pb_dst = nullptr;
    c->pb_tmp = c->pb_wn = nullptr;
    c->pb_len = nullptr;
    c->pb_ent_cap = c->pb_vcap = c->pb_table_cap = 0;
    c->pb_built = false;
}

template <typename T>
bool try_alloc_n(dynlp_ctx* c, T*& p, int64_t count) {
    p = static_cast<T*>(dev_try_alloc(c, (size_t)std::max<int64_t>(count, 1) * sizeof(T)));
    return p != nullptr;
}

// Lanes that share one (chunk, bin) run when it is written out (log2): the mean run length rounded up to a power of
// two, 16 .. 1,024 (8 / 16 / 32 lanes on runs of 11 entries: 1.79 / 1.71 / 1.73 ms per round).
int pb_run_lanes(int nbins) {
    int lg = 4;
    while (lg < 10 && ((int64_t)nbins << lg) < kPbChunk) ++lg;
    return lg;
}

// Receivers per bin (log2): the most (longer runs for the scatter pass) that leave two bins per CU, from 2^12 on.  A bin is a
// workgroup of the gather pass, one to a CU with 2^15 receivers and two below; 3M vertices are 92 such bins.  us per round with
// 2^15 / 14 / 13 / 12 / 11 receivers, synchronous (S) and conjugate (C): 2.2M of degree 5 S 92 / 66 / 70 / 67 / 73, 3M S 99 / 74 /
// 77 / 78 / 97, C 139 / 108 / 106 / 104 / 106, 5M of degree 7 S 202 / 209 / 199 / 203 / 292, 10M of degree 5 S 313 / 288 / 291 / 401, C
// 389 / 353 / 347 / 433, 20M S 564 / 556 / 774, C 765 / 742 / 947.
int pb_bin_bits(const dynlp_ctx* c) {
    if (c->binned > 0) return c->binned;
    int bits = kPbMaxBinBits;
    while (bits > 12 && ceil_div(c->n, (int64_t)1 << bits) < 2 * c->num_cu) --bits;
    return bits;
}

// LDS for the gather workgroups of any bin (always the same value: the attribute belongs to the kernel).
template <typename K>
void allow_gather_lds(dynlp_ctx* c, K* kernel) {
    HIPCHK(c, hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                  (int)pb_gather_lds(kPbMaxBinBits)));
}

// Slots, per-slot receiver offsets and normalised weights for the graph as it stands.  False (and nothing kept)
// when the arrays cannot be allocated: the caller then runs ordinary rounds.
bool build_binned(dynlp_ctx* c) {
    const int bits = pb_bin_bits(c);
    const int nbins = (int)ceil_div(std::max<int64_t>(c->n, 1), (int64_t)1 << bits);
    const int chunks = (int)ceil_div(std::max<int64_t>(c->entries, 1), kPbChunk);
    bool ok = true;
    if ((int64_t)chunks * kPbChunk > c->pb_ent_cap) {
        void* old[] = {c->pb_src, c->pb_sp, c->pb_row0, c->pb_lpos, c->pb_tmp, c->pb_dst, c->pb_wn, c->pb_val};
        for (void* q : old) dev_free(c, q);
        c->pb_src = c->pb_val = c->pb_row0 = c->pb_sp = nullptr;
        c->pb_lpos = c->pb_dst = nullptr;
        c->pb_tmp = c->pb_wn = nullptr;
        c->pb_ent_cap = 0;
        const int64_t cap = round_up(c->entries + c->entries / 8 + 1, kPbChunk);
        ok = try_alloc_n(c, c->pb_src, cap) && try_alloc_n(c, c->pb_sp, cap) &&
             try_alloc_n(c, c->pb_row0, cap / kPbChunk + 1) && try_alloc_n(c, c->pb_lpos, cap) &&
             try_alloc_n(c, c->pb_tmp, cap) && try_alloc_n(c, c->pb_dst, cap) && try_alloc_n(c, c->pb_wn, cap) &&
             try_alloc_n(c, c->pb_val, cap);
        if (ok) c->pb_ent_cap = cap;
    }
    if (ok && c->n > c->pb_vcap) {
        void* old[] = {c->pb_len, c->pb_upd, c->pb_first, c->pb_block};
        for (void* q : old) dev_free(c, q);
        c->pb_len = nullptr;
        c->pb_upd = c->pb_first = c->pb_block = nullptr;
        c->pb_vcap = 0;
        ok = try_alloc_n(c, c->pb_len, c->n_cap) && try_alloc_n(c, c->pb_upd, c->n_cap / 32 + 64) &&
             try_alloc_n(c, c->pb_first, c->n_cap + 1) && try_alloc_n(c, c->pb_block, c->n_cap / kBlock + 2);
        if (ok) c->pb_vcap = c->n_cap;
    }
    if (ok && !c->pb_bin) ok = try_alloc_n(c, c->pb_bin, 2 * (kPbMaxBins + 1));
    // rows 0 .. chunks of the table, then kPbSegs rows of segment sums
    if (ok && ((int64_t)chunks + 1 + kPbSegs) * nbins > c->pb_table_cap) {
        dev_free(c, c->pb_table);
        c->pb_table = nullptr;
        c->pb_table_cap = 0;
        const int64_t cap = ((int64_t)chunks + 1 + kPbSegs) * nbins + (int64_t)chunks * nbins / 8;
        ok = try_alloc_n(c, c->pb_table, cap);
        if (ok) c->pb_table_cap = cap;
    }
    if (!ok) {
        free_binned(c);
        return false;
    }
    unsigned int* bin_count = c->pb_bin;
    unsigned int* bin_off = c->pb_bin + (kPbMaxBins + 1);
    const unsigned int* num_entries = c->pb_first + c->n;
    const unsigned int vblocks = grid_for(c->n);
    hipLaunchKernelGGL(k_pb_receivers, dim3(grid_for(round_up(c->n, 64))), dim3(kBlock), 0, c->stream, c->n, c->meta,
                       c->seed_class, c->pb_len, c->pb_upd);
    hipLaunchKernelGGL(k_pb_row_blocks, dim3(vblocks), dim3(kBlock), 0, c->stream, c->n, c->meta, c->pb_block);
    hipLaunchKernelGGL(k_pb_scan_blocks, dim3(1), dim3(kBlock), 0, c->stream, (int64_t)vblocks, c->pb_block);
    hipLaunchKernelGGL(k_pb_row_first, dim3(vblocks), dim3(kBlock), 0, c->stream, c->n, c->meta, c->pb_block, c->pb_first);
    HIPCHK(c, hipGetLastError());
    // every array above is sized from the host's count of stored entries: it must be the device's
    unsigned int device_entries = 0;
    HIPCHK(c, hipMemcpyAsync(&device_entries, num_entries, sizeof device_entries, hipMemcpyDeviceToHost, c->stream));
    HIPCHK(c, hipStreamSynchronize(c->stream));
    if ((int64_t)device_entries != c->entries) {
        c->err = "internal error: the stored rows hold " + std::to_string(device_entries) + " entries, the context counts " +
                 std::to_string(c->entries);
        c->poisoned = true;
        throw Fail{DYNLP_ERR_STATE};
    }
    unsigned int* ecol = c->pb_val;  // scratch until the first scatter pass overwrites it
    unsigned int* too_wide = c->pb_row0 + c->pb_ent_cap / kPbChunk;  // the word after the last chunk's
    HIPCHK(c, hipMemsetAsync(too_wide, 0, sizeof(unsigned int), c->stream));
    hipLaunchKernelGGL(k_pb_expand, dim3(grid_for(c->n * 16)), dim3(kBlock), 0, c->stream, c->n, c->meta, c->pool, c->pb_first,
                       c->pb_src, ecol, c->pb_tmp, c->pb_row0);

    hipLaunchKernelGGL(k_pb_count, dim3(chunks), dim3(kBlock), 0, c->stream, num_entries, bits, nbins, ecol, c->pb_upd,
                       c->pb_table);
    unsigned int* seg = c->pb_table + ((size_t)chunks + 1) * nbins;
    const dim3 col_grid(grid_for(nbins), kPbSegs);
    hipLaunchKernelGGL(k_pb_seg_sums, col_grid, dim3(kBlock), 0, c->stream, nbins, chunks, c->pb_table, seg);
    hipLaunchKernelGGL(k_pb_seg_scan, dim3(grid_for(nbins)), dim3(kBlock), 0, c->stream, nbins, chunks, seg, c->pb_table,
                       bin_count);
    hipLaunchKernelGGL(k_pb_chunk_bases, col_grid, dim3(kBlock), 0, c->stream, nbins, chunks, seg, c->pb_table);
    hipLaunchKernelGGL(k_pb_offsets, dim3(1), dim3(kBlock), 0, c->stream, nbins, bin_count, bin_off);
    hipLaunchKernelGGL(k_pb_place, dim3(chunks), dim3(kPbPlaceThreads), 0, c->stream, num_entries, bits, nbins,
                       pb_run_lanes(nbins), ecol, c->pb_tmp, c->pb_upd, c->pb_table, bin_off, c->pb_lpos, c->pb_dst, c->pb_wn);
    hipLaunchKernelGGL(k_pb_pack, dim3(grid_for(c->entries)), dim3(kBlock), 0, c->stream, num_entries, c->pb_src, c->pb_lpos,
                       c->pb_row0, c->pb_sp, too_wide);
    hipLaunchKernelGGL(k_pb_normalise, dim3(nbins * kPbNormParts), dim3(kBlock), 0, c->stream, bits, bin_off, c->pb_dst,
                       c->deg, c->pb_wn);
    HIPCHK(c, hipGetLastError());
    c->pb_bits = bits;
    c->pb_bins = nbins;
    c->pb_chunks = chunks;
    // In-place mode: the round updates the vertices range by range (whole bins each) and publishes a range's new
    // labels before the next range is updated, which is what "a new row replaces the old one at once" means for
    // two streaming passes; fewer rounds are needed than with all ranges updated from the round-start labels.
    // Synchronous mode: one range.
    // A range's gather runs one workgroup per bin and one workgroup fills a CU: ranges of about one bin per CU keep
    // the whole chip busy (50M vertices, 1,526 bins, in-place batch: 2 / 4 / 6 / 8 / 16 ranges give 802 / 681 / 616 /
    // 622 / 731 ms against 956 ms with one).  Graphs with fewer bins than CUs keep one range.
    // (in the largest bins, where two workgroups share a CU)
    const int want_parts = c->update_mode != DYNLP_UPDATE_IN_PLACE ? 1
                           : c->binned > 0                         ? (int)ceil_div(nbins, std::max(1, c->num_cu))
                                           : (int)ceil_div(ceil_div(c->n, (int64_t)1 << kPbMaxBinBits), (int64_t)std::max(1, c->num_cu));
    const int parts = std::max(1, std::min({want_parts, kPbMaxParts, nbins}));
    c->pb_parts = parts;
    std::vector<unsigned int> first_at(parts + 1, 0u);
    unsigned int wide = 1;
    HIPCHK(c, hipMemcpyAsync(&wide, too_wide, sizeof wide, hipMemcpyDeviceToHost, c->stream));
    for (int i = 0; i <= parts; ++i) {
        const int b = (int)(((int64_t)nbins * i) / parts);
        c->pb_part_bin[i] = b;
        const int64_t v = std::min<int64_t>(c->n, (int64_t)b << bits);
        HIPCHK(c, hipMemcpyAsync(&first_at[i], c->pb_first + v, sizeof(unsigned int), hipMemcpyDeviceToHost, c->stream));
    }
    HIPCHK(c, hipStreamSynchronize(c->stream));
    for (int i = 0; i < parts; ++i) {
        c->pb_part_chunk[i][0] = (int)(first_at[i] / kPbChunk);
        c->pb_part_chunk[i][1] = (int)std::min<int64_t>(chunks, ceil_div((int64_t)first_at[i + 1], kPbChunk));
        if (first_at[i + 1] == first_at[i]) c->pb_part_chunk[i][1] = c->pb_part_chunk[i][0];  // no entries: nothing to publish
    }
    c->pb_packed_ok = wide == 0;
    c->pb_built = true;
    return true;
}

// One binned round: scatter pass + gather pass (arguments as for the fused round).
void launch_pb_scatter(dynlp_ctx* c, const RoundCtr* prev, int chunk0, int nchunks, const float* F, const unsigned int* bits,
                       unsigned int* moved_clear, RoundCtr* ctr_zero, const unsigned int* bits_also = nullptr, int flags = 0) {
    if (nchunks <= 0 && !ctr_zero && !moved_clear) return;
    const int lg = pb_run_lanes(c->pb_bins);
    const dim3 grid(8 * (unsigned int)std::max<int64_t>(1, ceil_div(nchunks, 8)));
    const unsigned int* bin_off = c->pb_bin + (kPbMaxBins + 1);
#define DYNLP_SCATTER(NB, PACKED, SRC)                                                                                     \
    hipLaunchKernelGGL((k_pb_scatter<NB, PACKED>), grid, dim3(kPbScatterThreads), 0, c->stream, prev, c->pb_first + c->n,      \
                       (unsigned int)chunk0, (unsigned int)std::max(nchunks, 0), c->pb_bins, lg, SRC, c->pb_row0, c->pb_lpos,  \
                       c->pb_table, bin_off, F, bits, bits_also, moved_clear, (unsigned int)c->moved_words, c->pb_val,         \
                       flags, ctr_zero)
    if (c->pb_bins <= 2048 && c->pb_packed_ok) DYNLP_SCATTER(2048, true, c->pb_sp);
    else if (c->pb_bins <= 2048) DYNLP_SCATTER(2048, false, c->pb_src);
    else if (c->pb_packed_ok) DYNLP_SCATTER(kPbMaxBins, true, c->pb_sp);
    else DYNLP_SCATTER(kPbMaxBins, false, c->pb_src);
#undef DYNLP_SCATTER
}

// One binned round (arguments as for the fused round).  `first_of_stretch`: no binned round has run since the slots
// were last brought up to date with the labels.
// One range (synchronous mode): scatter all labels, gather all bins: a Jacobi round.
// Several ranges (in-place mode): the slots are kept up to date between rounds; the round updates range after range,
// each gather followed by the scatter that publishes the range's new labels, so that later ranges of the same round
// already read them.  A published label carries "the sender moved in this round or in the previous one": ranges that
// come later in this round and ranges that come earlier in the next one both have to learn that it moved, and each
// sees only one publication.  V_aff of a round is then a superset of Alg. 2's (a row may be updated once more than
// needed), as with any in-place round that reads rows the same round has already replaced.
void launch_pb_gather(dynlp_ctx* c, const PullRoundArgs& a, int b0, int b1) {
    const unsigned int* bin_off = c->pb_bin + (kPbMaxBins + 1);
    allow_gather_lds(c, k_pb_gather);
    hipLaunchKernelGGL(k_pb_gather, dim3(b1 - b0), dim3(kPbGatherThreads), pb_gather_lds(c->pb_bits), c->stream, a.prev, c->n, c->pb_bits, (unsigned int)b0,
                       bin_off, c->pb_dst, c->pb_wn, c->pb_val, c->pb_len, a.F_in, a.F_out, a.moved_prev, a.moved_cur, a.tol,
                       a.flags, a.omega, a.ctr);
}

void launch_binned_round(dynlp_ctx* c, const PullRoundArgs& a, int round, bool first_of_stretch) {
    hipEvent_t e1 = open_timed_span(c, round, 1);
    if (c->pb_parts <= 1 || (a.flags & kRoundAll)) {  // rounds over all rows are Jacobi rounds in both modes
        launch_pb_scatter(c, a.prev, 0, c->pb_chunks, a.F_in, a.moved_prev, a.moved_clear, a.ctr_zero, nullptr, a.flags);
        launch_pb_gather(c, a, 0, c->pb_bins);
    } else {
        // bring every slot up to date once (labels and "moved in the previous round" bits); this launch also clears
        // the next round's counter slot and bitmap, as the first launch of every round does
        if (first_of_stretch) launch_pb_scatter(c, a.prev, 0, c->pb_chunks, a.F_in, a.moved_prev, nullptr, nullptr);
        for (int i = 0; i < c->pb_parts; ++i) {
            const int b0 = c->pb_part_bin[i], b1 = c->pb_part_bin[i + 1];
            if (i == 0) launch_pb_scatter(c, a.prev, 0, 0, a.F_in, a.moved_prev, a.moved_clear, a.ctr_zero);
            if (b1 > b0) launch_pb_gather(c, a, b0, b1);
            launch_pb_scatter(c, a.prev, c->pb_part_chunk[i][0], c->pb_part_chunk[i][1] - c->pb_part_chunk[i][0], a.F_out,
                              a.moved_cur, nullptr, nullptr, a.moved_prev);
        }
    }
    HIPCHK(c, hipGetLastError());
    close_timed_span(c, e1);
}

// ---- packed rounds (dynlp_packed.h) -----------------------------------------------------------------
// Below kPackedMinRows a round over all rows is a launch and its drain whichever kernel it runs (20,000 vertices of
// degree 8: 9 us with the row update) and the layout of the entries is one more thing to wait for.
constexpr unsigned int kPackedMinRows = 32768;
// kPackedShare: see packed_rounds_pay; kPackedUneven: a part with more than this many times the mean entries would keep
// the round waiting for one CU (us per round, row update / packed, largest part 1 / 2 / 3 / 4 times the mean: 150,000 vertices
// of degree 20 with 10 columns 61 / 37, 61 / 56, 63 / 77, 64 / 93; with 29 columns 73 / 49, 73 / 75, 72 / 102, 74 / 128;
// 400,000 with 10 columns 152 / 78, 151 / 133, 152 / 183, 155 / 235).  kPackedMaxRow: longer rows would show the unit of the
// packed sums (see dynlp_packed.h).
constexpr unsigned int kPackedMaxRow = 8192;
constexpr double kPackedShare = 0.6, kPackedUneven = 2.0;
// A row's share of a part's time, in entries: its sums are cleared, its old row read and its new one written.
constexpr unsigned int kPackedRowCost = 4;
// A longest row of more than one in kPackedSpread of a part's entries: its entries are spread over their buckets (k_pk_place).
constexpr double kPackedSpread = 16.0;
// Above kPackedMaxTol a synchronous run stops so far from the fixed point (the threshold times the steps of a random walk
// to a labelled vertex) that the last bits of a row decide visibly where: a row that moves by the threshold to within
// rounding enters V_aff or not and takes its neighbours along.  With tol = 1e-4 on 1,000,000 vertices two solves that
// agree to 7e-8 are 1.4e-4 apart after a batch (2-norm, relative).  Such runs keep the sums of the row update.
constexpr float kPackedMaxTol = 1e-5f;
struct PackedPlan {
    int rows, parts, col_bits, bucket_bits;  // rows: as many as a part may have
};

int packed_stride(const dynlp_ctx* c) { return c->Cs == 1 ? 1 : (c->Cs + 1) / 2 * 2; }

// Whether Jacobi rounds over nearly all vertices should run as packed rounds, and how the graph is cut for them.
bool packed_rounds_pay(const dynlp_ctx* c, const Frontier& universe, PackedPlan* plan) {
    // (a caller who fixes the lanes per row asks for the row update)
    if (c->group_lanes != 0 || (c->CP == 1 && c->binned != 0) || universe.size() < kPackedMinRows || c->entries >= ((int64_t)1 << 31)) return false;
    if (c->tol > kPackedMaxTol) return false;
    // parts: as many generations of one workgroup per CU as the sums need, of equal size
    const int row_bits8 = packed_stride(c) * 32 + 2;  // bits of LDS per row: the sums, "in V_aff", "moved"
    const int64_t rows_max = std::min<int64_t>((int64_t)(kPkLds - kPkFixedLds) * 8 / row_bits8 / 32 * 32, kPkMaxRows);
    const int64_t wide = c->num_cu;
    const int64_t gens = ceil_div(c->n, wide * rows_max);
    const int64_t rows = round_up(ceil_div(c->n, wide * gens), 32);
    int row_bits = 5, col_bits = 1;
    while (((int64_t)1 << row_bits) < rows) ++row_bits;
    while (((int64_t)1 << col_bits) < c->n) ++col_bits;
    // an entry keeps its row's place in the part and its neighbour's id in one word, which ends the packed rounds at about
    // 2^20 vertices with up to 15 columns, 2^21 with 17 to 33 and 2^22 with 50 and more
    if (row_bits + col_bits > 32) return false;
    int bucket_bits = 0;
    while (((c->n - 1) >> bucket_bits) >= kPkBuckets) ++bucket_bits;
    if (c->n * c->CP * 4 >= ((int64_t)1 << 32)) return false;  // byte offsets of label rows are 32-bit
    // Bytes over the fabric: every XCD reads the label matrix once per generation; the row update reads one or two
    // lines per entry.  Measured (share of the row update's bytes, time packed / ordinary): 1,000,000 vertices of degree
    // 20 with 10 columns 0.20, 0.45; 300,000 of degree 16 with 29 columns 0.50, 0.65; 1,000,000 of degree 38 with 50
    // columns would need 5 generations: 1.05 (not faster).
    const double packed = 8.0 * (double)gens * (double)c->n * c->CP * 4.0;
    const double ordinary = (double)c->entries * std::max(128.0, c->CP * 4.0);
    if (packed > kPackedShare * ordinary) return false;
    *plan = PackedPlan{(int)std::min<int64_t>(rows_max, (int64_t)1 << (32 - col_bits)), (int)ceil_div(c->n, rows), col_bits, bucket_bits};
    return true;
}

void free_packed(dynlp_ctx* c) {
    dev_free(c, c->pk_ent);
    dev_free(c, c->pk_len);
    dev_free(c, c->pk_deg);
    dev_free(c, c->pk_tab);
    c->pk_ent = nullptr;
    c->pk_len = nullptr;
    c->pk_deg = nullptr;
    c->pk_tab = nullptr;
    c->pk_ent_cap = c->pk_vcap = c->pk_tab_cap = 0;
    c->pk_built = false;
}

size_t packed_lds(const dynlp_ctx* c) { return (size_t)c->pk_rows * packed_stride(c) * 4 + (size_t)c->pk_rows / 32 * 8; }

template <int CP, int LANES>
struct PackedShape {
    static constexpr int cp = CP, lanes = LANES;
};

// Calls fn with the columns and lanes of the context's packed rounds.
template <typename Fn>
auto packed_kernel(const dynlp_ctx* c, Fn fn) {
    switch (c->CP > 4 ? (c->Cs + 3) / 4 : c->CP == 4 ? 1 : -c->CP) {
        case -1: return fn(PackedShape<1, 1>{});
        case -2: return fn(PackedShape<2, 1>{});
        case 1: return fn(PackedShape<4, 1>{});
        case 2: return fn(PackedShape<8, 2>{});
        case 3: return fn(PackedShape<16, 3>{});
        case 4: return fn(PackedShape<16, 4>{});
        case 5: return fn(PackedShape<32, 5>{});
        case 6: return fn(PackedShape<32, 6>{});
        case 7: return fn(PackedShape<32, 7>{});
        case 8: return fn(PackedShape<32, 8>{});
        case 9: return fn(PackedShape<64, 9>{});
        case 10: return fn(PackedShape<64, 10>{});
        case 11: return fn(PackedShape<64, 11>{});
        case 12: return fn(PackedShape<64, 12>{});
        case 13: return fn(PackedShape<64, 13>{});
        case 14: return fn(PackedShape<64, 14>{});
        case 15: return fn(PackedShape<64, 15>{});
        default: return fn(PackedShape<64, 16>{});
    }
}

// Lays the entries of the graph as it stands out for the packed rounds (universe: all updatable vertices).  False: no
// memory, parts so uneven that the largest would keep a round waiting, or a row that is too long (no array of entries is
// kept); the caller then runs ordinary rounds.
bool build_packed(dynlp_ctx* c, const Frontier& universe, const PackedPlan& plan) {
    const int64_t parts = plan.parts, ent = std::max<int64_t>(c->entries, 1), granules = ceil_div(c->n, 32);
    const int64_t tab = 2 * (parts + 1) + 3 + granules;
    bool ok = true;
    if (c->n > c->pk_vcap) {
        dev_free(c, c->pk_len);
        dev_free(c, c->pk_deg);
        c->pk_len = nullptr;
        c->pk_deg = nullptr;
        c->pk_vcap = 0;
        ok = try_alloc_n(c, c->pk_len, c->n_cap) && try_alloc_n(c, c->pk_deg, c->n_cap);
        if (ok) c->pk_vcap = c->n_cap;
    }
    if (ok && tab > c->pk_tab_cap) {
        dev_free(c, c->pk_tab);
        c->pk_tab = nullptr;
        c->pk_tab_cap = 0;
        ok = try_alloc_n(c, c->pk_tab, tab + tab / 8);
        if (ok) c->pk_tab_cap = tab + tab / 8;
    }
    c->pk_parts = plan.parts;
    c->pk_bits = plan.col_bits;
    if (ok) {
        // always the same value: the attribute belongs to the kernel, not to this context
        hipError_t e = packed_kernel(c, [&](auto shape) {
            using S = decltype(shape);
            const void* kernels[] = {reinterpret_cast<const void*>(&k_pk_round<S::cp, S::lanes>),
                                     reinterpret_cast<const void*>(&k_pk_product<S::cp, S::lanes>)};
            hipError_t worst = hipSuccess;
            for (const void* k : kernels) {
                const hipError_t r = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, kPkLds - kPkFixedLds);
                if (r != hipSuccess) worst = r;
            }
            return worst;
        });
        if (e == hipSuccess)
            e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_pk_place), hipFuncAttributeMaxDynamicSharedMemorySize,
                                    kPkPlaceLds);
        if (e != hipSuccess) {
            (void)hipGetLastError();
            ok = false;
        }
    }
    if (!ok) {
        free_packed(c);
        return false;
    }
    unsigned int* start = c->pk_tab;
    unsigned int* largest = start + parts + 1;
    unsigned int* bound = largest + 3;
    unsigned int* gran = bound + parts + 1;
    HIPCHK(c, hipMemsetAsync(largest + 2, 0, sizeof(unsigned int), c->stream));
    hipLaunchKernelGGL(k_pk_receivers, dim3(grid_for(c->n)), dim3(kBlock), 0, c->stream, c->n, c->meta, c->seed_class, c->deg,
                       c->pk_len, c->pk_deg, gran, largest + 2);
    hipLaunchKernelGGL(k_pk_bounds, dim3(1), dim3(kPkThreads), 0, c->stream, c->n, (int)granules, plan.parts, kPackedRowCost,
                       (unsigned int)plan.rows, gran, bound, start, largest);
    HIPCHK(c, hipGetLastError());
    unsigned int most[3] = {0, 0, 0};  // entries and rows of a part, longest row
    HIPCHK(c, hipMemcpyAsync(most, largest, sizeof most, hipMemcpyDeviceToHost, c->stream));
    HIPCHK(c, hipStreamSynchronize(c->stream));
    const bool refused = (double)most[0] > kPackedUneven * (double)ent / (double)parts || most[2] > kPackedMaxRow ||
                         most[1] > (unsigned int)plan.rows;
    c->pk_rows = (int)most[1];
    if (refused || ent > c->pk_ent_cap) {
        dev_free(c, c->pk_ent);
        c->pk_ent = nullptr;
        c->pk_ent_cap = 0;
        if (refused) return false;
        if (!try_alloc_n(c, c->pk_ent, ent + ent / 8)) {
            free_packed(c);
            return false;
        }
        c->pk_ent_cap = ent + ent / 8;
    }
    if (universe.nl)
        hipLaunchKernelGGL(k_pk_long_degrees, dim3(std::min<unsigned int>(universe.nl, (unsigned int)c->num_cu * 8)), dim3(kBlock), 0,
                           c->stream, universe.nl, universe.back, c->meta, c->pool, c->pk_deg);
    const int spread = (double)most[2] * kPackedSpread > (double)ent / (double)parts ? 1 : 0;
    // tiles as large as the running row lengths leave room for
    const size_t lengths = (size_t)(c->pk_rows + 1) * sizeof(unsigned int);
    unsigned int tile = kPkTile;
    while (tile * sizeof(PkEntry) + lengths > (size_t)kPkPlaceLds) tile /= 2;
    hipLaunchKernelGGL(k_pk_place, dim3(plan.parts), dim3(kPkThreads), tile * sizeof(PkEntry) + lengths, c->stream, c->n, bound, plan.col_bits,
                       plan.bucket_bits, tile, spread, c->meta, c->pool, c->pk_len, c->pk_deg, start, c->pk_ent);
    HIPCHK(c, hipGetLastError());
    c->pk_built = true;
    return true;
}

// One packed round (arguments as for the fused round).
void launch_packed_round(dynlp_ctx* c, const PullRoundArgs& a, int round) {
    hipEvent_t e1 = open_timed_span(c, round, 1);
    const PkRound r{a.prev, a.ctr, a.ctr_zero, c->n, c->pk_rows, c->pk_tab + c->pk_parts + 4, c->Cs, packed_stride(c), c->pk_bits, c->pk_ent, c->pk_tab,
                    c->pk_len, c->meta, c->pool, a.F_in, a.F_out, a.moved_prev, a.moved_cur, a.moved_clear,
                    (unsigned int)c->moved_words, a.tol, a.flags, a.omega};
    const dim3 grid((unsigned int)c->pk_parts), block(kPkThreads);
    packed_kernel(c, [&](auto shape) {
        using S = decltype(shape);
        hipLaunchKernelGGL((k_pk_round<S::cp, S::lanes>), grid, block, packed_lds(c), c->stream, r);
    });
    HIPCHK(c, hipGetLastError());
    close_timed_span(c, e1);
}

// Resolve the per-round events into the round log; returns the summed device time of all
// row-update launches.  (After a wait for the stream: that counters have arrived does not mean that events have.)
float collect_kernel_ms(dynlp_ctx* c) {
    float total = 0.f;
    for (size_t k = 0; 2 * k + 1 < c->events_used; ++k) {
        float a = 0.f;
        HIPCHK(c, hipEventElapsedTime(&a, c->events[c->ev_first[k]], c->events[c->ev_last[k]]));
        total += a;
        const int first = c->ev_round[k];
        if (first < 0) continue;
        const int last = std::min<int>(first + c->ev_count[k], (int)c->log.size());
        for (int t = first; t < last; ++t) c->log[t].ms_update += a / (float)std::max(1, last - first);
    }
    reset_timed_spans(c);
    return total;
}

dynlp_round_info round_info(const RoundCtr& r, int kind, int G) {
    dynlp_round_info ri;
    std::memset(&ri, 0, sizeof ri);
    ri.rows_short = r.rows_short;
    ri.rows_long = r.rows_long;
    ri.entries_short = (int64_t)r.edges;
    ri.entries_long = (int64_t)r.edges_long;
    std::memcpy(&ri.max_delta, &r.resid_bits, sizeof(float));
    ri.rows_moved = r.changed;
    ri.staged = kind;
    ri.group_lanes = G;
    return ri;
}

// flag bytes (or, with all_rows, every updatable vertex) -> frontier `out`; the two counts land in
// *count_short / *count_long, which must be zero beforehand.
void launch_compact(dynlp_ctx* c, const Frontier& out, unsigned int* count_short, unsigned int* count_long,
                    int all_rows) {
    if (c->n >= (16 << 20)) {
        const unsigned int blocks = (unsigned int)ceil_div(std::max<int64_t>(c->n, 1), 4 * kFlagsPerBlock);
        hipLaunchKernelGGL(k_compact<4>, dim3(blocks), dim3(kBlock), 0, c->stream, (unsigned int)c->n, c->flag, c->seed_class,
                           c->meta, all_rows, out.front, out.back, count_short, count_long);
    } else {
        const unsigned int blocks = (unsigned int)ceil_div(std::max<int64_t>(c->n, 1), kFlagsPerBlock);
        hipLaunchKernelGGL(k_compact<1>, dim3(blocks), dim3(kBlock), 0, c->stream, (unsigned int)c->n, c->flag, c->seed_class,
                           c->meta, all_rows, out.front, out.back, count_short, count_long);
    }
    HIPCHK(c, hipGetLastError());
}

// After a staged round over `f`: commit and next list (`out`; its counts as for launch_compact).
void launch_commit_compact(dynlp_ctx* c, const Frontier& f, const RoundCtr* prev, int64_t rows_bound, const Frontier& out,
                           unsigned int* count_short, unsigned int* count_long) {
    const int64_t items = rows_bound * (c->CP >= 4 ? c->CP / 4 : c->CP);
    const unsigned int commit = (unsigned int)std::max<int64_t>(1, std::min<int64_t>(ceil_div(items, kBlock), (int64_t)c->num_cu * 8));
    const int seg = c->n >= (16 << 20) ? 4 : 1;
    const unsigned int compact = (unsigned int)ceil_div(std::max<int64_t>(c->n, 1), seg * kFlagsPerBlock);
    auto kernel = seg == 4 ? k_commit_compact<4> : k_commit_compact<1>;
    hipLaunchKernelGGL(kernel, dim3(compact + commit), dim3(kBlock), 0, c->stream, compact, (unsigned int)c->n, c->flag, c->seed_class,
                       c->meta, out.front, out.back, count_short, count_long, prev, f.front, f.back, c->F2, c->F, c->CP);
    HIPCHK(c, hipGetLastError());
}

// Pull the next V_aff out of the round's "moved" bitmap straight into the frontier `out` (its counts go to
// *count_short / *count_long, zero beforehand); F_new holds the rows just written, F_old the round-start
// rows; `universe` lists every updatable vertex.
template <int SUB>
void launch_pull_frontier_inst(dynlp_ctx* c, const Frontier& universe, const unsigned int* moved, unsigned int* moved_next,
                               const float* F_new, float* F_old, const Frontier& out, unsigned int* count_short,
                               unsigned int* count_long) {
    const int64_t cap = (int64_t)c->num_cu * 8;
    const unsigned int long_blocks =
        (unsigned int)std::min<int64_t>(ceil_div(universe.nl, (kBlock / kWave) * SUB), cap / 2);
    const unsigned int short_blocks =
        (unsigned int)std::max<int64_t>(1, std::min<int64_t>(ceil_div(universe.ns, kBlock * SUB), cap));
    hipLaunchKernelGGL(k_pull_frontier<SUB>, dim3(long_blocks + short_blocks), dim3(kBlock), 0, c->stream, universe.ns,
                       universe.nl, long_blocks, universe.front, universe.back, moved, moved_next, (unsigned int)c->moved_words,
                       F_new, F_old, c->CP,
                       c->meta, c->pool, out.front, out.back, count_short, count_long);
    HIPCHK(c, hipGetLastError());
}

void launch_pull_frontier(dynlp_ctx* c, const Frontier& universe, double avg_len, const unsigned int* moved,
                          unsigned int* moved_next, const float* F_new, float* F_old, const Frontier& out,
                          unsigned int* count_short, unsigned int* count_long) {
    // measured: 10M vertices of mean degree 38 want the large chunks (0.21 vs 0.41 ms per round), 1M vertices of
    // degree 20, 100K vertices and 50M vertices of degree 5 the small ones
    if (universe.size() >= (2u << 20) && avg_len >= 16.0)
        launch_pull_frontier_inst<16>(c, universe, moved, moved_next, F_new, F_old, out, count_short, count_long);
    else
        launch_pull_frontier_inst<4>(c, universe, moved, moved_next, F_new, F_old, out, count_short, count_long);
}

// Whether a ping-pong stretch should run rounds that evaluate V_aff themselves (k_row_update_pull) rather than
// pairs of row update and pull.  The fused round saves the pull's pass over the graph but puts the membership test
// (one more dependent look-up for rows that did not move themselves) in front of every row's gathers.
bool fused_rounds_pay(const dynlp_ctx* c, double avg_len) {
    // Measured on MI355X, batches of 1% new vertices, whole batch, fused against separate: 1M vertices of mean
    // degree 20 with 10 / 32 / 64 classes 68 / 78 / 112 ms against 80 / 89 / 138 ms; 2M vertices of mean degree 38
    // with 10 / 20 classes 611 / 766 ms against 660 / 827 ms; 50M vertices of degree 5, one column, 1.54 s against
    // 1.89 s; but 10M vertices of mean degree 38 with 50 classes 14.9 ms per round against 14.3 + 0.2 ms.  The
    // rule below separates the two groups by the bytes a row's update reads.
    return avg_len * (double)(c->CP * 4 + 8) < 8192.0;
}

// Ping-pong stretches begin when V_aff holds at least kDenseEnter of the updatable vertices and end
// when it falls below kDenseLeave (the pull over all updatable vertices stops paying off).
constexpr double kDenseEnter = 0.90, kDenseLeave = 0.75;
// A binned round costs the same whatever the size of V_aff (two streams over the whole graph), about a quarter of an
// ordinary round over all rows, and a flag-marking round over a third of the rows already costs more: such stretches
// begin and end at smaller V_aff.  50M-vertex random graph, one batch, enter / leave at 0.50 / 0.35 against 0.35 / 0.20:
// synchronous 762 -> 738 ms, with supernode initialisation 367 -> 342 ms, in place with it 332 -> 270 ms (in place
// from uniform rows V_aff collapses within one chain of rounds and nothing changes); 0.20 / 0.10 is no better.
constexpr double kBinnedEnter = 0.35, kBinnedLeave = 0.20;
// A packed round costs about half an ordinary round over all rows while nearly all of them move; the fewer do, the more rows
// must look their neighbours up to know whether they are in V_aff (us per round with V_aff = 99%, packed / fused, all rows
// move - half do: 900,000 scalar rows of degree 6 56 / 77 - 94 / 88, two columns 58 / 96 - 104 / 104, 300,000 rows of 10
// columns 54 / 113 - 69 / 113), and the layout of the entries has to be earned.  Stretches therefore begin at a chain whose
// last round moved kPackedMoved of all rows (whole batches, without packed rounds / beginning at V_aff = 50% / now, tol =
// 1e-6: 1M planted blocks 5.2 / 6.4 / 5.2 ms, 500K 8.1 / 9.4 / 8.2, 900K scalar 3.0 / 3.7 / 3.0, 400K scalar 14.7 / 11.2 /
// 11.2, 60K kNN 20.6 / 17.2 / 17.2, 150K power law 38.7 / 29.9 / 30.5).
constexpr double kPackedMoved = 0.97, kPackedLeave = 0.35;

// The ping-pong partner must agree with F on every row a full sweep does not write (seeds,
// isolated vertices) before it can receive one.
void sync_partner(dynlp_ctx* c) {
    if (c->n > 0)
        HIPCHK(c, hipMemcpyAsync(c->F2, c->F, (size_t)c->n * c->CP * sizeof(float), hipMemcpyDeviceToDevice, c->stream));
}

void zero_ring(dynlp_ctx* c) {
    HIPCHK(c, hipMemsetAsync(c->ring, 0, sizeof(RoundCtr) * (kRing + 1), c->stream));
}

// Slot of round t; round -1 is the start slot that holds the size of the first frontier.
RoundCtr* slot_of(dynlp_ctx* c, int t) { return t < 0 ? c->ring + kRing : c->ring + (t % kRing); }

// Fold a copied slot's partial records into its header fields.
void fold_slot(RoundCtr& r) {
    r.resid_bits = 0;
    r.changed = 0;
    r.edges = 0;
    r.edges_long = 0;
    for (const RoundPart& p : r.part) {
        r.rows_short += p.rows_short;  // only rounds that find their own V_aff count rows here
        r.rows_long += p.rows_long;
        r.resid_bits = std::max(r.resid_bits, p.resid_bits);
        r.changed += p.changed;
        r.edges += p.edges;
        r.edges_long += p.edges_long;
    }
}

// Copy the slots of rounds [t0, t0 + count) to the host (count <= kRing) and wait for them.
void read_slots(dynlp_ctx* c, int t0, int count) {
    const int at = t0 % kRing, run = std::min(count, kRing - at);
    read_to_host(c, c->h_slot, c->ring + at, sizeof(RoundCtr) * (size_t)run, c->ring, sizeof(RoundCtr) * (size_t)(count - run));
    for (int i = 0; i < count; ++i) fold_slot(c->h_slot[i]);
}

// The start slot and the batch counters, in one copy.
void read_start(dynlp_ctx* c) {
    read_to_host(c, c->h_start, c->ring + kRing, sizeof(dynlp_ctx::HostStart));
}

// The first frontier of a batch (its size goes to the start slot) and the list of all updatable vertices; waits for their sizes.
void launch_compact_start(dynlp_ctx* c, const Frontier& out, const Frontier& universe, const BatchGate& gate) {
    // few vertices: more workgroups, each with one trip to memory; many: fewer additions to the four counters (us with 4 / 8 / 16
    // steps: 100,000 vertices 6.9 / 9.1 / 14.7, 300,000 9.6 / 10.0 / 14.3, 1M 18.5 / 15.8 / 17.7, 3M - / 33.3 / 29.5)
    const int steps = c->n >= (16 << 20) ? 64 : c->n >= (2 << 20) ? 16 : c->n >= (512 << 10) ? 8 : 4;
    const unsigned int blocks = (unsigned int)ceil_div(std::max<int64_t>(c->n, 1), start_block_rows(steps));
    auto kernel = steps == 64   ? k_compact_start<64>
                  : steps == 16 ? k_compact_start<16>
                  : steps == 8  ? k_compact_start<8>
                                : k_compact_start<4>;
    // the sizes go to the host with the last of few workgroups (many would queue for the counter that tells which is the last)
    const bool send = blocks <= 256;
    const StartToHost to{reinterpret_cast<unsigned long long*>(c->h_start), (unsigned int)(sizeof(dynlp_ctx::HostStart) / 8),
                         send ? c->h_flag : nullptr, send ? ++c->h_sent : 0u};
    hipLaunchKernelGGL(kernel, dim3(blocks), dim3(kBlock), 0, c->stream, (unsigned int)c->n, c->flag, c->seed_class, c->meta, out.front,
                       out.back, c->ring + kRing, universe.front, universe.back, c->bc, gate, to);
    HIPCHK(c, hipGetLastError());
    if (send) wait_for_flag(c, to.value);
    else read_start(c);
}

void read_slots_start(dynlp_ctx* c) {
    HIPCHK(c, hipMemcpyAsync(c->h_slot, c->ring + kRing, sizeof(RoundCtr), hipMemcpyDeviceToHost, c->stream));
    HIPCHK(c, hipStreamSynchronize(c->stream));
}

// ---- relaxed rounds (in-place mode) ----------------------------------------------------------------------------
// Rows updated in place need far fewer rounds than Jacobi rounds, but still one per step of the random walks that carry
// a label from the labelled vertices: 200 to 600 rounds at tol = 1e-6 on graphs with 1% labelled vertices.  While nearly
// every row is in V_aff and the threshold is tight, the in-place mode therefore relaxes all rows together,
//     F(k+1) = omega * (weighted mean of F(k)) + (1 - omega) * F(k-1)
// (second-order Richardson iteration, Golub and Varga 1961; the first round is an ordinary one, without which a component
// that oscillates would start with omega / (2 - omega) times its amplitude): it converges for every 0 < omega < 2 because the
// eigenvalues of the update lie in [-1, 1], and with omega = 2 / (1 + sqrt(1 - mu^2)) an error shrinks by
// sqrt(omega - 1) per round instead of mu, the update's largest eigenvalue.  mu is at least the Rayleigh quotient of the
// constant vector, 1 - (weight of the edges to labelled vertices) / (weight of all edges of updatable rows); kRelaxGap
// times the sampled quotient's distance from 1, kept above kRelaxMinGap, sets omega.  When rows stop moving, one ordinary
// round over all rows decides what is in V_aff, and Step 3 goes on as it is listed: the stop rule and what it guarantees
// stay what they are without relaxation.  A phase that does not settle within four times the rounds the theory gives for a
// factor of 1e-7 ends the same way, and so does one in which neither the largest move nor the number of rows that move has
// fallen by 1% in 32 rounds (128 while all rows move: the others may be on their way behind a few that do not settle):
// components without a labelled vertex can oscillate for ever (36,000 rows beside 39,000 such rows: 401 relaxed rounds
// without this rule, 105 with it).
// Measured, ms per call at tol = 1e-6 (second row: distance from the exact labels, 2-norm, relative):
//   kRelaxGap                       none     0.7     0.8     0.9     1.0    1.15     1.3     1.5     2.0
//   1M planted blocks, 10 classes   41.2    11.3    11.3     9.9     9.9     9.8    10.1    10.1    10.8
//                                 1.9e-4  3.7e-6  2.3e-6  6.7e-6  3.3e-5  4.6e-5  4.5e-5  5.2e-5  8.7e-5
//   300K planted blocks, 29         35.1     8.3     7.8     7.6     7.4     7.4     7.4     7.8     8.6
//   1M power law, 50 classes         627     114      98     115     124     134     144     157     183
//                                 4.7e-4  9.0e-5  1.5e-5  2.3e-5  3.7e-5  7.4e-5  8.7e-5  1.0e-4  1.3e-4
//   120K power law, 20 classes      24.4    3.70    3.42    3.73    3.85    4.12    4.28    4.54    5.20
//   100K kNN, 10 classes            18.9    2.50    2.57    2.84    3.01    3.24    3.43    3.72    3.95
//   50K kNN, 6 classes              12.4    1.75    1.71    1.92    2.01    2.15    2.36    2.50    2.77
//   50M scalar, one batch            371     204     197     187     188     178     176     186     187
// (50M: fastest of five; allocating its arrays takes 5 to 1,700 ms once the process has used all device memory before.)
// With 0.9 the phase can end a chain earlier and further off; three inputs, 0.8 / 0.85 / 0.9: 300K planted blocks from cold
// 4.9 / 4.8 / 4.6 ms at 1.0e-6 / 7e-7 / 1.0e-5, 600K 5.1 / 5.1 / 4.7 ms at 5e-7 / 1.3e-6 / 8e-6, 1M 11.2 / 11.1 / 10.6 ms at
// 1.1e-6 / 4.7e-6 / 9e-6, 100K kNN 2.65 / 2.70 / 2.79 ms at 6e-6 / 7e-6 / 7e-6, 1M power law 103 / 110 / 118 ms at 4.6e-5 /
// 9e-6 / 3.1e-5.
// kRelaxLeave, the share of moved rows below which the phase ends: 0.05 ... 0.25 within 12% of each other on these graphs;
// 0.5: 100K kNN 2.85 -> 2.48 ms, but 50K kNN 1.84 -> 3.96 ms (201 rounds); 0.75: 5.5 and 5.4 ms.
// kRelaxMinGap keeps omega from 2 where labels are scarce.  300K planted blocks, 0.1% labelled: 67 ms without relaxation,
// 9.0 / 9.2 / 11.5 / 14.1 / 16.9 ms with 5e-4 / 1e-3 / 2e-3 / 4e-3 / 8e-3; 0.01%: 406 ms, 43 / 52 / 57 / 41 / 29 ms at
// 1.3e-3 / 1.8e-3 / 3.6e-3 / 8.0e-3 / 1.5e-2 from the exact labels; 0.001%: 2.1 s without and with 2e-3, 51 ms with 1e-5.
// Not used: for loose thresholds, where Step 3 is over in ten or twenty rounds and the relaxed rounds would only go on past
// it (kRelaxMaxTol; tol = 3e-5, without and with: 300K planted blocks 2.6 / 5.5, 1M 3.2 / 5.5, 1M power law 80 / 67, 100K
// kNN 7.2 / 1.9 ms); for thresholds below what float32 rounding leaves moving (kRelaxMinTol; tol = 1e-7: 100K kNN 37 / 7.0,
// but one pass of five 141 ms, 50K kNN 19 / 29 ms).  Between kRelaxNowTol and kRelaxMaxTol a batch has one chain of ordinary
// rounds first, in which V_aff collapses on the graphs that need no more (ms without / at once / after a chain; tol = 1e-5:
// 1M planted blocks 3.7 / 6.9 / 3.3, 600K 2.1 / 3.7 / 1.9, 300K 15.9 / 6.1 / 4.9, 250K power law 9.1 / 3.6 / 4.2, 100K kNN
// 10.5 / 2.1 / 2.5; 5e-6: 5.1 / 8.3 / 4.0, 3.5 / 3.8 / 2.2, 21 / 6.2 / 5.5, 12.6 / 4.2 / 4.5, 12.6 / 2.3 / 2.7; 3e-6: 6.8 /
// 8.3 / 12.6, 8.5 / 4.4 / 4.7, 26 / 6.8 / 5.9, 14.6 / 4.2 / 4.8, 14.4 / 2.6 / 2.7; 2e-6, without / at once: 1M 24 / 9.5).
// kRelaxMinRows is where packed rounds begin; smaller graphs would gain as well (8,000 planted vertices 8.2 -> 1.2 ms,
// 16,000 kNN 7.1 -> 1.2 ms), but in-place calls on them are held to the number of rounds of the synchronous method.
constexpr unsigned int kRelaxMinRows = 32768;
constexpr float kRelaxMinTol = 2e-7f, kRelaxNowTol = 4e-6f, kRelaxMaxTol = 1e-5f;
constexpr double kRelaxStuck = 0.99;
constexpr double kRelaxGap = 0.85, kRelaxMinGap = 2e-3, kRelaxEnter = 0.90, kRelaxLeave = 0.25;

bool relaxed_rounds_pay(const dynlp_ctx* c, const Frontier& universe, float tol) {
    return c->update_mode == DYNLP_UPDATE_IN_PLACE && c->persist <= 0 && universe.size() >= kRelaxMinRows && tol >= kRelaxMinTol &&
           tol <= kRelaxMaxTol;
}

// What rounds over all updatable rows did (accelerate, conjugate).
struct DenseRounds {
    bool settled = true;        // conjugate rounds: ended because the residual was small enough
    int rounds = 0;             // executed, the ordinary round at the end included
    float last = 0.f;           // max change of the last round
    unsigned int changed = 0;   // rows it moved
    unsigned int last_map = 0;  // the bitmap that holds them
    double avg_len = 0.0;
};

// Rounds it, it + 1, ... (at most `budget`, which is not 0): relaxed rounds over `universe`, then one ordinary round over
// all of it.  That one is always run: only its moves tell how far the rows are from their neighbours' means (a relaxed row
// may stand still on its way past the fixed point).
DenseRounds accelerate(dynlp_ctx* c, const Frontier& universe, int G, float tol, int it, int budget, bool binned, bool packed) {
    DenseRounds out;
    sync_partner(c);
    for (unsigned int* mv : c->moved) HIPCHK(c, hipMemsetAsync(mv, 0, (size_t)c->moved_words * sizeof(unsigned int), c->stream));
    // share of the updatable rows' edge weight that leads to labelled vertices, from a sample of rows
    float sums[2] = {0.f, 0.f};
    {
        float* d_sums = reinterpret_cast<float*>(&c->bc->scan_total);
        HIPCHK(c, hipMemsetAsync(d_sums, 0, sizeof sums, c->stream));
        const unsigned int step = std::max(1u, universe.size() / 8192u);
        hipLaunchKernelGGL(k_labelled_share, dim3(grid_for((int64_t)(universe.size() / step + 1) * 16)), dim3(kBlock), 0, c->stream,
                           universe.ns, universe.nl, step, universe.front, universe.back, c->meta, c->pool, c->seed_class, d_sums);
        HIPCHK(c, hipGetLastError());
        HIPCHK(c, hipMemcpyAsync(sums, d_sums, sizeof sums, hipMemcpyDeviceToHost, c->stream));
        HIPCHK(c, hipStreamSynchronize(c->stream));
    }
    const double gap = std::min(0.5, std::max(kRelaxMinGap, kRelaxGap * (sums[1] > 0.f ? (double)sums[0] / sums[1] : 0.0)));
    const double omega = 2.0 / (1.0 + std::sqrt(gap * (2.0 - gap)));
    const int limit = (int)std::ceil(4.0 * 16.0 / -std::log(std::sqrt(omega - 1.0)));  // 16: log(1 / 1e-7)
    int q = 0;  // round of the stretch: bitmaps as in a fused stretch
    bool finish = budget == 1;
    struct Progress {
        float last;
        unsigned int changed;
    };
    std::vector<Progress> chains;  // after every chain
    for (;;) {
        const int r = finish ? 1 : std::min(kChain, budget - 1 - q);
        const size_t first_pair = c->events_used / 2;
        float* const buf[2] = {c->F, c->F2};
        for (int i = 0; i < r; ++i) {
            const int t = it + q + i, b = q + i;
            PullRoundArgs a{slot_of(c, t - 1), buf[i & 1], buf[(i + 1) & 1], c->moved[(b + 2) % 3], c->moved[b % 3],
                            c->moved[(b + 1) % 3], tol, slot_of(c, t), slot_of(c, t + 1)};
            a.flags = kRoundAll | (finish || b == 0 ? kRoundForce : 0);
            a.omega = finish || b == 0 ? 1.f : (float)omega;
            c->ev_adjacent = i > 0;
            if (binned) launch_binned_round(c, a, t, false);
            else if (packed) launch_packed_round(c, a, t);
            else launch_update_pull(c, G, universe, a, t);
        }
        read_slots(c, it + q, r);
        int executed = 0;
        for (int i = 0; i < r; ++i) {
            const RoundCtr& rc = c->h_slot[i];
            if (!rc.executed) break;
            ++executed;
            out.changed = rc.changed;
            std::memcpy(&out.last, &rc.resid_bits, sizeof(float));
            const unsigned int nq = rc.rows_short + rc.rows_long;
            if (nq) out.avg_len = (double)(rc.edges + rc.edges_long) / (double)nq;
            c->log.push_back(round_info(rc, binned ? 3 : 2, packed ? 0 : G));
        }
        if (executed & 1) std::swap(c->F, c->F2);
        if (c->time_kernels) trim_timed_spans(c, first_pair, it + q + executed);
        q += executed;
        out.last_map = (unsigned int)((q + 2) % 3);
        if (finish) break;
        chains.push_back({out.last, out.changed});
        const size_t k = chains.size(), back = (double)out.changed < kRelaxStuck * universe.size() ? 4 : 16;
        const bool stuck = k > back && (double)out.last >= kRelaxStuck * chains[k - 1 - back].last &&
                           (double)out.changed >= kRelaxStuck * chains[k - 1 - back].changed;
        finish = stuck || executed < r || (double)out.changed < kRelaxLeave * (double)universe.size() || q >= limit || q >= budget - 1;
    }
    out.rounds = q;
    return out;
}

// ---- conjugate rounds (in-place mode, dynlp_conjugate.h) -------------------------------------------------------
// They take the place of the relaxed rounds where the call leaves them enough rounds and there is memory for two more arrays
// of the size of the label matrix.
// A call may be cut by its round cap before the iteration has settled: 15 to 30 rounds on planted, kNN and power-law graphs,
// but 54 to 80 on random graphs of degree 3 to 5, and 120 to 500 and more on 2D grids with 1% to 0.1% of the vertices labelled.
// Of all combinations of the residuals so far a conjugate iterate is the nearest to the fixed point in the energy norm of the
// system, and a relaxed one is such a combination too; single rows may be further off.  64-bit models of both, 40,000
// vertices, 3 classes, from uniform rows; distance from the fixed point, 2-norm (largest), relaxed / conjugate:
//   rounds                            32                                64                                100
//   2D grid, 1% labelled     .14 (.45) / .11 (.42)        6.7e-2 (.24) / 1.9e-2 (5.6e-2)  3.3e-2 (.12) / 2.0e-3 (7.9e-3)
//   2D grid, 0.1%            .37 (.55) / .37 (.55)        .30 (.53) / .23 (.52)           .24 (.44) / .14 (.22)
//   random, degree 3, 0.1%   7.4e-2 (4.7e-2) / 1.8e-2 (.15)  5.6e-2 (2.7e-2) / 1.1e-5 (2.6e-4)  settled in 80
//   random, degree 5, 1%, weights over six decades        4.0e-2 (.47) / 2.5e-2 (.41)     3.0e-2 (.43) / 9.8e-3 (.29)
// After batches on converged labels (5 or 400 vertices labelled, 400 or 4,000 replaced; grids, random graphs, a path, planted
// blocks) single rows were further off after 32 rounds in 7 of 28 cases, after 64 and more in none that had not settled, and
// the 2-norm in one (a grid with 0.1%: 1.64e-2 against 1.53e-2 at 64, 1.36e-2 against 1.33e-2 at 80).  Smaller budgets keep the
// relaxed rounds.
constexpr int kCgMinBudget = 64;
// The iteration ends when no row would move by more than kCgStop * tol (in the recurrence's own residual), or when the largest
// move has not reached a new low (by 10%) in kCgPatience iterations, or when its coefficients are no numbers; relaxed rounds then
// go on.
constexpr float kCgStop = 0.5f;
constexpr int kCgPatience = 96;
// Solves and batches in a row that cannot run them (mode, threshold, round cap) after which their arrays are given back: not the
// first, since a program may alternate between two thresholds or modes, and to allocate and release is slow.
constexpr int kCgIdleCalls = 4;

void free_conjugate(dynlp_ctx* c) {
    dev_free(c, c->cg_z);
    dev_free(c, c->cg_p);
    c->cg_z = c->cg_p = nullptr;
    c->cg_cap = 0;
    c->cg_idle = 0;
}

// At the beginning of a solve or batch, when the stream is done with the call before.
void conjugate_idle(dynlp_ctx* c) {
    if (!c->cg_z) return;
    const bool usable = c->update_mode == DYNLP_UPDATE_IN_PLACE && c->tol >= kRelaxMinTol && c->tol <= kRelaxMaxTol &&
                        c->max_iter >= kCgMinBudget;
    c->cg_idle = usable ? 0 : c->cg_idle + 1;
    if (c->cg_idle >= kCgIdleCalls) free_conjugate(c);
}

bool conjugate_arrays(dynlp_ctx* c, const Frontier& universe, float** z, float** p) {
    if (!c->cg_ring) {
        c->cg_ring = static_cast<CgSlot*>(dev_try_alloc(c, sizeof(CgSlot) * kCgRing));
        if (!c->cg_ring) return false;
    }
    if (!c->h_cg) {
        size_t got = 0;
        c->h_cg = static_cast<CgSlot*>(pinned_try_alloc(c, sizeof(CgSlot) * kChain, &got));
        if (!c->h_cg) return false;
    }
    if (c->CP == 1) {  // one float per vertex: the two arrays of row lists that are idle meanwhile
        float* idle[2];
        int k = 0;
        for (int32_t* q : c->queue)
            if (q != universe.front && k < 2) idle[k++] = reinterpret_cast<float*>(q);
        *z = idle[0];
        *p = idle[1];
        return true;
    }
    if (c->n * c->CP > c->cg_cap) {
        free_conjugate(c);
        if (!try_alloc_n(c, c->cg_z, c->n_cap * c->CP) || !try_alloc_n(c, c->cg_p, c->n_cap * c->CP)) {
            free_conjugate(c);
            return false;
        }
        c->cg_cap = c->n_cap * c->CP;
    }
    *z = c->cg_z;
    *p = c->cg_p;
    return true;
}

template <int CP, int G>
void launch_row_product_inst(dynlp_ctx* c, const Frontier& universe, const CgRun& run, const float* p, float* v) {
    const int64_t cap = (int64_t)c->num_cu * 32;
    const unsigned int short_blocks =
        (unsigned int)std::max<int64_t>(1, std::min<int64_t>(ceil_div((int64_t)universe.ns, kBlock / G), cap));
    const unsigned int long_blocks = (unsigned int)std::min<int64_t>((int64_t)universe.nl, cap / 2);
    hipLaunchKernelGGL((k_row_product<CP, G>), dim3(short_blocks + long_blocks), dim3(kBlock), 0, c->stream, run, long_blocks,
                       universe.front, universe.back, universe.ns, universe.nl, c->meta, c->pool, p, v);
}

template <int CP>
void launch_row_product(dynlp_ctx* c, int G, const Frontier& universe, const CgRun& run, const float* p, float* v) {
    constexpr int LPN = CP >= 4 ? CP / 4 : 1;
#define DYNLP_CASE(GV)                                                   \
    case GV:                                                             \
        if constexpr (GV >= LPN) {                                       \
            launch_row_product_inst<CP, GV>(c, universe, run, p, v);     \
            return;                                                      \
        }                                                                \
        break;
    switch (G) {
        DYNLP_CASE(4)
        DYNLP_CASE(8)
        DYNLP_CASE(16)
        DYNLP_CASE(32)
        DYNLP_CASE(64)
        default: break;
    }
#undef DYNLP_CASE
    launch_row_product_inst<CP, 64>(c, universe, run, p, v);
}

// Calls fn with the padded number of columns.
template <typename Fn>
void with_columns(int CP, Fn fn) {
    switch (CP) {
        case 1: fn(std::integral_constant<int, 1>{}); break;
        case 2: fn(std::integral_constant<int, 2>{}); break;
        case 4: fn(std::integral_constant<int, 4>{}); break;
        case 8: fn(std::integral_constant<int, 8>{}); break;
        case 16: fn(std::integral_constant<int, 16>{}); break;
        case 32: fn(std::integral_constant<int, 32>{}); break;
        default: fn(std::integral_constant<int, 64>{}); break;
    }
}

void launch_product(dynlp_ctx* c, int G, const Frontier& universe, const CgRun& run, const float* p, float* v, bool binned, bool packed) {
    if (binned) {
        const int lg = pb_run_lanes(c->pb_bins);
        const dim3 grid(8 * (unsigned int)std::max<int64_t>(1, ceil_div(c->pb_chunks, 8)));
        const unsigned int* bin_off = c->pb_bin + (kPbMaxBins + 1);
#define DYNLP_SCATTER(NB, PACKED, SRC)                                                                                        \
    hipLaunchKernelGGL((k_pb_scatter_product<NB, PACKED>), grid, dim3(kPbScatterThreads), 0, c->stream, run, c->pb_first + c->n, \
                       (unsigned int)c->pb_chunks, c->pb_bins, lg, SRC, c->pb_row0, c->pb_lpos, c->pb_table, bin_off, p, c->pb_val)
        if (c->pb_bins <= 2048 && c->pb_packed_ok) DYNLP_SCATTER(2048, true, c->pb_sp);
        else if (c->pb_bins <= 2048) DYNLP_SCATTER(2048, false, c->pb_src);
        else if (c->pb_packed_ok) DYNLP_SCATTER(kPbMaxBins, true, c->pb_sp);
        else DYNLP_SCATTER(kPbMaxBins, false, c->pb_src);
#undef DYNLP_SCATTER
        allow_gather_lds(c, k_pb_product);
        hipLaunchKernelGGL(k_pb_product, dim3(c->pb_bins), dim3(kPbGatherThreads), pb_gather_lds(c->pb_bits), c->stream, run, c->n, c->pb_bits, bin_off,
                           c->pb_dst, c->pb_wn, reinterpret_cast<const float*>(c->pb_val), c->pb_len, c->deg, p, v);
    } else if (packed) {
        const PkProduct r{run, c->n, c->pk_rows, c->pk_tab + c->pk_parts + 4, c->Cs, packed_stride(c), c->pk_bits, c->pk_ent, c->pk_tab, c->pk_len, c->deg, p, v};
        packed_kernel(c, [&](auto shape) {
            using S = decltype(shape);
            hipLaunchKernelGGL((k_pk_product<S::cp, S::lanes>), dim3((unsigned int)c->pk_parts), dim3(kPkThreads), packed_lds(c),
                               c->stream, r);
        });
    } else {
        with_columns(c->CP, [&](auto cp) { launch_row_product<decltype(cp)::value>(c, G, universe, run, p, v); });
    }
    HIPCHK(c, hipGetLastError());
}

// One ordinary round over all updatable rows whatever moved before (F -> F2); the buffers are not swapped.
void launch_full_round(dynlp_ctx* c, const Frontier& universe, int G, float tol, int t, int q, bool binned, bool packed) {
    PullRoundArgs a{slot_of(c, t - 1), c->F, c->F2, c->moved[(q + 2) % 3], c->moved[q % 3], c->moved[(q + 1) % 3], tol,
                    slot_of(c, t), slot_of(c, t + 1)};
    a.flags = kRoundAll | kRoundForce;
    if (binned) launch_binned_round(c, a, t, false);
    else if (packed) launch_packed_round(c, a, t);
    else launch_update_pull(c, G, universe, a, t);
}

// Rounds it, it + 1, ... (at most `budget` >= kCgMinBudget): an ordinary round over all rows, whose moves are the first
// residual, conjugate rounds, and an ordinary round that decides what is in V_aff.
DenseRounds conjugate(dynlp_ctx* c, const Frontier& universe, int G, float tol, int it, int budget, bool binned, bool packed,
                      float* z, float* p) {
    DenseRounds out;
    sync_partner(c);
    for (unsigned int* mv : c->moved) HIPCHK(c, hipMemsetAsync(mv, 0, (size_t)c->moved_words * sizeof(unsigned int), c->stream));
    HIPCHK(c, hipMemsetAsync(c->cg_ring, 0, sizeof(CgSlot) * kCgRing, c->stream));
    const unsigned int blocks =
        (unsigned int)std::max<int64_t>(1, std::min<int64_t>(ceil_div(c->n * std::max(1, c->CP / 4), 2 * kBlock), (int64_t)c->num_cu * 8));
    launch_full_round(c, universe, G, tol, it, 0, binned, packed);
    with_columns(c->CP, [&](auto cp) {
        hipLaunchKernelGGL(k_cg_begin<decltype(cp)::value>, dim3(blocks), dim3(kBlock), 0, c->stream, c->n, c->deg, c->F, c->F2, z, p,
                           tol, c->cg_ring);
    });
    HIPCHK(c, hipGetLastError());
    const float stop = kCgStop * tol;
    auto log_round = [&](const RoundCtr& rc) {
        out.changed = rc.changed;
        std::memcpy(&out.last, &rc.resid_bits, sizeof(float));
        const unsigned int nq = rc.rows_short + rc.rows_long;
        if (nq) out.avg_len = (double)(rc.edges + rc.edges_long) / (double)nq;
        c->log.push_back(round_info(rc, binned ? 3 : 2, packed ? 0 : G));
    };
    dynlp_round_info full{};
    int k = 0;  // iterations executed
    int best_at = 0;
    float best = std::numeric_limits<float>::infinity();
    for (bool more = true; more;) {
        const int r = std::min(kChain, budget - 2 - k);
        if (r <= 0) {
            out.settled = false;
            break;
        }
        if (k > 0)
            for (int i = 1; i <= r;) {
                const int at = (k + i) % kCgRing, run = std::min(r + 1 - i, kCgRing - at);
                HIPCHK(c, hipMemsetAsync(c->cg_ring + at, 0, sizeof(CgSlot) * (size_t)run, c->stream));
                i += run;
            }
        const size_t first_pair = c->events_used / 2;
        for (int i = 1; i <= r; ++i) {
            const CgRun run{c->cg_ring + (k + i - 1) % kCgRing, c->cg_ring + (k + i) % kCgRing, stop, tol};
            c->ev_adjacent = i > 1;
            hipEvent_t e1 = open_timed_span(c, it + k + i, 1);
            launch_product(c, G, universe, run, p, c->F2, binned, packed);
            with_columns(c->CP, [&](auto cp) {
                hipLaunchKernelGGL(k_cg_step<decltype(cp)::value>, dim3(blocks), dim3(kBlock), 0, c->stream, run, c->n, c->deg, c->F, z,
                                   p, c->F2);
            });
            HIPCHK(c, hipGetLastError());
            close_timed_span(c, e1);
        }
        const int at = (k + 1) % kCgRing, run = std::min(r, kCgRing - at);
        read_to_host(c, c->h_cg, c->cg_ring + at, sizeof(CgSlot) * (size_t)run, c->cg_ring, sizeof(CgSlot) * (size_t)(r - run));
        if (k == 0) {
            read_slots(c, it, 1);
            log_round(c->h_slot[0]);
            full = c->log.back();
            if (!(out.last > stop)) more = false;
        }
        int executed = 0;
        for (int i = 0; i < r && more; ++i) {
            if (c->h_cg[i].broken) {  // not a round
                out.settled = more = false;
                break;
            }
            unsigned int zmax = 0, moved = 0;
            for (const CgPart& part : c->h_cg[i].part) {
                zmax = std::max(zmax, part.zmax);
                moved += part.moved;
            }
            ++executed;
            dynlp_round_info ri = full;
            std::memcpy(&ri.max_delta, &zmax, sizeof(float));
            ri.rows_moved = moved;
            ri.launch_rounds = -1.f;
            c->log.push_back(ri);
            if (ri.max_delta < 0.9f * best) {
                best = ri.max_delta;
                best_at = k + executed;
            }
            if (!(ri.max_delta > stop)) more = false;
        }
        k += executed;
        if (c->time_kernels) trim_timed_spans(c, first_pair, it + k + 1);
        if (more && k - best_at >= kCgPatience) {
            out.settled = false;
            more = false;
        }
    }
    with_columns(c->CP, [&](auto cp) {
        hipLaunchKernelGGL(k_cg_end<decltype(cp)::value>, dim3(blocks), dim3(kBlock), 0, c->stream, c->cg_ring + k % kCgRing, c->n, c->Cs,
                           c->deg, c->seed_class, z, p, c->F, c->F2);
    });
    HIPCHK(c, hipGetLastError());
    const int t = it + k + 1;
    for (int s : {t - 1, t}) HIPCHK(c, hipMemsetAsync(slot_of(c, s), 0, sizeof(RoundCtr), c->stream));
    launch_full_round(c, universe, G, tol, t, 1, binned, packed);
    read_slots(c, t, 1);
    log_round(c->h_slot[0]);
    std::swap(c->F, c->F2);
    out.last_map = 1;
    out.rounds = k + 2;
    return out;
}

// The rounds over all rows of a call in in-place mode: conjugate ones where they can run, else (or where they do not settle)
// relaxed ones.
DenseRounds dense_rounds(dynlp_ctx* c, const Frontier& universe, int G, float tol, int it, int budget, bool binned, bool packed) {
    float *z = nullptr, *p = nullptr;
    if (budget < kCgMinBudget || !conjugate_arrays(c, universe, &z, &p)) return accelerate(c, universe, G, tol, it, budget, binned, packed);
    DenseRounds out = conjugate(c, universe, G, tol, it, budget, binned, packed, z, p);
    if (out.settled || out.last <= tol || out.rounds >= budget) return out;
    const int before = out.rounds;
    out = accelerate(c, universe, G, tol, it + before, budget - before, binned, packed);
    out.rounds += before;
    return out;
}

void fill_stats_zero(dynlp_stats* s) {
    if (s) std::memset(s, 0, sizeof *s);
}

// ---- host-side argument checks (host-pointer mode): errors without touching the device ----------
bool host_check_seeds(std::string& err, int64_t s, int64_t n_total, int C, const int32_t* sv, const int32_t* sc) {
    std::unordered_map<int32_t, int32_t> seen;
    for (int64_t i = 0; i < s; ++i) {
        if (sv[i] < 0 || sv[i] >= n_total) { err = format_validation(kErrSeedVertex, i); return false; }
        if (sc[i] < 0 || sc[i] >= C) { err = format_validation(kErrSeedClass, i); return false; }
        auto it = seen.find(sv[i]);
        if (it != seen.end() && it->second != sc[i]) { err = format_validation(kErrSeedConflict, i); return false; }
        seen[sv[i]] = sc[i];
    }
    return true;
}

bool host_check_csr(std::string& err, int64_t n, const int64_t* row_ptr, const int32_t* col, const float* w) {
    if (row_ptr[0] != 0) { err = format_validation(kErrRowPtr, 0); return false; }
    for (int64_t u = 0; u < n; ++u)
        if (row_ptr[u + 1] < row_ptr[u]) { err = format_validation(kErrRowPtr, u); return false; }
    for (int64_t u = 0; u < n; ++u) {
        for (int64_t j = row_ptr[u]; j < row_ptr[u + 1]; ++j) {
            if (col[j] < 0 || col[j] >= n) { err = format_validation(kErrColRange, j); return false; }
            if (col[j] == u) { err = format_validation(kErrSelfLoop, j); return false; }
            if (!(w[j] > 0.f) || !std::isfinite(w[j])) { err = format_validation(kErrWeight, j); return false; }
        }
    }
    return true;
}

bool host_check_edges(std::string& err, int64_t m, int64_t n_total, const int32_t* eu, const int32_t* ev,
                      const float* ew) {
    for (int64_t i = 0; i < m; ++i) {
        if (eu[i] < 0 || eu[i] >= n_total || ev[i] < 0 || ev[i] >= n_total) {
            err = format_validation(kErrEndpoint, i);
            return false;
        }
        if (eu[i] == ev[i]) { err = format_validation(kErrSelfLoop, i); return false; }
        if (!(ew[i] > 0.f) || !std::isfinite(ew[i])) { err = format_validation(kErrWeight, i); return false; }
    }
    return true;
}

void destroy_ctx(dynlp_ctx* c) {
    if (!c) return;
    (void)hipSetDevice(c->device);
    if (c->stream || c->meta) c->idle = hipStreamSynchronize(c->stream) == hipSuccess;
    if (c->copy_stream) c->idle = hipStreamSynchronize(c->copy_stream) == hipSuccess && c->idle;
    void* ptrs[] = {c->meta, c->pool, c->F, c->F2, c->seed_class, c->flag, c->queue[0], c->queue[1], c->queue[2], c->moved[0], c->moved[1], c->moved[2], c->add_cnt,
                    c->deg, c->touched, c->reloc_off, c->he_rank, c->b_eu, c->b_ev, c->b_ew, c->b_sv, c->b_sc, c->b_del, c->d_io,
                    c->cc_par, c->cc_dense, c->cc_comp, c->cc_block, c->cc_kept, c->cc_W,
                    c->pb_src, c->pb_sp, c->pb_row0, c->pb_lpos, c->pb_tmp, c->pb_dst, c->pb_wn, c->pb_val, c->pb_len, c->pb_upd,
                    c->pb_first, c->pb_block, c->pb_bin, c->pb_table, c->pk_ent, c->pk_len, c->pk_deg, c->pk_tab,
                    c->cg_z, c->cg_p, c->cg_ring};
    for (void* p : ptrs) dev_free(c, p);
    std::vector<void*> left;  // arrays an interrupted call never got to free
    for (const auto& l : c->live) left.push_back(l.first);
    for (void* p : left) dev_free(c, p);
    dev_free(c, c->cc_ctr);
    if (c->h_cc) (void)hipHostFree(c->h_cc);
    for (hipEvent_t e : c->init_ev)
        if (e) (void)hipEventDestroy(e);
    dev_free(c, c->ring);
    dev_free(c, c->xcd);
    dev_free(c, c->persist_ctl);
    for (void* b : c->bounce)
        if (b) (void)hipHostFree(b);
    for (hipEvent_t e : c->ingest_ev)
        if (e) (void)hipEventDestroy(e);
    if (c->copy_stream) (void)hipStreamDestroy(c->copy_stream);
    if (c->idle) {
        pinned_free(c, c->h_fixed, c->h_fixed_bytes);
        pinned_free(c, c->h_io, (size_t)c->h_io_cap);
    } else {
        if (c->h_fixed) (void)hipHostFree(c->h_fixed);
        if (c->h_io) (void)hipHostFree(c->h_io);
    }
    if (c->h_cg) (void)hipHostFree(c->h_cg);
    for (hipEvent_t e : c->events) (void)hipEventDestroy(e);
    delete c;
    (void)g_kept.release_older(kKeepMs);
}

// ---- Alg. 2 Step 1 (components of the sparsified batch-internal graph) + Step 2 (supernode rows) ----
void ensure_init_scratch(dynlp_ctx* c, int64_t k, int64_t m) {
    if (!c->cc_ctr) {
        c->cc_ctr = static_cast<InitCtr*>(dev_alloc(c, sizeof(InitCtr)));
        size_t got = 0;
        c->h_cc = static_cast<InitCtr*>(pinned_alloc(c, sizeof(InitCtr), &got));
        for (hipEvent_t& e : c->init_ev) HIPCHK(c, hipEventCreate(&e));
    }
    if (k > c->cc_vcap) {
        dev_free(c, c->cc_par);
        dev_free(c, c->cc_dense);
        dev_free(c, c->cc_comp);
        dev_free(c, c->cc_block);
        c->cc_par = c->cc_dense = c->cc_comp = nullptr;
        c->cc_block = nullptr;
        c->cc_vcap = 0;
        const int64_t cap = k + k / 2;
        c->cc_par = dev_alloc_n<int32_t>(c, cap);
        c->cc_dense = dev_alloc_n<int32_t>(c, cap);
        c->cc_comp = dev_alloc_n<int32_t>(c, cap);
        c->cc_block = dev_alloc_n<unsigned int>(c, ceil_div(cap, kBlock) + 1);
        c->cc_vcap = cap;
    }
    if (m > c->cc_ecap) {
        dev_free(c, c->cc_kept);
        c->cc_kept = nullptr;
        c->cc_ecap = 0;
        const int64_t cap = m + m / 2;
        c->cc_kept = dev_alloc_n<int2>(c, cap);
        c->cc_ecap = cap;
    }
}

void read_init_ctr(dynlp_ctx* c) {
    HIPCHK(c, hipMemcpyAsync(c->h_cc, c->cc_ctr, sizeof(InitCtr), hipMemcpyDeviceToHost, c->stream));
    HIPCHK(c, hipStreamSynchronize(c->stream));
}

// Runs after the batch's edges are in the CSR and its seeds are clamped; rewrites only the rows of
// the k inserted, unlabelled vertices n0 .. n0+k-1.
void run_supernode_init(dynlp_ctx* c, int64_t n0, int64_t k, int64_t m, const int32_t* d_eu, const int32_t* d_ev,
                        const float* d_ew) {
    ensure_init_scratch(c, k, m);
    HIPCHK(c, hipEventRecord(c->init_ev[0], c->stream));
    HIPCHK(c, hipMemsetAsync(c->cc_ctr, 0, sizeof(InitCtr), c->stream));
    hipLaunchKernelGGL(k_cc_reset, dim3(grid_for(k)), dim3(kBlock), 0, c->stream, k, c->cc_par);
    if (m > 0)
        hipLaunchKernelGGL(k_cc_filter, dim3(grid_for(ceil_div(m, kAppendItems))), dim3(kBlock), 0, c->stream, m, n0, k, d_eu, d_ev, d_ew, c->tau,
                           c->cc_kept, c->cc_ctr);
    const unsigned int hook_grid = (unsigned int)std::min<int64_t>(grid_for(std::max<int64_t>(m, 1)), (int64_t)c->num_cu * 8);
    int hook_steps = 0;
    for (;;) {
        for (int i = 0; i < kInitChain; ++i) {
            hipLaunchKernelGGL(k_cc_hook, dim3(hook_grid), dim3(kBlock), 0, c->stream, i, c->cc_kept, c->cc_par, c->cc_ctr);
            hipLaunchKernelGGL(k_cc_jump, dim3(grid_for(k)), dim3(kBlock), 0, c->stream, i, k, c->cc_par, c->cc_ctr);
        }
        HIPCHK(c, hipGetLastError());
        read_init_ctr(c);
        for (int i = 0; i < kInitChain; ++i)
            if (i == 0 || c->h_cc->changed[i - 1]) ++hook_steps;
        if (c->h_cc->changed[kInitChain - 1] == 0u) break;  // a hook step found every kept edge inside one tree
        HIPCHK(c, hipMemsetAsync(c->cc_ctr->changed, 0, sizeof(unsigned int) * kInitChain, c->stream));
    }
    const int64_t nb = ceil_div(k, kBlock);
    hipLaunchKernelGGL(k_cc_count_roots, dim3((unsigned int)nb), dim3(kBlock), 0, c->stream, k, c->cc_par, c->cc_block);
    hipLaunchKernelGGL(k_cc_scan_blocks, dim3(1), dim3(kBlock), 0, c->stream, nb, c->cc_block, c->cc_ctr);
    hipLaunchKernelGGL(k_cc_number_roots, dim3((unsigned int)nb), dim3(kBlock), 0, c->stream, k, c->cc_par, c->cc_block,
                       c->cc_dense);
    hipLaunchKernelGGL(k_cc_label, dim3(grid_for(k)), dim3(kBlock), 0, c->stream, k, c->cc_par, c->cc_dense, c->cc_comp);
    HIPCHK(c, hipGetLastError());
    read_init_ctr(c);
    const int64_t comps = c->h_cc->components;
    if (comps * c->C > c->cc_wcap) {
        dev_free(c, c->cc_W);
        c->cc_W = nullptr;
        c->cc_wcap = 0;
        const int64_t cap = comps * c->C + comps * c->C / 2;
        c->cc_W = dev_alloc_n<double>(c, cap);
        c->cc_wcap = cap;
    }
    hipLaunchKernelGGL(k_fill_f64, dim3(grid_for(comps * c->C)), dim3(kBlock), 0, c->stream, comps * c->C, c->cc_W, 0.0);
    hipLaunchKernelGGL(k_supernode_weights, dim3((unsigned int)ceil_div(k, kSwRows)), dim3(kBlock), 0, c->stream, n0, k, c->C, c->meta,
                       c->pool, c->seed_class, c->cc_comp, c->cc_W);
    hipLaunchKernelGGL(k_supernode_rows, dim3(grid_for(k * c->CP)), dim3(kBlock), 0, c->stream, n0, k, c->C, c->Cs, c->coff, c->CP,
                       c->seed_class, c->cc_comp, c->cc_W, c->F);
    HIPCHK(c, hipGetLastError());
    HIPCHK(c, hipEventRecord(c->init_ev[1], c->stream));
    c->last_init.vertices = k;
    c->last_init.kept_edges = c->h_cc->kept;
    c->last_init.components = comps;
    c->last_init.hook_steps = hook_steps;
    c->last_init.ms = 0.f;  // filled in after the call's final synchronisation
}

// Prefix offsets of per-row values already stored (caps in meta / lens in an array) need the
// scanned block sums; this runs the middle step and returns the grand total.
int64_t scan_block_sums(dynlp_ctx* c, int64_t nb, int64_t* sums) {
    hipLaunchKernelGGL(k_scan_block_sums, dim3(1), dim3(kBlock), 0, c->stream, nb, sums, &c->bc->scan_total);
    HIPCHK(c, hipGetLastError());
    read_bc(c);
    return (int64_t)c->h_bc->scan_total;
}

// Labels in the caller's format: soft (n x C, no padding) and / or hard (argmax, lowest index on ties) into
// device buffers.  Every row is overwritten, so the buffers need no clearing.
void launch_label_output(dynlp_ctx* c, float* d_soft, int32_t* d_hard) {
    const int64_t n = c->n;
    if (!d_soft && !d_hard) return;
    if (c->coff)
        hipLaunchKernelGGL(k_scalar_labels, dim3(grid_for(n)), dim3(kBlock), 0, c->stream, n, c->F, d_soft, d_hard);
    else
        hipLaunchKernelGGL(k_labels, dim3(grid_for(n * (c->CP >= 4 ? c->CP / 4 : 1))), dim3(kBlock), 0, c->stream, n, c->C, c->CP, c->F,
                           d_soft, d_hard);
    HIPCHK(c, hipGetLastError());
}

}  // namespace

// =================================================================================================
// C ABI
// =================================================================================================
extern "C" {

void dynlp_default_options(dynlp_options* opt) {
    if (!opt) return;
    std::memset(opt, 0, sizeof *opt);
    opt->slack_factor = 1.25f;
}

const char* dynlp_last_error(const dynlp_ctx* ctx) { return ctx ? ctx->err.c_str() : g_create_error.c_str(); }

int64_t dynlp_num_vertices(const dynlp_ctx* ctx) { return ctx ? ctx->n : -1; }
int64_t dynlp_num_entries(const dynlp_ctx* ctx) { return ctx ? ctx->entries : -1; }
int32_t dynlp_num_classes(const dynlp_ctx* ctx) { return ctx ? ctx->C : -1; }

void dynlp_destroy(dynlp_ctx* ctx) { destroy_ctx(ctx); }

dynlp_status dynlp_create(dynlp_ctx** out, int64_t n, const int64_t* row_ptr, const int32_t* col, const float* w,
                          int32_t num_classes, int64_t num_seeds, const int32_t* seed_vertex,
                          const int32_t* seed_class, const dynlp_options* opt) {
    if (out) *out = nullptr;
    g_create_error.clear();
    auto bad = [&](const std::string& msg) {
        g_create_error = msg;
        return DYNLP_ERR_INVALID_ARG;
    };
    if (!out) return bad("out is NULL");
    if (n < 0 || n > 0x7ffffffeLL) return bad("n must be in [0, 2^31-2]");
    if (num_classes < 1 || num_classes > DYNLP_MAX_CLASSES) return bad("num_classes must be in [1, DYNLP_MAX_CLASSES]");
    if (!row_ptr) return bad("row_ptr is NULL");
    if (num_seeds < 0) return bad("num_seeds is negative");
    if (num_seeds > 0 && (!seed_vertex || !seed_class)) return bad("seed arrays are NULL");
    dynlp_options o;
    dynlp_default_options(&o);
    if (opt) o = *opt;
    if (!(o.slack_factor > 1.0f)) o.slack_factor = 1.25f;
    if (o.slack_factor > 8.0f) return bad("slack_factor must be <= 8");
    if (o.reserve_vertices < 0 || o.reserve_edges < 0) return bad("reserve counts must be >= 0");
    if (o.persistent_rounds < -1 || o.persistent_rounds > 1) return bad("persistent_rounds must be -1, 0 or 1");
    if (o.persistent_spin_limit < 0) return bad("persistent_spin_limit must be >= 0");
    if (o.ingest_chunk_edges < 0 || o.ingest_chunk_edges > ((int64_t)1 << 28)) return bad("ingest_chunk_edges must be in [0, 2^28]");
    if ((o.alloc == nullptr) != (o.dealloc == nullptr)) return bad("alloc and dealloc must be given together");
    if (o.binary_scalar != 0 && num_classes != 2) return bad("binary_scalar needs num_classes == 2");
    const int Cs = o.binary_scalar != 0 ? 1 : num_classes;  // stored columns
    const int CP = padded_classes(Cs);
    if (o.binned_rounds != 0 && o.binned_rounds != -1 && (o.binned_rounds < kPbMinBinBits || o.binned_rounds > kPbMaxBinBits))
        return bad("binned_rounds must be 0 (automatic), -1 (never) or a number of bin bits from 8 to 15");
    if (o.group_lanes != 0) {
        const int g = o.group_lanes;
        if (!(g == 4 || g == 8 || g == 16 || g == 32 || g == 64) || g < lanes_per_neighbour(CP))
            return bad("group_lanes must be 0 or one of 4, 8, 16, 32, 64 and at least padded_classes/4");
    }
    // Host-pointer mode: everything that can be checked without a GPU is checked first.
    int64_t nnz = -1;
    if (!o.ptrs_on_device) {
        nnz = row_ptr[n];
        if (nnz < 0) return bad(format_validation(kErrRowPtr, n));
        if (nnz > 0 && (!col || !w)) return bad("col / w are NULL");
        std::string e;
        if (!host_check_csr(e, n, row_ptr, col, w)) return bad(e);
        if (!host_check_seeds(e, num_seeds, n, num_classes, seed_vertex, seed_class)) return bad(e);
    }

    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || ndev <= 0 || o.device < 0 || o.device >= ndev) {
        (void)hipGetLastError();
        g_create_error = "no usable GPU (hipGetDeviceCount found " + std::to_string(ndev) + " devices, device " +
                         std::to_string(o.device) + " requested); libdynlp has no CPU path";
        return DYNLP_ERR_DEVICE;
    }
    dynlp_ctx* c = new (std::nothrow) dynlp_ctx;
    if (!c) {
        g_create_error = "host allocation failed";
        return DYNLP_ERR_OOM;
    }
    const AtWork at_work(o.device);
    dynlp_status result = DYNLP_OK;
    int64_t* block_sums = nullptr;
    try {
        c->device = o.device;
        c->stream = static_cast<hipStream_t>(o.stream);
        c->dev_ptrs = o.ptrs_on_device != 0;
        c->slack = o.slack_factor;
        c->time_kernels = o.time_kernels != 0;
        c->group_lanes = o.group_lanes;
        c->binned = o.binned_rounds;
        c->persist = o.persistent_rounds;
        if (o.persistent_spin_limit > 0) c->persist_spin = (unsigned int)o.persistent_spin_limit;
        c->ingest_chunk = o.ingest_chunk_edges > 0 ? o.ingest_chunk_edges : ((int64_t)4 << 20);
        c->alloc_fn = o.alloc;
        c->dealloc_fn = o.dealloc;
        c->alloc_user = o.alloc_user;
        c->C = num_classes;
        c->Cs = Cs;
        c->coff = num_classes - Cs;  // 1 in the binary scalar layout (column 0 holds class 1), else 0
        c->CP = CP;
        HIPCHK(c, hipSetDevice(c->device));
        resolve_static_scratch(c->device);  // for dynlp_get_labels_static; a failure is reported by that call
        (void)g_kept.release_older(kKeepMs);
        int cus = 0;  // (one attribute: all properties take 0.2 ms)
        HIPCHK(c, hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, c->device));
        c->num_cu = cus > 0 ? cus : 256;
        c->persist_ctl = static_cast<unsigned int*>(dev_alloc(c, kBarWords * sizeof(unsigned int)));
        c->ring = static_cast<RoundCtr*>(dev_alloc(c, sizeof(RoundCtr) * (kRing + 1) + sizeof(BatchCtr)));
        c->bc = reinterpret_cast<BatchCtr*>(c->ring + kRing + 1);
        c->xcd = static_cast<XcdCtl*>(dev_alloc(c, sizeof(XcdCtl)));
        HIPCHK(c, hipMemsetAsync(c->xcd, 0, sizeof(XcdCtl), c->stream));
        constexpr size_t kSlotBytes = sizeof(RoundCtr) * kRing, kStartBytes = (sizeof(dynlp_ctx::HostStart) + 63) / 64 * 64;
        constexpr size_t kResultBytes = (sizeof(XcdResult) + 63) / 64 * 64;
        c->h_fixed = pinned_alloc(c, kSlotBytes + kStartBytes + kResultBytes + 64, &c->h_fixed_bytes);
        unsigned char* const fixed = static_cast<unsigned char*>(c->h_fixed);
        c->h_slot = reinterpret_cast<RoundCtr*>(fixed);
        c->h_start = reinterpret_cast<dynlp_ctx::HostStart*>(fixed + kSlotBytes);
        c->h_bc = &c->h_start->bc;
        c->h_xcd = reinterpret_cast<XcdResult*>(fixed + kSlotBytes + kStartBytes);
        c->h_flag = reinterpret_cast<unsigned int*>(fixed + kSlotBytes + kStartBytes + kResultBytes);
        *c->h_flag = 0u;
        HIPCHK(c, hipDeviceGetAttribute(&c->clock_khz, hipDeviceAttributeWallClockRate, c->device));
        std::memset(c->h_bc, 0, sizeof(BatchCtr));
        write_bc(c);
        zero_ring(c);

        if (c->dev_ptrs) {
            HIPCHK(c, hipMemcpyAsync(&nnz, row_ptr + n, sizeof(int64_t), hipMemcpyDeviceToHost, c->stream));
            HIPCHK(c, hipStreamSynchronize(c->stream));
            if (nnz < 0) {
                c->err = format_validation(kErrRowPtr, n);
                throw Fail{DYNLP_ERR_INVALID_ARG};
            }
            if (nnz > 0 && (!col || !w)) {
                c->err = "col / w are NULL";
                throw Fail{DYNLP_ERR_INVALID_ARG};
            }
        }
        const int64_t reserve_v = o.reserve_vertices > 0 ? o.reserve_vertices : std::max<int64_t>(1024, n / 8);
        c->n = 0;  // nothing to preserve while the arrays are first allocated
        alloc_vertex_arrays(c, n + reserve_v);
        c->n = n;

        DevIn<int64_t> d_rp(c, row_ptr, n + 1);
        DevIn<int32_t> d_col(c, col, nnz);
        DevIn<float> d_w(c, w, nnz);
        DevIn<int32_t> d_sv(c, seed_vertex, num_seeds);
        DevIn<int32_t> d_sc(c, seed_class, num_seeds);

        // validate row_ptr and the seed list
        if (n > 0)
            hipLaunchKernelGGL(k_validate_row_ptr, dim3(grid_for(n)), dim3(kBlock), 0, c->stream, n, d_rp.ptr, nnz, c->bc);
        if (num_seeds > 0) {
            hipLaunchKernelGGL(k_validate_seeds, dim3(grid_for(num_seeds)), dim3(kBlock), 0, c->stream, num_seeds, n,
                               (int64_t)0, c->C, d_sv.ptr, d_sc.ptr, c->seed_class, c->add_cnt, c->bc);
            hipLaunchKernelGGL(k_clear_seed_tmp, dim3(grid_for(num_seeds)), dim3(kBlock), 0, c->stream, num_seeds, n,
                               d_sv.ptr, c->add_cnt);
        }
        HIPCHK(c, hipGetLastError());
        read_bc(c);
        if (c->h_bc->err) {
            c->err = format_validation(error_code(*c->h_bc), error_index(*c->h_bc));
            throw Fail{DYNLP_ERR_INVALID_ARG};
        }

        // slack layout: capacities, offsets (scan), entries
        const int64_t nb = grid_for(n);
        block_sums = dev_alloc_n<int64_t>(c, nb);
        int64_t tail = 0;
        if (n > 0) {
            hipLaunchKernelGGL(k_row_caps, dim3(nb), dim3(kBlock), 0, c->stream, n, d_rp.ptr, c->slack, c->meta, block_sums);
            HIPCHK(c, hipGetLastError());
            tail = scan_block_sums(c, nb, block_sums);
            hipLaunchKernelGGL(k_row_offsets, dim3(nb), dim3(kBlock), 0, c->stream, n, c->meta, block_sums);
            HIPCHK(c, hipGetLastError());
        }
        c->pool_tail = tail;
        const int64_t extra = tail / 4 + 4 * o.reserve_edges + (1 << 16);
        c->pool_cap = 0;
        grow_pool(c, tail + extra);
        c->h_bc->pool_tail = (unsigned long long)tail;
        c->h_bc->err = 0;
        write_bc(c);
        if (nnz > 0) {
            hipLaunchKernelGGL(k_scatter_entries, dim3(grid_for(nnz)), dim3(kBlock), 0, c->stream, nnz, n, d_rp.ptr,
                               d_col.ptr, d_w.ptr, c->meta, c->pool, c->bc);
            HIPCHK(c, hipGetLastError());
        }
        read_bc(c);
        if (c->h_bc->err) {
            c->err = format_validation(error_code(*c->h_bc), error_index(*c->h_bc));
            throw Fail{DYNLP_ERR_INVALID_ARG};
        }
        c->entries = nnz;

        // labels
        hipLaunchKernelGGL(k_fill_i32, dim3(grid_for(c->n_cap)), dim3(kBlock), 0, c->stream, (int64_t)0, c->n_cap,
                           c->seed_class, -1);
        if (num_seeds > 0)
            hipLaunchKernelGGL(k_set_seed_class, dim3(grid_for(num_seeds)), dim3(kBlock), 0, c->stream, num_seeds,
                               d_sv.ptr, d_sc.ptr, c->seed_class);
        if (n > 0) {
            hipLaunchKernelGGL(k_init_labels, dim3(grid_for(n * c->CP)), dim3(kBlock), 0, c->stream, (int64_t)0, n, c->C,
                               c->Cs, c->coff, c->CP, c->seed_class, c->F);
            hipLaunchKernelGGL(k_row_degree, dim3(grid_for(n * 16)), dim3(kBlock), 0, c->stream, n, c->meta, c->pool,
                               c->deg);
        }
        HIPCHK(c, hipGetLastError());
        HIPCHK(c, hipStreamSynchronize(c->stream));
    } catch (const Fail& f) {
        result = f.st;
    } catch (const std::bad_alloc&) {
        c->err = "host allocation failed";
        result = DYNLP_ERR_OOM;
    }
    if (block_sums) scratch_free(c, block_sums);
    if (result != DYNLP_OK) {
        g_create_error = c->err;
        destroy_ctx(c);
        return result;
    }
    *out = c;
    return DYNLP_OK;
}

dynlp_status dynlp_set_params(dynlp_ctx* ctx, float tol, int32_t max_iter) {
    if (!ctx) return DYNLP_ERR_INVALID_ARG;
    if (!(tol >= 0.f) || !std::isfinite(tol) || max_iter < 0) {
        ctx->err = "tol must be finite and >= 0, max_iter >= 0";
        return DYNLP_ERR_INVALID_ARG;
    }
    ctx->tol = tol;
    ctx->max_iter = max_iter;
    return DYNLP_OK;
}

dynlp_status dynlp_stream_bandwidth(dynlp_ctx* c, int64_t bytes, int32_t repetitions, double* copy_gb_per_s,
                                    double* read_gb_per_s) {
    if (!c) return DYNLP_ERR_INVALID_ARG;
    if (bytes < 16 || repetitions < 1) {
        c->err = "bytes < 16 or repetitions < 1";
        return DYNLP_ERR_INVALID_ARG;
    }
    hipEvent_t ev[3] = {nullptr, nullptr, nullptr};
    try {
        HIPCHK(c, hipSetDevice(c->device));
        const int64_t n16 = bytes / 16;
        const unsigned int blocks = (unsigned int)std::min<int64_t>(grid_for(n16), (int64_t)c->num_cu * 16);
        Temp<float4> src_t(c, n16);
        Temp<float4> dst_t(c, std::max<int64_t>(n16, ceil_div((int64_t)blocks * kBlock * (int64_t)sizeof(float), 16)));
        float4 *src = src_t.ptr, *dst = dst_t.ptr;
        HIPCHK(c, hipMemsetAsync(src, 0, (size_t)n16 * 16, c->stream));
        for (hipEvent_t& e : ev) HIPCHK(c, hipEventCreate(&e));
        hipLaunchKernelGGL(k_stream_copy, dim3(blocks), dim3(kBlock), 0, c->stream, n16, src, dst);  // warm-up
        HIPCHK(c, hipEventRecord(ev[0], c->stream));
        for (int r = 0; r < repetitions; ++r)
            hipLaunchKernelGGL(k_stream_copy, dim3(blocks), dim3(kBlock), 0, c->stream, n16, src, dst);
        HIPCHK(c, hipEventRecord(ev[1], c->stream));
        for (int r = 0; r < repetitions; ++r)
            hipLaunchKernelGGL(k_stream_read, dim3(blocks), dim3(kBlock), 0, c->stream, n16, src,
                               reinterpret_cast<float*>(dst));
        HIPCHK(c, hipEventRecord(ev[2], c->stream));
        HIPCHK(c, hipGetLastError());
        HIPCHK(c, hipEventSynchronize(ev[2]));
        float ms_copy = 0.f, ms_read = 0.f;
        HIPCHK(c, hipEventElapsedTime(&ms_copy, ev[0], ev[1]));
        HIPCHK(c, hipEventElapsedTime(&ms_read, ev[1], ev[2]));
        const double moved = (double)n16 * 16.0 * repetitions;
        if (copy_gb_per_s) *copy_gb_per_s = 2.0 * moved / ((double)ms_copy * 1e6);  // bytes read + bytes written
        if (read_gb_per_s) *read_gb_per_s = moved / ((double)ms_read * 1e6);
        for (hipEvent_t e : ev) (void)hipEventDestroy(e);
        return DYNLP_OK;
    } catch (const SoftOom&) {
        return DYNLP_ERR_OOM;
    } catch (const Fail& f) {
        for (hipEvent_t e : ev)
            if (e) (void)hipEventDestroy(e);
        return f.st;
    }
}

dynlp_status dynlp_gather_bandwidth(dynlp_ctx* c, int64_t table_rows, int32_t row_bytes, int64_t gathers,
                                    int32_t repetitions, double* gathers_per_s, double* gb_per_s) {
    if (!c) return DYNLP_ERR_INVALID_ARG;
    if (table_rows < 1 || table_rows > 0x7fffffffLL || gathers < 1 || repetitions < 1 ||
        !(row_bytes == 16 || row_bytes == 32 || row_bytes == 64 || row_bytes == 128 || row_bytes == 256)) {
        c->err = "table_rows in [1, 2^31), row_bytes one of 16, 32, 64, 128, 256, gathers >= 1, repetitions >= 1";
        return DYNLP_ERR_INVALID_ARG;
    }
    hipEvent_t ev[2] = {nullptr, nullptr};
    try {
        HIPCHK(c, hipSetDevice(c->device));
        const int lpn = row_bytes / 16;
        const unsigned int blocks = (unsigned int)std::min<int64_t>(grid_for(ceil_div(gathers, 8) * lpn), (int64_t)c->num_cu * 32);
        Temp<float4> table(c, table_rows * lpn);
        Temp<float> sink(c, (int64_t)blocks * kBlock);
        HIPCHK(c, hipMemsetAsync(table.ptr, 0, (size_t)table_rows * row_bytes, c->stream));
        for (hipEvent_t& e : ev) HIPCHK(c, hipEventCreate(&e));
        auto launch = [&]() {
            switch (lpn) {
                case 1: hipLaunchKernelGGL(k_gather_probe<1>, dim3(blocks), dim3(kBlock), 0, c->stream, table.ptr, (unsigned int)table_rows, (unsigned long long)gathers, sink.ptr); break;
                case 2: hipLaunchKernelGGL(k_gather_probe<2>, dim3(blocks), dim3(kBlock), 0, c->stream, table.ptr, (unsigned int)table_rows, (unsigned long long)gathers, sink.ptr); break;
                case 4: hipLaunchKernelGGL(k_gather_probe<4>, dim3(blocks), dim3(kBlock), 0, c->stream, table.ptr, (unsigned int)table_rows, (unsigned long long)gathers, sink.ptr); break;
                case 8: hipLaunchKernelGGL(k_gather_probe<8>, dim3(blocks), dim3(kBlock), 0, c->stream, table.ptr, (unsigned int)table_rows, (unsigned long long)gathers, sink.ptr); break;
                default: hipLaunchKernelGGL(k_gather_probe<16>, dim3(blocks), dim3(kBlock), 0, c->stream, table.ptr, (unsigned int)table_rows, (unsigned long long)gathers, sink.ptr); break;
            }
        };
        launch();  // warm-up
        HIPCHK(c, hipEventRecord(ev[0], c->stream));
        for (int r = 0; r < repetitions; ++r) launch();
        HIPCHK(c, hipEventRecord(ev[1], c->stream));
        HIPCHK(c, hipGetLastError());
        HIPCHK(c, hipEventSynchronize(ev[1]));
        float ms = 0.f;
        HIPCHK(c, hipEventElapsedTime(&ms, ev[0], ev[1]));
        const double per_s = (double)gathers * repetitions / ((double)ms * 1e-3);
        if (gathers_per_s) *gathers_per_s = per_s;
        if (gb_per_s) *gb_per_s = per_s * row_bytes / 1e9;
        for (hipEvent_t e : ev) (void)hipEventDestroy(e);
        return DYNLP_OK;
    } catch (const SoftOom&) {
        for (hipEvent_t e : ev)
            if (e) (void)hipEventDestroy(e);
        return DYNLP_ERR_OOM;
    } catch (const Fail& f) {
        for (hipEvent_t e : ev)
            if (e) (void)hipEventDestroy(e);
        return f.st;
    }
}

dynlp_status dynlp_storage_info(const dynlp_ctx* c, int64_t* pool_used, int64_t* pool_capacity) {
    if (!c) return DYNLP_ERR_INVALID_ARG;
    if (pool_used) *pool_used = c->pool_tail;
    if (pool_capacity) *pool_capacity = c->pool_cap;
    return DYNLP_OK;
}

dynlp_status dynlp_compact_storage(dynlp_ctx* c) {
    if (!c) return DYNLP_ERR_INVALID_ARG;
    if (c->poisoned) {
        c->err = "context is unusable after an earlier device or memory error";
        return DYNLP_ERR_STATE;
    }
    if (c->n == 0) return DYNLP_OK;
    try {
        HIPCHK(c, hipSetDevice(c->device));
        const int64_t n = c->n;
        const int64_t nb = grid_for(n);
        HIPCHK(c, hipStreamSynchronize(c->stream));
        free_conjugate(c);
        // the new layout is built beside the old one; the context switches over only when all of it exists, so
        // running out of memory here leaves graph and labels as they were
        Temp<RowMeta> meta_new(c, c->n_cap);
        Temp<int64_t> block_sums(c, nb);
        hipLaunchKernelGGL(k_recap_rows, dim3(nb), dim3(kBlock), 0, c->stream, n, c->meta, c->slack, meta_new.ptr, block_sums.ptr);
        HIPCHK(c, hipGetLastError());
        const int64_t tail = scan_block_sums(c, nb, block_sums.ptr);
        hipLaunchKernelGGL(k_row_offsets, dim3(nb), dim3(kBlock), 0, c->stream, n, meta_new.ptr, block_sums.ptr);
        const int64_t cap = round_up(tail + tail / 4 + (1 << 16), kRowAlign);
        Temp<Edge> pool_new(c, cap);
        hipLaunchKernelGGL(k_copy_rows, dim3(grid_for(n * 16)), dim3(kBlock), 0, c->stream, n, c->meta, meta_new.ptr, c->pool,
                           pool_new.ptr);
        HIPCHK(c, hipGetLastError());
        HIPCHK(c, hipStreamSynchronize(c->stream));
        dev_free(c, c->meta);
        dev_free(c, c->pool);
        c->meta = meta_new.release();
        c->pool = pool_new.release();
        c->pool_cap = cap;
        c->pool_tail = tail;
        (void)g_kept.release_older(0.f);
        return DYNLP_OK;
    } catch (const SoftOom&) {
        (void)hipStreamSynchronize(c->stream);
        return DYNLP_ERR_OOM;
    } catch (const Fail& f) {
        return f.st;
    } catch (const std::bad_alloc&) {
        c->err = "host allocation failed";
        return DYNLP_ERR_OOM;
    }
}

dynlp_status dynlp_set_update_mode(dynlp_ctx* ctx, int32_t mode) {
    if (!ctx) return DYNLP_ERR_INVALID_ARG;
    if (mode != DYNLP_UPDATE_SYNCHRONOUS && mode != DYNLP_UPDATE_IN_PLACE) {
        ctx->err = "mode must be DYNLP_UPDATE_SYNCHRONOUS or DYNLP_UPDATE_IN_PLACE";
        return DYNLP_ERR_INVALID_ARG;
    }
    ctx->update_mode = mode;
    return DYNLP_OK;
}

dynlp_status dynlp_set_final_check(dynlp_ctx* ctx, int32_t on) {
    if (!ctx) return DYNLP_ERR_INVALID_ARG;
    if (on != 0 && on != 1) {
        ctx->err = "on must be 0 or 1";
        return DYNLP_ERR_INVALID_ARG;
    }
    ctx->final_check = on != 0;
    return DYNLP_OK;
}

int64_t dynlp_release_kept_memory(void) { return (int64_t)g_kept.release_older(0.f); }

dynlp_status dynlp_set_shared_rounds(dynlp_ctx* c, int32_t workgroups, int64_t from_launch, int32_t last_launch) {
    if (!c) return DYNLP_ERR_INVALID_ARG;
    if (workgroups < -1 || workgroups > kXcdGroups || from_launch < 0 || last_launch < -1 || last_launch > (int32_t)kXcdLaunches) {
        c->err = "workgroups must be in [-1, 32], from_launch >= 0 and last_launch in [-1, 2^24 - 1]";
        return DYNLP_ERR_INVALID_ARG;
    }
    if (c->poisoned) {
        c->err = "context is unusable after an earlier device or memory error";
        return DYNLP_ERR_STATE;
    }
    try {
        if (last_launch >= 0) {  // (numbers that do not follow each other: from cleared words)
            HIPCHK(c, hipSetDevice(c->device));
            HIPCHK(c, hipMemsetAsync(c->xcd, 0, sizeof(XcdCtl), c->stream));
            HIPCHK(c, hipStreamSynchronize(c->stream));
            c->xcd_launches = (unsigned int)last_launch;
        }
    } catch (const Fail& f) {
        return f.st;
    }
    c->xcd_groups = workgroups;
    c->xcd_from = from_launch;
    c->xcd_asked = 0;
    return DYNLP_OK;
}

dynlp_status dynlp_set_initialiser(dynlp_ctx* ctx, int32_t mode, float tau) {
    if (!ctx) return DYNLP_ERR_INVALID_ARG;
    if (mode != DYNLP_INIT_UNIFORM && mode != DYNLP_INIT_SUPERNODE) {
        ctx->err = "mode must be DYNLP_INIT_UNIFORM or DYNLP_INIT_SUPERNODE";
        return DYNLP_ERR_INVALID_ARG;
    }
    if (mode == DYNLP_INIT_SUPERNODE && (!std::isfinite(tau) || tau < 0.f)) {
        ctx->err = "tau must be finite and >= 0";
        return DYNLP_ERR_INVALID_ARG;
    }
    ctx->init_mode = mode;
    ctx->tau = tau;
    return DYNLP_OK;
}

dynlp_status dynlp_mean_edge_weight(dynlp_ctx* c, double* mean) {
    if (!c) return DYNLP_ERR_INVALID_ARG;
    if (!mean) {
        c->err = "mean is NULL";
        return DYNLP_ERR_INVALID_ARG;
    }
    if (c->poisoned) {
        c->err = "context is unusable after an earlier device or memory error";
        return DYNLP_ERR_STATE;
    }
    *mean = 0.0;
    if (c->entries == 0) return DYNLP_OK;
    try {
        HIPCHK(c, hipSetDevice(c->device));
        const unsigned int blocks = (unsigned int)std::min<int64_t>(grid_for(c->n * 16), (int64_t)c->num_cu * 4);
        Temp<double> d_part(c, blocks);
        std::vector<double> part(blocks);
        hipLaunchKernelGGL(k_weight_partial, dim3(blocks), dim3(kBlock), 0, c->stream, c->n, c->meta, c->pool, d_part.ptr);
        HIPCHK(c, hipGetLastError());
        HIPCHK(c, hipMemcpyAsync(part.data(), d_part.ptr, sizeof(double) * blocks, hipMemcpyDeviceToHost, c->stream));
        HIPCHK(c, hipStreamSynchronize(c->stream));
        double tot = 0.0;
        for (double v : part) tot += v;
        *mean = tot / (double)c->entries;
        return DYNLP_OK;
    } catch (const SoftOom&) {
        return DYNLP_ERR_OOM;
    } catch (const Fail& f) {
        return f.st;
    } catch (const std::bad_alloc&) {
        c->err = "host allocation failed";
        return DYNLP_ERR_OOM;
    }
}

dynlp_status dynlp_last_components(dynlp_ctx* c, int64_t cap, int32_t* comp, dynlp_init_info* info) {
    if (!c) return DYNLP_ERR_INVALID_ARG;
    if (info) *info = c->last_init;
    if (!comp || c->last_init.vertices == 0) return DYNLP_OK;
    if (cap < c->last_init.vertices) {
        c->err = "comp holds fewer entries than the last batch inserted vertices";
        return DYNLP_ERR_INVALID_ARG;
    }
    if (c->poisoned) {
        c->err = "context is unusable after an earlier device or memory error";
        return DYNLP_ERR_STATE;
    }
    try {
        HIPCHK(c, hipSetDevice(c->device));
        HIPCHK(c, hipMemcpyAsync(comp, c->cc_comp, sizeof(int32_t) * (size_t)c->last_init.vertices,
                                 c->dev_ptrs ? hipMemcpyDeviceToDevice : hipMemcpyDeviceToHost, c->stream));
        HIPCHK(c, hipStreamSynchronize(c->stream));
        return DYNLP_OK;
    } catch (const Fail& f) {
        return f.st;
    }
}

dynlp_status dynlp_static_solve(dynlp_ctx* c, float tol, int32_t max_iter, dynlp_stats* stats) {
    if (!c) return DYNLP_ERR_INVALID_ARG;
    fill_stats_zero(stats);
    if (c->poisoned) {
        c->err = "context is unusable after an earlier device or memory error";
        return DYNLP_ERR_STATE;
    }
    dynlp_status st = dynlp_set_params(c, tol, max_iter);
    if (st != DYNLP_OK) return st;
    const auto t0 = Clock::now();
    const AtWork at_work(c->device);
    try {
        HIPCHK(c, hipSetDevice(c->device));
        (void)g_kept.release_older(kKeepMs);
        conjugate_idle(c);
        c->log.clear();
        reset_timed_spans(c);
        const bool in_place = c->update_mode == DYNLP_UPDATE_IN_PLACE;
        if (!in_place) sync_partner(c);
        zero_ring(c);
        const Frontier f = frontier_of(c, 0);
        RoundCtr* start = slot_of(c, -1);
        launch_compact(c, f, &start->next_count, &start->next_long, 1);
        read_slots_start(c);
        const unsigned int nq = c->h_slot[0].next_count + c->h_slot[0].next_long;
        c->h_slot_start_long = c->h_slot[0].next_long;
        int it = 0;
        float last = 0.f;
        bool converged = nq == 0;
        int64_t edges = 0;
        const int G = choose_group(c, c->n > 0 ? (double)c->entries / (double)std::max<int64_t>(1, nq) : 1.0);
        const auto t_it = Clock::now();
        // sweeps whose max change repeats exactly 16 times are in a float32 limit cycle (a nearly bipartite, weakly
        // tied component): the remaining sweeps average old and new rows (same fixed point, no such cycle)
        int same_run = 0;
        bool lazy = false;
        unsigned int prev_bits = 0xffffffffu;
        // Scalar labels on a large graph: every sweep after the first as a binned round (dynlp_binned.h) in which
        // every updatable vertex counts as moved, so that V_aff is all of them; a binned round does nothing once
        // its predecessor moved no row by more than tol, which is the stop rule of the static solve.
        Frontier all_rows = f;
        all_rows.ns = c->h_slot[0].next_count;
        all_rows.nl = c->h_slot[0].next_long;
        c->pb_built = false;
        const bool binned = !converged && binned_rounds_pay(c, all_rows) && build_binned(c);
        PackedPlan pk_plan;
        c->pk_built = false;
        const bool relaxed = in_place && !converged && max_iter > 0 && relaxed_rounds_pay(c, all_rows, tol);
        const bool can_pack = !converged && !binned && (relaxed || !in_place) && packed_rounds_pay(c, all_rows, &pk_plan);
        // (synchronous sweeps: after the first chain, since a solve with a loose threshold may end within it)
        bool packed = can_pack && relaxed && build_packed(c, all_rows, pk_plan);
        bool pack_tried = packed || !can_pack || relaxed;
        if (relaxed) {
            const DenseRounds done = dense_rounds(c, all_rows, G, tol, 0, max_iter, binned, packed);
            it = done.rounds;
            last = done.last;
            converged = last <= tol;
            for (const dynlp_round_info& ri : c->log) edges += ri.entries_short + ri.entries_long;
            // sweeps that follow find the size of their row list in the last slot
            if (!converged && it < max_iter)
                HIPCHK(c, hipMemcpyAsync(&slot_of(c, it - 1)->next_count, &start->next_count, 2 * sizeof(unsigned int),
                                         hipMemcpyDeviceToDevice, c->stream));
        }
        bool pb_fresh = true;  // the slots of the binned rounds do not yet hold the current labels
        // synchronous: sweep t reads buf[t & 1], writes buf[(t + 1) & 1]; in place: every sweep reads and writes F
        float* const buf[2] = {c->F, in_place ? c->F : c->F2};
        if (binned) HIPCHK(c, hipMemsetAsync(c->moved[0], 0xff, (size_t)c->moved_words * sizeof(unsigned int), c->stream));
        bool one_xcd = !relaxed && !binned && !packed && xcd_rounds_pay(c, all_rows, G, true);
        while (!converged && it < max_iter) {
            if (one_xcd && it % kChain == 0) {
                const unsigned int sig[3] = {0u, 0u, prev_bits};
                const size_t first_pair = c->events_used / 2;
                run_xcd(c, G, 0, it, std::min<int>(xcd_rounds_at_once(c, it), max_iter - it), buf[it & 1], buf[(it + 1) & 1], true, lazy, tol, 0, same_run, sig);
                const int executed = (int)c->h_xcd->rounds;
                if (c->time_kernels) trim_timed_spans(c, first_pair, it + executed);
                if (executed == 0) one_xcd = false;
                for (int i = 0; i < executed; ++i) {
                    const RoundCtr rc = xcd_round(c->h_xcd->round[i]);
                    std::memcpy(&last, &rc.resid_bits, sizeof(float));
                    edges += (int64_t)rc.edges;
                    c->log.push_back(round_info(rc, 0, G));
                    same_run = rc.resid_bits == prev_bits ? same_run + 1 : 0;
                    prev_bits = rc.resid_bits;
                    if (same_run >= kSameRounds) lazy = true;
                }
                it += executed;
                converged = executed > 0 && last <= tol;
                continue;
            }
            // a chain of sweeps; each checks on the device whether its predecessor already met the stop rule
            const int r = std::min<int>(kChain, max_iter - it);
            const bool chain_binned = binned && !lazy;  // the averaged sweeps of a limit cycle are ordinary ones
            if (!pack_tried && it > 0) {
                pack_tried = true;
                packed = build_packed(c, all_rows, pk_plan);
                if (packed) HIPCHK(c, hipMemsetAsync(c->moved[0], 0xff, (size_t)c->moved_words * sizeof(unsigned int), c->stream));
            }
            const bool chain_packed = packed && !in_place && !lazy;
            for (int i = 0; i < r; ++i) {
                const int t = it + i;
                c->ev_adjacent = i > 0;  // a chain of sweeps is nothing but these launches
                if ((chain_binned || chain_packed) && t > 0) {
                    const PullRoundArgs a{slot_of(c, t - 1), buf[t & 1], buf[(t + 1) & 1], c->moved[0], c->moved[1], c->moved[2],
                                          tol, slot_of(c, t), slot_of(c, t + 1)};
                    if (chain_packed) {
                        launch_packed_round(c, a, t);
                        continue;
                    }
                    launch_binned_round(c, a, t, t == 1 || pb_fresh);
                    pb_fresh = false;
                    continue;
                }
                const UpdateArgs a{slot_of(c, t - 1), t == 0 ? 1 : 2, buf[t & 1], buf[(t + 1) & 1], nullptr, tol,
                                   slot_of(c, t), slot_of(c, t + 1), (int64_t)nq, (int64_t)c->h_slot_start_long,
                                   lazy ? kRowLazy : 0};
                launch_update<false>(c, G, f, a, t);
            }
            const size_t first_pair = c->events_used / 2 - (c->time_kernels ? (size_t)r : 0);
            read_slots(c, it, r);
            {
                int done = 0;
                while (done < r && c->h_slot[done].executed) ++done;
                if (c->time_kernels) trim_timed_spans(c, first_pair, it + done);
            }
            if (!c->h_slot[0].executed) break;  // cannot happen while the stop rule is unmet; never spin on it
            for (int i = 0; i < r; ++i) {
                const RoundCtr& rc = c->h_slot[i];
                if (!rc.executed) break;
                std::memcpy(&last, &rc.resid_bits, sizeof(float));
                edges += (int64_t)(rc.edges + rc.edges_long);
                c->log.push_back(round_info(rc, chain_binned && it > 0 ? 3 : 0, chain_packed && it > 0 ? 0 : G));
                ++it;
                same_run = rc.resid_bits == prev_bits ? same_run + 1 : 0;
                prev_bits = rc.resid_bits;
                if (same_run >= kSameRounds) lazy = true;
                if (last <= tol) {
                    converged = true;
                    break;
                }
            }
        }
        // the labels of the last executed sweep
        if (!in_place) {
            c->F = buf[it & 1];
            c->F2 = buf[(it + 1) & 1];
        }
        // (the counters of the last sweep have arrived, with everything before them, but the events may not have; no wait without
        // them, it costs the release of a context 1 to 2 ms now and then)
        if (c->time_kernels) HIPCHK(c, hipStreamSynchronize(c->stream));
        const float kernel_ms_total = c->time_kernels ? collect_kernel_ms(c) : 0.f;
        if (stats) {
            stats->iterations = it;
            stats->converged = converged ? 1 : 0;
            stats->final_max_delta = last;
            stats->rows_updated = (int64_t)nq * it;
            stats->edges_traversed = edges;
            stats->frontier_initial = nq;
            stats->frontier_peak = nq;
            stats->update_launches = it;
            stats->ms_iterate = ms_since(t_it);
            stats->ms_update_kernel = kernel_ms_total;
            stats->ms_total = ms_since(t0);
        }
        reset_timed_spans(c);
        return converged ? DYNLP_OK : DYNLP_NOT_CONVERGED;
    } catch (const Fail& f) {
        return f.st;
    } catch (const std::bad_alloc&) {
        c->err = "host allocation failed";
        return DYNLP_ERR_OOM;
    }
}

dynlp_status dynlp_apply_batch(dynlp_ctx* c, int64_t k, int64_t m, const int32_t* eu, const int32_t* ev,
                               const float* ew, int64_t s, const int32_t* sv, const int32_t* sc, dynlp_stats* stats) {
    return dynlp_apply_update(c, 0, nullptr, k, m, eu, ev, ew, s, sv, sc, stats);
}

dynlp_status dynlp_apply_update(dynlp_ctx* c, int64_t nd, const int32_t* del, int64_t k, int64_t m, const int32_t* eu,
                                const int32_t* ev, const float* ew, int64_t s, const int32_t* sv, const int32_t* sc,
                                dynlp_stats* stats) {
    if (!c) return DYNLP_ERR_INVALID_ARG;
    fill_stats_zero(stats);
    if (c->poisoned) {
        c->err = "context is unusable after an earlier device or memory error";
        return DYNLP_ERR_STATE;
    }
    auto bad = [&](const std::string& msg) {
        c->err = msg;
        return DYNLP_ERR_INVALID_ARG;
    };
    if (k < 0 || m < 0 || s < 0 || nd < 0) return bad("counts must be >= 0");
    if (nd > 0 && !del) return bad("deleted_vertex is NULL");
    if (m > 0 && (!eu || !ev || !ew)) return bad("edge arrays are NULL");
    if (s > 0 && (!sv || !sc)) return bad("seed arrays are NULL");
    const int64_t n0 = c->n, n1 = c->n + k;
    if (n1 > 0x7ffffffeLL) return bad("vertex count would exceed 2^31-2");
    if (m > 0x3fffffffLL) return bad("too many edges in one batch");
    // a host-resident edge list of more than one chunk is sent in a pipeline (ingest_edges) and checked on the
    // device chunk by chunk as it arrives; a smaller one is checked here, before any device work
    const bool pipelined = !c->dev_ptrs && nd == 0 && m > c->ingest_chunk;
    if (!c->dev_ptrs) {
        std::string e;
        if (!pipelined && !host_check_edges(e, m, n1, eu, ev, ew)) return bad(e);
        if (!host_check_seeds(e, s, n1, c->C, sv, sc)) return bad(e);
        for (int64_t i = 0; i < nd; ++i)
            if (del[i] < 0 || del[i] >= n0) return bad(format_validation(kErrDeleted, i));
    }
    const auto t0 = Clock::now();
    const AtWork at_work(c->device);
    bool mutated = false;
    try {
        HIPCHK(c, hipSetDevice(c->device));
        (void)g_kept.release_older(kKeepMs);
        conjugate_idle(c);
        c->log.clear();
        reset_timed_spans(c);
        // ---- capacity for new vertices; their rows start empty, unlabelled, uniform ----
        if (n1 > c->n_cap) alloc_vertex_arrays(c, n1 + std::max<int64_t>(n1 / 2, 1024));
        BinnedInsert bins(c);
        const bool in_order = m > 0 && 2 * m >= n1 / kInOrderShare;  // many of the rows are touched
        ensure_batch_scratch(c, nd, m, s);
        if (in_order && !pipelined) bins.choose(m, n1);
        if (!bins.on) ensure_ranks(c, m);
        // (with ranks the rows' lengths stay what they are until the rows are sorted)
        const bool use_rank = !bins.on && c->he_rank != nullptr;
        bool small = !pipelined && !bins.on && small_batch(c, nd, k, m, s);
        unsigned int pieces = 0;  // of 16 bytes: the batch in pinned memory, which k_small_check fetches
        const int32_t *d_eu = eu, *d_ev = ev, *d_sv = sv, *d_sc = sc, *d_del = del;
        const float* d_ew = ew;
        c->ingest_chunks_last = 0;
        if (!c->dev_ptrs) {
            // one copy of everything where it is little (six copies of a few hundred bytes cost 5 us each), else one per array
            const void* from[6] = {pipelined ? nullptr : eu, pipelined ? nullptr : ev, pipelined ? nullptr : ew, sv, sc, del};
            const int64_t count[6] = {pipelined ? 0 : m, pipelined ? 0 : m, pipelined ? 0 : m, s, s, nd};
            int64_t at[6], bytes = 0;
            for (int i = 0; i < 6; ++i) {
                at[i] = bytes;
                bytes += round_up(count[i] * 4, 64);
            }
            bool together = bytes > 0 && ensure_pinned(c, bytes);
            if (together && bytes > c->d_io_cap) {
                dev_free(c, c->d_io);
                c->d_io_cap = 0;
                c->d_io = static_cast<unsigned char*>(dev_try_alloc(c, (size_t)c->h_io_cap));
                if (c->d_io) c->d_io_cap = c->h_io_cap;
                else together = false;
            }
            if (together) {
                for (int i = 0; i < 6; ++i)
                    if (count[i] > 0) std::memcpy(c->h_io + at[i], from[i], (size_t)count[i] * 4);
                if (small) pieces = (unsigned int)(bytes / 16);
                else HIPCHK(c, hipMemcpyAsync(c->d_io, c->h_io, (size_t)bytes, hipMemcpyHostToDevice, c->stream));
            } else {
                void* const to[6] = {c->b_eu, c->b_ev, c->b_ew, c->b_sv, c->b_sc, c->b_del};
                for (int i = 0; i < 6; ++i)
                    if (count[i] > 0) HIPCHK(c, hipMemcpyAsync(to[i], from[i], (size_t)count[i] * 4, hipMemcpyHostToDevice, c->stream));
            }
            auto where = [&](int i, void* own) { return together ? static_cast<void*>(c->d_io + at[i]) : own; };
            d_eu = static_cast<int32_t*>(pipelined ? c->b_eu : where(0, c->b_eu));
            d_ev = static_cast<int32_t*>(pipelined ? c->b_ev : where(1, c->b_ev));
            d_ew = static_cast<float*>(pipelined ? c->b_ew : where(2, c->b_ew));
            d_sv = static_cast<int32_t*>(where(3, c->b_sv));
            d_sc = static_cast<int32_t*>(where(4, c->b_sc));
            d_del = static_cast<int32_t*>(where(5, c->b_del));
        }
        const auto step1 = Clock::now();

        // ---- Alg. 2 Step 1.  Everything up to the first list of rows is queued without a wait: the kernels that change the
        // graph look at the result of the checks and at the planned size of the pool themselves (BatchGate).  Deletions come
        // first; the whole batch is checked before anything changes ----
        const unsigned int zero_words = (unsigned int)((sizeof(RoundCtr) * (kRing + 1)) / sizeof(unsigned int)) + kBatchClear;
        int32_t* const dropping = reinterpret_cast<int32_t*>(c->reloc_off);  // (not in use before the plan)
        SmallBatch sb{reinterpret_cast<const uint4*>(c->h_io), reinterpret_cast<uint4*>(c->d_io), pieces,
                      reinterpret_cast<uint4*>(c->ring), (unsigned int)(sizeof(RoundCtr) * (kRing + 1) / 16), (unsigned long long)c->pool_tail, nd, m, s, k, n0, n1, d_del, d_eu,
                      d_ev, d_sv, d_sc, d_ew, c->C, c->Cs, c->coff, c->CP, c->slack, c->bc, c->meta, c->pool, (unsigned long long)c->pool_cap,
                      c->seed_class, c->add_cnt, c->touched, dropping, use_rank ? c->he_rank : nullptr, c->reloc_off, c->flag, c->deg, c->F};
        if (small) {
            hipLaunchKernelGGL(k_small_check, dim3(1 + kSmallClear), dim3(kSmallThreads), 0, c->stream, sb);
        } else {
            hipLaunchKernelGGL(k_batch_begin, dim3(64), dim3(kBlock), 0, c->stream, reinterpret_cast<unsigned int*>(c->ring), zero_words,
                               c->bc, (unsigned long long)c->pool_tail);
            const int64_t checked = nd + (pipelined ? 0 : m) + s;
            if (checked > 0)
                hipLaunchKernelGGL(k_validate_batch, dim3(grid_for(checked)), dim3(kBlock), 0, c->stream, nd, d_del, pipelined ? 0 : m, d_eu,
                                   d_ev, d_ew, s, d_sv, d_sc, n1, n0, c->C, c->seed_class, c->add_cnt, c->bc);
            if (nd + s + k > 0)
                hipLaunchKernelGGL(k_batch_prepare, dim3(grid_for(nd + s + k)), dim3(kBlock), 0, c->stream, c->bc, nd, d_del, s, d_sv, n1,
                                   c->add_cnt, n0, k, c->meta, c->deg, c->seed_class);
        }
        const unsigned int most_blocks = (unsigned int)c->num_cu * 32;  // of kernels that find the number of their rows on the device
        if (nd > 0) {
            mutated = true;
            if (!small)
                hipLaunchKernelGGL(k_delete_rows, dim3(grid_for(nd * 16)), dim3(kBlock), 0, c->stream, nd, d_del, c->C, c->Cs, c->CP,
                                   c->meta, c->pool, c->seed_class, c->flag, c->add_cnt, dropping, c->deg, c->F, c->bc);
            // (rows that lose entries: as many as the deleted rows have entries, which the host does not know; the mean tells)
            const double guess = 16.0 * (double)nd * std::max(1.0, (double)c->entries / (double)std::max<int64_t>(1, c->n));
            hipLaunchKernelGGL(k_drop_deleted_entries, dim3(std::min<unsigned int>(grid_for((int64_t)std::min(guess, 1e9)), most_blocks)),
                               dim3(kBlock), 0, c->stream, c->bc, dropping, c->meta, c->pool, c->seed_class, c->add_cnt, c->deg);
        }
        // where many of the rows are touched, they are listed in the order of their ids after the counting
        int32_t* const as_touched = in_order ? nullptr : c->touched;
        if (small) {
            if (m + nd + k > 0) hipLaunchKernelGGL(k_small_insert, dim3(1), dim3(kSmallThreads), 0, c->stream, sb);
        } else if (pipelined) {
            ingest_edges(c, m, n1, eu, ev, ew, as_touched);
        } else if (m + nd > 0) {
            if (bins.on) bins.launch_count(m, n1, d_eu, d_ev, d_ew);
            const unsigned int count_blocks = m > 0 && !bins.on ? grid_for(ceil_div(2 * m, kAppendItems)) : 0u;
            if (count_blocks > 0 || nd > 0)
                hipLaunchKernelGGL(k_count_halfedges, dim3(count_blocks + (nd > 0 ? grid_for(nd) : 0u)), dim3(kBlock), 0, c->stream, m, n1,
                                   d_eu, d_ev, c->add_cnt, as_touched, c->bc, use_rank ? c->he_rank : nullptr,
                                   use_rank ? c->he_rank + m : nullptr, count_blocks, nd, d_del, c->seed_class);
        }
        if (in_order && !small)
            hipLaunchKernelGGL(k_list_touched, dim3(grid_for(ceil_div(n1, 16))), dim3(kBlock), 0, c->stream, n1, c->add_cnt, c->touched, c->bc);
        // room at the pool tail for the rows whose slack is too small
        const int64_t most_touched = std::min<int64_t>(2 * m, n1);
        if (m > 0 && !small)
            hipLaunchKernelGGL((most_touched >= kPlanItems ? k_plan_reserve<kAppendItems> : k_plan_reserve<1>),
                               dim3(std::min<unsigned int>(grid_for(ceil_div(most_touched, most_touched >= kPlanItems ? kAppendItems : 1)), most_blocks)),
                               dim3(kBlock), 0, c->stream, c->touched, c->meta, c->add_cnt, c->slack, c->reloc_off, c->bc);
        HIPCHK(c, hipGetLastError());
        c->last_init = dynlp_init_info{};
        Frontier universe = frontier_of(c, 2);
        mutated = true;
        c->n = n1;
        for (;;) {
            const BatchGate gate{c->bc, (unsigned long long)c->pool_cap};
            if (k > 0 && !small)
                hipLaunchKernelGGL(k_init_labels, dim3(grid_for(k * c->CP)), dim3(kBlock), 0, c->stream, n0, n1, c->C, c->Cs, c->coff,
                                   c->CP, c->seed_class, c->F);
            if (m > 0) {
                if (!small)
                    hipLaunchKernelGGL(k_relocate, dim3(std::min<unsigned int>(grid_for(most_touched), most_blocks)), dim3(kBlock), 0,
                                       c->stream, c->touched, c->meta, c->add_cnt, c->slack, c->reloc_off, c->pool, gate);
                if (bins.on) bins.launch_write(m, n1, gate);
                else if (!small)
                    hipLaunchKernelGGL(k_write_halfedges, dim3(grid_for(2 * m)), dim3(kBlock), 0, c->stream, m, d_eu, d_ev, d_ew,
                                       c->meta, c->pool, use_rank ? c->he_rank : nullptr, gate);
                // the batch's entries of every row in a fixed order, then degree, scratch and V_aff flag of the row (the
                // relocation offsets are no longer needed: their array holds the lists of rows with long appended segments
                // and of hubs)
                int32_t* long_list = reinterpret_cast<int32_t*>(c->reloc_off);
                int32_t* hub_list = long_list + c->touched_cap;
                // (the mean number of half-edges per touched row, if all rows are touched: the least it can be)
                const int lanes = in_order && most_touched >= kSortRows8 && 2 * m < kSortLanes8 * n1 ? 8 : 16;
                auto sort_finish = lanes == 8 ? k_sort_finish<8> : k_sort_finish<16>;
                const SortFinish f{c->meta, c->pool, c->add_cnt, use_rank ? 1 : 0, long_list, hub_list, c->touched_cap, c->bc, c->deg, c->flag};
                hipLaunchKernelGGL(sort_finish, dim3(std::min<unsigned int>(grid_for(most_touched * lanes), 2 * most_blocks)), dim3(kBlock), 0,
                                   c->stream, c->touched, f, gate);
                // (a context without vertices has none to touch, whatever edges it is given: they are refused)
                hipLaunchKernelGGL(k_sort_long_segments, dim3((unsigned int)std::max<int64_t>(1, std::min<int64_t>(most_touched, 512))), dim3(kSortThreads), 0,
                                   c->stream, f);
            }
            // seeds: clamp one-hot, their neighbours join V_aff; first frontier from the flags (its size goes to the start
            // slot), and the list of all updatable vertices
            if (s > 0)
                hipLaunchKernelGGL(k_apply_seeds, dim3(grid_for(s * 16)), dim3(kBlock), 0, c->stream, s, d_sv, d_sc, c->Cs, c->coff, c->CP,
                                   c->seed_class, c->F, c->meta, c->pool, c->flag, gate);
            launch_compact_start(c, frontier_of(c, 0), universe, gate);
            if (c->h_bc->err || (int64_t)c->h_bc->pool_tail <= c->pool_cap) break;
            // the pool is too small for the plan and nothing has been inserted yet
            const int64_t tail = (int64_t)c->h_bc->pool_tail;
            const int64_t larger = tail + (tail - c->pool_tail) / 2;
            if (bins.on && !grow_pool(c, larger, false)) {
                bins.release();  // the graph needs their memory: places from atomics on the rows' lengths
                bins.on = false;
            }
            if (c->pool_cap < tail) grow_pool(c, larger);
            small = false;  // (sb has the old pool)
        }
        bins.release();
        if (c->h_bc->err) {
            c->n = n0;
            const unsigned int nt = c->h_bc->touched;
            if (nt) hipLaunchKernelGGL(k_clear_counts, dim3(grid_for(nt)), dim3(kBlock), 0, c->stream, nt, c->touched, c->add_cnt);
            HIPCHK(c, hipStreamSynchronize(c->stream));
            return bad(format_validation(error_code(*c->h_bc), error_index(*c->h_bc)));
        }
        c->entries += 2 * m - (int64_t)c->h_bc->removed;
        c->pool_tail = (int64_t)c->h_bc->pool_tail;
        const int64_t relocated = c->h_bc->relocated;
        const auto listed = Clock::now();
        if (c->init_mode == DYNLP_INIT_SUPERNODE && k > 0) run_supernode_init(c, n0, k, m, d_eu, d_ev, d_ew);
        universe.ns = c->h_bc->upd_short;
        universe.nl = c->h_bc->upd_long;
        unsigned int known = c->h_start->start.next_count + c->h_start->start.next_long;  // |V_aff| the host knows of
        // (the host has just waited for Step 1 and will wait for Step 3, so its clock does; four events in the stream and what they
        // are asked for took 32 us of a call of 163, 5 to 20 of one of 270 to 1,500)
        const auto step3 = Clock::now();

        // ---- Step 3: rounds over V_aff, queued in chains of kChain rounds per host round trip ----
        const int64_t frontier_initial = known;
        int64_t peak = known, rows = 0, edges = 0;
        int it = 0, cur = 0;  // round `it` reads the frontier of parity `cur`
        unsigned int known_before = 0;  // |V_aff| when the chain before was queued
        float last = 0.f;
        double avg_len = c->n > 0 ? (double)c->entries / (double)c->n : 1.0;
        bool pingpong = false;
        int stretch_start = 0;  // first round of the running ping-pong stretch
        bool fused = false;     // the stretch's rounds evaluate V_aff themselves (no frontier list, no pull)
        bool binned = false;    // ... as scatter + gather passes (scalar labels)
        bool bin_failed = false;
        bool packed = false;    // ... as packed rounds
        bool pack_failed = false;
        unsigned int moved_last = 0;  // rows that the last round moved
        bool pack_now = false;  // a stretch of packed rounds may begin
        // Rounds that repeat themselves exactly (same |V_aff|, rows moved and max change, 16 times in a row) are in
        // a period-2 cycle kept alive by float32 rounding (in-place rounds too: the few rows of such a V_aff run side
        // by side in one wave and read each other's old values); the rest of the batch's flag-marking rounds then
        // average old and new row (kRowLazy), which has the same fixed point and no such cycle.
        int same_run = 0;
        bool lazy = false;
        unsigned int prev_sig[3] = {0xffffffffu, 0xffffffffu, 0xffffffffu};
        c->pb_built = c->pk_built = false;    // the batch changed the graph
        PackedPlan pk_plan{};
        c->persist_failed = false;
        c->persist_launches_last = c->persist_aborts_last = 0;
        const bool in_place = c->update_mode == DYNLP_UPDATE_IN_PLACE;
        // dynlp_set_final_check: when V_aff has emptied, one more round over every updatable row; rows it moves by
        // more than tol (and their neighbours) start Step 3 again.  check_round = index of the running check round.
        int final_checks = 0, check_round = -1;
        bool relaxed = false;  // the batch has had its relaxed rounds (accelerate)
        bool relax_now = c->tol <= kRelaxNowTol;  // else after one more chain, if V_aff is still that large
        bool verified = !c->final_check;
        // How the rounds run (lanes per row, stretches, averaged rows) is decided where a chain begins, every kChain
        // rounds from round chain0 on.  A launch of k_tail_rounds that ends inside a chain leaves the rest of it to
        // ordinary rounds, so that the order of every row's sum is the same whether or not rounds share launches.
        int chain0 = 0, G = 16;
        // chains without a shared launch after one that found too many entries in its first list: 1, 2, 4, ... 64
        int tail_wait = 0, tail_refused = 0;
        bool xcd_failed = false;  // rounds on one XCD were refused
        bool xcd_dense = false;   // ... stand for rounds of a ping-pong stretch (round log)
        for (;;) {
        while (known > 0 && it < c->max_iter) {
            const int chain_off = (it - chain0) % kChain;
            const bool new_chain = chain_off == 0;
            if (new_chain) G = choose_group(c, avg_len);
            // (32,768 vertices, none of them labelled: relaxed and conjugate rounds are possible and stay first)
            if (!xcd_failed && !pingpong && xcd_rounds_pay(c, universe, G, false) && !relaxed_rounds_pay(c, universe, c->tol)) {
                const bool few = tail_rounds_pay(c, known, known_before, avg_len);  // (V_aff of one workgroup's size)
                const size_t first_pair = c->events_used / 2;
                run_xcd(c, G, cur, it, std::min<int>(xcd_rounds_at_once(c, it) - chain_off, c->max_iter - it), c->F, in_place ? c->F : c->F2, false, lazy,
                        c->tol, chain_off, same_run, prev_sig);
                const int executed = (int)c->h_xcd->rounds;
                if (c->time_kernels) trim_timed_spans(c, first_pair, it + executed);
                if (executed == 0) {
                    xcd_failed = true;
                    continue;
                }
                known_before = known;
                for (int i = 0; i < executed; ++i) {
                    const RoundCtr rc = xcd_round(c->h_xcd->round[i]);
                    const unsigned int nq = rc.rows_short;
                    std::memcpy(&last, &rc.resid_bits, sizeof(float));
                    rows += nq;
                    edges += (int64_t)rc.edges;
                    avg_len = nq ? (double)rc.edges / (double)nq : avg_len;
                    // the log has the kind of round this one stands for
                    bool begins = false;
                    if ((chain_off + i) % kChain == 0) {
                        begins = !xcd_dense && (double)nq >= kDenseEnter * (double)universe.size();
                        xcd_dense = xcd_dense ? (double)nq >= kDenseLeave * (double)universe.size() : begins;
                    }
                    c->log.push_back(round_info(rc, !xcd_dense ? 1 : begins ? 0 : 2, G));
                    if (few) c->log.back().launch_rounds = (float)executed;
                    if (it + i == check_round) verified = rc.changed == 0u;
                    const unsigned int sig[3] = {nq, rc.changed, rc.resid_bits};
                    same_run = std::memcmp(sig, prev_sig, sizeof sig) == 0 ? same_run + 1 : 0;
                    std::memcpy(prev_sig, sig, sizeof sig);
                    if (same_run >= kSameRounds) lazy = true;
                    peak = std::max<int64_t>(peak, nq);
                }
                known = c->h_xcd->next;
                if (!xcd_dense) peak = std::max<int64_t>(peak, known);  // (a stretch does not count the rows of the round after)
                if (!in_place && (executed & 1)) std::swap(c->F, c->F2);
                cur ^= executed & 1;
                it += executed;
                continue;
            }
            const bool may_relax = new_chain && !relaxed && it != check_round &&
                                   (double)known >= kRelaxEnter * (double)universe.size() && relaxed_rounds_pay(c, universe, c->tol);
            const bool relax = may_relax && relax_now;
            relax_now = relax_now || may_relax;
            if (relax) {
                relaxed = true;
                const bool use_bins = binned_rounds_pay(c, universe) && (c->pb_built || build_binned(c));
                const bool use_pack = !use_bins && packed_rounds_pay(c, universe, &pk_plan) && (c->pk_built || build_packed(c, universe, pk_plan));
                const size_t logged = c->log.size();
                const DenseRounds done = dense_rounds(c, universe, G, c->tol, it, c->max_iter - it, use_bins, use_pack);
                it += done.rounds;
                last = done.last;
                if (done.avg_len > 0.0) avg_len = done.avg_len;
                for (size_t i = logged; i < c->log.size(); ++i) {
                    const dynlp_round_info& ri = c->log[i];
                    rows += ri.rows_short + ri.rows_long;
                    edges += ri.entries_short + ri.entries_long;
                    peak = std::max<int64_t>(peak, ri.rows_short + ri.rows_long);
                }
                pingpong = false;
                known = done.changed;
                if (known > 0) {
                    // V_aff after the ordinary round over all rows, as a list
                    RoundCtr* slot = slot_of(c, it - 1);
                    HIPCHK(c, hipMemsetAsync(&slot->next_count, 0, 2 * sizeof(unsigned int), c->stream));
                    launch_pull_frontier(c, universe, avg_len, c->moved[done.last_map], c->moved[(done.last_map + 1) % 3], c->F,
                                         nullptr, frontier_of(c, cur), &slot->next_count, &slot->next_long);
                    read_slots(c, it - 1, 1);
                    known = c->h_slot[0].next_count + c->h_slot[0].next_long;
                }
                chain0 = it;
                continue;
            }
            // A stretch of ping-pong rounds starts when V_aff covers nearly every updatable vertex (one copy
            // of F makes the partner buffer agree on every row outside V_aff) and ends when V_aff has shrunk.
            // Both kinds of round are correct for any V_aff, so the choice is only made between chains.
            // Inside a stretch no frontier list exists: its first round works on the list it was handed, the
            // later ones evaluate V_aff = {u : u or a neighbour moved in the previous round} per row, from
            // the bitmap of moved rows.  Leaving a stretch pulls the list out of the last bitmap once.
            bool can_bin = !bin_failed && binned_rounds_pay(c, universe);
            if (can_bin && new_chain && !pingpong && !c->pb_built && (double)known >= kBinnedEnter * (double)universe.size() &&
                !build_binned(c)) {
                bin_failed = true;  // no memory for the binned arrays: ordinary rounds for this batch
                can_bin = false;
            }
            const bool can_pack = !pack_failed && !in_place && !can_bin && !persistent_rounds_pay(c, universe) &&
                            packed_rounds_pay(c, universe, &pk_plan);
            if (new_chain) {
                pack_now = can_pack && (double)moved_last >= kPackedMoved * (double)universe.size();
                if (pack_now && !c->pk_built && !build_packed(c, universe, pk_plan)) {
                    pack_failed = true;
                    pack_now = false;
                }
            }
            const double enter = can_bin ? kBinnedEnter : pack_now ? kPackedMoved : kDenseEnter;
            // graphs whose rounds run many per launch stay in one stretch from the first round to the last: a round
            // over a small V_aff costs them no more than a launch
            // (not once rounds repeat themselves exactly: the averaged rows that end such a cycle are staged rounds)
            const bool stay = !lazy && !can_bin && fused_rounds_pay(c, avg_len) && persistent_rounds_pay(c, universe);
            if (new_chain && !pingpong && (stay || (double)known >= enter * (double)universe.size())) {
                if (!in_place) sync_partner(c);
                for (unsigned int* mv : c->moved)
                    HIPCHK(c, hipMemsetAsync(mv, 0, (size_t)c->moved_words * sizeof(unsigned int), c->stream));
                pingpong = true;
                stretch_start = it;
                binned = can_bin;
                packed = pack_now;
                fused = binned || packed || fused_rounds_pay(c, avg_len);
            } else if (new_chain && pingpong && fused && !binned && !packed && pack_now) {
                packed = true;  // the stretch goes on as packed rounds (same bitmaps, same buffers)
            } else if (pingpong && !(stay && fused && !binned) &&
                       (double)known < (binned ? kBinnedLeave : packed ? kPackedLeave : kDenseLeave) * (double)universe.size()) {
                pingpong = false;
                if (fused) {
                    // rows of the last round are in F (the buffers were swapped to make it so)
                    const int last = it - 1 - stretch_start;
                    RoundCtr* slot = slot_of(c, it - 1);
                    launch_pull_frontier(c, universe, avg_len, c->moved[last % 3], c->moved[(last + 1) % 3], c->F,
                                         in_place ? nullptr : c->F2, frontier_of(c, cur), &slot->next_count, &slot->next_long);
                }
            }
            // a stretch of short rounds runs many rounds per launch (k_rounds_persistent); its first round, which still
            // works on a frontier list, is an ordinary launch
            const bool persist = pingpong && fused && !binned && persistent_rounds_pay(c, universe);
            // (callers who fix the lanes per row or ask for binned rounds get them; rows so long that they are worth more
            // than 16 lanes do not come in numbers that one CU should handle)
            if (new_chain && tail_wait > 0) --tail_wait;
            const bool tail = !pingpong && tail_wait == 0 && c->group_lanes == 0 && G <= 16 && !(can_bin && c->binned > 0) &&
                              tail_rounds_pay(c, known, known_before, avg_len);
            // where every row that is affected now may bring its neighbours and V_aff then holds nearly every vertex, the
            // first chain is one round: the rounds over all rows that follow cost half a flag-marking round (1M planted blocks,
            // two such rounds / one: 345 us each, whole batch 5.53 / 5.25 ms; 100K kNN 1.44 / 1.40 ms)
            const bool short_first = it == 0 && !pingpong && relaxed_rounds_pay(c, universe, c->tol) &&
                                     (double)known * avg_len >= (double)universe.size();
            const int r = std::min<int>(persist ? kPersistRounds : tail ? kTailRounds : short_first ? 1 : kChain - chain_off, c->max_iter - it);
            const size_t first_pair = c->events_used / 2;
            // ping-pong: round it+i reads buf[i & 1], writes buf[(i + 1) & 1]; in place: always F
            float* const buf[2] = {c->F, in_place ? c->F : c->F2};
            bool persist_launched = false;
            int persist_first = r;  // chain position of the first round that ran inside a persistent launch
            known_before = known;
            if (tail)
                launch_tail(c, G, cur, it, r, (in_place ? kRowByVertex : 0) | (lazy ? kRowLazy : 0), chain_off, same_run, prev_sig);
            for (int i = 0; i < (tail ? 0 : r); ++i) {
                const int t = it + i;
                RoundCtr* slot = slot_of(c, t);
                const Frontier f = frontier_of(c, cur);
                if (pingpong) {
                    const int q = t - stretch_start;  // round of the stretch
                    if (!fused) {
                        // new rows go straight into the partner buffer; the next V_aff is pulled from the bitmap
                        // of rows that moved
                        unsigned int* mv = c->moved[q & 1];
                        const UpdateArgs a{slot_of(c, t - 1), 0, buf[i & 1], buf[(i + 1) & 1], mv, c->tol,
                                           slot, slot_of(c, t + 1), (int64_t)universe.size(), (int64_t)universe.nl};
                        launch_update<false>(c, G, f, a, t);
                        launch_pull_frontier(c, universe, avg_len, mv, c->moved[(q + 1) & 1], buf[(i + 1) & 1],
                                             in_place ? nullptr : buf[i & 1], frontier_of(c, cur ^ 1), &slot->next_count,
                                             &slot->next_long);
                        cur ^= 1;
                    } else if (q == 0) {
                        const UpdateArgs a{slot_of(c, t - 1), 0, buf[i & 1], buf[(i + 1) & 1], c->moved[0], c->tol,
                                           slot, slot_of(c, t + 1), (int64_t)universe.size(), (int64_t)universe.nl};
                        launch_update<false>(c, G, f, a, t);
                    } else {
                        c->ev_adjacent = i > 0;  // fused rounds of one chain follow each other with nothing in between
                        if (persist && !c->persist_failed) {
                            // rounds t .. it + r - 1 in one launch
                            PersistArgs pa;
                            pa.ring = c->ring;
                            pa.t0 = t;
                            pa.rounds = r - i;
                            pa.long_blocks_max = 0;
                            pa.front = universe.front;
                            pa.back = universe.back;
                            pa.ns = universe.ns;
                            pa.nl = universe.nl;
                            pa.meta = c->meta;
                            pa.pool = c->pool;
                            pa.buf0 = buf[i & 1];
                            pa.buf1 = buf[(i + 1) & 1];
                            pa.moved0 = c->moved[0];
                            pa.moved1 = c->moved[1];
                            pa.moved2 = c->moved[2];
                            pa.q0 = q;
                            pa.words = (unsigned int)c->moved_words;
                            pa.tol = c->tol;
                            pa.barrier = c->persist_ctl;
                            pa.spin_limit = c->persist_spin;
                            if (launch_persistent(c, G, universe, pa, t)) {
                                persist_launched = true;
                                persist_first = i;
                                ++c->persist_launches_last;
                                break;
                            }
                            c->persist_failed = true;  // refused: ordinary rounds for the rest of the chain and the batch
                        }
                        const PullRoundArgs a{slot_of(c, t - 1), buf[i & 1], buf[(i + 1) & 1], c->moved[(q - 1) % 3],
                                              c->moved[q % 3], c->moved[(q + 1) % 3], c->tol, slot, slot_of(c, t + 1)};
                        if (binned)
                            launch_binned_round(c, a, t, q == 1);
                        else if (packed)
                            launch_packed_round(c, a, t);
                        else
                            launch_update_pull(c, G, universe, a, t);
                    }
                } else {
                    // rows are staged by frontier position and committed after the kernel; rows that moved mark
                    // themselves and their neighbours
                    // (in-place mode: written straight into F, nothing to commit)
                    const UpdateArgs a{slot_of(c, t - 1), 0, c->F, in_place ? c->F : c->F2, nullptr, c->tol,
                                       slot, slot_of(c, t + 1), (int64_t)universe.size(), (int64_t)universe.nl,
                                       (in_place ? kRowByVertex : 0) | (lazy ? kRowLazy : 0)};
                    launch_update<true>(c, G, f, a, t);
                    if (in_place)
                        launch_compact(c, frontier_of(c, cur ^ 1), &slot->next_count, &slot->next_long, 0);
                    else
                        launch_commit_compact(c, f, slot_of(c, t - 1), (int64_t)universe.size(), frontier_of(c, cur ^ 1),
                                              &slot->next_count, &slot->next_long);
                    cur ^= 1;
                }
            }
            if (persist_launched) {
                // did a workgroup give up at the barrier?  (the rounds whose slots say "executed" are complete either way)
                unsigned int ctl[2] = {0, 0};
                HIPCHK(c, hipMemcpyAsync(ctl, c->persist_ctl, sizeof ctl, hipMemcpyDeviceToHost, c->stream));
                HIPCHK(c, hipStreamSynchronize(c->stream));
                if (ctl[1] != 0u) {
                    c->persist_failed = true;
                    ++c->persist_aborts_last;
                }
            }
            read_slots(c, it, r);
            int executed = 0;
            for (int i = 0; i < r; ++i) {
                const RoundCtr& rc = c->h_slot[i];
                if (!rc.executed) break;
                ++executed;
                const unsigned int nq = rc.rows_short + rc.rows_long;
                std::memcpy(&last, &rc.resid_bits, sizeof(float));
                rows += nq;
                edges += (int64_t)(rc.edges + rc.edges_long);
                avg_len = nq ? (double)(rc.edges + rc.edges_long) / (double)nq : avg_len;
                // the first round of a fused stretch still works on a frontier list
                c->log.push_back(round_info(rc, !pingpong ? 1 : (fused && it + i > stretch_start ? (binned ? 3 : i >= persist_first ? 4 : 2) : 0),
                                            pingpong && packed && it + i > stretch_start ? 0 : G));
                // inside a stretch the next V_aff is not counted: this round's size stands in for it while
                // rows still move
                moved_last = rc.changed;
                known = pingpong && fused ? (rc.changed ? std::max(nq, 1u) : 0u) : rc.next_count + rc.next_long;
                if (it + i == check_round) verified = rc.changed == 0u;  // the check round moved no row by more than tol
                const unsigned int sig[3] = {nq, rc.changed, rc.resid_bits};
                same_run = std::memcmp(sig, prev_sig, sizeof sig) == 0 ? same_run + 1 : 0;
                std::memcpy(prev_sig, sig, sizeof sig);
                if (same_run >= kSameRounds) lazy = true;
                peak = std::max<int64_t>(peak, known);
            }
            if (pingpong && !in_place && (executed & 1)) std::swap(c->F, c->F2);  // the output of the last executed round
            if (c->time_kernels) trim_timed_spans(c, first_pair, it + executed);
            // a persistent launch that gave up at a barrier stops short without V_aff being empty
            const bool cut_short = persist_launched && executed < r && executed > 0 && c->h_slot[executed - 1].changed != 0u;
            it += executed;
            for (int i = tail ? 0 : persist_first; i < executed; ++i)
                c->log[c->log.size() - executed + i].launch_rounds = (float)(tail ? executed : executed - persist_first);
            if (tail) {
                cur ^= executed & 1;
                if (executed > 0) tail_refused = 0;
                else tail_wait = 1 + (1 << std::min(tail_refused++, 6));
                continue;  // V_aff is empty, has outgrown the launch, or the launch has run all its rounds
            }
            if (cut_short || short_first) chain0 = it;
            if (cut_short) continue;
            if (executed < r) known = 0;  // a round found V_aff empty
        }
        if (verified || known > 0 || it >= c->max_iter || universe.size() == 0) break;
        // V_aff is empty: make every updatable vertex the frontier of round `it` (list into the current parity's
        // array, sizes into the slot the round reads them from; a slot past the last executed round is all zero)
        {
            pingpong = false;  // the check round starts a stretch of its own (fresh bitmaps, partner buffer in step)
            RoundCtr* slot = slot_of(c, it - 1);
            HIPCHK(c, hipMemsetAsync(slot, 0, sizeof(RoundCtr), c->stream));
            launch_compact(c, frontier_of(c, cur), &slot->next_count, &slot->next_long, 1);
            known = universe.size();
            check_round = chain0 = it;
            ++final_checks;
        }
        }
        // not converged: max_iter cut the rounds, or cut them before a requested final check had passed
        const unsigned int nq = known > 0 ? known : (verified || universe.size() == 0 ? 0u : 1u);
        HIPCHK(c, hipStreamSynchronize(c->stream));
        const float ms_iterate = ms_since(step3);
        const float kernel_ms_total = c->time_kernels ? collect_kernel_ms(c) : 0.f;
        if (c->last_init.vertices > 0) (void)hipEventElapsedTime(&c->last_init.ms, c->init_ev[0], c->init_ev[1]);
        if (stats) {
            stats->iterations = it;
            stats->converged = nq == 0 ? 1 : 0;
            stats->final_max_delta = last;
            stats->rows_updated = rows;
            stats->edges_traversed = edges;
            stats->frontier_initial = frontier_initial;
            stats->frontier_peak = peak;
            stats->rows_relocated = relocated;
            stats->update_launches = it;
            stats->final_checks = final_checks;
            stats->ingest_chunks = c->ingest_pinned_last ? c->ingest_chunks_last : -c->ingest_chunks_last;
            stats->ms_update_kernel = kernel_ms_total;
            const double insert = c->clock_khz > 0 ? (double)(c->h_bc->clock[1] - c->h_bc->clock[0]) / (double)c->clock_khz : 0.0;
            double both = std::chrono::duration<double, std::milli>(step3 - step1).count();
            // (what of the initialisation the device still had to do when the host went on)
            const double late = std::max(0.0, c->last_init.ms - std::chrono::duration<double, std::milli>(step3 - listed).count());
            both += std::min<double>(late, ms_iterate);
            stats->ms_insert = (float)std::min(insert, both);
            stats->ms_seed = (float)both - stats->ms_insert;
            stats->ms_iterate = (float)(ms_iterate - std::min<double>(late, ms_iterate));
            stats->ms_total = ms_since(t0);
        }
        reset_timed_spans(c);
        return nq == 0 ? DYNLP_OK : DYNLP_NOT_CONVERGED;
    } catch (const Fail& f) {
        if (mutated) c->poisoned = true;
        return f.st;
    } catch (const std::bad_alloc&) {
        c->err = "host allocation failed";
        if (mutated) c->poisoned = true;
        return DYNLP_ERR_OOM;
    }
}

dynlp_status dynlp_get_labels(dynlp_ctx* c, float* soft, int32_t* hard) {
    if (!c) return DYNLP_ERR_INVALID_ARG;
    if (c->poisoned) {
        c->err = "context is unusable after an earlier device or memory error";
        return DYNLP_ERR_STATE;
    }
    const int64_t n = c->n;
    if (n == 0 || (!soft && !hard)) return DYNLP_OK;
    const AtWork at_work(c->device);
    unsigned char* d_out = nullptr;
    dynlp_status st = DYNLP_OK;
    try {
        HIPCHK(c, hipSetDevice(c->device));
        const int64_t soft_bytes = soft ? n * c->C * (int64_t)sizeof(float) : 0, hard_off = round_up(soft_bytes, 64);
        const int64_t out_bytes = hard_off + (hard ? n * (int64_t)sizeof(int32_t) : 0);
        if (c->dev_ptrs) {
            launch_label_output(c, soft, hard);
            HIPCHK(c, hipStreamSynchronize(c->stream));
            return DYNLP_OK;
        }
        // up to kIoBytes: written by the kernel straight into pinned host memory (us for the call, staged and copied / straight:
        // 0.3 MB 39 / 28, 0.6 MB 52 / 41, 1 MB 70 / 58; a context with an allocator of its own asks that for staging from
        // kIoOutBytes on, and copies by way of the pinned memory); else staged in device memory (one array; without memory for it
        // the call fails and the context stays usable)
        const bool pinned = ensure_pinned(c, out_bytes);
        const bool direct = pinned && (out_bytes <= kIoOutBytes || !c->alloc_fn);
        if (!direct) d_out = Temp<unsigned char>(c, out_bytes).release();
        unsigned char* const to = direct ? c->h_io : d_out;
        launch_label_output(c, soft ? reinterpret_cast<float*>(to) : nullptr, hard ? reinterpret_cast<int32_t*>(to + hard_off) : nullptr);
        if (pinned && !direct) HIPCHK(c, hipMemcpyAsync(c->h_io, d_out, (size_t)out_bytes, hipMemcpyDeviceToHost, c->stream));
        if (!pinned && soft) HIPCHK(c, hipMemcpyAsync(soft, d_out, (size_t)soft_bytes, hipMemcpyDeviceToHost, c->stream));
        if (!pinned && hard) HIPCHK(c, hipMemcpyAsync(hard, d_out + hard_off, (size_t)n * sizeof(int32_t), hipMemcpyDeviceToHost, c->stream));
        HIPCHK(c, hipStreamSynchronize(c->stream));
        if (pinned && soft) std::memcpy(soft, c->h_io, (size_t)soft_bytes);
        if (pinned && hard) std::memcpy(hard, c->h_io + hard_off, (size_t)n * sizeof(int32_t));
    } catch (const SoftOom&) {
        st = DYNLP_ERR_OOM;
    } catch (const Fail& f) {
        st = f.st;
    }
    scratch_free(c, d_out);
    return st;
}

int64_t dynlp_static_scratch_bytes(void) { return (int64_t)kStaticScratchBytes; }

dynlp_status dynlp_get_labels_static(dynlp_ctx* c, float* soft, int32_t* hard) {
    if (!c) return DYNLP_ERR_INVALID_ARG;
    if (c->poisoned) {
        c->err = "context is unusable after an earlier device or memory error";
        return DYNLP_ERR_STATE;
    }
    const int64_t n = c->n;
    if (n == 0 || (!soft && !hard)) return DYNLP_OK;
    // staging layout: [soft: n*C floats][padding to 256 bytes][hard: n int32]
    const size_t soft_bytes = soft ? (size_t)n * c->C * sizeof(float) : 0;
    const size_t hard_off = (size_t)round_up((int64_t)soft_bytes, 256);
    const size_t need = hard_off + (hard ? (size_t)n * sizeof(int32_t) : 0);
    if (need > kStaticScratchBytes) {
        c->err = "dynlp_get_labels_static: the labels of " + std::to_string(n) + " vertices need " + std::to_string(need) +
                 " bytes of staging, the static scratch holds " + std::to_string(kStaticScratchBytes) +
                 "; use dynlp_get_labels";
        return DYNLP_ERR_INVALID_ARG;
    }
    void* base = c->device >= 0 && c->device < kMaxDevices ? g_scratch_ptr[c->device] : nullptr;
    if (!base) {
        c->err = std::string("dynlp_get_labels_static: the address of the static scratch could not be resolved on this device (") +
                 (c->device >= 0 && c->device < kMaxDevices ? hipGetErrorString(g_scratch_err[c->device]) : "device ordinal too large") + ")";
        return DYNLP_ERR_DEVICE;
    }
    try {
        HIPCHK(c, hipSetDevice(c->device));
        float* d_soft = soft ? static_cast<float*>(base) : nullptr;
        int32_t* d_hard = hard ? reinterpret_cast<int32_t*>(static_cast<unsigned char*>(base) + hard_off) : nullptr;
        launch_label_output(c, d_soft, d_hard);
        if (soft) HIPCHK(c, hipMemcpyAsync(soft, d_soft, soft_bytes, hipMemcpyDeviceToHost, c->stream));
        if (hard) HIPCHK(c, hipMemcpyAsync(hard, d_hard, (size_t)n * sizeof(int32_t), hipMemcpyDeviceToHost, c->stream));
        HIPCHK(c, hipStreamSynchronize(c->stream));
        return DYNLP_OK;
    } catch (const Fail& f) {
        return f.st;
    }
}

dynlp_status dynlp_export_graph(dynlp_ctx* c, int64_t* row_ptr, int32_t* col, float* w, float* degree,
                                int32_t* seed_class) {
    if (!c) return DYNLP_ERR_INVALID_ARG;
    if (c->poisoned) {
        c->err = "context is unusable after an earlier device or memory error";
        return DYNLP_ERR_STATE;
    }
    if (!row_ptr || (c->entries > 0 && (!col || !w))) {
        c->err = "row_ptr / col / w are NULL";
        return DYNLP_ERR_INVALID_ARG;
    }
    const int64_t n = c->n, nnz = c->entries;
    int64_t *d_rp = nullptr, *sums = nullptr;
    int32_t* d_col = nullptr;
    float* d_w = nullptr;
    dynlp_status st = DYNLP_OK;
    const hipMemcpyKind kind = c->dev_ptrs ? hipMemcpyDeviceToDevice : hipMemcpyDeviceToHost;
    try {
        HIPCHK(c, hipSetDevice(c->device));
        const int64_t nb = grid_for(n);
        d_rp = Temp<int64_t>(c, n + 1).release();
        sums = Temp<int64_t>(c, nb).release();
        int64_t total = 0;
        if (n > 0) {
            hipLaunchKernelGGL(k_row_lens, dim3(nb), dim3(kBlock), 0, c->stream, n, c->meta, d_rp, sums);
            HIPCHK(c, hipGetLastError());
            total = scan_block_sums(c, nb, sums);
            hipLaunchKernelGGL(k_lens_to_row_ptr, dim3(nb), dim3(kBlock), 0, c->stream, n, d_rp, sums);
            HIPCHK(c, hipGetLastError());
        }
        HIPCHK(c, hipMemcpyAsync(d_rp + n, &total, sizeof(int64_t), hipMemcpyHostToDevice, c->stream));
        if (total != nnz) {
            c->err = "internal: entry count mismatch";
            throw Fail{DYNLP_ERR_STATE};
        }
        if (nnz > 0) {
            int32_t* ocol = c->dev_ptrs ? col : (d_col = Temp<int32_t>(c, nnz).release());
            float* ow = c->dev_ptrs ? w : (d_w = Temp<float>(c, nnz).release());
            hipLaunchKernelGGL(k_export_rows, dim3(grid_for(n * 16)), dim3(kBlock), 0, c->stream, n, c->meta, c->pool, d_rp,
                               ocol, ow);
            HIPCHK(c, hipGetLastError());
            if (!c->dev_ptrs) {
                HIPCHK(c, hipMemcpyAsync(col, ocol, (size_t)nnz * 4, hipMemcpyDeviceToHost, c->stream));
                HIPCHK(c, hipMemcpyAsync(w, ow, (size_t)nnz * 4, hipMemcpyDeviceToHost, c->stream));
            }
        }
        HIPCHK(c, hipMemcpyAsync(row_ptr, d_rp, (size_t)(n + 1) * sizeof(int64_t), kind, c->stream));
        if (degree && n > 0) HIPCHK(c, hipMemcpyAsync(degree, c->deg, (size_t)n * sizeof(float), kind, c->stream));
        if (seed_class && n > 0)
            HIPCHK(c, hipMemcpyAsync(seed_class, c->seed_class, (size_t)n * sizeof(int32_t), kind, c->stream));
        HIPCHK(c, hipStreamSynchronize(c->stream));
    } catch (const SoftOom&) {
        (void)hipStreamSynchronize(c->stream);
        st = DYNLP_ERR_OOM;
    } catch (const Fail& f) {
        st = f.st;
    }
    dev_free(c, d_rp);
    dev_free(c, sums);
    dev_free(c, d_col);
    dev_free(c, d_w);
    return st;
}

int64_t dynlp_round_log(const dynlp_ctx* ctx, int64_t cap, dynlp_round_info* out) {
    if (!ctx) return -1;
    const int64_t rounds = (int64_t)ctx->log.size();
    const int64_t k = std::max<int64_t>(0, std::min(cap, rounds));
    if (out && k > 0) std::copy(ctx->log.begin(), ctx->log.begin() + k, out);
    return rounds;
}

}  // extern "C"

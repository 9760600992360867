// scratch.cpp -- device memory of whole calls, kept between calls.
//
// An allocation and its release cost a short call more than its kernels do
// (the release also waits for the whole device): a 128x128x32 forward
// projection took 97 us with them for 39 us of kernels.  So blocks that a call
// gives back stay, for the next calls on any geometry, thread or stream: up to
// KEPT_MAX bytes per device, in use and idle ones together, until the last
// geometry is destroyed or memory runs out.
#include <hip/hip_runtime.h>

#include <mutex>
#include <vector>

#include "internal.h"

namespace petos {

namespace {

constexpr size_t KEPT_MAX = (size_t)256 << 20;
constexpr int KEPT_BLOCKS = 16;

struct Block {
    void* p = nullptr;
    size_t bytes = 0;
    int device = -1;
    hipEvent_t done = nullptr;      // made when first needed
    bool pending = false;           // done marks the end of work that may still use the block,
    hipStream_t stream = nullptr;   // queued here
    bool lent = false;
    unsigned long long use = 0;     // larger: given back later
};

// While another stream of this thread (or, in global mode, of any) is being
// captured, allocations, releases and event queries end that capture with an
// error unless the thread is in relaxed mode.  No call here queues anything on a
// capturing stream.
struct Relaxed {
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    Relaxed() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
    ~Relaxed() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
};

std::mutex g_mu;                    // never held across a call that waits
std::vector<Block> g_blocks;
unsigned long long g_use = 0;

void free_blocks(std::vector<Block>& old) {
    for (auto& b : old) {
        if (b.pending) (void)hipEventSynchronize(b.done);
        if (b.done) (void)hipEventDestroy(b.done);
        (void)hipFree(b.p);
    }
    old.clear();
}

// (g_mu held) whether the block's work is over
bool is_done(Block& b) {
    if (b.pending) {
        const Relaxed relaxed;
        if (hipEventQuery(b.done) == hipSuccess) b.pending = false;
        else (void)hipGetLastError();
    }
    return !b.pending;
}

// (g_mu held) whether one block of `bytes` more keeps the device's bounds, with
// idle blocks taken out for it where `evict` is given, the longest idle first
bool has_room(int device, size_t bytes, std::vector<Block>* evict) {
    for (;;) {
        size_t total = bytes;
        int n = 1;
        auto oldest = g_blocks.end();
        for (auto it = g_blocks.begin(); it != g_blocks.end(); ++it) {
            if (it->device != device) continue;
            total += it->bytes;
            ++n;
            if (!it->lent && is_done(*it) && (oldest == g_blocks.end() || it->use < oldest->use)) oldest = it;
        }
        if (total <= KEPT_MAX && n <= KEPT_BLOCKS) return true;
        if (evict == nullptr || bytes > KEPT_MAX || oldest == g_blocks.end()) return false;
        evict->push_back(*oldest);
        g_blocks.erase(oldest);
    }
}

}  // namespace

void scratch_release() {
    std::vector<Block> old;
    {
        std::lock_guard<std::mutex> lk(g_mu);
        std::vector<Block> lent;
        for (auto& b : g_blocks) (b.lent ? lent : old).push_back(b);
        g_blocks.swap(lent);
    }
    free_blocks(old);
}

bool device_alloc(void** p, size_t bytes) {
    if (hipMalloc(p, bytes) == hipSuccess) return true;
    (void)hipGetLastError();
    scratch_release();              // what is kept may be what is missing
    if (hipMalloc(p, bytes) == hipSuccess) return true;
    (void)hipGetLastError();        // (the next launch would report it again)
    *p = nullptr;
    return false;
}

// A block whose work is done, the smallest that fits, else another block.  A
// call never waits for another stream's work.  Its own stream's blocks can be
// used again at once, but the wait for an event that was just recorded leaves
// a gap of 2 us between the kernels (back-projections of 127x125x29, 10 angles,
// one after the other 60.7 us with one block, 58.6 with three): so the longest
// idle of QUEUED blocks.
//
// A call that is asynchronous (async) takes no block that it would have to free
// or wait for: none if there is no room among the kept ones.
void* scratch_take(size_t bytes, const hipStream_t* s, bool async) {
    constexpr int QUEUED = 3;
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) return nullptr;
    bool kept = false;
    unsigned long long tag = 0;
    std::vector<Block> old;
    Block got;
    {
        std::lock_guard<std::mutex> lk(g_mu);
        Block *done = nullptr, *mine = nullptr;
        int fits = 0;
        for (auto& b : g_blocks) {
            if (b.lent || b.device != dev || b.bytes < bytes) continue;
            ++fits;
            if (is_done(b)) {
                if (done == nullptr || b.bytes < done->bytes) done = &b;
            } else if (s != nullptr && b.stream == *s) {
                if (mine == nullptr || b.use < mine->use) mine = &b;
            }
        }
        Block* take = done;
        if (take == nullptr && (fits >= QUEUED || !has_room(dev, bytes, nullptr))) take = mine;
        if (take == nullptr) kept = has_room(dev, bytes, async ? nullptr : &old);
        if (take != nullptr) {
            take->lent = true;
            got = *take;
        } else if (kept) {
            // (its place, before the memory)
            Block b;
            b.bytes = bytes;
            b.device = dev;
            b.lent = true;
            tag = b.use = ++g_use;
            g_blocks.push_back(b);
        } else if (async) {
            return nullptr;
        }
    }
    if (got.p != nullptr) {
        // (a stream made after another may have its handle)
        if (got.pending && hipStreamWaitEvent(*s, got.done, 0) != hipSuccess) (void)hipEventSynchronize(got.done);
        return got.p;
    }
    const Relaxed relaxed;
    free_blocks(old);
    void* p = nullptr;
    if (!async) {
        (void)device_alloc(&p, bytes);
    } else if (hipMalloc(&p, bytes) != hipSuccess) {
        (void)hipGetLastError();
        p = nullptr;
    }
    if (kept) {
        std::lock_guard<std::mutex> lk(g_mu);
        for (auto it = g_blocks.begin(); it != g_blocks.end(); ++it) {
            if (it->p != nullptr || it->use != tag) continue;
            if (p != nullptr) it->p = p;
            else g_blocks.erase(it);
            break;
        }
    }
    return p;
}

void scratch_give(void* p, const hipStream_t* after) {
    hipEvent_t ev = nullptr;
    bool kept = false;
    {
        std::lock_guard<std::mutex> lk(g_mu);
        for (auto& b : g_blocks)
            if (b.p == p) {
                kept = true;
                ev = b.done;
            }
    }
    bool pending = false;
    if (after) {
        const Relaxed relaxed;
        pending = kept && (ev != nullptr || hipEventCreateWithFlags(&ev, hipEventDisableTiming) == hipSuccess) &&
                  hipEventRecord(ev, *after) == hipSuccess;
        if (!pending) (void)hipStreamSynchronize(*after);
    }
    if (!kept) {
        const Relaxed relaxed;
        (void)hipFree(p);
        return;
    }
    std::lock_guard<std::mutex> lk(g_mu);
    for (auto& b : g_blocks)
        if (b.p == p) {
            b.done = ev;
            b.pending = pending;
            b.stream = after ? *after : nullptr;
            b.lent = false;
            b.use = ++g_use;
        }
}

}  // namespace petos

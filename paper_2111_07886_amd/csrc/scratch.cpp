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
    bool pending = false;           // done marks the end of work that may still use the block
    bool lent = false;
    unsigned long long use = 0;     // larger: given back later
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

// (g_mu held) take idle blocks out, the longest idle first, until one of
// `bytes` more keeps the device's bounds; whether it does
bool make_room(int device, size_t bytes, std::vector<Block>& out) {
    for (;;) {
        size_t total = bytes;
        int n = 1;
        auto oldest = g_blocks.end();
        for (auto it = g_blocks.begin(); it != g_blocks.end(); ++it) {
            if (it->device != device) continue;
            total += it->bytes;
            ++n;
            if (!it->lent && (oldest == g_blocks.end() || it->use < oldest->use)) oldest = it;
        }
        if (total <= KEPT_MAX && n <= KEPT_BLOCKS) return true;
        if (bytes > KEPT_MAX || oldest == g_blocks.end()) return false;
        out.push_back(*oldest);
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

void* scratch_take(size_t bytes, const hipStream_t* s) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) return nullptr;
    bool kept = false;
    std::vector<Block> old;
    Block got;
    {
        std::lock_guard<std::mutex> lk(g_mu);
        Block* best = nullptr;
        for (auto& b : g_blocks)
            if (!b.lent && b.device == dev && b.bytes >= bytes && (best == nullptr || b.bytes < best->bytes)) best = &b;
        if (best != nullptr) {
            best->lent = true;
            got = *best;
        } else {
            kept = make_room(dev, bytes, old);
        }
    }
    if (got.p != nullptr) {
        if (got.pending && (s ? hipStreamWaitEvent(*s, got.done, 0) : hipEventSynchronize(got.done)) != hipSuccess)
            (void)hipDeviceSynchronize();
        return got.p;
    }
    free_blocks(old);
    void* p = nullptr;
    if (!device_alloc(&p, bytes)) return nullptr;
    if (kept) {
        // (another thread may have taken the room: then the block is not kept)
        std::lock_guard<std::mutex> lk(g_mu);
        if (make_room(dev, bytes, old)) {
            Block b;
            b.p = p;
            b.bytes = bytes;
            b.device = dev;
            b.lent = true;
            g_blocks.push_back(b);
        }
    }
    free_blocks(old);
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
        pending = kept && (ev != nullptr || hipEventCreateWithFlags(&ev, hipEventDisableTiming) == hipSuccess) &&
                  hipEventRecord(ev, *after) == hipSuccess;
        if (!pending) (void)hipStreamSynchronize(*after);
    }
    if (!kept) {
        (void)hipFree(p);
        return;
    }
    std::lock_guard<std::mutex> lk(g_mu);
    for (auto& b : g_blocks)
        if (b.p == p) {
            b.done = ev;
            b.pending = pending;
            b.lent = false;
            b.use = ++g_use;
        }
}

}  // namespace petos

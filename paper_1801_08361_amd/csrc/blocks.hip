// Device memory of short-lived objects, kept for the next one of the same
// sizes: a forest's tables are 21 allocations, and giving them to the driver
// and taking them back cost more than a small room's frames (create and
// destroy 0.2 + 0.6 ms of 2.3 ms for 9 frames in a 267 MB forest, and 5.4 ms
// for the destruction alone where the driver's free lists had got into a slow
// state, which quick rebuilding brings about).
//
// A kept block belongs to nobody: whoever gives one back has waited for the
// device, so that any stream or thread can take it, and its contents are as
// undefined as new memory's. At most KEEP_BYTES are kept per process (the
// oldest go first); what was not taken within KEEP_TIME goes back to the
// driver at the next return, and everything kept on a device when an
// allocation there fails.
#include <chrono>
#include <mutex>
#include <vector>

#include "common.h"

namespace rl {

namespace {
using Clock = std::chrono::steady_clock;
constexpr size_t KEEP_BYTES = 4ull << 30;   // a full-size forest (3.5 GB), 1/64 of the device
constexpr std::chrono::seconds KEEP_TIME{10};

struct Block {
    void *p;
    size_t bytes;
    int device;
    Clock::time_point since;
};

struct Kept {
    std::mutex mu;
    std::vector<Block> blocks;   // oldest first
    size_t bytes = 0;
};

// never destroyed: objects may outlive static ones
Kept &kept()
{
    static Kept *k = new Kept();
    return *k;
}

size_t rounded(size_t bytes) { return ((bytes < 1 ? 1 : bytes) + 4095) & ~(size_t)4095; }
}  // namespace

hipError_t block_alloc(void **p, size_t bytes)
{
    const size_t n = rounded(bytes);
    int device = 0;
    hipError_t e = hipGetDevice(&device);
    if (e != hipSuccess) return e;
    Kept &k = kept();
    {
        std::lock_guard<std::mutex> g(k.mu);
        for (size_t i = k.blocks.size(); i-- > 0;)
            if (k.blocks[i].bytes == n && k.blocks[i].device == device) {
                *p = k.blocks[i].p;
                k.bytes -= n;
                k.blocks.erase(k.blocks.begin() + (std::ptrdiff_t)i);
                return hipSuccess;
            }
    }
    e = hipMalloc(p, n);
    if (e != hipErrorOutOfMemory) return e;
    // what is kept on this device goes back before the allocation fails
    bool any = false;
    for (;;) {
        void *q = nullptr;
        {
            std::lock_guard<std::mutex> g(k.mu);
            for (size_t i = 0; i < k.blocks.size() && !q; ++i)
                if (k.blocks[i].device == device) {
                    q = k.blocks[i].p;
                    k.bytes -= k.blocks[i].bytes;
                    k.blocks.erase(k.blocks.begin() + (std::ptrdiff_t)i);
                }
        }
        if (!q) break;
        (void)hipFree(q);
        any = true;
    }
    if (!any) return e;
    (void)hipGetLastError();
    return hipMalloc(p, n);
}

void block_return(void *p, size_t bytes, int device)
{
    const size_t n = rounded(bytes);
    int current = -1;
    // (the caller waited for the current device only)
    if (n > KEEP_BYTES || hipGetDevice(&current) != hipSuccess || current != device) {
        (void)hipFree(p);
        return;
    }
    Kept &k = kept();
    const Clock::time_point now = Clock::now();
    bool in = false;
    for (;;) {
        void *q = nullptr;
        {
            std::lock_guard<std::mutex> g(k.mu);
            if (!in) {
                try {
                    k.blocks.push_back(Block{p, n, device, now});
                } catch (...) {
                    q = p;
                }
                if (!q) k.bytes += n;
                in = true;
            }
            if (!q && !k.blocks.empty() && (k.bytes > KEEP_BYTES || now - k.blocks.front().since > KEEP_TIME)) {
                q = k.blocks.front().p;
                k.bytes -= k.blocks.front().bytes;
                k.blocks.erase(k.blocks.begin());
            }
        }
        if (!q) return;
        (void)hipFree(q);
    }
}

}  // namespace rl

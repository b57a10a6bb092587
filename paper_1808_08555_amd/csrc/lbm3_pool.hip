// Device workspaces kept from one handle for the next.
//
// A differentiable run creates a lattice, its checkpoints and the reverse sweep's workspace (1 GB
// at 256^2 and 100 steps a segment, 4 GB at 1100 x 900 and 20), and releases them with the
// result.  The driver clears the memory it hands out at 25-35 GB/s, so allocating them afresh
// took 60 ms of a 256^2 gradient of 100 steps and 230 ms of an 1100 x 900 one of 20, whose
// kernels run 5 and 8 ms.
//
// Blocks of 1 MiB or more that a handle gives back are kept, per device, up to 1/32 of the
// device's memory in all (9 GB of 288; a larger one is given back at once, and a run that needs
// one, such as 1100 x 900 with 100 steps a segment, pays for it each time); the oldest go back to the driver beyond that, all of
// them when an allocation of the library finds no memory, and on lbm3_release_cached.  A block
// has one owner at a time.  The owner has waited for its streams before it gives a block back:
// only buffers that never leave the library go through here (a lattice's state, which its
// callers may read on streams of their own, does not).
#include <list>
#include <mutex>

#include "lbm3_handle.h"

namespace tcg {
namespace {

struct Block {
    int device;
    void* p;
    size_t bytes, most;  // most: what the pool keeps on this device in all
    bool lent;
};
struct Pool {
    std::mutex mu;
    std::list<Block> all;  // lent and kept; the kept ones in the order they came back
};
// never destroyed: the driver may be gone when a static's destructor runs
Pool& pool()
{
    static Pool* p = new Pool();
    return *p;
}

constexpr size_t kLeast = (size_t)1 << 20;

// with the lock held
size_t kept_bytes(const Pool& P, int device)
{
    size_t n = 0;
    for (const Block& b : P.all)
        if (!b.lent && b.device == device) n += b.bytes;
    return n;
}

void give_back(std::list<Block>& out)
{
    for (const Block& b : out) (void)hipFree(b.p);
    out.clear();
}

}  // namespace

size_t pool_kept()
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    Pool& P = pool();
    std::lock_guard<std::mutex> lock(P.mu);
    return kept_bytes(P, dev);
}

void pool_trim()
{
    Pool& P = pool();
    std::list<Block> out;
    {
        std::lock_guard<std::mutex> lock(P.mu);
        for (auto i = P.all.begin(); i != P.all.end();) {
            const auto b = i++;
            if (!b->lent) out.splice(out.end(), P.all, b);
        }
    }
    give_back(out);
}

hipError_t device_malloc(void** p, size_t bytes)
{
    hipError_t e = hipMalloc(p, bytes);
    if (e == hipErrorOutOfMemory) {
        (void)hipGetLastError();
        pool_trim();
        e = hipMalloc(p, bytes);
    }
    return e;
}

hipError_t pool_malloc(void** p, size_t bytes)
try {
    *p = nullptr;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    Pool& P = pool();
    if (bytes >= kLeast) {
        // the smallest kept block that holds it and is not more than a quarter larger
        std::lock_guard<std::mutex> lock(P.mu);
        Block* best = nullptr;
        for (Block& b : P.all)
            if (!b.lent && b.device == dev && b.bytes >= bytes && b.bytes - bytes <= bytes / 4 &&
                (!best || b.bytes < best->bytes))
                best = &b;
        if (best) {
            best->lent = true;
            *p = best->p;
            return hipSuccess;
        }
    }
    size_t total = 0;  // (smaller blocks are not kept)
    if (bytes >= kLeast && hipDeviceTotalMem(&total, dev) != hipSuccess) total = 0;
    std::list<Block> node(1, Block{dev, nullptr, bytes, total / 32, true});
    e = device_malloc(p, bytes);
    if (e != hipSuccess) return e;
    node.front().p = *p;
    std::lock_guard<std::mutex> lock(P.mu);
    P.all.splice(P.all.end(), node);
    return hipSuccess;
} catch (...) {  // no host memory for the list's node: nothing has been allocated yet
    return hipErrorOutOfMemory;
}

void pool_free(void* p)
{
    if (!p) return;
    Pool& P = pool();
    std::list<Block> out;
    {
        std::lock_guard<std::mutex> lock(P.mu);
        auto b = P.all.begin();
        while (b != P.all.end() && b->p != p) ++b;
        if (b == P.all.end()) return;
        if (b->bytes < kLeast || b->bytes > b->most) {
            out.splice(out.end(), P.all, b);
        } else {
            b->lent = false;
            const int dev = b->device;
            const size_t most = b->most;
            P.all.splice(P.all.end(), P.all, b);  // the latest of the kept ones
            size_t n = kept_bytes(P, dev);
            for (auto i = P.all.begin(); n > most && i != P.all.end();) {
                const auto c = i++;
                if (c->lent || c->device != dev) continue;
                n -= c->bytes;
                out.splice(out.end(), P.all, c);
            }
        }
    }
    give_back(out);
}

}  // namespace tcg

extern "C" int lbm3_release_cached(void)
{
    tcg::pool_trim();
    return LBM3_OK;
}

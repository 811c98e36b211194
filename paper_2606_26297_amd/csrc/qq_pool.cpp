// qq_pool.cpp -- the pool behind DevBuf (qq_pool.h).
#include "qq_pool.h"

#include <map>
#include <mutex>
#include <vector>

namespace qq {
namespace {

struct Block {
    void *p;
    size_t bytes;
};

struct Pool {
    std::vector<Block> free;  // oldest first
    size_t held = 0;
    int problems = 0;
};

// Never destroyed: at process exit the HIP runtime may be gone before static destructors run.
std::mutex &mutex()
{
    static std::mutex *m = new std::mutex;
    return *m;
}
Pool &pool(int device)
{
    static std::map<int, Pool> *m = new std::map<int, Pool>;
    return (*m)[device];
}

size_t bound(const Pool &q) { return q.problems > 0 ? kPoolKeep : kPoolRest; }

// Blocks to free, oldest first, until the pool holds at most `limit` bytes.  The lock is held.
std::vector<Block> evict(Pool &q, size_t limit)
{
    std::vector<Block> out;
    size_t k = 0;
    while (k < q.free.size() && q.held > limit) {
        q.held -= q.free[k].bytes;
        out.push_back(q.free[k++]);
    }
    q.free.erase(q.free.begin(), q.free.begin() + (long)k);
    return out;
}

void free_all(const std::vector<Block> &v)
{
    for (const Block &b : v) (void)hipFree(b.p);
}

}  // namespace

size_t pool_trim(int device)
{
    std::vector<Block> all;
    {
        std::lock_guard<std::mutex> lock(mutex());
        all = evict(pool(device), 0);
    }
    size_t bytes = 0;
    for (const Block &b : all) bytes += b.bytes;
    free_all(all);
    return bytes;
}

hipError_t DevBuf::get(int dev, size_t n, bool lasting)
{
    release();
    device = dev;
    const size_t unit = n >= (2u << 20) ? (2u << 20) : 4096;
    const size_t want = (n + unit - 1) / unit * unit;
    {
        std::lock_guard<std::mutex> lock(mutex());
        Pool &q = pool(dev);
        // the smallest block that fits and is not too large
        const size_t most = lasting ? want + want / 8 : want > (512u << 10) ? 2 * want : (size_t)(1u << 20);
        size_t best = q.free.size();
        for (size_t i = 0; i < q.free.size(); ++i) {
            const size_t b = q.free[i].bytes;
            if (b < want || b > most) continue;
            if (best == q.free.size() || b < q.free[best].bytes) best = i;
        }
        if (best != q.free.size()) {
            p = q.free[best].p;
            bytes = q.free[best].bytes;
            q.held -= bytes;
            q.free.erase(q.free.begin() + (long)best);
            return hipSuccess;
        }
    }
    hipError_t e = hipMalloc(&p, want);
    if (e != hipSuccess) {
        (void)hipGetLastError();  // not for the next launch's check to find
        // the kept blocks may be what is missing
        if (pool_trim(dev) > 0) {
            e = hipMalloc(&p, want);
            if (e != hipSuccess) (void)hipGetLastError();
        }
    }
    if (e != hipSuccess) {
        p = nullptr;
        return e;
    }
    bytes = want;
    return hipSuccess;
}

void DevBuf::release()
{
    const bool was_idle = idle;
    idle = false;
    if (!p) return;
    std::vector<Block> out;
    bool kept = false;
    if (was_idle && bytes <= kPoolKeep) {
        std::lock_guard<std::mutex> lock(mutex());
        Pool &q = pool(device);
        if (bytes <= bound(q)) {
            q.free.push_back({p, bytes});
            q.held += bytes;
            out = evict(q, bound(q));
            kept = true;
        }
    }
    free_all(out);
    if (!kept) (void)hipFree(p);
    p = nullptr;
    bytes = 0;
}

void pool_problem_added(int device)
{
    std::lock_guard<std::mutex> lock(mutex());
    ++pool(device).problems;
}

void pool_problem_removed(int device)
{
    std::vector<Block> out;
    {
        std::lock_guard<std::mutex> lock(mutex());
        Pool &q = pool(device);
        --q.problems;
        out = evict(q, bound(q));
    }
    free_all(out);
}

}  // namespace qq

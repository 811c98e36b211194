// The device-memory pool (qq_pool.cpp) on a counted stand-in for the device's allocator: fit of kept blocks,
// bounds, eviction, the retry after a failing allocation, trimming, and several threads at once.
// Built and run by test_pool_cpu.py.
#include <cstdio>
#include <cstdlib>
#include <map>
#include <mutex>
#include <thread>
#include <vector>

#include "../paper_2606_26297_amd/csrc/qq_pool.h"

namespace {
std::mutex g_lock;
std::map<void *, size_t> g_live;  // blocks handed out by the stand-in
size_t g_bytes = 0, g_capacity = ~(size_t)0;
int g_mallocs = 0, g_frees = 0, g_bad = 0;
bool g_error = false;
char *g_next = reinterpret_cast<char *>(0x100000);
}  // namespace

extern "C" hipError_t hipMalloc(void **p, size_t n)
{
    std::lock_guard<std::mutex> l(g_lock);
    if (g_bytes + n > g_capacity) {
        g_error = true;
        return hipErrorOutOfMemory;
    }
    *p = g_next;
    g_next += n + 4096;
    g_live[*p] = n;
    g_bytes += n;
    ++g_mallocs;
    return hipSuccess;
}
extern "C" hipError_t hipFree(void *p)
{
    std::lock_guard<std::mutex> l(g_lock);
    auto it = g_live.find(p);
    if (it == g_live.end()) {
        ++g_bad;
        return hipErrorInvalidValue;
    }
    g_bytes -= it->second;
    g_live.erase(it);
    ++g_frees;
    return hipSuccess;
}
extern "C" hipError_t hipGetLastError()
{
    const bool e = g_error;
    g_error = false;
    return e ? hipErrorOutOfMemory : hipSuccess;
}

#define CHECK(x)                                                   \
    do {                                                           \
        if (!(x)) {                                                \
            std::printf("line %d: %s\n", __LINE__, #x);            \
            std::exit(1);                                          \
        }                                                          \
    } while (0)

using qq::DevBuf;
constexpr size_t M = 1u << 20, G = 1u << 30;

static void *once(size_t n, bool lasting = false, bool idle = true)
{
    DevBuf b;
    CHECK(b.get(0, n, lasting) == hipSuccess && b.bytes >= n);
    void *p = b.p;
    if (idle) b.done();
    return p;
}

int main()
{
    qq::pool_problem_added(0);
    // a kept block serves the next request that fits; one never declared idle does not
    void *a = once(10 * M);
    CHECK(once(9 * M) == a && once(10 * M) == a);
    CHECK(once(4 * M) != a);  // less than half: not for a call
    CHECK(qq::pool_trim(0) == 14 * M && g_bytes == 0 && g_live.empty());
    a = once(10 * M, false, false);
    CHECK(g_bytes == 0);

    // a handle's request takes an eighth more at most
    a = once(16 * M);
    {
        DevBuf h;
        CHECK(h.get(0, 12 * M, true) == hipSuccess && h.p != a && h.bytes == 12 * M);
        DevBuf k;
        CHECK(k.get(0, 15 * M, true) == hipSuccess && k.p == a);
        k.done();
        h.done();
    }
    CHECK(qq::pool_trim(0) == 28 * M);

    // done() on an empty buffer does not mark the block that it holds later
    {
        DevBuf b;
        b.done();
        CHECK(b.get(0, 8 * M) == hipSuccess);
    }
    CHECK(g_bytes == 0);

    // bounds: 4 GiB while a problem lives, oldest blocks first; larger blocks are not kept
    std::vector<DevBuf> v(6);
    for (auto &b : v) CHECK(b.get(0, G) == hipSuccess);
    for (auto &b : v) b.done();
    v.clear();
    CHECK(g_bytes == qq::kPoolKeep);
    once(5 * G);
    CHECK(g_bytes == qq::kPoolKeep);
    // a second problem leaves the bound, the last one's end lowers it
    qq::pool_problem_added(0);
    qq::pool_problem_removed(0);
    CHECK(g_bytes == qq::kPoolKeep);
    once(64 * M);
    qq::pool_problem_removed(0);
    CHECK(g_bytes <= qq::kPoolRest);
    qq::pool_trim(0);
    CHECK(g_bytes == 0);

    // a failing allocation empties the pool and is tried again; a second failure is reported, and no error is
    // left for the next launch's check
    qq::pool_problem_added(0);
    g_capacity = 3 * G;
    once(2 * G);
    {
        DevBuf b;
        CHECK(b.get(0, 3 * G) == hipSuccess && g_bytes == 3 * G && !g_error);
        DevBuf c;
        CHECK(c.get(0, G) == hipErrorOutOfMemory && c.p == nullptr && !g_error);
        b.done();
    }
    qq::pool_trim(0);
    g_capacity = ~(size_t)0;

    // several threads: no block is handed to two owners
    std::mutex own_lock;
    std::map<void *, int> own;
    std::vector<std::thread> threads;
    for (int t = 0; t < 8; ++t)
        threads.emplace_back([&, t] {
            unsigned r = 12345u + (unsigned)t;
            for (int i = 0; i < 3000; ++i) {
                r = r * 1664525u + 1013904223u;
                DevBuf b;
                CHECK(b.get(0, 1 + (r >> 8) % (3 * M), r & 1) == hipSuccess);
                {
                    std::lock_guard<std::mutex> l(own_lock);
                    CHECK(own[b.p]++ == 0);
                }
                if ((r >> 4) % 97 == 0) qq::pool_trim(0);
                {
                    std::lock_guard<std::mutex> l(own_lock);
                    own[b.p]--;
                }
                if (r & 2) b.done();
            }
        });
    for (auto &t : threads) t.join();
    qq::pool_trim(0);
    CHECK(g_bytes == 0 && g_bad == 0 && g_mallocs == g_frees);
    std::printf("pool ok\n");
    return 0;
}

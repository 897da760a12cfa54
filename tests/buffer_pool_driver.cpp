// Driver of the buffer pool on the host: a memory of a given size behind the
// allocator interface, with injected failures; built with sanitizers by
// test_buffer_pool_host.py.
#include <stdio.h>
#include <stdlib.h>

#include <map>
#include <mutex>
#include <thread>
#include <vector>

#include "buffer_pool.h"

static std::mutex g_lock;
static std::map<void *, size_t> g_live;
static size_t g_held, g_limit = (size_t)1 << 40;
static int g_tries, g_fail;  // g_fail: error to return whatever the memory (0: none)
constexpr int kOom = 2, kOther = 7;

struct Memory {
    static int alloc(void **ptr, size_t bytes)
    {
        std::lock_guard<std::mutex> hold(g_lock);
        ++g_tries;
        if (g_fail)
            return g_fail;
        if (g_held + bytes > g_limit)
            return kOom;
        *ptr = malloc(16);
        g_live[*ptr] = bytes;
        g_held += bytes;
        return 0;
    }
    static bool out_of_memory(int e) { return e == kOom; }
    static void free(void *ptr)
    {
        std::lock_guard<std::mutex> hold(g_lock);
        g_held -= g_live.at(ptr);  // throws on a foreign pointer or a second free
        g_live.erase(ptr);
        ::free(ptr);
    }
};
using Pool = wcs::BufferPool<Memory>;
using Buffer = Pool::Buffer;

static int g_bad;
#define CHECK(x)                                        \
    do {                                                \
        if (!(x)) {                                     \
            printf("line %d: %s\n", __LINE__, #x);      \
            ++g_bad;                                    \
        }                                               \
    } while (0)

constexpr size_t MB = 1 << 20;

int main()
{
    {  // reuse: the smallest that holds it and is not four times too large
        Pool p;
        Buffer a, b, c;
        CHECK(p.take(10 * MB, &a) == 0 && p.take(30 * MB, &b) == 0);
        void *pa = a.ptr, *pb = b.ptr;
        p.give(&a, true);
        p.give(&b, true);
        CHECK(!a.ptr && !b.ptr && g_held == 40 * MB);
        CHECK(p.take(8 * MB, &c) == 0 && c.ptr == pa && c.bytes == 10 * MB);
        CHECK(p.take(9 * MB, &a) == 0 && a.ptr == pb);
        p.give(&a, true);
        CHECK(p.take(7 * MB, &b) == 0 && b.ptr != pb && g_held == 47 * MB);
        p.give(&b, false);  // work may be in flight: freed, not kept
        CHECK(g_held == 40 * MB);
        p.give(&c, true);
    }
    CHECK(g_held == 0);
    {  // bounds: four buffers, 256 MiB in all, oldest out first
        Pool p;
        Buffer b[8];
        for (auto &x : b)
            CHECK(p.take(1 * MB, &x) == 0);
        void *last = b[7].ptr;
        for (auto &x : b)
            p.give(&x, true);
        CHECK(g_held == 4 * MB);
        Buffer big;
        CHECK(p.take(Pool::kMaxBytes - 2 * MB, &big) == 0);
        p.give(&big, true);
        CHECK(g_held == Pool::kMaxBytes);
        CHECK(p.take(1 * MB, &big) == 0 && g_held == Pool::kMaxBytes);
        CHECK(big.ptr != last || p.take(1 * MB, &b[0]) == 0);
        p.give(&big, true);
        p.give(&b[0], true);
        CHECK(p.take(Pool::kMaxBytes + 1, &big) == 0);
        p.give(&big, true);
        CHECK(g_held <= Pool::kMaxBytes);
    }
    CHECK(g_held == 0);
    {  // no memory: whatever the pool keeps goes, for its own and other allocations
        Pool p;
        Buffer a, b, c;
        g_limit = 100 * MB;
        CHECK(p.take(40 * MB, &a) == 0 && p.take(40 * MB, &b) == 0);
        p.give(&a, true);
        p.give(&b, true);
        g_tries = 0;
        CHECK(p.take(5 * MB, &c) == 0 && g_tries == 1);  // fits beside them
        CHECK(p.take(90 * MB, &a) == 0 && g_tries == 3 && g_held == 95 * MB);
        CHECK(p.take(90 * MB, &b) == kOom && !b.ptr && b.bytes == 0 && g_held == 95 * MB);
        CHECK(g_tries == 4);  // nothing kept: no second try
        p.give(&a, true);
        void *ptr = nullptr;
        CHECK(p.alloc(&ptr, 60 * MB) == 0 && ptr && g_held == 65 * MB);
        Memory::free(ptr);
        p.give(&c, true);
        g_fail = kOther;  // another error: neither freed nor tried again
        g_tries = 0;
        CHECK(p.take(50 * MB, &a) == kOther && !a.ptr && g_tries == 1 && g_held == 5 * MB);
        g_fail = 0;
        g_limit = (size_t)1 << 40;
    }
    CHECK(g_held == 0);
    {  // several threads
        Pool p;
        std::vector<std::thread> ts;
        for (int t = 0; t < 4; ++t)
            ts.emplace_back([&p, t] {
                for (int r = 0; r < 500; ++r) {
                    Buffer a, b;
                    if (p.take((size_t)(1 + (r * 7 + t) % 90) * MB, &a) || p.take(3 * MB, &b))
                        ++g_bad;
                    p.give(&a, true);
                    p.give(&b, r % 5 != 0);
                    if (r % 50 == t)
                        p.release();
                }
            });
        for (auto &t : ts)
            t.join();
        CHECK(g_held <= Pool::kMaxBytes);
    }
    CHECK(g_held == 0 && g_live.empty());
    printf("buffer pool %s\n", g_bad ? "FAILED" : "ok");
    return g_bad ? 1 : 0;
}

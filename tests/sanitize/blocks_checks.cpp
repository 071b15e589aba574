// The device blocks kept between indexes (csrc/z3_blocks.hip), compiled for the host against a
// stand-in of the few runtime calls it makes: a block may reach a new owner only after a wait
// for its device's work has succeeded.  Exit status 0 when every check holds.
#include <stdio.h>
#include <stdlib.h>

#include <atomic>
#include <map>
#include <mutex>
#include <set>
#include <thread>
#include <vector>

#include "z3_internal.h"

// ---- the runtime's stand-in -----------------------------------------------------------------
static thread_local int t_dev = 0;
static std::atomic<bool> wait_refused{false}, free_refused{false};
static std::atomic<size_t> fail_above{SIZE_MAX}, held{0};
static std::atomic<int> waits{0}, frees{0};
static std::mutex size_mu;
static std::map<uintptr_t, size_t> sizes;
static uintptr_t next_address = 0x1000;

extern "C" {
hipError_t hipGetDevice(int *d) { *d = t_dev; return hipSuccess; }
hipError_t hipSetDevice(int d) { t_dev = d; return hipSuccess; }
hipError_t hipDeviceSynchronize(void)
{
    ++waits;
    return wait_refused ? hipErrorStreamCaptureUnsupported : hipSuccess;
}
hipError_t hipGetLastError(void) { return hipSuccess; }
// addresses that stand for blocks, never used twice; nothing reads them
hipError_t hipMalloc(void **p, size_t bytes)
{
    if (held + bytes > fail_above) return hipErrorOutOfMemory;
    std::lock_guard<std::mutex> lk(size_mu);
    next_address += 256;
    sizes[next_address] = bytes;
    held += bytes;
    *p = reinterpret_cast<void *>(next_address);
    return hipSuccess;
}
hipError_t hipFree(void *p)
{
    if (free_refused) return hipErrorStreamCaptureUnsupported;
    std::lock_guard<std::mutex> lk(size_mu);
    const auto it = sizes.find(reinterpret_cast<uintptr_t>(p));
    if (it == sizes.end()) abort();
    held -= it->second;
    sizes.erase(it);
    ++frees;
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t, unsigned)
{
    std::lock_guard<std::mutex> lk(size_mu);
    *p = reinterpret_cast<void *>(next_address += 256);
    return hipSuccess;
}
hipError_t hipHostFree(void *) { return hipSuccess; }
}

namespace z3 {
z3_status fail(z3_status s, const char *, ...) { return s; }
z3_status check_hip(hipError_t e, const char *)
{
    return e == hipSuccess ? Z3_OK : (e == hipErrorOutOfMemory ? Z3_ERR_OUT_OF_MEMORY : Z3_ERR_HIP);
}
z3_status alloc_allowed(size_t, const char *) { return Z3_OK; }
}  // namespace z3

using namespace z3;

static int failures = 0;
#define CHECK(c)                                                          \
    do {                                                                  \
        if (!(c)) { fprintf(stderr, "line %d: %s\n", __LINE__, #c); ++failures; } \
    } while (0)

static void *take(size_t bytes)
{
    void *p = nullptr;
    CHECK(device_block(&p, bytes, "test") == Z3_OK && p);
    return p;
}

int main()
{
    const size_t MB = 1 << 20, GB = 1 << 30;
    // given back after a wait: the next owner gets it
    void *a = take(MB);
    CHECK(wait_device(0) == Z3_OK);
    return_block(a, 0);
    CHECK(take(MB) == a);

    // given back where the wait was refused: nobody gets it, until a wait has succeeded
    wait_refused = true;
    CHECK(wait_device(0) != Z3_OK);
    return_block(a, -1);
    void *b = take(MB);
    CHECK(b != a);
    CHECK(wait_device(0) != Z3_OK);
    void *c = take(MB);
    CHECK(c != a && c != b);
    wait_refused = false;
    CHECK(wait_device(0) == Z3_OK);
    CHECK(take(MB) == a);

    // a wait for another device says nothing about this one's work
    t_dev = 1;
    void *d = take(MB);
    return_block(d, 0);  // device 0 was waited for, the block is device 1's
    void *e = take(MB);
    CHECK(e != d);
    CHECK(wait_device(0) == Z3_OK && t_dev == 1);
    void *f = take(MB);
    CHECK(f != d && f != e);
    t_dev = 0;
    CHECK(wait_device(1) == Z3_OK && t_dev == 0);
    t_dev = 1;
    CHECK(take(MB) == d);
    return_block(d, 1);
    return_block(e, 1);
    return_block(f, 1);
    t_dev = 0;
    CHECK(take(MB) != d);

    // bounds: 4 GiB idle a device, the oldest leaving first, larger blocks at once
    release_idle(1);
    std::vector<void *> big;
    for (int i = 0; i < 6; ++i) big.push_back(take(GB + i));
    for (void *p : big) return_block(p, 0);
    int kept = 0;
    for (int i = 5; i >= 0; --i) {
        const int before = frees;
        void *p = take(GB + i);
        kept += p == big[i];
        CHECK(frees == before);
        big[i] = p;
    }
    CHECK(kept == 3);  // three of 1 GiB and a little
    for (void *p : big) return_block(p, 0);
    void *huge = take(5 * GB);
    const size_t h0 = held;
    return_block(huge, 0);
    CHECK(held == h0 - 5 * GB);

    // a failing allocation gives the idle blocks back first, those set aside after a wait too
    big.clear();
    for (int i = 0; i < 3; ++i) big.push_back(take(GB));
    return_block(big[0], 0);
    return_block(big[1], -1);
    release_idle(0);
    const size_t floor_held = held;
    CHECK(floor_held < 3 * GB);
    for (int i = 0; i < 2; ++i) big[i] = take(GB);
    return_block(big[0], 0);
    return_block(big[1], -1);
    fail_above = floor_held + GB + GB / 2;
    void *g = take(GB + 4096);  // fits no idle block's bounds nor the memory beside them
    CHECK(g != big[0] && g != big[1]);
    fail_above = SIZE_MAX;
    // a refused hipFree keeps the block
    return_block(g, 0);
    free_refused = true;
    const size_t h1 = held;
    release_idle(0);
    CHECK(held == h1);
    free_refused = false;
    CHECK(take(GB + 4096) == g);

    // threads that take, give back (with refused waits now and then) and wait: an address has one
    // owner at a time
    std::mutex mu;
    std::set<void *> owned;
    std::atomic<int> twice{0};
    std::vector<std::thread> threads;
    for (int k = 0; k < 4; ++k)
        threads.emplace_back([&, k] {
            unsigned r = 12345u + (unsigned)k;
            for (int i = 0; i < 3000; ++i) {
                r = r * 1664525u + 1013904223u;
                void *p = nullptr;
                if (device_block(&p, 4096 * (1 + r % 7), "test") != Z3_OK) { ++twice; continue; }
                { std::lock_guard<std::mutex> lk(mu); if (!owned.insert(p).second) ++twice; }
                { std::lock_guard<std::mutex> lk(mu); owned.erase(p); }
                const bool ok = r >> 28 != 0 && wait_device(0) == Z3_OK;
                return_block(p, ok ? 0 : -1);
            }
        });
    for (std::thread &t : threads) t.join();
    CHECK(twice == 0);

    // pinned buffers: one that a copy may still write to is not handed on
    void *p = nullptr, *q = nullptr;
    CHECK(pinned_take(&p) == Z3_OK);
    pinned_give(p, true);
    CHECK(pinned_take(&q) == Z3_OK && q == p);
    pinned_give(q, false);
    CHECK(pinned_take(&q) == Z3_OK && q != p);

    if (!failures) printf("block checks ok\n");
    return failures != 0;
}

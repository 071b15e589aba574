// Device memory of the indexes, and pinned host buffers of their builds, kept between them.
//
// An index takes a dozen arrays and gives them back when it is freed; a program that makes an
// index per catalogue paid hipMalloc and hipFree for each (20 of each per build: 4 + 2.6 us
// apiece for 4,000 points, 36 + 20 us for 491,000, 158 + 51 us for 3.1e6: 4 ms of a 65 ms
// estimate).  Blocks given back are kept for the next index, at most kIdleBytes and
// kIdleBlocks per device, the oldest leaving first; all idle blocks are given back to the
// runtime when an allocation fails.
//
// A block is live (it has an owner), idle (no work that uses it is in flight on any stream, so
// the next owner may use it anywhere) or set aside: its owner gave it back but could not wait for
// its work (the runtime refuses a device-wide wait while some stream is being captured).  A
// block set aside has no new owner until a later wait has succeeded.
#include <mutex>
#include <vector>

#include "z3_internal.h"

namespace z3 {

enum class BlockState : unsigned char { live, idle, aside };
struct DevBlock {
    int dev;
    void *p;
    size_t bytes;
    BlockState state;
    uint64_t stamp;  // order in which blocks were given back
};
constexpr size_t kIdleBytes = (size_t)4 << 30;
constexpr size_t kIdleBlocks = 96;
static std::mutex g_mu;
static std::vector<DevBlock> g_blocks;
static uint64_t g_stamp = 0;

// Gives idle blocks of `dev` back to the runtime until at most `bytes` in at most `count` blocks
// are left: those larger than that by themselves first, then the oldest.
static void trim_idle(int dev, size_t bytes, size_t count)
{
    for (;;) {
        void *p = nullptr;
        {
            std::lock_guard<std::mutex> lk(g_mu);
            size_t held = 0, n = 0;
            DevBlock *out = nullptr;
            for (DevBlock &b : g_blocks) {
                if (b.dev != dev || b.state != BlockState::idle) continue;
                held += b.bytes;
                ++n;
                const bool big = b.bytes > bytes, out_big = out && out->bytes > bytes;
                if (!out || (big != out_big ? big : b.stamp < out->stamp)) out = &b;
            }
            if (held <= bytes && n <= count) return;
            out->state = BlockState::live;  // ours while it is being freed
            p = out->p;
        }
        const bool freed = hipFree(p) == hipSuccess;
        if (!freed) (void)hipGetLastError();
        std::lock_guard<std::mutex> lk(g_mu);
        for (DevBlock &b : g_blocks) {
            if (b.p != p) continue;
            if (freed) {
                b = g_blocks.back();
                g_blocks.pop_back();
            } else {
                b.state = BlockState::idle;  // refused (a capture elsewhere): kept
            }
            break;
        }
        if (!freed) return;
    }
}

z3_status device_block(void **p, size_t bytes, const char *what)
{
    *p = nullptr;
    z3_status st = alloc_allowed(bytes, what);
    if (st != Z3_OK) return st;
    int dev = 0;
    if ((st = check_hip(hipGetDevice(&dev), "hipGetDevice")) != Z3_OK) return st;
    {
        // the smallest idle block that fits and is not wasted on a much smaller array
        std::lock_guard<std::mutex> lk(g_mu);
        DevBlock *best = nullptr;
        for (DevBlock &b : g_blocks)
            if (b.dev == dev && b.state == BlockState::idle && b.bytes >= bytes && b.bytes <= 2 * bytes + 65536 &&
                (!best || b.bytes < best->bytes))
                best = &b;
        if (best) {
            best->state = BlockState::live;
            *p = best->p;
            return Z3_OK;
        }
    }
    hipError_t e = hipMalloc(p, bytes);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        release_idle(dev);
        e = hipMalloc(p, bytes);
    }
    if ((st = check_hip(e, what)) != Z3_OK) {
        *p = nullptr;
        return st;
    }
    try {
        std::lock_guard<std::mutex> lk(g_mu);
        g_blocks.push_back(DevBlock{dev, *p, bytes, BlockState::live, 0});
    } catch (...) {
        (void)hipFree(*p);
        *p = nullptr;
        return fail(Z3_ERR_OUT_OF_MEMORY, "%s: host allocation failed", what);
    }
    return Z3_OK;
}

void return_block(void *p, int waited_dev)
{
    if (!p) return;
    {
        std::lock_guard<std::mutex> lk(g_mu);
        for (DevBlock &b : g_blocks)
            if (b.p == p && b.state == BlockState::live) {
                b.state = b.dev == waited_dev ? BlockState::idle : BlockState::aside;
                b.stamp = ++g_stamp;
                break;
            }
    }
    if (waited_dev >= 0) trim_idle(waited_dev, kIdleBytes, kIdleBlocks);
}

z3_status wait_device(int dev)
{
    uint64_t before;
    {
        std::lock_guard<std::mutex> lk(g_mu);
        before = g_stamp;
    }
    int cur = dev;
    hipError_t e = hipGetDevice(&cur);
    if (e == hipSuccess && cur != dev) e = hipSetDevice(dev);
    if (e == hipSuccess) e = hipDeviceSynchronize();
    if (cur != dev) (void)hipSetDevice(cur);
    const z3_status st = check_hip(e, "hipDeviceSynchronize");
    if (st != Z3_OK) {
        (void)hipGetLastError();  // reported by the status alone
        return st;
    }
    {
        std::lock_guard<std::mutex> lk(g_mu);
        for (DevBlock &b : g_blocks)
            if (b.dev == dev && b.state == BlockState::aside && b.stamp <= before) b.state = BlockState::idle;
    }
    trim_idle(dev, kIdleBytes, kIdleBlocks);
    return Z3_OK;
}

void release_idle(int dev)
{
    bool aside = false;
    {
        std::lock_guard<std::mutex> lk(g_mu);
        for (const DevBlock &b : g_blocks) aside = aside || (b.dev == dev && b.state == BlockState::aside);
    }
    if (aside) (void)wait_device(dev);
    trim_idle(dev, 0, 0);
}

// ---- pinned host buffers ------------------------------------------------------------------
// For the sizes a build reads back (one per build running at a time).
constexpr size_t kPinnedIdle = 8;
static std::mutex g_pin_mu;
static std::vector<void *> g_pin_idle = [] { std::vector<void *> v; v.reserve(kPinnedIdle); return v; }();

z3_status pinned_take(void **p)
{
    *p = nullptr;
    {
        std::lock_guard<std::mutex> lk(g_pin_mu);
        if (!g_pin_idle.empty()) {
            *p = g_pin_idle.back();
            g_pin_idle.pop_back();
            return Z3_OK;
        }
    }
    return check_hip(hipHostMalloc(p, kPinnedBytes, hipHostMallocPortable), "pinned host buffer");
}

void pinned_give(void *p, bool waited)
{
    if (!p) return;
    if (waited) {
        std::lock_guard<std::mutex> lk(g_pin_mu);
        if (g_pin_idle.size() < kPinnedIdle) {
            g_pin_idle.push_back(p);
            return;
        }
    }
    if (hipHostFree(p) != hipSuccess) (void)hipGetLastError();
}

}  // namespace z3

// Device memory of the library's handles and setup scratch.
//
// hipMalloc and hipFree cost about 30 and 45 us each and grow with the block
// (mapping, unmapping, the device-wide wait of hipFree).  An AMG setup makes
// some 270 pairs of them, more time than its kernels take below a few million
// cells.  Freed blocks are therefore kept per device for the next allocation
// of about their size.
//
// A block that is freed may still be in use by work in flight on any stream
// (as with hipFree, whose wait covered that): it waits in `pending`, and is
// handed out again only after a device synchronisation, one for all that
// wait.  An allocation that fails gives everything back and tries again; and
// when the last live block of a device is freed, nothing is kept at all.
//
// What is kept is out of reach of the process's other allocators (torch's
// caching one among them), so it is bounded, larger blocks given back first: by
// kPoolBytes per device (FVPCG_POOL_MB sets another bound, 0 keeps nothing),
// and past kSmallBytes by an eighth of what the device has free.  An AMG setup
// leaves about 1.1 to 1.6 KB per cell (0.4 GiB at 64^3, 3.2 at 128^3, 7.4 at
// 192^3), all of it kept while 64 GiB are free.
//
// No call into the runtime is made with the lock held: one that waits for a
// device (hipDeviceSynchronize, hipFree) would keep every other thread from
// its memory for that long, on other devices too.  The blocks such a call is
// about are out of both lists meanwhile (`moving`).
#include <algorithm>
#include <chrono>
#include <condition_variable>
#include <cstdlib>
#include <map>
#include <mutex>
#include <unordered_map>

#include "memory.hpp"

namespace fvpcg {

namespace {

constexpr size_t kPoolBytes = (size_t)8 << 30, kSmallBytes = (size_t)256 << 20;

using Clock = std::chrono::steady_clock;
// The device's free memory is asked for no more often than this: a
// setup frees some 270 blocks in a few milliseconds.
constexpr auto kLookEvery = std::chrono::milliseconds(50);

using Blocks = std::multimap<size_t, void*>;

struct Pool {
    Blocks clean, pending;
    size_t kept = 0;  // bytes in both, and in `pending` blocks being synchronised
    size_t live = 0;  // blocks handed out
    int moving = 0;   // threads that hold some of the pool's blocks for a call
    size_t share = ~(size_t)0;  // an eighth of the free memory, kept blocks included, when last looked at
    Clock::time_point looked{};
};

struct Block {
    int device;
    size_t bytes;
};

// Never destroyed: handles may be freed while the process ends.
struct Registry {
    std::mutex mu;
    std::condition_variable settled;  // a pool's `moving` has dropped
    std::map<int, Pool> pools;
    std::unordered_map<void*, Block> blocks;
};
Registry& registry() {
    static Registry* r = new Registry();
    return *r;
}

// 512 B steps, then an eighth of the size's power of two, then 2 MiB steps.
size_t rounded(size_t bytes) {
    size_t step = 512;
    if (bytes > ((size_t)64 << 20)) {
        step = (size_t)2 << 20;
    } else if (bytes > 4096) {
        size_t p = 4096;
        while (p * 2 <= bytes) p *= 2;
        step = p / 8;
    }
    return (bytes + step - 1) / step * step;
}

// Bytes of device memory free now; false if they cannot be told (for instance
// while a capture is under way).
bool device_free(int device, size_t* bytes) {
    int now = 0;
    size_t all = 0;
    bool ok = hipGetDevice(&now) == hipSuccess && (now == device || hipSetDevice(device) == hipSuccess);
    if (ok) {
        ok = hipMemGetInfo(bytes, &all) == hipSuccess;
        if (now != device) (void)hipSetDevice(now);
    }
    if (!ok) (void)hipGetLastError();
    return ok;
}

size_t pool_bytes() {
    const char* env = getenv("FVPCG_POOL_MB");
    return env && *env ? (size_t)std::max(0.0, atof(env) * 1048576.0) : kPoolBytes;
}

// Moves everything kept into `out`.
void drop_all(Pool& p, Blocks& out) {
    for (Blocks* m : {&p.pending, &p.clean}) {
        for (auto& b : *m) p.kept -= b.first;
        out.merge(*m);
    }
}

// Moves the largest blocks into `out` until at most `limit` bytes are kept.
void drop_above(Pool& p, size_t limit, Blocks& out) {
    while (p.kept > limit && !(p.clean.empty() && p.pending.empty())) {
        Blocks& m = p.clean.empty() || (!p.pending.empty() && p.pending.rbegin()->first > p.clean.rbegin()->first)
                        ? p.pending
                        : p.clean;
        auto last = std::prev(m.end());
        p.kept -= last->first;
        out.insert(m.extract(last));
    }
}

// hipFree of `out`, which was taken from p with the lock held: `lock` is
// released meanwhile.
void give_back(Registry& r, Pool& p, Blocks& out, std::unique_lock<std::mutex>& lock) {
    if (out.empty()) return;
    p.moving += 1;
    lock.unlock();
    for (auto& b : out) (void)hipFree(b.second);
    lock.lock();
    p.moving -= 1;
    r.settled.notify_all();
}

// A kept block of at least `bytes`, at most a quarter larger.
Blocks::iterator fitting(Blocks& m, size_t bytes) {
    auto it = m.lower_bound(bytes);
    return it == m.end() || it->first > bytes + bytes / 4 ? m.end() : it;
}
void* take(Pool& p, size_t bytes, size_t* got) {
    auto it = fitting(p.clean, bytes);
    if (it == p.clean.end()) return nullptr;
    void* q = it->second;
    *got = it->first;
    p.kept -= it->first;
    p.clean.erase(it);
    return q;
}

hipError_t alloc(void** out, size_t bytes) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const size_t need = rounded(bytes ? bytes : 1);
    Registry& r = registry();
    std::unique_lock<std::mutex> lock(r.mu);
    Pool& p = r.pools[dev];
    size_t got = 0;
    void* q = take(p, need, &got);
    if (!q && fitting(p.pending, need) != p.pending.end()) {
        Blocks waiting;
        waiting.swap(p.pending);
        p.moving += 1;
        lock.unlock();
        const bool ok = hipDeviceSynchronize() == hipSuccess;
        if (!ok) (void)hipGetLastError();  // e.g. a capture is under way: a new block
        lock.lock();
        (ok ? p.clean : p.pending).merge(waiting);
        p.moving -= 1;
        r.settled.notify_all();
        q = take(p, need, &got);
    }
    if (!q) {
        got = need;
        lock.unlock();
        e = hipMalloc(&q, need);
        lock.lock();
        if (e != hipSuccess) {
            (void)hipGetLastError();
            // what other threads have in their hands comes back first
            r.settled.wait(lock, [&] { return p.moving == 0; });
            Blocks all;
            drop_all(p, all);
            give_back(r, p, all, lock);
            lock.unlock();
            e = hipMalloc(&q, need);
            lock.lock();
            if (e != hipSuccess) {
                (void)hipGetLastError();
                return e;
            }
        }
    }
    try {
        r.blocks[q] = {dev, got};
    } catch (...) {
        lock.unlock();
        (void)hipFree(q);
        throw;
    }
    p.live += 1;
    *out = q;
    return hipSuccess;
}

}  // namespace

hipError_t pool_alloc(void** out, size_t bytes) noexcept {
    *out = nullptr;
    try {
        return alloc(out, bytes);
    } catch (...) {  // no host memory for the bookkeeping
        return hipErrorOutOfMemory;
    }
}

void pool_free(void* q) noexcept {
    if (!q) return;
    Registry& r = registry();
    std::unique_lock<std::mutex> lock(r.mu);
    auto it = r.blocks.find(q);
    if (it == r.blocks.end()) {
        lock.unlock();
        (void)hipFree(q);
        return;
    }
    const Block b = it->second;
    r.blocks.erase(it);
    Pool& p = r.pools[b.device];
    p.live -= 1;
    bool listed = true;
    try {
        p.pending.insert({b.bytes, q});
        p.kept += b.bytes;
    } catch (...) {  // no host memory to list it: freed below
        listed = false;
    }
    Blocks out;
    if (p.live == 0) {
        drop_all(p, out);
    } else {
        if (p.kept > kSmallBytes && Clock::now() - p.looked > kLookEvery) {
            p.looked = Clock::now();  // other threads need not look now
            lock.unlock();
            size_t bytes = 0;
            const bool told = device_free(b.device, &bytes);
            lock.lock();
            if (told) p.share = (bytes + p.kept) / 8;
        }
        drop_above(p, std::min(pool_bytes(), std::max(kSmallBytes, p.share)), out);
    }
    give_back(r, p, out, lock);
    lock.unlock();
    if (!listed) (void)hipFree(q);
}

}  // namespace fvpcg

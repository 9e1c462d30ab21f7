// The library's memory pool (memory.hip) on a stand-in HIP runtime in host
// memory: run with a scenario's name, exit status 0 if it holds.
#include <hip/hip_runtime_api.h>

#include <atomic>
#include <chrono>
#include <condition_variable>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <new>
#include <string>
#include <thread>
#include <vector>

#include "memory.hpp"

namespace {
constexpr size_t MiB = (size_t)1 << 20, GiB = (size_t)1 << 30;

// the stand-in runtime: addresses are handed out, nothing is stored there
std::mutex mu;
std::condition_variable cv;
std::map<void*, size_t> blocks;
size_t total = (size_t)288 << 30, used = 0, next_addr = (size_t)1 << 40;
std::atomic<int> syncs{0}, frees{0};
thread_local int device = 0;
std::atomic<bool> info_fails{false};
std::atomic<bool> hold{false}, held{false};  // calls that wait for the device are held back; one is
std::atomic<int> new_fails{-1};              // the how-manieth operator new from now throws (-1: none)

void wait_for_device() {
    std::unique_lock<std::mutex> l(mu);
    if (!hold) return;
    held = true;
    cv.notify_all();
    cv.wait_for(l, std::chrono::seconds(3), [] { return !hold; });
}
void until_held() {
    std::unique_lock<std::mutex> l(mu);
    cv.wait_for(l, std::chrono::seconds(3), [] { return held.load(); });
}
void let_go() {
    std::lock_guard<std::mutex> l(mu);
    hold = false;
    held = false;
    cv.notify_all();
}
}  // namespace

extern "C" {
hipError_t hipGetDevice(int* d) { return *d = device, hipSuccess; }
hipError_t hipSetDevice(int d) { return device = d, hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipDeviceSynchronize() {
    ++syncs;
    wait_for_device();
    return hipSuccess;
}
hipError_t hipMalloc(void** p, size_t n) {
    std::lock_guard<std::mutex> l(mu);
    if (used + n > total) return hipErrorOutOfMemory;
    used += n;
    *p = (void*)next_addr;
    next_addr += n;
    const int f = new_fails.exchange(-1);
    blocks[*p] = n;
    new_fails = f;
    return hipSuccess;
}
hipError_t hipFree(void* p) {
    ++frees;
    wait_for_device();
    std::lock_guard<std::mutex> l(mu);
    auto it = blocks.find(p);
    if (it == blocks.end()) std::abort();
    used -= it->second;
    blocks.erase(it);
    return hipSuccess;
}
hipError_t hipMemGetInfo(size_t* f, size_t* t) {
    if (info_fails) return hipErrorUnknown;
    std::lock_guard<std::mutex> l(mu);
    *f = total - used;
    *t = total;
    return hipSuccess;
}
}

void* operator new(size_t n) {
    if (new_fails >= 0 && new_fails-- == 0) throw std::bad_alloc();
    if (void* p = std::malloc(n ? n : 1)) return p;
    throw std::bad_alloc();
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, size_t) noexcept { std::free(p); }

namespace {
using fvpcg::pool_alloc;
using fvpcg::pool_free;

#define CHECK(c)                                               \
    do {                                                       \
        if (!(c)) {                                            \
            std::printf("line %d: %s\n", __LINE__, #c);        \
            std::fflush(stdout);                               \
            std::_Exit(1);                                     \
        }                                                      \
    } while (0)

void* get(size_t n) {
    void* p = nullptr;
    CHECK(pool_alloc(&p, n) == hipSuccess && p);
    return p;
}

// f in a thread of its own: does it end while the device is held?
template <typename F>
bool ends(F f) {
    std::atomic<bool> done{false};
    std::thread t([&] {
        f();
        done = true;
    });
    for (int i = 0; i < 100 && !done; ++i) std::this_thread::sleep_for(std::chrono::milliseconds(10));
    const bool in_time = done;
    let_go();
    t.join();
    return in_time;
}

// Blocks come back after one synchronisation, and all go when the last is freed.
void reuse() {
    void* live = get(MiB);
    void* a = get(40 * MiB);
    pool_free(a);
    CHECK(get(40 * MiB) == a && syncs == 1);
    pool_free(a);
    pool_free(live);
    CHECK(used == 0 && blocks.empty());
}

// One thread's wait for the device does not keep others from the pool: neither
// the synchronisation before a block is handed out again ...
void wait_in_alloc() {
    void *live = get(MiB), *a = get(40 * MiB), *b = get(3 * MiB);
    (void)hipSetDevice(1);
    void* live1 = get(MiB);
    (void)hipSetDevice(0);
    pool_free(a);
    hold = true;
    std::thread waits([&] { CHECK(get(40 * MiB) == a); });
    until_held();
    CHECK(held);
    CHECK(ends([&] {
        void* c = get(5 * MiB);
        pool_free(b);
        (void)hipSetDevice(1);
        pool_free(get(7 * MiB));
        (void)c;
    }));
    waits.join();
    (void)live;
    (void)live1;
}

// ... nor a hipFree.
void wait_in_free() {
    void *live = get(MiB), *b = get(3 * MiB);
    (void)hipSetDevice(1);
    void* last = get(9 * MiB);  // the only block of device 1: given back at once
    (void)hipSetDevice(0);
    hold = true;
    std::thread waits([&] { pool_free(last); });
    until_held();
    CHECK(held);
    CHECK(ends([&] {
        void* c = get(5 * MiB);
        pool_free(b);
        (void)c;
    }));
    waits.join();
    (void)live;
}

// An allocation that fails gets what is kept, also what another thread is
// waiting for just then.
void full() {
    total = 100 * MiB;
    void *live = get(MiB), *a = get(60 * MiB);
    pool_free(a);
    void* b = get(90 * MiB);
    pool_free(b);
    void* c = get(50 * MiB);
    pool_free(c);
    hold = true;
    std::thread waits([&] { pool_free(get(50 * MiB)); });
    until_held();
    std::thread release([] {
        std::this_thread::sleep_for(std::chrono::milliseconds(200));
        let_go();
    });
    void* d = nullptr;
    CHECK(pool_alloc(&d, 95 * MiB) == hipSuccess);
    release.join();
    waits.join();
    pool_free(d);
    pool_free(live);
    CHECK(used == 0);
}

// Threads at random: every block of one owner at a time, all given back at the end.
void threads() {
    total = 40 * MiB;
    std::vector<std::thread> ts;
    std::mutex m;
    std::map<void*, int> owner;
    for (int t = 0; t < 8; ++t)
        ts.emplace_back([&, t] {
            unsigned r = 12345u + (unsigned)t;
            std::vector<void*> mine;
            for (int i = 0; i < 4000; ++i) {
                r = r * 1664525u + 1013904223u;
                if (mine.size() < 4 && (r >> 30)) {
                    void* p = nullptr;
                    if (pool_alloc(&p, (r >> 8) % (2 * MiB) + 1) != hipSuccess) continue;
                    std::lock_guard<std::mutex> l(m);
                    CHECK(owner.emplace(p, t).second);
                    mine.push_back(p);
                } else if (!mine.empty()) {
                    void* p = mine.back();
                    mine.pop_back();
                    {
                        std::lock_guard<std::mutex> l(m);
                        CHECK(owner.erase(p) == 1);
                    }
                    pool_free(p);
                }
            }
            for (void* p : mine) {
                {
                    std::lock_guard<std::mutex> l(m);
                    owner.erase(p);
                }
                pool_free(p);
            }
        });
    for (auto& t : ts) t.join();
    // a thread that waited while the last block went may have kept some
    pool_free(get(1));
    CHECK(used == 0 && blocks.empty());
}
// No memory for the bookkeeping: an allocation fails with the runtime's code
// and leaks nothing, a free still frees; neither throws (frees run in
// destructors).
void no_host_memory() {
    void* live = get(MiB);
    for (int k = 0; k < 6; ++k) {
        const size_t before = used;
        void* p = nullptr;
        new_fails = k;
        const hipError_t e = pool_alloc(&p, 3 * MiB);
        const bool failed = new_fails == -1;
        new_fails = -1;
        CHECK(failed ? e == hipErrorOutOfMemory && !p && used == before : e == hipSuccess && p);
        if (p) pool_free(p);
    }
    for (int k = 0; k < 3; ++k) {
        void* p = get((5 + k) * MiB);
        new_fails = k;
        pool_free(p);
        new_fails = -1;
        CHECK(get((5 + k) * MiB) != nullptr);  // whatever became of it
    }
    (void)live;
}
// What is kept stays within an eighth of the free memory (looked at every 50 ms)
// and the bound that the environment sets; the block just freed counts.
void bounds() {
    void* live = get(MiB);
    auto keep = [&](size_t each, int n) {
        std::vector<void*> v;
        for (int i = 0; i < n; ++i) v.push_back(get(each + (size_t)i * 4096));
        for (void* q : v) {
            std::this_thread::sleep_for(std::chrono::milliseconds(51));
            pool_free(q);
        }
        return used - MiB;  // all but `live`
    };
    CHECK(keep(GiB, 12) <= 8 * GiB && used >= 7 * GiB);
    total = 24 * GiB;
    CHECK(keep(GiB, 12) <= 3 * GiB && used >= 2 * GiB);
    CHECK(keep(64 * MiB, 30) >= 256 * MiB);
    total = used + 200 * MiB;  // the rest of the process has taken the device
    std::this_thread::sleep_for(std::chrono::milliseconds(51));
    void* a = nullptr;
    CHECK(pool_alloc(&a, 100 * MiB) == hipSuccess);
    pool_free(a);
    total = (size_t)288 << 30;
    setenv("FVPCG_POOL_MB", "100", 1);
    CHECK(keep(30 * MiB, 10) <= 100 * MiB);
    setenv("FVPCG_POOL_MB", "0", 1);
    void* b = get(MiB);
    pool_free(b);
    CHECK(blocks.size() == 1);
    pool_free(live);
    CHECK(used == 0);
}

// Where the free memory cannot be told (a capture is under way) nothing is
// given back for it: hipFree is no better off there.
void no_info() {
    void* live = get(MiB);
    std::vector<void*> v;
    for (int i = 0; i < 6; ++i) v.push_back(get(GiB));
    for (int i = 0; i < 3; ++i) pool_free(v[(size_t)i]);
    CHECK(frees == 0);
    info_fails = true;
    std::this_thread::sleep_for(std::chrono::milliseconds(51));
    for (int i = 3; i < 6; ++i) pool_free(v[(size_t)i]);
    CHECK(frees == 0);
    (void)live;
}
}  // namespace

int main(int argc, char** argv) {
    const std::map<std::string, void (*)()> scenarios = {{"reuse", reuse},
                                                         {"wait_in_alloc", wait_in_alloc},
                                                         {"wait_in_free", wait_in_free},
                                                         {"full", full},
                                                         {"threads", threads},
                                                         {"no_host_memory", no_host_memory},
                                                         {"bounds", bounds},
                                                         {"no_info", no_info}};
    auto it = scenarios.find(argc > 1 ? argv[1] : "");
    if (it == scenarios.end()) return 2;
    it->second();
    return 0;
}

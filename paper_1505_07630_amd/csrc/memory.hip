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
// wait.  At most kPoolBytes per device are kept, larger blocks first given
// back; an allocation that fails gives everything back and tries again; and
// when the last live block of a device is freed, nothing is kept at all.
#include <map>
#include <mutex>
#include <unordered_map>
#include <vector>

#include "common.hpp"

namespace fvpcg {

namespace {

constexpr size_t kPoolBytes = (size_t)8 << 30;

struct Pool {
    std::multimap<size_t, void*> clean, pending;
    size_t kept = 0;  // bytes in both
    size_t live = 0;  // blocks handed out
};

struct Block {
    int device;
    size_t bytes;
};

// Never destroyed: handles may be freed while the process ends.
struct Registry {
    std::mutex mu;
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

void release(std::multimap<size_t, void*>& m, size_t* kept) {
    for (auto& b : m) {
        (void)hipFree(b.second);
        *kept -= b.first;
    }
    m.clear();
}

void release_all(Pool& p) {
    release(p.pending, &p.kept);
    release(p.clean, &p.kept);
}

// A kept block of at least `bytes`, at most a quarter larger.
void* take(std::multimap<size_t, void*>& m, size_t bytes, size_t* got) {
    auto it = m.lower_bound(bytes);
    if (it == m.end() || it->first > bytes + bytes / 4) return nullptr;
    void* q = it->second;
    *got = it->first;
    m.erase(it);
    return q;
}

}  // namespace

hipError_t pool_alloc(void** out, size_t bytes) {
    *out = nullptr;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const size_t need = rounded(bytes ? bytes : 1);
    Registry& r = registry();
    std::lock_guard<std::mutex> lock(r.mu);
    Pool& p = r.pools[dev];
    size_t got = 0;
    void* q = take(p.clean, need, &got);
    if (!q && !p.pending.empty()) {
        auto it = p.pending.lower_bound(need);
        if (it != p.pending.end() && it->first <= need + need / 4) {
            if (hipDeviceSynchronize() == hipSuccess) {
                p.clean.insert(p.pending.begin(), p.pending.end());
                p.pending.clear();
                q = take(p.clean, need, &got);
            } else {
                (void)hipGetLastError();  // e.g. a capture is under way: a new block
            }
        }
    }
    if (q) {
        p.kept -= got;
    } else {
        got = need;
        e = hipMalloc(&q, need);
        if (e != hipSuccess) {
            (void)hipGetLastError();
            release_all(p);
            e = hipMalloc(&q, need);
            if (e != hipSuccess) {
                (void)hipGetLastError();
                return e;
            }
        }
    }
    r.blocks[q] = {dev, got};
    p.live += 1;
    *out = q;
    return hipSuccess;
}

void pool_free(void* q) {
    if (!q) return;
    Registry& r = registry();
    std::lock_guard<std::mutex> lock(r.mu);
    auto it = r.blocks.find(q);
    if (it == r.blocks.end()) {
        (void)hipFree(q);
        return;
    }
    const Block b = it->second;
    r.blocks.erase(it);
    Pool& p = r.pools[b.device];
    p.live -= 1;
    p.pending.insert({b.bytes, q});
    p.kept += b.bytes;
    if (p.live == 0) {
        release_all(p);
        return;
    }
    while (p.kept > kPoolBytes) {
        std::multimap<size_t, void*>& m =
            p.clean.empty() || (!p.pending.empty() && p.pending.rbegin()->first > p.clean.rbegin()->first) ? p.pending
                                                                                                             : p.clean;
        auto last = std::prev(m.end());
        (void)hipFree(last->second);
        p.kept -= last->first;
        m.erase(last);
    }
}

}  // namespace fvpcg

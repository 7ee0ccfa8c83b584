// Device memory for indexes and their builds (see hv_internal.h).
#include <mutex>
#include <vector>

#include "hv_internal.h"

namespace hv {
namespace {

struct Block {
    void *p;
    size_t bytes;
    int device;
};

std::mutex g_mu;
std::vector<Block> g_free;  // oldest first
size_t g_free_bytes = 0;

void drop(size_t k) {
    (void)hipFree(g_free[k].p);
    g_free_bytes -= g_free[k].bytes;
    g_free.erase(g_free.begin() + (std::ptrdiff_t)k);
}

bool trim() {  // (g_mu held)
    const bool any = !g_free.empty();
    while (!g_free.empty()) drop(g_free.size() - 1);
    return any;
}

}  // namespace

bool device_trim() {
    std::lock_guard<std::mutex> g(g_mu);
    return trim();
}

hipError_t device_acquire(void **p, size_t bytes, size_t *held) {
    *p = nullptr;
    *held = 0;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    std::lock_guard<std::mutex> g(g_mu);
    // the smallest block that holds the request and is not much larger
    size_t best = g_free.size();
    for (size_t k = 0; k < g_free.size(); ++k)
        if (g_free[k].device == dev && g_free[k].bytes >= bytes && g_free[k].bytes / 2 <= bytes &&
            (best == g_free.size() || g_free[k].bytes < g_free[best].bytes))
            best = k;
    if (best < g_free.size()) {
        *p = g_free[best].p;
        *held = g_free[best].bytes;
        g_free_bytes -= *held;
        g_free.erase(g_free.begin() + (std::ptrdiff_t)best);
        return hipSuccess;
    }
    const size_t want = bytes ? bytes : 1;
    e = hipMalloc(p, want);
    if (e != hipSuccess && trim()) {
        (void)hipGetLastError();
        e = hipMalloc(p, want);
    }
    if (e == hipSuccess) *held = want;
    else *p = nullptr;
    return e;
}

void device_release(void *p, size_t held) {
    int dev = 0;
    hipPointerAttribute_t at;
    if (held > kPoolBytes / 2 || hipGetDevice(&dev) != hipSuccess || hipPointerGetAttributes(&at, p) != hipSuccess ||
        at.device != dev || hipDeviceSynchronize() != hipSuccess) {
        (void)hipGetLastError();
        (void)hipFree(p);
        return;
    }
    std::lock_guard<std::mutex> g(g_mu);
    g_free.push_back(Block{p, held, dev});
    g_free_bytes += held;
    while (g_free_bytes > kPoolBytes) drop(0);
}

}  // namespace hv

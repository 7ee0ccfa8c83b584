// The library's host code without a GPU: this program defines the HIP calls that
// libhv.so makes -- device memory is host memory, kernels are recorded and not
// run -- and takes commands on its standard input, a line each, to which it
// answers with a line each.  Tests read from it what the host code launches,
// allocates and gives back.
#include <cxxabi.h>
#include <hip/hip_runtime_api.h>

#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <iostream>
#include <map>
#include <mutex>
#include <sstream>
#include <string>
#include <thread>
#include <vector>

#include "hv.h"

namespace {
std::mutex mu;
std::map<void *, size_t> live;
size_t live_bytes = 0, most_bytes = 0, limit_bytes = size_t(1) << 40;
// (filled while libhv.so is loaded, before this program's own objects exist)
std::map<const void *, std::string> &names() { static std::map<const void *, std::string> m; return m; }
std::map<const void *, std::vector<char>> &vars() { static std::map<const void *, std::vector<char>> m; return m; }
std::vector<std::string> launches;
struct Graph { std::vector<std::string> nodes; };
thread_local Graph *capturing = nullptr;
thread_local dim3 cfg_grid, cfg_block;
thread_local size_t cfg_lds;
thread_local hipStream_t cfg_stream;

hipError_t take(void **p, size_t n) {
    std::lock_guard<std::mutex> g(mu);
    *p = nullptr;
    if (live_bytes + n > limit_bytes) return hipErrorOutOfMemory;
    *p = aligned_alloc(256, (n + 255) / 256 * 256);
    memset(*p, 0, n);
    live[*p] = n;
    live_bytes += n;
    if (live_bytes > most_bytes) most_bytes = live_bytes;
    return hipSuccess;
}
hipError_t give(void *p) {
    std::lock_guard<std::mutex> g(mu);
    auto at = live.find(p);
    if (at == live.end()) abort();
    live_bytes -= at->second;
    live.erase(at);
    free(p);
    return hipSuccess;
}
}  // namespace

extern "C" {
void **__hipRegisterFatBinary(const void *) { static void *h; return &h; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, void *, void *, int *) {
    int st = 0;
    char *d = abi::__cxa_demangle(name, nullptr, nullptr, &st);
    std::string s = d ? d : name;
    free(d);
    const size_t k = s.find("k_");  // hv::(anonymous namespace)::k_name<...>(...)
    names()[host] = s.substr(k, s.find('(', k) - k);
}
void __hipRegisterVar(void **, void *var, char *, char *, int, size_t size, int, int) { vars()[var].resize(size); }
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, hipStream_t s) {
    cfg_grid = g, cfg_block = b, cfg_lds = lds, cfg_stream = s;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *lds, hipStream_t *s) {
    *g = cfg_grid, *b = cfg_block, *lds = cfg_lds, *s = cfg_stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3 g, dim3 b, void **, size_t lds, hipStream_t) {
    std::ostringstream s;
    s << names()[f] << ":" << g.x << ":" << b.x << ":" << lds;
    std::string t = s.str();
    for (size_t k; (k = t.find(", ")) != std::string::npos;) t.erase(k + 1, 1);
    std::lock_guard<std::mutex> l(mu);
    (capturing ? capturing->nodes : launches).push_back(t);
    return hipSuccess;
}
hipError_t hipMalloc(void **p, size_t n) { return take(p, n); }
hipError_t hipMallocAsync(void **p, size_t n, hipStream_t) { return take(p, n); }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { *p = calloc(1, n); return hipSuccess; }
hipError_t hipFree(void *p) { return p ? give(p) : hipSuccess; }
hipError_t hipFreeAsync(void *p, hipStream_t) { return give(p); }
hipError_t hipHostFree(void *p) { free(p); return hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) {
    if (!capturing) memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemsetAsync(void *p, int v, size_t n, hipStream_t) { memset(p, v, n); return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
const char *hipGetErrorString(hipError_t e) { return e == hipErrorOutOfMemory ? "out of memory" : "error"; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipGetSymbolAddress(void **p, const void *s) { *p = vars()[s].data(); return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) { *e = (hipEvent_t)malloc(1); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) { free((void *)e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { *ms = 1.0f; return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { *s = (hipStream_t)malloc(1); return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t s) { free((void *)s); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { capturing = new Graph; return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *g) { *g = (hipGraph_t)capturing; capturing = nullptr; return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t *x, hipGraph_t g, hipGraphNode_t *, char *, size_t) { *x = (hipGraphExec_t)g; return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t x, hipStream_t) {
    std::lock_guard<std::mutex> l(mu);
    for (auto &n : ((Graph *)x)->nodes) launches.push_back(n);
    return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t g) { delete (Graph *)g; return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int threads, size_t) { *n = 1024 / threads; return hipSuccess; }
hipError_t hipPointerGetAttributes(hipPointerAttribute_t *a, const void *) {
    memset(a, 0, sizeof *a);
    a->type = hipMemoryTypeDevice;
    return hipSuccess;
}
}

int main() {
    std::map<std::string, hv_index *> ix;
    std::map<std::string, hv_batcher *> batchers;
    static unsigned char dummy[256] __attribute__((aligned(256)));
    uint8_t *const out = dummy;  // (never written: no kernel runs)
    double *const objects = (double *)dummy;
    std::string line;
    while (std::getline(std::cin, line)) {
        std::istringstream in(line);
        std::string cmd, name;
        in >> cmd;
        int rc = 0;
        std::ostringstream extra;
        launches.clear();
        auto shape = [&](hv_launch *l) -> hv_launch * {  // region waves objs_per_lane cand_cap grid_wgs; none: default
            memset(l, 0, sizeof *l);
            return in >> l->region >> l->waves_per_wg >> l->objs_per_lane >> l->cand_cap >> l->grid_wgs ? l : nullptr;
        };
        hv_launch l;
        if (cmd == "limit") in >> limit_bytes;
        else if (cmd == "trim") hv_trim();
        else if (cmd == "memory") extra << " " << live_bytes << " " << most_bytes;
        else if (cmd == "build") {  // build NAME KIND N
            int kind;
            int64_t n;
            in >> name >> kind >> n;
            ix[name] = hv_index_build(objects, kind, n);
            hv_info info = {};
            if (!ix[name]) rc = -1;
            else hv_index_info(ix[name], &info);
            extra << " " << info.device_bytes;
        } else if (cmd == "polygons") {  // polygons NAME N: triangles
            int64_t n;
            in >> name >> n;
            std::vector<int64_t> first;
            for (int64_t k = 0; k <= n; k += 3) first.push_back(k);
            ix[name] = hv_polygon_index_build(objects, n, first.data(), n / 3, 0);
            hv_info info = {};
            if (!ix[name]) rc = -1;
            else hv_index_info(ix[name], &info);
            extra << " " << info.device_bytes;
        } else if (cmd == "free") {
            in >> name;
            hv_free(ix[name]);
        } else if (cmd == "batch" || cmd == "aa" || cmd == "tune" || cmd == "run" || cmd == "fill") {
            // CMD NAME Z N [shape]: N requests at zoom Z (run NAME BATCHER Z N K: K of
            // them there, the others at zoom 22)
            std::string b;
            int z;
            int64_t n, there;
            in >> name;
            if (cmd == "run") in >> b;
            in >> z >> n;
            there = n;
            if (cmd == "run") in >> there;
            hv_launch *const L = cmd == "run" ? nullptr : shape(&l);
            std::vector<hv_request> rq((size_t)n);
            std::vector<hv_tile> tiles((size_t)n);
            for (int64_t k = 0; k < n; ++k) {
                memset(&tiles[k], 0, sizeof tiles[k]);
                tiles[k].z = z;
                rq[k] = hv_request{ix[name], k < there ? z : 22, 0, 0, 0, 2.0};
            }
            if (cmd == "batch") rc = hv_render_batch(rq.data(), n, out, L);
            else if (cmd == "aa") rc = hv_render_batch_aa(rq.data(), n, out, L);
            else if (cmd == "fill") rc = hv_render_fill(ix[name], tiles.data(), n, out, L);
            else if (cmd == "run") rc = hv_batcher_run(batchers[b], rq.data(), n, out);
            else {
                rc = hv_autotune(rq.data(), n, out, &l, nullptr);
                extra << " " << l.region << ":" << l.waves_per_wg << ":" << l.objs_per_lane << ":" << l.cand_cap << ":" << l.grid_wgs;
            }
        } else if (cmd == "batcher") {  // batcher NAME MAX
            int64_t n;
            in >> name >> n;
            batchers[name] = hv_batcher_create(n, 4, 8, shape(&l));
            rc = batchers[name] ? 0 : -1;
        } else if (cmd == "threads") {  // threads K: each builds and frees indexes of its own
            int k;
            in >> k;
            std::atomic<int> bad{0};
            std::vector<std::thread> ts;
            for (int t = 0; t < k; ++t)
                ts.emplace_back([&, t] {
                    for (int j = 0; j < 40; ++j) {
                        hv_index *a = hv_index_build(objects, t & 1, 1000 + 4000 * ((t + j) % 7));
                        hv_index *b = hv_index_build(objects, 0, 100000);
                        if (!a || !b) ++bad;
                        hv_free(a);
                        hv_free(b);
                    }
                });
            for (auto &t : ts) t.join();
            rc = bad;
        } else rc = -2;
        std::cout << rc << extra.str();
        if (cmd == "batch" || cmd == "aa" || cmd == "tune" || cmd == "run" || cmd == "fill")
            for (auto &s : launches) std::cout << " " << s;
        if (rc) fprintf(stderr, "%s: %s\n", line.c_str(), hv_last_error());
        std::cout << std::endl;
    }
    _Exit(0);
}

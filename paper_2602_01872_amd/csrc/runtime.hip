// Error reporting and per-kernel event timing for libgrappa_hip.so.
#include "common.h"

#include <map>
#include <mutex>
#include <vector>

namespace grp {

static thread_local std::string g_err;

void set_error(const char* fmt, ...) {
    char buf[1024];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_err = buf;
}

grp_status fail(grp_status code, const char* fmt, ...) {
    char buf[1024];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_err = buf;
    return code;
}

struct ProfRec {
    std::string name;
    hipEvent_t a, b;
    double flops, bytes;
};
static std::mutex g_prof_mu;
static bool g_prof_on = false;
static std::vector<ProfRec> g_prof;
static thread_local hipEvent_t g_open_end = nullptr;
static bool g_prof_detail = false;           // enable value 2: kernel names carry the launch shape
static thread_local char g_detail[96] = {0};

void prof_detail(const char* fmt, ...) {
    if (!g_prof_on || !g_prof_detail) return;
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_detail, sizeof g_detail, fmt, ap);
    va_end(ap);
}

bool prof_enabled() { return g_prof_on; }
void prof_begin(const char* name, hipStream_t st, double flops, double bytes) {
    if (!g_prof_on) return;
    ProfRec r{name, nullptr, nullptr, flops, bytes};
    if (g_prof_detail && g_detail[0]) { r.name += g_detail; }
    g_detail[0] = 0;
    if (hipEventCreate(&r.a) != hipSuccess || hipEventCreate(&r.b) != hipSuccess) return;
    (void)hipEventRecord(r.a, st);
    g_open_end = r.b;
    std::lock_guard<std::mutex> lk(g_prof_mu);
    g_prof.push_back(r);
}

void prof_end(hipStream_t st) {
    if (!g_prof_on || !g_open_end) return;
    (void)hipEventRecord(g_open_end, st);
    g_open_end = nullptr;
}

// ---------------------------------------------------------------- device memory of the builders
// A builder makes a dozen allocations and its handle is freed when the next one exists; hipMalloc and hipFree cost a few
// microseconds when the runtime has the pages at hand and up to a millisecond each when it has to map them (a partition of 3e5 nodes
// out of 6.2e7 edges: 1.5 ms of kernels and transfers inside 10 ms).  Freed blocks are therefore kept and handed out again.
//   - hipFree waits for the device; a freed block waits in `pending` instead, and the first request that one of those
//     could serve waits for the device once and makes all of them ready.  So a block never changes hands while work that
//     was queued before its release, on any stream, can still use it.
//   - A request takes the smallest ready block of at most 1.25 times its size.
//   - At most 1/64 of the device's memory is kept; the block that was freed longest ago goes first.  A block that 64 later
//     requests have passed over is given back.  Everything kept is given back when an allocation fails, when the last block in use on
//     the device is freed (no handle is left there), and by grp_release_memory.
//   - One cache per device, one lock.
namespace {
struct PoolBlock { void* p; size_t bytes; uint64_t freed_at; bool pending; };
struct Pool {
    std::vector<PoolBlock> kept;                 // in the order they were freed
    size_t kept_bytes = 0, bound = 0;
    int64_t live = 0;                            // blocks in use
    uint64_t clock = 0;                          // requests so far
};
std::mutex g_pool_mu;
std::map<int, Pool> g_pools;
std::map<void*, std::pair<int, size_t>> g_pool_live;      // blocks handed out: device and size

void pool_drop(Pool& pool, size_t i) {           // give a kept block back to the runtime
    (void)hipFree(pool.kept[i].p);
    pool.kept_bytes -= pool.kept[i].bytes;
    pool.kept.erase(pool.kept.begin() + (long)i);
}
void pool_drop_all(Pool& pool) {
    while (!pool.kept.empty()) pool_drop(pool, pool.kept.size() - 1);
}
}  // namespace

hipError_t pool_alloc(void** out, size_t bytes) {
    *out = nullptr;
    int dev = 0;
    const hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    size_t unit = 256;                           // sizes are rounded up to eighths of a power of two, so that similar builds fit each other's blocks
    while (unit * 16 <= bytes) unit *= 2;
    const size_t want = (bytes + unit - 1) / unit * unit;
    std::lock_guard<std::mutex> lk(g_pool_mu);
    Pool& pool = g_pools[dev];
    ++pool.clock;
    for (int pass = 0; pass < 2; ++pass) {       // ready blocks first, then, after one wait, the pending ones
        size_t best = pool.kept.size();
        bool waits = false;
        for (size_t i = 0; i < pool.kept.size(); ++i) {
            const PoolBlock& b = pool.kept[i];
            if (b.bytes < want || b.bytes > want + want / 4) continue;
            if (b.pending) { waits = true; continue; }
            if (best == pool.kept.size() || b.bytes < pool.kept[best].bytes) best = i;
        }
        if (best < pool.kept.size()) {
            *out = pool.kept[best].p;
            g_pool_live[*out] = {dev, pool.kept[best].bytes};
            pool.kept_bytes -= pool.kept[best].bytes;
            pool.kept.erase(pool.kept.begin() + (long)best);
            break;
        }
        if (!waits) break;
        if (hipDeviceSynchronize() != hipSuccess) {            // (another thread may be capturing a graph)
            (void)hipGetLastError();
            break;
        }
        for (PoolBlock& b : pool.kept) b.pending = false;
    }
    while (!pool.kept.empty() && pool.clock - pool.kept.front().freed_at > 64) pool_drop(pool, 0);
    if (*out) { ++pool.live; return hipSuccess; }
    hipError_t r = hipMalloc(out, want ? want : 256);
    if (r != hipSuccess && !pool.kept.empty()) {
        (void)hipGetLastError();
        pool_drop_all(pool);
        r = hipMalloc(out, want ? want : 256);
    }
    if (r != hipSuccess) { *out = nullptr; return r; }
    g_pool_live[*out] = {dev, want ? want : 256};
    ++pool.live;
    return hipSuccess;
}

void pool_free(void* p) {
    if (!p) return;
    std::lock_guard<std::mutex> lk(g_pool_mu);
    const auto it = g_pool_live.find(p);
    if (it == g_pool_live.end()) { (void)hipFree(p); return; }
    const int dev = it->second.first;
    const size_t bytes = it->second.second;
    g_pool_live.erase(it);
    Pool& pool = g_pools[dev];
    if (--pool.live == 0) {
        (void)hipFree(p);
        pool_drop_all(pool);
        return;
    }
    if (pool.bound == 0) {
        size_t free_b = 0, total = 0;
        pool.bound = hipMemGetInfo(&free_b, &total) == hipSuccess && total ? total / 64 : 1;
    }
    pool.kept.push_back({p, bytes, pool.clock, true});
    pool.kept_bytes += bytes;
    while (pool.kept_bytes > pool.bound) pool_drop(pool, 0);
}

hipError_t pool_release() {
    int dev = 0;
    const hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    std::lock_guard<std::mutex> lk(g_pool_mu);
    pool_drop_all(g_pools[dev]);
    return hipSuccess;
}

// One helper stream (default priority, not synchronising with the legacy stream) and its events per caller
// stream and device, created at the first request and kept until the process ends.
SideLane* side_lane(hipStream_t main) {
    static std::mutex mu;
    static std::map<std::pair<int, hipStream_t>, SideLane*> lanes;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) { (void)hipGetLastError(); return nullptr; }
    std::lock_guard<std::mutex> lk(mu);
    auto it = lanes.find({dev, main});
    if (it != lanes.end()) return it->second;
    if (main) {            // nothing is created while the caller's stream is being captured
        hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
        if (hipStreamIsCapturing(main, &cs) != hipSuccess || cs != hipStreamCaptureStatusNone) {
            (void)hipGetLastError();
            return nullptr;
        }
    }
    SideLane* lane = new SideLane();
    bool ok = hipStreamCreateWithFlags(&lane->stream, hipStreamNonBlocking) == hipSuccess;
    for (int l = 0; ok && l < GRP_MAX_LAYERS; ++l)
        ok = hipEventCreateWithFlags(&lane->fork[l], hipEventDisableTiming) == hipSuccess;
    ok = ok && hipEventCreateWithFlags(&lane->join, hipEventDisableTiming) == hipSuccess;
    if (!ok) {             // the step then runs on the caller's stream alone; what was created stays allocated
        (void)hipGetLastError();
        return nullptr;
    }
    lanes[{dev, main}] = lane;
    return lane;
}

}  // namespace grp

extern "C" const char* grp_last_error(void) { return grp::g_err.c_str(); }

extern "C" grp_status grp_release_memory(void) {
    GRP_HIP(grp::pool_release());
    return GRP_OK;
}

extern "C" grp_status grp_profile_enable(int32_t on) {
    std::lock_guard<std::mutex> lk(grp::g_prof_mu);
    grp::g_prof_on = on != 0;
    grp::g_prof_detail = on == 2;
    return GRP_OK;
}

extern "C" grp_status grp_profile_report(char* buf, size_t cap) {
    if (!buf || cap == 0) return grp::fail(GRP_EINVAL, "grp_profile_report: null buffer");
    std::vector<grp::ProfRec> recs;
    {
        std::lock_guard<std::mutex> lk(grp::g_prof_mu);
        recs.swap(grp::g_prof);
    }
    struct Acc { long n; double ms, flops, bytes; };
    std::map<std::string, Acc> acc;
    std::vector<std::string> order;
    for (auto& r : recs) {
        float ms = 0.f;
        if (hipEventSynchronize(r.b) == hipSuccess && hipEventElapsedTime(&ms, r.a, r.b) == hipSuccess) {
            auto it = acc.find(r.name);
            if (it == acc.end()) {
                order.push_back(r.name);
                acc[r.name] = Acc{1, ms, r.flops, r.bytes};
            } else {
                it->second.n += 1;
                it->second.ms += ms;
                it->second.flops += r.flops;
                it->second.bytes += r.bytes;
            }
        }
        (void)hipEventDestroy(r.a);
        (void)hipEventDestroy(r.b);
    }
    std::string out;
    char line[320];
    for (auto& nm : order) {
        const Acc& a = acc[nm];
        snprintf(line, sizeof line, "%s %ld %.6f %.6e %.6e\n", nm.c_str(), a.n, a.ms, a.flops, a.bytes);
        out += line;
    }
    if (out.size() + 1 > cap) out.resize(cap - 1);
    memcpy(buf, out.c_str(), out.size() + 1);
    return GRP_OK;
}

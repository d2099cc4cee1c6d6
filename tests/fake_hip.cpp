// A stand-in for the HIP runtime over host memory, and for the kernels, so that
// the host side of uploads (csrc/merf_api.hip) runs on the CPU: a device of a
// chosen size, allocations of every kind, and counts of the calls that would
// wait for the whole device.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <new>

#include "merf_internal.h"

namespace {

struct Pool {
    size_t reserved = 0, used = 0;
    uint64_t threshold = 0;
};
struct Block {
    size_t n;
    Pool *pool;                       // of a pool allocation
};
std::mutex mu;
// the fail_at-th allocation of the code under test throws (0: none)
long fail_at = 0;
thread_local int inside = 0;          // this file's own allocations never do
struct Own {
    Own() { ++inside; }
    ~Own() { --inside; }
};
std::map<void *, Block> device, host;
size_t capacity = SIZE_MAX, plain = 0;
Pool *only = nullptr;                 // one scratch pool (one device)
size_t pool_reserved() { return only ? only->reserved : 0; }
size_t peak = 0;
bool octants_together = false;
long waits = 0;                       // hipFree, hipHostFree, hipStreamDestroy, hipDeviceSynchronize
hipError_t last = hipSuccess;

hipError_t done(hipError_t e) {
    if (e != hipSuccess) last = e;
    return e;
}
hipError_t take(void **p, size_t n, Pool *pool) {
    Own own;
    std::lock_guard<std::mutex> lk(mu);
    *p = nullptr;
    const size_t grow = pool ? std::max(pool->reserved, pool->used + n) - pool->reserved : n;
    if (plain + pool_reserved() + grow > capacity) return done(hipErrorOutOfMemory);
    if (!(*p = std::malloc(std::max<size_t>(n, 1)))) return done(hipErrorOutOfMemory);
    if (pool) {
        pool->reserved += grow;
        pool->used += n;
    } else {
        plain += n;
    }
    peak = std::max(peak, plain + pool_reserved());
    device[*p] = {n, pool};
    return hipSuccess;
}
hipError_t give(void *p) {
    if (!p) return hipSuccess;
    std::lock_guard<std::mutex> lk(mu);
    auto it = device.find(p);
    if (it == device.end()) return done(hipErrorInvalidValue);
    if (Pool *q = it->second.pool) {
        q->used -= it->second.n;
        q->reserved = std::max(q->used, std::min<size_t>(q->reserved, q->threshold));
    } else {
        plain -= it->second.n;
    }
    device.erase(it);
    std::free(p);
    return hipSuccess;
}
// bytes of the device allocation that holds p, from p on
size_t room(const void *p) {
    std::lock_guard<std::mutex> lk(mu);
    auto it = device.upper_bound(const_cast<void *>(p));
    if (it == device.begin()) return 0;
    --it;
    const size_t at = static_cast<const char *>(p) - static_cast<const char *>(it->first);
    return at < it->second.n ? it->second.n - at : 0;
}

}  // namespace

void *operator new(size_t n) {
    if (!inside && fail_at > 0 && __atomic_sub_fetch(&fail_at, 1, __ATOMIC_RELAXED) == 0) throw std::bad_alloc();
    if (void *p = std::malloc(std::max<size_t>(n, 1))) return p;
    throw std::bad_alloc();
}
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, size_t) noexcept { std::free(p); }

extern "C" {

hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetLastError() { const hipError_t e = last; last = hipSuccess; return e; }
hipError_t hipPeekAtLastError() { return last; }
const char *hipGetErrorString(hipError_t e) { return e == hipErrorOutOfMemory ? "out of memory" : "an error"; }
hipError_t hipDeviceSynchronize() { ++waits; return hipSuccess; }
hipError_t hipMalloc(void **p, size_t n) { return take(p, n, nullptr); }
hipError_t hipFree(void *p) { ++waits; return give(p); }
hipError_t hipMallocAsync(void **p, size_t n, hipStream_t) { return take(p, n, nullptr); }
hipError_t hipFreeAsync(void *p, hipStream_t) { return give(p); }
hipError_t hipMemPoolCreate(hipMemPool_t *p, const hipMemPoolProps *) {
    Own own;
    only = new Pool();
    *p = reinterpret_cast<hipMemPool_t>(only);
    return hipSuccess;
}
hipError_t hipMemPoolDestroy(hipMemPool_t) { return hipSuccess; }
hipError_t hipMemPoolSetAttribute(hipMemPool_t p, hipMemPoolAttr, void *v) {
    reinterpret_cast<Pool *>(p)->threshold = *static_cast<uint64_t *>(v);
    return hipSuccess;
}
hipError_t hipMemPoolTrimTo(hipMemPool_t p, size_t n) {
    std::lock_guard<std::mutex> lk(mu);
    Pool *q = reinterpret_cast<Pool *>(p);
    q->reserved = std::max(q->used, std::min(q->reserved, n));
    return hipSuccess;
}
hipError_t hipMallocFromPoolAsync(void **p, size_t n, hipMemPool_t pool, hipStream_t) {
    return take(p, n, reinterpret_cast<Pool *>(pool));
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned) {
    Own own;
    *p = std::malloc(n);
    std::lock_guard<std::mutex> lk(mu);
    host[*p] = {n, nullptr};
    return hipSuccess;
}
hipError_t hipHostFree(void *p) {
    ++waits;
    std::lock_guard<std::mutex> lk(mu);
    host.erase(p);
    std::free(p);
    return hipSuccess;
}
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t) { std::memset(d, v, n); return hipSuccess; }
hipError_t hipPointerGetAttributes(hipPointerAttribute_t *a, const void *p) {
    a->type = room(p) ? hipMemoryTypeDevice : hipMemoryTypeUnregistered;
    return hipSuccess;
}
hipError_t hipGetSymbolAddress(void **, const void *) { return hipErrorInvalidSymbol; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { *s = reinterpret_cast<hipStream_t>(std::malloc(1)); return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t s) { ++waits; std::free(s); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamGetDevice(hipStream_t, hipDevice_t *d) { *d = 0; return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *s) { *s = hipStreamCaptureStatusNone; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { *e = reinterpret_cast<hipEvent_t>(std::malloc(1)); return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t e) { std::free(e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }

// ---- what the tests set and read
void fake_capacity(size_t n) { capacity = n; }
size_t fake_held() { std::lock_guard<std::mutex> lk(mu); return plain + pool_reserved(); }
size_t fake_pool_kept() { std::lock_guard<std::mutex> lk(mu); return only ? only->reserved - only->used : 0; }
size_t fake_pinned() {
    std::lock_guard<std::mutex> lk(mu);
    size_t n = 0;
    for (auto &h : host) n += h.second.n;
    return n;
}
size_t fake_peak(int reset) { const size_t v = peak; if (reset) peak = plain + pool_reserved(); return v; }
int fake_octants_together() { return octants_together; }
// the n-th allocation from now on fails; returns how many are left of that
long fake_fail_new(long n) { const long left = fail_at; fail_at = n; return left; }
long fake_waits() { return waits; }
int fake_upload_on(const merf_scene_desc *d, merf_scene_t *out) { return merf::scene_upload_on(d, reinterpret_cast<hipStream_t>(8), out); }
static merf::SceneImage image;
static char *image_bytes = nullptr;
int fake_image(merf_scene_t s) {
    const size_t n = merf_scene_bytes(s);
    image_bytes = static_cast<char *>(std::malloc(n));
    return merf::scene_image_on(s, image_bytes, n, reinterpret_cast<hipStream_t>(8), &image);
}
int fake_restore(merf_scene_t *out) {
    return merf::scene_from_image_on(image, image_bytes, reinterpret_cast<hipStream_t>(8), out);
}
void fake_release_unused() { merf::release_unused(); }
int fake_release_on(merf_scene_t s) { return merf::scene_release_on(s, reinterpret_cast<hipStream_t>(8)); }

}  // extern "C"

namespace merf {

hipError_t launch_render(const DevScene &, const RenderBatch &, hipStream_t) { return hipSuccess; }
hipError_t launch_dequant(const uint8_t *, int64_t, float, float, int, void *, hipStream_t) { return hipSuccess; }
hipError_t launch_maxpool(const uint8_t *, int, const int32_t *, int, uint8_t *const *, hipStream_t) { return hipSuccess; }
hipError_t launch_tile_order(const DevScene &, const RenderBatch &, uint8_t *, uint32_t *, int32_t *, hipStream_t) { return hipSuccess; }
hipError_t launch_pack_bricks(const uint8_t *, const int32_t *, const int32_t *, int, int, uint8_t *, hipStream_t) { return hipSuccess; }
hipError_t launch_distance_grid(const OccLevels &, uint8_t *, uint8_t *, uint8_t *, hipStream_t) { return hipSuccess; }
hipError_t launch_mlp_fragments(const float *, uint32_t *, hipStream_t) { return hipSuccess; }
hipError_t launch_identity_order(int32_t *, int, hipStream_t) { return hipSuccess; }
hipError_t launch_octant_extents(const OccLevels &lv, bool together, uint8_t *scratch, uint8_t *, hipStream_t) {
    octants_together = together;
    return room(scratch) >= octant_scratch_bytes(lv.res[lv.n - 1], together) ? hipSuccess : hipErrorInvalidValue;
}

}  // namespace merf

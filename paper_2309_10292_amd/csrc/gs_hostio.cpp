// Reading device fields to host FP64 arrays (gs_read, gs_batch_read).
//
// What bounds a large read: the copy over PCIe (57 GB/s into pinned memory, 18 GB/s
// into pageable memory) and the first touch of the caller's arrays, which the kernel
// hands out page by page. One thread that copies a field into a fresh pageable buffer
// and then widens it takes 48 ms for both FP32 fields of 256^3 (FP64 26, BF16 30). Here the fields go
// in slices through a ring of pinned buffers that the handle keeps, and a few threads
// widen the slices that have arrived into the caller's arrays while the next ones are
// copied: 5.9 ms (FP64 7.8, BF16 4.8), of which the copy over PCIe is 2.4.
#include "../../include/gs.h"
#include "gs_internal.hpp"

#include <sched.h>
#include <string.h>

#include <algorithm>
#include <atomic>
#include <exception>
#include <memory>
#include <new>
#include <thread>
#include <vector>

namespace gsapi {

namespace {

float from_bf16(uint16_t b)
{
    const uint32_t w = (uint32_t)b << 16;
    float f;
    memcpy(&f, &w, 4);
    return f;
}

// IEEE half, with integer operations and normal FP32 operands alone, so that the
// calling thread's treatment of denormals does not matter: a normal half is its bits in
// place with the exponent rebiased by 127 - 15, a subnormal one its mantissa times 2^-24,
// and the largest exponent (infinities, NaN) stays the largest.
float from_f16(uint16_t b)
{
    const uint32_t m = b & 0x3ffu, e = b & 0x7c00u;
    const float small = (float)(int32_t)m * 0x1p-24f;
    uint32_t w;
    memcpy(&w, &small, 4);
    w = e ? ((uint32_t)(b & 0x7fffu) << 13) + (e == 0x7c00u ? 224u << 23 : 112u << 23) : w;
    w |= (uint32_t)(b & 0x8000u) << 16;
    float f;
    memcpy(&f, &w, 4);
    return f;
}

// n stored values of field f (0 = u, 1 = v) as FP64.
void widen(int32_t storage, int field, const void *src, double *__restrict__ dst, size_t n)
{
    if (storage == GS_F64) {
        memcpy(dst, src, n * 8);
    } else if (storage == GS_F32) {
        const float *x = (const float *)src;
        for (size_t i = 0; i < n; ++i) dst[i] = x[i];
    } else if (storage == GS_BF16 || (storage == GS_BF16C && field == 1)) {
        const uint16_t *x = (const uint16_t *)src;
        for (size_t i = 0; i < n; ++i) dst[i] = from_bf16(x[i]);
    } else if (storage == GS_BF16C) {
        const uint16_t *x = (const uint16_t *)src;
        for (size_t i = 0; i < n; ++i) dst[i] = 1.0 - (double)from_bf16(x[i]);
    } else {
        const uint16_t *x = (const uint16_t *)src;
        for (size_t i = 0; i < n; ++i) dst[i] = from_f16(x[i]);
    }
}

// Memory that the runtime does not know: copies into it are staged.
bool pageable(const void *p)
{
    hipPointerAttribute_t a;
    memset(&a, 0, sizeof a);
    if (hipPointerGetAttributes(&a, p) != hipSuccess) {
        (void)hipGetLastError();
        return true;
    }
    return a.type == hipMemoryTypeUnregistered;
}

// Allocations and frees are refused while any thread captures a graph in the global
// mode, and end that capture; in the relaxed mode they are not.
struct Relaxed {
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    Relaxed() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
    ~Relaxed() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
};

constexpr size_t k_slot = (size_t)2 << 20;   // bytes of a ring slot
constexpr size_t k_part = (size_t)256 << 10; // bytes a thread widens at a time
constexpr int k_parts = (int)(k_slot / k_part);
constexpr int k_threads = 8;
constexpr size_t k_min = 448 << 10;          // values of a field from which the ring is used
// Rings that handles keep between reads, in all (of 8 MB each, which cannot be paged
// out); a handle beyond that makes one for each read (0.7 ms) and gives it back.
constexpr int k_kept = 16;
std::atomic<int> g_rings{0}; // rings there are

// One field in a plain copy.
gs_status read_plain(const void *dev, int32_t storage, size_t n, double *host, hipStream_t st, int field)
{
    std::unique_ptr<unsigned char[]> tmp; // (not cleared)
    void *to = host;
    if (storage != GS_F64) {
        tmp.reset(new (std::nothrow) unsigned char[n * storage_bytes(storage)]);
        if (!tmp) return fail(GS_ERR_INVALID_ARG, "out of host memory");
        to = tmp.get();
    }
    hipError_t e = hipMemcpyAsync(to, dev, n * storage_bytes(storage), hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) return hip_fail(e, "device-to-host copy");
    if (storage != GS_F64) widen(storage, field, to, host, n);
    return GS_OK;
}

} // namespace

// The ring, made at the first large read (or, unless kept, at each). False where it cannot serve: no memory, or
// a stream of another device than the current one or the ring's.
bool ReadStage::prepare(hipStream_t st)
{
    int now = -1, of_stream = -1;
    if (hipGetDevice(&now) != hipSuccess || (st && hipStreamGetDevice(st, &of_stream) != hipSuccess)) {
        (void)hipGetLastError();
        return false;
    }
    if (st && of_stream != now) return false;
    if (ring) return device == now;
    Relaxed relaxed;
    void *p = nullptr;
    if (hipHostMalloc(&p, k_slot * SLOTS, hipHostMallocDefault) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    for (int i = 0; i < SLOTS; ++i)
        if (hipEventCreateWithFlags(&arrived[i], hipEventDisableTiming) != hipSuccess) {
            (void)hipGetLastError();
            while (i > 0) (void)hipEventDestroy(arrived[--i]);
            (void)hipHostFree(p);
            return false;
        }
    ring = static_cast<unsigned char *>(p);
    device = now;
    kept = g_rings.fetch_add(1) < k_kept;
    return true;
}

void ReadStage::release()
{
    if (!ring) return;
    Relaxed relaxed;
    for (hipEvent_t e : arrived) (void)hipEventDestroy(e);
    (void)hipHostFree(ring);
    ring = nullptr;
    g_rings.fetch_sub(1);
}

gs_status read_fields(ReadStage &stage, const void *const dev[2], int32_t storage, size_t n, double *const host[2],
                      hipStream_t st)
{
    if (host[0] && host[1]) {
        const uintptr_t u = (uintptr_t)host[0], v = (uintptr_t)host[1];
        if ((u < v ? v - u : u - v) < n * sizeof(double)) { // overlapping arrays: all of u, then all of v
            double *const one[2] = {host[0], nullptr}, *const other[2] = {nullptr, host[1]};
            const gs_status r = read_fields(stage, dev, storage, n, one, st);
            return r != GS_OK ? r : read_fields(stage, dev, storage, n, other, st);
        }
    }
    const size_t es = storage_bytes(storage), bytes = n * es;
    const size_t chunks = (bytes + k_slot - 1) / k_slot; // of a field
    int field[2], nf = 0;
    for (int f = 0; f < 2; ++f)
        if (host[f]) field[nf++] = f;
    // Below 3.5 MB of FP64 a first read would lose more to making the ring (0.7 ms) than
    // it gains (72^3 FP64 0.36 -> 1.13 ms; 80^3 1.84 -> 1.19, FP32 1.35 -> 0.88), and
    // later ones gain little. FP64 into memory that the runtime knows needs no staging.
    std::unique_lock<std::mutex> lock(stage.mu, std::defer_lock);
    bool ringed = nf > 0 && n >= k_min;
    if (storage == GS_F64)
        for (int i = 0; i < nf; ++i) ringed = ringed && pageable(host[field[i]]);
    if (ringed) {
        lock.lock();
        ringed = stage.prepare(st);
    }
    if (!ringed) {
        for (int i = 0; i < nf; ++i) {
            const gs_status r = read_plain(dev[field[i]], storage, n, host[field[i]], st, field[i]);
            if (r != GS_OK) return r;
        }
        return GS_OK;
    }

    struct GiveBack {
        ReadStage &stage;
        ~GiveBack()
        {
            if (!stage.kept) stage.release();
        }
    } give_back{stage};
    constexpr int K = ReadStage::SLOTS;
    const size_t total = chunks * nf;
    auto chunk_bytes = [&](size_t c) { return std::min(k_slot, bytes - c % chunks * k_slot); };
    std::atomic<size_t> ready{0}, next{0}; // chunks that have arrived, the next part to widen
    std::atomic<size_t> widened[K];        // parts widened from each slot so far
    for (auto &w : widened) w = 0;
    std::atomic<bool> stop{false};
    // Parts are taken in order: part q is part q mod k_parts of chunk q / k_parts (a
    // chunk that is not full has empty parts at its end).
    auto part = [&](size_t q) {
        const size_t c = q / k_parts, off = q % k_parts * k_part, cb = chunk_bytes(c);
        if (off < cb)
            widen(storage, field[c / chunks], stage.ring + c % K * k_slot + off,
                  host[field[c / chunks]] + (c % chunks * k_slot + off) / es, std::min(k_part, cb - off) / es);
        widened[c % K].fetch_add(1, std::memory_order_release);
    };
    auto work = [&]() {
        for (size_t q; (q = next.fetch_add(1)) < total * k_parts; part(q))
            while (ready.load(std::memory_order_acquire) <= q / k_parts) {
                if (stop.load(std::memory_order_relaxed)) return;
                std::this_thread::yield();
            }
    };
    // This thread widens only what has arrived: it is the one that issues the copies.
    auto help = [&]() {
        size_t q = next.load();
        while (q < total * k_parts && q / k_parts < ready.load(std::memory_order_relaxed))
            if (next.compare_exchange_weak(q, q + 1)) {
                part(q);
                return true;
            }
        return false;
    };
    std::vector<std::thread> pool;
    hipError_t e = hipSuccess;
    size_t issued = 0;
    for (size_t c = 0; c < total && e == hipSuccess; ++c) {
        // keep the ring full: a chunk takes the slot of the one K before, once that is widened
        for (; issued < total && issued < c + K && e == hipSuccess; ++issued) {
            std::atomic<size_t> &w = widened[issued % K];
            const size_t before = issued / K * k_parts;
            if (issued > c && w.load(std::memory_order_acquire) < before) break;
            while (w.load(std::memory_order_acquire) < before)
                if (!help()) std::this_thread::yield();
            e = hipMemcpyAsync(stage.ring + issued % K * k_slot,
                               static_cast<const char *>(dev[field[issued / chunks]]) + issued % chunks * k_slot,
                               chunk_bytes(issued), hipMemcpyDeviceToHost, st);
            if (e == hipSuccess) e = hipEventRecord(stage.arrived[issued % K], st);
        }
        if (e == hipSuccess) e = hipEventSynchronize(stage.arrived[c % K]);
        if (e != hipSuccess) break;
        ready.store(c + 1, std::memory_order_release);
        if (c == 0) { // the stream has reached the read: nobody spins on the work before it
            cpu_set_t cpus;
            const int usable = sched_getaffinity(0, sizeof cpus, &cpus) == 0 ? CPU_COUNT(&cpus) : 1;
            try {
                pool.reserve(k_threads);
                for (int i = 0; i < std::min(k_threads, usable - 1); ++i) pool.emplace_back(work);
            } catch (const std::exception &) { // fewer threads, or none
            }
        }
    }
    if (e != hipSuccess) stop = true;
    else while (help()) {}
    for (auto &t : pool) t.join();
    if (e != hipSuccess) {
        (void)hipStreamSynchronize(st); // no copy into the ring is left behind
        return hip_fail(e, "device-to-host copy");
    }
    return GS_OK;
}

} // namespace gsapi

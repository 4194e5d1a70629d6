// fb_transfer.cpp -- pinned host memory that the runtime's transfers go
// through, and the read-back of device ranges into the caller's arrays.
#include "fb_runtime_internal.h"

#include <algorithm>
#include <atomic>
#include <cstring>
#include <exception>
#include <mutex>
#include <new>
#include <thread>
#include <vector>

namespace fb {
namespace rt {

namespace {

// Blocks given back, by device and size, for the next taker: allocating pinned
// memory takes longer than a small call's whole transfer.  At most kKeep of
// each size and device are kept, the others freed.
constexpr int kDevices = 64, kKeep = 16;
std::mutex g_mu;
std::vector<HostBlock> g_free[kDevices][2];

int size_class(size_t bytes) { return bytes <= kHostPage ? 0 : 1; }

void destroy(HostBlock &b)
{
    if (b.stream)
        (void)hipStreamDestroy(b.stream);
    if (b.p)
        (void)hipHostFree(b.p);
    b = HostBlock();
}

}  // namespace

fb_status take_block(size_t bytes, HostBlock &out)
{
    int dev = 0;
    FB_HIP(hipGetDevice(&dev));
    const int c = size_class(bytes);
    if (dev >= 0 && dev < kDevices) {
        std::lock_guard<std::mutex> lk(g_mu);
        std::vector<HostBlock> &v = g_free[dev][c];
        if (!v.empty()) {
            out = v.back();
            v.pop_back();
            return FB_OK;
        }
    }
    HostBlock b;
    b.device = dev;
    b.bytes = c ? kHostBlock : kHostPage;
    FB_HIP(hipHostMalloc((void **)&b.p, b.bytes, hipHostMallocPortable));
    out = b;
    return FB_OK;
}

void give_block(HostBlock &b)
{
    if (!b.p)
        return;
    const int c = size_class(b.bytes);
    if (b.device >= 0 && b.device < kDevices) {
        std::lock_guard<std::mutex> lk(g_mu);
        std::vector<HostBlock> &v = g_free[b.device][c];
        if ((int)v.size() < kKeep) {
            try {
                v.push_back(b);
                b = HostBlock();
                return;
            } catch (const std::bad_alloc &) {
            }
        }
    }
    destroy(b);
}

namespace {

// The chunks of a read-back: megabytes of one part after another.
struct Chunks {
    const HostPart *parts;
    int n;

    static size_t of(const HostPart &p) { return p.to ? (p.bytes + kHostBlock - 1) / kHostBlock : 0; }
    size_t count() const
    {
        size_t c = 0;
        for (int i = 0; i < n; ++i)
            c += of(parts[i]);
        return c;
    }
    HostPart at(size_t k) const
    {
        int i = 0;
        for (; k >= of(parts[i]); ++i)
            k -= of(parts[i]);
        const HostPart &p = parts[i];
        const size_t off = k * kHostBlock;
        return HostPart{static_cast<char *>(p.to) + off, static_cast<const char *>(p.from) + off,
                        std::min(kHostBlock, p.bytes - off)};
    }
};

// One worker's share of the chunks: each through this worker's own block and
// stream, so while one copies out of its block another's transfer runs.
hipError_t drain(const Chunks &chunks, const size_t count, std::atomic<size_t> &next, HostBlock &b)
{
    if (!b.stream) {
        const hipError_t e = hipStreamCreateWithFlags(&b.stream, hipStreamNonBlocking);
        if (e != hipSuccess)
            return e;
    }
    for (size_t k; (k = next.fetch_add(1)) < count;) {
        const HostPart p = chunks.at(k);
        hipError_t e = hipMemcpyAsync(b.p, p.from, p.bytes, hipMemcpyDeviceToHost, b.stream);
        if (e == hipSuccess)
            e = hipStreamSynchronize(b.stream);
        if (e != hipSuccess)
            return e;
        std::memcpy(p.to, b.p, p.bytes);
    }
    return hipSuccess;
}

bool is_pinned(const void *p)
{
    hipPointerAttribute_t a;
    if (hipPointerGetAttributes(&a, p) != hipSuccess) {
        (void)hipGetLastError();   // ordinary memory is reported as an error
        return false;
    }
    return a.type == hipMemoryTypeHost;
}

// All chunks into the host arrays by several workers, on the current device.
fb_status drain_all(const Chunks &chunks)
{
    const size_t count = chunks.count();
    if (count == 0)
        return FB_OK;
    HostBlock own;
    const fb_status st = take_block(kHostBlock, own);
    if (st != FB_OK)
        return st;
    std::atomic<size_t> next{0};
    std::atomic<int> failed{(int)hipSuccess};
    std::thread threads[kReadWorkers - 1];
    for (int k = 0; k < kReadWorkers - 1 && (size_t)k + 1 < count; ++k) {
        try {
            threads[k] = std::thread([&, dev = own.device] {
                HostBlock b;
                hipError_t e = hipSetDevice(dev);
                if (e == hipSuccess && take_block(kHostBlock, b) == FB_OK) {
                    e = drain(chunks, count, next, b);
                    give_block(b);
                }   // without a block the other workers take all chunks
                if (e != hipSuccess)
                    failed = (int)e;
            });
        } catch (const std::exception &) {
            break;   // no thread, or no memory for one: those that there are take all chunks
        }
    }
    hipError_t err = drain(chunks, count, next, own);
    for (std::thread &t : threads)
        if (t.joinable())
            t.join();
    if (err == hipSuccess)
        err = (hipError_t)failed.load();
    give_block(own);
    return err == hipSuccess ? FB_OK : hip_fail(err, "read-back");
}

}  // namespace

// The caller's arrays are ordinary memory, often fresh: a copy straight into
// them is staged and copied out by one thread of the runtime, page faults
// included, one array after another.  Four workers, each with a block and a
// stream, a megabyte at a time: 131072 x 3 bodies (21.5 MB) 1290 -> 590 us
// (two workers 820, half megabytes 590, quarters 700, six workers with halves
// 540), 16384 x 6 (5 MB) 200.  What fits one block is a single transfer.
fb_status read_to_host(const HostPart *parts, int n, hipStream_t s, int device)
{
    if (n > kMostParts)
        return fail(FB_E_INVAL, "too many parts");
    size_t total = 0;
    const char *lo = nullptr, *hi = nullptr;
    for (int i = 0; i < n; ++i) {
        if (!parts[i].to || !parts[i].bytes)
            continue;
        const char *f = static_cast<const char *>(parts[i].from);
        lo = lo ? std::min(lo, f) : f;
        hi = hi ? std::max(hi, f + parts[i].bytes) : f + parts[i].bytes;
        total += parts[i].bytes;
    }
    if (total == 0) {
        FB_HIP(hipStreamSynchronize(s));
        return FB_OK;
    }
    if ((size_t)(hi - lo) <= kHostBlock) {
        HostBlock own;
        const fb_status st = take_block(kHostBlock, own);
        if (st != FB_OK)
            return st;
        hipError_t e = hipMemcpyAsync(own.p, lo, (size_t)(hi - lo), hipMemcpyDeviceToHost, s);
        if (e == hipSuccess)
            e = hipStreamSynchronize(s);
        if (e == hipSuccess)
            for (int i = 0; i < n; ++i)
                if (parts[i].to && parts[i].bytes)
                    std::memcpy(parts[i].to, own.p + (static_cast<const char *>(parts[i].from) - lo), parts[i].bytes);
        give_block(own);
        return e == hipSuccess ? FB_OK : hip_fail(e, "read-back");
    }
    HostPart rest[kMostParts];
    hipError_t err = hipSuccess;
    for (int i = 0; i < n; ++i) {
        rest[i] = parts[i];
        if (err == hipSuccess && parts[i].to && parts[i].bytes && is_pinned(parts[i].to)) {   // no second copy needed
            err = hipMemcpyAsync(parts[i].to, parts[i].from, parts[i].bytes, hipMemcpyDeviceToHost, s);
            rest[i].to = nullptr;
        }
    }
    // the workers copy on streams of their own; and no copy of s is left
    // behind by an error
    const hipError_t es = hipStreamSynchronize(s);
    FB_HIP(err);
    FB_HIP(es);
    int current = device;
    FB_HIP(hipGetDevice(&current));
    if (current == device)
        return drain_all(Chunks{rest, n});
    FB_HIP(hipSetDevice(device));   // the streams belong where the data is
    const fb_status st = drain_all(Chunks{rest, n});
    FB_HIP(hipSetDevice(current));
    return st;
}

}  // namespace rt
}  // namespace fb

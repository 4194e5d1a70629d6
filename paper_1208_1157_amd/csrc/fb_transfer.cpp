// fb_transfer.cpp -- pinned host memory that the runtime's transfers go
// through, and the read-back of device ranges into the caller's arrays.
#include "fb_runtime_internal.h"

#include <algorithm>
#include <atomic>
#include <cstring>
#include <mutex>
#include <system_error>
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

// Chunk of a read-back.
struct Piece {
    char *to;
    const char *from;
    size_t bytes;
};

// One worker's share of the pieces: each through this worker's own block and
// stream, so while one copies out of its block another's transfer runs.
hipError_t drain(const std::vector<Piece> &pieces, std::atomic<size_t> &next, HostBlock &b)
{
    if (!b.stream) {
        const hipError_t e = hipStreamCreateWithFlags(&b.stream, hipStreamNonBlocking);
        if (e != hipSuccess)
            return e;
    }
    for (size_t i; (i = next.fetch_add(1)) < pieces.size();) {
        const Piece &p = pieces[i];
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

}  // namespace

// The caller's arrays are ordinary memory, often fresh: a copy straight into
// them is staged and copied out by one thread of the runtime, page faults
// included, one array after another.  Four workers, each with a block and a
// stream, a megabyte at a time: 131072 x 3 bodies (21.5 MB) 1290 -> 590 us
// (two workers 820, half megabytes 590, quarters 700, six workers with halves
// 540), 16384 x 6 (5 MB) 200.  What fits one block is a single transfer.
fb_status read_to_host(const HostPart *parts, int n, hipStream_t s)
{
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
    HostBlock own;
    fb_status st = take_block(kHostBlock, own);
    if (st != FB_OK)
        return st;
    if ((size_t)(hi - lo) <= own.bytes) {
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
    hipError_t err = hipSuccess;
    std::vector<Piece> pieces;
    for (int i = 0; i < n && err == hipSuccess; ++i) {
        char *to = static_cast<char *>(parts[i].to);
        const char *from = static_cast<const char *>(parts[i].from);
        if (!to || !parts[i].bytes)
            continue;
        if (is_pinned(to)) {   // no second copy needed
            err = hipMemcpyAsync(to, from, parts[i].bytes, hipMemcpyDeviceToHost, s);
            continue;
        }
        for (size_t at = 0; at < parts[i].bytes; at += kHostBlock)
            pieces.push_back({to + at, from + at, std::min(kHostBlock, parts[i].bytes - at)});
    }
    std::atomic<size_t> next{0};
    std::atomic<int> failed{(int)hipSuccess};
    if (err == hipSuccess)   // the workers copy on streams of their own
        err = hipStreamSynchronize(s);
    const int workers = (int)std::min<size_t>(pieces.size(), kReadWorkers);
    std::vector<std::thread> threads;
    if (err == hipSuccess) {
        for (int k = 1; k < workers; ++k) {
            try {
                threads.emplace_back([&, dev = own.device] {
                    HostBlock b;
                    hipError_t e = hipSetDevice(dev);
                    if (e == hipSuccess && take_block(kHostBlock, b) == FB_OK) {
                        e = drain(pieces, next, b);
                        give_block(b);
                    }   // without a block the other workers take all pieces
                    if (e != hipSuccess)
                        failed = (int)e;
                });
            } catch (const std::system_error &) {
                break;   // no more threads: those that there are take all pieces
            }
        }
        err = drain(pieces, next, own);
        for (std::thread &t : threads)
            t.join();
        if (err == hipSuccess)
            err = (hipError_t)failed.load();
    }
    give_block(own);
    return err == hipSuccess ? FB_OK : hip_fail(err, "read-back");
}

}  // namespace rt
}  // namespace fb

// Read-back of device ranges (fb_transfer.cpp) on the CPU: the HIP calls it
// makes are stood in for here, "device" memory being ordinary memory, and
// operator new fails on demand.  Prints one "name value" line per check.
#include "fb_runtime_internal.h"

#include <algorithm>
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>
#include <set>
#include <vector>

namespace {
std::atomic<int> news_left{-1};   // >= 0: allocations until one fails
std::atomic<int> copies{0}, fail_copy{-1};
std::atomic<int> wrong_device{0};
std::atomic<int> pending{0};      // copies on the caller's stream that nobody has waited for
thread_local int device = 0;
int want_device = 0;
hipStream_t const kCaller = reinterpret_cast<hipStream_t>(0x10);
std::set<const void *> pinned;
}  // namespace

void *operator new(std::size_t n)
{
    int left = news_left.load();
    while (left >= 0 && !news_left.compare_exchange_weak(left, left - 1)) {
    }
    if (left == 0)
        throw std::bad_alloc();
    if (void *p = std::malloc(n ? n : 1))
        return p;
    throw std::bad_alloc();
}
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, std::size_t) noexcept { std::free(p); }

extern "C" {
hipError_t hipGetDevice(int *d) { *d = device; return hipSuccess; }
hipError_t hipSetDevice(int d) { device = d; return hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { *p = std::malloc(n); return *p ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipHostFree(void *p) { std::free(p); return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned)
{
    wrong_device += device != want_device;
    *s = reinterpret_cast<hipStream_t>(0x1000);
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s)
{
    if (s == kCaller)
        pending = 0;
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *to, const void *from, size_t n, hipMemcpyKind, hipStream_t s)
{
    if (copies++ == fail_copy.load())
        return hipErrorUnknown;
    if (s == kCaller)
        ++pending;
    std::memcpy(to, from, n);
    return hipSuccess;
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t *a, const void *p)
{
    std::memset(a, 0, sizeof *a);
    a->type = pinned.count(p) ? hipMemoryTypeHost : hipMemoryTypeUnregistered;
    return hipSuccess;
}
hipError_t hipGetLastError(void) { return hipSuccess; }
}

namespace fb {
namespace rt {
fb_status fail(fb_status code, const char *, ...) { return code; }
fb_status hip_fail(hipError_t, const char *) { return FB_E_DEVICE; }
}  // namespace rt
}  // namespace fb

int main()
{
    using namespace fb::rt;
    const size_t MB = 1 << 20, sizes[5] = {3 * MB + 17, MB, 5 * MB - 8, 40, 2 * MB + 1};
    std::vector<char> from(12 * MB + 64), want(from.size());
    for (size_t i = 0; i < from.size(); ++i)
        from[i] = want[i] = (char)(i * 2654435761u >> 13);
    std::vector<char> to(from.size());
    HostPart parts[5];
    size_t at = 0;
    for (int i = 0; i < 5; ++i) {
        parts[i] = HostPart{i == 1 ? nullptr : to.data() + at, from.data() + at, sizes[i]};
        at += sizes[i];
    }
    auto right = [&](bool whole) {
        for (int i = 0; i < 5; ++i) {
            const size_t o = static_cast<const char *>(parts[i].from) - from.data();
            const bool have = std::memcmp(to.data() + o, want.data() + o, sizes[i]) == 0;
            if (have != (parts[i].to && whole))
                return false;
        }
        return true;
    };
    auto read = [&](int dev) {
        std::fill(to.begin(), to.end(), 0);
        copies = 0;
        return read_to_host(parts, 5, kCaller, dev);
    };
    std::printf("plain %d\n", read(0) == FB_OK && right(true));
    pinned.insert(parts[2].to);
    std::printf("pinned %d\n", read(0) == FB_OK && right(true) && pending == 0);

    // the streams of the copies are made on the ensemble's device
    want_device = 1;
    std::printf("device %d\n", read(1) == FB_OK && right(true) && wrong_device == 0 && device == 0);
    want_device = 0;

    // a failed copy is reported, with nothing left under way
    bool ok = true;
    for (int k = 0; k < 8; ++k) {
        fail_copy = k;
        ok = ok && read(0) == FB_E_DEVICE && pending == 0;
    }
    fail_copy = -1;
    std::printf("errors %d\n", ok);

    // an allocation that fails, whichever it is, costs a worker at most
    ok = true;
    for (int k = 0; k < 24; ++k) {
        news_left = k;
        fb_status st = FB_E_STATE;
        try {
            st = read(0);
        } catch (...) {
            ok = false;
        }
        news_left = -1;
        ok = ok && st == FB_OK && right(true);
    }
    std::printf("no_memory %d\n", ok);
    return 0;
}

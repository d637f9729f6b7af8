// Reads of large device arrays through pinned staging buffers (btrt_transfer.h).
//
// The runtime copies to pageable memory through one staging buffer and one thread: 134 MB into
// freshly allocated pages took 15.2 ms, of which the transfer itself is 2.4 (57 GB/s from pinned memory)
// and the rest one thread's copy and page faults. Here up to kThreads threads each move every kThreads-th
// chunk through two pinned buffers of their own, so transfers, copies and page faults overlap. A kernel
// moves the words into the (device-visible) pinned buffer: the first copy-engine transfer of a new stream
// took 20 ms. 134 MB into fresh pages now take 6.5 ms. (Uploads stay with the runtime, which reads
// pageable memory faster than a kernel reads a pinned buffer.)

#include "btrt_transfer.h"

#include <algorithm>
#include <cstdint>
#include <cstring>
#include <mutex>
#include <thread>

namespace btrth {
namespace {

// n16 16-byte words, and one 8-byte word more where tail is set.
__global__ __launch_bounds__(256) void copy_words_kernel(ulonglong2* __restrict__ dst, const ulonglong2* __restrict__ src,
                                                         unsigned n16, int tail)
{
    const unsigned k = blockIdx.x * 256u + threadIdx.x;
    if (k < n16) dst[k] = src[k];
    if (tail && k == 0)
        reinterpret_cast<unsigned long long*>(dst)[2 * static_cast<size_t>(n16)] =
            reinterpret_cast<const unsigned long long*>(src)[2 * static_cast<size_t>(n16)];
}

// bytes: a multiple of 8, at most a chunk; both pointers 16-byte aligned.
hipError_t copy_words(void* dst, const void* src, size_t bytes, hipStream_t s)
{
    const unsigned n16 = static_cast<unsigned>(bytes / 16);
    hipLaunchKernelGGL(copy_words_kernel, dim3(std::max(1u, (n16 + 255) / 256)), dim3(256), 0, s,
                       static_cast<ulonglong2*>(dst), static_cast<const ulonglong2*>(src), n16, bytes % 16 ? 1 : 0);
    return hipGetLastError();
}

constexpr size_t kChunk = size_t(1) << 19;       // bytes per buffer
constexpr int kThreads = 8;
constexpr size_t kBuffers = 2 * kChunk;          // a thread's pinned buffers, one allocation
constexpr size_t kPerThread = size_t(1) << 20;   // at least this much work for a thread

// Buffers for at most kThreads threads are kept idle, while anything that copies is alive; concurrent
// copies take more, which go back when they end. One allocation per thread: 1 MB of pinned memory took 15 us,
// 2 MB and more 300 to 600 in a single one (all eight threads' together made the first read of a new
// 900 x 700 handle 1.2 ms instead of 0.4).
std::mutex g_lock;
void* g_idle[kThreads];
int g_idles = 0;
int g_users = 0;

// One thread's share of a copy: chunks first, first + step, ... through two buffers.
hipError_t copy_share(char* host, const char* dev, size_t bytes, int first, int step, char* pinned, int device,
                      hipStream_t s)
{
    hipError_t e = hipSetDevice(device);
    hipEvent_t ev[2] = {nullptr, nullptr};
    size_t at[2] = {0, 0}, len[2] = {0, 0};  // chunk in flight in each buffer (len 0: none)
    for (int b = 0; b < 2 && e == hipSuccess; ++b) e = hipEventCreateWithFlags(&ev[b], hipEventDisableTiming);
    // Waits for buffer b and empties it.
    auto finish = [&](int b) {
        if (len[b] == 0) return;
        const hipError_t w = hipEventSynchronize(ev[b]);
        if (e == hipSuccess) e = w;
        if (e == hipSuccess) std::memcpy(host + at[b], pinned + b * kChunk, len[b]);
        len[b] = 0;
    };
    int b = 0;
    for (size_t off = static_cast<size_t>(first) * kChunk; off < bytes && e == hipSuccess;
         off += static_cast<size_t>(step) * kChunk, b ^= 1) {
        finish(b);
        if (e != hipSuccess) break;
        const size_t m = std::min(kChunk, bytes - off);
        e = copy_words(pinned + b * kChunk, dev + off, m, s);
        if (e == hipSuccess) e = hipEventRecord(ev[b], s);
        if (e == hipSuccess) {
            at[b] = off;
            len[b] = m;
        }
    }
    finish(b);
    finish(b ^ 1);
    for (hipEvent_t x : ev)
        if (x) (void)hipEventDestroy(x);
    return e;
}

}  // namespace

void* staging_get(size_t* bytes)
{
    *bytes = kBuffers;
    {
        std::lock_guard<std::mutex> guard(g_lock);
        if (g_idles > 0) return g_idle[--g_idles];
    }
    void* p = nullptr;
    if (hipHostMalloc(&p, kBuffers, hipHostMallocPortable) != hipSuccess) {
        (void)hipGetLastError();
        return nullptr;
    }
    return p;
}

void staging_put(void* p)
{
    if (!p) return;
    {
        std::lock_guard<std::mutex> guard(g_lock);
        if (g_idles < kThreads && g_users > 0) {
            g_idle[g_idles++] = p;
            return;
        }
    }
    (void)hipHostFree(p);
}

void staging_retain()
{
    std::lock_guard<std::mutex> guard(g_lock);
    ++g_users;
}

void staging_release()
{
    void* p[kThreads];
    int n = 0;
    {
        std::lock_guard<std::mutex> guard(g_lock);
        if (--g_users == 0) {
            n = g_idles;
            std::copy(g_idle, g_idle + n, p);
            g_idles = 0;
        }
    }
    for (int i = 0; i < n; ++i) (void)hipHostFree(p[i]);
}

hipError_t copy_to_host(void* dst, const void* src, size_t bytes, int device, hipStream_t s)
{
    char* const host = static_cast<char*>(dst);
    const char* const dev = static_cast<const char*>(src);
    // Words the kernel could not move are left to the runtime's own path (64^2 FP64, the whole read: 33 us
    // by that, 19 by the kernel; 500^2 126 and 90 us).
    const bool words = bytes % 8 == 0 && reinterpret_cast<uintptr_t>(dev) % 16 == 0;
    // hipStreamPerThread names another stream in each thread, where nothing would order a share behind the
    // work on the caller's: those reads stay on the calling thread.
    const size_t threads = s == hipStreamPerThread ? 1 : kThreads;
    const int most = static_cast<int>(std::max<size_t>(1, std::min<size_t>(threads, bytes / kPerThread)));
    char* pinned[kThreads];
    int want = 0;
    size_t got = 0;
    while (words && want < most && (pinned[want] = static_cast<char*>(staging_get(&got))) != nullptr) ++want;
    if (want == 0) {
        const hipError_t e = hipMemcpyAsync(dst, src, bytes, hipMemcpyDeviceToHost, s);
        return e == hipSuccess ? hipStreamSynchronize(s) : e;
    }
    hipError_t err[kThreads] = {};
    std::thread pool[kThreads];
    int started = 1;  // the calling thread is the first
    // The shares are fixed by `want`; a share whose thread could not be started is done here.
    for (int t = 1; t < want; ++t) {
        try {
            pool[t] = std::thread([=, &err, &pinned] { err[t] = copy_share(host, dev, bytes, t, want, pinned[t], device, s); });
        } catch (...) {
            break;
        }
        ++started;
    }
    err[0] = copy_share(host, dev, bytes, 0, want, pinned[0], device, s);
    for (int t = started; t < want; ++t) err[t] = copy_share(host, dev, bytes, t, want, pinned[t], device, s);
    for (int t = 1; t < started; ++t) pool[t].join();
    hipError_t e = hipSuccess;
    for (int t = 0; t < want; ++t)
        if (e == hipSuccess) e = err[t];
    if (e != hipSuccess) (void)hipStreamSynchronize(s);  // nothing may still use the buffers
    for (int t = 0; t < want; ++t) staging_put(pinned[t]);
    return e;
}

}  // namespace btrth

// Shared host/device definitions for the SYK HIP library.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <memory>
#include <stdexcept>
#include <string>
#include <vector>

#include "../../include/syk.h"

namespace syk {

// Interleaved complex numbers, matching the caller's complex128 / complex64 buffers.
template <typename R>
struct alignas(2 * sizeof(R)) cplx {
    R re, im;
};
using c128 = cplx<double>;
using c64 = cplx<float>;

// Error carrying a status code across the internal layers; the C-ABI turns it
// into a return value and the thread-local message of syk_last_error().
struct Error : std::runtime_error {
    syk_status code;
    Error(syk_status c, const std::string& m) : std::runtime_error(m), code(c) {}
};

inline void hip_check(hipError_t e, const char* what, const char* file, int line)
{
    if (e != hipSuccess) {
        char buf[512];
        std::snprintf(buf, sizeof buf, "%s failed at %s:%d: %s", what, file, line, hipGetErrorString(e));
        throw Error(SYK_EHIP, buf);
    }
}
#define SYK_HIP(call) ::syk::hip_check((call), #call, __FILE__, __LINE__)

inline void require(bool ok, const std::string& msg)
{
    if (!ok) throw Error(SYK_EINVAL, msg);
}

inline size_t elem_bytes(syk_dtype d) { return d == SYK_C128 ? 16 : 8; }

// Device buffer owned by the library (workspaces, tables).
struct DevBuf {
    void* p = nullptr;
    size_t bytes = 0;
    DevBuf() = default;
    DevBuf(const DevBuf&) = delete;
    DevBuf& operator=(const DevBuf&) = delete;
    ~DevBuf() { release(); }
    void release()
    {
        if (p) {
            (void)hipDeviceSynchronize();   // work enqueued earlier may still read it
            (void)hipFree(p);
        }
        p = nullptr;
        bytes = 0;
    }
    void ensure(size_t n)
    {
        if (n <= bytes) return;
        release();
        hipError_t e = hipMalloc(&p, n);
        if (e != hipSuccess) {
            p = nullptr;
            throw Error(e == hipErrorOutOfMemory ? SYK_ENOMEM : SYK_EHIP,
                        std::string("hipMalloc of ") + std::to_string(n) + " bytes: " + hipGetErrorString(e));
        }
        bytes = n;
    }
    template <typename T>
    T* as() const { return static_cast<T*>(p); }
};

// A device table built on first use.  `ready` is set once the work that fills it
// has finished: after a launch or a wait that failed, the next use fills it again.
struct TableBuf : DevBuf {
    bool ready = false;
};

// Scratch that grows but never moves what it gave out, so that launches captured
// in a graph keep valid addresses: a buffer it has outgrown lives on with it.  Each
// is at least twice the one before (up to `most`), so the old ones together are
// no larger than the newest.
struct KeptBuf {
    std::vector<std::unique_ptr<DevBuf>> bufs;
    size_t bytes() const { return bufs.empty() ? 0 : bufs.back()->bytes; }
    void* get(size_t n, size_t most)
    {
        if (n > bytes()) {
            std::unique_ptr<DevBuf> b(new DevBuf());
            b->ensure(std::max(n, std::min(2 * bytes(), most)));
            bufs.push_back(std::move(b));
        }
        return bufs.empty() ? nullptr : bufs.back()->p;
    }
};

// Pinned host buffer owned by the library, read by the host after the stream
// that wrote it is synchronised.
struct PinnedBuf {
    void* p = nullptr;
    size_t bytes = 0;
    int asked = 0;
    PinnedBuf() = default;
    PinnedBuf(const PinnedBuf&) = delete;
    PinnedBuf& operator=(const PinnedBuf&) = delete;
    ~PinnedBuf() { release(); }
    void release()
    {
        if (p) {
            (void)hipDeviceSynchronize();   // work enqueued earlier may still write it
            (void)hipHostFree(p);
        }
        p = nullptr;
        bytes = 0;
    }
    void* get(size_t n)
    {
        if (n <= bytes) return p;
        release();
        n = n < 16384 ? 16384 : n;
        hipError_t e = hipHostMalloc(&p, n, hipHostMallocDefault);
        if (e != hipSuccess) {
            p = nullptr;
            throw Error(SYK_ENOMEM, std::string("hipHostMalloc of ") + std::to_string(n) + " bytes: " + hipGetErrorString(e));
        }
        bytes = n;
        return p;
    }
    // The buffer, or NULL for the first four requests it would have to grow for:
    // allocating it takes 70 us, a copy from device memory instead 9, and a handle
    // may be used only once or twice.
    void* get_if_used(size_t n) { return n > bytes && asked++ < 4 ? nullptr : get(n); }
};

}  // namespace syk

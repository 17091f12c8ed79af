// The HIP stub of tests/hoststub with a device of bounded memory: hipMalloc fails beyond
// hipmem::capacity() bytes, and a failure stays the thread's last error until
// hipGetLastError has returned it, also after later calls that succeed (as the ROCm 7
// runtime does).  Test infrastructure only.
#pragma once
#define hipMalloc hipMalloc_unbounded
#define hipFree hipFree_unbounded
#define hipGetLastError hipGetLastError_none
#include "../../hoststub/hip/hip_runtime.h"
#undef hipMalloc
#undef hipFree
#undef hipGetLastError
#include <map>

namespace hipmem {
inline size_t &capacity() { static size_t n = (size_t)1 << 40; return n; }
inline size_t &used() { static size_t n = 0; return n; }
inline size_t &peak() { static size_t n = 0; return n; }
inline long &failures() { static long n = 0; return n; }
inline hipError_t &last_error() { static hipError_t e = hipSuccess; return e; }
inline std::map<void *, size_t> &sizes() { static std::map<void *, size_t> m; return m; }
}  // namespace hipmem

inline hipError_t hipMalloc(void **p, size_t n) {
    if (hipmem::used() + n > hipmem::capacity()) {
        *p = nullptr;
        ++hipmem::failures();
        return hipmem::last_error() = hipErrorOutOfMemory;
    }
    const hipError_t e = hipMalloc_unbounded(p, n);
    if (e != hipSuccess) return hipmem::last_error() = e;
    hipmem::sizes()[*p] = n;
    hipmem::used() += n;
    if (hipmem::used() > hipmem::peak()) hipmem::peak() = hipmem::used();
    return hipSuccess;
}
inline hipError_t hipFree(void *p) {
    auto it = hipmem::sizes().find(p);
    if (it != hipmem::sizes().end()) {
        hipmem::used() -= it->second;
        hipmem::sizes().erase(it);
    }
    return hipFree_unbounded(p);
}
inline hipError_t hipGetLastError() {
    const hipError_t e = hipmem::last_error();
    hipmem::last_error() = hipSuccess;
    return e;
}

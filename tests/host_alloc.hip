// Host side of the library's allocation helpers, driven by test_host_alloc.py:
// compiled for the host alone, with a global operator new that can be made to
// fail and an allocator of this file's own in place of the device's.
#include <cstdlib>
#include <new>

#include "agal_internal.hpp"

static bool g_fail_new = false;
void *operator new(size_t n) {
    if (g_fail_new) throw std::bad_alloc();
    void *p = std::malloc(n ? n : 1);
    if (!p) throw std::bad_alloc();
    return p;
}
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, size_t) noexcept { std::free(p); }

namespace agal {
agal_status fail(agal_status s, const char *, ...) { return s; }
static size_t g_bytes = 0;
void *Allocator::alloc(size_t bytes, hipStream_t) const {
    g_bytes = bytes;
    return reinterpret_cast<void *>(uintptr_t(1) << 40);
}
}  // namespace agal

// n arrays of counts[i] doubles in one block: the status, the block's bytes and
// the arrays' offsets in it; -1 when an exception came out.
extern "C" __attribute__((visibility("default"))) int slab(int n, const size_t *counts, size_t *bytes, size_t *at) {
    static double *arrays[64];
    alignas(agal::Allocator) static char room[sizeof(agal::Allocator)];
    agal::Allocator *a = new (room) agal::Allocator();
    for (double *&p : arrays) p = nullptr;
    g_fail_new = true;
    int st;
    try {
        agal::Slab s;
        for (int i = 0; i < n; ++i) s.add(&arrays[i], counts[i]);
        void *base = nullptr;
        st = (int)s.get(*a, &base, nullptr);
    } catch (...) {
        st = -1;
    }
    g_fail_new = false;
    *bytes = agal::g_bytes;
    for (int i = 0; i < n && st == 0; ++i) at[i] = (size_t)((uintptr_t)arrays[i] - (uintptr_t(1) << 40));
    a->~Allocator();
    return st;
}

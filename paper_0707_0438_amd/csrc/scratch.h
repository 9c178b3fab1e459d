// Device memory that a context owns.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>

namespace nb {

// Goes with its owner (whose device is current then).
struct DevBuf {
    void* p = nullptr;
    size_t bytes = 0;
    DevBuf() = default;
    DevBuf(const DevBuf&) = delete;
    DevBuf& operator=(const DevBuf&) = delete;
    ~DevBuf() {
        if (p) (void)hipFree(p);
    }
};

// Grows b to `bytes` with memory from get(bytes), which returns NULL when
// there is none: then b stays as it is (other calls still need it) and the
// result is false.
template <class Get>
bool grow_or_keep(DevBuf& b, size_t bytes, Get get) {
    if (b.bytes >= bytes) return true;
    void* const p = get(bytes);
    if (!p) return false;
    if (b.p) (void)hipFree(b.p);
    b.p = p;
    b.bytes = bytes;
    return true;
}

}  // namespace nb

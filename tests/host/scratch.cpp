// Host-only check of optional scratch: a failed growth leaves the buffer.
#include <cstdio>

#include "scratch.h"

int main() {
    char mem[64];
    nb::DevBuf b;
    b.p = mem;
    b.bytes = sizeof mem;
    int asked = 0;
    auto none = [&](size_t) -> void* { return ++asked, nullptr; };
    const bool same = nb::grow_or_keep(b, 64, none), more = nb::grow_or_keep(b, 65, none);
    const bool ok = same && !more && asked == 1 && b.p == mem && b.bytes == sizeof mem;
    b.p = nullptr;   // not device memory
    return ok ? 0 : 1;
}

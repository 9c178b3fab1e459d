// Host-only check of the pair-symmetric launch shapes: for many set sizes,
// the pieces of every band cover each block's stretch, every two blocks meet
// exactly once, the rows fit in the bytes asked for, and offsets stay within
// int32.
#include <cstdio>
#include <vector>

#include "launch_shape.h"

int main() {
    int bad = 0;
    auto fail = [&](long long n, const char* what) {
        printf("n %lld: %s\n", n, what);
        ++bad;
    };
    std::vector<long long> sizes = {nb::kSymMin, nb::kSymMin + 1, 25600, 25601, 40000, 65535, 65536, 65537, 100003,
                                    131072, 262144, 262145, 1 << 20, (1 << 20) + 1, 1 << 24, nb::kSymMax - 7, nb::kSymMax};
    for (long long n : sizes)
        for (int tj : {64, 256})
            for (int q : {4, 7}) {
                const nb::SymShape s = nb::sym_shape(n, tj, q);
                const long long ring = (long long)s.nb * s.lb;
                if (s.lb != 1 << s.lbs || s.lb % nb::kSymGroup || ring < n || ring - n >= s.lb) fail(n, "blocks");
                if (s.lp <= 0 || s.lp % tj || (long long)s.lp * s.np < ((long long)s.nd << s.lbs)) fail(n, "pieces");
                if (s.dists != s.nb / 2 + 1 || s.nd < 1 || s.nd > s.dists) fail(n, "distances");
                const long long row = 8LL * q * nb::sym_stride(n);
                if (nb::sym_stride(n) < n || nb::sym_stride(n) % 4) fail(n, "stride");
                if ((long long)s.bytes != row * (s.nd + s.np)) fail(n, "bytes");
                if ((long long)s.bytes > nb::kSymBytes) fail(n, "limit");
                if (2 * ring + s.lp > 2147483647LL || (long long)s.np * s.nb > 2147483647LL) fail(n, "int32 range");
                if (s.nb > 4096) continue;
                // every unordered pair of blocks once, over all bands
                std::vector<char> met((size_t)s.nb * s.nb, 0);
                for (int d0 = 0; d0 < s.dists; d0 += s.nd) {
                    const int d1 = std::min(s.dists, d0 + s.nd);
                    const bool half = d1 == s.dists && s.nb % 2 == 0;
                    for (int A = 0; A < s.nb; ++A)
                        for (int d = d0; d < d1 - (half && A >= s.nb / 2 ? 1 : 0); ++d) {
                            const int B = (A + d) % s.nb;
                            ++met[(size_t)std::min(A, B) * s.nb + std::max(A, B)];
                        }
                }
                for (int A = 0; A < s.nb; ++A)
                    for (int B = A; B < s.nb; ++B)
                        if (met[(size_t)A * s.nb + B] != 1) {
                            fail(n, "pairs of blocks");
                            A = s.nb;
                            break;
                        }
            }
    return bad ? 1 : 0;
}

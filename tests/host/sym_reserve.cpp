// Host-only check of the pre-sizing of pair-symmetric scratch: what is asked
// for up to `most` particles holds the rows of every set of up to that many,
// in the j-tile that it is evaluated with, jerk or not.
#include <cstdio>

#include "launch_shape.h"

int main() {
    size_t need = 0;
    int bad = 0;
    for (long long n = nb::kSymMin; n <= (1 << 18); ++n) {
        for (int kind = 0; kind < 2; ++kind) {
            const int tj = nb::default_tile_kind(kind, 1, n, n).tile_j;
            need = std::max(need, nb::sym_shape(n, tj, kind == 1 ? 4 : 7).bytes);
        }
        const long long r = n % nb::kSymGroup;
        if (r > 1 && r < nb::kSymGroup - 1 && n % 128) continue;
        const size_t have = nb::sym_bytes_upto(n);
        if (have < need && bad++ < 10) printf("up to %lld: %zu bytes, %zu needed\n", n, have, need);
    }
    for (long long n = 1 << 18; n <= nb::kSymMax; n += 99991)
        for (int q : {4, 7})
            if (nb::sym_shape(n, 256, q).bytes > nb::sym_bytes_upto(n) && bad++ < 10) printf("%lld: beyond\n", n);
    return bad ? 1 : 0;
}

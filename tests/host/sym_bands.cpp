// Prints the pair-symmetric launch shape of each (bodies, kind) pair of the
// arguments in the default j-tile: bodies kind distances distances-a-band
// block-length blocks.
#include <cstdio>
#include <cstdlib>

#include "launch_shape.h"

int main(int argc, char** argv) {
    for (int k = 1; k + 1 < argc; k += 2) {
        const long long n = atoll(argv[k]);
        const int kind = atoi(argv[k + 1]);
        const int tj = nb::default_tile_kind(kind, 1, n, n).tile_j;
        const nb::SymShape s = nb::sym_shape(n, tj, kind == 1 ? 4 : 7);
        printf("%lld %d %d %d %d %d\n", n, kind, s.dists, s.nd, s.lb, s.nb);
    }
    return 0;
}

// Host-only check of the pre-sizing of split partials: what is asked for up
// to max_i i-particles against max_j j holds the partials of every call of no
// more of either, of each kind and precision, in its default shape.
#include <cmath>
#include <cstdio>
#include <random>

#include "launch_shape.h"

static nbody_tile shape(int kind, int prec, int64_t n, int64_t m) {
    nbody_tile t = nb::default_tile_kind(kind, prec, n, m);
    t.split = nb::choose_split(prec, n, m, t, kind);
    return t;
}

int main() {
    std::mt19937_64 g(5);
    auto size = [&](int64_t hi) { return (int64_t)exp(std::uniform_real_distribution<double>(0, log(hi + 0.99))(g)); };
    int bad = 0;
    for (int it = 0; it < 600; ++it) {
        const int64_t max_i = size(3000000), max_j = it % 2 ? max_i : size(3000000);
        int64_t have = 0;
        for (int kind = 0; kind < 3; ++kind)
            for (int prec = 0; prec < 2; ++prec)
                have = std::max(have, nb::part_rows_upto(prec, max_i, max_j, [&](int64_t n, int64_t m) {
                                    return nb::default_tile_kind(kind, prec, n, m);
                                }));
        for (int c = 0; c < 2000; ++c) {
            int64_t n = c % 8 ? size(max_i) : max_i, m = c % 3 ? size(max_j) : max_j;
            if (c % 5 == 4) n = m = std::min(n, m);
            for (int kind = 0; kind < 3; ++kind)
                for (int prec = 0; prec < 2; ++prec) {
                    const nbody_tile t = shape(kind, prec, n, m);
                    int nb, S, jc;
                    nb::split_plan(n, m, t.wg * t.ipt, t.tile_j, t.split, &nb, &S, &jc);
                    if (S > 1 && S * n > have && bad++ < 10)
                        printf("reserve %lld x %lld, call %lld x %lld kind %d prec %d: %lld rows, %lld reserved\n",
                               (long long)max_i, (long long)max_j, (long long)n, (long long)m, kind, prec,
                               (long long)(S * n), (long long)have);
                }
        }
    }
    printf("%d short\n", bad);
    return bad ? 1 : 0;
}

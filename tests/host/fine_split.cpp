// Host-only check of the finer split of mid-size DS evaluations: where five
// tiles a range set it, a range is five tiles, not six.
#include <cstdio>

#include "launch_shape.h"

int main() {
    int bad = 0;
    const long long cases[][2] = {{400, 262144}, {256, 524288}, {128, 700000}, {128, 1 << 20}, {12000, 12000},
                                  {1000, 131072}, {4096, 32768}, {10000, 10000}, {129, 600001}};
    for (const auto& c : cases) {
        const nbody_tile t = nb::default_tile(1, c[0], c[1]);
        int nb, S, jc;
        nb::split_plan(c[0], c[1], t.wg * t.ipt, t.tile_j, nb::choose_split(1, c[0], c[1], t), &nb, &S, &jc);
        if (t.tile_j != 64 || jc != 5 * t.tile_j) {
            printf("%lld x %lld: ranges of %d records\n", c[0], c[1], jc);
            ++bad;
        }
    }
    return bad ? 1 : 0;
}

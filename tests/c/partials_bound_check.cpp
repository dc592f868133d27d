// Host-side check of force_partials_bound (csrc/force.hip): no shape that the
// library chooses for ni sinks and nj sources, ni, nj <= n, has more partials,
// for every policy. Linked against the library; no device is touched. Prints
// "ok" and exits 0, or names the failure.
#include <cstdio>
#include <cstdlib>

#include "common.h"

using namespace nb;

static uint64_t state = 1;
static int64_t draw(int64_t lo, int64_t hi) {
    state = state * 6364136223846793005ull + 1442695040888963407ull;
    return lo + (int64_t)((state >> 33) % (uint64_t)(hi - lo + 1));
}

static void check(int prec, int64_t ni, int64_t nj, int64_t n) {
    for (Pick pick : {Pick::Best, Pick::Least}) {
        const Shape s = choose_force_shape(prec, ni, nj, pick);
        if (s.split > 1 && force_partials_bytes(s, ni) > force_partials_bound(prec, n)) {
            std::printf("FAIL: prec %d ni %lld nj %lld: %d ranges\n", prec, (long long)ni,
                        (long long)nj, s.split);
            std::exit(1);
        }
    }
}

int main() {
    for (int prec = NB_F64; prec <= NB_MIX_TILEC; ++prec) {
        check(prec, 16653, 20522, 20522);
        for (int64_t n = 60; n < 90000; n += 17 + n / 50)
            for (int k = 0; k < 60; ++k) {
                const int64_t i = draw(1, n);
                check(prec, i, n, n);
                check(prec, n, i, n);
                check(prec, i, draw(1, n), n);
            }
        for (int64_t n : {int64_t(1) << 17, int64_t(1) << 20, int64_t(1) << 23, int64_t(1) << 30})
            for (int k = 0; k < 4000; ++k) check(prec, draw(1, k % 2 ? n : 100000), n, n);
    }
    std::printf("ok\n");
    return 0;
}

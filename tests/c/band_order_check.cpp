// Host-side check of the two orders in which a band's work items are dealt
// (band_item of csrc/common.h): in either, the items of band [I0, I1) are the
// block pairs (I, J), I0 <= I < I1, I <= J < nb, each once; the triangle comes
// before the rectangle, and the diagonal is last in the triangle or in its
// rows' places. Prints "ok" and exits 0, or names the failure.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "common.h"

using namespace nb;

static void check(int nb, int I0, int I1, bool last) {
    const SymLayout L{(int64_t)nb * 64, 64, nb, 3, 4, 8};
    const int64_t items = sym_band_items(L, I0, I1), R = I1 - I0;
    std::vector<char> seen((size_t)nb * nb, 0);
    for (int64_t t = 0; t < items; ++t) {
        int I = -1, J = -1;
        if (last)
            band_item<true>(t, I0, I1, I, J);
        else
            band_item<false>(t, I0, I1, I, J);
        const bool in = I >= I0 && I < I1 && J >= I && J < nb;
        const bool part = (t < R * (R + 1) / 2) == (J < I1);
        const bool diag = last ? (I == J) == (t >= R * (R - 1) / 2 && t < R * (R + 1) / 2)
                               : J >= I1 || t == (int64_t)(J - I0) * (J - I0 + 1) / 2 + (I - I0);
        if (!in || !part || !diag || seen[(size_t)I * nb + J]++) {
            std::printf("FAIL: nb %d band %d..%d last %d item %lld -> %d %d\n", nb, I0, I1, last,
                        (long long)t, I, J);
            std::exit(1);
        }
    }
}

int main() {
    for (bool last : {true, false})
        for (int nb : {1, 2, 3, 7, 48, 64, 65, 130, 700})
            for (int I0 = 0; I0 < nb; I0 += 1 + nb / 9)
                for (int I1 = I0 + 1; I1 <= nb; I1 += 1 + nb / 7) {
                    check(nb, I0, I1, last);
                    check(nb, I0, nb, last);
                }
    // far into a large triangle, where its index needs more than 32 bits
    for (int64_t j : {int64_t(1), int64_t(65535), int64_t(131071), int64_t(500000)})
        for (int64_t i : {int64_t(0), j / 2, j - 1}) {
            int I, J;
            band_item<true>(j * (j - 1) / 2 + i, 0, 1 << 20, I, J);
            if (I != i || J != j) std::printf("FAIL: far item\n"), std::exit(1);
            band_item<false>(j * (j + 1) / 2 + i, 0, 1 << 20, I, J);
            if (I != i || J != j) std::printf("FAIL: far item\n"), std::exit(1);
        }
    std::printf("ok\n");
    return 0;
}

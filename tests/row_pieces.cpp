// The pieces of every row of small ballot arrays: what is loaded lies inside the
// array, and the entries are the row's.  Prints the first mistake, or "ok".
#include <stdio.h>
#include <string.h>

#include <vector>

#include "../paper_2505_12976_amd/csrc/row_pieces.h"

template <bool I32, bool LONG>
static bool check(int n, int L, int shift) {
    using P = RowPieces<I32, LONG>;
    using Id = typename std::conditional<I32, uint32_t, uint16_t>::type;
    constexpr int FLY = 3;
    alignas(16) static Id buffer[4096];
    memset(buffer, 0x5A, sizeof buffer);
    Id *b = buffer + 64 + shift;  // (ids from one on; around them 0x5A5A..)
    for (int i = 0; i < n * L; ++i) b[i] = (Id)(i + 1);
    const char *lo = (const char *)b, *hi = (const char *)(b + n * L);
    for (int row = 0; row < n; ++row) {
        const P p(b, n, L, row);
        std::vector<int> seen(L, 0);
        for (int lane = 0; lane < 64; ++lane)
            for (int j0 = 0; j0 < p.count; j0 += 64 * FLY) {
                for (int u = 0; u < FLY; ++u) {
                    const char *q = p.source(p.piece(j0 + lane + 64 * u));
                    if (p.spare ? q < lo || q + 16 > hi || (uintptr_t)q % 16 : p.inside(p.piece(j0 + lane + 64 * u))) {
                        printf("n=%d L=%d shift=%d row=%d lane=%d: reads at %td .. of %td bytes\n", n, L, shift, row, lane,
                               q - lo, hi - lo);
                        return false;
                    }
                }
                v4u x[FLY];
                p.template load<FLY>(x, j0 + lane);
                for (int u = 0; u < FLY; ++u)
                    p.each(x[u], j0 + lane + 64 * u, L, [&](int32_t t, uint32_t raw) {
                        if (j0 + lane + 64 * u >= p.count) return;
                        seen[t] += raw == (uint32_t)(row * L + t + 1) ? 1 : 1000;
                    });
            }
        for (int t = 0; t < L; ++t)
            if (seen[t] != 1) {
                printf("n=%d L=%d shift=%d row=%d entry %d: %d\n", n, L, shift, row, t, seen[t]);
                return false;
            }
    }
    return true;
}

static bool both(int n, int L, int shift) {
    if (!check<false, false>(n, L, shift) || (L > 64 && !check<false, true>(n, L, shift))) return false;
    return shift >= 4 || (check<true, false>(n, L, shift) && (L <= 64 || check<true, true>(n, L, shift)));
}

int main() {
    for (int n = 1; n <= 4; ++n)
        for (int L = 1; L <= 70; ++L)
            for (int shift = 0; shift < 8; ++shift)
                if (!both(n, L, shift)) return 1;
    for (int L : {255, 256, 257, 777})
        for (int shift = 0; shift < 8; ++shift)
            if (!both(3, L, shift)) return 1;
    printf("ok\n");
    return 0;
}

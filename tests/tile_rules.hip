// Host-only checks of rules in fft_tile.h: the form of a direct stage, over every radix,
// length and width that a tile takes, and the walk over rows-contiguous data. Exit status
// 0 when all hold.
#include <algorithm>
#include <cstdio>
#include <vector>

#include "fft_tile.h"

using namespace ips;

static int g_fail = 0;

static void expect(bool ok, const char *what, int R, int NR, int lgs)
{
    if (ok) return;
    if (++g_fail < 20) std::printf("FAILED: %s (R = %d, positions %d, 2^%d sequences)\n", what, R, NR, lgs);
}

// rounds of a thread over the items of ST x QT outputs
template <int NT>
static int rounds(int R, int NR, int lgs, int ST, int QT)
{
    return ((NR << lgs) / ST * ((R + QT - 1) / QT) + NT - 1) / NT;
}

template <bool F64, int MAXE, int NT>
static void check(int maxn)
{
    constexpr int Q2 = F64 ? 2 : 4;
    for (int R = 7; R < maxn; ++R) {
        bool prime = true;
        for (int q = 2; q * q <= R; ++q) prime = prime && R % q != 0;
        if (!prime) continue;
        for (int NR = 2; NR * R <= maxn; NR += 2)
            for (int lgs = 0; (NR * R) << lgs <= MAXE * NT && lgs <= 4; ++lgs) {
                const bool sh = direct_shared<F64, NT>(R, NR, lgs);
                const int ST = lgs > 0 ? 2 : 1, QT = lgs > 0 ? Q2 : 2 * Q2;
                const int r1 = rounds<NT>(R, NR, lgs, 1, 1), rs = rounds<NT>(R, NR, lgs, ST, QT);
                expect(r1 <= direct_items<MAXE, 1, 1>(), "held items, one output at a time", R, NR, lgs);
                expect(rs <= (lgs > 0 ? direct_items<MAXE, 2, Q2>() : direct_items<MAXE, 1, 2 * Q2>()),
                       "held items, shared", R, NR, lgs);
                // tiles without an output per thread never share, and a thread that
                // shares reads less than one that does not
                expect(r1 > 1 || !sh, "a tile of fewer outputs than threads shares", R, NR, lgs);
                expect(sh == (rs * (ST + QT) <= 2 * r1), "LDS reads of the shared form", R, NR, lgs);
            }
    }
}

// by_columns: every element once, and no thread with more rows than an even split leaves
template <int NT>
static void check_columns()
{
    constexpr int NW = NT / 64;
    for (int lgW = 1; lgW <= 5; ++lgW)
        for (int ncols = 1; ncols <= 1 << lgW; ++ncols)
            for (int nrows : {1, 63, 64, 65, 255, 256, 257, 1023, 1025, 5999}) {
                std::vector<int> seen((size_t)ncols * nrows, 0);
                int most = 0;
                for (int t = 0; t < NT; ++t) {
                    int n = 0;
                    by_columns<NT>(lgW, ncols, nrows, t, [&](int c, int r) {
                        ++seen[(size_t)c * nrows + r];
                        ++n;
                    });
                    most = std::max(most, n);
                }
                const int W = 1 << lgW, waves = std::max(1, NW / W); // per column
                expect(std::all_of(seen.begin(), seen.end(), [](int v) { return v == 1; }), "every element once", ncols,
                       nrows, lgW);
                expect(most <= (ncols + NW - 1) / NW * ((nrows + 64 * waves - 1) / (64 * waves)), "idle waves", ncols,
                       nrows, lgW);
            }
}

int main()
{
    check_columns<256>();
    check_columns<1024>();
    check<true, 4, 256>(2048);
    check<true, 8, 256>(2048);
    check<true, 16, 256>(2048);
    check<false, 4, 256>(2048);
    check<false, 8, 256>(2048);
    check<false, 16, 256>(2048);
    check<true, 4, 1024>(4096);
    check<true, 8, 1024>(8192);
    check<false, 4, 1024>(4096);
    check<false, 8, 1024>(8192);
    if (g_fail) return 1;
    std::printf("tile rules hold\n");
    return 0;
}

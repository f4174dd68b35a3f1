// Counts which items of a launch the eight XCDs get (XcdShare), over many numbers of items, and whether tile_cost of the stage path's
// contractions counts the rounds of workgroups that the busiest XCD then has. Host code only: nothing is launched.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "taq_gemm_op.h"

#define CHECK(cond)                                                                       \
    do {                                                                                  \
        if (!(cond)) {                                                                    \
            std::fprintf(stderr, "%s:%d: check failed: %s\n", __FILE__, __LINE__, #cond); \
            std::exit(1);                                                                 \
        }                                                                                 \
    } while (0)

using namespace taq;

static long busiest(unsigned n) {
    long count[8] = {}, most = 0;
    std::vector<char> seen(n, 0);
    long last[8];
    for (long& l : last) l = -1;
    for (unsigned block = 0; block < XcdShare::grid(n); ++block) {
        const int i = XcdShare::item(block, n), x = block & 7;
        if (i < 0) continue;
        CHECK((unsigned)i < n && !seen[i] && (last[x] < 0 || i == last[x] + 1));  // one after the other
        seen[i] = 1;
        last[x] = i;
        ++count[x];
    }
    for (char s : seen) CHECK(s);
    for (int x = 0; x < 8; ++x) {
        most = count[x] > most ? count[x] : most;
        CHECK(count[x] >= (long)n / 8);
        if (x && last[x] >= 0 && last[x - 1] >= 0) CHECK(last[x] > last[x - 1]);  // the XCDs follow one another in the order of the items
    }
    CHECK(most == ((long)n + 7) / 8);
    return most;
}

int main() {
    for (unsigned n = 1; n < 3000; ++n) busiest(n);
    for (unsigned n : {65535u, 65536u, 1000003u, 1u << 22}) busiest(n);
    for (unsigned x = 0; x < 8; ++x) {  // no overflow at the largest number
        const unsigned n = (unsigned)XcdShare::MOST;
        CHECK(XcdShare::item(x, n) == (int)(n / 8 * x) && XcdShare::item(x + (n - 8), n) == (int)(n / 8 * (x + 1)) - 1 && XcdShare::item(x + n, n) == -1);
    }
    // tile_cost: an XCD has 32 compute units
    long checked = 0;
    for (int tiles = 1; tiles <= 1100; tiles += 1 + tiles / 100)
        for (int H : {4, 6, 8, 12, 20})
            for (int tph : {1, 3, 4, 5, 10})
                for (int mb : {2, 4, 6, 8})
                    for (int nb : {4, 5, 8, 10}) {
                        GemmOpArgs a = {};
                        a.tiles = tiles;
                        a.H = H;
                        a.tph = tph;
                        const int mx = (tiles + mb - 1) / mb, nx = (H * tph + nb - 1) / nb;
                        const long rounds = (busiest(mx * nx) + 31) / 32;
                        const int step = 4 * mb * nb > 16 * (mb + nb) ? 4 * mb * nb : 16 * (mb + nb);
                        CHECK(tile_cost(a, mb, nb) == (rounds > 1 ? rounds * step : step + 60));
                        ++checked;
                    }
    std::printf("xcd_share: ok (%ld)\n", checked);
    return 0;
}

// Walks every expert count and form of the price solve: a pass writes (2 * bins + 1) rows of its columns into one copy of the
// tables, which must end before the next copy begins.
#include <cstdio>

#include "price_tables.h"

int main()
{
    using namespace maxscore;
    int bad = 0;
    for (int E = 2; E <= kPriceMaxE; ++E)
        for (int extra = 0; extra < 2; ++extra) {
            const int bins = E <= 256 ? 20 : 10, columns = (E + extra + 3) / 4 * 4, written = (2 * bins + 1) * columns;
            if (price_bins(E) != bins || price_columns(E, extra == 0) != columns || price_table_ints(E, extra == 0) != written ||
                written > kPTableInts) {
                std::printf("E=%d extra=%d: %d words written, a copy has %d\n", E, extra, written, kPTableInts);
                ++bad;
            }
            // (with spare capacity one more row of bins)
            const int more = price_table_ints(E, true, true) - price_table_ints(E, true);
            if (more < bins || more % 4 != 0 || price_table_ints(E, true, true) > kPTableInts) {
                std::printf("E=%d: %d more words with spare capacity\n", E, more);
                ++bad;
            }
        }
    std::puts(bad ? "tables overlap" : "ok");
    return bad != 0;
}

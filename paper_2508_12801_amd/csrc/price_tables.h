// Sizes of the tables a price pass adds to.  Plain C++: the host test that walks all expert counts includes it too.
#pragma once

namespace maxscore {

constexpr int kPriceMaxE = 512;
constexpr int kPBins = 20;                        // margin bins per side: ten octaves, two bins each (one beyond 256 experts)

constexpr int price_bins(int E) { return E <= 256 ? kPBins : kPBins / 2; }
// Columns: one per expert, and one for the unfilled slots where demand exceeds capacity; whole 16-byte pieces.
constexpr int price_columns(int E, bool no_extra) { return (E + (no_extra ? 0 : 1) + 3) & ~3; }
// Margins of the holds, margins of the newcomers, and one row of holds per expert; with spare capacity behind them the margins of the experts
// that have a price together (a row of bins: as one more column they took 0.3 us of a pass over 10007 rows of 96 experts).
constexpr int price_table_ints(int E, bool no_extra, bool spare = false)
{
    return (2 * price_bins(E) + 1) * price_columns(E, no_extra) + (spare ? (price_bins(E) + 3) & ~3 : 0);
}

// The largest table of any expert count.  (It is that of 512 experts with one more column, not that of 256: half as many bins
// of twice as many columns, but the row of holds does not halve.)
constexpr int price_table_most(int E_first, int E_last)
{
    int most = 0;
    for (int E = E_first; E <= E_last; ++E) {
        const int n = price_table_ints(E, false), m = price_table_ints(E, true, true);
        most = n > most ? n : most;
        most = m > most ? m : most;
    }
    return most;
}
constexpr int kPTableInts = price_table_most(1, kPriceMaxE);

}  // namespace maxscore

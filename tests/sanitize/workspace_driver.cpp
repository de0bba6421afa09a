// The iterative assignment's tiles and tables inside the workspace, over token counts around the block sizes, all the expert
// counts and slots that matter, and at the largest sizes: they end before the next region begins.  Linked with api.cpp and the stubs.
#include <cstdio>

#include "common.h"

int main()
{
    using namespace maxscore;
    const int Ts[] = {1, 3, 63, 64, 65, 255, 4097, 65536, (1 << 21) - 63, 1 << 21}, Es[] = {1, 2, 64, 65, 128, 129, 511, 1024}, ks[] = {1, 2, 16, 17, 34, 35, 64};
    int bad = 0;
    for (int T : Ts)
        for (int E : Es)
            for (int k : ks) {
                if (k > E) continue;
                const WorkspaceLayout L = workspace_layout(T, E, k);
                const size_t blocks = ((size_t)T + 63) / 64;
                // tables, sums and pairs per block, a word per (slot, block)
                const size_t tables = 4 * (size_t)kMaxE * 11 + 16 + 256 + (8 + 4) * blocks + 4 * k * blocks;
                const size_t tiles = iter_tiles_off(L, T, E), words = k * blocks * E;
                const bool fit = tiles + 4 * words <= L.price_off;
                if (tiles < L.wcnt_off + 4 * blocks * E || tiles % 256 != 0 || fit != iter_tiles_are_words(L, T, E, k) ||
                    (!fit && (E <= 128 || k <= 34)) || tiles + words > L.price_off || L.price_off + tables > L.wt_off) {
                    std::printf("T=%d E=%d k=%d: a region is too small\n", T, E, k);
                    ++bad;
                }
            }
    // two tables of a byte per (token, expert) on either side of the pairs' keys, counts and arcs: nothing that grows with all three
    const size_t most = maxscore_workspace_bytes(1 << 21, 0, 1024, 64, 1 << 21);
    const double T = 1 << 21, pairs = T * 64;
    const double limit = 2 * T * 1024 + pairs * (8 + 1024 / 256. + 3) + T * (1 + 8 + 48 + 8) + (4 << 20);
    std::printf("%.3f GB of %.3f\n", most * 1e-9, limit * 1e-9);
    if (most > limit) ++bad;
    std::puts(bad ? "failed" : "ok");
    return bad != 0;
}

// Walks expert, slot and block counts of the rerouting rounds that one workgroup takes: what it asks for fits a launch, at every size, and
// it is refused only where it would not.
#include <cstdio>

#include "iter_tail.h"

int main()
{
    using namespace maxscore;
    int bad = 0, refused = 0;
    for (int E = 1; E <= 1024; E += E < 70 ? 1 : 61)
        for (int k = 1; k <= 64 && k <= E; ++k)
            for (int n_wg = 1; n_wg <= 32768; n_wg += n_wg < 4 ? 1 : 97) {
                const int most = tail_most(E, k, n_wg);
                if (most >= 0) {
                    bad += tail_words(most, E, k, n_wg) * 4 > 62 * 1024 || most < 1 || most > kTailMost || most * k > kTailSlots || k > 32;
                } else if (k <= kTailMaxK && n_wg <= kTailMaxBlocks) {
                    ++refused;
                    bad += k < 6 || n_wg * 64 < 300000;
                }
            }
    std::printf("%d refused, %d wrong\n", refused, bad);
    return bad != 0 || refused == 0;
}

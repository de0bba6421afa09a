// The host's wait for the words that end a call, against a model: words that come in any order, late, or never, and a launch that fails.
#include <cstdio>
#include <initializer_list>

#include "done_wait.h"

using namespace maxscore;

struct Model {
    int n, at[40], fail, sync_rc, never;       // at: looks before word i is there
    int looks = 0, syncs = 0, launches = 0;
    bool idle = false;
    unsigned number(int i)
    {
        ++looks;
        if (i == never) return 6;
        return idle || looks > at[i] ? 7 : 6;
    }
    void pause() {}
    bool late() const { return looks > 2000; }
    int sync() { ++syncs; idle = true; return sync_rc; }
    int lost() const { return -9; }
    int launch() { ++launches; return fail; }
};

int main()
{
    int bad = 0;
    for (int n = 0; n < 32; n += n < 3 ? 1 : 7)
        for (int order = 0; order < 4; ++order)
            for (int scale : {0, 1, 40, 300}) {
                Model m = {n, {}, 0, 0, -1};
                int longest = 0;
                for (int i = 0; i <= n; ++i) {
                    m.at[i] = scale * (order == 0 ? i : order == 1 ? n - i : order == 2 ? i * 7 % (n + 1) : n);
                    longest = m.at[i] > longest ? m.at[i] : longest;
                }
                bad += tell_and_wait(m, 7, n) != 0 || m.launches != 1 || m.syncs != (longest > 2300 ? 1 : m.syncs) || (longest < 1500 && m.syncs != 0) || m.syncs > 1;
            }
    Model launch = {3, {}, -5, 0, -1};              // the launch fails: the stream is waited for all the same
    bad += tell_and_wait(launch, 7, 3) != -5 || launch.syncs != 1 || launch.looks != 0;
    Model stream = {3, {1 << 30, 1 << 30, 1 << 30, 1 << 30}, 0, -5, -1};          // an error of the stream
    bad += tell_and_wait(stream, 7, 3) != -5 || stream.syncs != 1;
    Model never = {3, {}, 0, 0, 2};                 // a word that never comes
    bad += tell_and_wait(never, 7, 3) != -9 || never.syncs != 1;
    std::printf("%d wrong\n", bad);
    return bad != 0;
}

// Walks the host's loop over the passes of a price solve against a model of the stream: the prices are done behind a pass of any number, some of
// the words that the launches tell are lost, and the hint that the end is near comes at any time.  The end runs once, behind the last pass.
#include <cstdio>
#include <vector>

#include "price_loop.h"

using namespace maxscore;

struct Model {
    int done_behind;             // passes after which the prices are done
    unsigned lost;               // bit i: the i-th word is lost
    unsigned soon;               // bit t: the hint of the launch before pass t
    int far;
    struct Launch { bool end; int t; };
    std::vector<Launch> queue;
    size_t ran = 0;
    int passes = 0, ends = 0, early = 0, words = 0, late = 0, looks = 0;
    PriceSeen word = {false, 0, false, false};

    bool done() const { return passes >= done_behind; }
    void tell(int t)
    {
        if (lost >> (words++ & 31) & 1) return;
        if (done()) word.done = true;
        else if (t > 0) word = {word.done, t, far != 0, (soon >> t & 1) != 0};
    }
    void run_one()
    {
        if (ran == queue.size()) return;
        const Launch l = queue[ran++];
        if (l.end) {
            if (l.t) tell(l.t);
            if (l.t && !done()) ++early;
            else ++ends;
            return;
        }
        tell(l.t);
        if (ends) ++late;
        if (!done()) ++passes;
    }
    void pass(int t) { queue.push_back({false, t}); }
    void end(int t) { queue.push_back({true, t}); }
    PriceSeen told()
    {
        if (++looks % 3 == 0) run_one();
        return word;
    }
    int idle() const { return ran == queue.size() ? 1 : 0; }
    int state(int t, PriceSeen *seen) { *seen = {done(), t, far != 0, false}; return 0; }
    void pause() {}
    int seen(int t, PriceSeen *now) { return price_seen(*this, t, now); }
};

int main()
{
    int bad = 0, again = 0, early = 0;
    for (int n_pass = 4; n_pass <= 7; ++n_pass)
        for (int look : {-1, n_pass - 2})
            for (int far = 0; far < 2; ++far)
                for (int rest = 0; rest < 2; ++rest)
                    for (int done_behind = 0; done_behind <= n_pass + 5; ++done_behind)
                        for (unsigned lost : {0u, ~0u, 0x55555555u, 0xaaaaaaaau, 1u, 2u, 4u, 8u, 16u, 32u, 64u, 128u, 12u, 24u, 48u, 96u})
                            for (unsigned soon : {0u, ~0u, 4u, 8u, 16u, 32u, 40u, 80u}) {
                                Model m = {done_behind, lost, soon, far};
                                if (rest) bad += price_passes(m, n_pass, look, 4, true, false) != 0 || m.queue.size() != kPriceAhead;
                                bad += price_passes(m, n_pass, look, 4, false, rest != 0) != 0;
                                while (m.ran < m.queue.size()) m.run_one();
                                const int most = n_pass + (far && look >= 0 ? 4 : 0), want = done_behind < most ? done_behind : most;
                                if (m.ends != 1 || m.late || m.passes != want) {
                                    if (!bad++) std::printf("passes %d done behind %d lost %x soon %x: %d ends, %d passes\n", n_pass, done_behind, lost, soon, m.ends, m.passes);
                                }
                                again += m.ends > 1;
                                early += m.early;
                            }
    std::printf("%d wrong, %d with a second end, %d ends came too early\n", bad, again, early);
    return bad != 0 || early == 0;
}

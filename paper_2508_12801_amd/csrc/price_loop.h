// How the host enqueues the passes of a price solve and its end.  Plain C++: the host test that walks it includes it too.
#pragma once

namespace maxscore {

constexpr int kPriceAhead = 2;                    // passes that are enqueued before the first is looked at

// What the passes before some pass have come to.
struct PriceSeen {
    bool done;         // the prices need no further pass
    int passes;        // passes that have ended
    bool far, soon;    // many tokens are still too many; few: the next pass may be the last
};

// Pass t is enqueued when pass t - 1 has begun, so that one stays queued behind the one that runs: a pass that is still queued when the
// prices are done costs two empty launches (5 us).  So where the pass that runs is likely to be the last, the end is enqueued behind it
// instead, which looks at the prices first; if these are not done, that costs as much.
//
// q.pass(t) enqueues a pass and its step, q.end(t) the end, with t > 0 unless the passes turn out to go on with pass t.  q.seen(t, &seen) waits
// until the passes before pass t have ended, or the prices are done, and says so by the state of the solve itself where nobody has told: an end that has
// run must not be enqueued again.  It returns an error or 0.  `look`: pass t = look + 2 is preceded by a look at whether `more` passes are needed.
// begin: the first passes alone, for which nothing is waited for; rest: what follows these.
template <class Q>
int price_passes(Q &q, int n_pass, int look, int more, bool begin, bool rest)
{
    for (int t = rest ? kPriceAhead : 0;; ++t) {
        if (begin && t >= kPriceAhead) return 0;
        if (t >= kPriceAhead && (t < n_pass || t == look + 2)) {
            PriceSeen now = {false, 0, false, false};
            int rc = q.seen(t - 1, &now);
            if (rc) return rc;
            if (t == look + 2 && now.far) n_pass += more;
            if (now.done) break;
            if (t < n_pass && now.soon) {
                q.end(t);
                rc = q.seen(t, &now);
                if (rc || now.done) return rc;
            }
        }
        if (t >= n_pass) break;
        q.pass(t);
    }
    q.end(0);
    return 0;
}

// q.seen by words that the kernels tell: told() gives what they say, idle() 1 if the stream has nothing left to do (0: it has; else an error), state() the solve's
// own state then (all that has been enqueued has ended).  Words may be lost: passes that were begun and given up in another stream
// may tell theirs in the same place.
template <class W>
int price_seen(W &w, int t, PriceSeen *seen)
{
    for (unsigned spin = 1;; ++spin) {
        *seen = w.told();
        if (seen->done || seen->passes >= t) return 0;
        if ((spin & 4095) == 0) {
            const int idle = w.idle();
            if (idle < 0) return idle;
            if (idle) {
                *seen = w.told();
                if (seen->done || seen->passes >= t) return 0;
                return w.state(t, seen);
            }
        }
        w.pause();
    }
}

}  // namespace maxscore

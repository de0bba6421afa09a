// How the host waits for the words that end a call.  Plain C++: the host test that walks it includes it too.
#pragma once

namespace maxscore {

// Until all of words 0 .. n carry the number of the wait.  w.number(i) is what word i carries, w.late() whether it has taken long: then w.sync(),
// which sleeps until the stream has nothing left to do and reports an error of it, goes on (it returns an error or 0), and behind it a word that is not there is
// an error too.
template <class W>
int wait_told(W &w, unsigned number, int n)
{
    int have = 0;
    for (unsigned spin = 1; have <= n; ++spin) {
        if (w.number(have) == number) ++have;
        else w.pause();
        if ((spin & 255) == 0 && have <= n && w.late()) {
            const int rc = w.sync();
            if (rc) return rc;
            while (have <= n && w.number(have) == number) ++have;
            return have > n ? 0 : w.lost();
        }
    }
    return 0;
}

// w.launch() enqueues the kernel that writes the words.  If it cannot, nothing of the call is left running on the caller's buffers either.
template <class W>
int tell_and_wait(W &w, unsigned number, int n)
{
    const int rc = w.launch();
    if (rc) {
        (void)w.sync();
        return rc;
    }
    return wait_told(w, number, n);
}

}  // namespace maxscore

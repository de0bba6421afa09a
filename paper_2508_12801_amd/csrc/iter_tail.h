// Sizes of the rerouting rounds that one workgroup goes through by itself.  Plain C++: the host test that walks them includes it too.
#pragma once

#include <algorithm>

namespace maxscore {

// Pairs that one workgroup takes through the rounds that are left: as many as it proposes for in the time of a round of two launches
// (a row takes 150 instructions of eight lanes, and one compute unit issues them all: with 2048 pairs 14493 tokens of 32 experts 193 us a
// call, with 1024 173).
constexpr int kTailMost = 1024, kTailEntries = 1 << 16, kTailSlots = 8192, kTailMaxK = 32, kTailMaxBlocks = 8192;
constexpr int kTailLds = 62 * 1024;               // bytes it may ask for: a launch has 64 KB, of which the kernel itself declares less than 2

// LDS of the tail, in words: tokens, open slots and slots of its rows, room and proposals per expert, its pairs twice, their proposals
// (half words), proposals per (64 pairs, expert), before that open slots per (64 rows, slot).  The blocks' first rows lie where the pairs go.
constexpr int tail_words(int most, int E, int k, int n_wg)
{
    const int tiles = (most + 63) / 64, pairs = 2 * most + (most + 1) / 2, tab = tiles * std::max(E, kTailMaxK) + 1;
    return (2 + k) * most + 2 * E + std::max(pairs + tab, n_wg + 1);
}

// Pairs it takes at most, -1 if it is not to be used: from some 5000 blocks on (320000 tokens) the blocks' first rows do not fit beside eight
// and more slots of 1024 rows.
constexpr int tail_most(int E, int k, int n_wg)
{
    if (k > kTailMaxK || n_wg > kTailMaxBlocks) return -1;
    const int most = std::min(kTailMost, std::min(kTailEntries / E, kTailSlots / k));
    return tail_words(most, E, k, n_wg) * 4 <= kTailLds ? most : -1;
}

}  // namespace maxscore

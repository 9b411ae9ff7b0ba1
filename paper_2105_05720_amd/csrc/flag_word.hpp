// How a launch's waves agree on the overflow flag through the state word (see FlagCount in kernels.hip.h, where the reasons are).  No HIP
// in here: the host can run it as well.  `Words` are the two words: the state word's read, exchange and compare-exchange, and
// raise(), which stores 1 into the flag.
#pragma once

#include "piece_order.hpp"

namespace ccf {

constexpr unsigned long long kStateBad = 1ull, kStateCleared = 2ull;
CCF_ANYWHERE unsigned long long state_of(uint32_t tag, unsigned long long mark) { return ((unsigned long long)tag << 2) | mark; }

// The launch's last arrival, once its 0 has been performed in the flag.
template <class Words> CCF_ANYWHERE void flag_cleared(Words words, uint32_t tag)
{
    if (words.exchange(state_of(tag, kStateCleared)) == state_of(tag, kStateBad)) words.raise();
}

// A wave that has something to report, at any time after its arrival.  (A plain store of 1 would not do: the 0 may come after it.)
template <class Words> CCF_ANYWHERE void flag_report(Words words, uint32_t tag)
{
    const unsigned long long bad = state_of(tag, kStateBad), cleared = state_of(tag, kStateCleared);
    unsigned long long cur = words.read();
    while (true) {
        if (cur == cleared) {                 // the flag was cleared before: this store comes after the 0
            words.raise();
            break;
        }
        if (cur == bad) break;                // another wave has reported for this launch already
        if (words.replace(cur, bad)) break;   // the last arrival's exchange will return this report
    }
}

}  // namespace ccf

// How many targets are walked and listed at a time (host only, no HIP).
#pragma once
#include <stdint.h>

#include <algorithm>

namespace tr {

// The largest chunk whose scratch can be had: want, halved while take(n) fails,
// down to least (1 <= least <= want).  take leaves nothing behind when it
// fails.  0: not even least.
template <typename Take>
int64_t take_chunk(int64_t want, int64_t least, Take &&take)
{
    for (int64_t n = want;; n = std::max(least, n / 2)) {
        if (take(n)) return n;
        if (n <= least) return 0;
    }
}

}  // namespace tr

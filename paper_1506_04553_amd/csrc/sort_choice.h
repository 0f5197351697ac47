// sort_choice.h -- whether a build sorts whole keys at once, or tries the short
// sort first (tree.hip: leading bits, then runs of equal ones).
#pragma once

#include <stdint.h>

namespace p3t {

// A short sort that meets a run it cannot order costs its passes and a host wait
// before the whole sort: 2^20 particles with one far away, whose cluster lies in few
// cells of 40 bits, take 1.07 ms to build so, 0.89 sorted whole at once (and 0.58
// without that one).  What decides is where the particles lie, which changes little
// from one build to the next while their number may change in each; so after such a
// build the next `wait` sort whole keys, whatever their number, and then one tries
// again.  A dense system loses little (0.90 ms on average over 40 builds of different
// numbers), and one that was dense for a while comes back to the short sort.
struct SortChoice {
    static constexpr int32_t kFirst = 16, kMost = 1024;
    int32_t wait = kFirst;   // builds of whole keys after the next failure
    int32_t left = 0;        // builds that still are
    // the next build's choice
    bool whole() {
        if (left == 0) return false;
        --left;
        return true;
    }
    // how a short sort ended
    void tried(bool longer) {
        left = longer ? wait : 0;
        wait = !longer ? kFirst : wait < kMost ? 2 * wait : kMost;
    }
};

}  // namespace p3t

// What a launch of workgroups that wait for each other comes to: kept or given
// up, the same for all of them.  The rule alone (no HIP), so that it can be
// checked on the CPU over every order of events.
//
// One word per launch, OPEN at its start and changed once.  A workgroup that
// has waited too long gives the launch up, unless a workgroup that got through
// the launch's last meeting has kept it; one that got through keeps it before
// it stores anything, unless it has been given up.  A launch is kept only when
// every workgroup has brought its word to the last meeting, so a workgroup
// that is told so finds all words there and gets through as well.
//
// W: load() is the word as it is or was; swap(from, to) sets it to `to` if it
// is `from` and returns what it was.
#pragma once

#include <cstdint>

#ifdef __HIPCC__
#define DSM_RULE __host__ __device__ __forceinline__
#else
#define DSM_RULE inline
#endif

namespace dsm {

enum Outcome : uint32_t { OUTCOME_OPEN = 0, OUTCOME_GIVEN_UP = 1, OUTCOME_KEPT = 2 };

// A waiting workgroup, `late` once its time is up: whether it stops waiting.
template <class W>
DSM_RULE bool outcome_gives_up(W w, bool late) {
    uint32_t was = w.load();
    if (was == OUTCOME_OPEN && late) {
        was = w.swap(OUTCOME_OPEN, OUTCOME_GIVEN_UP);
        if (was == OUTCOME_OPEN) was = OUTCOME_GIVEN_UP;
    }
    return was == OUTCOME_GIVEN_UP;
}

// A workgroup past the last meeting: whether it may store its results.
template <class W>
DSM_RULE bool outcome_keeps(W w) {
    return w.swap(OUTCOME_OPEN, OUTCOME_KEPT) != OUTCOME_GIVEN_UP;
}

}  // namespace dsm

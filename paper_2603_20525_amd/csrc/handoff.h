// How one wave hands a state to another through memory, by a flag with three
// values. The giver writes the state and then calls handoff_give once; the taker
// calls handoff_take once, and if that succeeded reads the state and then calls
// handoff_release. Either may come first and the taker may give up, in which case
// it does without; whoever comes last puts the flag back to rest. Host and device
// code alike: Flag has load, store, exchange, compare_exchange (which returns the
// value before) and pause.
#pragma once

#ifdef __HIP__
#define PLAN_HANDOFF_FN __attribute__((device, always_inline)) inline
#else
#define PLAN_HANDOFF_FN inline
#endif

namespace plan {

enum : int { HANDOFF_REST = 0, HANDOFF_READY = 1, HANDOFF_GIVEN_UP = 2 };

template <class Flag>
PLAN_HANDOFF_FN void handoff_give(const Flag &f) {
    if (f.exchange(HANDOFF_READY) == HANDOFF_GIVEN_UP) f.store(HANDOFF_REST);
}

// Whether the state is there, looked for up to `looks` times and once more with
// the decision not to wait any longer.
template <class Flag>
PLAN_HANDOFF_FN bool handoff_take(const Flag &f, int looks) {
    for (int i = 0; i < looks; ++i) {
        if (f.load() == HANDOFF_READY) return true;
        f.pause();
    }
    return f.compare_exchange(HANDOFF_REST, HANDOFF_GIVEN_UP) == HANDOFF_READY;
}

template <class Flag>
PLAN_HANDOFF_FN void handoff_release(const Flag &f) {
    f.store(HANDOFF_REST);
}

}  // namespace plan

"""The hand-off of a state between two waves (csrc/handoff.h), compiled for the
host: every order of its two sides, the taker waiting for any number of looks
and giving up included, hands on the whole state or none, and leaves the flag at
rest for the next launch."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2603_20525_amd", "csrc")

PROGRAM = r'''
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <thread>
#include <vector>
#include "handoff.h"

static void require(bool ok, const char *what) {
    if (!ok) {
        std::printf("failed: %s\n", what);
        std::exit(1);
    }
}

// Runs both sides one access at a time, the order taken from a bit string: a
// side that wants to touch the flag waits until its turn comes.
struct Turns {
    unsigned order;
    int steps;
    std::atomic<int> at{0};
    std::atomic<int> done{0};  // bit per side that has ended
    bool mine(int side) {
        const int s = at.load();
        const int next = s < steps ? (int)(order >> s & 1) : side;
        return next == side || (done.load() & (1 << (1 - side)));
    }
};

struct SteppedFlag {
    std::atomic<int> *v;
    Turns *t;
    int side;
    template <class F>
    int turn(F f) const {
        while (!t->mine(side)) std::this_thread::yield();
        const int r = f();
        t->at.fetch_add(1);
        return r;
    }
    int load() const { return turn([&] { return v->load(); }); }
    void store(int x) const { turn([&] { v->store(x); return 0; }); }
    int exchange(int x) const { return turn([&] { return v->exchange(x); }); }
    int compare_exchange(int e, int x) const {
        return turn([&] { v->compare_exchange_strong(e, x); return e; });
    }
    void pause() const {}
};

struct FreeFlag {
    std::atomic<int> *v;
    int load() const { return v->load(); }
    void store(int x) const { v->store(x); }
    int exchange(int x) const { return v->exchange(x); }
    int compare_exchange(int e, int x) const { v->compare_exchange_strong(e, x); return e; }
    void pause() const { std::this_thread::yield(); }
};

// one hand-off of `value`; returns what the taker saw, or -1
template <class FlagG, class FlagT>
int hand_over(FlagG give, FlagT take, int *slot, int value, int looks, std::atomic<int> *done) {
    int got = -1;
    std::thread giver([&] {
        *slot = value;
        plan::handoff_give(give);
        if (done) done->fetch_or(1);
    });
    if (plan::handoff_take(take, looks)) {
        got = *slot;
        plan::handoff_release(take);
    }
    if (done) done->fetch_or(2);
    giver.join();
    return got;
}

int main() {
    std::atomic<int> flag{plan::HANDOFF_REST};
    int slot = -2, value = 0, taken = 0, given_up = 0;
    for (int looks = 0; looks <= 3; ++looks)
        for (int steps = looks + 4, order = 0; order < 1 << steps; ++order) {
            Turns t{(unsigned)order, steps};
            const int got = hand_over(SteppedFlag{&flag, &t, 0}, SteppedFlag{&flag, &t, 1}, &slot,
                                      ++value, looks, &t.done);
            require(got == -1 || got == value, "state of this hand-off or none");
            require(flag.load() == plan::HANDOFF_REST, "flag at rest after both sides");
            (got == -1 ? given_up : taken)++;
        }
    // given up where all of the taker's looks + 1 accesses come first: 2^3 orders each
    require(given_up == 4 * 8 && taken == 16 + 32 + 64 + 128 - given_up, "both endings happen");
    // the giver first is always taken, also by a taker that does not wait
    for (int looks = 0; looks <= 2; ++looks) {
        Turns t{0u, 1};
        require(hand_over(SteppedFlag{&flag, &t, 0}, SteppedFlag{&flag, &t, 1}, &slot, 7, looks,
                          &t.done) == 7, "giver first");
    }
    // free running, the next hand-off on the same flag right after the last
    for (int i = 0; i < 3000; ++i) {
        const int got = hand_over(FreeFlag{&flag}, FreeFlag{&flag}, &slot, i, i % 5, nullptr);
        require(got == -1 || got == i, "free running: state of this hand-off or none");
        require(flag.load() == plan::HANDOFF_REST, "free running: flag at rest");
    }
    std::printf("ok %d %d\n", taken, given_up);
    return 0;
}
'''


def test_every_order_leaves_the_flag_at_rest(tmp_path):
    src, exe = tmp_path / "handoff.cpp", tmp_path / "handoff"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-pthread", "-I", CSRC,
                    str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0 and r.stdout.startswith("ok"), r.stdout + r.stderr


def test_a_taker_that_leaves_the_flag_given_up_is_noticed(tmp_path):
    """The same program fails for a giver that does not put the flag back."""
    broken = tmp_path / "handoff.h"
    with open(os.path.join(CSRC, "handoff.h")) as f:
        text = f.read()
    line = "if (f.exchange(HANDOFF_READY) == HANDOFF_GIVEN_UP) f.store(HANDOFF_REST);"
    assert line in text
    broken.write_text(text.replace(line, "f.exchange(HANDOFF_READY);"))
    src, exe = tmp_path / "handoff.cpp", tmp_path / "handoff"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-I", str(tmp_path), str(src), "-o",
                    str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=100)
    assert r.returncode != 0 and "failed" in r.stdout

// Who sets which mark when, for workgroups of one launch that wait for each other and never rely on one another.
//
// Nothing here knows of a GPU: W is a wavefront's way to the marks (arrivals.h has the device's), so that the CPU tests can
// run this very code through every order in which stores and loads may take effect (tests/handshake).  W has
//   set(mark, value)           a store that others see some time later
//   get(mark)                  a load
//   settle()                   returns when everything this wavefront has set can be seen by everybody
//   swap(mark, from, to)       compare and exchange, one step for everybody; true if the mark was `from`
//   wait_until(f, ticks)       calls f until it says so or the time is up; which of the two
//
// No wait is unbounded, and none relies on all workgroups running at the same time (another stream's kernel may keep some of
// them out for as long as it likes).  A waiter whose time is up says so in a mark and looks once more; if somebody is still
// missing it leaves, and whoever arrives last finds that mark and does its work.
//
// That holds because nobody looks at a mark before its own has settled, neither who arrives nor who leaves: of an arrival and
// a departure that miss each other, each would have to look before the other's store, and so before its own.  A store
// followed by a load of another mark is no such order by itself: the two are served apart, and the load may be first.  (The
// wait in front of the first look costs nothing: the others cannot see the mark sooner either.  Step on 512 tokens 8.3 us
// without it, 8.2 with it.)
#pragma once

namespace reader {

// The low bits of a mark, which a token leaves free: kLeft, kTaken, and the XCD its workgroup runs on.
typedef unsigned long long mark_t;
constexpr mark_t kLeft = 1, kTaken = 3, kStateBits = 3, kMarkBits = 63;
constexpr int kXccShift = 2;
constexpr mark_t kTokenStep = kMarkBits + 1;

// How long a wait lasts at most, in ticks of the device's 100 MHz counter: 30 us, or what is asked for (0: one look), but never more
// than 10 ms.  A keeper waits for the longest of all shares and keeps nobody from running: four times as long.
constexpr long long kWaitTicks = 3000, kMostWaitTicks = 1000000, kKeeperPatience = 4;
constexpr int wait_ticks(long long asked) { return (int)(asked < 0 ? kWaitTicks : asked > kMostWaitTicks ? kMostWaitTicks : asked); }

// Workgroups that all have their part done and go on together: `here` is this one's arrival, everybody() looks at all marks.
// True: all have arrived; false: this one has left, and its share of what comes next is done by one of those who come later,
// who see its mark with kLeft.
template <class W, class F>
__device__ __forceinline__ bool meet(W &&w, mark_t *mine, mark_t here, F &&everybody, unsigned long long ticks) {
    w.set(mine, here);
    w.settle();
    if (w.wait_until(everybody, ticks)) return true;
    w.set(mine, here | kLeft);
    w.settle();
    return everybody();
}

// A keeper, which acts when everybody() has arrived (and is waited for by nobody).  True: it acts; false: it has left, and exactly
// one of those who arrive later acts for it (act_for_those_who_left).
template <class W, class F>
__device__ __forceinline__ bool keep(W &&w, mark_t *mine, mark_t *any_left, mark_t token, F &&everybody, unsigned long long ticks) {
    if (w.wait_until(everybody, ticks)) return true;
    w.set(mine, token | kLeft);
    w.settle();
    w.set(any_left, token);
    w.settle();
    return everybody() && w.swap(mine, token | kLeft, token | kTaken);
}

// An arrival that keepers wait for.  True: a keeper has left, so this workgroup has to look whether it was the last.
template <class W>
__device__ __forceinline__ bool arrive(W &&w, mark_t *mine, const mark_t *any_left, mark_t token) {
    w.set(mine, token);
    w.settle();
    return w.get(any_left) == token;
}

// What keepers that have left still have to do, by a workgroup that has arrived: act(k) for each of them, if it is the last.
template <class W, class F, class A>
__device__ __forceinline__ void act_for_those_who_left(W &&w, mark_t *keepers, int n, mark_t token, F &&everybody, A &&act) {
    if (!everybody()) return;
#pragma unroll 1
    for (int k = 0; k < n; ++k)
        if (w.get(keepers + k) == (token | kLeft) && w.swap(keepers + k, token | kLeft, token | kTaken)) act(k);
}

}  // namespace reader

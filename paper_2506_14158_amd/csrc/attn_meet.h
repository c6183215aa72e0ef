// How the workgroups that attend over the runs of one divided unit agree, in the launch itself, on which of them merge its parts: the
// protocol alone, which also compiles for the host (tests/host/attn_meet.cpp plays it).
//
// A workgroup only ever waits for workgroups that have started.  Those hold a CU, wait for nobody before they have handed their part
// over, and so come to it whatever else the GPU runs: no number of overlapping launches, streams or processes can hold
// a launch up, and there is no waiting limit that could run out.  (Merging workgroups of their own behind the attention's in the grid wait for workgroups that may
// not have started: the order of a grid holds within an eighth of the chip only.  Three overlapping launches of them stood
// still until a limit ran out.  Counting the parts in, the last one merging, takes read-modify-write operations across the
// chip's separate L2s, which cost tens of microseconds, and leaves a unit's merge to one CU.)
//
// Every workgroup has a word that it alone writes until the end:
//   kStarted   at its start.
//   kStays     its part is handed over, and before that it had seen every workgroup of the unit started: it waits until
//              all have handed theirs over, and merges a share of the unit;
//   kLeaves    its part is handed over, and some workgroup had not started: it is gone, without a share.
//   kKnows     it stayed, and has seen every part handed over: who stays is then the same to everybody.
// The workgroup whose first word is the last to be written sees everybody started, so somebody stays.
//
// Words lie in memory that may hold anything: they count under the call's tag only, which no other call of the process has.
// A captured graph replays a call, tag and all, so the words must be gone when the launch ends: a workgroup that
// stayed writes kKnows, then looks, and clears all words of the unit if nobody is on the way any more.  The one whose kKnows
// is the last to be written sees that, if it does not see words that another one has cleared already.
#pragma once
#include <stdint.h>

#if defined(__HIPCC__)
#define S4C_MEET __device__ __forceinline__
#else
#define S4C_MEET inline
#endif

namespace s4c {
namespace meet {

enum State { kAbsent = 0, kStarted = 1, kStays = 2, kLeaves = 3, kKnows = 4 };
constexpr uint64_t kStateBits = 7;                     // of a word; the others are the tag's, whose own are 0

S4C_MEET uint64_t word_of(uint64_t tag, int state) { return tag | (uint64_t)state; }
S4C_MEET int state_of(uint64_t tag, uint64_t word) { return (word & ~kStateBits) == tag ? (int)(word & kStateBits) : (int)kAbsent; }

// W: a workgroup's view of the unit's words.
//   tell(s)      writes this workgroup's own
//   settle()     waits until whatever it has written can be seen by everybody
//   look()       reads them all
//   all(p)       whether p(state) holds for every other workgroup's, as last read
//   which(p)     the workgroups whose state is one that p holds for, as last read, and this one: a bit set
//   clear()      writes something without a tag over all of them

// At a workgroup's start.
template <class W>
S4C_MEET void begin(W& w) {
    w.tell(kStarted);
}
// Before it hands its part over.
template <class W>
S4C_MEET void look_round(W& w) {
    w.settle();
    w.look();
}
// Its part can be seen by everybody (what it saw before decides whether it stays).  The workgroups that stay, if it does.
template <class W>
S4C_MEET uint64_t hand_over(W& w) {
    const bool stays = w.all([](int s) { return s >= kStarted; });
    w.tell(stays ? kStays : kLeaves);
    if (!stays) return 0;
    do w.look();
    while (!w.all([](int s) { return s >= kStays; }));
    w.tell(kKnows);
    return w.which([](int s) { return s == kStays || s == kKnows; });
}
// Of a workgroup that stayed, any time behind that.
template <class W>
S4C_MEET void end(W& w) {
    w.settle();
    w.look();
    if (w.all([](int s) { return s >= kLeaves; })) w.clear();
}

}  // namespace meet
}  // namespace s4c

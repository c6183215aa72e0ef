// How one workgroup tells another one of its launch something, when that one does not wait for ever: the protocol alone, which also compiles
// for the host (tests/host/told.cpp plays it).
//
// A word and a mark beside it, both in memory that may hold anything: they count under the call's tag only.  The writer writes the word.  The
// reader takes it when it finds it, or gives up: it leaves its mark and then looks once more.  The writer looks for a mark some time
// behind its word, always: nothing is known of which of the two starts first (the order of a grid holds within an eighth of the
// chip only), so the reader may be gone before the writer begins.  At least one of the two sees the other, and neither word nor mark of the
// call is left for a replay of a captured graph, tag and all, to find.  (Writers that looked only when they had been running for half the waiting time
// left words behind where they were started later than that.)
#pragma once
#include <stdint.h>

#if defined(__HIPCC__)
#define S4C_TOLD __device__ __forceinline__
#else
#define S4C_TOLD inline
#endif

namespace s4c {
namespace told {

// P: one word and its mark.
//   word(), mark()                reads
//   set_word(v), set_mark(v)      writes
//   settle()                      waits until whatever this thread has written can be seen by everybody

// ---- the writer
template <class P>
S4C_TOLD void tell(P& p, uint64_t tag) {
    p.set_word(tag);
}
// Some time behind that; what it gives goes to `end`.
template <class P>
S4C_TOLD uint64_t look_back(P& p) {
    p.settle();
    return p.mark();
}
// Whether the reader had given up.
template <class P>
S4C_TOLD bool end(P& p, uint64_t tag, uint64_t mark) {
    if (mark != tag) return false;
    p.set_word(~tag);
    p.set_mark(~tag);
    return true;
}

// ---- the reader
template <class P>
S4C_TOLD bool take(P& p, uint64_t tag) {
    if (p.word() != tag) return false;
    p.set_word(~tag);
    return true;
}
// It has waited long enough: whether the word is here after all.
template <class P>
S4C_TOLD bool give_up(P& p, uint64_t tag) {
    p.set_mark(tag);
    p.settle();
    const bool came = take(p, tag);
    if (came) p.set_mark(~tag);
    return came;
}

}  // namespace told
}  // namespace s4c

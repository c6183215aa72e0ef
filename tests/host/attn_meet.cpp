// Plays csrc/attn_meet.h: the workgroups of one divided unit, an access to memory at a time, in any order.  A write becomes
// visible any time before the workgroup has waited for it; workgroups start as places come free (the fewest: one), so that some are through
// before others begin.  One workspace is used by several launches, most of them replays under the same tag, whose parts are other numbers.
// Checks that every launch ends with nobody waiting, that every piece of the unit is merged, from parts of this launch, once,
// and that no word of the launch's tag is left.
// Usage: attn_meet TRIALS; prints the first wrong trial, exit status 1
#include <ucontext.h>

#include <cstdio>
#include <cstdlib>
#include <deque>
#include <random>
#include <vector>

#include "attn_meet.h"

using namespace s4c;

namespace {

std::mt19937 rng;
int pick(int lo, int hi) { return lo + (int)(rng() % (unsigned)(hi - lo + 1)); }

struct Memory {
    std::vector<uint64_t> words;
    std::vector<int> part;             // the launch whose part lies there
};

struct Player;
Player* running;
struct Player {
    ucontext_t here, back;
    std::vector<char> stack = std::vector<char>(64 << 10);
    std::deque<std::pair<int, uint64_t>> written;      // on the way to memory: (word, value); word -1: the part
    bool ended = false;
    void step() {
        running = this;
        swapcontext(&back, &here);
    }
    void pause() { swapcontext(&here, &back); }
};

struct Launch {
    Memory* mem;
    int n, number;
    uint64_t tag;
    std::vector<int> merged;
};
Launch* launch;

// A write lands whenever the scheduler says so; `written` is emptied in order per address only, so any entry may go first unless an
// earlier one is to the same word.
void land(Player& p, size_t i) {
    for (size_t j = 0; j < i; ++j)
        if (p.written[j].first == p.written[i].first) i = j;
    if (p.written[i].first < 0) launch->mem->part[p.written[i].second] = launch->number;
    else launch->mem->words[p.written[i].first] = p.written[i].second;
    p.written.erase(p.written.begin() + i);
}

struct View {
    Player* p;
    int me;
    std::vector<int> states;
    void tell(int s) {
        p->written.push_back({me, meet::word_of(launch->tag, s)});
        p->pause();
    }
    void settle() {
        while (!p->written.empty()) p->pause();
    }
    void look() {
        states.assign(launch->n, 0);
        std::vector<int> order(launch->n);
        for (int i = 0; i < launch->n; ++i) order[i] = i;
        for (int i = launch->n - 1; i > 0; --i) std::swap(order[i], order[rng() % (i + 1)]);
        for (int i : order) {                                  // one load, but its lanes are served one by one
            states[i] = meet::state_of(launch->tag, launch->mem->words[i]);
            p->pause();
        }
    }
    template <class P>
    bool all(P pred) const {
        for (int i = 0; i < launch->n; ++i)
            if (i != me && !pred(states[i])) return false;
        return true;
    }
    template <class P>
    uint64_t which(P pred) const {
        uint64_t m = 1ull << me;
        for (int i = 0; i < launch->n; ++i)
            if (i != me && pred(states[i])) m |= 1ull << i;
        return m;
    }
    void clear() {
        for (int i = 0; i < launch->n; ++i) {
            p->written.push_back({i, 0});
            p->pause();
        }
    }
};

int pieces;                            // of the unit, to be merged
const char* wrong;

void workgroup(int me) {
    Player* const p = running;
    View w{p, me, {}};
    meet::begin(w);
    for (int i = pick(0, 40); i > 0; --i) p->pause();          // attends
    meet::look_round(w);
    p->written.push_back({-1, (uint64_t)me});
    w.settle();
    const uint64_t who = meet::hand_over(w);
    if (who) {
        if (!(who >> me & 1)) wrong = "a workgroup that stays is not among those that do";
        const int rank = __builtin_popcountll(who & ((1ull << me) - 1)), all = __builtin_popcountll(who);
        for (int t = rank; t < pieces; t += all) {
            for (int i = 0; i < launch->n; ++i) {
                if (launch->mem->part[i] != launch->number) wrong = "a part of another launch is merged";
                p->pause();
            }
            ++launch->merged[t];
        }
        meet::end(w);
    }
    w.settle();
    p->ended = true;
    for (;;) p->pause();
}

const char* play(Launch& l) {
    launch = &l;
    wrong = nullptr;
    pieces = pick(0, 8);
    l.merged.assign(pieces, 0);
    std::deque<Player> players(l.n);
    std::vector<int> order(l.n);
    for (int i = 0; i < l.n; ++i) order[i] = i;
    for (int i = l.n - 1; i > 0; --i) std::swap(order[i], order[rng() % (i + 1)]);     // other launches hold places of some XCDs
    const unsigned lazy = 1u << pick(0, 5);
    const int places = rng() % 3 == 0 ? 1 : pick(1, l.n);
    std::vector<int> here;
    int next = 0, gone = 0;
    for (long steps = 0; gone < l.n; ++steps) {
        if (steps > 2000000) return "a launch does not end";
        while ((int)here.size() < places && next < l.n && (here.empty() || rng() % 16 == 0)) {
            Player& p = players[order[next]];
            getcontext(&p.here);
            p.here.uc_stack.ss_sp = p.stack.data();
            p.here.uc_stack.ss_size = p.stack.size();
            p.here.uc_link = nullptr;
            makecontext(&p.here, (void (*)())workgroup, 1, order[next]);
            here.push_back(order[next++]);
        }
        const size_t k = rng() % here.size();
        Player& p = players[here[k]];
        if (!p.written.empty() && rng() % lazy == 0) land(p, rng() % p.written.size());
        else p.step();
        if (wrong) return wrong;
        if (p.ended && p.written.empty()) {
            here.erase(here.begin() + k);
            ++gone;
        }
    }
    for (int t : l.merged)
        if (t != 1) return "a piece is not merged once";
    for (uint64_t w : l.mem->words)
        if (meet::state_of(l.tag, w)) return "a word is left";
    return nullptr;
}

}  // namespace

int main(int argc, char** argv) {
    const int trials = argc > 1 ? atoi(argv[1]) : 100;
    for (int t = 0; t < trials; ++t) {
        rng.seed(t + 1);
        const int n = t % 4 ? pick(2, 6) : pick(2, 24);
        Memory mem;
        mem.words.resize(n);
        for (uint64_t& w : mem.words) w = rng() % 2 ? ~0ull : ((uint64_t)rng() << 32 | rng());
        mem.part.assign(n, -1);
        const uint64_t tag = ((uint64_t)rng() << 32 | rng()) & ~meet::kStateBits;
        for (int i = 0; i < 4; ++i) {
            Launch l{&mem, n, i, i == 2 ? tag ^ (1ull << 40) : tag, {}};
            if (const char* why = play(l)) {
                printf("trial %d, %d workgroups, launch %d: %s\n", t, n, i, why);
                return 1;
            }
        }
    }
    printf("%d trials\n", trials);
    return 0;
}

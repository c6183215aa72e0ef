// Plays csrc/told.h: a writer and a reader of one word, an access to memory at a time, in any order; either may be through before the other begins,
// and a write becomes visible any time before its thread has waited for it.  Several launches, most of them replays under one tag, on memory that
// holds anything.  Checks that a reader that hears something hears what was told in its own launch, that one that gives up too early is the only
// one that does not, and that neither the word nor the mark of the tag is left.
// Usage: told TRIALS; prints the first wrong trial, exit status 1
#include <ucontext.h>

#include <cstdio>
#include <cstdlib>
#include <deque>
#include <random>
#include <vector>

#include "told.h"

using namespace s4c;

namespace {

std::mt19937 rng;
uint64_t memory[2];                    // word, mark

struct Thread {
    ucontext_t here, back;
    std::vector<char> stack = std::vector<char>(64 << 10);
    std::deque<std::pair<int, uint64_t>> written;
    bool begun = false, ended = false;
    void land(size_t i) {
        for (size_t j = 0; j < i; ++j)
            if (written[j].first == written[i].first) i = j;
        memory[written[i].first] = written[i].second;
        written.erase(written.begin() + i);
    }
    void pause() { swapcontext(&here, &back); }
};
struct Pair {
    Thread* t;
    uint64_t read(int i) {
        t->pause();
        for (size_t j = t->written.size(); j-- > 0;)
            if (t->written[j].first == i) return t->written[j].second;       // a thread sees its own writes
        return memory[i];
    }
    void write(int i, uint64_t v) {
        t->written.push_back({i, v});
        t->pause();
    }
    uint64_t word() { return read(0); }
    uint64_t mark() { return read(1); }
    void set_word(uint64_t v) { write(0, v); }
    void set_mark(uint64_t v) { write(1, v); }
    void settle() {
        while (!t->written.empty()) t->pause();
    }
};

uint64_t tag;
int patience, work, told_at, clock_now;            // reader's looks; the writer's other work
bool heard, gone;
Thread* threads;                     // the writer, the reader

void writer() {
    Pair p{&threads[0]};
    for (int i = rng() % 4; i > 0; --i) p.t->pause();
    told_at = clock_now;
    told::tell(p, tag);
    for (int i = work; i > 0; --i) p.t->pause();
    const uint64_t mark = told::look_back(p);
    for (int i = rng() % 4; i > 0; --i) p.t->pause();
    gone = told::end(p, tag, mark);
    p.settle();
    p.t->ended = true;
    for (;;) p.t->pause();
}
void reader() {
    Pair p{&threads[1]};
    heard = false;
    for (int i = 0; i < patience && !heard; ++i) heard = told::take(p, tag);
    if (!heard) heard = told::give_up(p, tag);
    if (heard && told_at < 0) { printf("heard before it was told\n"); exit(1); }
    p.settle();
    p.t->ended = true;
    for (;;) p.t->pause();
}

const char* play() {
    std::vector<Thread> two(2);
    threads = &two[0];
    Thread* t[2] = {&two[0], &two[1]};
    told_at = -1;
    clock_now = 0;
    gone = false;
    patience = rng() % 6;
    work = rng() % 8;
    const int late = rng() % 3, wait = rng() % 60;             // one starts so much later, or (late == 2) both at once
    const unsigned lazy = 1u << rng() % 5;
    for (long steps = 0;; ++steps, ++clock_now) {
        if (steps > 100000) return "a launch does not end";
        int open = 0;
        for (int i = 0; i < 2; ++i) open += !(t[i]->ended && t[i]->written.empty());
        if (!open) break;
        const int k = rng() % 2;
        Thread& a = *t[k];
        if (!a.begun) {
            if (k == late && steps < wait) continue;
            a.begun = true;
            getcontext(&a.here);
            a.here.uc_stack.ss_sp = a.stack.data();
            a.here.uc_stack.ss_size = a.stack.size();
            a.here.uc_link = nullptr;
            makecontext(&a.here, k ? reader : writer, 0);
        }
        threads = t[0];
        if (!a.written.empty() && rng() % lazy == 0) a.land(rng() % a.written.size());
        else swapcontext(&a.back, &a.here);
    }
    if (!heard && !gone) return "nobody knows that it was not heard";
    if (memory[0] == tag) return "a word is left";
    if (memory[1] == tag) return "a mark is left";
    return nullptr;
}

}  // namespace

int main(int argc, char** argv) {
    const int trials = argc > 1 ? atoi(argv[1]) : 1000;
    for (int i = 0; i < trials; ++i) {
        rng.seed(i + 1);
        tag = (uint64_t)rng() << 32 | rng();
        for (uint64_t& m : memory) m = rng() % 2 ? ~tag : (uint64_t)rng() << 32 | rng();
        for (int l = 0; l < 4; ++l)
            if (const char* why = play()) {
                printf("trial %d, launch %d: %s\n", i, l, why);
                return 1;
            }
    }
    printf("%d trials\n", trials);
    return 0;
}

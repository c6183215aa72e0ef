// Plays pairs of calls of sequential acceptance on two streams (csrc/resample_plan.h): an XCD starts the workgroups of a launch in
// order as CUs have room, but which stream it serves first is drawn anew for every XCD and changes on the way; a team goes on, and
// leaves, once all its workgroups have started; a node's workgroup leaves by itself, and the one that follows a sequence's decisions
// once all of them have started.  Prints the first pair that gets stuck, exit status 1.
// Usage: resample_plan TRIALS B N V [B N V ...]: every pair of the calls, TRIALS times each
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "resample_plan.h"

using namespace s4c;

namespace {

constexpr int kXcds = 8, kCus = 32;            // CUs of an XCD; two places on each, of which a team kernel's workgroup takes one or both

struct Wait { int team, cu; };
struct Stream {
    int B, N, G, size, next = 0, n = 0;        // size: places that a workgroup takes; next: first sequence of the next launch
    bool rows;
    ResampleLaunch l;
    std::vector<int> head, started;            // per XCD: workgroups started; per sequence of the launch: likewise
    std::vector<std::vector<Wait>> here;       // per XCD: started and not gone
    bool left = false;                         // all of the launch's workgroups have

    Stream(int B_, int N_, int V) : B(B_), N(N_) {
        rows = resample_by_rows(B, N, V, kXcds * kCus);
        G = rows ? 1 : resample_team(B, V, kXcds * kCus);
        const int iters = resample_iters((resample_blocks(V) + G - 1) / G);
        size = resample_per_cu(iters) > 1 ? 1 : 2;
        l = resample_launch(B, G, iters, kXcds * kCus);
        launch();
    }
    int grid() const { return rows ? B * (N + 1) : resample_grid(n, G, l.groups); }
    int awaited() const { return rows ? N : G; }
    ResampleMember member(int i) const {
        if (!rows) return resample_member(i, G, l.groups);
        return i < B * N ? ResampleMember{i / N, i % N} : ResampleMember{i - B * N, N};
    }
    void launch() {
        n = B - next < l.sequences ? B - next : l.sequences;
        next += n;
        head.assign(kXcds, 0);
        started.assign(n, 0);
        here.assign(kXcds, {});
        left = false;
    }
    bool done() const { return left && next == B; }
};

bool play(Stream (&s)[2], std::mt19937& rng) {
    std::vector<std::vector<int>> room(kXcds, std::vector<int>(kCus, 2));
    int first[kXcds];
    for (int& f : first) f = rng() & 1;
    while (!s[0].done() || !s[1].done()) {
        bool moved = false;
        for (int x = 0; x < kXcds; ++x)
            for (int k = 0; k < 2; ++k) {
                Stream& a = s[first[x] ^ k];
                for (;;) {                                             // one after the other, while there is room
                    const int i = a.head[x] * kXcds + x;
                    if (i >= a.grid()) break;
                    const ResampleMember m = a.member(i);
                    int cu = -1;
                    for (int c = 0; c < kCus; ++c)
                        if (room[x][c] >= a.size && (cu < 0 || room[x][c] > room[x][cu])) cu = c;
                    if (m.sequence < a.n) {
                        if (cu < 0) break;
                        if (!a.rows || m.g == a.N) {
                            room[x][cu] -= a.size;
                            a.here[x].push_back({m.sequence, cu});
                        }
                        if (!a.rows || m.g < a.N) ++a.started[m.sequence];
                    }
                    ++a.head[x];
                    moved = true;
                }
            }
        for (Stream& a : s) {
            for (int x = 0; x < kXcds; ++x) {
                std::vector<Wait> left;
                for (const Wait& w : a.here[x])
                    if (a.started[w.team] == a.awaited()) { room[x][w.cu] += a.size; moved = true; }
                    else left.push_back(w);
                a.here[x] = left;
            }
            a.left = true;
            for (int x = 0; x < kXcds; ++x) a.left &= a.head[x] * kXcds + x >= a.grid() && a.here[x].empty();
            if (a.left && a.next < a.B) { a.launch(); moved = true; }
        }
        if (!moved) return false;
        if (rng() % 4 == 0) first[rng() % kXcds] ^= 1;
    }
    return true;
}

}  // namespace

int main(int argc, char** argv) {
    const int trials = atoi(argv[1]);
    std::vector<std::vector<int>> calls;
    for (int i = 2; i + 2 < argc; i += 3) calls.push_back({atoi(argv[i]), atoi(argv[i + 1]), atoi(argv[i + 2])});
    std::mt19937 rng(1);
    for (const auto& p : calls)
        for (const auto& q : calls)
            for (int t = 0; t < trials; ++t) {
                Stream s[2] = {Stream(p[0], p[1], p[2]), Stream(q[0], q[1], q[2])};
                for (const Stream& a : s) {                            // every workgroup of every team exactly once
                    const int per = a.rows ? a.N + 1 : a.G;
                    std::vector<int> seen(a.n * per, 0);
                    for (int i = 0; i < a.grid(); ++i) {
                        const ResampleMember m = a.member(i);
                        if (m.sequence < a.n && seen[m.sequence * per + m.g]++) return printf("twice: %d x %d\n", a.B, per), 1;
                    }
                    for (int n : seen)
                        if (n != 1) return printf("never: %d x %d\n", a.B, per), 1;
                }
                if (!play(s, rng)) {
                    printf("stuck: %d x %d, V %d beside %d x %d, V %d\n", p[0], p[1], p[2], q[0], q[1], q[2]);
                    return 1;
                }
            }
    return 0;
}

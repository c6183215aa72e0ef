// Plays verification steps of one launch on several streams: an XCD starts the workgroups of a launch in order while a CU of it is free, but which
// stream it serves first is drawn anew for every XCD and changes on the way.  Attention and scanning workgroups leave by
// themselves (those that merge wait for workgroups that have started: attn_meet.h), collectors wait for both, copiers for the
// collectors; each is taken to need a CU to itself.  Prints the first launches that get stuck, exit status 1.
// Usage: attn_waiting TRIALS OVERLAP B Hkv ATTENTION SCAN [...]: OVERLAP launches at a time of those described, drawn TRIALS times,
// and that many of each
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "attn_division.h"

using namespace s4c;

namespace {

constexpr int kXcds = 8, kCus = 32, kMostCopiers = 8;
enum Role { kWork, kScan, kCollect, kCopy, kRoles };
typedef std::vector<int> Call;                                  // B, Hkv, workgroups that attend, workgroups that scan

struct Launch {
    std::vector<Role> grid;
    int total[kRoles] = {}, left[kRoles] = {};                 // workgroups of a role, and how many have gone
    std::vector<int> head = std::vector<int>(kXcds, 0);         // per XCD: workgroups started
    std::vector<std::vector<Role>> here = std::vector<std::vector<Role>>(kXcds);
    explicit Launch(const Call& x) {
        const int heads = heads_of_copier(x[0], x[1], kMostCopiers, kXcds * kCus), copiers = copiers_of(x[1], heads);
        if (copiers > kMostCopiers || copiers * heads < x[1]) exit(2);
        const int n[kRoles] = {x[2], x[3], x[0], x[0] * copiers};
        for (int r = 0; r < kRoles; ++r) {
            total[r] = n[r];
            grid.insert(grid.end(), n[r], (Role)r);
        }
    }
    bool gone(Role r) const { return left[r] == total[r]; }
    bool goes(Role r) const {
        return r == kWork || r == kScan || (r == kCollect && gone(kWork) && gone(kScan)) || (r == kCopy && gone(kCollect));
    }
    bool done() const { return gone(kWork) && gone(kScan) && gone(kCollect) && gone(kCopy); }
};

bool play(std::vector<Launch> s, std::mt19937& rng) {
    const int K = (int)s.size();
    int room[kXcds], first[kXcds];
    for (int x = 0; x < kXcds; ++x) room[x] = kCus, first[x] = rng() % K;
    auto done = [&] {
        for (const Launch& l : s)
            if (!l.done()) return false;
        return true;
    };
    while (!done()) {
        bool moved = false;
        for (int x = 0; x < kXcds; ++x)
            for (int k = 0; k < K; ++k) {
                Launch& a = s[(first[x] + k) % K];
                for (int i; room[x] > 0 && (i = a.head[x] * kXcds + x) < (int)a.grid.size(); ++a.head[x], --room[x], moved = true)
                    a.here[x].push_back(a.grid[i]);
            }
        for (Launch& a : s)
            for (int x = 0; x < kXcds; ++x) {
                std::vector<Role> stay;
                for (Role r : a.here[x])
                    if (a.goes(r)) ++a.left[r], ++room[x], moved = true;
                    else stay.push_back(r);
                a.here[x] = stay;
            }
        if (!moved) return false;
        if (rng() % 4 == 0) first[rng() % kXcds] = rng() % K;
    }
    return true;
}

}  // namespace

int main(int argc, char** argv) {
    const int trials = atoi(argv[1]), overlap = atoi(argv[2]);
    std::vector<Call> calls;
    for (int i = 3; i + 3 < argc; i += 4) calls.push_back({atoi(argv[i]), atoi(argv[i + 1]), atoi(argv[i + 2]), atoi(argv[i + 3])});
    std::mt19937 rng(1);
    for (int t = 0; t < trials * (int)(calls.size() + 1); ++t) {
        std::vector<Launch> s;
        std::vector<int> which;
        for (int k = 0; k < overlap; ++k) {
            which.push_back(t < trials * (int)calls.size() ? t / trials : rng() % calls.size());
            s.emplace_back(calls[which.back()]);
        }
        if (!play(s, rng)) {
            printf("stuck:");
            for (int i : which) printf(" %d x %d", calls[i][0], calls[i][1]);
            printf("\n");
            return 1;
        }
    }
    return 0;
}

// Plays pairs of attention launches on two streams: an XCD starts the workgroups of a launch in order while a CU of it is free, but which
// stream it serves first is drawn anew for every XCD and changes on the way.  Attention and scanning workgroups leave by
// themselves, merging workgroups wait for the attention, collectors for both, copiers for the collectors; each is taken to need a
// CU to itself.  Prints the first pair that gets stuck, exit status 1.
// Usage: attn_waiting TRIALS B Hkv MERGING ATTENTION SCAN [...]: every pair of the launches, TRIALS times each.  MERGING: workgroups that would
// merge in one turn; SCAN 0: attention alone
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "attn_division.h"

using namespace s4c;

namespace {

constexpr int kXcds = 8, kCus = 32, kMostCopiers = 8;
enum Role { kWork, kScan, kCollect, kMerge, kCopy, kRoles };

struct Launch {
    std::vector<Role> grid;
    int total[kRoles] = {}, left[kRoles] = {};                 // workgroups of a role, and how many have gone
    std::vector<int> head = std::vector<int>(kXcds, 0);         // per XCD: workgroups started
    std::vector<std::vector<Role>> here = std::vector<std::vector<Role>>(kXcds);
    Launch(const int* x) {
        const int B = x[4] > 0 ? x[0] : 0, Hkv = x[1];
        const AttnWaiting w = plan_waiting(x[2], B, Hkv, kMostCopiers, kXcds * kCus);
        const int copiers = B > 0 ? copiers_of(Hkv, w.heads) : 0;
        if (copiers > kMostCopiers || (long long)copiers * w.heads < (B > 0 ? Hkv : 0) || (x[2] > 0 && w.merging < 1)) exit(2);
        const int n[kRoles] = {x[3], x[4], B, w.merging, B * copiers};
        for (int r = 0; r < kRoles; ++r) {
            total[r] = n[r];
            grid.insert(grid.end(), n[r], (Role)r);
        }
    }
    bool gone(Role r) const { return left[r] == total[r]; }
    bool goes(Role r) const {
        return r == kWork || r == kScan || (r == kMerge && gone(kWork)) || (r == kCollect && gone(kWork) && gone(kScan)) || (r == kCopy && gone(kCollect));
    }
    bool done() const { return gone(kWork) && gone(kScan) && gone(kCollect) && gone(kMerge) && gone(kCopy); }
};

bool play(Launch* s, std::mt19937& rng) {
    int room[kXcds], first[kXcds];
    for (int x = 0; x < kXcds; ++x) room[x] = kCus, first[x] = rng() & 1;
    while (!s[0].done() || !s[1].done()) {
        bool moved = false;
        for (int x = 0; x < kXcds; ++x)
            for (int k = 0; k < 2; ++k) {
                Launch& a = s[first[x] ^ k];
                for (int i; room[x] > 0 && (i = a.head[x] * kXcds + x) < (int)a.grid.size(); ++a.head[x], --room[x], moved = true)
                    a.here[x].push_back(a.grid[i]);
            }
        for (int k = 0; k < 2; ++k)
            for (int x = 0; x < kXcds; ++x) {
                std::vector<Role> stay;
                for (Role r : s[k].here[x])
                    if (s[k].goes(r)) ++s[k].left[r], ++room[x], moved = true;
                    else stay.push_back(r);
                s[k].here[x] = stay;
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
    for (int i = 2; i + 4 < argc; i += 5) calls.push_back({atoi(argv[i]), atoi(argv[i + 1]), atoi(argv[i + 2]), atoi(argv[i + 3]), atoi(argv[i + 4])});
    std::mt19937 rng(1);
    for (const auto& p : calls)
        for (const auto& q : calls)
            for (int t = 0; t < trials; ++t) {
                Launch s[2] = {Launch(p.data()), Launch(q.data())};
                if (!play(s, rng)) {
                    printf("stuck: %d x %d, %d merging beside %d x %d, %d merging\n", p[0], p[1], p[2], q[0], q[1], q[2]);
                    return 1;
                }
            }
    return 0;
}

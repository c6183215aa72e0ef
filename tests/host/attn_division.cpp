// Plays every workgroup of attention launches through csrc/attn_division.h on the host, over random shapes and sequence
// lengths, and checks what the kernels and the merge rely on:
//   every key tile of every unit is walked exactly once, and no workspace slot is written twice;
//   a unit that one team covered alone is not merged, and a unit that is merged was written by no team alone;
//   every part that the merge reads was written by this call, and it reads every part of its unit (equal runs: a region for
//   every team; balanced shares: slots, which teams note).
// Usage: attn_division split|balanced LAUNCHES; prints the first wrong launch and their number, exit status 1 if any.
//        attn_division plan B Hkv N M max_cache_len ROWS KEYS PER_CU WIDE CUS; prints the plan's teams, split and parts
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <random>
#include <vector>

#include "attn_division.h"

using namespace s4c;

namespace {

struct Args {
    int B, Hkv, N, M, S_cap, max_cache_len, teams, split, tile_keys, tile_shift;
    int32_t* ws_parts;
};

struct Order;
struct Lens {
    typedef ::Order Order;
    const std::vector<int>* len;
    int tiles(const Args& a, int b) const { return work::tiles_of(a, work::usable(a, (*len)[b])); }
};
struct Order {
    int total = 0;
    std::vector<int> first;
    Order(const Args& a, const Lens& lens) {
        for (int b = 0; b < a.B; ++b) {
            first.push_back(total);
            total += lens.tiles(a, b) * a.Hkv;
        }
    }
    int begin(const Args&, const Lens&, int b) const { return first[b]; }
    int seq_of(const Args& a, const Lens&, int x) const {
        int b = a.B - 1;
        while (first[b] > x) --b;
        return b;
    }
};

const char* wrong(const Args& a, const AttnDivision& d, const Lens& lens) {
    const int units = a.B * a.Hkv, kNobody = -1, kEmpty = -2;
    if (a.split > 32) return "more runs than a wave has bits and words for";
    std::vector<std::vector<int>> walked(units);
    for (int u = 0; u < units; ++u) walked[u].assign(lens.tiles(a, u / a.Hkv), 0);
    std::vector<int> whole(units, 0), slots((size_t)a.teams * 2, kNobody), parts_of(units, 0);
    for (int i = 0; i < 2 * units; ++i) a.ws_parts[i] = -7;
    std::vector<int> seen(a.teams, 0);
    for (int wg = 0; wg < (a.teams + 7) / 8 * 8; ++wg) {
        const int team = work::team_id(a, wg & 7, wg >> 3);
        if (team < a.teams && seen[team]++) return "a team number is used twice";
        work::Walk w = a.split > 0 ? work::walk_run(a, lens, team) : work::walk_share(a, lens, team);
        if (w.b < 0 && work::leaves_empty(a, team)) slots[team] = kEmpty;
        while (w.b >= 0) {
            const int u = w.b * a.Hkv + w.kvh;
            if (w.b >= a.B || w.kvh >= a.Hkv || w.tile < 0 || w.tile >= w.tile_end || w.tile_end > (int)walked[u].size())
                return "a segment outside its unit";
            for (int t = w.tile; t < w.tile_end; ++t) ++walked[u][t];
            if (a.split == 0) work::note_parts(a, team, w);
            if (work::walk_is_whole(a, w)) {
                ++whole[u];
            } else {
                int& s = slots[a.split > 0 ? (size_t)team : work::part_row(a, team, work::part_slot(w)) / a.M];
                if (s != kNobody) return "a workspace slot is written twice";
                s = u;
                ++parts_of[u];
            }
            w = work::walk_next(a, lens, w);
        }
    }
    for (int t = 0; t < a.teams; ++t)
        if (!seen[t]) return "a team has no workgroup";
    for (int u = 0; u < units; ++u) {
        for (int n : walked[u])
            if (n != 1) return "a tile is not walked once";
        if (d.split == 1) {                                  // no merge is launched
            if (whole[u] != 1) return "nobody writes a unit's output";
            continue;
        }
        if (a.split > 0) {                                   // every team of the unit leaves a part, and all are merged
            int read = 0;
            for (int k = 0; k < a.split; ++k) {
                const int s = slots[u * a.split + k];
                if (s != u && s != kEmpty) return "the merge reads a part that this call did not write for the unit";
                read += s == u;
            }
            if (whole[u] || read != parts_of[u]) return "the merge misses a part";
            continue;
        }
        const work::Parts p(a, u);
        if (p.first < 0 || p.last < p.first || p.last >= a.teams) return "a unit's teams were not noted";
        if (p.first == p.last) {
            if (whole[u] != 1 || parts_of[u]) return "nobody writes a unit's output";
            continue;
        }
        if (whole[u]) return "a unit that is written already is merged";
        int read = 0;
        for (int t = p.first; t <= p.last; ++t) {
            const int s = slots[work::part_row(a, t, p.slot(t)) / a.M];
            if (s != u && s != kEmpty) return "the merge reads a part that this call did not write for the unit";
            read += s == u;
        }
        if (read != parts_of[u]) return "the merge misses a part";
    }
    return nullptr;
}

}  // namespace

int main(int argc, char** argv) {
    if (argc == 12 && !strcmp(argv[1], "plan")) {
        int n[10];
        for (int i = 0; i < 10; ++i) n[i] = atoi(argv[2 + i]);
        const AttnDivision d = plan_division(n[0], n[1], n[2], n[3], n[4], AttnTile{n[5], n[6], n[7], n[8] != 0}, n[9]);
        printf("%d %d %d\n", d.teams, d.split, d.parts);
        return 0;
    }
    const bool split = argc > 1 && !strcmp(argv[1], "split");
    const int launches = argc > 2 ? atoi(argv[2]) : 1000;
    std::mt19937 rng(20250614);
    auto pick = [&](int lo, int hi) { return (int)(lo + rng() % (unsigned)(hi - lo + 1)); };
    auto log_pick = [&](int lo, int hi) {
        const double x = std::uniform_real_distribution<double>(std::log((double)lo), std::log((double)hi + 1))(rng);
        return (int)std::exp(x);
    };
    // rows, keys and workgroups per CU of the kernels' configurations
    const AttnTile tiles[] = {{128, 64, 1, true}, {128, 64, 2, false}, {256, 64, 1, true}, {256, 64, 1, false}, {32, 32, 1, true}, {32, 32, 1, false}, {32, 32, 2, false},
                              {64, 32, 1, false}, {64, 32, 2, true}, {64, 32, 2, false}};
    int played = 0, bad = 0, divided = 0;
    while (played < launches) {
        Args a;
        a.B = log_pick(1, 80);
        a.Hkv = log_pick(1, 40);
        a.N = rng() % 4 ? pick(1, 128) : pick(1, 20);
        const AttnTile t = tiles[rng() % 10];
        const int G = t.rows <= 64 && rng() % 2 ? 1 : log_pick(1, 16);
        a.M = a.N * G;
        a.max_cache_len = rng() % 8 ? log_pick(1, 40000) : 0;
        a.S_cap = a.max_cache_len + pick(0, 200);
        const AttnDivision d = plan_division(a.B, a.Hkv, a.N, a.M, a.max_cache_len, t, rng() % 4 ? 256 : pick(1, 38) * 8);
        if ((d.split > 0) != split) continue;
        ++played;
        divided += d.split != 1;
        a.teams = d.teams;
        a.split = d.split;
        a.tile_keys = t.keys;
        a.tile_shift = t.keys == 64 ? 6 : 5;
        std::vector<int32_t> parts((size_t)a.B * a.Hkv * 2);
        a.ws_parts = parts.data();
        // full, ragged, short or empty sequences under the same max_cache_len, some of an invalid length
        std::vector<int> len(a.B);
        const int regime = rng() % 5;
        for (int& n : len) {
            const int most = a.max_cache_len;
            n = regime == 0 ? most : regime == 1 ? pick(0, most) : regime == 2 ? pick(0, most < 64 ? most : 64) : regime == 3 ? 0 : log_pick(1, most + 1) - 1;
            const int special = rng() % 16;
            if (special == 0) n = 0;
            if (special == 1) n = rng() % 2 ? -1 : most + 1;
        }
        if (const char* why = wrong(a, d, Lens{&len})) {
            if (!bad++) {
                printf("B %d Hkv %d N %d M %d max_cache_len %d tile %d x %d teams %d split %d: %s; lengths", a.B, a.Hkv, a.N, a.M,
                       a.max_cache_len, t.rows, t.keys, a.teams, a.split, why);
                for (int n : len) printf(" %d", n);
                printf("\n");
            }
        }
    }
    printf("%d launches, %d divided, %d wrong\n", played, divided, bad);
    return bad ? 1 : 0;
}

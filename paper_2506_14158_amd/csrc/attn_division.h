// How a launch of the attention kernels divides its work: the arithmetic alone, which also compiles for the host
// (tests/host/attn_division.cpp plays every workgroup of a launch through it).
//
// The work of one (sequence, KV head) "unit" is a run of key tiles: its prefix tiles, then its tree tiles.  A
// team is the workgroups that walk the same keys for the row tiles of one unit (a single workgroup when all query
// rows fit one).  Two divisions:
//   split     every unit's tiles (of its ACTUAL length) are cut into `split` equal runs, a team each; a team walks
//             one run.  split = 1: nothing to merge.  For launches whose teams all fit on the chip at once.
//   balanced  (split = 0) all units' tiles are laid end to end, sequence by sequence with their actual lengths, and
//             the teams take equal consecutive shares (sizes differ by one tile).  A share may end inside a unit.  Equal
//             shares are what keeps every CU busy to the end: 104 units on 256 CUs leave 48 of them idle at two runs per
//             unit, and with ragged lengths the rest wait for the longest sequence.
// A part of a unit that several teams share goes to the workspace unnormalised, and a unit's parts are combined in order: equal
// runs by attn_parts.h, balanced shares by attn_merge.h.
// The shares are a function of the shape and of cache_len, so results are deterministic for given inputs.
//
// `A` is AttnArgs, or what a host program has with the same members; `L` tells the sequences' lengths, L::Order their
// end-to-end order (attn_work.h has the kernels').
#pragma once
#include <stddef.h>
#include <stdint.h>

#if defined(__HIPCC__)
#define S4C_WORK __device__ __forceinline__
#define S4C_UNIFORM(x) __builtin_amdgcn_readfirstlane(x)
#else
#define S4C_WORK inline
#define S4C_UNIFORM(x) (x)
#endif

namespace s4c {

// What one workgroup of the kernel for a shape takes: query rows, keys per tile, and how many fit on a CU; `wide`: 16-bit
// data of head size 128; part_keys: waves that share the columns of a row when it writes.
struct AttnTile { int rows, keys, per_cu; bool wide; int part_keys = 1; };

constexpr int kMostRuns = 24;              // of a unit; up to 32 (attn_parts.h)

struct AttnDivision {
    int teams, split, mtiles;
    int parts;                 // most parts a unit is divided into when no sequence is shorter than max_cache_len
};

// How the key tiles of a shape are divided between workgroups: a fixed function of its sizes and max_cache_len, so that
// the workspace query and the launch agree.  M: query rows of a unit; cus: compute units of the device.
inline AttnDivision plan_division(int B, int Hkv, int N, int M, int max_cache_len, AttnTile t, int cus) {
    AttnDivision p;
    p.mtiles = (M + t.rows - 1) / t.rows;
    const long long slots = (long long)cus * t.per_cu;
    const long long units = (long long)B * Hkv;
    const long long tiles = (max_cache_len + t.keys - 1) / t.keys + (N + t.keys - 1) / t.keys;   // of the longest unit
    // Teams: one round of the chip, a team's workgroups all on one XCD (an eighth of it); fewer when a share would get
    // shorter than kMinKeys keys, below which a part's fixed costs (prologue, partial results, its share of the merge)
    // outweigh what the extra workgroups stream, but never fewer than units for that: whole units have no parts, and several
    // short ones in a row are a chain (512 units of 20 keys + 20 nodes: 28.0 us on 192 teams, 8.6 on 512).  At most
    // kMostRuns per unit.
    const long long kMinKeys = 256, per_xcd = slots / 8;
    long long teams = per_xcd >= p.mtiles ? per_xcd / p.mtiles * 8 : 8;
    long long most = units * tiles * t.keys / kMinKeys;
    if (most < units) most = units;
    if (teams > most) teams = most;
    if (teams > units * kMostRuns) teams = units * kMostRuns;
    // A share that ends inside a unit has a second segment to start and finish, which costs as much as kSwitchKeys keys:
    // whole numbers of runs per unit where the longer runs cost less than that, and where no unit would get a second.
    //
    // And a unit that is not divided has no parts, of as many rows as a workgroup has, to write and to merge, nor a merge at
    // all if no unit is.  Undivided units leave part of the chip's (last) round idle, `idle` keys of each team's time.  Whole
    // and divided, us (where they meet depends on the rows that go through the workspace):
    //   prefixes below kShortKeys, unless most of the chip would be idle: 160 units, 60 rows, 500 keys 15.7 and 20.2; 24 units, 80 rows 17.8 and 15.8
    //   the kernel with 32-key tiles, two workgroups a CU, at three units on four CUs (it waits for memory, of which a workgroup that has a
    //     CU to itself gets more): 224 units, 60 rows, 1200 keys 27.1 and 32.8, 2600 keys 60.6 and 60.9; 20 rows, 1200 keys 26.2 and 29.2,
    //     2600 keys 57.3 and 53.5; 320 units, 60 rows, 1200 keys 38.4 and 47.2; a step of 240 units of 5 rows, 8253 keys 221 and 192
    //   the kernel with 64-key tiles, one round: 136 units, 240 rows, 500 keys 24.6 and 40.0, 5000 keys 131 and 120; 200 units, 80 rows,
    //     1200 keys 31.1 and 39.5 (at lengths between half and all of 2184, 88 rows: a step of 66 and 60)
    //   more than one round: 1280 units, 60 rows, 1200 keys 164 and 180; 544 units of 4800 keys 291 and 269 (20 rows: 285 and 242);
    //     264 units, 80 rows, 150 keys 23.9 and 27.2, 300 keys 31.1 and 30.6, 1200 keys 58.9 and 45.8
    // (Several rounds of equal shares that are whole units need no merge either, and load a unit behind the last one.)
    // fp32 data and head size 64 do more arithmetic per byte, and shares win from short prefixes on: 136 units, 80 rows, 800 keys
    // of fp32 130 and 87 (640 units of head size 64, 40 keys + 20 nodes: 18.1 and 19.9).
    const long long kSwitchKeys = 256, kShortKeys = 512;
    const long long rounds = (units + teams - 1) / teams, idle = tiles * t.keys * (rounds * teams - units) / (rounds * teams);
    const long long rows = M < t.rows ? M : t.rows;
    long long split = 0;
    // beyond the kernels' 32-bit tile numbers, or offsets in the parts of a unit (8 M 128 bytes each: PartRegion)
    if (units * tiles > 0x3FFFFFFFll || M > (int)(0xFFFFFFFFu / (8u * 128u * kMostRuns))) split = 1;
    else if (teams >= units) {
        const long long q = teams / units;
        if ((tiles + q - 1) / q * t.keys <= units * tiles * t.keys / teams + kSwitchKeys) split = q;
        if (t.wide && (max_cache_len < kShortKeys ? units * p.mtiles * 8 > cus
                       : t.keys == 32             ? t.per_cu == 2 && units * 4 >= cus * 3ll && idle <= 400 + 50 * rows
                                                  : q == 1 && idle <= 200 + 5 * rows / 2))
            split = 1;
    } else if (units * p.mtiles <= slots || (units % teams != 0 && (tiles * t.keys <= 128 || (t.wide && idle * 16 <= rows * (t.keys == 32 ? 256 : 28))))) {
        split = 1;
    }
    p.split = (int)split;
    p.teams = (int)(split > 0 ? units * split : teams < 1 ? 1 : teams);
    if (split == 1) {
        p.parts = 1;
    } else {
        const long long share = units * tiles / p.teams;                     // >= 1: kMinKeys is several tiles
        p.parts = (int)(split > 0 ? split : share % tiles == 0 && units * tiles % p.teams == 0 ? 1 : (tiles + share - 1) / share + 1);
    }
    return p;
}

// Where a team of a launch of equal runs leaves its part: a region with room for 2 M rows of D floats, of which the slabs (8 columns of a
// row block of 32; a lane's 16 bytes are 4 columns of a row) need M.  In the other half lie the rows' (maximum in log2 units, sum) for every
// wave that wrote columns of its own, 4 of them at most, and behind them a word for each tile of the unit's rows (attn_meet.h).
template <int D>
struct PartRegion {
    static S4C_WORK uint32_t bytes(int M) { return 8u * M * D; }
    static S4C_WORK uint32_t slab(int M, int block, int s, int lane) {
        const int rows = M - 32 * block < 32 ? M - 32 * block : 32;
        return 4u * (32 * block * D + ((2 * s + (lane >> 5)) * rows + (lane & 31)) * 4);
    }
    static S4C_WORK uint32_t stats(int M, int block, int key, int lane) { return 4u * M * D + 8u * (key * M + 32 * block + (lane & 31)); }
    static S4C_WORK uint32_t word(int M, int mt) { return 4u * M * D + 4 * 8u * M + 8u * mt; }
};

// Workgroups of a step's only launch that wait for others of it: a collector for each sequence, and its copiers.  Every XCD starts a launch's
// workgroups in order, but which of several streams it serves first is its own affair: with one XCD full of waiting workgroups of
// some calls and another full of others', nobody's attention would be started until the waits run out.  Four calls can run at once (the hardware
// queues that a process has unless it asks for more), so the waiting workgroups of three leave a CU of an XCD to the fourth: a launch
// has at most a third of an XCD's CUs but one waiting, 80 of 256 altogether.  (So many that eight calls could overlap, 32, and one copier for each of 12
// sequences of 32 heads: 15.7 -> 16.5 us.)
// Returns the KV heads of a copier.
inline int copiers_of(int Hkv, int heads) { return (Hkv + heads - 1) / heads; }
// sequences: at most an eighth of the CUs; most: copiers of a sequence
inline int heads_of_copier(int sequences, int Hkv, int most, int cus) {
    const int waiting = (cus / 8 - 1) / 3 * 8;
    int copiers = waiting / sequences - 1;
    copiers = copiers < 1 ? 1 : copiers > most ? most : copiers;
    return (Hkv + copiers - 1) / copiers;
}

namespace work {

// prefix length used for the division: an out-of-range cache_len (the sequence is flagged) counts as empty
template <class A>
S4C_WORK int usable(const A& a, int P) { return (P < 0 || P > a.max_cache_len || P > a.S_cap) ? 0 : P; }
template <class A>
S4C_WORK int tiles_of(const A& a, int P) {
    return ((P + a.tile_keys - 1) >> a.tile_shift) + ((a.N + a.tile_keys - 1) >> a.tile_shift);
}

// The team that runs on slot k of an XCD: neighbours in the end-to-end order share an XCD, so an XCD's workgroups
// walk one eighth of the cache and not pieces of all of it.
template <class A>
S4C_WORK int team_id(const A& a, int xcd, int k) { return xcd * ((a.teams + 7) >> 3) + k; }

// Team g's share begins at tile floor(g total / teams): equal shares, and whole units where the numbers divide.
struct Shares {
    int total, teams, per, rem;
    S4C_WORK Shares(int total_, int teams_) : total(total_), teams(teams_), per(total_ / teams_), rem(total_ % teams_) {}
    S4C_WORK int begin(int g) const { return g * per + (int)((unsigned)g * (unsigned)rem / (unsigned)teams); }   // teams < 2^16
};

// One team's walk over its share: a segment is a run of tiles [tile, tile_end) of one unit.  The kernels keep two: one
// runs ahead and issues loads, one follows and multiplies, so that the loads never pause where a segment ends.
struct Walk {
    int b, kvh;            // unit of the current segment; b < 0: no segment
    int tiles;             // tiles of that unit
    int tile, tile_end;    // the segment
    int left;              // tiles of the share after this segment
};

// ... of a launch of equal runs, or of whole units (split = 1): the only segment of team's share
template <class A, class L>
S4C_WORK Walk walk_run(const A& a, const L& lens, int team) {
    Walk w = {-1, 0, 0, 0, 0, 0};
    if (team >= a.teams) return w;
    const int unit = team / a.split, k = team - unit * a.split;
    w.b = unit / a.Hkv;
    w.kvh = unit - w.b * a.Hkv;
    w.tiles = lens.tiles(a, w.b);
    const int run = (w.tiles + a.split - 1) / a.split;
    w.tile = k * run;
    w.tile_end = w.tiles < w.tile + run ? w.tiles : w.tile + run;
    if (w.tile >= w.tile_end) w.b = -1;         // (an empty run: see leaves_empty)
    return w;
}
// ... of a balanced launch: the first segment
template <class A, class L>
S4C_WORK Walk walk_share(const A& a, const L& lens, int team) {
    Walk w = {-1, 0, 0, 0, 0, 0};
    if (team >= a.teams) return w;
    const typename L::Order order(a, lens);
    // Fewer tiles than teams (short sequences under a large max_cache_len): as many teams as tiles, so that every team
    // between the one that begins a unit and the one that ends it has a part of it.
    const Shares s(order.total, a.teams < order.total ? a.teams : order.total);
    if (team >= s.teams) return w;
    const int x = S4C_UNIFORM(s.begin(team)), n = S4C_UNIFORM(s.begin(team + 1)) - x;
    if (n <= 0) return w;
    w.b = order.seq_of(a, lens, x);
    w.tiles = lens.tiles(a, w.b);
    const int first = order.begin(a, lens, w.b);
    w.kvh = S4C_UNIFORM((x - first) / w.tiles);
    w.tile = (x - first) - w.kvh * w.tiles;
    w.tile_end = w.tiles < w.tile + n ? w.tiles : w.tile + n;
    w.left = n - (w.tile_end - w.tile);
    return w;
}

// (by value: a walk stays in scalar registers)
template <class A, class L>
S4C_WORK Walk walk_next(const A& a, const L& lens, const Walk w) {
    Walk n = w;
    n.b = -1;
    if (w.left > 0) {
        const bool next_seq = w.kvh + 1 == a.Hkv;
        n.b = next_seq ? w.b + 1 : w.b;
        n.kvh = next_seq ? 0 : w.kvh + 1;
        n.tiles = lens.tiles(a, n.b);
        n.tile = 0;
        n.tile_end = n.tiles < w.left ? n.tiles : w.left;
        n.left = w.left - n.tile_end;
    }
    return n;
}

// This segment is the unit's output rather than a part of it (evaluate before the walk's `tile` moves): it covers the
// unit, and the merge will not look at it.  A split launch of several runs merges every unit: one of a single tile (an
// empty prefix, a flagged sequence) is one part and empty ones.
template <class A>
S4C_WORK bool walk_is_whole(const A& a, const Walk& w) { return a.split <= 1 && w.tile == 0 && w.tile_end == w.tiles; }
// Workspace slot of a part in a balanced launch: a team leaves at most one part that ends a unit or lies inside it (slot 0) and one
// that begins a unit (slot 1).
S4C_WORK int part_slot(const Walk& w) { return w.tile == 0 ? 1 : 0; }
template <class A>
S4C_WORK size_t part_row(const A& a, int team, int slot) { return ((size_t)team * 2 + slot) * a.M; }

// A team without tiles in a split launch leaves empty parts (sum 0), so that who merges need not know how many teams had
// some.
template <class A>
S4C_WORK bool leaves_empty(const A& a, int team) { return a.split > 1 && team < a.teams; }

// Tells the merge which teams share a unit (balanced launches): the team that begins it and the team that ends it.
template <class A>
S4C_WORK void note_parts(const A& a, int team, const Walk& w) {
    const size_t unit = (size_t)w.b * a.Hkv + w.kvh;
    if (w.tile == 0) a.ws_parts[2 * unit] = team;
    if (w.tile_end == w.tiles) a.ws_parts[2 * unit + 1] = team;
}

// The teams whose parts make up a unit of a balanced launch, as they noted: slot 1 of the first one, slot 0 of the others; one team
// alone has written the unit's output itself.
struct Parts {
    int first, last;
    template <class A>
    S4C_WORK Parts(const A& a, int unit) : first(a.ws_parts[2 * unit]), last(a.ws_parts[2 * unit + 1]) {}
    S4C_WORK int slot(int team) const { return team == first ? 1 : 0; }
};

}  // namespace work
}  // namespace s4c

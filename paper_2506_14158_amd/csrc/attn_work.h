// How a launch of the attention kernels divides its work (device side of plan_attn in s4c_api.hip).
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
// A part of a unit that several teams share goes to the workspace unnormalised; attn_merge_kernel combines a unit's
// parts in order.
// The shares are a function of the shape and of cache_len, so results are deterministic for given inputs.
#pragma once
#include "common.h"

namespace s4c {
namespace work {

// prefix length used for the division: an out-of-range cache_len (the sequence is flagged) counts as empty
__device__ __forceinline__ int usable(const AttnArgs& a, int P) { return (P < 0 || P > a.max_cache_len || P > a.S_cap) ? 0 : P; }
__device__ __forceinline__ int tiles_of(const AttnArgs& a, int P) {
    return ((P + a.tile_keys - 1) >> a.tile_shift) + ((a.N + a.tile_keys - 1) >> a.tile_shift);
}

// The team that runs on slot k of an XCD: neighbours in the end-to-end order share an XCD, so an XCD's workgroups
// walk one eighth of the cache and not pieces of all of it.
__device__ __forceinline__ int team_id(const AttnArgs& a, int xcd, int k) { return xcd * ((a.teams + 7) >> 3) + k; }

// Every function below is called by whole wavefronts and returns wave-uniform values.

// cache_len of the batch, read once: lane l holds sequence l's (batches beyond 64 are read as they are needed)
struct Lens {
    int mine;
    __device__ __forceinline__ explicit Lens(const AttnArgs& a) {
        const int lane = threadIdx.x & 63;
        mine = lane < a.B ? a.cache_len[lane] : 0;
    }
    __device__ __forceinline__ int at(const AttnArgs& a, int b) const {
        return b < 64 ? __builtin_amdgcn_readlane(mine, b) : __builtin_amdgcn_readfirstlane(a.cache_len[b]);
    }
    __device__ __forceinline__ int tiles(const AttnArgs& a, int b) const { return tiles_of(a, usable(a, at(a, b))); }
    // tiles of sequence c + lane (all its KV heads), 0 past the end of the batch
    __device__ __forceinline__ int lane_tiles(const AttnArgs& a, int c) const {
        const int b = c + (threadIdx.x & 63);
        if (b >= a.B) return 0;
        return tiles_of(a, usable(a, c == 0 ? mine : a.cache_len[b])) * a.Hkv;
    }
};

__device__ __forceinline__ int wave_inclusive(int x) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int y = __shfl_up(x, off);
        if (lane >= off) x += y;
    }
    return x;
}

// The end-to-end order of the batch's tiles: one prefix sum over the sequences (batches beyond 64: over each 64)
struct Order {
    int incl, total;       // this lane's inclusive sum over sequences 0 .. lane; all tiles
    __device__ __forceinline__ Order(const AttnArgs& a, const Lens& lens) {
        if (a.B == 1) {
            total = incl = lens.tiles(a, 0) * a.Hkv;
            return;
        }
        incl = wave_inclusive(lens.lane_tiles(a, 0));
        total = __builtin_amdgcn_readlane(incl, 63);
        for (int c = 64; c < a.B; c += 64) total += __builtin_amdgcn_readlane(wave_inclusive(lens.lane_tiles(a, c)), 63);
    }
    // first tile of sequence b
    __device__ __forceinline__ int begin(const AttnArgs& a, const Lens& lens, int b) const {
        if (b <= 64) return b == 0 ? 0 : __builtin_amdgcn_readlane(incl, b - 1);
        int t = __builtin_amdgcn_readlane(incl, 63);
        for (int c = 64; c < b; c += 64) {
            const int n = lens.lane_tiles(a, c);
            t += __builtin_amdgcn_readlane(wave_inclusive(c + (int)(threadIdx.x & 63) < b ? n : 0), 63);
        }
        return t;
    }
    // sequence that holds tile x (0 <= x < total)
    __device__ __forceinline__ int seq_of(const AttnArgs& a, const Lens& lens, int x) const {
        if (a.B == 1) return 0;
        unsigned long long after = __ballot(incl > x);
        int base = __builtin_amdgcn_readlane(incl, 63), c = 0;
        while (!after) {
            c += 64;
            const int in = base + wave_inclusive(lens.lane_tiles(a, c));
            after = __ballot(in > x);
            base = __builtin_amdgcn_readlane(in, 63);
        }
        return __builtin_amdgcn_readfirstlane(c + __ffsll((long long)after) - 1);
    }
};

// Team g's share begins at tile floor(g total / teams): equal shares, and whole units where the numbers divide.
struct Shares {
    int total, teams, per, rem;
    __device__ __forceinline__ Shares(int total_, int teams_) : total(total_), teams(teams_), per(total_ / teams_), rem(total_ % teams_) {}
    __device__ __forceinline__ int begin(int g) const { return g * per + (int)((unsigned)g * (unsigned)rem / (unsigned)teams); }   // teams < 2^16
};

// One team's walk over its share: a segment is a run of tiles [tile, tile_end) of one unit.  The kernels keep two: one
// runs ahead and issues loads, one follows and multiplies, so that the loads never pause where a segment ends.
struct Walk {
    int b, kvh;            // unit of the current segment; b < 0: no segment
    int tiles;             // tiles of that unit
    int tile, tile_end;    // the segment
    int left;              // tiles of the share after this segment
};

__device__ __forceinline__ Walk walk_first(const AttnArgs& a, const Lens& lens, int team) {
    Walk w = {-1, 0, 0, 0, 0, 0};
    if (team >= a.teams) return w;
    if (a.split > 0) {
        const int unit = team / a.split, k = team - unit * a.split;
        w.b = unit / a.Hkv;
        w.kvh = unit - w.b * a.Hkv;
        w.tiles = lens.tiles(a, w.b);
        const int run = (w.tiles + a.split - 1) / a.split;
        w.tile = k * run;
        w.tile_end = min(w.tiles, w.tile + run);
        if (w.tile >= w.tile_end) w.b = -1;         // (an empty run: see note_empty)
        return w;
    }
    const Order order(a, lens);
    const Shares s(order.total, a.teams);
    const int x = __builtin_amdgcn_readfirstlane(s.begin(team)), n = __builtin_amdgcn_readfirstlane(s.begin(team + 1)) - x;
    if (n <= 0) return w;
    w.b = order.seq_of(a, lens, x);
    w.tiles = lens.tiles(a, w.b);
    const int first = order.begin(a, lens, w.b);
    w.kvh = __builtin_amdgcn_readfirstlane((x - first) / w.tiles);
    w.tile = (x - first) - w.kvh * w.tiles;
    w.tile_end = min(w.tiles, w.tile + n);
    w.left = n - (w.tile_end - w.tile);
    return w;
}

// (by value: a walk stays in scalar registers)
__device__ __forceinline__ Walk walk_next(const AttnArgs& a, const Lens& lens, const Walk w) {
    Walk n = w;
    n.b = -1;
    if (w.left > 0) {
        const bool next_seq = w.kvh + 1 == a.Hkv;
        n.b = next_seq ? w.b + 1 : w.b;
        n.kvh = next_seq ? 0 : w.kvh + 1;
        n.tiles = lens.tiles(a, n.b);
        n.tile = 0;
        n.tile_end = min(n.tiles, w.left);
        n.left = w.left - n.tile_end;
    }
    return n;
}

// a walk's unit is covered by this segment alone (evaluate before the walk's `tile` moves)
__device__ __forceinline__ bool walk_is_whole(const Walk& w) { return w.tile == 0 && w.tile_end == w.tiles; }
// workspace rows of a part: a team leaves at most one part that ends a unit or lies inside it (slot 0) and one
// that begins a unit (slot 1)
__device__ __forceinline__ size_t part_row(const AttnArgs& a, int team, int slot) { return ((size_t)team * 2 + slot) * a.M; }

// ---- what a workgroup needs to know about a sequence besides its length (each wavefront finds out by itself: no barrier)
// parent[] (in LDS) is not a tree
__device__ __forceinline__ bool tree_is_bad(const AttnArgs& a, const int32_t* spar) {
    const int lane = threadIdx.x & 63;
    bool bad = false;
#pragma unroll
    for (int i = lane; i < kMaxNodes; i += 64)
        if (i < a.N) bad = bad || spar[i] < -1 || spar[i] >= i;
    return __any(bad) != 0;
}
// a page that the prefix of length P touches is not a page of the pool
__device__ __forceinline__ bool pages_are_bad(const AttnArgs& a, int b, int P) {
    bool bad = false;
    for (int i = threadIdx.x & 63; i < ((P + (1 << a.page_shift) - 1) >> a.page_shift); i += 64) {
        const int id = a.block_table[(size_t)b * a.max_blocks + i];
        bad = bad || id < 0 || id >= a.num_pages;
    }
    return __any(bad) != 0;
}
// 128-bit ancestor-or-self masks of a valid tree, from `spar`; the caller's barrier makes them visible
__device__ __forceinline__ void build_masks(const AttnArgs& a, const int32_t* spar, uint32_t* anc) {
    const int tid = threadIdx.x;
    if (tid < a.N) {
        uint32_t m[4] = {0, 0, 0, 0};
        for (int j = tid; j >= 0; j = spar[j]) m[j >> 5] |= 1u << (j & 31);
        *(uint4*)(anc + tid * 4) = make_uint4(m[0], m[1], m[2], m[3]);
    }
}
// node of query row r (r / G without an integer division per row)
__device__ __forceinline__ int node_of_row(int r, int G, float inv_G) {
    int q = (int)((float)r * inv_G);
    const int rem = r - q * G;
    return rem < 0 ? q - 1 : rem >= G ? q + 1 : q;
}

// A team without tiles in a split launch leaves empty parts (sum 0), so that the merge kernel need not know how many
// teams had some.
__device__ __forceinline__ void note_empty(const AttnArgs& a, int team, int mt, int rows) {
    if (a.split > 1 && team < a.teams)
        for (int r = mt * rows + (int)threadIdx.x; r < min(a.M, (mt + 1) * rows); r += blockDim.x)
            *(float2*)(a.ws_ml + (part_row(a, team, team % a.split == 0 ? 1 : 0) + r) * 2) = make_float2(-INFINITY, 0.f);
}

// Tells the merge kernel which teams share a unit (balanced launches): the team that begins it and the team that ends it.
__device__ __forceinline__ void note_parts(const AttnArgs& a, int team, const Walk& w) {
    const size_t unit = (size_t)w.b * a.Hkv + w.kvh;
    if (w.tile == 0) a.ws_parts[2 * unit] = team;
    if (w.tile_end == w.tiles) a.ws_parts[2 * unit + 1] = team;
}

}  // namespace work
}  // namespace s4c

// What the attention kernels need to know about a launch's work: the division (attn_division.h) over the batch's actual
// lengths, and the state of a sequence.
#pragma once
#include "common.h"

namespace s4c {
namespace work {

// Every function below is called by whole wavefronts and returns wave-uniform values.

// cache_len of the batch, read once: lane l holds sequence l's (batches beyond 64 are read as they are needed)
struct Order;
struct Lens {
    typedef work::Order Order;
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

}  // namespace work
}  // namespace s4c

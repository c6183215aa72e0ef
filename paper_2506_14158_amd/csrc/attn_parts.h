// Parts of divided units in a launch of equal runs (attn_division.h, split > 1): how a workgroup hands its part over, and how the
// parts of a unit are merged, by the unit's own workgroups in the same launch (attn_meet.h) or, in a step of two launches, by the next one.
//
// A launch of its own for the merge costs the end of one kernel and the start of another for a few microseconds of
// latency-bound work.  In the same launch the chip's L2s have to be got round, which are not coherent between its eighths: a part
// is written through to memory (device-coherent 16-byte stores, a kilobyte per instruction: the accumulator's registers as they are,
// one "slab" of 8 columns x 32 rows after the other), and the workgroup hands it over when its stores are acknowledged.  (8-byte stores in row order
// made a launch 1.3 to 1.9 times as long as two.)  A merging wave requests everything it needs at once.
#pragma once
#include "attn_meet.h"
#include "attn_work.h"
#include "mfma_common.h"

namespace s4c {

namespace parts {

using namespace mfma;

enum Elem { kB16 = 0, kH16 = 1, kF32 = 2 };  // bf16, fp16, fp32
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
constexpr int kCoherent = 16;                // cache policy of the buffer instructions: sc1, device scope
// What the workgroups of a kernel walk, and what becomes of units in parts.  kWhole: a unit each.  kShares: balanced shares, their parts for attn_merge.h.
// Equal runs: kHere merges them in this launch; kNext leaves them to the next one, where that has other work to do meanwhile (the acceptance of a step behind the
// attention: 8 x 32/8 heads, 8192 keys 115.1 us merged here, 113.8 there).
// (In one kernel for all of them, whole units kept the values of the others: 29 scalar registers spilled
// instead of none, 27 layers of 3 x 4 heads, 73 nodes 461.5 us against 459.0.)
enum Merge { kWhole, kShares, kHere, kNext };

template <int D>
struct Region : PartRegion<D> {
    static __device__ __forceinline__ unsigned char* of(const AttnArgs& a, int team) { return (unsigned char*)a.ws_o + (size_t)team * PartRegion<D>::bytes(a.M); }
};

// (its bounds are checked by the hardware)
__device__ __forceinline__ __amdgpu_buffer_rsrc_t resource(const void* p, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc((void*)uniform((const unsigned char*)p), 0, uniform((int)bytes), 0x00020000);
}

// 4 columns of a row's output
template <Elem E>
__device__ __forceinline__ void store_out(void* out, size_t at, f32x4 v) {
    if constexpr (E == kF32) *(f32x4*)((float*)out + at) = v;
    else *(uint2*)((bf16_t*)out + at) = make_uint2(round1<E == kH16>(v[0]) | (round1<E == kH16>(v[1]) << 16),
                                                   round1<E == kH16>(v[2]) | (round1<E == kH16>(v[3]) << 16));
}

// ---- A wave writes its columns of a row block: KEYS such waves have equal shares of the D / 8 slabs, this one is number
// `key`.  `slab(q)` is its slab q: columns 8 (key slabs + q) + 4 (lane / 32) .. + 3 of row 32 block + lane % 32.  m, l: the row's.
// LATE: the places are found here rather than kept while tiles are multiplied, for a kernel that has no registers left (it kept them in
// scratch: 8 layers of 4 x 64/8 heads, 20 nodes 166 us against 162.5, a step of 32/8 heads, 4000 keys 27.1 against 26.4; in the kernel for few rows,
// which has room, it costs 0.15 us a launch).
template <int D, int KEYS, Merge MERGE, bool LATE = false, class Slab>
__device__ __forceinline__ void put(const AttnArgs& a, int team, int block, int key, float m, float l, Slab slab) {
    constexpr int kSlabs = D / 8 / KEYS, kPolicy = MERGE == kHere ? kCoherent : 0;
    typedef Region<D> R;
    int lane = threadIdx.x & 63;
    if constexpr (LATE) asm volatile("" : "+v"(lane));
    if (32 * block + (lane & 31) >= a.M) return;
    const __amdgpu_buffer_rsrc_t r = resource(R::of(a, team), R::bytes(a.M));
    if (lane < 32) {
        const u32x2 v = {__float_as_uint(m), __float_as_uint(l)};
        __builtin_amdgcn_raw_buffer_store_b64(v, r, R::stats(a.M, block, key, lane), 0, kPolicy);
    }
#pragma unroll
    for (int q = 0; q < kSlabs; ++q)
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, slab(q)), r, R::slab(a.M, block, key * kSlabs + q, lane), 0, kPolicy);
}
// the part of a team without tiles: nothing seen by any row
template <int D, int KEYS, Merge MERGE>
__device__ __forceinline__ void put_empty(const AttnArgs& a, int team, int block, int key) {
    put<D, KEYS, MERGE>(a, team, block, key, -INFINITY, 0.f, [](int) { return f32x4{0.f, 0.f, 0.f, 0.f}; });
}

// ---- A wave merges SLABS slabs of a row block of one unit from number `slab` on, its parts in the order of the runs => deterministic.
// BATCH parts are in flight together (4 SLABS + 2 registers each).
template <int D, Elem E, Merge MERGE, int SLABS, int BATCH>
__device__ __forceinline__ void take(const AttnArgs& a, int unit, int block, int slab) {
    typedef Region<D> R;
    constexpr int kPolicy = MERGE == kHere ? kCoherent : 0;
    const int lane = threadIdx.x & 63, n = a.split;
    const int key = slab * a.part_keys / (D / 8);
    const int b = unit / a.Hkv, kvh = unit - b * a.Hkv;
    const int r = 32 * block + (lane & 31);
    if (r >= a.M) return;
    f32x4 o[SLABS];
    float m = -INFINITY, l = 0.f;
#pragma unroll
    for (int q = 0; q < SLABS; ++q) o[q] = f32x4{0.f, 0.f, 0.f, 0.f};
    // (one resource for all parts: one for each took more scalar registers than there are)
    const uint32_t bytes = R::bytes(a.M);
    const __amdgpu_buffer_rsrc_t all = resource(R::of(a, unit * n), bytes * n);
    f32x4 v[BATCH][SLABS];
    u32x2 st[BATCH];
    auto fetch = [&](int p0, bool slabs) __attribute__((always_inline)) {
#pragma unroll
        for (int p = 0; p < BATCH; ++p) {
            st[p] = u32x2{0, 0};
            if (p0 + p < n) {
                st[p] = __builtin_amdgcn_raw_buffer_load_b64(all, R::stats(a.M, block, key, lane), (p0 + p) * bytes, kPolicy);
                if (slabs) {
#pragma unroll
                    for (int q = 0; q < SLABS; ++q)
                        v[p][q] = __builtin_bit_cast(
                            f32x4, __builtin_amdgcn_raw_buffer_load_b128(all, R::slab(a.M, block, slab + q, lane), (p0 + p) * bytes, kPolicy));
                }
            }
        }
    };
    auto highest = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int p = 0; p < BATCH; ++p) m = fmaxf(m, __uint_as_float(st[p][1]) > 0.f ? __uint_as_float(st[p][0]) : -INFINITY);
    };
    // the maximum of all parts first, so that the result does not depend on BATCH: the first parts' last, with their slabs
    for (int p0 = BATCH; p0 < n; p0 += BATCH) {
        fetch(p0, false);
        highest();
    }
    fetch(0, true);
    highest();
    for (int p0 = 0;;) {
#pragma unroll
        for (int p = 0; p < BATCH; ++p)
            if (p0 + p < n) {
                const float pl = __uint_as_float(st[p][1]);
                const float w = pl > 0.f ? fast_exp2(__uint_as_float(st[p][0]) - m) : 0.f;       // 0: the part saw nothing visible
                l = fmaf(pl, w, l);
#pragma unroll
                for (int q = 0; q < SLABS; ++q)
#pragma unroll
                    for (int e = 0; e < 4; ++e) o[q][e] = fmaf(v[p][q][e], w, o[q][e]);
            }
        if ((p0 += BATCH) >= n) break;
        fetch(p0, true);
    }
    const float inv = l > 0.f ? 1.f / l : 0.f;
    const int node = r / a.G, g = r - node * a.G;
    const size_t o0 = (((size_t)b * a.N + node) * a.Hq + kvh * a.G + g) * D + 8 * slab + 4 * (lane >> 5);
#pragma unroll
    for (int q = 0; q < SLABS; ++q) store_out<E>(a.out, o0 + 8 * q, o[q] * inv);
}

// The merging waves of the next launch, 32 columns each.
__host__ __device__ inline int tasks(const AttnArgs& a) { return a.split > 1 ? a.B * a.Hkv * ((a.M + 31) / 32) * (a.D / 32) : 0; }
template <int D, Elem E, int BATCH>
__device__ __forceinline__ void take_task(const AttnArgs& a, int task) {
    if (task >= tasks(a)) return;
    const int blocks = (a.M + 31) / 32, at = task / (D / 32);
    take<D, E, kNext, 4, BATCH>(a, at / blocks, at % blocks, task % (D / 32) * 4);
}

// ---- The workgroups of a unit's runs (for one tile of its rows) meet, seen from a wave of one of them (attn_meet.h).
// Lane p has the word of run p; split <= 24.
template <int D>
struct Words {
    uint64_t *mine, *of_lane;
    uint64_t tag;
    int n, me, state;
    __device__ __forceinline__ Words(const AttnArgs& a, int team, int mt) : tag(a.tag), n(a.split), state(0) {
        const int unit = team / n, lane = threadIdx.x & 63;
        me = team - unit * n;
        auto word = [&](int t) __attribute__((always_inline)) { return (uint64_t*)(Region<D>::of(a, t) + Region<D>::word(a.M, mt)); };
        mine = word(team);
        of_lane = word(unit * n + (lane < n ? lane : me));
    }
    static __device__ __forceinline__ void store(uint64_t* p, uint64_t v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
    __device__ __forceinline__ void tell(int s) const {
        if ((threadIdx.x & 63) == 0) store(mine, meet::word_of(tag, s));
    }
    __device__ __forceinline__ void settle() const { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
    __device__ __forceinline__ void look() { state = meet::state_of(tag, __hip_atomic_load(of_lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)); }
    template <class P>
    __device__ __forceinline__ bool all(P pred) const {
        const int lane = threadIdx.x & 63;
        return __all(lane >= n || lane == me || pred(state)) != 0;
    }
    template <class P>
    __device__ __forceinline__ uint64_t which(P pred) const {
        const int lane = threadIdx.x & 63;
        return __ballot(lane < n && (lane == me || pred(state)));
    }
    __device__ __forceinline__ void clear() const {
        if ((threadIdx.x & 63) < n) store(of_lane, 0);
    }
};
template <int D>
__device__ __forceinline__ void begin(const AttnArgs& a, int team, int mt) {          // the first wave
    if (team >= a.teams) return;
    Words<D> w(a, team, mt);
    meet::begin(w);
}
// The end of a workgroup: `part()` writes its waves' parts; then its share of the unit's merge, if it has one.  Waves of BLOCKS row
// blocks; smem: free once every wave is here.
template <int D, Elem E, Merge MERGE, int WAVES, int BLOCKS, class Part>
__device__ __forceinline__ void finish(const AttnArgs& a, int team, int mt, unsigned char* smem, Part part) {
    if constexpr (MERGE == kNext) {
        part();
        return;
    }
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    Words<D> w(a, team, mt);
    if (wave == 0) meet::look_round(w);
    part();
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (wave == 0) {
        const uint64_t who = meet::hand_over(w);
        if (threadIdx.x == 0) *(uint64_t*)smem = who;
    }
    __syncthreads();
    const uint64_t who = *(const uint64_t*)smem;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)who), hi = __builtin_amdgcn_readfirstlane((uint32_t)(who >> 32));
    if ((lo | hi) == 0) return;
    asm volatile("" ::: "memory");
    const int unit = team / a.split, me = team - unit * a.split;      // (me < 32)
    const int rank = __builtin_popcount(lo & ((1u << me) - 1u)), stay = __builtin_popcount(lo) + __builtin_popcount(hi);
    const int blocks = min(BLOCKS, (a.M + 31) / 32 - mt * BLOCKS);
    // Over the workgroups first: 16 parts of 108 rows, merged by the waves of four of the 16 CUs, took 0.6 us longer a launch.  32 columns a wave of
    // up to eight parts, all in flight together; of more, 8 columns, all of them in flight too.  (Batches of eight parts one after the other: a
    // step of 32/8 heads, 4000 keys, 16 parts 22.8 us and 21.0; 21 parts of 56 rows of size 64 32.5 and 30.4.)
    auto share = [&](auto slabs, auto batch) __attribute__((always_inline)) {
        constexpr int kSlabs = decltype(slabs)::value, kTasks = D / 8 / kSlabs;
        for (int t = wave * stay + rank; t < blocks * kTasks; t += stay * WAVES)
            take<D, E, kHere, kSlabs, decltype(batch)::value>(a, unit, mt * BLOCKS + t / kTasks, t % kTasks * kSlabs);
    };
    if (a.split <= 8) share(std::integral_constant<int, 4>{}, std::integral_constant<int, 8>{});
    else share(std::integral_constant<int, 1>{}, std::integral_constant<int, kMostRuns>{});
    if (wave == 0) meet::end(w);
}

}  // namespace parts
}  // namespace s4c

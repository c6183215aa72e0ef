// Parts of divided units in a launch of equal runs (attn_division.h, split > 1): how a workgroup hands its part over, and how a
// merging wave picks the parts up, behind the attention workgroups in the same launch or in the next one.
//
// A launch of its own for the merge costs the end of one kernel and the start of another for a few microseconds of
// latency-bound work.  In the same launch the chip's L2s have to be got round, which are not coherent between its eighths: a part
// is written through to memory (device-coherent 16-byte stores, a kilobyte per instruction: the accumulator's registers as they are,
// one "slab" of 8 columns x 32 rows after the other), the wave waits until its stores are acknowledged, and then publishes a word for
// every merging wave that will take some of it.  (8-byte stores in row order made a launch 1.3 to 1.9 times as long
// as two.)  A merging wave looks at the words of all its parts with one load, then requests everything at once.  It
// only waits for workgroups before it in the grid, which are dispatched before it, and they wait for nobody.
//
// A part is published under the call's 64-bit tag, so the words need no initialisation and what a workspace held before is not
// taken for one.  A merging wave changes the word when it has seen it, so that a captured graph can replay the call, tag
// and all.  Its wait is bounded by wall-clock time; then the sequence is flagged S4C_SEQ_TIMEOUT and its rows are zero.
#pragma once
#include "attn_work.h"
#include "mfma_common.h"

namespace s4c {

// ---- words under a tag, one writer and one reader each, a mark of the reader's beside every word
namespace word {
struct Pair { uint64_t word, mark; };
__device__ __forceinline__ uint64_t load(const uint64_t* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void store(uint64_t* p, uint64_t v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
// A reader that gives up leaves its mark and then looks once more; the writer publishes and then looks for a mark: at least one of
// the two sees the other, and no word of this call stays behind for a replay to find.  Readers start after
// the writer (`started`, 100 MHz wall clock) and wait for `ticks`, so there can only be marks after half that time.
__device__ __forceinline__ void publish(Pair* p, uint64_t tag, long long started, long long ticks) {
    store(&p->word, tag);
    if ((long long)wall_clock64() - started >= ticks / 2) {
        __threadfence();
        if (load(&p->mark) == tag) {
            store(&p->word, ~tag);
            store(&p->mark, ~tag);
        }
    }
}
__device__ __forceinline__ bool here(const Pair* p, uint64_t tag) { return load(&p->word) == tag; }
__device__ __forceinline__ void taken(Pair* p, uint64_t tag) { store(&p->word, ~tag); }
// The reader has waited long enough: whether the word is here after all.  If not, the writer takes it back.
__device__ __forceinline__ bool give_up(Pair* p, uint64_t tag) {
    store(&p->mark, tag);
    __threadfence();
    const bool came = here(p, tag);
    if (came) store(&p->mark, ~tag);
    return came;
}
}  // namespace word

namespace parts {

using namespace mfma;

enum Elem { kB16 = 0, kH16 = 1, kF32 = 2 };  // bf16, fp16, fp32
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
constexpr int kCoherent = 16;                // cache policy of the buffer instructions: sc1, device scope
constexpr int kTake = 4;                     // slabs of a merging wave (32 columns)

// A team's region: room for 2 M rows of D floats, of which a launch of equal runs needs M for the slabs.  In the other half lie
// a pair of words for every row block of 32 and merging wave, and a copy of the rows' (maximum in log2 units, sum) for every wave that wrote
// columns of its own (a.part_keys of them): 16 M / 32 D / 32 + 16 + 8 * 4 M bytes at most, of 4 M D.
template <int D>
struct Region {
    static __device__ __forceinline__ uint32_t bytes(int M) { return 8u * M * D; }
    static __device__ __forceinline__ unsigned char* of(const AttnArgs& a, int team) { return (unsigned char*)a.ws_o + (size_t)team * bytes(a.M); }
    static __device__ __forceinline__ uint32_t slab(int M, int block, int s, int lane) {
        const int rows = min(32, M - 32 * block);
        return 4u * (32 * block * D + ((2 * s + (lane >> 5)) * rows + (lane & 31)) * 4);
    }
    static __device__ __forceinline__ uint32_t words(int M, int block) { return 4u * M * D + sizeof(word::Pair) * (D / 32) * block; }
    static __device__ __forceinline__ uint32_t stats(int M, int block, int key, int lane) {
        return words(M, (M + 31) / 32) + 8u * (key * M + 32 * block + (lane & 31));
    }
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

// ---- A wave hands over its columns of a row block: KEYS such waves have equal shares of the D / 8 slabs, this one is number
// `key`.  `slab(q)` is its slab q: columns 8 (key slabs + q) + 4 (lane / 32) .. + 3 of row 32 block + lane % 32.  m, l: the row's.
// LATE: the places are found here rather than kept while tiles are multiplied, for a kernel that has no registers left (it kept them, and the
// tag, in scratch: 8 layers of 4 x 64/8 heads, 20 nodes 166 us against 162.5, a step of 32/8 heads, 4000 keys 27.1 against 26.4; in the kernel for few rows,
// which has room, it costs 0.15 us a launch).
template <int D, int KEYS, bool LATE = false, class Slab>
__device__ __forceinline__ void put(const AttnArgs& a, int team, int block, int key, float m, float l, long long started, Slab slab) {
    constexpr int kSlabs = D / 8 / KEYS;
    typedef Region<D> R;
    int lane = threadIdx.x & 63;
    if constexpr (LATE) asm volatile("" : "+v"(lane));
    if (32 * block >= a.M) return;
    const __amdgpu_buffer_rsrc_t r = resource(R::of(a, team), R::bytes(a.M));
    auto store = [&](auto policy) __attribute__((always_inline)) {
        if (32 * block + (lane & 31) < a.M) {
            if (lane < 32) {
                const u32x2 v = {__float_as_uint(m), __float_as_uint(l)};
                __builtin_amdgcn_raw_buffer_store_b64(v, r, R::stats(a.M, block, key, lane), 0, policy);
            }
#pragma unroll
            for (int q = 0; q < kSlabs; ++q)
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, slab(q)), r, R::slab(a.M, block, key * kSlabs + q, lane), 0, policy);
        }
    };
    if (a.tag == 0) {                                      // merged by the next launch
        store(std::integral_constant<int, 0>{});
        return;
    }
    store(std::integral_constant<int, kCoherent>{});
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if (lane < kSlabs / kTake)
        word::publish((word::Pair*)(R::of(a, team) + R::words(a.M, block)) + key * (kSlabs / kTake) + lane, a.tag, started, a.wait_ticks);
}
// the part of a team without tiles: nothing seen by any row
template <int D, int KEYS>
__device__ __forceinline__ void put_empty(const AttnArgs& a, int team, int block, int key, long long started) {
    put<D, KEYS>(a, team, block, key, -INFINITY, 0.f, started, [](int) { return f32x4{0.f, 0.f, 0.f, 0.f}; });
}

// ---- Merging wave `task` of a launch: 32 columns of a row block of one unit, its parts in the order of the runs => deterministic.
__host__ __device__ inline int tasks(const AttnArgs& a) { return a.split > 1 ? a.B * a.Hkv * ((a.M + 31) / 32) * (a.D / 32) : 0; }

// BATCH parts are in flight together (18 registers each).
template <int D, Elem E, int BATCH>
__device__ __forceinline__ void take(const AttnArgs& a, int task) {
    typedef Region<D> R;
    if (task >= tasks(a)) return;
    const int lane = threadIdx.x & 63, blocks = (a.M + 31) / 32, n = a.split;
    const int quarter = task % (D / 32), block = task / (D / 32) % blocks, unit = task / (D / 32) / blocks;
    const int key = quarter * a.part_keys / (D / 32);
    const int b = unit / a.Hkv, kvh = unit - b * a.Hkv;
    bool late = false;
    if (a.tag != 0) {
        word::Pair* const p = (word::Pair*)(R::of(a, unit * n + (lane < n ? lane : 0)) + R::words(a.M, block)) + quarter;     // n <= 64
        const long long deadline = (long long)wall_clock64() + a.wait_ticks;
        bool mine = lane >= n || word::here(p, a.tag);
        while (!__all(mine)) {
            if ((long long)wall_clock64() - deadline >= 0) {
                if (!mine) mine = word::give_up(p, a.tag);
                late = !__all(mine);
                break;
            }
            __builtin_amdgcn_s_sleep(1);
            mine = lane >= n || word::here(p, a.tag);
        }
        if (lane < n && mine) word::taken(p, a.tag);
    }
    asm volatile("" ::: "memory");
    const int r = 32 * block + (lane & 31);
    f32x4 o[kTake];
    float m = -INFINITY, l = 0.f;
#pragma unroll
    for (int q = 0; q < kTake; ++q) o[q] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (late) {
        // (behind what an attention workgroup of the sequence may be about to write there)
        for (const long long until = (long long)wall_clock64() + 500000; (long long)wall_clock64() - until < 0;) __builtin_amdgcn_s_sleep(64);
        if (a.status && lane == 0) atomicOr(a.status + b, S4C_SEQ_TIMEOUT);
    }
    auto combine = [&](auto policy) __attribute__((always_inline)) {
        auto from = [&](int p) __attribute__((always_inline)) { return resource(R::of(a, unit * n + p), R::bytes(a.M)); };
        f32x4 v[BATCH][kTake];
        u32x2 st[BATCH];
        auto fetch = [&](int p0, bool slabs) __attribute__((always_inline)) {
#pragma unroll
            for (int p = 0; p < BATCH; ++p) {
                st[p] = u32x2{0, 0};
                if (p0 + p < n) {
                    st[p] = __builtin_amdgcn_raw_buffer_load_b64(from(p0 + p), R::stats(a.M, block, key, lane), 0, policy);
                    if (slabs) {
#pragma unroll
                        for (int q = 0; q < kTake; ++q)
                            v[p][q] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(
                                from(p0 + p), R::slab(a.M, block, quarter * kTake + q, lane), 0, policy));
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
                    for (int q = 0; q < kTake; ++q)
#pragma unroll
                        for (int e = 0; e < 4; ++e) o[q][e] = fmaf(v[p][q][e], w, o[q][e]);
                }
            if ((p0 += BATCH) >= n) break;
            fetch(p0, true);
        }
    };
    if (r >= a.M) return;
    if (a.tag == 0) combine(std::integral_constant<int, 0>{});
    else if (!late) combine(std::integral_constant<int, kCoherent>{});
    const float inv = l > 0.f ? 1.f / l : 0.f;
    const int node = r / a.G, g = r - node * a.G;
    const size_t o0 = (((size_t)b * a.N + node) * a.Hq + kvh * a.G + g) * D + 32 * quarter + 4 * (lane >> 5);
#pragma unroll
    for (int q = 0; q < kTake; ++q) store_out<E>(a.out, o0 + 8 * q, o[q] * inv);
}

}  // namespace parts
}  // namespace s4c

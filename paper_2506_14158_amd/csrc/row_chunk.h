// Shared by the kernels that scan logits rows in chunks of 8192 (acceptance statistics,
// candidate-tree construction): a workgroup of 256 threads holds one chunk in registers,
// 32 logits per thread, read once with 16-byte loads.
#pragma once
#include "common.h"

namespace s4c {
namespace rowchunk {

constexpr int kThreads = 256;
constexpr int kPerThread = 32;                       // logits per thread
constexpr int kChunk = kThreads * kPerThread;        // logits per workgroup

struct MaxIdx {
    float v;
    int32_t i;
};

__device__ __forceinline__ MaxIdx better(MaxIdx a, MaxIdx b) {
    // larger value wins; equal values: lower index wins (never depends on reduction order)
    const bool take_b = (b.v > a.v) || (b.v == a.v && b.i < a.i);
    return take_b ? b : a;
}

// Reductions over a wavefront, the result in every lane.  Data parallel primitives: each of the six steps is one instruction of the
// vector ALU, where an exchange through LDS takes a round trip of it (the twelve of a (value, index) maximum: 0.6 us).
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp_or(uint32_t x, uint32_t none) {        // lanes without a source: none
    return (uint32_t)__builtin_amdgcn_update_dpp((int)none, (int)x, CTRL, ROWS, 0xF, false);
}
template <class Op>
__device__ __forceinline__ uint32_t wave_reduce(uint32_t x, uint32_t none, Op op) {
    x = op(x, dpp_or<0x111, 0xF>(x, none));          // row_shr:1, 2, 4, 8: inside each row of 16
    x = op(x, dpp_or<0x112, 0xF>(x, none));
    x = op(x, dpp_or<0x114, 0xF>(x, none));
    x = op(x, dpp_or<0x118, 0xF>(x, none));
    x = op(x, dpp_or<0x142, 0xA>(x, none));          // row_bcast:15 into rows 1 and 3
    x = op(x, dpp_or<0x143, 0xC>(x, none));          // row_bcast:31 into rows 2 and 3
    return (uint32_t)__builtin_amdgcn_readlane((int)x, 63);
}
__device__ __forceinline__ float wave_max(float x) {
    return __uint_as_float(wave_reduce(__float_as_uint(x), 0xFF800000u, [](uint32_t a, uint32_t b) {
        return __float_as_uint(fmaxf(__uint_as_float(a), __uint_as_float(b)));
    }));
}
__device__ __forceinline__ float wave_sum(float x) {
    return __uint_as_float(wave_reduce(__float_as_uint(x), 0u, [](uint32_t a, uint32_t b) {
        return __float_as_uint(__uint_as_float(a) + __uint_as_float(b));
    }));
}
__device__ __forceinline__ MaxIdx wave_best(MaxIdx x) {
    const float v = wave_max(x.v);
    const uint32_t i = x.v == v ? (uint32_t)x.i : 0xFFFFFFFFu;                  // (indices are not negative)
    return MaxIdx{v, (int32_t)wave_reduce(i, 0xFFFFFFFFu, [](uint32_t a, uint32_t b) { return a < b ? a : b; })};
}

template <typename T> struct Vec16;   // 16-byte vector of T
template <> struct Vec16<float> { static constexpr int n = 4; };
template <> struct Vec16<bf16_t> { static constexpr int n = 8; };
template <> struct Vec16<f16_t> { static constexpr int n = 8; };

// A logits row read in chunks of kChunk elements with 16-byte loads whatever its alignment: chunks are counted from the
// 16-byte boundary at or below the row's start, `head` elements before it.  Vector j of a thread holds the Vec16<T>::n
// elements from idx(chunk, j) on; elements outside [0, V) read as -inf.  Only the vectors that contain such
// elements (the first and the last of a row) are put together element by element, so every load lies in the row.
// (Rows of an odd length used to be read two bytes at a time.)
template <typename T>
struct RowReader {
    static constexpr int VN = Vec16<T>::n;
    static constexpr int NV = kPerThread / VN;
    // (named as global memory: where the compiler lost track of that, the loads became flat ones, which wait for LDS too)
    typedef const __attribute__((address_space(1))) T* Ptr;
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    Ptr base;
    int V, head;
    __device__ __forceinline__ RowReader(const void* logits, size_t row, int V_) : base((Ptr)((const T*)logits + row * (size_t)V_)), V(V_) {
        head = (int)(((uintptr_t)base & 15) / sizeof(T));
    }
    __device__ __forceinline__ int idx(int chunk, int j) const { return chunk * kChunk + (j * kThreads + (int)threadIdx.x) * VN - head; }
    __device__ __forceinline__ uint4 vec(int e) const {
        const u32x4 w = *(const __attribute__((address_space(1))) u32x4*)(base + e);
        return make_uint4(w[0], w[1], w[2], w[3]);
    }
    __device__ __forceinline__ void fetch(int chunk, uint4 (&raw)[NV]) const {
        const int lo = chunk * kChunk - head;
        if (lo >= 0 && lo <= V - kChunk) {                             // wave-uniform
#pragma unroll
            for (int j = 0; j < NV; ++j) raw[j] = vec(idx(chunk, j));
            return;
        }
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            const int e0 = idx(chunk, j);
            constexpr uint32_t kNegInf = sizeof(T) == 4 ? 0xFF800000u : __is_same(T, f16_t) ? 0xFC00FC00u : 0xFF80FF80u;
            raw[j] = make_uint4(kNegInf, kNegInf, kNegInf, kNegInf);
            if (e0 >= 0 && e0 + VN <= V) {
                raw[j] = vec(e0);
            } else if (e0 + VN > 0 && e0 < V) {
                uint32_t w[4] = {kNegInf, kNegInf, kNegInf, kNegInf};
#pragma unroll
                for (int k = 0; k < VN; ++k)
                    if (e0 + k >= 0 && e0 + k < V) {
                        if constexpr (sizeof(T) == 4) {
                            w[k] = __builtin_bit_cast(uint32_t, base[e0 + k]);
                        } else {
                            const uint32_t x = __builtin_bit_cast(uint16_t, base[e0 + k]);
                            w[k / 2] = (k & 1) ? (w[k / 2] & 0xFFFFu) | (x << 16) : (w[k / 2] & 0xFFFF0000u) | x;
                        }
                    }
                raw[j] = make_uint4(w[0], w[1], w[2], w[3]);
            }
        }
    }
};
// the elements of one vector, as floats
template <typename T>
__device__ __forceinline__ void decode(const uint4& raw, float (&x)[Vec16<T>::n]) {
    if constexpr (sizeof(T) == 4) {
        x[0] = __uint_as_float(raw.x);
        x[1] = __uint_as_float(raw.y);
        x[2] = __uint_as_float(raw.z);
        x[3] = __uint_as_float(raw.w);
    } else {
        unpack2<T>(raw.x, x[0], x[1]);
        unpack2<T>(raw.y, x[2], x[3]);
        unpack2<T>(raw.z, x[4], x[5]);
        unpack2<T>(raw.w, x[6], x[7]);
    }
}

// Thread tid's 32 logits of the chunk [c0, cend) of the row at `base`, which begins and ends on a 16-byte boundary, as
// floats: vector j of the thread holds the Vec16<T>::n consecutive tokens starting at idx0[j] (ascending in j and
// inside a vector).  Tokens at or beyond cend read as -inf.
template <typename T>
__device__ __forceinline__ void load_chunk(const T* base, int c0, int cend, int tid, float (&x)[kPerThread],
                                           int32_t (&idx0)[kPerThread / Vec16<T>::n]) {
    constexpr int VN = Vec16<T>::n;
#pragma unroll
    for (int j = 0; j < kPerThread / VN; ++j) {
        const int e0 = c0 + (j * kThreads + tid) * VN;
        idx0[j] = e0;
        float v[VN];
        if (e0 + VN <= cend) decode<T>(*(const uint4*)(base + e0), v);
#pragma unroll
        for (int q = 0; q < VN; ++q) x[j * VN + q] = e0 + VN <= cend ? v[q] : -INFINITY;
    }
}

}  // namespace rowchunk
}  // namespace s4c

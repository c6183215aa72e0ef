// Combines the parts of the (sequence, KV head) units that the attention kernels' teams divided between them
// (attn_division.h): out = sum_p 2^(m_p - m) O_p / sum_p 2^(m_p - m) l_p, parts in tile order => deterministic.
//
// A workgroup takes a chunk of query rows of one unit and leaves at once if the unit was not divided.  32 lanes per
// row (D = 128: one float4 each, D = 64: float2); every part's statistics and the first eight parts' outputs are in
// flight together: the kernel is a few microseconds of latency, not of work.
#pragma once
#include "attn_work.h"

namespace s4c {
namespace merge {

constexpr int kRows = 8;            // rows per workgroup and pass
constexpr int kBatch = 8;           // partial outputs in flight together

// rows [(chunk * passes) * kRows ..) of one unit, by a workgroup of 256 threads
template <typename T, int D>
__device__ __forceinline__ void merge_rows(const AttnArgs& a, int unit, int chunk, int passes) {
    constexpr int VW = D / 32;                                   // floats per lane
    const int sub = threadIdx.x & 31;
    const int b = unit / a.Hkv, kvh = unit - b * a.Hkv;
    const work::Parts parts(a, unit);
    const int g0 = parts.first, g1 = parts.last;
    if (g0 == g1) return;                                        // written by its one team already
    for (int pass = 0; pass < passes; ++pass) {
        const int r = (chunk * passes + pass) * kRows + (threadIdx.x >> 5);
        if (r >= a.M) return;                                    // (all 32 lanes of a row together)
        float m = -INFINITY, l = 0.f, o[VW];
#pragma unroll
        for (int j = 0; j < VW; ++j) o[j] = 0.f;
        for (int gb = g0; gb <= g1; gb += 32) {                  // (more than 32 parts only if a sequence is much the longest)
            const int n = min(32, g1 + 1 - gb);
            auto part = [&](int p) { return work::part_row(a, gb + p, parts.slot(gb + p)) + r; };
            // lane p of the row holds part p's maximum and sum; the first outputs are requested with them
            const float2 ml = sub < n ? *(const float2*)(a.ws_ml + part(sub) * 2) : make_float2(-INFINITY, 0.f);
            float v[kBatch][VW];
            auto fetch = [&](int p0) {
#pragma unroll
                for (int p = 0; p < kBatch; ++p)
                    if (p0 + p < n) {
#pragma unroll
                        for (int j = 0; j < VW; ++j) v[p][j] = a.ws_o[part(p0 + p) * D + sub * VW + j];
                    }
            };
            fetch(0);
            float mb = ml.y > 0.f ? ml.x : -INFINITY;
#pragma unroll
            for (int off = 16; off >= 1; off >>= 1) mb = fmaxf(mb, __shfl_xor(mb, off, 32));
            mb = fmaxf(mb, m);
            const float w = ml.y > 0.f ? fast_exp2(ml.x - mb) : 0.f;         // 0: the part saw nothing visible
            float lb = ml.y * w;
#pragma unroll
            for (int off = 16; off >= 1; off >>= 1) lb += __shfl_xor(lb, off, 32);
            const float w0 = m > -INFINITY ? fast_exp2(m - mb) : 0.f;
            l = fmaf(l, w0, lb);
            m = mb;
#pragma unroll
            for (int j = 0; j < VW; ++j) o[j] *= w0;
            for (int p0 = 0; p0 < n; p0 += kBatch) {
                if (p0 > 0) fetch(p0);
#pragma unroll
                for (int p = 0; p < kBatch; ++p)
                    if (p0 + p < n) {
                        const float wp = __shfl(w, p0 + p, 32);
#pragma unroll
                        for (int j = 0; j < VW; ++j) o[j] = wp > 0.f ? fmaf(v[p][j], wp, o[j]) : o[j];   // (0: v may never have been written)
                    }
            }
        }
        const float inv = (l > 0.f) ? 1.f / l : 0.f;
        const int node = r / a.G, g = r - node * a.G;
        T* dst = (T*)a.out + (((size_t)b * a.N + node) * a.Hq + (kvh * a.G + g)) * D + sub * VW;
        T packed[VW];
#pragma unroll
        for (int j = 0; j < VW; ++j) packed[j] = from_f32<T>(o[j] * inv);
        __builtin_memcpy(__builtin_assume_aligned(dst, sizeof(packed)), packed, sizeof(packed));
    }
}

struct Grid { int units, chunks, passes; };    // workgroups: units x chunks
// one pass per workgroup, more where that would be over about 2048 workgroups (units that are not divided should cost little)
inline Grid grid_of(const AttnArgs& a) {
    const long units = (long)a.B * a.Hkv, chunks = (a.M + kRows - 1) / kRows;
    const int passes = (int)((units * chunks + 2047) / 2048);
    return Grid{(int)units, (int)((chunks + passes - 1) / passes), passes};
}

}  // namespace merge
}  // namespace s4c

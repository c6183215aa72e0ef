// Whether a verification step that fits one launch (attn_step.h) is also faster so: the arithmetic alone, which also compiles for the host
// (tests/host/step_plan.cpp).
//
// Beside the attention the scan has the places that are left, few where the attention has most of the chip, and a workgroup's scan may outlast it; behind
// the attention it has the whole chip, but begins 2 us after the attention's end and ends in a chain of memory round trips.  Measured, 900 steps of random sizes
// (1 - 32 sequences, 2 - 32 KV heads of 1 - 8 query heads, 4 - 100 nodes, 64 - 6000 keys, V 1000 - 128256):
//   a scanning workgroup takes 0.5 us for a chunk of 8192 16-bit logits and 1.7 us for every row that it ends (its threads' results meet, which
//     waits for the chunks in flight), about two thirds of it in stochastic mode, which skips the leaves' rows;
//   a key tile takes 0.75 us of the kernel for few rows (1.5 and more in fp32) and 1.7 us of the one for many;
//   behind the attention a step takes 6 us, and 0.16 us a megabyte of logits (0.06 in stochastic mode), longer than the attention alone.
// One and two launches, us, where the estimates below are closest to each other: one 22.5, two 23.9 (19 x 8 x 8 heads, 24 nodes, 84 keys, V 4900) and one
// 43.6, two 41.7 (26 x 8 heads, 10 nodes, 1527 keys, V 45984) are left to two; one 30.7, two 32.6 (11 x 8 heads of size 64, 64 nodes, 742 keys, V 35697) and one
// 121.8, two 114.4 (13 x 16 x 4 heads, 51 nodes, 3356 keys, V 9580) to one.  Far from the line: one 189, two 87 (27 x 16 heads, 55 nodes, 1654
// keys, V 1558) and one 19.9, two 32.9 (2 x 32 heads, 94 nodes, 184 keys, V 128256).
// (The line used to be 4 chunks more than key tiles, of whatever kind: those two were on its wrong sides.)
#pragma once

namespace s4c {

struct StepScan {
    long long chunks;          // of a scanning workgroup beside the attention, at most
    long long row_chunks;      // of a row of logits
    long long tiles;           // key tiles of an attention workgroup, at most
    long long logits_bytes;    // of the batch
    bool fp32, greedy;
    bool large;                // the attention's kernel for many rows (attn_division.h)
    int per_cu;                // its workgroups on a CU
};

inline bool one_launch_pays(const StepScan& s) {
    const long long rows = (s.chunks + s.row_chunks - 1) / s.row_chunks;
    long long scan = s.chunks * (s.fp32 ? 800 : 550) + rows * 1800;                              // ns
    if (!s.greedy) scan = scan * 7 / 10;
    if (s.large && s.per_cu == 2) scan += 8000;                                                  // (many rows of head size 64, two workgroups a CU: 8 us later)
    const long long attention = s.tiles * (s.fp32 ? 1500 : s.large ? 1700 : 750);
    const long long behind = 4000 + (s.logits_bytes * (s.greedy ? 100 : 50) >> 20);
    return scan <= attention + behind;
}

}  // namespace s4c

// Whether a verification step that fits one launch (attn_step.h) is also faster so: the arithmetic alone, which also compiles for the host
// (tests/host/step_plan.cpp).
//
// Beside the attention the scan has the places that are left, few where the attention has most of the chip, and a workgroup's scan may outlast it; behind
// the attention it has the whole chip, but begins 2 us after the attention's end and ends in a chain of memory round trips.  Measured, 1500 steps of random sizes
// (1 - 32 sequences, 2 - 32 KV heads of 1 - 8 query heads, 4 - 100 nodes, 64 - 6000 keys, V 1000 - 128256):
//   a scanning workgroup takes 0.5 us for a chunk of 8192 16-bit logits and 1.5 us for every row that it ends (its threads' results meet, which
//     waits for the chunks in flight); beside long attention on the matrix cores, which lowers the clock, 0.8 to 1 us for a whole chunk (one 83.6, two 60.6: 8 x 8 heads,
//     87 nodes, 16904 keys, V 97351); stochastic mode skips the leaves' rows, which only the device knows: two thirds of them in the trees of
//     this measurement, a fifth to a third in others;
//   a key tile takes 0.5 to 0.8 us of the kernel for few rows (1 to 2.3 in fp32) and 1.1 to 2 us of the one for many;
//   behind the attention a step takes 6 us, and 0.16 us a megabyte of logits that are scanned, longer than the attention alone;
//     an attention workgroup takes 6 us more than its tiles in the kernel for many rows, 2.5 in fp32.
// The estimates below lean towards two launches: 1150 of the steps go in one, none slower so, and of the others one was the faster way for 104 by
// more than 3 %.  One and two launches, us, left to two: 28.4 and 28.1 (9 x 4 x 4 heads of size 64, 92 nodes, 381 keys, V 3661), 26.0 and 24.8 (2 x 8 x 4 heads, 29
// nodes, 3777 keys, V 32000); sent in one: 85.7 and 88.5 (fp32, 2 x 8 x 8 heads, 19 nodes, 4831 keys, V 32000), 38.0 and 39.0 (fp32, 2 x 8 heads of size 64, 81
// nodes, 4722 keys).  Far from the line: one 189, two 87 (27 x 16 heads, 55 nodes, 1654
// keys, V 1558) and one 19.9, two 32.9 (2 x 32 heads, 94 nodes, 184 keys, V 128256).
// Counting too few rows in stochastic mode costs most: trees of 6 levels, 7 x 32 heads, 107 nodes, 2095 keys, V 12941, in one 104.2, in two 66.3.  The other way round
// 11 x 8 x 4 heads, 39 nodes, 266 keys, V 128256: 22.7 and 33.1.
// (The line used to be 4 chunks more than key tiles, of whatever kind: the two far from it were on its wrong sides.)
#pragma once

namespace s4c {

struct StepScan {
    long long chunks;          // of a scanning workgroup beside the attention, at most
    long long row_chunks;      // of a row of logits
    long long tiles;           // key tiles of an attention workgroup, at most
    long long logits_bytes;    // of the batch
    bool fp32, greedy;
    bool large;                // the attention's kernel for many rows (attn_division.h)
    int head;                  // size
};

inline bool one_launch_pays(const StepScan& s) {
    const long long rows = (s.chunks + s.row_chunks - 1) / s.row_chunks;
    long long scan = s.chunks * (s.fp32 ? 850 : s.large && s.row_chunks > 1 && s.tiles > 16 ? 750 : 600) + rows * 1800;                              // ns
    long long whole = s.logits_bytes * 100 >> 20;                                                // on the whole chip
    if (!s.greedy) {
        scan = scan * 8 / 10;
        whole = whole * 8 / 10;
    }
    const long long tile = s.fp32 ? (s.head == 64 ? 1000 : 2000) : s.large ? (s.head == 64 ? 1100 : 1700) : s.head == 64 ? 450 : 750;
    const long long behind = (s.fp32 ? 6500 : s.large ? 10000 : 4000) + whole;
    return scan <= s.tiles * tile + behind;
}

}  // namespace s4c

// How the candidate-tree scan cuts its rows: the arithmetic alone, which also compiles for the host
// (tests/host/build_plan.cpp).
#pragma once

namespace s4c {

constexpr int kBuildListsInRegisters = 64;     // lists of a row (four a segment) that its merging wavefront holds, one a lane

// Chunks in a segment, of rows of `chunks` chunks.  Up to 8 (a segment's first chunk fills the lists, later ones seldom change
// them), fewer where that would leave fewer than about 2048 workgroups counting all rows, of which about half have children: four
// fit on a CU, and the last turn of the chip should not be a long one; but not so few that a row has more lists than registers
// hold, because then the row kernel reads all of them again for every child (more lists, and 64 at most: 1 x 64, 256000 34.9 and
// 21.2; 1 x 127, 256000 46.0 and 23.9; 1 x 128, 151936 34.0 and 23.2; 1 x 64, 500000 60.3 and 27.8; 1 x 20, 256000 fp32 31.3 and 19.1).
// With 1024 workgroups (us a call) and with 2048: 16 rows x 30 nodes, V 50000 27.6 and 21.3; 8 x 128, 32000
// 34.6 and 27.1; 4 x 100, 128256 37.2 and 30.6; 2 x 128, 128256 32.9 and 28.1; 8 x 100, 60001 fp32 39.5 and 36.6; 16 x 128, 128256 (8
// chunks in both) 83.6; with 4096: 16 x 60, 128256 51.5 (45.2), 8 x 100 fp32 45.2.  Equal runs of chunks across the rows' ends, as the acceptance scan has
// them, measured 87 on the largest: the scan is bound by its selection and exponentials, not by its last turn.
inline int build_segment(long long rows, int chunks) {
    long long seg = rows * chunks / 2048;
    const int few = (4 * chunks + kBuildListsInRegisters - 1) / kBuildListsInRegisters;
    if (seg < few) seg = few;
    if (seg > 8) seg = 8;
    if (seg > chunks) seg = chunks;
    return seg < 1 ? 1 : (int)seg;
}

}  // namespace s4c

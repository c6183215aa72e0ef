// How a call of sequential acceptance is divided between workgroups: the arithmetic alone, which also compiles for the host
// (tests/host/resample_plan.cpp).
#pragma once

#if defined(__HIPCC__)
#define S4C_PLAN __host__ __device__ inline
#else
#define S4C_PLAN inline
#endif

namespace s4c {

constexpr int kResampleWaves = 8;              // of a workgroup
constexpr int kResampleBlock = 512;            // tokens per (wave, iteration)
constexpr int kResampleMaxIters = 8;           // blocks per wave (registers: see decide)
constexpr int kResampleMaxSlice = kResampleMaxIters * kResampleWaves * kResampleBlock;      // tokens of a workgroup: 32768
constexpr int kResampleMaxRow = kResampleMaxSlice / 2;      // longest row that one workgroup decides alone (resample_by_rows)
constexpr int kResampleTeam = 16;              // workgroups per sequence (more only where a slice would outgrow the registers)

S4C_PLAN int resample_blocks(int V) { return (V + kResampleBlock - 1) / kResampleBlock; }
// Blocks per wave, as kernels are built for, of a workgroup that has this many.
S4C_PLAN int resample_iters(int blocks) {
    const int n = (blocks + kResampleWaves - 1) / kResampleWaves;
    return n <= 1 ? 1 : n <= 2 ? 2 : n <= 4 ? 4 : 8;
}
// Workgroups of a team kernel that a CU has room for (by the registers that its launch bounds leave it).
S4C_PLAN constexpr int resample_per_cu(int iters) { return iters <= 2 ? 2 : 1; }

// Workgroups per sequence: enough blocks per workgroup to keep its waves busy, at most 16, and few enough that all
// teams are resident together (one workgroup per CU is certain), but no slice larger than a workgroup's registers hold
// (which makes up to 64 of them for rows beyond 524288).
S4C_PLAN int resample_team(int B, int V, int cus) {
    int G = (resample_blocks(V) + kResampleWaves - 1) / kResampleWaves;
    if (G > kResampleTeam) G = kResampleTeam;
    while (G > 1 && (long long)B * G > cus) G >>= 1;
    const int least = (V + kResampleMaxSlice - 1) / kResampleMaxSlice;
    return G < least ? least : G;
}

// One launch of teams of G: how many sequences it takes, and how many groups of CUs its teams keep to.
//
// Workgroups of a team wait for each other, so two calls on two streams must not each hold CUs that the other one's teams
// are incomplete without.  Workgroup i runs on XCD i modulo the number of XCDs, and every XCD starts a launch's workgroups
// in order, but one XCD may serve one stream first and the next XCD the other.  A launch is therefore of one of three kinds,
// and of any two launches of them one goes on:
//   two fit on a CU      at most one workgroup per CU; two launches fit on the chip together
//   one fills a CU       at most one workgroup for every other CU, likewise
//   one fills a CU, more: a team's workgroups all on one XCD (groups = XCDs, resample_member).  Of the workgroups that an XCD
//                        has started all teams but the last one are complete, and an incomplete one takes at most G - 1
//                        of its 32 CUs: with two such launches, or one and half of the CUs, there is room for the next workgroup.
// (Launches of half the chip in place of the third kind would take twice the time.  us a call, teams spread over the XCDs and one on each:
// 17 x 64 nodes, V 128256 59.6 and 55.6; 64 x 64, 128256 108.6 and 107.0; 40 x 40, 151936 102.8 and 100.5.)
struct ResampleLaunch { int sequences, groups; };
S4C_PLAN ResampleLaunch resample_launch(int B, int G, int iters, int cus) {
    if (G == 1) return {B, 1};                                 // waits for nobody
    if (resample_per_cu(iters) > 1) return {cus / G < 1 ? 1 : cus / G, 1};
    const int per_xcd = cus % 32 == 0 ? 32 : cus, xcds = cus / per_xcd;
    if ((long long)B * G <= cus / 2 || 2 * G > per_xcd) return {cus / 2 / G < 1 ? 1 : cus / 2 / G, 1};
    return {xcds * (per_xcd / G), xcds};
}
S4C_PLAN int resample_grid(int sequences, int G, int groups) { return (sequences + groups - 1) / groups * groups * G; }
// Workgroup i of a launch: its sequence (of the launch; there may be a few more than it has) and its number in the team.
struct ResampleMember { int sequence, g; };
S4C_PLAN ResampleMember resample_member(int i, int G, int groups) {
    const int slot = i / groups;
    return {slot / G * groups + i % groups, slot % G};
}

// Whether every node is decided at once, a workgroup each: up to two turns of the chip of rows of 16384 tokens, or as many
// tokens in shorter rows; half of that where rows lie on odd addresses and are read by the element.  Teams and rows, us a call
// (B x N, V): 1 x 20, 1000: 13.5 and 7.8; 3 x 64, 16000 fp32: 29.3 and 15.7; 4 x 128, 16384: 40.4 and 24.8; 8 x 128, 16384: 38.7
// and 42.0; 16 x 40, 8000: 36.5 and 19.6; 16 x 128, 8000: 35.9 and 38.8; 16 x 128, 4000: 26.2 and 22.6; 8 x 64, 16001: 39.5 and
// 42.0.  Rows of 32000 would fit the registers too, but the slowest node (many children, all rejected) is alone on its CU
// then: 4 x 64: 33.2 and, as the kernels were before, 42.3.
// The sequences' own workgroups wait for the nodes': no more of them than half of the places on the chip, so that whatever a
// second call has waiting, there is room for the nodes' (which wait for nobody).  That also keeps most calls of many sequences with few nodes
// each from this route, where a workgroup a sequence is as good: 512 x 4, 4000: 18.3 and 22.9; 1000 x 2, 1000: 23.6 and 19.8.
S4C_PLAN bool resample_by_rows(int B, int N, int V, int cus) {
    const long long tokens = (long long)B * N * (V < 4096 ? 4096 : V);
    return V <= kResampleMaxRow && tokens <= (V % 8 == 0 ? 2ll : 1ll) * cus * kResampleMaxRow &&
           2 * B <= cus * resample_per_cu(resample_iters(resample_blocks(V)));
}

}  // namespace s4c

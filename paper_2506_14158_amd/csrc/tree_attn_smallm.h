// Tree-masked attention on the matrix cores for few query rows per KV head (M = N*G <= 64 rows), and for fp32 data
// at any M (64 rows at a time): paper Sec. 3.2; every drafted node attends to the whole prefix, so with 64 rows a
// K/V byte of 16-bit data only feeds 64 FLOP and the kernel is a stream over K and V.
//
// With so few rows one (sequence, KV head) cannot occupy a CU by splitting rows, so the waves of a workgroup split
// the KEYS instead: wave w owns row block w % RBW (32 rows) and key group w / RBW.  A round is one 32-key tile per
// key group; a ring of NR rounds lives in LDS (direct-to-LDS loads, XOR-swizzled), NR - 1 of them in flight while
// one is consumed.  Every wave keeps its own online-softmax state over its key group; at the end of a segment (a run
// of tiles of one unit, attn_division.h) the states of a row are merged through LDS, while the ring already fills for the
// next segment, and written.  Tree rows are the unit's last tiles, masked with the 128-bit ancestor sets built
// from parent[].
//   16-bit data: v_mfma_f32_32x32x16, K read as 16-byte row pieces, V^T through the transposing LDS read.
//   fp32 data:   v_mfma_f32_32x32x2_f32 (fp32 products and sums, 256 FLOP/clock/CU -- what the vector ALUs have, but
//                fed by one LDS value per 32 products instead of two per product).  The reduction index of Q.K is
//                permuted (lane half g takes elements 8 t + 4 g .. + 3) so that both operands are 16-byte reads, and
//                P^T is used straight out of the score accumulator: register j of lane half g holds key
//                8 (j/4) + 4 g + j%4, so step j multiplies V rows that far apart.
#pragma once
#include "attn_step.h"

namespace s4c {

namespace {

using namespace mfma;
using parts::Elem;
using parts::kB16;
using parts::kF32;
using parts::kH16;

constexpr int kBN = 32;                      // keys per tile
// By how much (log2) a row's maximum may outgrow the reference that its exponentials are taken against.  Where the
// probabilities keep all their bits (fp32 data, or Prob's parts) any reference gives the same result, and a lagging one saves
// rescaling the output.  Where they are rounded to the storage type the reference is the maximum: the largest ones, 1 or close below, round
// with the least error then.  Error against 64 bits (2-norm; 32 heads, 1024 keys + 60 nodes, bf16) 2.27e-3 lagging,
// 2.10e-3 with the maximum; fp16, 731 keys: 2.84e-4 and 2.66e-4.
template <bool ROUNDED>
constexpr float kLagLog2 = ROUNDED ? 0.0f : 8.0f;
constexpr int kAuxB = kMaxNodes * 16 + kMaxNodes * 4;

// KG key groups x RBW row blocks of 32 = waves; NR rounds in the ring.
template <Elem E, int D_, int KG_, int RBW_, int NR_>
struct Cfg {
    static constexpr Elem kElem = E;
    static constexpr int kD = D_, kKG = KG_, kRBW = RBW_, kNR = NR_;
    static constexpr int kEs = E == kF32 ? 4 : 2;
    static constexpr int kRowB = kD * kEs;               // bytes per K/V row
    static constexpr int kTileKB = kBN * kRowB;          // K (or V) bytes of a tile
    static constexpr int kTileB = 2 * kTileKB;           // K then V
    static constexpr int kRoundB = kKG * kTileB;
    static constexpr int kRingB = kNR * kRoundB;
    static constexpr int kWaves = kKG * kRBW;
    static constexpr int kThreads = 64 * kWaves;
    static constexpr int kCH = kTileKB / 1024 / kRBW;    // direct-to-LDS loads per wave for its share of K (or V)
    // Where the key groups' states of a row meet (a region of its own, so that the ring keeps filling for the next segment): every
    // wave's (maximum, sum), and two of the eight-column pieces it sends.  kOwners groups share the output's 32-column blocks;
    // each adds up kOwn blocks of all groups.
    static constexpr int kDB = kD / 32, kOwners = kKG < kDB ? kKG : kDB, kOwn = kDB / kOwners;
    static constexpr int kMergeB = kWaves * (32 * 8 + 2 * 1024);
    static constexpr int kLdsBytes = kRingB + kAuxB + kMergeB;
    static_assert(kWaves * kDB * 4096 <= kRingB, "after a launch's only segment they meet in the ring");
    static_assert(sizeof(accept::Shared) <= kRingB, "the ring is also what the other workgroups of a step have");
    static constexpr int kPerCu = 2 * kLdsBytes <= 160 * 1024 ? 2 : 1;
    static_assert(kLdsBytes <= 160 * 1024, "LDS of one CU");
    static_assert(kCH >= 1 && 2 * kCH * (kNR - 1) < 64, "loads in flight are counted in vmcnt");
    // 16-byte chunk swizzle of row r: K is read as one chunk of 16 (or 32) consecutive rows at a time, V as 4 rows x
    // 64 bytes (16-bit) or two rows 4 apart x 128 bytes (fp32); both spread over all banks
    static __device__ __forceinline__ int k_swz(int r) {
        if constexpr (kRowB == 128) return (r >> 1) & 7;
        else return r & 15;
    }
    static __device__ __forceinline__ int v_swz(int r) {
        if constexpr (kElem == kF32) return ((r >> 2) & 1) << 3;
        else if constexpr (kRowB == 128) return ((r >> 1) & 1) << 2;
        else return (r & 3) << 2;
    }
};

template <class C, bool PAGED, StepKind STEP, parts::Merge MERGE>
__global__ __launch_bounds__(C::kThreads) __attribute__((amdgpu_waves_per_eu(C::kPerCu * C::kWaves / 4, 2)))
void tree_attn_smallm_kernel(AttnArgs a, StepTail<STEP> tail) {
    constexpr int kD = C::kD, kKG = C::kKG, kRBW = C::kRBW, kNR = C::kNR, kRowB = C::kRowB;
    constexpr int kThreads = C::kThreads, kCH = C::kCH;
    constexpr bool kIs32 = C::kElem == kF32, F16 = C::kElem == kH16;
    constexpr int kDB = C::kDB, kOwners = C::kOwners, kOwn = C::kOwn;
    constexpr int kParts = Prob<F16, kD>::kParts;             // (16-bit data)
    constexpr float kShift = kIs32 ? 0.f : Prob<F16, kD>::kShift;
    constexpr float kLag = kLagLog2<!kIs32 && kParts == 1>;
    constexpr int kLPR = kRowB / 16;                          // lanes (16-byte chunks) per row in a direct-to-LDS load
    constexpr int kRPI = 64 / kLPR;                           // rows per load instruction
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    if constexpr (STEP != kNoStep)
        if (__builtin_expect(blockIdx.y > 0, 0)) {          // (the attention's code first: a far jump at its start costs a fetch)
            rest_of_launch<C::kElem, STEP>(smem);
            return;
        }
    uint32_t* anc = (uint32_t*)(smem + C::kRingB);            // [kMaxNodes][4]
    int32_t* spar = (int32_t*)(anc + kMaxNodes * 4);          // [kMaxNodes]
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_u8*)smem;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rb = wave % kRBW, kg = wave / kRBW;
    const int N = a.N, G = a.G, M = a.M;
    const int g32 = lane >> 5;

    // the workgroups of a team (row tiles that walk the same keys) take consecutive slots of one XCD
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    const int team = work::team_id(a, xcd, slot / a.mtiles), mt = slot % a.mtiles;

    // per-lane offsets: direct-to-LDS loads (instruction ii covers rows kRPI ii ..), fragment reads inside a tile
    uint32_t kvo_k[kCH], kvo_v[kCH];
#pragma unroll
    for (int c = 0; c < kCH; ++c) {
        const int row = kRPI * (rb * kCH + c) + lane / kLPR, pc = lane % kLPR;
        kvo_k[c] = row * kRowB + ((pc ^ C::k_swz(row)) << 4);
        kvo_v[c] = row * kRowB + ((pc ^ C::v_swz(row)) << 4);
    }
    const int i16 = lane & 15, dhalf = (lane >> 4) & 1;
    constexpr int kKT = kIs32 ? kD / 8 : kD / 16;             // 16-byte K pieces per row and lane half
    // (block db of the accumulator is column block (db + kg kOwn) % kDB of the output, so that the blocks a group adds up are its first ones)
    uint32_t k_off[kKT], v_off[kDB];
    auto column_block = [&](int db) __attribute__((always_inline)) { return (db + kg * kOwn) % kDB; };
#pragma unroll
    for (int tt = 0; tt < kKT; ++tt) k_off[tt] = (lane & 31) * kRowB + (((2 * tt + g32) ^ C::k_swz(lane & 31)) << 4);
#pragma unroll
    for (int db = 0; db < kDB; ++db) {
        if constexpr (kIs32) {
            // element d = 32 db + lane % 32 of row 4 g32 (rows 8 q + 4 g32 + e follow at constant distances)
            const int d = 32 * column_block(db) + (lane & 31);
            v_off[db] = C::kTileKB + 4 * g32 * kRowB + (((d >> 2) ^ (g32 << 3)) << 4) + 4 * (d & 3);
        } else {
            const int vrow = 4 * g32 + (i16 >> 2);
            v_off[db] = C::kTileKB + vrow * kRowB + (((4 * column_block(db) + 2 * dhalf + ((i16 & 3) >> 1)) ^ C::v_swz(vrow)) << 4) + 8 * (i16 & 1);
        }
    }
    const ptrdiff_t v_minus_k = (const unsigned char*)a.v_cache - (const unsigned char*)a.k_cache;
    const ptrdiff_t vt_minus_kt = (const unsigned char*)a.v_tree - (const unsigned char*)a.k_tree;
    const uint32_t tree_stride = (uint32_t)a.Hkv * kRowB;

    const work::Lens lens(a);
    // ---- while the lengths are on their way: this lane's query row, and where its pieces of the wave's Q rows lie in a unit's
    const int rq0 = (mt * kRBW + rb) * 32;
    const int rq = rq0 + (lane & 31);
    const bool rvalid = rq < M;
    const int node = rvalid ? rq / G : 0, gh = rvalid ? rq - node * G : 0;
    size_t q_off[C::kTileKB / 1024];
    {
        // rows rq0 + kRPI c + lane / kLPR, one step of kRPI rows after the other; past the last row: the last
        const int r0 = rq0 + lane / kLPR, step_nd = kRPI / G, step_g = kRPI - step_nd * G;
        int nd = r0 / G, g = r0 - nd * G;
        const size_t last = (size_t)(N - 1) * a.Hq + (G - 1);
#pragma unroll
        for (int c = 0; c < C::kTileKB / 1024; ++c) {
            const int row = kRPI * c + lane / kLPR, pc = lane % kLPR;
            const size_t at = (size_t)nd * a.Hq + g;
            q_off[c] = (at < last ? at : last) * kRowB + ((pc ^ C::k_swz(row)) << 4);
            nd += step_nd;
            g += step_g;
            if (g >= G) { g -= G; ++nd; }
        }
    }
    if constexpr (MERGE == parts::kHere)
        if (wave == 0) parts::begin<kD>(a, team, mt);
    constexpr bool kOne = MERGE != parts::kShares;            // a share is one segment
    work::Walk cw;                                        // what is multiplied
    if constexpr (kOne) cw = work::walk_run(a, lens, team); else cw = work::walk_share(a, lens, team);
    if (cw.b < 0) {
        if constexpr (STEP != kNoStep) {
            __syncthreads();
            lens_read(tail, a, lens);
        }
        if constexpr (MERGE == parts::kHere || MERGE == parts::kNext)
            if (work::leaves_empty(a, team))
                parts::finish<kD, C::kElem, MERGE, C::kWaves, kRBW>(a, team, mt, smem, [&]() __attribute__((always_inline)) {
                    if (kg < kOwners) parts::put_empty<kD, kOwners, MERGE>(a, team, mt * kRBW + rb, kg);
                });
        lens_end<STEP>(lens_look_back<STEP>());
        return;
    }
    work::Walk pw = cw;                                   // what is loaded
    int issued = 0, done = 0;                             // rounds

    // Loads the next round: tile kg of the KG tiles from pw.tile on (a round does not reach past its segment; a group
    // without a tile in a segment's last round fetches the segment's last tile again, so that every wave has the same
    // number of loads in flight, and does not compute on it).  Every address is in bounds whatever the inputs hold:
    // prefix rows lie below the usable length, page ids are clamped to the pool (a sequence with a bad one is
    // flagged and its result discarded).  Rounds of full prefix tiles take the short way: p_full of them are left in
    // the segment, this group's next tile at p_k (or, paged, at key p_key).
    int p_full = 0, p_key = 0;
    const unsigned char* p_k = nullptr;
    auto page_addr = [&](int k0) __attribute__((always_inline)) {               // (a tile never straddles pages: pages are powers of two >= 64 rows)
        int id = scalar_load_i32(uniform((const unsigned char*)(a.block_table + (size_t)pw.b * a.max_blocks)),
                                 (uint32_t)uniform(k0 >> a.page_shift) * 4u);
        id = (unsigned)id < (unsigned)a.num_pages ? id : 0;
        return uniform((const unsigned char*)a.k_cache +
                       ((((size_t)id * a.Hkv + pw.kvh) << a.page_shift) + (size_t)(k0 & ((1 << a.page_shift) - 1))) * kRowB);
    };
    auto cache_addr = [&](int k0) __attribute__((always_inline)) {
        return uniform((const unsigned char*)a.k_cache + (((size_t)pw.b * a.Hkv + pw.kvh) * (size_t)a.S_cap + k0) * kRowB);
    };
    auto begin_segment = [&]() __attribute__((always_inline)) {
        p_full = uniform(max(0, min(work::usable(a, lens.at(a, pw.b)) / kBN, pw.tile_end) - pw.tile) / kKG);
        p_key = (pw.tile + kg) * kBN;
        if constexpr (!PAGED) p_k = cache_addr(p_key);
    };
    begin_segment();
    auto stage_base = [&]() __attribute__((always_inline)) {
        return __builtin_amdgcn_readfirstlane(lds0 + ((uint32_t)issued % kNR) * C::kRoundB + kg * C::kTileB + rb * kCH * 1024);
    };
    auto issue_full = [&]() __attribute__((always_inline)) {
        const uint32_t sbase = stage_base();
        const unsigned char* kgp = PAGED ? page_addr(p_key) : uniform(p_k);
        const unsigned char* vgp = uniform(kgp + v_minus_k);
#pragma unroll
        for (int c = 0; c < kCH; ++c) {
            dma16(kgp, kvo_k[c], sbase + c * 1024);
            dma16(vgp, kvo_v[c], sbase + c * 1024 + C::kTileKB);
        }
        if constexpr (PAGED) p_key += kKG * kBN; else p_k += kKG * kBN * kRowB;
    };
    auto end_round = [&]() __attribute__((always_inline)) {
        if (pw.tile >= pw.tile_end) {
            if constexpr (kOne) pw.b = -1; else pw = work::walk_next(a, lens, pw);
            if (!kOne && pw.b >= 0) begin_segment();
        }
    };
    auto issue_round = [&]() __attribute__((always_inline)) {
        if (p_full > 0) {
            issue_full();
            --p_full;
        } else {
            const int P = work::usable(a, lens.at(a, pw.b)), u_pref = (P + kBN - 1) / kBN;
            const uint32_t sbase = stage_base();
            const int t = uniform(min(pw.tile + kg, pw.tile_end - 1));
            const bool tree = t >= u_pref;
            const int k0 = (tree ? t - u_pref : t) * kBN;
            const unsigned char* kgp;
            if (tree) kgp = uniform((const unsigned char*)a.k_tree + (((size_t)pw.b * N + k0) * a.Hkv + pw.kvh) * kRowB);
            else kgp = PAGED ? page_addr(k0) : cache_addr(k0);
            kgp = uniform(kgp);
            const unsigned char* vgp = uniform(kgp + (tree ? vt_minus_kt : v_minus_k));
            const int last = (tree ? N : P) - 1 - k0;                      // >= 0: last valid row of the tile
            const uint32_t rstride = tree ? tree_stride : (uint32_t)kRowB;
#pragma unroll
            for (int c = 0; c < kCH; ++c) {
                const int row = kRPI * (rb * kCH + c) + lane / kLPR, pc = lane % kLPR;
                const uint32_t roff = (uint32_t)min(row, last) * rstride;
                dma16(kgp, roff + ((pc ^ C::k_swz(row)) << 4), sbase + c * 1024);
                dma16(vgp, roff + ((pc ^ C::v_swz(row)) << 4), sbase + c * 1024 + C::kTileKB);
            }
        }
        ++issued;
        pw.tile += kKG;
        end_round();
    };
    // ---- The first segment's start is a chain of memory latencies, so everything it needs is requested at once:
    // parent[], this wave's 32 Q rows (into the ring's last round, swizzled like K rows), and the first NR - 1
    // rounds.  All of it goes straight to LDS, so that waiting for Q does not mean waiting for the rounds behind it
    // (the compiler knows nothing of these loads; a wait of its own for a register load counts them in).
    const uint32_t q_stage = (uint32_t)(kNR - 1) * C::kRoundB + wave * C::kTileKB;
    bool len_bad = work::usable(a, lens.at(a, cw.b)) != lens.at(a, cw.b);
    if constexpr (PAGED) len_bad = len_bad || work::pages_are_bad(a, cw.b, work::usable(a, lens.at(a, cw.b)));
    if (wave < 2 && wave * 64 + lane < N)
        dma4(a.parent + (size_t)cw.b * N + wave * 64 + lane,
             __builtin_amdgcn_readfirstlane(lds0 + C::kRingB + kMaxNodes * 16 + wave * 256));
    {
        const unsigned char* qb = (const unsigned char*)a.q + ((size_t)cw.b * N * a.Hq + cw.kvh * G) * kRowB;
#pragma unroll
        for (int c = 0; c < C::kTileKB / 1024; ++c) dma16(qb + q_off[c], __builtin_amdgcn_readfirstlane(lds0 + q_stage + c * 1024));
    }
#pragma unroll
    for (int r = 0; r < kNR - 1; ++r)
        if (pw.b >= 0) issue_round();
    if constexpr (STEP != kNoStep) {
        __syncthreads();
        lens_read(tail, a, lens);
    }
    if (issued == kNR - 1) wait_vmcnt<2 * kCH * (kNR - 1)>(); else wait_vmcnt<0>();

    // ---- this lane's query row; a later segment's Q fragments (and parent[]) are loaded before the previous one is
    // written out
    uint4 qf[kKT];           // 16-bit: elements 16 t + 8 g32 .. + 7; fp32: elements 8 t + 4 g32 .. + 3
#pragma unroll
    for (int t = 0; t < kKT; ++t) {
        qf[t] = *(const uint4*)(smem + q_stage + k_off[t]);
        if (!rvalid) qf[t] = make_uint4(0, 0, 0, 0);
    }
    auto load_q = [&](int b, int kvh) __attribute__((always_inline)) {
        const unsigned char* qrow = (const unsigned char*)a.q + ((((size_t)b * N + node) * a.Hq + kvh * G + gh) * kD) * C::kEs + g32 * 16;
#pragma unroll
        for (int t = 0; t < kKT; ++t) {
            qf[t] = make_uint4(0, 0, 0, 0);
            if (rvalid) qf[t] = *(const uint4*)(qrow + 32 * t);
        }
    };
    int parent = -1, b_known = cw.b;
    bool masks = false;                                       // anc[] holds b_known's masks
    while (cw.b >= 0) {
        const int b = cw.b, kvh = cw.kvh;
        const int P = work::usable(a, lens.at(a, b)), u_pref = (P + kBN - 1) / kBN;
        const int t_end = uniform(cw.tile_end);
        if (b != b_known) {
            b_known = b;
            masks = false;
            len_bad = P != lens.at(a, b);
            if constexpr (PAGED) len_bad = len_bad || work::pages_are_bad(a, b, P);
            __syncthreads();                                  // the previous sequence's parent[] is no longer read
            if (tid < N) spar[tid] = parent;
            __syncthreads();
        }
        // ancestor words of this row, pre-shifted for this half of the wave
        uint32_t amask[4] = {0, 0, 0, 0};
        if (t_end > u_pref) {
            if (!masks) {
                __syncthreads();                              // (the first segment: parent[] has landed)
                if (!work::tree_is_bad(a, spar)) work::build_masks(a, spar, anc);
                else if (tid < N) *(uint4*)(anc + tid * 4) = make_uint4(0, 0, 0, 0);
                __syncthreads();
                masks = true;
            }
            if (rvalid) {
#pragma unroll
                for (int q = 0; q < 4; ++q) amask[q] = anc[node * 4 + q] >> (4 * g32);
            }
        }

        f32x16 o[kDB];
#pragma unroll
        for (int db = 0; db < kDB; ++db)
#pragma unroll
            for (int j = 0; j < 16; ++j) o[db][j] = 0.f;
        float m_run = -INFINITY, l_run = 0.f;

        // one 32-key tile: S^T = K Q^T, (mask,) online softmax, O^T += V^T P^T
        // masked: bit 8 (j/4) + j%4 of `visible` tells whether register j's key counts for this lane's row
        auto tile = [&](auto masked_tag, uint32_t visible) __attribute__((always_inline)) {
            constexpr bool MASKED = decltype(masked_tag)::value;
            const lds_u8* stage = (const lds_u8*)smem + ((uint32_t)done % kNR) * C::kRoundB + kg * C::kTileB;
            f32x16 s;
#pragma unroll
            for (int j = 0; j < 16; ++j) s[j] = 0.f;
            if constexpr (kIs32) {
                typedef __attribute__((address_space(3))) f32x4 lds_f32x4;
#pragma unroll
                for (int t0 = 0; t0 < kKT; t0 += 8) {
                    f32x4 kf[8];
#pragma unroll
                    for (int t = 0; t < 8; ++t) kf[t] = *(const lds_f32x4*)(stage + k_off[t0 + t]);
#pragma unroll
                    for (int t = 0; t < 8; ++t) {
                        const f32x4 q4 = __builtin_bit_cast(f32x4, qf[t0 + t]);
#pragma unroll
                        for (int e = 0; e < 4; ++e) s = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[t][e], q4[e], s, 0, 0, 0);
                    }
                }
            } else {
                bf16x8 kf[kKT];
#pragma unroll
                for (int tt = 0; tt < kKT; ++tt) kf[tt] = *(const lds_bf16x8*)(stage + k_off[tt]);
                f32x16 s1;
#pragma unroll
                for (int j = 0; j < 16; ++j) s1[j] = 0.f;
#pragma unroll
                for (int tt = 0; tt < kKT; tt += 2) {        // two chains over the head dimension, summed below
                    s = mma32<F16>(kf[tt], __builtin_bit_cast(bf16x8, qf[tt]), s);
                    s1 = mma32<F16>(kf[tt + 1], __builtin_bit_cast(bf16x8, qf[tt + 1]), s1);
                }
#pragma unroll
                for (int j = 0; j < 16; ++j) s[j] += s1[j];
            }
            if constexpr (MASKED) {
#pragma unroll
                for (int j = 0; j < 16; ++j)
                    if (!((visible >> ((j >> 2) * 8 + (j & 3))) & 1u)) s[j] = -INFINITY;
            }
            float mx = s[0];
#pragma unroll
            for (int j = 1; j < 16; j += 2) mx = __builtin_fmaxf(__builtin_fmaxf(mx, s[j]), s[(j + 1) & 15]);
            mx = max_across_halves(mx) * a.scale_log2;
            // The reference moves only when some row of the wave outgrew it by more than 2^kLag (always at its first
            // visible key); until then the accumulator is not touched.
            if (__any(mx > m_run + kLag)) {
                const float m_new = fmaxf(m_run, mx);
                float alpha = fast_exp2(m_run - m_new);                      // first tile: exp2(-inf) = 0
                if constexpr (MASKED) alpha = (m_new == -INFINITY) ? 1.f : alpha;
                l_run *= alpha;
#pragma unroll
                for (int db = 0; db < kDB; ++db)
#pragma unroll
                    for (int j = 0; j < 16; ++j) o[db][j] *= alpha;
                m_run = m_new;
            }
            float m_ref = m_run;
            if constexpr (MASKED) m_ref = (m_run == -INFINITY) ? 0.f : m_run;     // nothing visible yet: all terms are 0
            float psum = 0.f;
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                const float p = fast_exp2(fmaf(s[j], a.scale_log2, kShift - m_ref));
                s[j] = p;
                psum += p;
            }
            l_run += psum;

            if constexpr (kIs32) {
                typedef __attribute__((address_space(3))) float lds_f32;
#pragma unroll
                for (int jq = 0; jq < 4; ++jq)
#pragma unroll
                    for (int db = 0; db < kDB; ++db) {
                        float vf[4];
#pragma unroll
                        for (int e = 0; e < 4; ++e) vf[e] = *(const lds_f32*)(stage + v_off[db] + (8 * jq + e) * kRowB);
#pragma unroll
                        for (int e = 0; e < 4; ++e) o[db] = __builtin_amdgcn_mfma_f32_32x32x2f32(vf[e], s[4 * jq + e], o[db], 0, 0, 0);
                    }
            } else {
                auto vfrag = [&](const lds_u8* p) __attribute__((always_inline)) {
                    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)p);
                    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p + 8 * kRowB));
                    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
                };
                bf16x8 vf[2][kDB];
#pragma unroll
                for (int st = 0; st < 2; ++st)
#pragma unroll
                    for (int db = 0; db < kDB; ++db) vf[st][db] = vfrag(stage + st * 16 * kRowB + v_off[db]);
#pragma unroll
                for (int part = 0; part < kParts; ++part)
#pragma unroll
                    for (int st = 0; st < 2; ++st) {
                        const bf16x8 pb = part + 1 < kParts ? take8<F16>(s, 8 * st) : round8<F16>(s, 8 * st);
#pragma unroll
                        for (int db = 0; db < kDB; ++db) o[db] = mma32<F16>(vf[st][db], pb, o[db]);
                    }
            }
        };

        // ---- round pipeline.  Settle the Q fragments here, so that the compiler places no vmcnt wait of its own
        // inside the round loop (which would also wait for the rounds just issued).
#pragma unroll
        for (int t = 0; t < kKT; ++t) asm volatile("" : "+v"(qf[t].x), "+v"(qf[t].y), "+v"(qf[t].z), "+v"(qf[t].w));
        auto sync_and_prefetch = [&]() __attribute__((always_inline)) {
            // this wave's share of round `done` has landed once at most NR - 2 younger rounds are outstanding
            if (kNR > 2 && issued - done == kNR - 1) wait_vmcnt<2 * kCH * (kNR - 2)>(); else wait_vmcnt<0>();
            __syncthreads();           // everybody's has; the round before it is no longer read
            if (pw.b >= 0) issue_round();
        };
        int t = uniform(cw.tile);
        for (const int e = min(P / kBN, t_end) - kKG; t <= e; t += kKG, ++done) {
            sync_and_prefetch();
            tile(std::integral_constant<bool, false>{}, 0u);
        }
        for (; t < t_end; t += kKG, ++done) {
            sync_and_prefetch();
            const int my = t + kg;
            if (my >= t_end) continue;
            uint32_t visible;
            if (my >= u_pref) {
                const int word = my - u_pref;                            // 32-node word of this tile (< 4 since N <= 128)
                visible = (word == 0 ? amask[0] : word == 1 ? amask[1] : word == 2 ? amask[2] : amask[3]);
            } else {
                const int nvalid = P - my * kBN;                         // the ragged last prefix tile: 1 .. 31 keys
                visible = (nvalid >= kBN ? 0xFFFFFFFFu : (1u << nvalid) - 1u) >> (4 * g32);
            }
            tile(std::integral_constant<bool, true>{}, visible);
        }

        work::Walk nw = cw;
        if constexpr (!kOne) {
            nw = work::walk_next(a, lens, cw);
            if (nw.b >= 0) {
                if (nw.b != b && tid < N) parent = a.parent[(size_t)nw.b * N + tid];
                load_q(nw.b, nw.kvh);
            }
        }
        const int flagged = (work::tree_is_bad(a, spar) ? S4C_SEQ_BAD_TREE : 0) | (len_bad ? S4C_SEQ_BAD_LEN : 0);
        if (a.status && tid == 0 && cw.tile == 0 && kvh == 0 && mt == 0) a.status[b] = flagged;
        float l_tot = l_run + __shfl_xor(l_run, 32);
        if (flagged) {                                        // zero output, whatever was read in place of a bad page
            l_tot = 0.f;
#pragma unroll
            for (int db = 0; db < kDB; ++db)
#pragma unroll
                for (int j = 0; j < 16; ++j) o[db][j] = 0.f;
        }
        // ---- The key groups of each row meet in LDS: a group sends its later blocks and adds up its first kOwn.  The sums of
        // block db come from the groups that are db / kOwn before this one, modulo kOwners.
        // (One group that added up everything, a block at a time: 1.8 us from the last tile to the last store; 1.1 so.)
        float* const mml = (float*)(smem + C::kRingB + kAuxB);                // [waves][32 rows][2]
        if (g32 == 0) *(float2*)(mml + (wave * 32 + lane) * 2) = make_float2(m_run, l_tot);
        float m_max = -INFINITY, w_own = 0.f;
        auto weight = [&](int g) __attribute__((always_inline)) {             // 0: the group saw nothing visible
            const float2 ml = *(const float2*)(mml + ((g * kRBW + rb) * 32 + (lane & 31)) * 2);
            return ml.y > 0.f ? fast_exp2(ml.x - m_max) : 0.f;
        };
        auto meet = [&](auto alone_tag) __attribute__((always_inline)) {
            // the launch's only segment: the ring is free once every wave is through, and holds everything at once;
            // else two pieces of every wave at a time
            constexpr bool ALONE = decltype(alone_tag)::value;
            constexpr int kJ = ALONE ? 4 : 2;
            f32x4* const ex = (f32x4*)(ALONE ? smem : (unsigned char*)(mml + C::kWaves * 64));
            auto at = [&](int w, int db, int jq) __attribute__((always_inline)) { return ex + (ALONE ? (w * kDB + db) * 4 + jq : w * 2 + (jq & 1)) * 64 + lane; };
            auto send = [&](int db, int j0) __attribute__((always_inline)) {
                if (db < kOwn && kg < kOwners) return;
#pragma unroll
                for (int jq = j0; jq < j0 + kJ; ++jq)
                    *at(wave, db, jq) = f32x4{o[db][4 * jq], o[db][4 * jq + 1], o[db][4 * jq + 2], o[db][4 * jq + 3]};
            };
            constexpr int kFirst = kKG > kOwners ? 0 : kOwn;                  // first block that some group sends
            if constexpr (ALONE) {
                __syncthreads();
#pragma unroll
                for (int db = kFirst; db < kDB; ++db) send(db, 0);
            } else {
                send(kFirst, 0);
            }
            __syncthreads();
            l_tot = 0.f;
#pragma unroll
            for (int g = 0; g < kKG; ++g) {
                const float2 ml = *(const float2*)(mml + ((g * kRBW + rb) * 32 + (lane & 31)) * 2);
                m_max = fmaxf(m_max, ml.y > 0.f ? ml.x : -INFINITY);
            }
#pragma unroll
            for (int g = 0; g < kKG; ++g) l_tot = fmaf(mml[((g * kRBW + rb) * 32 + (lane & 31)) * 2 + 1], weight(g), l_tot);
            w_own = weight(kg);
            if (kg < kOwners)                                                 // (the others send what is left as it is: who adds it up weights it)
#pragma unroll
                for (int db = 0; db < kOwn; ++db)
#pragma unroll
                    for (int j = 0; j < 16; ++j) o[db][j] *= w_own;
#pragma unroll
            for (int db = kFirst; db < kDB; ++db)
#pragma unroll
                for (int j0 = 0; j0 < 4; j0 += kJ) {
                    if (!ALONE && (db > kFirst || j0 > 0)) {
                        __syncthreads();
                        send(db, j0);
                        __syncthreads();
                    }
                    if (kg < kOwners)
#pragma unroll
                        for (int g0 = 0; g0 < kKG; g0 += kOwners) {
                            const int g = g0 + (kg - db / kOwn + kOwners) % kOwners;
                            if (g == kg) continue;
                            const float w = weight(g);
#pragma unroll
                            for (int jq = j0; jq < j0 + kJ; ++jq) {
                                const f32x4 v = *at(g * kRBW + rb, db, jq);
#pragma unroll
                                for (int e = 0; e < 4; ++e) o[db % kOwn][4 * jq + e] = fmaf(v[e], w, o[db % kOwn][4 * jq + e]);
                            }
                        }
                }
        };
        meet(std::integral_constant<bool, kOne>{});
        if (!kOne && mt == 0 && tid == 0) work::note_parts(a, team, cw);
        // ---- the row's columns: d = 32 column_block(db) + 8 (j/4) + 4 g32 + (j%4)
        auto piece = [&](int q) __attribute__((always_inline)) {
            return f32x4{o[q >> 2][4 * (q & 3)], o[q >> 2][4 * (q & 3) + 1], o[q >> 2][4 * (q & 3) + 2], o[q >> 2][4 * (q & 3) + 3]};
        };
        const uint64_t left = lens_look_back<STEP>();
        if constexpr (MERGE == parts::kHere || MERGE == parts::kNext) {
            parts::finish<kD, C::kElem, MERGE, C::kWaves, kRBW>(a, team, mt, smem, [&]() __attribute__((always_inline)) {
                if (kg < kOwners) parts::put<kD, kOwners, MERGE>(a, team, mt * kRBW + rb, kg, m_max, l_tot, piece);
            });
            lens_end<STEP>(left);
            return;
        }
        if (MERGE == parts::kWhole || work::walk_is_whole(a, cw)) {
            const float inv = (l_tot > 0.f) ? 1.f / l_tot : 0.f;
            const size_t o0 = (((size_t)b * a.N + node) * a.Hq + kvh * G + gh) * kD + 32 * kOwn * kg + 4 * g32;
            if (rvalid && kg < kOwners)
#pragma unroll
                for (int q = 0; q < 4 * kOwn; ++q) parts::store_out<C::kElem>(a.out, o0 + 8 * q, piece(q) * inv);
        } else if (rvalid && kg < kOwners) {
            const size_t prow = work::part_row(a, team, work::part_slot(cw)) + rq;
            float* orow = a.ws_o + prow * kD + 32 * kOwn * kg + 4 * g32;
#pragma unroll
            for (int q = 0; q < 4 * kOwn; ++q) *(f32x4*)(orow + 8 * q) = piece(q);
            if (kg == 0 && g32 == 0) *(float2*)(a.ws_ml + prow * 2) = make_float2(m_max, l_tot);
        }
        lens_end<STEP>(left);
        if constexpr (kOne) return;
        cw = nw;
    }
}

template <class C, bool PAGED, StepKind STEP, parts::Merge MERGE>
hipError_t launch(AttnArgs a, StepTail<STEP> tail, hipStream_t st) {
    static std::atomic<uint64_t> lds_set{0};
    const hipError_t ea = ensure_dynamic_lds((const void*)tree_attn_smallm_kernel<C, PAGED, STEP, MERGE>, C::kLdsBytes, lds_set);
    if (ea != hipSuccess) return ea;
    a.attn_wgs = attn_workgroups(a);
    const dim3 grid = launch_grid(a, rest_of(a, tail)), block(C::kThreads);
    hipLaunchKernelGGL((tree_attn_smallm_kernel<C, PAGED, STEP, MERGE>), grid, block, C::kLdsBytes, st, a, tail);
    return hipGetLastError();
}
template <class C, bool PAGED, StepKind STEP>
hipError_t launch(const AttnArgs& a, const StepTail<STEP>& tail, hipStream_t st) {
    if (a.split == 1) return launch<C, PAGED, STEP, parts::kWhole>(a, tail, st);
    if constexpr (STEP == kNoStep)
        if (a.split == 0) return launch<C, PAGED, STEP, parts::kShares>(a, tail, st);
    if constexpr (!PAGED && STEP == kNoStep)
        if (a.tag == 0) return launch<C, PAGED, STEP, parts::kNext>(a, tail, st);
    return launch<C, PAGED, STEP, parts::kHere>(a, tail, st);
}

// The configuration for an element type, head size and rows per workgroup (attn_tile_small), handed to `use` as a type.
// 32 rows: one row block, four key groups, so that no wave works on rows that do not exist.
template <Elem E, class Use>
auto with_cfg(int D, int rows, Use use) {
    if constexpr (E == kF32) {
        if (D == 64) return rows == 32 ? use(Cfg<E, 64, 4, 1, 2>{}) : use(Cfg<E, 64, 2, 2, 2>{});
        return use(Cfg<E, 128, 2, 2, 2>{});          // (four key groups of 32 KB tiles would not fit twice)
    } else {
        // (64 rows of head size 64: tiles of 8 KB, so four rounds are the same 64 KB of loads in flight)
        if (D == 64) return rows == 32 ? use(Cfg<E, 64, 4, 1, 2>{}) : use(Cfg<E, 64, 2, 2, 4>{});
        return rows == 32 ? use(Cfg<E, 128, 4, 1, 2>{}) : use(Cfg<E, 128, 2, 2, 2>{});
    }
}
// A launch for one element type; instantiated in a translation unit of its own each (they take a minute to compile).
template <Elem E>
hipError_t launch_smallm(const AttnArgs& a, const StepTail<kGreedyStep>* step, hipStream_t st) {
    return with_cfg<E>(a.D, a.tile_rows, [&](auto c) {
        typedef decltype(c) C;
        if (step)
            return step->accept.mode == S4C_GREEDY ? launch<C, false>(a, StepTail<kGreedyStep>(*step), st)
                                                   : launch<C, false>(a, StepTail<kStochasticStep>(*step), st);
        return a.block_table ? launch<C, true>(a, StepTail<kNoStep>(), st) : launch<C, false>(a, StepTail<kNoStep>(), st);
    });
}

}  // namespace

}  // namespace s4c

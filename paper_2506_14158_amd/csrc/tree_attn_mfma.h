// Tree-masked attention on the CDNA4 matrix cores (paper Sec. 3.2, Fig. 3): bf16 or fp16 in, fp32
// accumulate, more than 64 query rows per KV head (fewer: tree_attn_smallm.h); head size 64 or 128.
//
// The N tree nodes times the G query heads that share one KV head form a dense tile of
// M = N*G query rows, so both contractions run on v_mfma_f32_32x32x16_bf16 (_f16 for fp16 data).
//   * One workgroup = WR waves; wave w owns 32 query rows.  All waves share the K/V tiles
//     (64 keys) that the workgroup streams from HBM straight into LDS with
//     global_load_lds_dwordx4 (no staging registers), through a ring of NS tiles: the loads of
//     tile t+NS-1 are issued before tile t is consumed, so several tiles are in flight per CU
//     while the matrix cores work.
//   * Scores are computed transposed, S^T = K Q^T (A = K rows from LDS, B = Q^T kept in
//     registers), so every lane owns one query row: the running max / sum and the rescaling of
//     the output accumulator need no cross-lane traffic (one v_permlane32_swap joins the two
//     halves of a row), and the exponentiated scores already sit in the B-operand layout of the
//     second contraction O^T += V^T P^T.
//   * V^T fragments come from the row-major V tile through the transposing LDS read
//     (ds_read_b64_tr_b16), so V is never transposed in memory.
//   * A direct-to-LDS load writes 1 KB contiguous per wave, so rows cannot be padded; instead the
//     16-byte chunks of a row are XOR-swizzled (K: chunk ^ (row & 15); V: chunk ^ ((row & 3) << 2)),
//     applied on the global-address side of the load.  That makes the 16-byte row reads of K and
//     the 4-row x 64-byte transposing reads of V bank-conflict free.  (Head size 64: two rows share
//     256 bytes of banks, so K uses chunk ^ ((row >> 1) & 7) and V chunk ^ (((row >> 1) & 1) << 2).)
//   * Full prefix tiles run a mask-free body.  The ragged last prefix tile and the tree rows
//     (extra tiles whose scores are kept only where the key node is the query node or one of its
//     ancestors; 128-bit masks built from parent[] in LDS) run a masked copy of the body.  Rows
//     past the end of a ragged tile are clamped to its last valid row (in bounds, finite).
//   * The keys are divided between teams of workgroups (attn_division.h); parts of a divided unit are written
//     unnormalised (attn_parts.h, attn_merge.h).
#pragma once
#include "attn_step.h"

namespace s4c {

namespace {

using namespace mfma;

constexpr int kBN = 64;                     // keys per tile
constexpr float kLazyLog2 = 8.0f;           // full tiles rescale only when a row maximum grew by more than 2^8
constexpr int lds_bytes_for(int ns, int d) { return ns * 2 * kBN * d * 2 + kMaxNodes * 16 + kMaxNodes * 4; }

template <int WR, int NS, int WPE, bool PAGED, bool F16, int kD, StepKind STEP, parts::Merge MERGE>
__global__ __launch_bounds__(WR * 64) __attribute__((amdgpu_waves_per_eu(WPE, WPE)))
void tree_attn_mfma_kernel(AttnArgs a, StepTail<STEP> tail) {
    constexpr int NT = WR * 64;
    constexpr int BM = WR * 32;
    constexpr int kRowB = kD * 2;                // bytes per K/V row
    constexpr int kTileB = kBN * kRowB;          // bytes per K (or V) tile
    constexpr int kStageB = 2 * kTileB;          // K then V
    constexpr int kLPR = kRowB / 16;             // lanes (16-byte chunks) per row in a direct-to-LDS load
    constexpr int kRPI = 64 / kLPR;              // rows per load instruction
    constexpr int kKT = kD / 16, kDB = kD / 32;  // MFMA steps of the scores; 32-column blocks of the output
    constexpr int kParts = Prob<F16, kD>::kParts;
    constexpr float kShift = Prob<F16, kD>::kShift;
    auto k_swz = [](int r) { return kD == 64 ? (r >> 1) & 7 : r & 15; };
    auto v_swz = [](int r) { return kD == 64 ? ((r >> 1) & 1) << 2 : (r & 3) << 2; };
    constexpr int CH = (kBN * kD / 8) / NT;      // direct-to-LDS loads per thread per K (or V) tile
    static_assert(CH >= 1, "tile smaller than the workgroup");
    static_assert(NS >= 2 && 2 * CH * (NS - 2) < 64, "too many loads in flight for vmcnt");

    static_assert(sizeof(accept::Shared) <= NS * kStageB, "the ring is also what the other workgroups of a step have");
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    constexpr parts::Elem kElem = F16 ? parts::kH16 : parts::kB16;
    if constexpr (STEP != kNoStep)
        if (__builtin_expect(blockIdx.y > 0, 0)) {          // (the attention's code first: a far jump at its start costs a fetch)
            rest_of_launch<kElem, STEP>(smem);
            return;
        }
    uint32_t* anc = (uint32_t*)(smem + NS * kStageB);        // [kMaxNodes][4]
    int32_t* spar = (int32_t*)(anc + kMaxNodes * 4);         // [kMaxNodes]
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_u8*)smem;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int N = a.N, G = a.G, M = a.M;

    // Workgroups are handed to the 8 XCDs round-robin by linear id.  The workgroups of a team -- the row tiles of
    // one unit, walking the same keys -- take consecutive slots of ONE XCD and share the K/V rows through its L2.
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    const int team = work::team_id(a, xcd, slot / a.mtiles), mt = slot % a.mtiles;

    // ---- direct-to-LDS tile loads.  Load c of a wave (instruction ii = wave + WR c of the tile) covers rows
    // kRPI ii .. : lane -> (row, physical chunk) and fetches the logical chunk that the swizzle maps there.  For full
    // prefix tiles the per-lane byte offsets are loop invariants and the tile base advances in scalar registers.
    uint32_t kvo_k[CH], kvo_v[CH];
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        const int row = kRPI * (wave + WR * c) + lane / kLPR, pc = lane % kLPR;
        kvo_k[c] = row * kRowB + ((pc ^ k_swz(row)) << 4);
        kvo_v[c] = row * kRowB + ((pc ^ v_swz(row)) << 4);
    }
    // per-lane LDS byte offsets inside a stage
    const int g32 = lane >> 5;                    // which half of the wave
    const int i16 = lane & 15, dhalf = (lane >> 4) & 1;
    uint32_t k_off[kKT], v_off[kDB];
#pragma unroll
    for (int tt = 0; tt < kKT; ++tt) k_off[tt] = (lane & 31) * kRowB + (((2 * tt + g32) ^ k_swz(lane & 31)) << 4);
#pragma unroll
    for (int db = 0; db < kDB; ++db) {
        const int vrow = 4 * g32 + (i16 >> 2);
        v_off[db] = kTileB + vrow * kRowB + (((4 * db + 2 * dhalf + ((i16 & 3) >> 1)) ^ v_swz(vrow)) << 4) + 8 * (i16 & 1);
    }

    const work::Lens lens(a);
    // ---- while the lengths are on their way: this lane's query row, and where its pieces of the wave's Q rows lie in a unit's
    const int rq0 = mt * BM + wave * 32;
    const bool wave_on = rq0 < M;                         // some of this wave's rows exist
    const int rq = rq0 + (lane & 31);
    const bool rvalid = rq < M;
    const int node = rvalid ? rq / G : 0, g = rvalid ? rq - node * G : 0;
    size_t q_off[32 / kRPI];
    {
        // rows rq0 + kRPI c + lane / kLPR, one step of kRPI rows after the other; past the last row: the last
        const int r0 = rq0 + lane / kLPR, step_nd = kRPI / G, step_g = kRPI - step_nd * G;
        int nd = r0 / G, gg = r0 - nd * G;
        const size_t last = (size_t)(N - 1) * a.Hq + (G - 1);
#pragma unroll
        for (int c = 0; c < 32 / kRPI; ++c) {
            const int row = kRPI * c + lane / kLPR, pc = lane % kLPR;
            const size_t at = (size_t)nd * a.Hq + gg;
            q_off[c] = (at < last ? at : last) * kRowB + ((pc ^ k_swz(row)) << 4);
            nd += step_nd;
            gg += step_g;
            if (gg >= G) { gg -= G; ++nd; }
        }
    }
    if constexpr (MERGE == parts::kHere)
        if (wave == 0) parts::begin<kD>(a, team, mt);
    constexpr bool kOne = MERGE != parts::kShares;        // a share is one segment
    work::Walk cw;                                        // what is multiplied
    if constexpr (kOne) cw = work::walk_run(a, lens, team); else cw = work::walk_share(a, lens, team);
    if (cw.b < 0) {
        if constexpr (STEP != kNoStep) {
            __syncthreads();
            lens_read(tail, a, lens);
        }
        if constexpr (MERGE == parts::kHere || MERGE == parts::kNext)
            if (work::leaves_empty(a, team))
                parts::finish<kD, kElem, MERGE, WR, WR>(a, team, mt, smem, [&]() __attribute__((always_inline)) { parts::put_empty<kD, 1, MERGE>(a, team, mt * WR + wave, 0); });
        lens_end<STEP>(lens_look_back<STEP>());
        return;
    }
    work::Walk pw = cw;                                   // what is loaded
    const int n_share = uniform(cw.left + cw.tile_end - cw.tile);
    int issued = 0, done = 0;
    const ptrdiff_t v_minus_k = (const unsigned char*)a.v_cache - (const unsigned char*)a.k_cache;
    const ptrdiff_t vt_minus_kt = (const unsigned char*)a.v_tree - (const unsigned char*)a.k_tree;
    const uint32_t tree_stride = (uint32_t)a.Hkv * kRowB;

    // Loads the next tile of the share (tile `issued`, ring stage issued % NS).  Every address is in bounds whatever
    // the inputs hold: prefix rows lie below the usable length, page ids are clamped to the pool (a sequence with a bad
    // one is flagged and its result discarded).  Full prefix tiles take the short way: p_full of them are left in the
    // segment, the next one at p_k (or, paged, at key p_key).
    int p_full = 0, p_key = 0;
    const unsigned char* p_k = nullptr;
    auto page_addr = [&](int k0) __attribute__((always_inline)) {               // (a tile never straddles pages: pages are powers of two >= the tile)
        int id = scalar_load_i32(uniform((const unsigned char*)(a.block_table + (size_t)pw.b * a.max_blocks)),
                                 (uint32_t)uniform(k0 >> a.page_shift) * 4u);
        id = (unsigned)id < (unsigned)a.num_pages ? id : 0;
        return uniform((const unsigned char*)a.k_cache +
                       ((((size_t)id * a.Hkv + pw.kvh) << a.page_shift) + (size_t)(k0 & ((1 << a.page_shift) - 1))) * kRowB);
    };
    auto begin_segment = [&]() __attribute__((always_inline)) {
        p_full = uniform(max(0, min(work::usable(a, lens.at(a, pw.b)) / kBN, pw.tile_end) - pw.tile));
        p_key = pw.tile * kBN;
        if constexpr (!PAGED)
            p_k = uniform((const unsigned char*)a.k_cache + (((size_t)pw.b * a.Hkv + pw.kvh) * (size_t)a.S_cap + p_key) * kRowB);
    };
    begin_segment();
    auto stage_base = [&]() __attribute__((always_inline)) {
        return __builtin_amdgcn_readfirstlane(lds0 + ((uint32_t)issued % NS) * kStageB + wave * 1024);
    };
    auto issue_full = [&]() __attribute__((always_inline)) {
        const uint32_t sbase = stage_base();
        const unsigned char* kg = PAGED ? page_addr(p_key) : uniform(p_k);
        const unsigned char* vg = uniform(kg + v_minus_k);
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            dma16(kg, kvo_k[c], sbase + WR * c * 1024);
            dma16(vg, kvo_v[c], sbase + WR * c * 1024 + kTileB);
        }
        if constexpr (PAGED) p_key += kBN; else p_k += kBN * kRowB;
    };
    auto end_tile = [&]() __attribute__((always_inline)) {
        if (pw.tile == pw.tile_end) {
            if constexpr (kOne) pw.b = -1; else pw = work::walk_next(a, lens, pw);
            if (!kOne && pw.b >= 0) begin_segment();
        }
    };
    auto issue_next = [&]() __attribute__((always_inline)) {
        ++pw.tile;
        if (p_full > 0) {
            issue_full();
            --p_full;
        } else {
            const int P = work::usable(a, lens.at(a, pw.b)), u_pref = (P + kBN - 1) / kBN;
            const uint32_t sbase = stage_base();
            const bool tree = pw.tile > u_pref;
            const int k0 = (pw.tile - 1 - (tree ? u_pref : 0)) * kBN;
            const unsigned char* kg;
            if (tree) kg = uniform((const unsigned char*)a.k_tree + (((size_t)pw.b * N + k0) * a.Hkv + pw.kvh) * kRowB);
            else kg = PAGED ? page_addr(k0) : uniform(p_k);
            kg = uniform(kg);
            const unsigned char* vg = uniform(kg + (tree ? vt_minus_kt : v_minus_k));
            const int last = (tree ? N : P) - 1 - k0;                       // >= 0: last valid row of the tile
            const uint32_t rstride = tree ? tree_stride : (uint32_t)kRowB;
#pragma unroll
            for (int c = 0; c < CH; ++c) {
                const int row = kRPI * (wave + WR * c) + lane / kLPR, pc = lane % kLPR;
                const uint32_t roff = (uint32_t)min(row, last) * rstride;
                dma16(kg, roff + ((pc ^ k_swz(row)) << 4), sbase + WR * c * 1024);
                dma16(vg, roff + ((pc ^ v_swz(row)) << 4), sbase + WR * c * 1024 + kTileB);
            }
        }
        ++issued;
        end_tile();
    };

    // ---- The first segment's start is a chain of memory latencies, so everything it needs is requested at once:
    // parent[], this wave's 32 Q rows (into the ring's last two stages, swizzled like K rows), and the tiles of the
    // other stages.  All of it goes straight to LDS, so that waiting for Q does not mean waiting for the tiles behind it
    // (the compiler knows nothing of these loads; a wait of its own for a register load counts them in).
    const uint32_t q_stage = (NS - 2) * kStageB + wave * (32 * kRowB);
    bool len_bad = work::usable(a, lens.at(a, cw.b)) != lens.at(a, cw.b);
    if constexpr (PAGED) len_bad = len_bad || work::pages_are_bad(a, cw.b, work::usable(a, lens.at(a, cw.b)));
    if (wave < 2 && wave * 64 + lane < N)
        dma4(a.parent + (size_t)cw.b * N + wave * 64 + lane,
             __builtin_amdgcn_readfirstlane(lds0 + NS * kStageB + kMaxNodes * 16 + wave * 256));
    {
        const unsigned char* qb = (const unsigned char*)a.q + ((size_t)cw.b * N * a.Hq + cw.kvh * G) * kRowB;
#pragma unroll
        for (int c = 0; c < 32 / kRPI; ++c) dma16(qb + q_off[c], __builtin_amdgcn_readfirstlane(lds0 + q_stage + c * 1024));
    }
    for (int t = 0; t < NS - 2 && t < n_share; ++t) issue_next();
    if (issued == NS - 2) wait_vmcnt<2 * CH * (NS - 2)>(); else wait_vmcnt<0>();

    // ---- this lane's query row.  Q^T fragments: B operand of step t holds d = 16 t + 8 g32 + (0..7) of the row.
    // A later segment's fragments (and parent[]) are loaded before the previous one is written out.
    bf16x8 qf[kKT];
#pragma unroll
    for (int t = 0; t < kKT; ++t) {
        uint4 raw = *(const uint4*)(smem + q_stage + k_off[t]);
        if (!rvalid) raw = make_uint4(0, 0, 0, 0);
        qf[t] = __builtin_bit_cast(bf16x8, raw);
    }
    auto load_q = [&](int b, int kvh) __attribute__((always_inline)) {
        const bf16_t* qrow = (const bf16_t*)a.q + (((size_t)b * N + node) * a.Hq + kvh * G + g) * kD + g32 * 8;
#pragma unroll
        for (int t = 0; t < kKT; ++t) {
            uint4 raw = make_uint4(0, 0, 0, 0);
            if (rvalid) raw = *(const uint4*)(qrow + 16 * t);
            qf[t] = __builtin_bit_cast(bf16x8, raw);
        }
    };
#pragma unroll
    for (int t = 0; t < kKT; ++t) asm volatile("" : "+v"(qf[t]));          // in registers before the barrier
    __syncthreads();                                      // Q and parent[] are here, their stages free
    if constexpr (STEP != kNoStep) lens_read(tail, a, lens);
    while (issued < NS - 1 && issued < n_share) issue_next();

    int parent = -1, b_known = cw.b;
    bool masks = false;                                   // anc[] holds b_known's masks
    while (cw.b >= 0) {
    const int b = cw.b, kvh = cw.kvh;
    const int P = work::usable(a, lens.at(a, b)), u_pref = (P + kBN - 1) / kBN, t_end = uniform(cw.tile_end);
    if (b != b_known) {
        b_known = b;
        masks = false;
        len_bad = P != lens.at(a, b);
        if constexpr (PAGED) len_bad = len_bad || work::pages_are_bad(a, b, P);
        __syncthreads();                                  // the previous sequence's parent[] is no longer read
        if (tid < N) spar[tid] = parent;
        __syncthreads();
    }
    uint32_t amask[4] = {0, 0, 0, 0};
    if (t_end > u_pref) {
        if (!masks) {
            if (!work::tree_is_bad(a, spar)) work::build_masks(a, spar, anc);
            else if (tid < N) *(uint4*)(anc + tid * 4) = make_uint4(0, 0, 0, 0);
            __syncthreads();
            masks = true;
        }
        if (rvalid) {
            const uint4 m = *(const uint4*)(anc + node * 4);
            amask[0] = m.x; amask[1] = m.y; amask[2] = m.z; amask[3] = m.w;
        }
    }

    f32x16 o[kDB];
#pragma unroll
    for (int db = 0; db < kDB; ++db)
#pragma unroll
        for (int j = 0; j < 16; ++j) o[db][j] = 0.f;
    float m_run = -INFINITY, l_run = 0.f;      // l_run: this lane's half of the keys only

    // ---- one tile: scores, (mask,) online softmax, accumulate
    // kTail: keys >= arg masked; kTree: tree tile `arg` of the unit, ancestor mask
    auto tile_body = [&](auto mode_tag, int arg) __attribute__((always_inline)) {
        constexpr int MODE = decltype(mode_tag)::value;
        const lds_u8* stage = (const lds_u8*)smem + ((uint32_t)done % NS) * kStageB;     // LDS address space throughout

        // S^T = K Q^T for the two 32-key blocks.  The two accumulator chains are interleaved (a
        // dependent MFMA cannot start before its predecessor retires); the K fragments of the
        // second half of the head dimension are requested while the first half is multiplied.
        f32x16 s[2];
        {
            bf16x8 kf[2][4];
#pragma unroll
            for (int tt = 0; tt < 4; ++tt) {
                kf[0][tt] = *(const lds_bf16x8*)(stage + k_off[tt]);
                kf[1][tt] = *(const lds_bf16x8*)(stage + 32 * kRowB + k_off[tt]);
            }
#pragma unroll
            for (int j = 0; j < 16; ++j) { s[0][j] = 0.f; s[1][j] = 0.f; }
            if constexpr (kKT == 8) {
#pragma unroll
                for (int tt = 0; tt < 4; ++tt) {
                    s[0] = mma32<F16>(kf[0][tt], qf[tt], s[0]);
                    kf[0][tt] = *(const lds_bf16x8*)(stage + k_off[tt + 4]);
                    s[1] = mma32<F16>(kf[1][tt], qf[tt], s[1]);
                    kf[1][tt] = *(const lds_bf16x8*)(stage + 32 * kRowB + k_off[tt + 4]);
                }
            }
#pragma unroll
            for (int tt = 0; tt < 4; ++tt) {
                s[0] = mma32<F16>(kf[0][tt], qf[tt + kKT - 4], s[0]);
                s[1] = mma32<F16>(kf[1][tt], qf[tt + kKT - 4], s[1]);
            }
            __builtin_amdgcn_sched_group_barrier(0x100, 8, 0);      // 8 LDS reads
            if constexpr (kKT == 8) {
#pragma unroll
                for (int tt = 0; tt < 8; ++tt) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // 1 MFMA
                    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);  // 1 LDS read
                }
            }
            __builtin_amdgcn_sched_group_barrier(0x008, 8, 0);      // 8 MFMAs
        }

        // key of register j of block kblk, relative to the tile: 32 kblk + 8 (j/4) + 4 g32 + (j%4)
        if constexpr (MODE == kTree) {
            const int w0 = arg * 2;                     // 32-node word of block 0
#pragma unroll
            for (int kblk = 0; kblk < 2; ++kblk) {
                const int w = w0 + kblk;
                const uint32_t word = (w == 0 ? amask[0] : w == 1 ? amask[1] : w == 2 ? amask[2] : amask[3]) >> (4 * g32);
#pragma unroll
                for (int j = 0; j < 16; ++j)
                    if (!((word >> ((j >> 2) * 8 + (j & 3))) & 1u)) s[kblk][j] = -INFINITY;
            }
        } else if constexpr (MODE == kTail) {
#pragma unroll
            for (int kblk = 0; kblk < 2; ++kblk)
#pragma unroll
                for (int j = 0; j < 16; ++j)
                    if (kblk * 32 + (j >> 2) * 8 + 4 * g32 + (j & 3) >= arg) s[kblk][j] = -INFINITY;
        }

        // online softmax for this lane's row (log2 units)
        float mx = fmaxf(s[0][0], s[1][0]);
#pragma unroll
        for (int j = 1; j < 16; ++j) mx = __builtin_fmaxf(__builtin_fmaxf(mx, s[0][j]), s[1][j]);    // v_max3_f32
        mx = max_across_halves(mx);
        float psum = 0.f;
        if constexpr (MODE == kPlain) {
            // Full prefix tiles move the row's reference maximum only when some row of the wave
            // outgrew it by more than 2^kLazyLog2: until then the exponentials are taken against the
            // stale reference (they stay below 2^kLazyLog2, exact in fp32 and in bf16's range), and the
            // 64 multiplications of the output accumulator are skipped.  Sum and accumulator stay
            // consistent with whatever reference is current, which is all the final division (or the
            // merge of KV splits) needs.
            const float mt = mx * a.scale_log2;
            if (__any(mt > m_run + kLazyLog2)) {
                const float m_new = fmaxf(m_run, mt);
                const float alpha = fast_exp2(m_run - m_new);          // first tile: exp2(-inf) = 0
                l_run *= alpha;
#pragma unroll
                for (int db = 0; db < kDB; ++db)
#pragma unroll
                    for (int j = 0; j < 16; ++j) o[db][j] *= alpha;
                m_run = m_new;
            }
#pragma unroll
            for (int kblk = 0; kblk < 2; ++kblk)
#pragma unroll
                for (int j = 0; j < 16; ++j) {
                    const float p = fast_exp2(fmaf(s[kblk][j], a.scale_log2, kShift - m_run));
                    s[kblk][j] = p;
                    psum += p;
                }
            l_run += psum;
        } else {
            const float m_new = fmaxf(m_run, mx * a.scale_log2);
            float m_safe = m_new;
            if constexpr (MODE == kTree) m_safe = (m_new == -INFINITY) ? 0.f : m_new;   // row with no visible key yet
            const float alpha = fast_exp2(m_run - m_safe);
#pragma unroll
            for (int kblk = 0; kblk < 2; ++kblk)
#pragma unroll
                for (int j = 0; j < 16; ++j) {
                    const float p = fast_exp2(fmaf(s[kblk][j], a.scale_log2, kShift - m_safe));
                    s[kblk][j] = p;
                    psum += p;
                }
            l_run = l_run * alpha + psum;
            if (__any(m_new > m_run)) {
#pragma unroll
                for (int db = 0; db < kDB; ++db)
#pragma unroll
                    for (int j = 0; j < 16; ++j) o[db][j] *= alpha;
            }
            m_run = m_new;
        }

        // O^T += V^T P^T in four steps of 16 keys; the V^T fragments of step i+1 are requested
        // before the MFMAs of step i.
        {
            bf16x8 pb[kParts][4];
#pragma unroll
            for (int part = 0; part < kParts; ++part)
#pragma unroll
                for (int st = 0; st < 4; ++st)
                    pb[part][st] = part + 1 < kParts ? take8<F16>(s[st >> 1], 8 * (st & 1)) : round8<F16>(s[st >> 1], 8 * (st & 1));
            auto vfrag = [&](const lds_u8* p) __attribute__((always_inline)) {     // 8 keys x 1 column of V^T: two transposing reads
                const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)p);
                const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p + 8 * kRowB));
                return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
            };
            bf16x8 vf[2][kDB];
#pragma unroll
            for (int db = 0; db < kDB; ++db) vf[0][db] = vfrag(stage + v_off[db]);
#pragma unroll
            for (int st = 0; st < 4; ++st) {
                if (st < 3) {
#pragma unroll
                    for (int db = 0; db < kDB; ++db) vf[(st + 1) & 1][db] = vfrag(stage + (st + 1) * 16 * kRowB + v_off[db]);
                }
#pragma unroll
                for (int part = 0; part < kParts; ++part)
#pragma unroll
                    for (int db = 0; db < kDB; ++db)
                        o[db] = mma32<F16>(vf[st & 1][db], pb[part][st], o[db]);
            }
            // A fragment's reads, one ahead of the product that takes it: left to itself the compiler reads as many as it has registers for, and
            // the products wait for the LDS in bursts (16 x 64/8 heads, 32768 keys + 128 nodes 1997 us, 1980 so).
            if constexpr (kParts == 1 && kDB == 4) {
                __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);      // LDS reads
#pragma unroll
                for (int i = 1; i < 4 * kDB; ++i) {
                    __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // MFMA
                }
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            }
        }
    };

    // The compiler does not see the direct-to-LDS loads; settle the Q fragments here, so that it places no
    // vmcnt wait of its own inside the tile loop.
#pragma unroll
    for (int t = 0; t < kKT; ++t) asm volatile("" : "+v"(qf[t]));

    auto sync = [&]() __attribute__((always_inline)) {
        // tile `done` has landed once at most NS-2 younger tiles of this wave are outstanding
        if (done + NS - 2 < n_share) wait_vmcnt<2 * CH * (NS - 2)>(); else wait_vmcnt<0>();
        __syncthreads();          // every wave's part of the tile is in LDS; the stage before it is free
        if (issued < n_share) issue_next();
    };
    int t = uniform(cw.tile);
    // While the loads run ahead inside this segment's full prefix tiles, nothing has to be decided per tile.
    if (uniform(pw.b) == uniform(b) && uniform(pw.kvh) == uniform(kvh)) {
        const int n = uniform(p_full);
        for (int i = 0; i < n; ++i, ++done) {
            wait_vmcnt<2 * CH * (NS - 2)>();
            __syncthreads();
            issue_full();
            ++issued;
            if (wave_on) tile_body(std::integral_constant<int, kPlain>{}, 0);
        }
        t += n;
        pw.tile += n;
        p_full = 0;
        end_tile();
    }
    for (const int e = min(P / kBN, t_end); t < e; ++t, ++done) {
        sync();
        if (wave_on) tile_body(std::integral_constant<int, kPlain>{}, 0);
    }
    for (const int e = min(u_pref, t_end); t < e; ++t, ++done) {
        sync();
        if (wave_on) tile_body(std::integral_constant<int, kTail>{}, P - t * kBN);
    }
    for (; t < t_end; ++t, ++done) {
        sync();
        if (wave_on) tile_body(std::integral_constant<int, kTree>{}, t - u_pref);
    }

    work::Walk nw = cw;
    if constexpr (!kOne) {
        nw = work::walk_next(a, lens, cw);
        if (nw.b >= 0) {
            if (nw.b != b && tid < N) parent = a.parent[(size_t)nw.b * N + tid];
            load_q(nw.b, nw.kvh);
        }
        if (mt == 0 && tid == 0) work::note_parts(a, team, cw);
    }
    // ---- write this lane's row: d = 32 db + 8 (j/4) + 4 g32 + (j%4)
    const int flagged = (work::tree_is_bad(a, spar) ? S4C_SEQ_BAD_TREE : 0) | (len_bad ? S4C_SEQ_BAD_LEN : 0);
    if (a.status && tid == 0 && cw.tile == 0 && kvh == 0 && mt == 0) a.status[b] = flagged;
    float l_tot = l_run + __shfl_xor(l_run, 32);
    if (flagged) {                             // zero output, whatever was read in place of a bad page
        l_tot = 0.f;
#pragma unroll
        for (int db = 0; db < kDB; ++db)
#pragma unroll
            for (int j = 0; j < 16; ++j) o[db][j] = 0.f;
    }
    const uint64_t left = lens_look_back<STEP>();
    if constexpr (MERGE == parts::kHere || MERGE == parts::kNext) {
        parts::finish<kD, kElem, MERGE, WR, WR>(Arguments().attn(), team, mt, smem, [&]() __attribute__((always_inline)) {
            parts::put<kD, 1, MERGE, true>(Arguments().attn(), team, mt * WR + wave, 0, m_run, l_tot, [&](int q) __attribute__((always_inline)) {
                return f32x4{o[q >> 2][4 * (q & 3)], o[q >> 2][4 * (q & 3) + 1], o[q >> 2][4 * (q & 3) + 2], o[q >> 2][4 * (q & 3) + 3]};
            });
        });
        lens_end<STEP>(left);
        return;
    }
    if (MERGE == parts::kWhole || work::walk_is_whole(a, cw)) {
        if (rvalid) {
        const float inv = (l_tot > 0.f) ? 1.f / l_tot : 0.f;
        bf16_t* orow = (bf16_t*)a.out + (((size_t)b * N + node) * a.Hq + kvh * G + g) * kD + 4 * g32;
#pragma unroll
        for (int db = 0; db < kDB; ++db)
#pragma unroll
            for (int jq = 0; jq < 4; ++jq) {
                uint2 pk;
                pk.x = round1<F16>(o[db][4 * jq + 0] * inv) | (round1<F16>(o[db][4 * jq + 1] * inv) << 16);
                pk.y = round1<F16>(o[db][4 * jq + 2] * inv) | (round1<F16>(o[db][4 * jq + 3] * inv) << 16);
                *(uint2*)(orow + 32 * db + 8 * jq) = pk;
            }
        }
    } else {
        if (rvalid) {
            const size_t prow = work::part_row(a, team, work::part_slot(cw)) + rq;
            float* orow = Arguments().attn().ws_o + prow * kD + 4 * g32;       // (not kept in scratch while tiles are multiplied)
#pragma unroll
            for (int db = 0; db < kDB; ++db)
#pragma unroll
                for (int jq = 0; jq < 4; ++jq)
                    *(float4*)(orow + 32 * db + 8 * jq) =
                        make_float4(o[db][4 * jq], o[db][4 * jq + 1], o[db][4 * jq + 2], o[db][4 * jq + 3]);
            if (g32 == 0) {
                a.ws_ml[prow * 2] = m_run;
                a.ws_ml[prow * 2 + 1] = l_tot;
            }
        }
    }
    lens_end<STEP>(left);
    if constexpr (kOne) return;
    cw = nw;
    }
}

int pick_wr(int M) { return M <= 128 ? 4 : 8; }

template <int WR, int NS, int WPE, bool PAGED, bool F16, int D, StepKind STEP, parts::Merge MERGE>
hipError_t launch(AttnArgs a, StepTail<STEP> tail, hipStream_t st) {
    constexpr int kLds = lds_bytes_for(NS, D);
    static std::atomic<uint64_t> lds_set{0};
    const hipError_t ea = ensure_dynamic_lds((const void*)tree_attn_mfma_kernel<WR, NS, WPE, PAGED, F16, D, STEP, MERGE>, kLds, lds_set);
    if (ea != hipSuccess) return ea;
    a.attn_wgs = attn_workgroups(a);
    const dim3 grid = launch_grid(a, rest_of(a, tail)), block(WR * 64);
    hipLaunchKernelGGL((tree_attn_mfma_kernel<WR, NS, WPE, PAGED, F16, D, STEP, MERGE>), grid, block, kLds, st, a, tail);
    return hipGetLastError();
}

// four waves (up to 128 rows): one workgroup per CU and wave per SIMD, or two of head size 64 (attn_tile_large), which 256 registers a thread allow (with 262
// there was one: 24 parts of 76 rows, 21000 keys 67.5 us and 53.0; 12 parts of 71 rows, 12000 keys 55.5 and 42.9); eight: two waves per SIMD
template <bool PAGED, bool F16, int D, StepKind STEP, parts::Merge MERGE>
hipError_t launch_rows(const AttnArgs& a, const StepTail<STEP>& tail, hipStream_t st) {
    return pick_wr(a.M) == 4 ? launch<4, 4, D == 64 ? 2 : 1, PAGED, F16, D, STEP, MERGE>(a, tail, st) : launch<8, 4, 2, PAGED, F16, D, STEP, MERGE>(a, tail, st);
}
template <bool PAGED, bool F16, int D, StepKind STEP>
hipError_t launch_rows(const AttnArgs& a, const StepTail<STEP>& tail, hipStream_t st) {
    if (a.split == 1) return launch_rows<PAGED, F16, D, STEP, parts::kWhole>(a, tail, st);
    if constexpr (STEP == kNoStep)
        if (a.split == 0) return launch_rows<PAGED, F16, D, STEP, parts::kShares>(a, tail, st);
    if constexpr (!PAGED && STEP == kNoStep)
        if (a.tag == 0) return launch_rows<PAGED, F16, D, STEP, parts::kNext>(a, tail, st);
    return launch_rows<PAGED, F16, D, STEP, parts::kHere>(a, tail, st);
}
template <bool F16, int D>
hipError_t launch_as(const AttnArgs& a, const StepTail<kGreedyStep>* step, hipStream_t st) {
    if (step)
        return step->accept.mode == S4C_GREEDY ? launch_rows<false, F16, D>(a, StepTail<kGreedyStep>(*step), st)
                                               : launch_rows<false, F16, D>(a, StepTail<kStochasticStep>(*step), st);
    return a.block_table ? launch_rows<true, F16, D>(a, StepTail<kNoStep>(), st) : launch_rows<false, F16, D>(a, StepTail<kNoStep>(), st);
}
template <bool F16>
hipError_t launch_by_shape(const AttnArgs& a, const StepTail<kGreedyStep>* step, hipStream_t st) {
    return a.D == 64 ? launch_as<F16, 64>(a, step, st) : launch_as<F16, 128>(a, step, st);
}

}  // namespace

}  // namespace s4c

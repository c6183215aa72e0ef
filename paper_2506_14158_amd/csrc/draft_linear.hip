// Input projection of a draft head (paper Eq. 3: h = Linear(concat[e, f])) on the CDNA4 matrix
// cores: out[t][o] = bias[o] + sum_k e[t][k] W[o][k] + sum_k f[t][k] W[o][H + k], bf16 in and
// out (fp16 likewise), fp32 accumulate.  The concatenation is never materialised: the K loop walks the first H
// columns of W against e and the last H against f.
//
//   * Both operands have the reduction index contiguous in memory (W is [Hout][2H], e and f are
//     [T][H]), which is what the matrix-core instruction wants for A and for B: a lane's 8 values
//     are 16 consecutive bytes of one row.  The product is formed transposed, D = W x^T (A = W
//     rows, B = token rows), so a lane ends up with 4 consecutive output features of one token
//     and stores them as one 8-byte word.
//   * v_mfma_f32_16x16x32_bf16 rather than the 32x32x16 shape: with random operands the chip is
//     power-limited and the smaller shape sustains a higher clock (measured 7 % faster here); the
//     wave tile keeps the LDS bytes per FLOP the same.
//   * Workgroup tile 256 output features x 256 tokens, stages of 64 reduction elements (a tile row is 128 bytes: whole cache
//     lines; half of that per row, as this kernel had it, cost twice the requests); wave (wo, wt) of 8 owns
//     128 features x 64 tokens = 8 x 4 accumulator blocks of 16 x 16.  W and token tiles stream from HBM / L2 straight into LDS
//     (global_load_lds_dwordx4), into a ring of five 32 KB slots, the whole 160 KB: with two stages of W and one and a half of
//     tokens under way the latency of memory (1.5 us under load, where a stage's products take 1.2) is covered.
//   * A stage is multiplied out of registers, half by half: while one half is multiplied the other's fragments are read, two
//     LDS reads to four products, and behind the stage's one barrier the loads follow one by one between the products too.
//     Issued in one go there (64 of them per CU, 16 cycles each) they held up every wave's products together.
//     2048 tokens, H 8192, us: 477 before; 422 with 128-byte rows and fragments read ahead, 394 with five slots and the
//     loads between the products (1.39 PFLOP/s; the clock falls as the matrix cores are busier).
//     Measured and not kept: a second, earlier request for every line, to have it in the L2 (441); four stages of 32 elements (460).
//   * 16-byte chunk c of row r sits at chunk c ^ (r & 7), applied on the global-address side of the direct-to-LDS load, so the
//     16-byte fragment reads of 8 consecutive rows fall into 8 different bank groups.
//   * The token tiles of one output-feature tile take consecutive slots of one XCD (workgroup id
//     modulo 8), so the W tile they all read is fetched from HBM once and shared through that L2.
//   * Few tiles: the reduction is divided (draft_linear_slices), fp32 partial sums, added in slice order by
//     draft_linear_reduce_kernel.
#include "mfma_common.h"

namespace s4c {

namespace {

using namespace mfma;

constexpr int kBO = 256;                   // output features per workgroup
constexpr int kBT = 256;                   // tokens per workgroup
constexpr int kBK = 64;                    // reduction elements per stage
constexpr int kRow = kBK * 2;              // bytes per tile row
constexpr int kSlot = kBO * kRow;          // bytes of the W (or token) part of a stage: 32 KB
constexpr int kSlots = 5;                  // all of a CU's LDS
constexpr int kWaves = 8;
constexpr int kTB = 2;                     // token blocks (of 32) per wave
constexpr int kCH = kBO / 8 / kWaves;      // direct-to-LDS loads per wave and half-stage

template <bool F16, bool SPLIT>
__global__ __launch_bounds__(kWaves * 64) __attribute__((amdgpu_waves_per_eu(2, 2)))
void draft_linear_kernel(LinearArgs a) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_u8*)smem;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    const int team = a.ttiles;
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    const int unit = (slot / team) * 8 + xcd;              // (slice of the reduction, output-feature tile)
    if (unit >= a.otiles * (SPLIT ? a.nslices : 1)) return;
    const int slice = SPLIT ? unit / a.otiles : 0;
    const int o0 = (unit - slice * a.otiles) * kBO, t0 = (slot % team) * kBT;
    const int H = a.H, T = a.T;
    const size_t wrow = (size_t)2 * H * 2;                 // bytes per W row
    const size_t xrow = (size_t)H * 2;                     // bytes per e / f row

    // ---- direct-to-LDS loads: instruction ii of a half-stage covers rows 8 ii .. 8 ii + 7,
    // lane -> (row 8 ii + lane / 8, physical chunk lane % 8); a wave issues ii = wave, wave + 8, ...
    const int lc = (lane & 7) ^ (lane >> 3);               // the logical chunk: physical ^ (row & 7)
    uint32_t wo_off[kCH], xo_off[kCH];
#pragma unroll
    for (int c = 0; c < kCH; ++c) {
        const int row = 8 * (wave + kWaves * c) + (lane >> 3);
        wo_off[c] = (uint32_t)((size_t)row * wrow) + lc * 16;
        xo_off[c] = (uint32_t)((size_t)min(t0 + row, T - 1) * xrow);              // rows past T: clamped, never stored
    }
    const unsigned char* wbase = (const unsigned char*)a.W + (size_t)o0 * wrow;
    const int nk_all = 2 * H / kBK;                        // stages (H is a multiple of 32)
    const int kb = SPLIT ? slice * a.kslice : 0, ke = SPLIT ? min(nk_all, kb + a.kslice) : nk_all;      // this workgroup's
    // One of the 2 kCH loads of a wave (the last stages are asked for again at the end, so that every step has as many loads).
    auto load_w = [&](int kt, uint32_t slot, int c) __attribute__((always_inline)) {
        dma16(uniform(wbase + (size_t)min(kt, ke - 1) * kRow), wo_off[c], __builtin_amdgcn_readfirstlane(lds0 + slot + (wave + kWaves * c) * 1024));
    };
    // (by lane, because H may be an odd multiple of 32: then one stage ends in e and begins in f)
    auto x_from = [&](int kt) __attribute__((always_inline)) {
        const int k = min(kt, ke - 1) * kBK + lc * 8;
        return k < H ? (const unsigned char*)a.e + (size_t)k * 2 : (const unsigned char*)a.f + (size_t)(k - H) * 2;
    };
    auto load_x = [&](const unsigned char* from, uint32_t slot, int c) __attribute__((always_inline)) {
        dma16(from + xo_off[c], __builtin_amdgcn_readfirstlane(lds0 + slot + (wave + kWaves * c) * 1024));
    };

    // ---- fragment addresses inside a stage (v_mfma_f32_16x16x32_bf16: a lane supplies row lane % 16,
    // reduction elements 8 (lane / 16) .. + 7, i.e. chunk lane / 16 of the row's first or second half); the swizzle is the
    // same for every block of 16 rows, so the blocks lie at constant distances
    const int wo = wave / (8 / kTB), wt = wave % (8 / kTB), g16 = lane >> 4, l16 = lane & 15;
    uint32_t w_off[2], x_off[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const uint32_t chunk = (uint32_t)((4 * h + g16) ^ (l16 & 7)) << 4;
        w_off[h] = (uint32_t)(wo * 128 + l16) * kRow + chunk;
        x_off[h] = (uint32_t)(wt * (32 * kTB) + l16) * kRow + chunk;
    }

    f32x4 acc[8][2 * kTB];
#pragma unroll
    for (int ob = 0; ob < 8; ++ob)
#pragma unroll
        for (int tb = 0; tb < 2 * kTB; ++tb)
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[ob][tb][j] = 0.f;

    struct Frags { bf16x8 w[8], x[2 * kTB]; };
    // read i of the 12 that fill f from the half h of a stage
    auto read = [&](Frags& f, int h, uint32_t ws, uint32_t xs, int i) __attribute__((always_inline)) {
        if (i < 2 * kTB) f.x[i] = *(const lds_bf16x8*)((const lds_u8*)smem + (xs + x_off[h]) + i * (16 * kRow));
        else f.w[i - 2 * kTB] = *(const lds_bf16x8*)((const lds_u8*)smem + (ws + w_off[h]) + (i - 2 * kTB) * (16 * kRow));
    };
    auto multiply = [&](const Frags& f, int ob) __attribute__((always_inline)) {
#pragma unroll
        for (int tb = 0; tb < 2 * kTB; ++tb) acc[ob][tb] = mma16<F16>(f.w[ob], f.x[tb], acc[ob][tb]);
    };
    // Ring of five slots; stage kt's W part is the 2 kt'th to enter it, its token part the 2 kt + 1'st.  W, which comes from
    // memory, is requested two stages ahead, the tokens, which every workgroup reads, one and a half.
    auto next = [](uint32_t slot) { return slot + 2 * kSlot < kSlots * kSlot ? slot + 2 * kSlot : slot + 2 * kSlot - kSlots * kSlot; };
    uint32_t ws = 0, xs = kSlot;                           // stage kt's slots
    Frags fa, fb;
#pragma unroll
    for (int c = 0; c < kCH; ++c) load_w(kb, ws, c);
#pragma unroll
    for (int c = 0; c < kCH; ++c) load_x(x_from(kb), xs, c);
#pragma unroll
    for (int c = 0; c < kCH; ++c) load_w(kb + 1, next(ws), c);
#pragma unroll
    for (int c = 0; c < kCH; ++c) load_x(x_from(kb + 1), next(xs), c);
#pragma unroll
    for (int c = 0; c < kCH; ++c) load_w(kb + 2, next(next(ws)), c);
    wait_vmcnt<3 * kCH>();
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 12; ++i) read(fa, 0, ws, xs, i);
    for (int kt = kb; kt < ke; ++kt) {
        // Products of the stage's first half, reads of its second.  (The barriers between the groups keep the compiler from
        // gathering the reads, and below the loads, in front of the products, where all waves would wait for each other's.)
#pragma unroll
        for (int g = 0; g < 8; ++g) {
            if (g < 6) { read(fb, 1, ws, xs, 2 * g); read(fb, 1, ws, xs, 2 * g + 1); }
            multiply(fa, g);
            __builtin_amdgcn_sched_barrier(0);
        }
        wait_vmcnt<kCH>();                                 // this wave's parts of stage kt + 1 have landed (W of kt + 2 is on its way)
        __syncthreads();                                   // everybody's have; stage kt is in registers and no longer read
        const uint32_t w1 = next(ws), x1 = next(xs), x2 = next(x1), w3 = next(next(w1));
        const unsigned char* from = x_from(kt + 2);
#pragma unroll
        for (int g = 0; g < 8; ++g) {
            if (g < kCH) load_x(from, x2, g); else load_w(kt + 3, w3, g - kCH);
            if (g < 6) { read(fa, 0, w1, x1, 2 * g); read(fa, 0, w1, x1, 2 * g + 1); }
            multiply(fb, g);
            __builtin_amdgcn_sched_barrier(0);
        }
        ws = w1;
        xs = x1;
    }
    wait_vmcnt<0>();                                       // (the loads asked for again)

    // ---- epilogue: per block a lane holds features 4 (lane / 16) .. + 3 of token lane % 16
    if constexpr (SPLIT) {
        float* part = a.ws + (size_t)slice * T * a.Hout + o0 + wo * 128 + 4 * g16;
#pragma unroll
        for (int tb = 0; tb < 2 * kTB; ++tb) {
            const int tok = t0 + wt * (32 * kTB) + tb * 16 + l16;
            if (tok >= T) continue;
#pragma unroll
            for (int ob = 0; ob < 8; ++ob) *(f32x4*)(part + (size_t)tok * a.Hout + ob * 16) = acc[ob][tb];
        }
        return;
    }
    const uint16_t* bias = (const uint16_t*)a.bias;
    auto elem = [](uint16_t bits) { return F16 ? (float)__builtin_bit_cast(_Float16, bits) : bf16_to_f32(bits); };
#pragma unroll
    for (int tb = 0; tb < 2 * kTB; ++tb) {
        const int tok = t0 + wt * (32 * kTB) + tb * 16 + l16;
        if (tok >= T) continue;
        uint16_t* orow = (uint16_t*)a.out + (size_t)tok * a.Hout + o0 + wo * 128 + 4 * g16;
#pragma unroll
        for (int ob = 0; ob < 8; ++ob) {
            float v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = acc[ob][tb][u];
            if (bias) {
                const uint16_t* bp = bias + o0 + wo * 128 + ob * 16 + 4 * g16;
#pragma unroll
                for (int u = 0; u < 4; ++u) v[u] += elem(bp[u]);
            }
            uint2 pk;
            pk.x = round1<F16>(v[0]) | (round1<F16>(v[1]) << 16);
            pk.y = round1<F16>(v[2]) | (round1<F16>(v[3]) << 16);
            *(uint2*)(orow + ob * 16) = pk;
        }
    }
}

}  // namespace

int draft_linear_tile_out() { return kBO; }
int draft_linear_tile_k() { return 32; }          // reduction elements that H is a multiple of

// Slices of the reduction, at most `most`: few output tiles leave CUs idle, so each tile's reduction goes to several workgroups,
// whose partial sums are written, read and added by a second launch.  What that costs and saves, us: a stage 1.3, the
// launch 3, a byte of the partial sums' way there and back at 3.5 TB/s; never more workgroups than CUs.
// Chosen and measured: 512 tokens, H 8192 4 slices, 140; 600, 8192 2 slices, 198 (one: 320); 1024, 8192 2 slices, 233 (337); 2048, 4096 2 slices, 128 (176);
// 150, 4096 11 slices, 34.0 (8: 35.4, 16: 36.5); 150, 1024 8 slices, 17.8 (4: 19.8).
int draft_linear_slices(int T, int H, int Hout, int cus, size_t most, int* kslice) {
    const int nk = 2 * H / kBK;
    const long long tiles = (long long)(Hout / kBO) * ((T + kBT - 1) / kBT);
    int best = 1;
    double best_us = 1.3 * nk;
    for (int n = 2; n <= nk && n * tiles <= cus && (size_t)n <= most; ++n) {
        const double us = 1.3 * ((nk + n - 1) / n) + 3.0 + (double)n * T * Hout * 8.0 / 3.5e6;
        if (us < best_us) { best_us = us; best = n; }
    }
    *kslice = (nk + best - 1) / best;
    return (nk + *kslice - 1) / *kslice;
}

template <bool F16, bool SPLIT>
static hipError_t launch_linear(const LinearArgs& a, hipStream_t st) {
    constexpr int kLds = kSlots * kSlot;
    static std::atomic<uint64_t> lds_set{0};
    const hipError_t ea = ensure_dynamic_lds((const void*)draft_linear_kernel<F16, SPLIT>, kLds, lds_set);
    if (ea != hipSuccess) return ea;
    LinearArgs k = a;
    k.ttiles = (a.T + kBT - 1) / kBT;
    k.otiles = a.Hout / kBO;
    const long units8 = ((long)k.otiles * (SPLIT ? a.nslices : 1) + 7) / 8 * 8;      // padded to whole XCD rounds
    hipLaunchKernelGGL((draft_linear_kernel<F16, SPLIT>), dim3((unsigned)(units8 * k.ttiles)), dim3(kWaves * 64), kLds, st, k);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess && SPLIT ? launch_draft_linear_reduce(a, st) : e;
}

hipError_t launch_draft_linear(const LinearArgs& a, hipStream_t st) {
    if (a.nslices > 1) return a.dtype == S4C_F16 ? launch_linear<true, true>(a, st) : launch_linear<false, true>(a, st);
    return a.dtype == S4C_F16 ? launch_linear<true, false>(a, st) : launch_linear<false, false>(a, st);
}

}  // namespace s4c

// Sibling-sequential acceptance with the correction token (paper Sec. 2, speculative-sampling
// paragraph: accept with probability min(1, p/q), redraw a rejected token from
// norm(max(0, p - q)); Sec. 3.2, second equation: the correction at a fork of the tree).
//
// The walk from the root is a chain of data-dependent decisions, each needing a reduction over the vocabulary.  What
// one node decides (which child is accepted; if none, the correction token) depends on its own two rows only, so:
//   rows    (few and short rows, see resample_by_rows) every node of every sequence is decided at the same time, a
//           workgroup each, whether the walk will come by or not, and a workgroup per sequence behind them follows the
//           decisions from the root.  A chain of a handful of reductions inside one CU instead of one of all levels'
//           across several.
//   teams   (the rest) a team of G workgroups walks one sequence, each with a slice of the vocabulary; the G partial
//           results are exchanged through a per-pass slot array in device memory (struct Team).  All G workgroups then add
//           the partials in slot order, obtain bit-identical sums and so take the same branches without any other
//           communication.  Workgroup 0 of the team is the only one that writes the sequence's outputs (the owner of
//           the correction token hands it over through one more slot), so what the caller sees is either a complete
//           result or, if workgroup 0 itself gave up anywhere, the flagged empty one -- never a mixture.
// Every poll is bounded: a workgroup that cannot complete an exchange exits.
//
// A node's rows are read once and stay in registers (8 tokens x NG blocks a thread: the weights as fp64 and, up to four blocks, the
// draft probabilities as fp32), so a rejected child costs arithmetic and a reduction, no memory:
//   a_0[v] = exp((l[v] - max l) / T)              S_0 = sum_v a_0[v]        (target row)
//   a_{j+1}[v] = max(0, a_j[v] - S_j q[v])        S_{j+1} = sum_v a_{j+1}[v] (after j+1 rejections)
// so that a_j / S_j is the j-times-corrected distribution.  A child with token x passes iff
// u q[x] < a_j[x] / S_j.  The correction token is the inverse CDF of a_j in token-id order.
// The arithmetic is fp64: the decisions compare sums of 10^5 terms against a uniform number,
// and the work is a few rows per sequence, so accuracy is worth more than VALU rate here.
//
// Vocabulary order: blocks of 512 tokens; workgroup g owns blocks [g*bpg, (g+1)*bpg), wave w of it the blocks
// [w*ipw, (w+1)*ipw) of those; in a block lane l owns the 8 tokens 8l..8l+7 (one 16-byte load of 16-bit logits,
// two of fp32).
#include "common.h"
#include "resample_plan.h"

namespace s4c {

namespace {

constexpr int kWaves = kResampleWaves;
constexpr int kThreads = 64 * kWaves;
constexpr int kBlock = kResampleBlock;
constexpr int kMaxRow = kResampleMaxRow;
constexpr int kMaxVocab = 1 << 21;
constexpr int kMaxTeam = kMaxVocab / kResampleMaxSlice;
constexpr int kSpinLimit = 1 << 20;    // default number of polls (each followed by a short sleep) before giving up

// lane's value of x from another lane of the row of 16 or from the row below, through the data-parallel-primitive path of the
// vector ALUs (a shuffle through LDS is several times the latency, and a walk is a chain of these); 0 where there is none
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp(double x) {
    const uint64_t u = (uint64_t)__double_as_longlong(x);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, ROWS, 0xF, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, ROWS, 0xF, false);
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}
__device__ __forceinline__ double of_lane(double x, int lane) {            // (lane wave-uniform)
    const uint64_t u = (uint64_t)__double_as_longlong(x);
    const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)u, lane), hi = __builtin_amdgcn_readlane((uint32_t)(u >> 32), lane);
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}
__device__ __forceinline__ float uniform_f32(float x) { return __uint_as_float((uint32_t)__builtin_amdgcn_readfirstlane((int)__float_as_uint(x))); }
// inclusive sums over the wave's lanes
__device__ __forceinline__ double wave_incl_scan(double x) {
    x += dpp<0x111, 0xF>(x);          // row_shr:1, 2, 4, 8: sums inside each row of 16
    x += dpp<0x112, 0xF>(x);
    x += dpp<0x114, 0xF>(x);
    x += dpp<0x118, 0xF>(x);
    x += dpp<0x142, 0xA>(x);          // row_bcast:15 into rows 1 and 3
    x += dpp<0x143, 0xC>(x);          // row_bcast:31 into rows 2 and 3
    return x;
}
__device__ __forceinline__ double wave_sum(double x) { return of_lane(wave_incl_scan(x), 63); }      // in every lane
template <int CTRL, int ROWS>
__device__ __forceinline__ float dpp_max(float x) {                         // (lanes without a source see their own value)
    const int i = (int)__float_as_uint(x);
    return fmaxf(x, __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(i, i, CTRL, ROWS, 0xF, false)));
}
__device__ __forceinline__ float wave_max(float x) {                        // in every lane
    x = dpp_max<0x118, 0xF>(dpp_max<0x114, 0xF>(dpp_max<0x112, 0xF>(dpp_max<0x111, 0xF>(x))));
    x = dpp_max<0x143, 0xC>(dpp_max<0x142, 0xA>(x));
    return __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(x), 63));
}

__device__ __forceinline__ double bits_to_f64(uint64_t u) { return __longlong_as_double((long long)u); }
__device__ __forceinline__ uint64_t f64_to_bits(double x) { return (uint64_t)__double_as_longlong(x); }

// One block after the other: interleaved, the blocks' temporaries would not fit the registers beside the weights.
__device__ __forceinline__ void keep_order() { __builtin_amdgcn_sched_barrier(0); }

struct Row {
    const void* lg;       // logits row
    const float* q;       // draft row
    int V;
    bool vec;             // 16-byte loads allowed for both rows
};

// the 8 logits (as float) of tokens base..base+7; tokens >= V read as -inf
template <typename T>
__device__ __forceinline__ void load_logits8(const Row& r, int base, float (&x)[8]) {
    const T* p = (const T*)r.lg;
    if (r.vec && base + 8 <= r.V) {
        if constexpr (sizeof(T) == 2) {
            const uint4 raw = *(const uint4*)(p + base);
            const uint32_t w[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
            for (int k = 0; k < 4; ++k) unpack2<T>(w[k], x[2 * k], x[2 * k + 1]);
        } else {
            const float4 a = *(const float4*)(p + base), b = *(const float4*)(p + base + 4);
            x[0] = a.x; x[1] = a.y; x[2] = a.z; x[3] = a.w; x[4] = b.x; x[5] = b.y; x[6] = b.z; x[7] = b.w;
        }
    } else {
#pragma unroll
        for (int k = 0; k < 8; ++k) x[k] = (base + k < r.V) ? to_f32<T>(p[base + k]) : -INFINITY;
    }
}

__device__ __forceinline__ void load_draft8(const Row& r, int base, float (&qv)[8]) {
    if (r.vec && base + 8 <= r.V) {
        const float4 a = *(const float4*)(r.q + base), b = *(const float4*)(r.q + base + 4);
        qv[0] = a.x; qv[1] = a.y; qv[2] = a.z; qv[3] = a.w; qv[4] = b.x; qv[5] = b.y; qv[6] = b.z; qv[7] = b.w;
    } else {
#pragma unroll
        for (int k = 0; k < 8; ++k) qv[k] = (base + k < r.V) ? r.q[base + k] : 0.f;
    }
}

// What the threads of a workgroup share.
struct Shared {
    int32_t par[kMaxNodes], tok[kMaxNodes], child[kMaxNodes];      // the tree; the current node's children
    int32_t count[2], fail, token;
    double ax[kMaxNodes], lhs[kMaxNodes];                          // per node: weight and u q of its token in its parent's rows
    double red[2][kWaves];
    float redf[kWaves];
    uint32_t got[4 * kMaxTeam];                                    // the team's words of an exchange: [4][G]
};

// A team's exchanges (a workgroup that works alone, G = 1, makes none).  Workgroup g's words of an exchange are 8-byte
// records (tag << 32) | 32 bits of payload, written with device-coherent stores by thread 0 and polled by all workgroups
// of the team.  Nothing has to be cleared before a call: a record without the tag is not there yet.  In the first exchange
// the tag is the call's nonce, and workgroup 0 adds the time; of nonce and time the tag of the later ones is made, so that a
// captured graph, which replays the call nonce and all, does not take the previous replay's records for its own.
// The first exchange's records are overwritten behind the second one, when everybody has read them.  (Clearing the
// slots in a launch of its own, as this did before, cost 3 to 5 us a call.)
struct Team {
    uint64_t* slots;      // of the sequence: [max_pass][4][G]
    int g, G, max_pass, spin_limit, pass;
    uint32_t nonce, tag;

    static __device__ __forceinline__ void put(uint64_t* p, uint32_t tag, uint32_t bits) {
        __hip_atomic_store(p, ((uint64_t)tag << 32) | bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    // the payload of a record; false if it never came
    __device__ __forceinline__ bool get(const uint64_t* p, uint32_t* bits) const {
        for (int spin = 0; spin < spin_limit; ++spin) {
            const uint64_t v = __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            *bits = (uint32_t)v;
            if ((uint32_t)(v >> 32) == tag) return true;
            __builtin_amdgcn_s_sleep(1);
        }
        return false;
    }
    // Everybody's a; with a maximum, everybody's b too (got[2]).
    template <bool MAX>
    __device__ __forceinline__ bool exchange(Shared& sh, double a, float b = 0.f) {
        if (pass >= max_pass) return false;                // (more than a valid tree can need)
        const bool first = pass == 0;                      // (an exchange with a maximum)
        uint64_t* const w = slots + (size_t)pass * 4 * G;
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));                      // (as in decide)
        const uint64_t bits = f64_to_bits(a);
        if (tid == 0) {
            put(w + g, tag, (uint32_t)(bits >> 32));
            put(w + G + g, tag, (uint32_t)bits);
            if (MAX) put(w + 2 * G + g, tag, __float_as_uint(b));
            if (MAX && first) put(w + 3 * G + g, tag, (uint32_t)wall_clock64());
        }
        if (tid < (!MAX ? 2 : first ? 4 : 3) * G) {
            uint32_t x = 0;
            if (!get(w + tid, &x)) sh.fail = 1;
            sh.got[tid] = x;
        }
        __syncthreads();
        if (__builtin_amdgcn_readfirstlane(sh.fail)) return false;
        if (first) tag = nonce ^ (sh.got[3 * G] * 0x9E3779B1u);
        else if (pass == 1) clear();
        ++pass;
        return true;
    }
    __device__ __forceinline__ double value(const Shared& sh, int i) const { return bits_to_f64(((uint64_t)sh.got[i] << 32) | sh.got[G + i]); }
    // this workgroup's records of the first exchange
    __device__ __forceinline__ void clear() const {
        if (threadIdx.x < 4) put(slots + threadIdx.x * G + g, ~nonce, 0u);
    }
};

// Decides node `cur`: its accepted child, or -1 and the correction token, or kLeave if the team could not complete an
// exchange.  (All threads of all workgroups of the team return the same; with several workgroups the token is known to
// workgroup 0 only.)
constexpr int kLeave = -2;
template <typename T, int NG, bool TEAM>
__device__ __forceinline__ int decide(const ResampleArgs& a, Shared& sh, Team& team, int b, int cur, int blk0, int blk1, int32_t* token) {
    // Registers: a block's weights take 16, its draft probabilities 8, its logits 8 until they are weights; the rest, the constants of the
    // exponential foremost, about 65.  A team's kernel has 89, 112 and 162 with 1, 2 and 4 blocks, and 244 with 8, whose draft probabilities
    // are read again at every use; nothing is spilled.  What that takes: the draft probabilities are requested when the logits are
    // weights; branches that all threads take alike are scalar ones, and the weights are not changed under a condition (both would keep
    // them twice); and the compiler must not know that a thread's number is the same for every node of a walk, or addresses and
    // the masks of a row's end are computed once and kept.  With all of it left out, 8 blocks took 256 registers and spilled
    // 497.  us a call, before and after: 256 x 32 nodes, V 32000 (8 blocks) 350 and 90; 16 x 128, 128256 (2) 57.4 and 47.4;
    // 4 x 64, 32000 (1) 41.5 and 37.3.
    int tid = threadIdx.x;
    if (TEAM) asm volatile("" : "+v"(tid));
    const int V = a.V, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), N = a.N;
    Row row;
    row.V = V;
    row.lg = (const T*)a.logits + ((size_t)b * N + cur) * V;
    row.q = a.draft + ((size_t)b * N + cur) * V;
    row.vec = (((uintptr_t)row.lg | (uintptr_t)row.q) & 15) == 0;
    const double invT = a.inv_temperature;

    constexpr bool kKeepQ = NG <= 4;                       // (eight blocks' weights leave no room for it: read again at every use)
    double w[NG][8];
    float q[kKeepQ ? NG : 1][8];
    {
        float x[NG][8];
#pragma unroll
        for (int it = 0; it < NG; ++it) {
            if (blk0 + it < blk1) {
                load_logits8<T>(row, (blk0 + it) * kBlock + lane * 8, x[it]);
            } else {
#pragma unroll
                for (int k = 0; k < 8; ++k) x[it][k] = -INFINITY;
            }
        }
        // ---- children of cur, in increasing node index (a token that is no token id is rejected, and nothing carried)
        const int tok = tid < N ? sh.tok[tid] : -1;
        const bool mine = tid < N && tid > cur && sh.par[tid] == cur && tok >= 0 && tok < V;
        float lx = 0.f, qx = 0.f, ux = 0.f;
        if (mine) {
            lx = to_f32<T>(((const T*)row.lg)[tok]);
            qx = row.q[tok];
            ux = a.uniforms[(size_t)b * N + tid];
        }
        const unsigned long long mask = __ballot(mine);
        if (wave < 2 && lane == 0) sh.count[wave] = __popcll(mask);
        __syncthreads();
        if (mine) sh.child[__popcll(mask & ((1ull << lane) - 1ull)) + (wave == 1 ? sh.count[0] : 0)] = tid;
        const int n_child = __builtin_amdgcn_readfirstlane(sh.count[0] + sh.count[1]);
        auto load_q = [&](int it, int at, float (&to)[8]) __attribute__((always_inline)) {
            if (n_child > 0 && blk0 + it < blk1) {
                load_draft8(row, (blk0 + it) * kBlock + at, to);
            } else {
#pragma unroll
                for (int k = 0; k < 8; ++k) to[k] = 0.f;
            }
        };
        auto load_all_q = [&]() __attribute__((always_inline)) {
            if constexpr (kKeepQ) {
#pragma unroll
                for (int it = 0; it < NG; ++it) load_q(it, lane * 8, q[it]);
            }
        };
        auto q_of = [&](int it) __attribute__((always_inline)) -> float (&)[8] {
            if constexpr (kKeepQ) return q[it];
            int at = lane * 8;
            asm volatile("" : "+v"(at));
            load_q(it, at, q[0]);
            return q[0];
        };
        if (!TEAM) load_all_q();
        // ---- row maximum (exact), the weights against the slice's, and their sum
        float ms = x[0][0];
#pragma unroll
        for (int it = 0; it < NG; ++it)
#pragma unroll
            for (int k = 0; k < 8; ++k) ms = fmaxf(ms, x[it][k]);
        ms = wave_max(ms);
        if (lane == 0) sh.redf[wave] = ms;
        __syncthreads();
        ms = sh.redf[0];
#pragma unroll
        for (int i = 1; i < kWaves; ++i) ms = fmaxf(ms, sh.redf[i]);
        ms = uniform_f32(ms);
        double s = 0.0;
        const double md = ms > -INFINITY ? (double)ms : 0.0;         // (a slice behind the vocabulary's end: no weights)
#pragma unroll
        for (int it = 0; it < NG; ++it) {
            keep_order();
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                if (TEAM && k % 2 == 0) keep_order();
                w[it][k] = exp(((double)x[it][k] - md) * invT);      // padding: exp(-inf) = 0
                s += w[it][k];
            }
        }
        if (TEAM) {              // (where the logits were; they arrive while the sums are exchanged)
            keep_order();
            load_all_q();
        }
        s = wave_sum(s);
        if (lane == 0) sh.red[0][wave] = s;
        __syncthreads();
        double sg = 0.0;
#pragma unroll
        for (int i = 0; i < kWaves; ++i) sg += sh.red[0][i];
        float m = ms;
        double f = 1.0;
        if (TEAM && team.G > 1) {
            if (!team.template exchange<true>(sh, sg, ms)) return kLeave;
            // lane i brings workgroup i's sum to the row's maximum
            const float mi = lane < team.G ? __uint_as_float(sh.got[2 * team.G + lane]) : -INFINITY;
            m = wave_max(mi);
            sg = wave_sum(mi > -INFINITY ? team.value(sh, lane) * exp(((double)mi - (double)m) * invT) : 0.0);
            f = ms > -INFINITY ? exp(((double)ms - (double)m) * invT) : 0.0;
        }
        if (TEAM) {              // (also where there is nothing to change: under the condition above, the weights would be kept twice)
#pragma unroll
            for (int it = 0; it < NG; ++it)
#pragma unroll
                for (int k = 0; k < 8; ++k) w[it][k] *= f;
        }
        if (mine) {
            sh.ax[tid] = exp(((double)lx - (double)m) * invT);
            sh.lhs[tid] = (double)ux * (double)qx;
        }
        __syncthreads();

        // ---- the children, one after the other (every thread of every workgroup of the team takes the same branches).
        // The weights in registers lag by the last rejection: w' = max(0, w - owed q).
        double S = sg, owed = 0.0;
        int buf = 1;
        for (int i = 0; i < n_child; ++i) {
            const int c = __builtin_amdgcn_readfirstlane(sh.child[i]);
            if (__builtin_amdgcn_readfirstlane(sh.lhs[c] < sh.ax[c] / S)) return c;
            double z = 0.0;                                          // rejected: mass of max(0, w' - S q)
#pragma unroll
            for (int it = 0; it < NG; ++it) {
                keep_order();
                float (&qi)[8] = q_of(it);
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    if (TEAM && k % 2 == 0) keep_order();
                    if (TEAM) asm volatile("" : "+v"(qi[k]));            // (or all of them would be held as doubles, converted in front of the loop)
                    const double qd = (double)qi[k];
                    w[it][k] = fmax(0.0, w[it][k] - owed * qd);
                    z += fmax(0.0, w[it][k] - S * qd);
                }
            }
            owed = 0.0;
            z = wave_sum(z);
            if (lane == 0) sh.red[buf][wave] = z;
            __syncthreads();
            double t = 0.0;
#pragma unroll
            for (int j = 0; j < kWaves; ++j) t += sh.red[buf][j];
            buf ^= 1;
            if (TEAM && team.G > 1) {
                if (!team.template exchange<false>(sh, t)) return kLeave;
                t = wave_sum(lane < team.G ? team.value(sh, lane) : 0.0);
            }
            if (t > 0.0) {                                           // same value in every thread; no mass left: nothing carried
                if (mine) sh.ax[tid] = fmax(0.0, sh.ax[tid] - S * (double)qx);
                owed = S;
                S = t;
            }
            __syncthreads();
        }
        // (behind this point w are the weights that the correction token is drawn from)
#pragma unroll
        for (int it = 0; it < NG; ++it) {
            keep_order();
            const float (&qi)[8] = q_of(it);
#pragma unroll
            for (int k = 0; k < 8; ++k) w[it][k] = fmax(0.0, w[it][k] - owed * (double)qi[k]);
        }
    }

    // ---- correction / bonus token: inverse CDF at u_resample, token-id order: the first of the team's workgroups, of its
    // waves, of the wave's blocks, of the block's lanes and of the lane's tokens whose inclusive sum exceeds the target; the
    // last one with any mass if none does (the target reaches the total by rounding only)
    double ls[NG], s = 0.0;
#pragma unroll
    for (int it = 0; it < NG; ++it) {
        ls[it] = ((w[it][0] + w[it][1]) + (w[it][2] + w[it][3])) + ((w[it][4] + w[it][5]) + (w[it][6] + w[it][7]));
        s += ls[it];
    }
    s = wave_sum(s);
    __syncthreads();
    if (lane == 0) sh.red[0][wave] = s;
    if (tid == 0) sh.token = 0;
    __syncthreads();
    double slice = 0.0;
#pragma unroll
    for (int i = 0; i < kWaves; ++i) slice += sh.red[0][i];
    double excl = 0.0, total = slice;
    int gsel = 0;
    double part = 0.0, incl_g = 0.0;                   // of workgroup `lane`: its sum, and the sum up to and with it
    if (TEAM && team.G > 1) {
        if (!team.template exchange<false>(sh, slice)) return kLeave;
        part = lane < team.G ? team.value(sh, lane) : 0.0;
        incl_g = wave_incl_scan(part);
        total = of_lane(incl_g, 63);
    }
    const double tgt = (double)a.u_resample[b] * total;
    if (TEAM && team.G > 1) {
        const unsigned long long hits = __ballot(part > 0.0 && incl_g > tgt), pos = __ballot(part > 0.0);
        gsel = hits ? __ffsll((long long)hits) - 1 : pos ? 63 - __clzll((long long)pos) : 0;
        if (gsel > 0) excl = of_lane(incl_g, gsel - 1);
    }
    if (team.g == gsel) {
        int wsel = -1, wlast = 0;
        double wexcl = excl, run = excl, wlexcl = excl;
        for (int i = 0; i < kWaves; ++i) {
            const double v = sh.red[0][i];
            if (v > 0.0) { wlast = i; wlexcl = run; }
            if (wsel < 0 && run + v > tgt) { wsel = i; wexcl = run; }
            run += v;
        }
        if (wsel < 0) { wsel = wlast; wexcl = wlexcl; }
        if (wave == wsel) {
            double incl[NG], e_sel = 0.0;
            int isel = -1, ilast = 0;
            double ilexcl = wexcl;
            run = wexcl;
#pragma unroll
            for (int it = 0; it < NG; ++it) {
                incl[it] = wave_incl_scan(ls[it]);
                const double v = of_lane(incl[it], 63);
                if (v > 0.0) { ilast = it; ilexcl = run; }
                if (isel < 0 && run + v > tgt) { isel = it; e_sel = run; }
                run += v;
            }
            if (isel < 0) { isel = ilast; e_sel = ilexcl; }
#pragma unroll
            for (int it = 0; it < NG; ++it)
                if (it == isel) {
                    const bool hit = (e_sel + incl[it] > tgt) && ls[it] > 0.0;
                    const unsigned long long hits = __ballot(hit), pos = __ballot(ls[it] > 0.0);
                    const int lsel = hits ? __ffsll((long long)hits) - 1 : 63 - __clzll((long long)(pos ? pos : 1ull));
                    if (lane == lsel) {
                        double r3 = e_sel + (incl[it] - ls[it]);
                        int pick = -1, lastpos = -1;
#pragma unroll
                        for (int k = 0; k < 8; ++k) {
                            r3 += w[it][k];
                            if (w[it][k] > 0.0) lastpos = k;
                            if (pick < 0 && r3 > tgt && w[it][k] > 0.0) pick = k;
                        }
                        if (pick < 0) pick = max(lastpos, 0);
                        sh.token = (blk0 + it) * kBlock + lane * 8 + pick;
                    }
                }
        }
    }
    __syncthreads();
    if (gsel != 0) {                                   // the token goes to workgroup 0, through one more slot
        if (team.pass >= team.max_pass) return kLeave;
        uint64_t* slot = team.slots + (size_t)team.pass++ * 4 * team.G;
        if (team.g == gsel && tid == 0) Team::put(slot, team.tag, (uint32_t)sh.token);
        if (team.g == 0 && tid == 0) {
            uint32_t x = 0;
            if (team.get(slot, &x)) sh.token = (int)x; else sh.fail = 1;
        }
        __syncthreads();
        if (__builtin_amdgcn_readfirstlane(sh.fail)) return kLeave;
    }
    *token = sh.token;
    return -1;
}

// The tree of sequence b into LDS; true if it is none: node 0 is the only root, parents precede children, depth < max_path.
__device__ __forceinline__ bool load_tree(const ResampleArgs& a, Shared& sh, int b, bool check) {
    const int tid = threadIdx.x, N = a.N;
    int bad = 0;
    if (tid == 0) sh.fail = 0;
    if (tid < N) {
        const int p = a.parent[(size_t)b * N + tid];
        sh.par[tid] = p;
        sh.tok[tid] = a.tokens[(size_t)b * N + tid];
        bad = (tid == 0) ? (p != -1) : (p < 0 || p >= tid);
    }
    bad = __syncthreads_or(bad);
    if (!check) return bad;
    if (!bad && tid < N) {
        int depth = 0;
        for (int i = tid; i > 0; i = sh.par[i]) ++depth;
        bad = depth >= a.max_path;
    }
    return __syncthreads_or(bad);
}

__device__ __forceinline__ void empty_path(const ResampleArgs& a, int b) {
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));                 // (as in decide)
    for (int k = tid; k < a.max_path; k += kThreads) {
        a.path[(size_t)b * a.max_path + k] = (k == 0) ? 0 : -1;
        a.accepted_tokens[(size_t)b * a.max_path + k] = -1;
    }
}
// nothing accepted, no token
__device__ __forceinline__ void write_empty(const ResampleArgs& a, int b, int status) {
    empty_path(a, b);
    if (threadIdx.x == 0) {
        a.accept_len[b] = 0;
        a.bonus_token[b] = -1;
        if (a.status) a.status[b] = status;
    }
}

// ---- teams: workgroup g of sequence b's team walks from the root
template <typename T, int NG>
__global__ __launch_bounds__(kThreads, resample_per_cu(NG) * kWaves / 4) void accept_resample_kernel(ResampleArgs a) {
    __shared__ Shared sh;
    const int G = a.team, tid = threadIdx.x;
    const ResampleMember me = resample_member(blockIdx.x, G, a.groups);
    const int b = a.first + me.sequence, g = me.g;
    if (b >= a.B) return;                                  // (fills up the last round of groups)
    if (load_tree(a, sh, b, true)) {                       // every workgroup of the team sees the same tree
        if (g == 0) write_empty(a, b, S4C_SEQ_BAD_TREE);
        return;
    }
    const int nblocks = (a.V + kBlock - 1) / kBlock;
    const int bpg = (nblocks + G - 1) / G, ipw = (bpg + kWaves - 1) / kWaves;              // blocks per workgroup and wave
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int gblk1 = min(nblocks, (g + 1) * bpg), blk0 = min(gblk1, g * bpg + wave * ipw), blk1 = min(gblk1, blk0 + ipw);
    Team team = {a.slots + (size_t)b * a.max_pass * 4 * G, g, G, a.max_pass, a.spin_limit, 0, a.nonce, a.nonce};
    int cur = 0, L = 0;
    int32_t token = -1;
    if (g == 0) empty_path(a, b);
    for (;;) {
        const int next = decide<T, NG, true>(a, sh, team, b, cur, blk0, blk1, &token);
        if (next == kLeave) {                              // workgroup 0 flags the sequence and empties its outputs
            __syncthreads();                               // (thread 0's earlier path entries come before)
            if (G > 1) team.clear();
            if (g == 0) write_empty(a, b, S4C_SEQ_TIMEOUT);
            return;
        }
        if (next < 0) break;
        ++L;
        if (g == 0 && threadIdx.x == 0) {
            a.path[(size_t)b * a.max_path + L] = next;
            a.accepted_tokens[(size_t)b * a.max_path + L - 1] = sh.tok[next];
        }
        cur = next;
        __syncthreads();                                   // the node's shared words are written again
    }
    if (g == 0 && tid == 0) {
        a.accept_len[b] = L;
        a.bonus_token[b] = token;
        if (a.status) a.status[b] = 0;
    }
}

// ---- rows: workgroup b N + i decides node i of sequence b and publishes (call nonce, decision); workgroup B N + b waits
// for its sequence's decisions, overwrites them (so that a captured graph can replay the call) and follows them.  A decision that
// it gave up on is overwritten by the node's own workgroup, which finds the word (~nonce, 1) left for it there (an exchange in place
// of a store: 1 x 20, V 1000 8.75 and 8.70 us, 3 x 64, 16000 fp32 17.7 and 17.9, 4 x 40, 8000 11.6 and 11.7).  Every
// XCD starts its share of the workgroups in grid order, the waiting ones behind the nodes', which wait for nobody.
constexpr uint32_t kAccepted = 0x80000000u;                // decision: kAccepted | child, or the correction token
template <typename T, int NG>
__global__ __launch_bounds__(kThreads) void resample_rows_kernel(ResampleArgs a) {
    __shared__ Shared sh;
    const int tid = threadIdx.x, N = a.N;
    if ((int)blockIdx.x < a.B * N) {
        const int b = blockIdx.x / N, node = blockIdx.x - b * N;
        load_tree(a, sh, b, false);                        // (whatever it holds: rows and tokens are checked where they are used)
        const int nblocks = (a.V + kBlock - 1) / kBlock, ipw = (nblocks + kWaves - 1) / kWaves;
        const int blk0 = min(nblocks, __builtin_amdgcn_readfirstlane(tid >> 6) * ipw), blk1 = min(nblocks, blk0 + ipw);
        Team team = {nullptr, 0, 1, 0, 0, 0, 0, 0};
        int32_t token = 0;
        const int next = decide<T, NG, false>(a, sh, team, b, node, blk0, blk1, &token);
        if (tid == 0) {
            const uint64_t before = __hip_atomic_exchange(a.slots + blockIdx.x, ((uint64_t)a.nonce << 32) | (next >= 0 ? kAccepted | (uint32_t)next : (uint32_t)token),
                                                          __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (before == (((uint64_t)(~a.nonce) << 32) | 1u))
                __hip_atomic_store(a.slots + blockIdx.x, (uint64_t)(~a.nonce) << 32, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        return;
    }
    const int b = blockIdx.x - a.B * N;
    const bool bad = load_tree(a, sh, b, true);
    __shared__ uint32_t s_said[kMaxNodes];
    int late = 0;
    if (tid < N) {
        uint64_t* const rec = a.slots + (size_t)b * N + tid;
        uint64_t v = 0;
        late = 1;
        for (int spin = 0; late && spin < a.spin_limit; ++spin) {
            v = __hip_atomic_load(rec, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            late = (uint32_t)(v >> 32) != a.nonce;
            if (late) __builtin_amdgcn_s_sleep(8);
        }
        s_said[tid] = (uint32_t)v;
        if (!late || (uint32_t)(__hip_atomic_exchange(rec, ((uint64_t)(~a.nonce) << 32) | 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >> 32) == a.nonce)
            __hip_atomic_store(rec, (uint64_t)(~a.nonce) << 32, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    late = __syncthreads_or(late);
    if (late || bad) {
        write_empty(a, b, late ? S4C_SEQ_TIMEOUT : S4C_SEQ_BAD_TREE);
        return;
    }
    // every thread follows the path, thread k writes entry k
    int cur = 0, L = 0, my_node = tid == 0 ? 0 : -1, my_tok = -1;
    while (s_said[cur] & kAccepted) {
        cur = (int)(s_said[cur] & ~kAccepted);
        ++L;
        if (L == tid) my_node = cur;
        if (L == tid + 1) my_tok = sh.tok[cur];
    }
    for (int k = tid; k < a.max_path; k += kThreads) {
        a.path[(size_t)b * a.max_path + k] = k == tid ? my_node : -1;         // (a path has at most kMaxNodes < kThreads nodes)
        a.accepted_tokens[(size_t)b * a.max_path + k] = k == tid ? my_tok : -1;
    }
    if (tid == 0) {
        a.accept_len[b] = L;
        a.bonus_token[b] = (int32_t)s_said[cur];
        if (a.status) a.status[b] = 0;
    }
}

template <typename T, int NG>
hipError_t launch(const ResampleArgs& a, hipStream_t st) {
    if constexpr (NG * kWaves * kBlock <= kMaxRow) if (a.team == 0) {
        hipLaunchKernelGGL((resample_rows_kernel<T, NG>), dim3((unsigned)(a.B * (a.N + 1))), dim3(kThreads), 0, st, a);
        return hipGetLastError();
    }
    const ResampleLaunch l = resample_launch(a.B, a.team, NG, a.cus);
    for (int b = 0; b < a.B; b += l.sequences) {
        ResampleArgs k = a;
        k.first = b;
        k.groups = l.groups;
        const int n = a.B - b < l.sequences ? a.B - b : l.sequences;
        hipLaunchKernelGGL((accept_resample_kernel<T, NG>), dim3((unsigned)resample_grid(n, a.team, l.groups)), dim3(kThreads), 0, st, k);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}
template <typename T>
hipError_t launch_sized(const ResampleArgs& a, hipStream_t st) {
    const int nblocks = resample_blocks(a.V), n = resample_iters(a.team ? (nblocks + a.team - 1) / a.team : nblocks);
    return n == 1 ? launch<T, 1>(a, st) : n == 2 ? launch<T, 2>(a, st) : n == 4 ? launch<T, 4>(a, st) : launch<T, 8>(a, st);
}

}  // namespace

int resample_max_vocab() { return kMaxVocab; }

// exchanges per sequence: one per visited node, one per rejected child, one for the sampling, one
// to hand the token to workgroup 0
int resample_max_pass(int N, int max_path) { return max_path + N + 2; }
int resample_default_spin_limit() { return kSpinLimit; }

size_t resample_slot_words(int B, int N, int V, int max_path, int cus) {
    const int G = resample_team(B, V, cus);
    return G == 1 ? 0 : (size_t)B * resample_max_pass(N, max_path) * 4 * G;
}

hipError_t launch_accept_resample(const ResampleArgs& a, hipStream_t st) {
    return a.dtype == S4C_F32 ? launch_sized<float>(a, st) : a.dtype == S4C_F16 ? launch_sized<f16_t>(a, st) : launch_sized<bf16_t>(a, st);
}

}  // namespace s4c

// Path acceptance (paper Sec. 3.2: per-node test, then the longest accepted path) in ONE launch; and the same launch
// extended to the rest of a verification step (last section of this comment).
//
// Scan (the HBM-bound part).  The rows to scan of a sequence -- every row in greedy mode (the bonus token may come from
// any), the rows of nodes that have children in stochastic mode -- are laid end to end and cut into equal runs of
// 8192-logit chunks, one for each of the sequence's scanning workgroups.  For batches of no more sequences than the chip
// holds workgroups (scan_plan) the scanning workgroups are resident at once on a free chip, so none of them waits for a second turn; what
// else the launch holds comes behind them in the grid.  (Fixed segments of up to 8 chunks made config 5 2612 workgroups on
// 1280 places, the third turn almost empty.)  Measured, whole calls back to back on one input, against fixed segments: 345 MB of bf16
// logits 72.3 -> 70.5 us, 131 MB 29.0 -> 28.0, 9 MB 11.9 -> 9.1, 4 MB 10.8 -> 6.7; 51 MB in rows of odd length 71.7 -> 18.7.
// About 6 us of that are the launch, the first loads and the collector's look.  With inputs that the last-level cache does not
// hold from the call before, 335 MB take 76 us and 131 MB 32: 4.8 - 5 TB/s behind those 6 us.
// A chunk is read exactly once with 16-byte loads, the next one in
// flight while it is reduced, across the ends of rows too.
//   Greedy: per thread a running maximum; the raw words of the chunk that holds it are kept aside, and its position
//   is looked up in them once per row; the 256 threads are then combined with an order-independent (value, lowest
//   index) reduction.
//   Stochastic: per thread a sum of exp2 against a reference that moves only when a logit outgrows it by more than
//   2^kLazyLog2 (any reference serves, as long as reference and sum go together).
//
// Path step.  A run publishes its statistics of each row it touches as two 8-byte records (call nonce in the upper
// half) with device-coherent stores.  The sequence's collector, a workgroup of its own behind the scanning ones in the
// grid, loads everything else the path step needs and then polls the records of the sequence until every one
// carries this call's nonce, combines them per row, applies the per-node test against the parent's row, ANDs along each
// node's ancestor chain and writes the deepest accepted node's path (lowest index among equals).  No second launch,
// no read-modify-write atomics (they serialise per address and take microseconds across the chip's separate L2s), no
// cache flush: only the records bypass the non-coherent part of the L2.
// A record needs no initialisation: anything without this call's nonce is "not there yet".  The
// collector overwrites what it consumed with the complement of the nonce, so a captured graph can
// replay the call, nonce and all.  The collector's wait is bounded by wall-clock time; when it runs
// out (which needs a GPU that stops scheduling the sequence's other workgroups) the sequence is
// flagged S4C_SEQ_TIMEOUT and gets the empty result.  Workgroups are dispatched in grid order within each
// eighth of the chip, so a collector seldom starts before the workgroups that it waits for; it may, where other streams hold places.
//
// step_kernel: the acceptance scan with its collectors, then the workgroups of the attention merge (it only needs the
// attention kernel to have ended; the other chain is the longer one), then workgroups that append the accepted path's K/V rows to the cache: a few per
// sequence, a group of KV heads each, which wait for a message from the collector (the path, the cache length it
// has read and advanced).  At batch 1 the three launches this replaces were 2 us of work each behind 2 us of launch, and a
// sequence's rows, copied by one workgroup, waited for one address translation after another (each KV head's
// rows lie in pages of their own): 13b, batch 4: 12.5 + 5.6 + 10.4 us in three launches.
#pragma once
#include "attn_merge.h"
#include "row_chunk.h"
#include "told.h"

namespace s4c {

namespace told {
// a word and its mark in device memory
struct Pair { uint64_t word, mark; };
struct At {
    Pair* p;
    static __device__ __forceinline__ uint64_t load(const uint64_t* at) { return __hip_atomic_load(at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
    static __device__ __forceinline__ void store(uint64_t* at, uint64_t v) { __hip_atomic_store(at, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
    __device__ __forceinline__ uint64_t word() const { return load(&p->word); }
    __device__ __forceinline__ uint64_t mark() const { return load(&p->mark); }
    __device__ __forceinline__ void set_word(uint64_t v) const { store(&p->word, v); }
    __device__ __forceinline__ void set_mark(uint64_t v) const { store(&p->mark, v); }
    __device__ __forceinline__ void settle() const { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
};
}  // namespace told

namespace accept {

using namespace rowchunk;

typedef unsigned long long rec_t;
// Scanning workgroups that a CU holds at once: 5 (96 registers a thread), each with 16 KB of logits in flight, where
// a CU needs about 50 KB to stream at its share of the memory's rate; 3 with 32 KB each for fp32 logits.
template <typename T>
constexpr int kWavesPerSimd = sizeof(T) == 4 ? 3 : 5;

__device__ __forceinline__ void publish(rec_t* p, uint32_t nonce, uint32_t bits) {
    __hip_atomic_store(p, ((rec_t)nonce << 32) | bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Loads the records of up to four consecutive runs of a row in one burst (the loads are
// independent round trips of a microsecond or two each, so they must not be taken one after the
// other) and repeats until every one carries the nonce or the deadline (100 MHz wall clock) has
// passed; returns whether they all arrived.  bits[2 s + w] = payload of word w of run s.
__device__ __forceinline__ bool await4(const rec_t* p, int runs, uint32_t nonce, long long deadline, uint32_t (&bits)[8]) {
    for (;;) {
        rec_t w[8];
#pragma unroll
        for (int e = 0; e < 8; ++e)
            w[e] = e < 2 * runs ? __hip_atomic_load(p + e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : ((rec_t)nonce << 32);
        bool all = true;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            all = all && ((uint32_t)(w[e] >> 32) == nonce);
            bits[e] = (uint32_t)w[e];
        }
        if (all) return true;
        if ((long long)wall_clock64() - deadline >= 0) return false;
        __builtin_amdgcn_s_sleep(2);
    }
}

// ---- the division of a sequence's scan
// The scanned nodes of sequence b in LDS, ascending, and their number (ranks: position of a node, -1 for a row that is
// not scanned).  All threads; ends with a barrier.
struct Rows {
    int32_t list[kMaxNodes], rank[kMaxNodes], has[kMaxNodes], count[2];
};
// What the workgroups here have in LDS.  (Given by the kernel: in an attention launch it is part of the tiles' ring.)
struct Shared {
    Rows rows;
    int32_t any[4];
    float v[4], s[4];                                        // a scanning workgroup's waves
    int32_t i[4];
    int32_t parent[kMaxNodes], g[kMaxNodes], node[kMaxNodes], best, len;     // a collector's nodes, its result
    uint64_t above[kMaxNodes][2], ok[2];                     // each node's ancestors and itself; the nodes that pass their test
    float m[kMaxNodes], S[kMaxNodes];
    int32_t msg[2 + kMaxNodes];                              // a copier's message
};
// Whether one of the kThreads threads says so.  (A kernel with more threads sends the others away first.)
__device__ __forceinline__ bool any_of(Shared& sh, bool mine) {
    const bool w = __any(mine) != 0;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh.any[threadIdx.x >> 6] = w;
    __syncthreads();
    return sh.any[0] | sh.any[1] | sh.any[2] | sh.any[3];
}
__device__ __forceinline__ int find_rows(const AcceptArgs& a, int b, Rows& r) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, N = a.N;
    if (a.mode == S4C_GREEDY) {
        if (tid < kMaxNodes) r.list[tid] = r.rank[tid] = tid;
        __syncthreads();
        return N;
    }
    // waves 0 and 1 hold one node per lane
    if (tid < kMaxNodes) r.has[tid] = 0;
    __syncthreads();
    if (tid >= 1 && tid < N) {
        const int p = a.parent[(size_t)b * N + tid];
        if (p >= 0 && p < N) r.has[p] = 1;                 // a malformed tree is reported by the path step
    }
    __syncthreads();
    const int has = tid < N ? r.has[tid] : 0;
    const unsigned long long mask = __ballot(has);
    if (lane == 0 && wave < 2) r.count[wave] = __popcll(mask);
    __syncthreads();
    if (tid < kMaxNodes) {
        const int rank = __popcll(mask & ((1ull << lane) - 1ull)) + (wave == 1 ? r.count[0] : 0);
        r.rank[tid] = has ? rank : -1;
        if (has) r.list[rank] = tid;
    }
    __syncthreads();
    return r.count[0] + r.count[1];
}
// Run j of `used`: `per` units, one more for the first `rem`; a unit is a chunk, or a whole row where rows are the shorter
// way to runs of plan.seg chunks.
struct Runs {
    int unit, used, per, rem;
    __device__ __forceinline__ Runs(const AcceptArgs& a, int rows) {
        unit = a.plan.slots == 1 ? a.chunks : 1;
        const int units = a.plan.slots == 1 ? rows : rows * a.chunks;
        used = max(1, min(a.plan.wgs, a.plan.slots == 1 ? rows : units / a.plan.seg));
        per = units / used;
        rem = units - per * used;
    }
    __device__ __forceinline__ int begin(int j) const { return (j * per + min(j, rem)) * unit; }       // first chunk
    __device__ __forceinline__ int of_chunk(int c) const {
        const int u = c / unit, big = rem * (per + 1);
        return u < big ? u / (per + 1) : rem + (u - big) / max(per, 1);
    }
};
constexpr float kLazyLog2 = 24.0f;

// ---- what a step adds
enum Part { kAlone, kBehindAttention, kBesideAttention };     // acceptance by itself; a step's second launch; its only one
struct StepArgs {
    CompactArgs compact;
    rec_t* messages;            // [B][copiers][kMessageWords]
    told::Pair* lens;           // in the launch of the attention: [B][attn_wgs], told by every attention workgroup when it has read cache_len
    int32_t attn_wgs;
    uint64_t tag;               // of these
    long long copy_ticks;       // how long a copier waits for its message (100 MHz wall clock)
    int32_t merge_wgs, merge_chunks, merge_passes;           // behind the attention.  balanced shares: attn_merge.h; equal runs: attn_parts.h, a wave each
    int32_t scan_wgs;
    int32_t copiers, heads;     // workgroups per sequence that append rows, KV heads of each
};
constexpr int kMessage = 2 + kMaxNodes;          // records: cache length (or -1), accepted length, path nodes
constexpr int kMessageWords = kMessage + 1;      // and one in which the copier tells that it has given up
constexpr int kMostCopiers = 8;

// The collector's half of the compaction, as s4c_kv_compact: checks that the rows fit, writes dst_index and status,
// advances cache_len, and tells the sequence's copiers, each in a message of its own (it clears the message when
// it has read it, so that a captured graph can replay the call).  Path of L + 1 nodes in `node`; all threads.
__device__ __forceinline__ void announce_path(const StepArgs& x, const AcceptArgs& a, Shared& sh, int b, int base, bool unread) {
    const CompactArgs& c = x.compact;
    const int i = threadIdx.x;
    const int L = sh.len;
    const bool bad = unread || base < 0 || (long long)base + L + 1 > c.S_cap;
    rec_t* const first = x.messages + (size_t)b * x.copiers * kMessageWords;
    if (i < kMessage) {
        const int32_t word = i == 0 ? (bad ? -1 : base) : i == 1 ? L : i - 2 <= L ? sh.node[i - 2] : -1;
        for (int w = 0; w < x.copiers; ++w) publish(first + w * kMessageWords + i, a.nonce, (uint32_t)word);
    }
    if (c.dst_index)
        for (int k = i; k < c.max_path; k += kThreads) c.dst_index[(size_t)b * c.max_path + k] = (!bad && k <= L) ? base + k : -1;
    if (i == 0) {
        if (c.status) c.status[b] = unread ? S4C_SEQ_TIMEOUT : bad ? S4C_SEQ_BAD_LEN : 0;
        if (!bad) c.cache_len[b] = base + L + 1;
    }
}
// The end of a collector: whether a copier has left before it was told (told.h, a message for a word).  Then rows are missing, so the sequence is
// flagged and its length is what it was; nothing of the message or of the mark stays behind.  (A copier waits longer than a
// collector does before it gives up, but a collector may begin later.)
__device__ __forceinline__ void look_for_leavers(const StepArgs& x, const AcceptArgs& a, Shared& sh, int b, int base) {
    const CompactArgs& c = x.compact;
    const int i = threadIdx.x;
    rec_t* const first = x.messages + (size_t)b * x.copiers * kMessageWords;
    auto left = [&](const rec_t* mark) { return (uint32_t)(__hip_atomic_load(mark, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >> 32) == a.nonce; };
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();                                       // every thread's words can be seen
    if (!any_of(sh, i < x.copiers && left(first + i * kMessageWords + kMessage))) return;
    for (int w = 0; w < x.copiers; ++w) {
        rec_t* const m = first + w * kMessageWords;
        const bool gone = left(m + kMessage);
        __syncthreads();                                   // every thread has looked before the mark is cleared
        if (gone && i <= kMessage) publish(m + i, ~a.nonce, 0u);
    }
    if (c.dst_index)
        for (int k = i; k < c.max_path; k += kThreads) c.dst_index[(size_t)b * c.max_path + k] = -1;
    if (i == 0) {
        if (c.status) c.status[b] |= S4C_SEQ_TIMEOUT;
        c.cache_len[b] = base;
    }
}

// A copier: waits for its message, appends the path's rows of its KV heads.
__device__ __forceinline__ void copy_rows(const StepArgs& x, const AcceptArgs& a, Shared& sh, int b, int w) {
    const CompactArgs& c = x.compact;
    int32_t* const s_msg = sh.msg;
    const int tid = threadIdx.x;
    rec_t* const m = x.messages + ((size_t)b * x.copiers + w) * kMessageWords;
    const int h0 = w * x.heads, nh = min(c.Hkv, h0 + x.heads) - h0, shift = 31 - __builtin_clz(c.row_bytes / 16);   // (vectors of a row: 8, 16 or 32)
    constexpr int kInFlight = 4;
    // vector e of the rows belongs to row k of the path and KV head h (those of the first pass are found before the message is here)
    int row[kInFlight], head[kInFlight];
    const size_t v16 = (size_t)(tid & ((1 << shift) - 1)) * 16;              // (kThreads is a multiple of a row's vectors)
    auto place = [&](int e0) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < kInFlight; ++u) {
            const int q = (e0 + u * kThreads) >> shift;
            row[u] = q / nh;
            head[u] = h0 + q - row[u] * nh;
        }
    };
    place(tid);
    // this thread's word, if it is this call's
    auto look = [&]() {
        const rec_t v = __hip_atomic_load(m + tid, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        s_msg[tid] = (int32_t)(uint32_t)v;
        return (uint32_t)(v >> 32) == a.nonce;
    };
    int late = 0;
    if (tid < kMessage) {
        const long long deadline = (long long)wall_clock64() + x.copy_ticks;
        while (!look()) {
            if ((long long)wall_clock64() - deadline >= 0) { late = 1; break; }
            __builtin_amdgcn_s_sleep(4);
        }
    }
    if (any_of(sh, late)) {
        if (tid == 0) publish(m + kMessage, a.nonce, 1u);
        __threadfence();
        __syncthreads();
        __threadfence();
        if (any_of(sh, tid < kMessage && !look())) return;       // the collector flags the sequence (look_for_leavers)
        if (tid == 0) publish(m + kMessage, ~a.nonce, 0u);
    }
    if (tid < kMessage) publish(m + tid, ~a.nonce, 0u);
    const int base = s_msg[0], L = s_msg[1];
    if (base < 0) return;
    const int total = (L + 1) * nh << shift;
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
#pragma unroll 1
    for (int e0 = tid; e0 < total; e0 += kThreads * kInFlight) {
        u32x4 kv[kInFlight], vv[kInFlight];
        if (e0 != tid) place(e0);
#pragma unroll
        for (int u = 0; u < kInFlight; ++u)
            if (e0 + u * kThreads < total) {
                const size_t src = (((size_t)b * c.N + s_msg[2 + row[u]]) * c.Hkv + head[u]) * c.row_bytes + v16;
                kv[u] = *(const u32x4*)((const char*)c.k_tree + src);
                vv[u] = *(const u32x4*)((const char*)c.v_tree + src);
            }
#pragma unroll
        for (int u = 0; u < kInFlight; ++u)
            if (e0 + u * kThreads < total) {
                const size_t dst = (((size_t)b * c.Hkv + head[u]) * c.S_cap + (size_t)(base + row[u])) * c.row_bytes + v16;
                *(u32x4*)((char*)c.k_cache + dst) = kv[u];
                *(u32x4*)((char*)c.v_cache + dst) = vv[u];
            }
    }
}

// Whether some attention workgroup of this launch has not read the lengths yet, which are about to change, and does not come to
// it in time.  This thread's share of them.
__device__ __forceinline__ bool lens_unread(const StepArgs& x, int b, long long started) {
    bool unread = false;
    for (int w = threadIdx.x; w < x.attn_wgs; w += kThreads) {
        told::At p{x.lens + (size_t)b * x.attn_wgs + w};
        bool here = told::take(p, x.tag);
        while (!here) {
            if ((long long)wall_clock64() - started >= x.copy_ticks / 2) { here = told::give_up(p, x.tag); break; }
            __builtin_amdgcn_s_sleep(4);
            here = told::take(p, x.tag);
        }
        unread = unread || !here;
    }
    return unread;
}

// The path step for sequence b, run by all kThreads threads of one workgroup (thread i = node i).  Everything that the tree alone
// decides (each node's ancestors, as a bit set; its depth) is found before the scan's records are there; behind them there is a
// ballot, a maximum over the accepted nodes, and the path's nodes are the deepest one's bit set in ascending order, all written at once.
// (From the records to the message: 4.5 us with a walk up the tree per node and one down the path, and the lengths' words looked at in between.)
template <typename T, Part PART>
__device__ __forceinline__ void path_step(const AcceptArgs& a, const StepArgs& x, Shared& sh, int b) {
    Rows& rows = sh.rows;
    const long long started = (long long)wall_clock64(), deadline = started + a.wait_ticks;
    const int i = threadIdx.x;
    const int N = a.N;
    const int base = PART != kAlone ? x.compact.cache_len[b] : 0;

    // ---- everything node i needs that does not depend on another load is requested up front (the
    // step is a chain of dependent memory latencies, not of work)
    int bad = 0;
    int tok = -1, par_i = -1;
    float u_i = 0.f, pd_i = 0.f;
    if (i < N) {
        const int p = par_i = a.parent[(size_t)b * N + i];
        tok = a.tokens[(size_t)b * N + i];
        if (a.mode == S4C_STOCHASTIC && i > 0) {
            u_i = a.uniforms[(size_t)b * N + i];
            pd_i = a.p_draft[(size_t)b * N + i];
        }
        // tree validation: node 0 is the only root, parents precede children
        sh.parent[i] = p;
        bad = (i == 0) ? (p != -1) : (p < 0 || p >= i);
    }
    // the target logit of this node's token in its parent's row (needs only parent and token)
    float lx = 0.f;
    if (a.mode == S4C_STOCHASTIC && i > 0 && i < N && !bad && tok >= 0 && tok < a.V)
        lx = to_f32<T>(((const T*)a.logits)[((size_t)b * N + par_i) * a.V + tok]);
    const int n_rows = find_rows(a, b, rows);
    if (i == 0) sh.best = 0;
    bad = any_of(sh, bad);
    uint64_t lo = 0, hi = 0;                                   // this node and its ancestors
    int depth = 0;
    if (!bad && i < N) {
        for (int j = i; j >= 0; j = sh.parent[j]) {
            if (j < 64) lo |= 1ull << j; else hi |= 1ull << (j - 64);
            ++depth;
        }
        --depth;
        sh.above[i][0] = lo;
        sh.above[i][1] = hi;
    }
    bool unread = false;
    if constexpr (PART == kBesideAttention) unread = lens_unread(x, b, started);
    const bool too_deep = any_of(sh, depth >= a.max_path);
    if constexpr (PART == kBesideAttention) unread = any_of(sh, unread);
    bad = bad || too_deep;

    // ---- combine the statistics of row i's runs.  In stochastic mode only the rows of nodes with
    // children were scanned, and only those are combined (nothing reads a leaf's statistics: a node
    // is tested against its PARENT's row, and that mode has no bonus token).
    float m = -INFINITY, S = 0.f;
    int32_t g = 0x7FFFFFFF;
    int late = 0;
    const Runs runs(a, n_rows);
    const int rank = i < N ? rows.rank[i] : -1;      // (of a malformed tree too: every record of the call is consumed)
    rec_t* const r = a.rec + ((size_t)b * N + i) * a.plan.slots * 2;
    const int parts = rank < 0 ? 0 : runs.of_chunk(rank * a.chunks + a.chunks - 1) - runs.of_chunk(rank * a.chunks) + 1;
    if (rank >= 0) {
        for (int c0 = 0; c0 < parts && !late; c0 += 4) {
            uint32_t bits[8];
            if (!await4(r + 2 * c0, min(4, parts - c0), a.nonce, deadline, bits)) { late = 1; break; }
            if (a.mode == S4C_GREEDY) {                        // runs ascend: strict '>' keeps the lowest index
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    const float v = __uint_as_float(bits[2 * s]);
                    if (c0 + s < parts && v > m) { m = v; g = (int32_t)bits[2 * s + 1]; }
                }
            } else {
                float mn = m;
#pragma unroll
                for (int s = 0; s < 4; ++s)
                    if (c0 + s < parts) mn = fmaxf(mn, __uint_as_float(bits[2 * s]));
                if (m > -INFINITY) S *= fast_exp2((m - mn) * a.inv_temp_log2);
                m = mn;
#pragma unroll
                for (int s = 0; s < 4; ++s)
                    if (c0 + s < parts && __uint_as_float(bits[2 * s]) > -INFINITY)
                        S += __uint_as_float(bits[2 * s + 1]) * fast_exp2((__uint_as_float(bits[2 * s]) - m) * a.inv_temp_log2);
            }
        }
    }
    // consumed: a replay of this very call (same nonce) must not mistake them for its own
    auto spend = [&]() __attribute__((always_inline)) {
        if (rank >= 0 && !late)
            for (int c = 0; c < 2 * parts; ++c) publish(r + c, ~a.nonce, 0u);
    };
    if (i < N) { sh.g[i] = g; sh.m[i] = m; sh.S[i] = S; }
    const bool some_late = any_of(sh, late);
    int32_t* pth = a.path + (size_t)b * a.max_path;
    int32_t* atk = a.accepted_tokens + (size_t)b * a.max_path;
    if (some_late || bad) {
        for (int k = i; k < a.max_path; k += kThreads) { pth[k] = (k == 0) ? 0 : -1; atk[k] = -1; }
        if (i == 0) {
            a.accept_len[b] = 0;
            a.bonus_token[b] = -1;
            if (a.status) a.status[b] = some_late ? S4C_SEQ_TIMEOUT : S4C_SEQ_BAD_TREE;
            sh.node[0] = sh.len = 0;
        }
        if constexpr (PART != kAlone) {
            __syncthreads();
            announce_path(x, a, sh, b, base, unread);
        }
        spend();
        if constexpr (PART != kAlone) look_for_leavers(x, a, sh, b, base);
        return;
    }
    // ---- local test of node i against its parent's row
    bool ok = i < N;
    if (ok && i > 0) {
        if (a.mode == S4C_GREEDY) {
            ok = tok == sh.g[par_i];
        } else if (tok < 0 || tok >= a.V) {
            ok = false;
        } else {
            const float pt = fast_exp2((lx - sh.m[par_i]) * a.inv_temp_log2) / sh.S[par_i];
            ok = u_i * pd_i < pt;
        }
    }
    const uint64_t passed = __ballot(ok);
    if (i < 128 && (i & 63) == 0) sh.ok[i >> 6] = passed;
    __syncthreads();
    // deepest accepted node, lowest index among equals: maximise depth*256 + (255 - i)
    if (i < N && !(lo & ~sh.ok[0]) && !(hi & ~sh.ok[1])) atomicMax(&sh.best, depth * 256 + (255 - i));
    __syncthreads();
    const int best = 255 - (sh.best & 255), L = sh.best >> 8;
    const uint64_t path_lo = sh.above[best][0], path_hi = sh.above[best][1];
    const bool on_path = i < N && (((i < 64 ? path_lo : path_hi) >> (i & 63)) & 1);
    if (on_path) {                                             // its ancestors have lower numbers: it is node `depth` of the path
        pth[depth] = i;
        if (depth > 0) atk[depth - 1] = tok;
        if constexpr (PART != kAlone) sh.node[depth] = i;
    }
    if (i == best) {
        if constexpr (PART != kAlone) sh.len = L;
        a.accept_len[b] = L;
        a.bonus_token[b] = (a.mode == S4C_GREEDY) ? g : -1;
        if (a.status) a.status[b] = 0;
    }
    if constexpr (PART != kAlone) {
        __syncthreads();
        announce_path(x, a, sh, b, base, unread);
    }
    for (int k = i; k < a.max_path; k += kThreads) {
        if (k > L) pth[k] = -1;
        if (k >= L) atk[k] = -1;
    }
    spend();
    if constexpr (PART != kAlone) look_for_leavers(x, a, sh, b, base);
}

// one workgroup of the scan: run j of sequence b.  AHEAD chunks are in flight behind the one that is reduced.
template <typename T, bool STOCHASTIC, int AHEAD>
__device__ __forceinline__ void scan_run(const AcceptArgs& a, Shared& sh, int b, int j) {
    constexpr int VN = RowReader<T>::VN, NV = RowReader<T>::NV;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    Rows& rows = sh.rows;
    const int n_rows = find_rows(a, b, rows);
    const Runs runs(a, n_rows);
    if (n_rows == 0 || j >= runs.used) return;
    const int c_end = runs.begin(j + 1);
    int c = runs.begin(j), rank = c / a.chunks, ch = c - rank * a.chunks;
    const size_t row0 = (size_t)b * a.N;
    // the chunks to come, of this row or of the next ones
    uint4 raw[AHEAD][NV];
    int p_left = c_end - c, p_rank = rank, p_ch = ch;
    RowReader<T> p_reader(a.logits, row0 + rows.list[rank], a.V);
    auto fetch = [&](uint4 (&to)[NV]) __attribute__((always_inline)) {
        if (p_left == 0) return;
        if (p_ch == a.chunks) {
            p_ch = 0;
            p_reader = RowReader<T>(a.logits, row0 + rows.list[++p_rank], a.V);
        }
        p_reader.fetch(p_ch++, to);
        --p_left;
    };
#pragma unroll
    for (int d = 0; d < AHEAD; ++d) fetch(raw[d]);
    while (c < c_end) {
        const int node = rows.list[rank], last = min(a.chunks, ch + c_end - c);       // this row's chunks ch .. last - 1
        float m_t = -INFINITY, s_t = 0.f;               // greedy: maximum; stochastic: reference and sum
        uint4 wbest[NV];
        int32_t cbest = 0;
        if constexpr (!STOCHASTIC) {
#pragma unroll
            for (int q = 0; q < NV; ++q) wbest[q] = make_uint4(0, 0, 0, 0);
        }
        const RowReader<T> here(a.logits, row0 + node, a.V);
        for (; ch < last; ++ch, ++c) {
            uint4 cur[NV];
#pragma unroll
            for (int q = 0; q < NV; ++q) cur[q] = raw[0][q];
#pragma unroll
            for (int d = 0; d + 1 < AHEAD; ++d)
#pragma unroll
                for (int q = 0; q < NV; ++q) raw[d][q] = raw[d + 1][q];
            fetch(raw[AHEAD - 1]);
            float m_c = -INFINITY;
#pragma unroll
            for (int q = 0; q < NV; ++q) {
                float x[VN];
                decode<T>(cur[q], x);
#pragma unroll
                for (int e = 0; e < VN; e += 2) m_c = __builtin_fmaxf(__builtin_fmaxf(m_c, x[e]), x[e + 1]);
            }
            if constexpr (!STOCHASTIC) {
                if (m_c > m_t) {                        // strict: an equal later chunk never replaces an earlier one
                    m_t = m_c;
                    cbest = ch;
#pragma unroll
                    for (int q = 0; q < NV; ++q) wbest[q] = cur[q];
                }
            } else {
                if ((m_c - m_t) * a.inv_temp_log2 > kLazyLog2) {               // (m_t = -inf: the first logit that is not padding)
                    s_t *= fast_exp2((m_t - m_c) * a.inv_temp_log2);
                    m_t = m_c;
                }
                const float ref = m_t > -INFINITY ? m_t * a.inv_temp_log2 : 0.f;
                float sum[2] = {0.f, 0.f};
                // (a reference beyond the range of fp32: rows masked with the type's lowest value, for one)
                const bool in_range = fabsf(ref) <= 3.0e38f;
#pragma unroll
                for (int q = 0; q < NV; ++q) {
                    float x[VN];
                    decode<T>(cur[q], x);
                    if (in_range) {
#pragma unroll
                        for (int e = 0; e < VN; ++e) sum[e & 1] += fast_exp2(fmaf(x[e], a.inv_temp_log2, -ref));   // padding: 0
                    } else {
#pragma unroll
                        for (int e = 0; e < VN; ++e) sum[e & 1] += fast_exp2((x[e] - m_t) * a.inv_temp_log2);
                    }
                }
                s_t += sum[0] + sum[1];
            }
        }
        // ---- the row's part is done: combine the 256 threads
        float out_v;
        uint32_t out_w;
        if constexpr (STOCHASTIC) {
            const float mw = wave_max(m_t);
            float sw = m_t > -INFINITY ? s_t * fast_exp2((m_t - mw) * a.inv_temp_log2) : 0.f;
            sw = wave_sum(sw);
            if (lane == 0) { sh.v[wave] = mw; sh.s[wave] = sw; }
            __syncthreads();
            out_v = fmaxf(fmaxf(sh.v[0], sh.v[1]), fmaxf(sh.v[2], sh.v[3]));
            float t = 0.f;
#pragma unroll
            for (int w = 0; w < 4; ++w)
                if (sh.v[w] > -INFINITY) t += sh.s[w] * fast_exp2((sh.v[w] - out_v) * a.inv_temp_log2);
            out_w = __float_as_uint(t);
        } else {
            // the thread's argmax: lowest index among its elements equal to its maximum (scan descending,
            // so that the lowest match is written last)
            MaxIdx best = {m_t, 0x7FFFFFFF};
            if (m_t > -INFINITY) {                      // (a thread of a ragged chunk may hold padding only)
#pragma unroll
                for (int q = NV - 1; q >= 0; --q) {
                    float x[VN];
                    decode<T>(wbest[q], x);
#pragma unroll
                    for (int e = VN - 1; e >= 0; --e)
                        if (x[e] == m_t) best.i = here.idx(cbest, q) + e;
                }
            }
            const MaxIdx wb = wave_best(best);
            if (lane == 0) { sh.v[wave] = wb.v; sh.i[wave] = wb.i; }
            __syncthreads();
            MaxIdx blk = {sh.v[0], sh.i[0]};
#pragma unroll
            for (int w = 1; w < 4; ++w) blk = better(blk, MaxIdx{sh.v[w], sh.i[w]});
            out_v = blk.v;
            out_w = (uint32_t)blk.i;
        }
        if (tid == 0) {
            rec_t* r = a.rec + ((row0 + node) * a.plan.slots + (j - runs.of_chunk(rank * a.chunks))) * 2;
            publish(r, a.nonce, __float_as_uint(out_v));
            publish(r + 1, a.nonce, out_w);
        }
        __syncthreads();                                // sh.v, sh.i, sh.s are written again for the next row
        ++rank;
        ch = 0;
    }
}

// Workgroup wg of the scan: the runs of all sequences (run number slowest, so that the ones without work are the last of
// the grid rather than interleaved with the working ones), then the sequences' collectors.
template <typename T, bool STOCHASTIC, Part PART, int AHEAD>
__device__ __forceinline__ void scan_or_collect(const AcceptArgs& a, const StepArgs& x, Shared& sh, int wg) {
    const int j = wg / a.B, b = wg - j * a.B;
    if (j < a.plan.wgs) scan_run<T, STOCHASTIC, AHEAD>(a, sh, b, j);
    else path_step<T, PART>(a, x, sh, b);
}

// (without a merge)
inline StepArgs make_step(const AcceptArgs& a, const CompactArgs& compact, rec_t* messages, long long copy_ticks) {
    StepArgs x;
    x.compact = compact;
    x.messages = messages;
    x.lens = nullptr;
    x.attn_wgs = 0;
    x.tag = 0;
    x.copy_ticks = copy_ticks;
    x.merge_wgs = 0;
    x.merge_chunks = x.merge_passes = 1;
    x.scan_wgs = (a.plan.wgs + 1) * a.B;
    x.heads = (compact.Hkv + kMostCopiers - 1) / kMostCopiers;
    x.copiers = (compact.Hkv + x.heads - 1) / x.heads;
    return x;
}

}  // namespace accept
}  // namespace s4c

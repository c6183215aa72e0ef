// Candidate-tree construction from the drafter's logits (paper Sec. 3.2: the top-1 continuation
// is drafted first, the next most probable tokens are placed beside it as alternatives).
//
// Kernel 1 (topk_chunk): the HBM-bound part, over the rows that have children; a workgroup walks a
// segment of consecutive 8192-logit chunks of one row, the next chunk in flight while the current
// one is searched.  Every wavefront keeps the nchild[row] largest logits of its quarter of the
// segment as a running sorted list (a chunk is only searched where a vote finds something above the
// list's last entry; ties to the lowest token id) and writes the list out at the end, next to the
// maximum and the sum of exponentials of its part: no barrier, no workgroup-level step, no
// cross-lane step per chunk unless the list changes.
// Kernel 2 (topk_row): one wavefront per row finds from the sequence's child counts which numbers its children have
// (level by level: a prefix sum), whether the counts describe a tree of exactly N nodes, merges the parts' candidates into the
// row's top nchild tokens, turns their logits into probabilities, and writes its children.  The numbering needs 128
// words that are requested with everything else, so doing it once per row costs less than a launch of its own did.
// HBM bounds kernel 1; kernel 2 is a chain of two memory latencies.
#include "build_plan.h"
#include "row_chunk.h"

namespace s4c {

namespace {

using namespace rowchunk;
constexpr int kK = 8;                 // most children per node

template <typename T, bool ALIGNED>
__global__ __launch_bounds__(kThreads) void topk_chunk_kernel(BuildArgs a) {
    constexpr int VN = Vec16<T>::n;
    constexpr int NV = kPerThread / VN;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int N = a.N;
    // workgroup -> (rank k among the sequence's rows that have children, sequence b, segment sg of consecutive
    // chunks), k slowest, so that the workgroups of rows without children are the last of the grid instead of
    // being interleaved
    const int sg = blockIdx.x % a.nseg;
    const int b = (blockIdx.x / a.nseg) % a.B;
    const int k = blockIdx.x / (a.nseg * a.B);
    __shared__ int32_t s_row, s_cnt0;
    const int my_nc = (tid < N) ? a.nchild[(size_t)b * N + tid] : 0;
    const int has = my_nc > 0 && my_nc <= a.kmax;       // (an invalid count is flagged by the row kernel)
    const unsigned long long mask = __ballot(has);
    if (tid == 0) { s_cnt0 = __popcll(mask); s_row = -1; }
    __syncthreads();
    if (wave < 2 && has) {
        const int rank = __popcll(mask & ((1ull << lane) - 1ull)) + (wave == 1 ? s_cnt0 : 0);
        if (rank == k) s_row = tid;
    }
    __syncthreads();
    if (s_row < 0) return;
    const int row = b * N + s_row;
    const int nc = a.nchild[row];
    const int V = a.V;
    const RowReader<T> reader(a.logits, row, V);
    const T* base = (const T*)a.logits + (size_t)row * V;
    const int ch0 = sg * a.seg, ch1 = min(a.chunks, ch0 + a.seg);

    // chunks are fetched one ahead as raw 16-byte words (ALIGNED: whole chunks; a row's last one is read in place)
    uint4 raw[NV];
    auto ahead = [&](int c) { return c < ch1 && (!ALIGNED || (c + 1) * kChunk <= V); };
    auto fetch = [&](int c) {
        if constexpr (ALIGNED) {
#pragma unroll
            for (int j = 0; j < NV; ++j) raw[j] = *(const uint4*)(base + c * kChunk + (j * kThreads + tid) * VN);
        } else {
            reader.fetch(c, raw);
        }
    };
    bool have = ahead(ch0);
    if (have) fetch(ch0);
    float m_e = -INFINITY, s_e = 0.f;                  // this thread's running maximum and sum of exponentials
    float lv[kK];                                      // the wavefront's list (uniform across lanes)
    int32_t li[kK];
#pragma unroll
    for (int e = 0; e < kK; ++e) { lv[e] = (e >= kK - nc) ? -INFINITY : INFINITY; li[e] = -1; }
  for (int ch = ch0; ch < ch1; ++ch) {
    float x[kPerThread];
    int32_t idx0[NV];
    if (!ALIGNED || have) {
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            idx0[j] = ALIGNED ? ch * kChunk + (j * kThreads + tid) * VN : reader.idx(ch, j);
            float v[VN];
            decode<T>(raw[j], v);
#pragma unroll
            for (int q = 0; q < VN; ++q) x[j * VN + q] = v[q];
        }
    } else {
        load_chunk<T>(base, ch * kChunk, min(V, (ch + 1) * kChunk), tid, x, idx0);
    }
    have = ahead(ch + 1);
    if (have) fetch(ch + 1);                           // in flight while this chunk is searched

    // this thread's share of the sum of exponentials, relative to its own running maximum (rescaled when that
    // grows): no cross-lane step per chunk
    float m_c = x[0];
#pragma unroll
    for (int e = 1; e < kPerThread; e += 2) m_c = __builtin_fmaxf(__builtin_fmaxf(m_c, x[e]), x[(e + 1) & (kPerThread - 1)]);
    if (m_c > -INFINITY) {
        const float m_new = fmaxf(m_e, m_c);
        float sum = 0.f;
#pragma unroll
        for (int e = 0; e < kPerThread; ++e) sum += fast_exp2((x[e] - m_new) * a.inv_temp_log2);   // padding: 0
        s_e = s_e * fast_exp2((m_e - m_new) * a.inv_temp_log2) + sum;                              // first chunk: 0 * 0
        m_e = m_new;
    }

    // Selection.  The wavefront keeps the nc largest logits it has seen in the segment so far as a sorted list
    // (value descending, token id ascending), the same in every lane.  A chunk can only change the list where a
    // lane holds something larger than the list's last entry, which a vote tells without any cross-lane data
    // movement; after the segment's first chunk most chunks pass with few or no insertions.  An insertion is a
    // wavefront maximum of the lanes' largest remaining logits, a lookup of the lowest token id that attains it
    // (ties to the lowest id), a shift of the list, and the owner retiring the element.
    float m_t = m_c;
    for (int r = 0; r < nc; ++r) {                       // at most nc entries of one chunk can enter
        const float tau = lv[kK - 1];                    // the list's last entry of the nc kept (see the shift below)
        if (!__any(m_t > tau)) break;                    // (an equal later logit has a higher token id: it stays out)
        float wm = m_t;
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) wm = fmaxf(wm, __shfl_xor(wm, off));
        int32_t mine = 0x7FFFFFFF;                       // lowest token id of this lane that attains the wave maximum
        if (m_t == wm) {
#pragma unroll
            for (int j = NV - 1; j >= 0; --j)
#pragma unroll
                for (int q = VN - 1; q >= 0; --q)
                    if (x[j * VN + q] == wm) mine = idx0[j] + q;
        }
        int32_t win = mine;
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) win = min(win, __shfl_xor(win, off));
        // insert (wm, win): entries are kept in slots kK - nc .. kK - 1, so that the last kept entry sits in
        // slot kK - 1 whatever nc is; everything smaller than the newcomer moves one slot down and the last drops
        // out.  Tokens of later chunks have higher ids, so the newcomer goes behind entries of equal value.
#pragma unroll
        for (int e = kK - 1; e >= 1; --e) {
            const bool moves = lv[e - 1] < wm;           // slot e takes slot e-1's entry
            const bool lands = !moves && lv[e] < wm;     // slot e takes the newcomer
            if (moves) { lv[e] = lv[e - 1]; li[e] = li[e - 1]; }
            else if (lands) { lv[e] = wm; li[e] = win; }
        }
        if (lv[0] < wm) { lv[0] = wm; li[0] = win; }
        if (mine == win) {                               // the owner removes the winner
#pragma unroll
            for (int j = 0; j < NV; ++j)
#pragma unroll
                for (int q = 0; q < VN; ++q)
                    if (idx0[j] + q == win) x[j * VN + q] = -INFINITY;
            m_t = x[0];
#pragma unroll
            for (int e = 1; e < kPerThread; e += 2) m_t = __builtin_fmaxf(__builtin_fmaxf(m_t, x[e]), x[(e + 1) & (kPerThread - 1)]);
        }
    }
  }
    // ---- the wavefront's part of the segment: maximum, sum of exponentials against it, and its list
    float wm = m_e;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) wm = fmaxf(wm, __shfl_xor(wm, off));
    float sum = (m_e > -INFINITY) ? s_e * fast_exp2((m_e - wm) * a.inv_temp_log2) : 0.f;
    sum = wave_sum(sum);
    const size_t o = ((size_t)row * a.nseg + sg) * 4 + wave;
    if (lane == 0) { a.ws_max[o] = wm; a.ws_sum[o] = sum; }
    if (lane < nc) {
        // entry r of the list sits in slot kK - nc + r; a slot that was never filled holds -inf / -1 ("part exhausted")
        float v = -INFINITY;
        int32_t t = -1;
#pragma unroll
        for (int e = 0; e < kK; ++e)
            if (e == kK - nc + lane) { v = lv[e]; t = li[e]; }
        a.ws_topv[o * kK + lane] = v;
        a.ws_topi[o * kK + lane] = t;
    }
}

__global__ __launch_bounds__(64) void topk_row_kernel(BuildArgs a) {
    const int row = blockIdx.x, lane = threadIdx.x, N = a.N;
    const int b = row / N, i = row - b * N;
    const int parts = a.nseg * 4;                            // a wavefront's quarter of a segment of chunks each
    const size_t o = (size_t)row * parts;
    // the sequence's child counts, this lane's part statistics and (few parts) its whole list are requested together: the
    // kernel is a chain of memory latencies, not of work
    const bool few = parts <= kBuildListsInRegisters, mine = lane < parts;
    const int32_t* counts = a.nchild + (size_t)b * N;
    const int c0 = lane < N ? counts[lane] : 0, c1 = lane + 64 < N ? counts[lane + 64] : 0;
    const int32_t root = i == 0 ? a.root_token[b] : -1;
    const float pm0 = (few && mine) ? a.ws_max[o + lane] : -INFINITY;
    const float ps0 = (few && mine) ? a.ws_sum[o + lane] : 0.f;
    float v[kK];
    int32_t t[kK];
#pragma unroll
    for (int e = 0; e < kK; ++e) {
        v[e] = (few && mine) ? a.ws_topv[(o + lane) * kK + e] : -INFINITY;      // (slots beyond nc hold leftovers: masked below)
        t[e] = (few && mine) ? a.ws_topi[(o + lane) * kK + e] : -1;
    }
    // ---- numbering: lane l holds the counts of nodes l and l + 64 and their inclusive sums (s0, s1)
    const bool ok0 = c0 >= 0 && c0 <= a.kmax, ok1 = c1 >= 0 && c1 <= a.kmax;
    int s0 = ok0 ? c0 : 0, s1 = ok1 ? c1 : 0;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int y0 = __shfl_up(s0, off), y1 = __shfl_up(s1, off);
        if (lane >= off) { s0 += y0; s1 += y1; }
    }
    s1 += __builtin_amdgcn_readlane(s0, 63);
    auto handed = [&](int n) { return n < 64 ? __builtin_amdgcn_readlane(s0, n) : __builtin_amdgcn_readlane(s1, n - 64); };  // by nodes 0 .. n
    // an invalid count, a node that would be a parent before it exists, or not exactly N nodes
    const bool early = (lane >= 1 && lane < N && s0 - c0 < lane) || (lane + 64 < N && s1 - c1 < lane + 64);
    const bool bad = __any(!ok0 || !ok1 || early) || handed(N - 1) != N - 1;
    if (lane == 0 && (i == 0 || bad)) {                      // the root, or any node of what is no tree
        a.parent[row] = -1;
        a.tokens[row] = root;
        a.p_draft[row] = 0.f;
        if (a.level) a.level[row] = 0;
        if (i == 0 && a.status) a.status[b] = bad ? S4C_SEQ_BAD_TREE : 0;
    }
    if (bad) return;
    const int first = 1 + (i > 0 ? handed(i - 1) : 0), nc = 1 + handed(i) - first;
    if (nc == 0) return;
    int lev = 1;                                             // the children's level: levels end where the previous one's children do
    for (int end = 1; end <= i; end = 1 + handed(end - 1)) ++lev;     // (grows every time: node `end` has a parent before it)
    // row maximum and sum of exponentials from the parts' statistics
    float m = pm0;
    if (!few)
        for (int c = lane; c < parts; c += 64) m = fmaxf(m, a.ws_max[o + c]);
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));
    float S = 0.f;
    if (few) {
        if (pm0 > -INFINITY) S = ps0 * fast_exp2((pm0 - m) * a.inv_temp_log2);
    } else {
        for (int c = lane; c < parts; c += 64) {
            const float pm = a.ws_max[o + c];
            if (pm > -INFINITY) S += a.ws_sum[o + c] * fast_exp2((pm - m) * a.inv_temp_log2);    // (a part beyond V is all padding)
        }
    }
    S = wave_sum(S);
    const float* cv = a.ws_topv + o * kK;
    const int32_t* ci = a.ws_topi + o * kK;
    auto emit = [&](int r, MaxIdx best) {
        if (lane == 0) {
            const bool found = best.i != 0x7FFFFFFF;
            const size_t c = (size_t)b * N + first + r;
            a.parent[c] = i;
            a.tokens[c] = found ? best.i : -1;
            a.p_draft[c] = found ? fast_exp2((best.v - m) * a.inv_temp_log2) / S : 0.f;
            if (a.level) a.level[c] = lev;
        }
    };
    if (few) {
        // Every part's candidates are a descending list of nc entries: lane p keeps part p's list in
        // registers (read once), offers its head in every round, and the lane that wins shifts its list.
#pragma unroll
        for (int e = 0; e < kK; ++e)
            if (e >= nc) { v[e] = -INFINITY; t[e] = -1; }
        for (int r = 0; r < nc; ++r) {
            const MaxIdx head = (t[0] >= 0) ? MaxIdx{v[0], t[0]} : MaxIdx{-INFINITY, 0x7FFFFFFF};
            const MaxIdx best = wave_best(head);
            emit(r, best);
            if (head.i == best.i && best.i != 0x7FFFFFFF) {          // candidates are distinct tokens: one lane matches
#pragma unroll
                for (int e = 0; e + 1 < kK; ++e) { v[e] = v[e + 1]; t[e] = t[e + 1]; }
                v[kK - 1] = -INFINITY;
                t[kK - 1] = -1;
            }
        }
        return;
    }
    // more than 64 parts (rows beyond 1048576 logits): nc rounds of "largest remaining candidate" over the lists in
    // memory; a lane owns candidates lane, lane+64, ...
    const int ncand = parts * kK;
    MaxIdx prev = {INFINITY, -1};                         // the winner of the previous round
    for (int r = 0; r < nc; ++r) {
        // candidates are distinct tokens, so "remaining" = strictly after the previous winner
        // in the order (value descending, token id ascending)
        MaxIdx best = {-INFINITY, 0x7FFFFFFF};
        for (int c = lane; c < ncand; c += 64) {
            const MaxIdx cand = {cv[c], ci[c]};
            if (c % kK >= nc || cand.i < 0) continue;       // slots beyond nc were not written
            const bool after = (cand.v < prev.v) || (cand.v == prev.v && cand.i > prev.i);
            if (after) best = better(best, cand);
        }
        best = wave_best(best);
        emit(r, best);
        prev = best;
        if (best.i == 0x7FFFFFFF) prev = MaxIdx{-INFINITY, 0x7FFFFFFF};   // nothing left: later rounds find nothing
    }
}

}  // namespace

int build_tree_max_children() { return kK; }
int build_tree_chunk_elems() { return kChunk; }

void build_tree_plan(BuildArgs& a) {
    a.seg = build_segment((long long)a.B * a.N, a.chunks);
    a.nseg = (a.chunks + a.seg - 1) / a.seg;
}

// Rows on 16-byte boundaries are read in plain chunks, others through RowReader.  Read through RowReader too, 335 MB of
// aligned bf16 rows take 88 us instead of 82; rows of odd length read two bytes at a time, as the plain chunks would be,
// 71.4 us instead of 43.6 (103 MB).
template <typename T>
static void launch_topk(const BuildArgs& a, hipStream_t st) {
    const dim3 grid((unsigned)((size_t)a.B * a.N * a.nseg));
    if (a.V % Vec16<T>::n == 0 && (((uintptr_t)a.logits) & 15) == 0)
        hipLaunchKernelGGL((topk_chunk_kernel<T, true>), grid, dim3(kThreads), 0, st, a);
    else
        hipLaunchKernelGGL((topk_chunk_kernel<T, false>), grid, dim3(kThreads), 0, st, a);
}

hipError_t launch_build_tree(const BuildArgs& a, hipStream_t st) {
    if (a.dtype == S4C_F32) launch_topk<float>(a, st);
    else if (a.dtype == S4C_F16) launch_topk<f16_t>(a, st);
    else launch_topk<bf16_t>(a, st);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(topk_row_kernel, dim3((unsigned)(a.B * a.N)), dim3(64), 0, st, a);
    return hipGetLastError();
}

}  // namespace s4c

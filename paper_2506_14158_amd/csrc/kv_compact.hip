// KV reuse (paper Sec. 3.2, last paragraph): append the accepted path's K/V rows to the cache.
//
// One workgroup per sequence (and layer): the path is read from device memory (no host round trip), all
// (path position, KV head) rows are copied with 16-byte accesses, and cache_len is bumped by
// the same workgroup after its copies were issued.  Moves at most max_path * Hkv * D * 2 rows of
// bytes per sequence, so the step is a chain of latencies: the path and the length, then the rows and the pages they go to
// (requested together, before either has been checked: a node is clamped to the tree, a page only used once every one is
// known to be the pool's), then the stores.
#include "common.h"

namespace s4c {

namespace {

constexpr int kThreads = 1024;
constexpr int kBatch = 4;       // independent 16-byte copies in flight per thread (x2: K and V)
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));      // (arrays of HIP's uint4 went through scratch memory here)

// Where the rows of a path come from and go to.
struct Rows {
    const char *k_tree, *v_tree;
    char *k_cache, *v_cache;
    const int32_t* table;          // the sequence's pages, null: contiguous
    int b, N, Hkv, S_cap, row_bytes, page_shift, num_pages;
};

// Appends the rows of the path's L + 1 nodes (s_path, then pth beyond kMaxNodes) behind `base` rows, which fit; false, and
// nothing written, if a node or a page is not valid.  All threads.
__device__ __forceinline__ bool append_rows(const Rows& r, const int32_t* s_path, const int32_t* pth, int base, int L) {
    const int tid = threadIdx.x, vpr = r.row_bytes / 16, total = (L + 1) * r.Hkv * vpr;
    auto node_at = [&](int k) { return k < kMaxNodes ? s_path[k] : pth[k]; };
    u32x4 kv[kBatch], vv[kBatch];
    size_t dst[kBatch];
    auto fetch = [&](int e0) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const int e = e0 + u * kThreads;
            if (e < total) {
                const int q = e / vpr, v = e - q * vpr, k = q / r.Hkv, h = q - k * r.Hkv, j = base + k;
                const int node = min(max(node_at(k), 0), r.N - 1);
                const size_t src = (((size_t)r.b * r.N + node) * r.Hkv + h) * r.row_bytes + (size_t)v * 16;
                kv[u] = *(const u32x4*)(r.k_tree + src);
                vv[u] = *(const u32x4*)(r.v_tree + src);
                size_t drow = ((size_t)r.b * r.Hkv + h) * r.S_cap + (size_t)j;
                if (r.table) drow = (((size_t)r.table[j >> r.page_shift] * r.Hkv + h) << r.page_shift) + (size_t)(j & ((1 << r.page_shift) - 1));
                dst[u] = drow * r.row_bytes + (size_t)v * 16;
            }
        }
    };
    fetch(tid);
    int bad = 0;
    for (int k = tid; k <= L; k += kThreads) {
        bad |= node_at(k) < 0 || node_at(k) >= r.N;
        if (r.table) {                             // the page of every written row must be a page of the pool
            const int id = r.table[(base + k) >> r.page_shift];
            bad |= id < 0 || id >= r.num_pages;
        }
    }
    if (__syncthreads_or(bad)) return false;
    for (int e0 = tid; e0 < total; e0 += kThreads * kBatch) {
        if (e0 != tid) fetch(e0);
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            if (e0 + u * kThreads < total) {
                *(u32x4*)(r.k_cache + dst[u]) = kv[u];
                *(u32x4*)(r.v_cache + dst[u]) = vv[u];
            }
        }
    }
    return true;
}

__global__ __launch_bounds__(kThreads) void kv_compact_kernel(CompactArgs a) {
    const int b = blockIdx.x, tid = threadIdx.x;
    const int32_t* pth = a.path + (size_t)b * a.max_path;
    // the three loads that everything else depends on go out together (path entries before the
    // accepted length is known; a real path has at most kMaxNodes nodes, longer ones are read in place)
    __shared__ int32_t s_path[kMaxNodes];
    const int L = a.accept_len[b];
    const int base = a.cache_len[b];
    if (tid < kMaxNodes) s_path[tid] = (tid < a.max_path) ? pth[tid] : -1;
    __syncthreads();                     // also orders every thread's read of cache_len before the bump
    const Rows rows = {(const char*)a.k_tree, (const char*)a.v_tree, (char*)a.k_cache, (char*)a.v_cache,
                       a.block_table ? a.block_table + (size_t)b * a.max_blocks : nullptr, b, a.N, a.Hkv, a.S_cap, a.row_bytes, a.page_shift, a.num_pages};
    const bool fits = L >= 0 && L < a.max_path && base >= 0 && (long long)base + L + 1 <= a.S_cap;
    const bool done = fits && append_rows(rows, s_path, pth, base, L);
    if (a.dst_index)
        for (int k = tid; k < a.max_path; k += kThreads)
            a.dst_index[(size_t)b * a.max_path + k] = (done && k <= L) ? base + k : -1;
    if (tid == 0) {
        if (a.status) a.status[b] = done ? 0 : S4C_SEQ_BAD_LEN;
        if (done) a.cache_len[b] = base + L + 1;
    }
}

// ---- all layers of a model (and the accepted nodes' feature rows) in one launch -------------
// grid (B, layers [+1]): workgroup (b, y) copies layer y's rows of sequence b; y == layers copies
// the feature rows.  No workgroup writes cache_len here -- all of a sequence's workgroups read it
// in no particular order -- a second one-thread-per-sequence kernel advances it afterwards.
__device__ __forceinline__ int commit_bad(const CommitArgs& a, int b, int tid, int nthreads) {
    const int L = a.accept_len[b];
    const int base = a.cache_len[b];
    const int32_t* pth = a.path + (size_t)b * a.max_path;
    int bad = (L < 0 || L >= a.max_path || base < 0 || (long long)base + L + 1 > a.S_cap);
    if (!bad)
        for (int k = tid; k <= L; k += nthreads) {
            bad |= (pth[k] < 0 || pth[k] >= a.N);
            if (a.block_table) {                       // the page of every written row must be a page of the pool
                const int id = a.block_table[(size_t)b * a.max_blocks + ((base + k) >> a.page_shift)];
                bad |= (id < 0 || id >= a.num_pages);
            }
        }
    return bad;
}

__global__ __launch_bounds__(kThreads) void commit_copy_kernel(CommitArgs a) {
    const int b = blockIdx.x, y = blockIdx.y, tid = threadIdx.x;
    const int32_t* pth = a.path + (size_t)b * a.max_path;
    __shared__ int32_t s_path[kMaxNodes];
    const int L = a.accept_len[b];
    const int base = a.cache_len[b];
    if (tid < kMaxNodes) s_path[tid] = (tid < a.max_path) ? pth[tid] : -1;
    __syncthreads();
    if (y == a.layers) {                                   // feature rows -> features_out[b][k]
        if (__syncthreads_or(commit_bad(a, b, tid, kThreads))) return;
        const int vpr = a.feature_bytes / 16;
        const int total = (L + 1) * vpr;
        for (int e = tid; e < total; e += kThreads) {
            const int k = e / vpr, v = e - k * vpr;
            const u32x4 x = *(const u32x4*)((const char*)a.features + ((size_t)b * a.N + pth[k]) * a.feature_bytes + (size_t)v * 16);
            *(u32x4*)((char*)a.features_out + ((size_t)b * a.max_path + k) * a.feature_bytes + (size_t)v * 16) = x;
        }
        return;
    }
    if (L < 0 || L >= a.max_path || base < 0 || (long long)base + L + 1 > a.S_cap) return;
    const Rows rows = {(const char*)a.k_tree + (size_t)y * a.tree_layer_bytes, (const char*)a.v_tree + (size_t)y * a.tree_layer_bytes,
                       (char*)a.k_cache + (size_t)y * a.cache_layer_bytes, (char*)a.v_cache + (size_t)y * a.cache_layer_bytes,
                       a.block_table ? a.block_table + (size_t)b * a.max_blocks : nullptr, b, a.N, a.Hkv, a.S_cap, a.row_bytes, a.page_shift, a.num_pages};
    append_rows(rows, s_path, pth, base, L);
}

// one thread per sequence: status, dst_index, and the single advance of cache_len
__global__ void commit_finish_kernel(CommitArgs a) {
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= a.B) return;
    const int bad = commit_bad(a, b, 0, 1);
    const int L = a.accept_len[b], base = a.cache_len[b];
    if (a.dst_index)
        for (int k = 0; k < a.max_path; ++k) a.dst_index[(size_t)b * a.max_path + k] = (!bad && k <= L) ? base + k : -1;
    if (a.status) a.status[b] = bad ? S4C_SEQ_BAD_LEN : 0;
    if (!bad) a.cache_len[b] = base + L + 1;
}

}  // namespace

hipError_t launch_commit(const CommitArgs& a, hipStream_t st) {
    const bool feats = a.features && a.features_out;
    hipLaunchKernelGGL(commit_copy_kernel, dim3(a.B, a.layers + (feats ? 1 : 0)), dim3(kThreads), 0, st, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(commit_finish_kernel, dim3((a.B + 255) / 256), dim3(256), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_compact(const CompactArgs& a, hipStream_t st) {
    hipLaunchKernelGGL(kv_compact_kernel, dim3(a.B), dim3(kThreads), 0, st, a);
    return hipGetLastError();
}

}  // namespace s4c

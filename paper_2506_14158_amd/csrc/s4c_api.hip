// C ABI of libs4c: argument checks, launch planning, kernel launches.  See include/s4c.h.
#include "attn_step.h"
#include "common.h"
#include "resample_plan.h"
#include "step_plan.h"

#include <math.h>
#include <stdlib.h>

#include <atomic>

using namespace s4c;

// Scratch of s4c_accept_path_static: one copy per GPU that loads the library, held until the process
// ends.  In host code this name is only a handle for hipGetSymbolAddress; the device address of each
// GPU's copy is looked up once per device (static_scratch) and that pointer is what kernels receive.
static __device__ __align__(256) unsigned char scratch[S4C_STATIC_SCRATCH_BYTES];

namespace {

constexpr int kMaxDevices = 64;

// Compute units of the current device (sizes the attention launch plan); the MI355X's 256 when no
// device can be asked (size queries on a host without a GPU).
int device_cus() {
    static std::atomic<int> cached[kMaxDevices];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return 256;
    int n = cached[dev].load(std::memory_order_relaxed);
    if (n <= 0) {
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
        cached[dev].store(n, std::memory_order_relaxed);
    }
    return n;
}

// Device address of the current GPU's copy of `scratch`.
hipError_t static_scratch(void** out) {
    static std::atomic<void*> addr[kMaxDevices];
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    void* p = addr[dev].load(std::memory_order_acquire);
    if (!p) {
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        addr[dev].store(p, std::memory_order_release);
    }
    *out = p;
    return hipSuccess;
}

bool aligned16(const void* p) { return (((uintptr_t)p) & 15) == 0; }

// A different number for every acceptance call of the process (the records of a workspace tell this
// call's statistics from older contents by it).  Never 0 or ~0: freshly allocated memory is often all
// zeros, which must read as "no record yet", and ~nonce marks a consumed record.
uint32_t next_nonce() {
    static std::atomic<uint32_t> counter{0};
    for (;;) {
        uint32_t x = counter.fetch_add(1, std::memory_order_relaxed) + 0x9E3779B9u;
        x ^= x >> 16; x *= 0x7FEB352Du; x ^= x >> 15; x *= 0x846CA68Bu; x ^= x >> 16;      // a bijection of 32-bit words
        if (x != 0u && x != 0xFFFFFFFFu) return x;
    }
}

// A different number for every attention call of the process, under which its workgroups' words count (attn_meet.h).  They lie where
// other calls keep numbers of any kind, so all bits are mixed: what is there is not taken for this call's.  Never 0.
uint64_t next_tag() {
    static std::atomic<uint64_t> counter{0};
    for (;;) {
        uint64_t x = counter.fetch_add(1, std::memory_order_relaxed) + 1;
        constexpr int half = 64 - __builtin_popcountll(meet::kStateBits);
        // a bijection of the words of that many bits: odd factors, and shifts to the right
        const uint64_t mask = (1ull << half) - 1;
        x = x * 0x9E3779B97F4A7C15ull & mask;
        x ^= x >> 30; x = x * 0xBF58476D1CE4E5B9ull & mask; x ^= x >> 27; x = x * 0x94D049BB133111EBull & mask; x ^= x >> 31;
        if (x != 0) return x << (64 - half);
    }
}

// A waiting time in microseconds, up to a minute, replaced by an environment variable (read at every call).
long long wait_us(const char* name, long long otherwise) {
    if (const char* env = getenv(name)) {
        char* end = nullptr;
        const long long v = strtoll(env, &end, 10);
        if (end != env && v >= 0 && v <= 60000000ll) return v;
    }
    return otherwise;
}

bool dtype_ok(int32_t d) { return d == S4C_F32 || d == S4C_BF16 || d == S4C_F16; }

bool shape_ok(const s4c_attn_shape* s, s4c_status* why) {
    if (s->B <= 0 || s->Hq <= 0 || s->Hkv <= 0 || s->D <= 0 || s->N <= 0 || s->S_cap < 0 ||
        s->Hq % s->Hkv != 0) {
        *why = S4C_ERR_SHAPE;
        return false;
    }
    if (s->N > kMaxNodes || (s->D != 64 && s->D != 128) || !dtype_ok(s->dtype) ||
        s->B > 65535 || s->Hkv > 65535) {
        *why = S4C_ERR_UNSUPPORTED;
        return false;
    }
    return true;
}

struct AttnPlan {
    bool large;                // more than 64 rows of 16-bit data: the kernel whose waves split the rows
    AttnTile tile;
    AttnDivision division;
    size_t ws_o_bytes, ws_ml_bytes, ws_parts_bytes;
};

// a fixed function of (shape, max_cache_len), so that the workspace query and the launch agree
AttnPlan plan_attn(const s4c_attn_shape& s, int32_t max_cache_len, AttnTile small) {
    AttnPlan p;
    const int M = s.N * (s.Hq / s.Hkv);
    p.large = s.dtype != S4C_F32 && M > 64;
    p.tile = p.large ? attn_tile_large(s) : small;
    p.division = plan_division(s.B, s.Hkv, s.N, M, max_cache_len, p.tile, device_cus());
    if (p.division.split == 1) {
        p.ws_o_bytes = p.ws_ml_bytes = p.ws_parts_bytes = 0;
    } else {
        const size_t prow = (size_t)p.division.teams * 2 * M;
        p.ws_o_bytes = prow * s.D * sizeof(float);
        p.ws_ml_bytes = ((prow * 2 * sizeof(float) + 255) / 256) * 256;
        p.ws_parts_bytes = (((size_t)s.B * s.Hkv * 2 * sizeof(int32_t) + 255) / 256) * 256;
    }
    return p;
}
AttnPlan plan_attn(const s4c_attn_shape& s, int32_t max_cache_len) {
    return plan_attn(s, max_cache_len, attn_tile_small(s, max_cache_len, device_cus()));
}
size_t workspace_bytes_of(const AttnPlan& p) { return p.ws_o_bytes + p.ws_ml_bytes + p.ws_parts_bytes; }

}  // namespace

extern "C" {
#pragma GCC visibility push(default)

const char* s4c_strerror(int code) {
    switch (code) {
        case S4C_OK: return "ok";
        case S4C_ERR_NULL: return "a required pointer is NULL";
        case S4C_ERR_SHAPE: return "non-positive or inconsistent sizes";
        case S4C_ERR_UNSUPPORTED: return "unsupported size, dtype or mode (N <= 128, D in {64,128})";
        case S4C_ERR_WORKSPACE: return "workspace missing or too small";
        case S4C_ERR_HIP: return "HIP kernel launch failed";
        case S4C_ERR_STATIC_SCRATCH: return "problem larger than the static scratch of s4c_accept_path_static";
    }
    return "unknown status";
}

size_t s4c_tree_attn_workspace_size(const s4c_attn_shape* shape, int32_t max_cache_len) {
    s4c_status why;
    if (!shape || !shape_ok(shape, &why) || max_cache_len < 0) return 0;
    // Also what short units' configuration takes, so that a workspace serves every call up to the length it was made for.
    const size_t own = workspace_bytes_of(plan_attn(*shape, max_cache_len));
    const size_t shorter = workspace_bytes_of(plan_attn(*shape, max_cache_len, attn_tile_small(*shape, 0, device_cus())));
    return own > shorter ? own : shorter;
}

int32_t s4c_tree_attn_num_splits(const s4c_attn_shape* shape, int32_t max_cache_len) {
    s4c_status why;
    if (!shape || !shape_ok(shape, &why) || max_cache_len < 0) return 0;
    return plan_attn(*shape, max_cache_len).division.parts;
}

#pragma GCC visibility pop
}  // extern "C"

namespace {
// log2 of a page size that is a power of two >= 64, else -1
int page_shift_of(int32_t page_size) {
    for (int sh = 6; sh < 31; ++sh)
        if (page_size == (1 << sh)) return sh;
    return -1;
}

// everything of an attention call but the launches
s4c_status tree_attn_prepare(const s4c_attn_shape* shape, const void* q, const void* k_tree, const void* v_tree,
                             const void* k_cache, const void* v_cache, const int32_t* block_table, int32_t max_blocks,
                             int32_t page_shift, int32_t num_pages, const int32_t* cache_len, const int32_t* parent,
                             int32_t max_cache_len, float scale, void* out, int32_t* status, void* workspace,
                             size_t workspace_bytes, AttnPlan* plan, AttnArgs* args) {
    if (!shape || !q || !k_tree || !v_tree || !cache_len || !parent || !out) return S4C_ERR_NULL;
    s4c_status why;
    if (!shape_ok(shape, &why)) return why;
    if (max_cache_len < 0 || max_cache_len > shape->S_cap) return S4C_ERR_SHAPE;
    if (max_cache_len > 0 && (!k_cache || !v_cache)) return S4C_ERR_NULL;
    if (!aligned16(q) || !aligned16(k_tree) || !aligned16(v_tree) || !aligned16(k_cache) || !aligned16(v_cache) ||
        !aligned16(out))
        return S4C_ERR_SHAPE;
    const AttnPlan p = plan_attn(*shape, max_cache_len);
    const size_t need = workspace_bytes_of(p);
    if (need > 0 && (!workspace || workspace_bytes < need || (((uintptr_t)workspace) & 255))) return S4C_ERR_WORKSPACE;

    AttnArgs& a = *args;
    a.q = q; a.k_tree = k_tree; a.v_tree = v_tree; a.k_cache = k_cache; a.v_cache = v_cache;
    a.cache_len = cache_len; a.parent = parent; a.out = out; a.status = status;
    a.ws_ml = (float*)workspace;
    a.ws_parts = (int32_t*)((char*)workspace + p.ws_ml_bytes);
    a.ws_o = (float*)((char*)workspace + p.ws_ml_bytes + p.ws_parts_bytes);
    a.B = shape->B; a.Hq = shape->Hq; a.Hkv = shape->Hkv; a.D = shape->D; a.N = shape->N;
    a.S_cap = shape->S_cap; a.G = shape->Hq / shape->Hkv; a.M = a.N * a.G;
    a.max_cache_len = max_cache_len; a.teams = p.division.teams; a.split = p.division.split; a.mtiles = p.division.mtiles;
    a.tile_rows = p.tile.rows; a.tile_keys = p.tile.keys; a.tile_shift = __builtin_ctz((unsigned)p.tile.keys);
    a.scale_log2 = (scale > 0.f ? scale : 1.0f / sqrtf((float)shape->D)) * kLog2e;
    a.block_table = block_table; a.max_blocks = max_blocks; a.page_shift = page_shift; a.num_pages = num_pages;
    a.part_keys = p.tile.part_keys;
    a.cus = device_cus();
    a.attn_wgs = 0;
    a.tag = a.split > 1 ? next_tag() : 0;
    *plan = p;
    return S4C_OK;
}

hipError_t launch_tree_attn(const AttnPlan& p, const AttnArgs& a, int dtype, const StepTail<kGreedyStep>* step, hipStream_t st) {
    return p.large ? launch_tree_attn_large(a, dtype, step, st) : launch_tree_attn_small(a, dtype, step, st);
}
// attention and its merge
hipError_t launch_attn_and_merge(const AttnPlan& p, const AttnArgs& a, int dtype, hipStream_t st) {
    const hipError_t e = launch_tree_attn(p, a, dtype, nullptr, st);
    return e == hipSuccess && a.split == 0 ? launch_attn_merge(a, dtype, st) : e;       // the parts of balanced shares
}

s4c_status tree_attn_impl(const s4c_attn_shape* shape, const void* q, const void* k_tree, const void* v_tree,
                          const void* k_cache, const void* v_cache, const int32_t* block_table, int32_t max_blocks,
                          int32_t page_shift, int32_t num_pages, const int32_t* cache_len, const int32_t* parent,
                          int32_t max_cache_len, float scale, void* out, int32_t* status, void* workspace,
                          size_t workspace_bytes, void* hip_stream) {
    AttnPlan p;
    AttnArgs a;
    const s4c_status ok = tree_attn_prepare(shape, q, k_tree, v_tree, k_cache, v_cache, block_table, max_blocks, page_shift, num_pages,
                                            cache_len, parent, max_cache_len, scale, out, status, workspace, workspace_bytes, &p, &a);
    if (ok != S4C_OK) return ok;
    return launch_attn_and_merge(p, a, shape->dtype, (hipStream_t)hip_stream) == hipSuccess ? S4C_OK : S4C_ERR_HIP;
}
}  // namespace

extern "C" {
#pragma GCC visibility push(default)

s4c_status s4c_tree_attn(const s4c_attn_shape* shape, const void* q, const void* k_tree,
                         const void* v_tree, const void* k_cache, const void* v_cache,
                         const int32_t* cache_len, const int32_t* parent, int32_t max_cache_len,
                         float scale, void* out, int32_t* status, void* workspace,
                         size_t workspace_bytes, void* hip_stream) {
    return tree_attn_impl(shape, q, k_tree, v_tree, k_cache, v_cache, nullptr, 0, 0, 0, cache_len, parent, max_cache_len,
                          scale, out, status, workspace, workspace_bytes, hip_stream);
}

s4c_status s4c_tree_attn_paged(const s4c_attn_shape* shape, const void* q, const void* k_tree, const void* v_tree,
                               const void* k_pool, const void* v_pool, const int32_t* block_table,
                               int32_t max_blocks, int32_t page_size, int32_t num_pages, const int32_t* cache_len,
                               const int32_t* parent, int32_t max_cache_len, float scale, void* out,
                               int32_t* status, void* workspace, size_t workspace_bytes, void* hip_stream) {
    if (!shape || !block_table || !k_pool || !v_pool) return S4C_ERR_NULL;
    const int sh = page_shift_of(page_size);
    if (sh < 0) return S4C_ERR_UNSUPPORTED;
    if (max_blocks <= 0 || num_pages <= 0 || (long long)max_blocks * page_size > 0x7FFFFFFFll) return S4C_ERR_SHAPE;
    if (shape->S_cap != max_blocks * page_size) return S4C_ERR_SHAPE;       // the logical capacity of a sequence
    return tree_attn_impl(shape, q, k_tree, v_tree, k_pool, v_pool, block_table, max_blocks, sh, num_pages, cache_len,
                          parent, max_cache_len, scale, out, status, workspace, workspace_bytes, hip_stream);
}

size_t s4c_accept_path_workspace_size(int32_t B, int32_t N, int32_t V) {
    if (B <= 0 || N <= 0 || V <= 0) return 0;
    int seg, nseg;
    accept_plan(B, N, V, &seg, &nseg);
    return (((size_t)B * N * nseg * 3 * sizeof(unsigned long long) + 255) / 256) * 256;   // room for two records per (row, run): scan_plan
}

#pragma GCC visibility pop
}  // extern "C"

namespace {
// checks shared by the two acceptance entry points; everything but the workspace
s4c_status accept_args_ok(int32_t B, int32_t N, int32_t V, int32_t logits_dtype, int32_t mode, float temperature,
                          const void* logits, const int32_t* parent, const int32_t* tokens, const float* p_draft,
                          const float* uniforms, int32_t max_path, int32_t* path, int32_t* accept_len,
                          int32_t* accepted_tokens, int32_t* bonus_token) {
    if (!logits || !parent || !tokens || !path || !accept_len || !accepted_tokens || !bonus_token)
        return S4C_ERR_NULL;
    if (B <= 0 || N <= 0 || V <= 0 || max_path <= 0) return S4C_ERR_SHAPE;
    if (N > kMaxNodes || !dtype_ok(logits_dtype) ||
        (mode != S4C_GREEDY && mode != S4C_STOCHASTIC))
        return S4C_ERR_UNSUPPORTED;
    if (mode == S4C_STOCHASTIC) {
        if (!p_draft || !uniforms) return S4C_ERR_NULL;
        if (!(temperature > 0.f)) return S4C_ERR_SHAPE;
    }
    const AcceptPlan p = scan_plan(B, N, V, 2, device_cus());
    if ((size_t)B * N * p.slots > 0x7FFFFFFFull || (size_t)N * p.chunks > 0x7FFFFFFFull) return S4C_ERR_UNSUPPORTED;
    return S4C_OK;
}

// `workspace` holds at least s4c_accept_path_workspace_size(B, N, V) bytes, 256-byte aligned
AcceptArgs accept_prepare(int32_t B, int32_t N, int32_t V, int32_t logits_dtype, int32_t mode, float temperature,
                          const void* logits, const int32_t* parent, const int32_t* tokens, const float* p_draft,
                          const float* uniforms, int32_t max_path, int32_t* path, int32_t* accept_len,
                          int32_t* accepted_tokens, int32_t* bonus_token, int32_t* status, void* workspace) {
    AcceptArgs a;
    a.logits = logits; a.parent = parent; a.tokens = tokens; a.p_draft = p_draft; a.uniforms = uniforms;
    a.path = path; a.accept_len = accept_len; a.accepted_tokens = accepted_tokens;
    a.bonus_token = bonus_token; a.status = status;
    a.rec = (unsigned long long*)workspace;
    a.nonce = next_nonce();
    // S4C_ACCEPT_WAIT_US (environment, >= 0): how long a sequence's collecting workgroup waits for the
    // statistics of the others before it flags the sequence.  A diagnostic knob: 0 makes a collector that
    // does not find everything at its first look give up, which exercises the flagged path on a healthy GPU.
    a.wait_ticks = wait_us("S4C_ACCEPT_WAIT_US", 2000000) * 100;
    a.B = B; a.N = N; a.V = V;
    const size_t es = logits_dtype == S4C_F32 ? 4 : 2;
    a.plan = scan_plan(B, N, V, (int)es, device_cus());
    a.chunks = (((uintptr_t)logits | ((size_t)V * es)) & 15) ? a.plan.chunks : (V + accept_chunk_elems() - 1) / accept_chunk_elems();
    a.max_path = max_path; a.mode = mode; a.dtype = logits_dtype;
    a.inv_temp_log2 = kLog2e / (mode == S4C_STOCHASTIC ? temperature : 1.0f);
    return a;
}

s4c_status accept_launch(const AcceptArgs& a, void* hip_stream) {
    return launch_accept(a, (hipStream_t)hip_stream) == hipSuccess ? S4C_OK : S4C_ERR_HIP;
}
}  // namespace

namespace {
s4c_status compact_prepare(const s4c_attn_shape* shape, const void* k_tree, const void* v_tree, void* k_cache, void* v_cache,
                           int32_t* cache_len, const int32_t* path, const int32_t* accept_len, int32_t max_path,
                           int32_t* dst_index, int32_t* status, CompactArgs* args) {
    if (!shape || !k_tree || !v_tree || !k_cache || !v_cache || !cache_len || !path || !accept_len)
        return S4C_ERR_NULL;
    s4c_attn_shape s = *shape;
    if (s.Hq <= 0) s.Hq = s.Hkv;          // Hq is not used by this call
    if (s.Hkv > 0 && s.Hq % s.Hkv != 0) s.Hq = s.Hkv;
    s4c_status why;
    if (!shape_ok(&s, &why)) return why;
    if (max_path <= 0 || s.S_cap <= 0) return S4C_ERR_SHAPE;
    CompactArgs& a = *args;
    a.k_tree = k_tree; a.v_tree = v_tree; a.k_cache = k_cache; a.v_cache = v_cache;
    a.cache_len = cache_len; a.path = path; a.accept_len = accept_len; a.dst_index = dst_index;
    a.status = status; a.B = s.B; a.Hkv = s.Hkv; a.N = s.N; a.S_cap = s.S_cap; a.max_path = max_path;
    a.row_bytes = s.D * (s.dtype == S4C_F32 ? 4 : 2);
    a.block_table = nullptr; a.max_blocks = a.page_shift = a.num_pages = 0;
    return S4C_OK;
}
}  // namespace

extern "C" {
#pragma GCC visibility push(default)

s4c_status s4c_accept_path(int32_t B, int32_t N, int32_t V, int32_t logits_dtype, int32_t mode,
                           float temperature, const void* logits, const int32_t* parent,
                           const int32_t* tokens, const float* p_draft, const float* uniforms,
                           int32_t max_path, int32_t* path, int32_t* accept_len,
                           int32_t* accepted_tokens, int32_t* bonus_token, int32_t* status,
                           void* workspace, size_t workspace_bytes, void* hip_stream) {
    const s4c_status ok = accept_args_ok(B, N, V, logits_dtype, mode, temperature, logits, parent, tokens, p_draft, uniforms,
                                         max_path, path, accept_len, accepted_tokens, bonus_token);
    if (ok != S4C_OK) return ok;
    const size_t need = s4c_accept_path_workspace_size(B, N, V);
    if (!workspace || workspace_bytes < need || (((uintptr_t)workspace) & 255)) return S4C_ERR_WORKSPACE;
    return accept_launch(accept_prepare(B, N, V, logits_dtype, mode, temperature, logits, parent, tokens, p_draft, uniforms, max_path, path,
                                        accept_len, accepted_tokens, bonus_token, status, workspace), hip_stream);
}

s4c_status s4c_accept_path_static(int32_t B, int32_t N, int32_t V, int32_t logits_dtype, int32_t mode,
                                  float temperature, const void* logits, const int32_t* parent,
                                  const int32_t* tokens, const float* p_draft, const float* uniforms,
                                  int32_t max_path, int32_t* path, int32_t* accept_len,
                                  int32_t* accepted_tokens, int32_t* bonus_token, int32_t* status,
                                  void* hip_stream) {
    const s4c_status ok = accept_args_ok(B, N, V, logits_dtype, mode, temperature, logits, parent, tokens, p_draft, uniforms,
                                         max_path, path, accept_len, accepted_tokens, bonus_token);
    if (ok != S4C_OK) return ok;
    if (s4c_accept_path_workspace_size(B, N, V) > (size_t)S4C_STATIC_SCRATCH_BYTES) return S4C_ERR_STATIC_SCRATCH;
    void* ws = nullptr;
    if (static_scratch(&ws) != hipSuccess) return S4C_ERR_HIP;
    return accept_launch(accept_prepare(B, N, V, logits_dtype, mode, temperature, logits, parent, tokens, p_draft, uniforms, max_path, path,
                                        accept_len, accepted_tokens, bonus_token, status, ws), hip_stream);
}

size_t s4c_accept_resample_workspace_size(int32_t B, int32_t N, int32_t V, int32_t max_path) {
    if (B <= 0 || N <= 0 || V <= 0 || max_path <= 0 || N > kMaxNodes || V > resample_max_vocab()) return 0;
    const size_t words = resample_slot_words(B, N, V, max_path, device_cus());
    const size_t rows = resample_by_rows(B, N, V, device_cus()) ? (size_t)B * N : 0;
    return (words > rows ? words : rows) * sizeof(uint64_t);
}

s4c_status s4c_accept_resample(int32_t B, int32_t N, int32_t V, int32_t logits_dtype, float temperature,
                               const void* logits, const float* draft_probs, const int32_t* parent,
                               const int32_t* tokens, const float* uniforms, const float* u_resample,
                               int32_t max_path, int32_t* path, int32_t* accept_len,
                               int32_t* accepted_tokens, int32_t* bonus_token, int32_t* status,
                               void* workspace, size_t workspace_bytes, void* hip_stream) {
    if (!logits || !draft_probs || !parent || !tokens || !uniforms || !u_resample || !path || !accept_len ||
        !accepted_tokens || !bonus_token)
        return S4C_ERR_NULL;
    if (B <= 0 || N <= 0 || V <= 0 || max_path <= 0 || !(temperature > 0.f)) return S4C_ERR_SHAPE;
    if (N > kMaxNodes || V > resample_max_vocab() || !dtype_ok(logits_dtype))
        return S4C_ERR_UNSUPPORTED;
    // (teams of one workgroup need no workspace; without one they do what the workgroups per node would)
    const size_t need = resample_slot_words(B, N, V, max_path, device_cus()) * sizeof(uint64_t);
    const bool usable = workspace && !(((uintptr_t)workspace) & 255);
    if (need > 0 && (!usable || workspace_bytes < need)) return S4C_ERR_WORKSPACE;
    const bool by_rows = resample_by_rows(B, N, V, device_cus()) && usable && workspace_bytes >= (size_t)B * N * sizeof(uint64_t);
    ResampleArgs a;
    a.logits = logits; a.draft = draft_probs; a.parent = parent; a.tokens = tokens; a.uniforms = uniforms;
    a.u_resample = u_resample; a.path = path; a.accept_len = accept_len; a.accepted_tokens = accepted_tokens;
    a.bonus_token = bonus_token; a.status = status; a.slots = (uint64_t*)workspace;
    a.B = B; a.N = N; a.V = V; a.max_path = max_path; a.dtype = logits_dtype; a.inv_temperature = 1.0 / (double)temperature;
    a.team = by_rows ? 0 : resample_team(B, V, device_cus());
    a.cus = device_cus();
    a.first = a.groups = 0;
    a.nonce = next_nonce();
    a.max_pass = resample_max_pass(N, max_path);
    // S4C_RESAMPLE_SPIN_LIMIT (environment, >= 0): polls before a workgroup gives up on an exchange.  A
    // diagnostic knob: 0 makes every exchange between several workgroups fail, which is how the give-up
    // path is exercised without a stuck GPU.
    a.spin_limit = resample_default_spin_limit();
    if (const char* env = getenv("S4C_RESAMPLE_SPIN_LIMIT")) {
        char* end = nullptr;
        const long v = strtol(env, &end, 10);
        if (end != env && v >= 0 && v <= 0x7FFFFFFFl) a.spin_limit = (int32_t)v;
    }
    return launch_accept_resample(a, (hipStream_t)hip_stream) == hipSuccess ? S4C_OK : S4C_ERR_HIP;
}

s4c_status s4c_kv_compact(const s4c_attn_shape* shape, const void* k_tree, const void* v_tree,
                          void* k_cache, void* v_cache, int32_t* cache_len, const int32_t* path,
                          const int32_t* accept_len, int32_t max_path, int32_t* dst_index,
                          int32_t* status, void* hip_stream) {
    CompactArgs a;
    const s4c_status ok = compact_prepare(shape, k_tree, v_tree, k_cache, v_cache, cache_len, path, accept_len, max_path, dst_index, status, &a);
    if (ok != S4C_OK) return ok;
    return launch_compact(a, (hipStream_t)hip_stream) == hipSuccess ? S4C_OK : S4C_ERR_HIP;
}

s4c_status s4c_kv_compact_paged(const s4c_attn_shape* shape, const void* k_tree, const void* v_tree, void* k_pool,
                                void* v_pool, const int32_t* block_table, int32_t max_blocks, int32_t page_size,
                                int32_t num_pages, int32_t* cache_len, const int32_t* path,
                                const int32_t* accept_len, int32_t max_path, int32_t* dst_index, int32_t* status,
                                void* hip_stream) {
    if (!shape || !k_tree || !v_tree || !k_pool || !v_pool || !block_table || !cache_len || !path || !accept_len)
        return S4C_ERR_NULL;
    const int sh = page_shift_of(page_size);
    if (sh < 0) return S4C_ERR_UNSUPPORTED;
    if (max_blocks <= 0 || num_pages <= 0 || (long long)max_blocks * page_size > 0x7FFFFFFFll) return S4C_ERR_SHAPE;
    s4c_attn_shape s = *shape;
    s.S_cap = max_blocks * page_size;
    if (s.Hq <= 0) s.Hq = s.Hkv;
    if (s.Hkv > 0 && s.Hq % s.Hkv != 0) s.Hq = s.Hkv;
    s4c_status why;
    if (!shape_ok(&s, &why)) return why;
    if (max_path <= 0) return S4C_ERR_SHAPE;
    CompactArgs a;
    a.k_tree = k_tree; a.v_tree = v_tree; a.k_cache = k_pool; a.v_cache = v_pool;
    a.cache_len = cache_len; a.path = path; a.accept_len = accept_len; a.dst_index = dst_index;
    a.status = status; a.B = s.B; a.Hkv = s.Hkv; a.N = s.N; a.S_cap = s.S_cap; a.max_path = max_path;
    a.row_bytes = s.D * (s.dtype == S4C_F32 ? 4 : 2);
    a.block_table = block_table; a.max_blocks = max_blocks; a.page_shift = sh; a.num_pages = num_pages;
    return launch_compact(a, (hipStream_t)hip_stream) == hipSuccess ? S4C_OK : S4C_ERR_HIP;
}

#pragma GCC visibility pop
}  // extern "C"

namespace {
struct BuildLayout { size_t chunks, off_sum, off_topv, off_topi, total; };
BuildLayout build_layout(int32_t B, int32_t N, int32_t V) {
    BuildLayout l;
    l.chunks = ((size_t)V + 7 + build_tree_chunk_elems() - 1) / build_tree_chunk_elems();   // a row may begin up to 7 elements into its first vector
    const size_t rows = (size_t)B * N, K = (size_t)build_tree_max_children();
    auto up = [](size_t x) { return (x + 255) / 256 * 256; };
    size_t o = 0;
    const size_t parts = l.chunks * 4;            // every wavefront of the scan reports its quarter of a chunk
    o += up(rows * parts * 4); l.off_sum = o;
    o += up(rows * parts * 4); l.off_topv = o;
    o += up(rows * parts * K * 4); l.off_topi = o;
    o += up(rows * parts * K * 4); l.total = o;
    return l;
}
}  // namespace

extern "C" {
#pragma GCC visibility push(default)

size_t s4c_build_tree_workspace_size(int32_t B, int32_t N, int32_t V) {
    if (B <= 0 || N <= 0 || V <= 0) return 0;
    return build_layout(B, N, V).total;
}

s4c_status s4c_build_tree(int32_t B, int32_t N, int32_t V, int32_t logits_dtype, float temperature,
                          const void* draft_logits, const int32_t* nchild, const int32_t* root_token,
                          int32_t kmax, int32_t* parent, int32_t* tokens, float* p_draft, int32_t* level,
                          int32_t* status, void* workspace, size_t workspace_bytes, void* hip_stream) {
    if (!draft_logits || !nchild || !root_token || !parent || !tokens || !p_draft) return S4C_ERR_NULL;
    if (B <= 0 || N <= 0 || V <= 0 || kmax <= 0 || !(temperature > 0.f)) return S4C_ERR_SHAPE;
    if (N > kMaxNodes || kmax > build_tree_max_children() || !dtype_ok(logits_dtype))
        return S4C_ERR_UNSUPPORTED;
    const BuildLayout l = build_layout(B, N, V);
    const size_t row_chunks = ((size_t)V + build_tree_chunk_elems() - 1) / build_tree_chunk_elems();
    if ((size_t)B * N * row_chunks * 4 * (size_t)build_tree_max_children() > 0x7FFFFFFFull) return S4C_ERR_UNSUPPORTED;
    if (!workspace || workspace_bytes < l.total || (((uintptr_t)workspace) & 255)) return S4C_ERR_WORKSPACE;
    BuildArgs a;
    a.logits = draft_logits; a.nchild = nchild; a.root_token = root_token; a.parent = parent; a.tokens = tokens;
    a.p_draft = p_draft; a.level = level; a.status = status;
    char* w = (char*)workspace;
    a.ws_max = (float*)w; a.ws_sum = (float*)(w + l.off_sum); a.ws_topv = (float*)(w + l.off_topv);
    a.ws_topi = (int32_t*)(w + l.off_topi);
    a.B = B; a.N = N; a.V = V; a.kmax = kmax; a.dtype = logits_dtype;
    {   // rows that begin inside a 16-byte vector may reach into one chunk more (row_chunk.h)
        const int vec = logits_dtype == S4C_F32 ? 4 : 8;
        const int head = V % vec == 0 && aligned16(draft_logits) ? 0 : vec - 1;
        a.chunks = (int)(((long long)V + head + build_tree_chunk_elems() - 1) / build_tree_chunk_elems());
        build_tree_plan(a);
    }
    a.inv_temp_log2 = kLog2e / temperature;
    return launch_build_tree(a, (hipStream_t)hip_stream) == hipSuccess ? S4C_OK : S4C_ERR_HIP;
}

#pragma GCC visibility pop
}  // extern "C"

namespace {
s4c_status commit_impl(const s4c_attn_shape* shape, int32_t layers, const void* k_tree, const void* v_tree,
                       void* k_cache, void* v_cache, const int32_t* block_table, int32_t max_blocks, int32_t page_shift,
                       int32_t num_pages, int32_t* cache_len, const int32_t* path, const int32_t* accept_len,
                       int32_t max_path, const void* features, int32_t feature_bytes, void* features_out,
                       int32_t* dst_index, int32_t* status, void* hip_stream) {
    if (!shape || !k_tree || !v_tree || !k_cache || !v_cache || !cache_len || !path || !accept_len)
        return S4C_ERR_NULL;
    s4c_attn_shape s = *shape;
    if (block_table) s.S_cap = max_blocks << page_shift;
    if (s.Hq <= 0) s.Hq = s.Hkv;          // Hq is not used by this call
    if (s.Hkv > 0 && s.Hq % s.Hkv != 0) s.Hq = s.Hkv;
    s4c_status why;
    if (!shape_ok(&s, &why)) return why;
    if (max_path <= 0 || s.S_cap <= 0 || layers <= 0 || layers > 65534) return S4C_ERR_SHAPE;
    const bool feats = features || features_out;
    if (feats) {
        if (!features || !features_out) return S4C_ERR_NULL;
        if (feature_bytes <= 0 || feature_bytes % 16 != 0) return S4C_ERR_SHAPE;
        if ((((uintptr_t)features) | ((uintptr_t)features_out)) & 15) return S4C_ERR_SHAPE;
    }
    CommitArgs a;
    a.k_tree = k_tree; a.v_tree = v_tree; a.k_cache = k_cache; a.v_cache = v_cache; a.cache_len = cache_len;
    a.path = path; a.accept_len = accept_len; a.features = features; a.features_out = features_out;
    a.dst_index = dst_index; a.status = status;
    a.B = s.B; a.Hkv = s.Hkv; a.N = s.N; a.S_cap = s.S_cap; a.max_path = max_path; a.layers = layers;
    a.row_bytes = s.D * (s.dtype == S4C_F32 ? 4 : 2);
    a.feature_bytes = feats ? feature_bytes : 0;
    a.tree_layer_bytes = (size_t)s.B * s.N * s.Hkv * a.row_bytes;
    a.cache_layer_bytes = block_table ? (((size_t)num_pages * s.Hkv) << page_shift) * a.row_bytes
                                      : (size_t)s.B * s.Hkv * s.S_cap * a.row_bytes;
    a.block_table = block_table; a.max_blocks = max_blocks; a.page_shift = page_shift; a.num_pages = num_pages;
    return launch_commit(a, (hipStream_t)hip_stream) == hipSuccess ? S4C_OK : S4C_ERR_HIP;
}
}  // namespace

extern "C" {
#pragma GCC visibility push(default)

s4c_status s4c_commit_path(const s4c_attn_shape* shape, int32_t layers, const void* k_tree, const void* v_tree,
                           void* k_cache, void* v_cache, int32_t* cache_len, const int32_t* path,
                           const int32_t* accept_len, int32_t max_path, const void* features,
                           int32_t feature_bytes, void* features_out, int32_t* dst_index, int32_t* status,
                           void* hip_stream) {
    return commit_impl(shape, layers, k_tree, v_tree, k_cache, v_cache, nullptr, 0, 0, 0, cache_len, path, accept_len,
                       max_path, features, feature_bytes, features_out, dst_index, status, hip_stream);
}

s4c_status s4c_commit_path_paged(const s4c_attn_shape* shape, int32_t layers, const void* k_tree, const void* v_tree,
                                 void* k_pool, void* v_pool, const int32_t* block_table, int32_t max_blocks,
                                 int32_t page_size, int32_t num_pages, int32_t* cache_len, const int32_t* path,
                                 const int32_t* accept_len, int32_t max_path, const void* features,
                                 int32_t feature_bytes, void* features_out, int32_t* dst_index, int32_t* status,
                                 void* hip_stream) {
    if (!block_table) return S4C_ERR_NULL;
    const int sh = page_shift_of(page_size);
    if (sh < 0) return S4C_ERR_UNSUPPORTED;
    if (max_blocks <= 0 || num_pages <= 0 || (long long)max_blocks * page_size > 0x7FFFFFFFll) return S4C_ERR_SHAPE;
    return commit_impl(shape, layers, k_tree, v_tree, k_pool, v_pool, block_table, max_blocks, sh, num_pages, cache_len,
                       path, accept_len, max_path, features, feature_bytes, features_out, dst_index, status, hip_stream);
}

#pragma GCC visibility pop
}  // extern "C"

namespace {
// Up to kNeedsWorkspace tokens a call must bring a workspace of at least this size: what the weight-streaming kernel's partial
// sums take.  More tokens than that kernel has room for go to the tiled one, which makes do with any workspace or none; for them the size, that of
// equal passes over the tokens, is only the line between calls that are taken and calls that are refused, which callers rely on.
constexpr int kNeedsWorkspace = 512;
size_t least_linear_bytes(int32_t T, int32_t H, int32_t Hout) {
    if (T > kNeedsWorkspace) return 0;
    const int step = draft_linear_small_max_tokens(), passes = (T + step - 1) / step, per = (T + passes - 1) / passes;
    size_t need = 0;
    for (int t0 = 0; t0 < T; t0 += per) {
        const int Tp = T - t0 < per ? T - t0 : per;
        int ksub, kslice, nslices;
        draft_linear_small_plan(Tp, H, Hout, device_cus(), &ksub, &kslice, &nslices);
        const size_t b = (size_t)nslices * Tp * Hout * sizeof(float);
        if (b > need) need = b;
    }
    return need;
}
// The tiled kernel rather than the one that streams W for few tokens: from 65 tokens on where W is large, whose stream the tiled kernel,
// all its loads asynchronous, keeps up better, and always where tokens would not fit the other.  Streamed and tiled, us: 128
// tokens H 2048 18.4 and 20.6, 4096 32.7 and 32.6, 5120 53.0 and 40.9, 8192 99.9 and 85.3; 80 tokens 4096 28.2 and 29.8, 5120 41.8
// and 37.9, 8192 88.7 and 82.2; 64 tokens 5120 36.8 and 35.9, 8192 81.2 and 79.5; 33 tokens 4096 22.9 and 26.6.  (More than 128
// tokens used to be streamed in passes up to 512, W each time: 150, 1024 21.9 and 17.8, 8192 145 and 91; 512, 8192 377 and 140.)
bool linear_is_tiled(int32_t T, int32_t H, int32_t Hout) {
    return T > draft_linear_small_max_tokens() || (T > 64 && (long long)H * Hout >= 5120ll * 5120);
}
size_t tiled_bytes(int32_t T, int32_t H, int32_t Hout) {
    int kslice;
    const int n = draft_linear_slices(T, H, Hout, device_cus(), ~(size_t)0, &kslice);
    return n > 1 ? (size_t)n * T * Hout * sizeof(float) : 0;
}
}  // namespace

extern "C" {
#pragma GCC visibility push(default)

size_t s4c_draft_linear_workspace_size(int32_t T, int32_t H, int32_t Hout) {
    if (T <= 0 || H <= 0 || Hout <= 0 || H % draft_linear_tile_k() != 0 || Hout % draft_linear_tile_out() != 0) return 0;
    const size_t least = least_linear_bytes(T, H, Hout), tiled = linear_is_tiled(T, H, Hout) ? tiled_bytes(T, H, Hout) : 0;
    return (((least > tiled ? least : tiled) + 255) / 256) * 256;
}

s4c_status s4c_draft_linear(int32_t T, int32_t H, int32_t Hout, int32_t dtype, const void* e, const void* f,
                            const void* W, const void* bias, void* out, void* workspace, size_t workspace_bytes,
                            void* hip_stream) {
    if (!e || !f || !W || !out) return S4C_ERR_NULL;
    if (T <= 0 || H <= 0 || Hout <= 0) return S4C_ERR_SHAPE;
    if ((dtype != S4C_BF16 && dtype != S4C_F16) || H % draft_linear_tile_k() != 0 || Hout % draft_linear_tile_out() != 0 ||
        (long long)T * H * 2 >= (1ll << 31) || H > 16384)
        return S4C_ERR_UNSUPPORTED;
    if ((((uintptr_t)e) | ((uintptr_t)f) | ((uintptr_t)W) | ((uintptr_t)out)) & 15) return S4C_ERR_SHAPE;
    LinearArgs a;
    a.e = e; a.f = f; a.W = W; a.bias = bias; a.out = out; a.ws = nullptr; a.T = T; a.H = H; a.Hout = Hout; a.dtype = dtype;
    a.ttiles = a.otiles = 0; a.ksub = a.kslice = a.nslices = 0;
    const bool usable = workspace && !(((uintptr_t)workspace) & 255);
    if (T <= kNeedsWorkspace && (!usable || workspace_bytes < least_linear_bytes(T, H, Hout))) return S4C_ERR_WORKSPACE;
    a.ws = (float*)workspace;
    hipError_t err;
    if (linear_is_tiled(T, H, Hout)) {
        // (as many slices as the workspace has room for)
        const size_t most = usable ? workspace_bytes / ((size_t)T * Hout * sizeof(float)) : 0;
        a.nslices = draft_linear_slices(T, H, Hout, device_cus(), most, &a.kslice);
        err = launch_draft_linear(a, (hipStream_t)hip_stream);
    } else {
        draft_linear_small_plan(T, H, Hout, device_cus(), &a.ksub, &a.kslice, &a.nslices);
        err = launch_draft_linear_small(a, (hipStream_t)hip_stream);
    }
    return err == hipSuccess ? S4C_OK : S4C_ERR_HIP;
}

#pragma GCC visibility pop
}  // extern "C"

namespace {
// what a step needs, and what one in a single launch needs behind it (a call without that much takes two)
size_t step_bytes(const s4c_attn_shape& s, int32_t V) {
    return s4c_accept_path_workspace_size(s.B, s.N, V) + (step_message_bytes(s.B, s.Hkv) + 255) / 256 * 256;
}
constexpr int kOneLaunchMostSequences = 32;           // (heads_of_copier)
size_t one_launch_bytes(const s4c_attn_shape& s) {
    return s.B > kOneLaunchMostSequences ? 0 : (size_t)s.B * device_cus() * 2 * sizeof(told::Pair);      // at most two workgroups a CU
}

// A step in one launch: where the attention leaves places for the collectors and for enough scanning workgroups (step_plan.h).
bool plan_one_launch(const s4c_step& p, const AttnPlan& plan, const AttnArgs& attn, AcceptArgs& accept) {
    if (p.logits_dtype != p.shape.dtype || attn.split == 0 || attn.B > kOneLaunchMostSequences || attn.B * 8 > attn.cus) return false;
    if (p.accept_workspace_bytes < step_bytes(p.shape, p.V) + (size_t)attn.B * attn_workgroups(attn) * sizeof(told::Pair)) return false;
    const int places = device_cus() * plan.tile.per_cu - attn_workgroups(attn) - attn.B;
    const int wgs = places / attn.B < accept.plan.wgs ? places / attn.B : accept.plan.wgs;
    if (wgs < 1) return false;
    const long long chunks = ((long long)attn.N * accept.chunks + wgs - 1) / wgs;
    const long long tiles = ((attn.max_cache_len + attn.tile_keys - 1) / attn.tile_keys + (attn.N + attn.tile_keys - 1) / attn.tile_keys + attn.split - 1) / attn.split;
    const StepScan scan = {chunks, accept.chunks, tiles, (long long)attn.B * attn.N * p.V * (p.logits_dtype == S4C_F32 ? 4 : 2), p.logits_dtype == S4C_F32,
                           p.mode == S4C_GREEDY, plan.large, attn.D};
    if (!one_launch_pays(scan)) return false;
    accept.plan.wgs = wgs;
    return true;
}
}  // namespace

extern "C" {
#pragma GCC visibility push(default)

size_t s4c_verify_step_workspace_size(const s4c_attn_shape* shape, int32_t V) {
    s4c_status why;
    if (!shape || !shape_ok(shape, &why) || V <= 0) return 0;
    return step_bytes(*shape, V) + one_launch_bytes(*shape);
}

s4c_status s4c_verify_step(const s4c_step* p, void* hip_stream) {
    if (!p) return S4C_ERR_NULL;
    hipStream_t st = (hipStream_t)hip_stream;
    AttnPlan plan;
    AttnArgs attn;
    CompactArgs compact;
    s4c_status ok = tree_attn_prepare(&p->shape, p->q, p->k_tree, p->v_tree, p->k_cache, p->v_cache, nullptr, 0, 0, 0, p->cache_len, p->parent,
                                      p->max_cache_len, p->scale, p->out, p->attn_status, p->attn_workspace, p->attn_workspace_bytes,
                                      &plan, &attn);
    if (ok != S4C_OK) return ok;
    const int32_t B = p->shape.B, N = p->shape.N, V = p->V;
    ok = accept_args_ok(B, N, V, p->logits_dtype, p->mode, p->temperature, p->logits, p->parent, p->tokens, p->p_draft, p->uniforms,
                        p->max_path, p->path, p->accept_len, p->accepted_tokens, p->bonus_token);
    if (ok != S4C_OK) return ok;
    if (!p->accept_workspace || p->accept_workspace_bytes < step_bytes(p->shape, V) ||
        (((uintptr_t)p->accept_workspace) & 255))
        return S4C_ERR_WORKSPACE;
    ok = compact_prepare(&p->shape, p->k_tree, p->v_tree, p->k_cache, p->v_cache, p->cache_len, p->path, p->accept_len, p->max_path,
                         p->dst_index, p->compact_status, &compact);
    if (ok != S4C_OK) return ok;
    AcceptArgs accept = accept_prepare(B, N, V, p->logits_dtype, p->mode, p->temperature, p->logits, p->parent, p->tokens, p->p_draft,
                                             p->uniforms, p->max_path, p->path, p->accept_len, p->accepted_tokens, p->bonus_token,
                                             p->accept_status, p->accept_workspace);
    accept::rec_t* const messages = (accept::rec_t*)((char*)p->accept_workspace + s4c_accept_path_workspace_size(B, N, V));
    // the copying workgroups wait 2 s longer than the collector they hear from (S4C_COPY_WAIT_US: that long)
    const long long copy_ticks = wait_us("S4C_COPY_WAIT_US", accept.wait_ticks / 100 + 2000000) * 100;
    hipError_t e;
    if (plan_one_launch(*p, plan, attn, accept)) {
        StepTail<kGreedyStep> tail;
        tail.accept = accept;
        tail.step = accept::make_step(accept, compact, messages, copy_ticks);
        tail.step.lens = (told::Pair*)((char*)p->accept_workspace + step_bytes(p->shape, V));
        tail.step.attn_wgs = attn_workgroups(attn);
        tail.step.tag = next_tag();
        e = launch_tree_attn(plan, attn, p->shape.dtype, &tail, st);
    } else if (p->logits_dtype == p->shape.dtype) {
        attn.tag = 0;
        e = launch_tree_attn(plan, attn, p->shape.dtype, nullptr, st);
        if (e == hipSuccess) e = launch_step(attn, accept, compact, messages, copy_ticks, st);
    } else {
        e = launch_attn_and_merge(plan, attn, p->shape.dtype, st);
        if (e == hipSuccess) e = launch_accept(accept, st);
        if (e == hipSuccess) e = launch_compact(compact, st);
    }
    return e == hipSuccess ? S4C_OK : S4C_ERR_HIP;
}

#pragma GCC visibility pop
}  // extern "C"

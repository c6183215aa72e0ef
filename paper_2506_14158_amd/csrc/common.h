// Internal declarations shared by the HIP translation units of libs4c (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "attn_division.h"
#include "s4c.h"

namespace s4c {

constexpr int kMaxNodes = 128;
constexpr float kLog2e = 1.4426950408889634f;

typedef uint16_t bf16_t;   // raw bf16 bits
typedef _Float16 f16_t;    // IEEE binary16

__device__ __forceinline__ float bf16_to_f32(bf16_t x) { return __uint_as_float(((uint32_t)x) << 16); }

// round-to-nearest-even; inputs are finite
__device__ __forceinline__ bf16_t f32_to_bf16(float f) {
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (bf16_t)(u >> 16);
}

template <typename T> __device__ __forceinline__ float to_f32(T x);
template <> __device__ __forceinline__ float to_f32<float>(float x) { return x; }
template <> __device__ __forceinline__ float to_f32<bf16_t>(bf16_t x) { return bf16_to_f32(x); }
template <> __device__ __forceinline__ float to_f32<f16_t>(f16_t x) { return (float)x; }

template <typename T> __device__ __forceinline__ T from_f32(float x);
template <> __device__ __forceinline__ float from_f32<float>(float x) { return x; }
template <> __device__ __forceinline__ bf16_t from_f32<bf16_t>(float x) { return f32_to_bf16(x); }
template <> __device__ __forceinline__ f16_t from_f32<f16_t>(float x) { return (f16_t)x; }   // round to nearest even

// the two 16-bit elements of a 32-bit word (low half first), as floats
template <typename T> __device__ __forceinline__ void unpack2(uint32_t w, float& lo, float& hi);
template <> __device__ __forceinline__ void unpack2<bf16_t>(uint32_t w, float& lo, float& hi) {
    lo = __uint_as_float(w << 16);
    hi = __uint_as_float(w & 0xFFFF0000u);
}
template <> __device__ __forceinline__ void unpack2<f16_t>(uint32_t w, float& lo, float& hi) {
    typedef _Float16 h2 __attribute__((ext_vector_type(2)));
    const h2 v = __builtin_bit_cast(h2, w);
    lo = (float)v[0];
    hi = (float)v[1];
}

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// Arguments of the attention kernels.  Row r of the M = N*G query rows of one (sequence, KV
// head) is node r / G, group head r % G.
struct AttnArgs {
    const void* q;
    const void* k_tree;
    const void* v_tree;
    const void* k_cache;
    const void* v_cache;
    const int32_t* cache_len;
    const int32_t* parent;
    void* out;
    int32_t* status;
    float* ws_o;    // [teams][2][M][D]  unnormalised outputs of the parts of divided units (attn_division.h)
    float* ws_ml;   // [teams][2][M][2]  (running max in log2 units, running sum)
    int32_t* ws_parts;    // [B][Hkv][2]  first and last team of a unit
    int32_t B, Hq, Hkv, D, N, S_cap, G, M;
    int32_t max_cache_len;
    int32_t teams;      // teams the work is divided between (attn_division.h)
    int32_t split;      // teams per (sequence, KV head); 0: equal shares of all units' tiles laid end to end
    int32_t mtiles;     // query-row tiles per (sequence, KV head) = workgroups per team
    int32_t tile_rows;  // query rows per workgroup
    int32_t tile_keys, tile_shift;   // keys per tile of the kernel that will run, and its log2
    int32_t part_keys;  // waves that share the columns of a row in a part (attn_parts.h)
    int32_t cus;        // compute units of the device
    int32_t attn_wgs;   // set by the launcher: workgroups of the launch that attend
    uint64_t tag;       // equal runs: the call's, under which its workgroups agree on the merge (attn_meet.h); 0: the next launch merges
    float scale_log2; // softmax scale * log2(e)
    // paged cache (block_table != null): k_cache / v_cache are pools [num_pages][Hkv][page][D],
    // row j of sequence b is row j & (page-1) of page block_table[b][j >> page_shift]
    const int32_t* block_table;   // [B][max_blocks] or null
    int32_t max_blocks, page_shift, num_pages;
};

// launchers (defined in the kernel translation units); return hipGetLastError()
// (`step`: with the rest of a verification step behind it, attn_step.h; the kind is accept.mode, known to the compiler)
enum StepKind { kNoStep = 0, kGreedyStep = 1, kStochasticStep = 2 };
template <StepKind KIND>
struct StepTail;
hipError_t launch_tree_attn_large(const AttnArgs& a, int dtype, const StepTail<kGreedyStep>* step, hipStream_t st);    // 16-bit data, more than 64 query rows
hipError_t launch_tree_attn_small(const AttnArgs& a, int dtype, const StepTail<kGreedyStep>* step, hipStream_t st);    // at most 64 query rows, or fp32 data
// (of one type each)
hipError_t launch_large_bf16(const AttnArgs& a, const StepTail<kGreedyStep>* step, hipStream_t st);
hipError_t launch_large_f16(const AttnArgs& a, const StepTail<kGreedyStep>* step, hipStream_t st);
hipError_t launch_smallm_bf16(const AttnArgs& a, const StepTail<kGreedyStep>* step, hipStream_t st);
hipError_t launch_smallm_f16(const AttnArgs& a, const StepTail<kGreedyStep>* step, hipStream_t st);
hipError_t launch_smallm_f32(const AttnArgs& a, const StepTail<kGreedyStep>* step, hipStream_t st);
hipError_t launch_attn_merge(const AttnArgs& a, int dtype, hipStream_t st);
AttnTile attn_tile_large(const s4c_attn_shape& s);
AttnTile attn_tile_small(const s4c_attn_shape& s, int32_t max_cache_len, int cus);

// How a call's scan is divided: see scan_plan in accept_path.hip
struct AcceptPlan {
    int32_t chunks;    // of a row of any alignment
    int32_t seg;       // fewest chunks of a workgroup's run
    int32_t slots;     // most runs that a row's chunks can lie in
    int32_t wgs;       // scanning workgroups per sequence
};
AcceptPlan scan_plan(int B, int N, int V, int elem_bytes, int cus);

struct AcceptArgs {
    const void* logits;
    const int32_t* parent;
    const int32_t* tokens;
    const float* p_draft;
    const float* uniforms;
    int32_t* path;
    int32_t* accept_len;
    int32_t* accepted_tokens;
    int32_t* bonus_token;
    int32_t* status;
    unsigned long long* rec;   // [B*N][slots][2] (call nonce << 32) | bits of (maximum, argmax) or (reference, sum of exponentials)
    uint32_t nonce;    // tells this call's records from whatever the words held before
    long long wait_ticks;   // how long a collector waits for its sequence's records (100 MHz wall clock)
    int32_t B, N, V, max_path, mode, dtype;
    AcceptPlan plan;
    int32_t chunks;    // of a row, for its alignment (<= plan.chunks)
    float inv_temp_log2;   // log2(e) / T
};
hipError_t launch_accept(const AcceptArgs& a, hipStream_t st);
struct AttnArgs;
struct CompactArgs;
// The rest of a verification step after the attention kernel in one launch: the merge of divided attention, acceptance, and the accepted path's rows appended to the cache.  All three of one element type.
hipError_t launch_step(const AttnArgs& attn, const AcceptArgs& accept, const CompactArgs& compact,
                       unsigned long long* messages, long long copy_ticks, hipStream_t st);
size_t step_message_bytes(int B, int Hkv);
int accept_chunk_elems();
void accept_plan(int B, int N, int V, int* seg, int* nseg);

struct ResampleArgs {
    const void* logits;
    const float* draft;        // [B][N][V]
    const int32_t* parent;
    const int32_t* tokens;
    const float* uniforms;     // [B][N]
    const float* u_resample;   // [B]
    int32_t* path;
    int32_t* accept_len;
    int32_t* accepted_tokens;
    int32_t* bonus_token;
    int32_t* status;
    uint64_t* slots;           // team > 1: [B][max_pass][4][team] exchange words; team == 0: [B][N] (nonce << 32) | decision
    int32_t B, N, V, max_path, dtype;
    int32_t team;              // workgroups per sequence; 0: one per node
    int32_t cus;               // of the device
    int32_t first, groups;     // set by the launcher: first sequence of a launch of teams, resample_launch
    uint32_t nonce;            // tells this call's words from whatever they held before
    int32_t max_pass;          // exchanges a sequence may need
    int32_t spin_limit;        // polls before a workgroup gives up on an exchange
    double inv_temperature;
};
hipError_t launch_accept_resample(const ResampleArgs& a, hipStream_t st);
int resample_max_vocab();
int resample_max_pass(int N, int max_path);
int resample_default_spin_limit();
size_t resample_slot_words(int B, int N, int V, int max_path, int cus);      // of the teams

struct CompactArgs {
    const void* k_tree;
    const void* v_tree;
    void* k_cache;
    void* v_cache;
    int32_t* cache_len;
    const int32_t* path;
    const int32_t* accept_len;
    int32_t* dst_index;
    int32_t* status;
    int32_t B, Hkv, N, S_cap, max_path;
    int32_t row_bytes;   // D * element size
    const int32_t* block_table;   // paged cache: [B][max_blocks] (S_cap = max_blocks << page_shift), else null
    int32_t max_blocks, page_shift, num_pages;
};
hipError_t launch_compact(const CompactArgs& a, hipStream_t st);

struct BuildArgs {
    const void* logits;        // draft logits [B][N][V]
    const int32_t* nchild;     // [B][N]
    const int32_t* root_token; // [B]
    int32_t* parent;
    int32_t* tokens;
    float* p_draft;
    int32_t* level;            // nullable
    int32_t* status;           // nullable
    float* ws_max;             // [B*N][chunks]
    float* ws_sum;             // [B*N][chunks]
    float* ws_topv;            // [B*N][chunks][8]
    int32_t* ws_topi;          // [B*N][chunks][8]
    int32_t B, N, V, chunks, kmax, dtype;
    int32_t seg, nseg;         // chunks per workgroup of the scan, workgroups per row
    float inv_temp_log2;
};
void build_tree_plan(BuildArgs& a);       // seg and nseg
hipError_t launch_build_tree(const BuildArgs& a, hipStream_t st);
int build_tree_max_children();
int build_tree_chunk_elems();

struct CommitArgs {
    const void* k_tree;        // [layers][B][N][Hkv][D]
    const void* v_tree;
    void* k_cache;             // [layers][B][Hkv][S_cap][D]
    void* v_cache;
    int32_t* cache_len;
    const int32_t* path;
    const int32_t* accept_len;
    const void* features;      // [B][N][feature_bytes] or null
    void* features_out;        // [B][max_path][feature_bytes] or null
    int32_t* dst_index;
    int32_t* status;
    size_t tree_layer_bytes, cache_layer_bytes;
    int32_t B, Hkv, N, S_cap, max_path, layers;
    int32_t row_bytes;         // D * element size
    int32_t feature_bytes;
    // paged pools (block_table != null): k_cache / v_cache are [layers][num_pages][Hkv][page][D], one
    // block table [B][max_blocks] serves every layer; S_cap = max_blocks << page_shift
    const int32_t* block_table;
    int32_t max_blocks, page_shift, num_pages;
};
hipError_t launch_commit(const CommitArgs& a, hipStream_t st);

struct LinearArgs {
    const void* e;       // [T][H] bf16 or fp16
    const void* f;       // [T][H]
    const void* W;       // [Hout][2H]
    const void* bias;    // [Hout] or null
    void* out;           // [T][Hout]
    float* ws;           // [nslices][T][Hout] partial sums
    int32_t T, H, Hout, dtype;
    int32_t ttiles, otiles;   // set by the launcher
    int32_t ksub, kslice, nslices;   // few tokens: reduction elements per LDS fill, per workgroup, workgroups per tile; tiled: stages and slices
};
hipError_t launch_draft_linear(const LinearArgs& a, hipStream_t st);         // nslices > 1: partial sums in ws
hipError_t launch_draft_linear_reduce(const LinearArgs& a, hipStream_t st);  // adds the slices' partial sums
int draft_linear_slices(int T, int H, int Hout, int cus, size_t most, int* kslice);      // of the tiled kernel, kslice stages each
hipError_t launch_draft_linear_small(const LinearArgs& a, hipStream_t st);   // T <= draft_linear_small_max_tokens()
int draft_linear_small_max_tokens();      // tokens that the weight-streaming kernel takes
void draft_linear_small_plan(int T, int H, int Hout, int cus, int* ksub, int* kslice, int* nslices);
int draft_linear_tile_out();
int draft_linear_tile_k();

}  // namespace s4c

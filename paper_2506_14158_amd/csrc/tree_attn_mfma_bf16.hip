// tree_attn_mfma.h for bf16 data, and what a shape takes.
#include "tree_attn_mfma.h"

namespace s4c {

// 32 rows per wave.  (Head size 64 leaves room for two four-wave workgroups on a CU.)
AttnTile attn_tile_large(const s4c_attn_shape& s) {
    const int wr = pick_wr(s.N * (s.Hq / s.Hkv));
    return AttnTile{32 * wr, kBN, wr == 4 && 2 * lds_bytes_for(4, s.D) <= 160 * 1024 ? 2 : 1, s.D == 128, 1};
}

hipError_t launch_large_bf16(const AttnArgs& a, const StepTail<kGreedyStep>* step, hipStream_t st) { return launch_by_shape<false>(a, step, st); }

hipError_t launch_tree_attn_large(const AttnArgs& a, int dtype, const StepTail<kGreedyStep>* step, hipStream_t st) {
    return dtype == S4C_F16 ? launch_large_f16(a, step, st) : launch_large_bf16(a, step, st);
}

}  // namespace s4c

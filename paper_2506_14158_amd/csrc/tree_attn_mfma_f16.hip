// tree_attn_mfma.h for fp16 data.
#include "tree_attn_mfma.h"

namespace s4c {

hipError_t launch_large_f16(const AttnArgs& a, const StepTail<kGreedyStep>* step, hipStream_t st) { return launch_by_shape<true>(a, step, st); }

}  // namespace s4c

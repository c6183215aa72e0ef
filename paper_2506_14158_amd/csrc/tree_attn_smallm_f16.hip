// tree_attn_smallm.h for fp16 data.
#include "tree_attn_smallm.h"

namespace s4c {

hipError_t launch_smallm_f16(const AttnArgs& a, const StepTail<kGreedyStep>* step, hipStream_t st) { return launch_smallm<kH16>(a, step, st); }

}  // namespace s4c

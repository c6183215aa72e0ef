// tree_attn_smallm.h for fp32 data, and which configuration a shape takes.
#include "tree_attn_smallm.h"

namespace s4c {

namespace {

template <class Use>
auto with_cfg(int dtype, int D, int rows, Use use) {
    if (dtype == S4C_F32) return with_cfg<kF32>(D, rows, use);
    return dtype == S4C_F16 ? with_cfg<kH16>(D, rows, use) : with_cfg<kB16>(D, rows, use);
}

}  // namespace

// Up to 32 rows take the configuration of one row block.  16-bit data of head size 128 only where a CU has more than
// 7168 keys to stream, in long units: four key groups fill a CU's LDS with one workgroup, and two workgroups hide each other's starts and
// merges (512 units of 20 rows, 20 keys: 28.0 us and 8.6 with two; 640 units of 300 keys 38 and 29, 2400 keys 151 and 150, 4800 keys
// 273 and 279; 256 units of 8192 keys 180 and 189; 1280 units of 900 to 1800 keys 192 and 167).
AttnTile attn_tile_small(const s4c_attn_shape& s, int32_t max_cache_len, int cus) {
    const bool deep = max_cache_len >= 4096 && (long long)s.B * s.Hkv * max_cache_len >= 7168ll * cus;
    const int rows = s.N * (s.Hq / s.Hkv) <= 32 && (s.D == 64 || (s.dtype != S4C_F32 && deep)) ? 32 : 64;
    return with_cfg(s.dtype, s.D, rows, [](auto c) {
        typedef decltype(c) C;
        return AttnTile{32 * C::kRBW, kBN, C::kPerCu, C::kElem != kF32 && C::kD == 128, C::kOwners};
    });
}


hipError_t launch_smallm_f32(const AttnArgs& a, const StepTail<kGreedyStep>* step, hipStream_t st) { return launch_smallm<kF32>(a, step, st); }

hipError_t launch_tree_attn_small(const AttnArgs& a, int dtype, const StepTail<kGreedyStep>* step, hipStream_t st) {
    return dtype == S4C_F32 ? launch_smallm_f32(a, step, st) : dtype == S4C_F16 ? launch_smallm_f16(a, step, st) : launch_smallm_bf16(a, step, st);
}

}  // namespace s4c

// A verification step in one launch (s4c_verify_step): what the launch holds behind its attention workgroups.
//
// Acceptance needs nothing of the attention, so its workgroups (accept_roles.h) run beside
// the attention's where those leave places on the chip free, instead of behind them: attention, scan, collectors, copiers,
// in this order.  The appended rows lie behind every key that the attention
// reads; the lengths, which all its workgroups read, are advanced when all of them have said that they have.
// Two launches and one, a whole step, us: fp32, 4 heads, 128 keys + 15 nodes 19.6 and 12.4; 32 heads, 1024 keys + 60 nodes, V 32000
// 19.7 and 15.6; 3 x 8 heads of size 64, 2049 keys 25.7 and 21.3; 4 x 40 heads, 4096 keys 81.1 and 73.9.  (Which of the two a step takes: step_plan.h.)
#pragma once
#include "accept_roles.h"
#include "attn_parts.h"

namespace s4c {

template <StepKind KIND>
struct StepTail {
    AcceptArgs accept;
    accept::StepArgs step;
    StepTail() = default;
    template <StepKind OTHER>
    explicit StepTail(const StepTail<OTHER>& t) : accept(t.accept), step(t.step) {}
};
template <>
struct StepTail<kNoStep> {};

// The attention kernels' arguments, (AttnArgs, StepTail), read when they are asked for.  As the named parameters, all that the
// whole kernel needs is loaded at its start and kept, and the attention's scalar registers do not hold it: a hundred values written
// to vector registers' lanes first, 0.2 us of every launch.
struct Arguments {
    typedef const __attribute__((address_space(4))) unsigned char* Ptr;
    Ptr at;
    __device__ __forceinline__ Arguments() : at((Ptr)__builtin_amdgcn_kernarg_segment_ptr()) { asm volatile("" : "+s"(at)); }
    __device__ __forceinline__ const AttnArgs& attn() const { return *(const AttnArgs*)at; }
    template <StepKind KIND>
    __device__ __forceinline__ const StepTail<KIND>& tail() const {
        constexpr size_t al = alignof(StepTail<KIND>);
        return *(const StepTail<KIND>*)(at + (sizeof(AttnArgs) + al - 1) / al * al);
    }
};

// What an attention workgroup says to the collectors, the first wave's lanes to one sequence's each: that all its waves have the lengths ...
template <StepKind KIND>
__device__ __forceinline__ void lens_read(const StepTail<KIND>& t, const AttnArgs& a, const work::Lens& lens) {
    asm volatile("" ::"v"(lens.mine));
    told::At p{t.step.lens + (size_t)threadIdx.x * a.attn_wgs + blockIdx.x};
    if (threadIdx.x < (unsigned)a.B) told::tell(p, t.step.tag);
}
// ... and its look for one that has given up, before its output and behind it.
template <StepKind KIND>
__device__ __forceinline__ uint64_t lens_look_back() {
    uint64_t mark = 0;
    if constexpr (KIND != kNoStep) {
        const Arguments args;
        const AttnArgs& a = args.attn();
        told::At p{args.tail<KIND>().step.lens + (size_t)threadIdx.x * a.attn_wgs + blockIdx.x};
        if (threadIdx.x < (unsigned)a.B) mark = told::look_back(p);
    }
    return mark;
}
template <StepKind KIND>
__device__ __forceinline__ void lens_end(uint64_t mark) {
    if constexpr (KIND != kNoStep) {
        const Arguments args;
        const AttnArgs& a = args.attn();
        const StepTail<KIND>& t = args.tail<KIND>();
        told::At p{t.step.lens + (size_t)threadIdx.x * a.attn_wgs + blockIdx.x};
        if (threadIdx.x < (unsigned)a.B) told::end(p, t.step.tag, mark);
    }
}

// workgroups of a launch: the attention's, whole rounds over the XCDs, and the others
inline int attn_workgroups(const AttnArgs& a) { return (int)(((long)a.teams + 7) / 8 * 8 * a.mtiles); }
template <StepKind KIND>
inline int rest_of(const AttnArgs& a, StepTail<KIND>& t) {
    if constexpr (KIND == kNoStep) return 0;
    else {
        t.step.heads = heads_of_copier(a.B, a.Hkv, accept::kMostCopiers, a.cus);
        t.step.copiers = copiers_of(a.Hkv, t.step.heads);
        return t.step.scan_wgs + a.B * t.step.copiers;
    }
}

// The attention's workgroups are row 0 of the grid, the others the rows behind it: told apart without waiting for an argument
// (which a kernel would do before it asks for the rest of them: 0.3 us).
inline dim3 launch_grid(const AttnArgs& a, int rest) { return dim3((unsigned)a.attn_wgs, (unsigned)(1 + (rest + a.attn_wgs - 1) / a.attn_wgs)); }

template <parts::Elem E, StepKind KIND>
__device__ __forceinline__ void rest_of_launch(unsigned char* smem) {
    const Arguments args;
    const AttnArgs& a = args.attn();
    const StepTail<KIND>& t = args.tail<KIND>();
    typedef typename std::conditional<E == parts::kF32, float, typename std::conditional<E == parts::kH16, f16_t, bf16_t>::type>::type T;
    accept::Shared& sh = *(accept::Shared*)smem;
    if (threadIdx.x >= accept::kThreads) return;              // (barriers count the waves that are left)
    int wg = (blockIdx.y - 1) * a.attn_wgs + blockIdx.x;
    if (wg < t.step.scan_wgs) {
        accept::scan_or_collect<T, KIND == kStochasticStep, accept::kBesideAttention, 4>(t.accept, t.step, sh, wg);
        return;
    }
    wg -= t.step.scan_wgs;
    if (wg < a.B * t.step.copiers) accept::copy_rows(t.step, t.accept, sh, wg / t.step.copiers, wg % t.step.copiers);      // (the grid's last row is not full)
}

}  // namespace s4c

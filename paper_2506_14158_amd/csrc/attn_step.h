// What an attention launch holds behind its attention workgroups: the merging waves of divided units (attn_parts.h) and, in a
// step's only launch, the rest of the verification step.
//
// A step in one launch (s4c_verify_step).  Acceptance needs nothing of the attention, so its workgroups (accept_roles.h) run beside
// the attention's where those leave places on the chip free, instead of behind them: attention, scan, collectors, merging waves, copiers,
// in this order, each waiting only for workgroups before it.  The appended rows lie behind every key that the attention
// reads; the lengths, which all its workgroups read, are advanced when all of them have said that they have.
// Two launches and one, a whole step, us: fp32, 4 heads, 128 keys + 15 nodes 20.9 and 13.4; 32 heads, 1024 keys + 60 nodes, V 32000
// 22.3 and 16.9; 3 x 8 heads of size 64, 2049 keys 28.1 and 23.4; 4 x 40 heads, 4096 keys 84.3 and 76.6 (merging waves in two turns;
// in one, more workgroups than plan_waiting allows: 74.5).
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

// the first wave, once all waves of the workgroup have the lengths
template <StepKind KIND>
__device__ __forceinline__ void lens_read(const StepTail<KIND>& t, const AttnArgs& a, const work::Lens& lens, long long started) {
    asm volatile("" ::"v"(lens.mine));
    const int lane = threadIdx.x;
    if (lane < a.B) word::publish(t.step.lens + (size_t)lane * a.attn_wgs + blockIdx.x, t.step.tag, started, t.step.copy_ticks);
}

// workgroups of a launch: the attention's, whole rounds over the XCDs, and the others
inline int attn_workgroups(const AttnArgs& a) { return (int)(((long)a.teams + 7) / 8 * 8 * a.mtiles); }
inline int merge_workgroups(const AttnArgs& a, int threads) { return a.tag != 0 ? (parts::tasks(a) + threads / 64 - 1) / (threads / 64) : 0; }
inline int rest_of(AttnArgs& a, StepTail<kNoStep>&, int threads) {
    return a.merge_wgs = plan_waiting(merge_workgroups(a, threads), 0, a.Hkv, 0, a.cus).merging;
}
template <StepKind KIND>
inline int rest_of(AttnArgs& a, StepTail<KIND>& t, int threads) {
    const AttnWaiting w = plan_waiting(merge_workgroups(a, threads), a.B, a.Hkv, accept::kMostCopiers, a.cus);
    a.merge_wgs = w.merging;
    t.step.heads = w.heads;
    t.step.copiers = copiers_of(a.Hkv, w.heads);
    return t.step.scan_wgs + a.merge_wgs + a.B * t.step.copiers;
}

// The attention's workgroups are row 0 of the grid, the others the rows behind it: told apart without waiting for an argument
// (which a kernel would do before it asks for the rest of them: 0.3 us).
inline dim3 launch_grid(const AttnArgs& a, int rest) { return dim3((unsigned)a.attn_wgs, (unsigned)(1 + (rest + a.attn_wgs - 1) / a.attn_wgs)); }

template <int D, parts::Elem E, int THREADS, StepKind KIND>
__device__ __forceinline__ void rest_of_launch(unsigned char* smem) {
    const Arguments args;
    const AttnArgs& a = args.attn();
    int wg = (blockIdx.y - 1) * a.attn_wgs + blockIdx.x;
    if constexpr (KIND != kNoStep) {
        const StepTail<KIND>& t = args.tail<KIND>();
        typedef typename std::conditional<E == parts::kF32, float, typename std::conditional<E == parts::kH16, f16_t, bf16_t>::type>::type T;
        const int merging = a.merge_wgs;
        accept::Shared& sh = *(accept::Shared*)smem;
        const bool scan = wg < t.step.scan_wgs, copy = !scan && wg - t.step.scan_wgs >= merging;
        if (scan || copy) {
            if (threadIdx.x >= accept::kThreads) return;      // (barriers count the waves that are left)
            if (copy && wg - t.step.scan_wgs - merging >= a.B * t.step.copiers) return;          // (the grid's last row is not full)
            if (scan) accept::scan_or_collect<T, KIND == kStochasticStep, accept::kBesideAttention, 4>(t.accept, t.step, sh, wg);
            else {
                wg -= t.step.scan_wgs + merging;
                accept::copy_rows(t.step, t.accept, sh, wg / t.step.copiers, wg % t.step.copiers);
            }
            return;
        }
        wg -= t.step.scan_wgs;
    }
    const int turn = a.merge_wgs * (THREADS / 64), all = parts::tasks(a);
    int task = wg * (THREADS / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (task >= turn) return;                                // (the grid's last row is not full)
    parts::take<D, E, 8>(a, task);
    // (Further turns have code of their own, units of few parts: as turns of one loop they cost the first 0.2 us.)
    if (__builtin_expect(turn < all, 0))
        while ((task += turn) < all) parts::take<D, E, 4>(Arguments().attn(), task);
}

}  // namespace s4c

// The acceptance kernels: accept_roles.h in launches of their own.
#include "accept_roles.h"
#include "attn_parts.h"

namespace s4c {

namespace {

using namespace accept;

template <typename T, bool STOCHASTIC>
__global__ __launch_bounds__(kThreads, kWavesPerSimd<T>) void accept_kernel(AcceptArgs a) {
    __shared__ Shared sh;
    scan_or_collect<T, STOCHASTIC, kAlone, 1>(a, StepArgs{}, sh, blockIdx.x);
}

template <typename T, bool STOCHASTIC>
__global__ __launch_bounds__(kThreads, kWavesPerSimd<T>) void step_kernel(AttnArgs attn, AcceptArgs a, StepArgs x) {
    __shared__ Shared sh;
    int wg = blockIdx.x;
    if (wg < x.scan_wgs) {
        scan_or_collect<T, STOCHASTIC, kBehindAttention, 1>(a, x, sh, wg);
        return;
    }
    wg -= x.scan_wgs;
    if (wg < x.merge_wgs) {
        if (attn.split > 0) {
            constexpr parts::Elem E = sizeof(T) == 4 ? parts::kF32 : std::is_same<T, f16_t>::value ? parts::kH16 : parts::kB16;
            const int task = wg * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
            if (attn.D == 64) parts::take_task<64, E, 3>(attn, task);
            else parts::take_task<128, E, 3>(attn, task);
            return;
        }
        const int unit = wg / x.merge_chunks, chunk = wg - unit * x.merge_chunks;
        if (attn.D == 64) merge::merge_rows<T, 64>(attn, unit, chunk, x.merge_passes);
        else merge::merge_rows<T, 128>(attn, unit, chunk, x.merge_passes);
        return;
    }
    wg -= x.merge_wgs;
    copy_rows(x, a, sh, wg / x.copiers, wg % x.copiers);
}

}  // namespace

int accept_chunk_elems() { return kChunk; }

// Segments by which the acceptance workspace is sized (scan_plan): up to 8 chunks of a row, fewer when that would leave less
// than about 1024 workgroups to spread over the chip.
void accept_plan(int B, int N, int V, int* seg, int* nseg) {
    const long long ch = ((long long)V + kChunk - 1) / kChunk;
    const long long units = (long long)B * N * ch;
    long long sg = units / 1024;
    if (sg > 8) sg = 8;
    if (sg > ch) sg = ch;
    if (sg < 1) sg = 1;
    *seg = (int)sg;
    *nseg = (int)((ch + sg - 1) / sg);
}

// A run is at least `seg` chunks long, so that a row's records take no more room than the three words that the workspace
// has for each segment of accept_plan.  A row's chunks lie in at most ceil(chunks / seg) + 1 runs; where seg is
// a whole row, runs are made of whole rows.
AcceptPlan scan_plan(int B, int N, int V, int elem_bytes, int cus) {
    int seg, nseg;
    accept_plan(B, N, V, &seg, &nseg);
    AcceptPlan p;
    p.chunks = (int)(((long long)V + 7 + kChunk - 1) / kChunk);          // a row may begin up to 7 elements into its first vector
    auto slots = [&](int sg) { return sg >= p.chunks ? 1 : sg == 1 ? p.chunks : (p.chunks + sg - 1) / sg + 1; };
    while (2 * slots(seg) > 3 * nseg) ++seg;
    p.seg = seg;
    p.slots = slots(seg);
    const long long resident = (long long)cus * (elem_bytes == 4 ? kWavesPerSimd<float> : kWavesPerSimd<bf16_t>);
    const long long runs = (long long)N * p.chunks / seg;
    long long wgs = resident / B;
    if (wgs > runs) wgs = runs;
    p.wgs = (int)(wgs < 1 ? 1 : wgs);
    return p;
}

template <typename T>
static hipError_t launch_accept_as(const AcceptArgs& a, hipStream_t st) {
    const dim3 grid((unsigned)((a.plan.wgs + 1) * a.B)), block(kThreads);
    if (a.mode == S4C_STOCHASTIC) hipLaunchKernelGGL((accept_kernel<T, true>), grid, block, 0, st, a);
    else hipLaunchKernelGGL((accept_kernel<T, false>), grid, block, 0, st, a);
    return hipGetLastError();
}
hipError_t launch_accept(const AcceptArgs& a, hipStream_t st) {
    static_assert(kThreads >= 2 * 64 && kThreads >= kMaxNodes, "the path step and the row lookup use one thread per node");
    return a.dtype == S4C_F32 ? launch_accept_as<float>(a, st) : a.dtype == S4C_F16 ? launch_accept_as<f16_t>(a, st) : launch_accept_as<bf16_t>(a, st);
}

template <typename T>
static hipError_t launch_step_as(const AttnArgs& attn, const AcceptArgs& a, const StepArgs& x, hipStream_t st) {
    const dim3 grid((unsigned)(x.merge_wgs + x.scan_wgs + a.B * x.copiers)), block(kThreads);
    if (a.mode == S4C_STOCHASTIC) hipLaunchKernelGGL((step_kernel<T, true>), grid, block, 0, st, attn, a, x);
    else hipLaunchKernelGGL((step_kernel<T, false>), grid, block, 0, st, attn, a, x);
    return hipGetLastError();
}

// up to kMostCopiers per sequence, whole KV heads each
size_t step_message_bytes(int B, int Hkv) {
    return (size_t)B * (Hkv < kMostCopiers ? Hkv : kMostCopiers) * kMessageWords * sizeof(rec_t);
}

hipError_t launch_step(const AttnArgs& attn, const AcceptArgs& a, const CompactArgs& compact, unsigned long long* messages,
                       long long copy_ticks, hipStream_t st) {
    StepArgs x = make_step(a, compact, messages, copy_ticks);
    if (attn.split > 1) {
        x.merge_wgs = (parts::tasks(attn) + 3) / 4;
    } else if (attn.split == 0) {
        const merge::Grid g = merge::grid_of(attn);
        x.merge_wgs = g.units * g.chunks;
        x.merge_chunks = g.chunks;
        x.merge_passes = g.passes;
    }
    return a.dtype == S4C_F32 ? launch_step_as<float>(attn, a, x, st) : a.dtype == S4C_F16 ? launch_step_as<f16_t>(attn, a, x, st)
                                                                                          : launch_step_as<bf16_t>(attn, a, x, st);
}

}  // namespace s4c

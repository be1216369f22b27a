// P2/P4 (FFT along b) kernels, FP64: one per radix plan of HARTREE_PLANS plus the run-time
// radix kernel (one translation unit per pass and precision so the build
// compiles them in parallel), and per plan kernels for tiles of 8 pencils with
// no pitch pad, whose tile shape is compiled in.
#include "fft_runtime.hpp"

namespace hartree {
namespace {
template <int R0, int R1, int R2, int R3>
hipError_t launch_one(int grid, size_t lds, hipStream_t s, const PassArgs &a)
{
    return launch_pass(k_fft_b<double, R0, R1, R2, R3>, grid, lds, s, a);
}
template <int R0, int R1, int R2, int R3>
hipError_t launch_fixed8(int grid, size_t lds, hipStream_t s, const PassArgs &a)
{
    constexpr int NT = threads8<double>(1, plan_length(R0, R1, R2, R3));
    return launch_pass(k_fft_b<double, R0, R1, R2, R3, 8, NT>, grid, lds, s, a, NT);
}
#define HARTREE_ENTRY(R0, R1, R2, R3) &launch_one<R0, R1, R2, R3>,
const PassLaunchFn kTable[] = {HARTREE_PLANS(HARTREE_ENTRY)};
#undef HARTREE_ENTRY
#define HARTREE_ENTRY(R0, R1, R2, R3) &launch_fixed8<R0, R1, R2, R3>,
const PassLaunchFn kFixed8[] = {HARTREE_PLANS(HARTREE_ENTRY)};
#undef HARTREE_ENTRY
}  // namespace

hipError_t run_b_f64(int plan, int maxn, int grid, hipStream_t s, const PassArgs &a)
{
    const size_t lds = pass_lds_bytes<double>(a, maxn);
    if (plan == kMultiPlan) return hipErrorInvalidValue;  // multi-plan launches are FP32 only
    if (plan < 0 || plan >= int(sizeof(kTable) / sizeof(kTable[0])))
        return launch_b_rt<double>(plan == kRuntimeWide, maxn, grid, s, a);
    if (a.pad == 0 && a.p_log2 == 3 && lane_offsets_fit<double>(a, threads8<double>(1, maxn)))
        return kFixed8[plan](grid, lds, s, a);
    return kTable[plan](grid, lds, s, a);
}
}  // namespace hartree

// P2/P4 (FFT along b) kernels, FP32: one per radix plan of HARTREE_PLANS plus the run-time
// radix kernel (one translation unit per pass and precision so the build
// compiles them in parallel), and per plan kernels for tiles of 4, 8 and 16
// pencils with no pitch pad, whose tile shape is compiled in.
#include "fft_runtime.hpp"

namespace hartree {
namespace {
template <int R0, int R1, int R2, int R3, int CP>
hipError_t launch_one(int grid, size_t lds, hipStream_t s, const PassArgs &a)
{
    return launch_pass(k_fft_b<float, R0, R1, R2, R3, CP>, grid, lds, s, a);
}
template <int R0, int R1, int R2, int R3>
hipError_t launch_fixed8(int grid, size_t lds, hipStream_t s, const PassArgs &a)
{
    constexpr int NT = threads8<float>(1, plan_length(R0, R1, R2, R3));
    return launch_pass(k_fft_b<float, R0, R1, R2, R3, 8, NT>, grid, lds, s, a, NT);
}
#define HARTREE_ENTRY(R0, R1, R2, R3) &launch_one<R0, R1, R2, R3, 0>,
const PassLaunchFn kTable[] = {HARTREE_PLANS(HARTREE_ENTRY)};
#undef HARTREE_ENTRY
#define HARTREE_ENTRY(R0, R1, R2, R3) &launch_one<R0, R1, R2, R3, 4>,
const PassLaunchFn kFixed4[] = {HARTREE_PLANS(HARTREE_ENTRY)};
#undef HARTREE_ENTRY
#define HARTREE_ENTRY(R0, R1, R2, R3) &launch_fixed8<R0, R1, R2, R3>,
const PassLaunchFn kFixed8[] = {HARTREE_PLANS(HARTREE_ENTRY)};
#undef HARTREE_ENTRY
#define HARTREE_ENTRY(R0, R1, R2, R3) &launch_one<R0, R1, R2, R3, 16>,
const PassLaunchFn kFixed16[] = {HARTREE_PLANS(HARTREE_ENTRY)};
#undef HARTREE_ENTRY
}  // namespace

hipError_t run_b_f32(int plan, int maxn, int grid, hipStream_t s, const PassArgs &a)
{
    const size_t lds = pass_lds_bytes<float>(a, maxn);
    if (plan == kMultiPlan) {
        if (a.p_log2 == multi_log_p(1, 0))
            return launch_pass(k_fft_b_multi<float, 1 << multi_log_p(1, 0)>, grid, lds, s, a);
        if (a.p_log2 == multi_log_p(1, 1))
            return launch_pass(k_fft_b_multi<float, 1 << multi_log_p(1, 1)>, grid, lds, s, a);
        if (a.p_log2 == kMultiAutoLog)
            return launch_pass(k_fft_b_multi<float, 0>, grid, multi_auto_lds<float>(1, maxn), s, a);
        return hipErrorInvalidValue;
    }
    if (plan < 0 || plan >= int(sizeof(kTable) / sizeof(kTable[0])))
        return launch_b_rt<float>(plan == kRuntimeWide, maxn, grid, s, a);
    // the compiled tiles address their pencils with 32-bit lane offsets
    if (a.pad == 0 && lane_offsets_fit<float>(a, a.p_log2 == 3 ? threads8<float>(1, maxn) : kPassThreads)) {
        if (a.p_log2 == 2) return kFixed4[plan](grid, lds, s, a);
        if (a.p_log2 == 3) return kFixed8[plan](grid, lds, s, a);
        if (a.p_log2 == 4) return kFixed16[plan](grid, lds, s, a);
    }
    return kTable[plan](grid, lds, s, a);
}
}  // namespace hartree

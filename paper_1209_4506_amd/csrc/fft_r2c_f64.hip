// P1 (r2c along c) kernels, FP64: one per radix plan of HARTREE_PLANS plus the run-time
// radix kernel (one translation unit per pass and precision so the build
// compiles them in parallel).
#include "fft_runtime.hpp"

namespace hartree {
namespace {
template <int R0, int R1, int R2, int R3>
hipError_t launch_one(int grid, size_t lds, hipStream_t s, const PassArgs &a)
{
    // forward: rho.  Backward (mode 1): grad_v + s rho, grad_v alone (no
    // grad_e), or s rho alone (no grad_v); the host never passes neither.
    if (a.mode == 0 || a.grad_e == nullptr) return launch_pass(k_r2c_mode<double, 0, R0, R1, R2, R3>, grid, lds, s, a);
    if (a.in != nullptr) return launch_pass(k_r2c_mode<double, 1, R0, R1, R2, R3>, grid, lds, s, a);
    return launch_pass(k_r2c_mode<double, 2, R0, R1, R2, R3>, grid, lds, s, a);
}
#define HARTREE_ENTRY(R0, R1, R2, R3) &launch_one<R0, R1, R2, R3>,
const PassLaunchFn kTable[] = {HARTREE_PLANS(HARTREE_ENTRY)};
#undef HARTREE_ENTRY
}  // namespace

hipError_t run_r2c_f64(int plan, int maxn, int grid, hipStream_t s, const PassArgs &a)
{
    const size_t lds = pass_lds_bytes<double>(a, maxn);
    if (plan == kMultiPlan) return hipErrorInvalidValue;  // multi-plan launches are FP32 only
    if (plan < 0 || plan >= int(sizeof(kTable) / sizeof(kTable[0])))
        return launch_r2c_rt<double>(plan == kRuntimeWide, maxn, grid, s, a);
    return kTable[plan](grid, lds, s, a);
}
}  // namespace hartree

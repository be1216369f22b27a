// P3 (fused FFT along a) kernels, FP64: one per radix plan of HARTREE_PLANS plus the run-time
// radix kernel (one translation unit per pass and precision so the build
// compiles them in parallel), and per plan kernels for tiles of 4 and 8
// pencils with no pitch pad, whose tile shape is compiled in: the pass is short
// of wavefronts (170 registers and more, two per SIMD), and without the strides
// and bounds a kernel needs 96 to 157.  192^3: 38 -> 29 us a pass; 300^3: 119 ->
// 90; 600^3: 1,366 -> 901; 360^3 as 10 x 6 x 6 with 4 pencils: 219 -> 194 (a copy
// of its bytes: 145).  (Along b, 120 registers as it is, the same gave 0 to 2 %.)
#include "fft_runtime.hpp"

namespace hartree {
namespace {
template <int R0, int R1, int R2, int R3>
hipError_t launch_one(int grid, size_t lds, hipStream_t s, const PassArgs &a)
{
    return launch_pass(k_fft_a<double, R0, R1, R2, R3>, grid, lds, s, a);
}
#define HARTREE_ENTRY(R0, R1, R2, R3) &launch_one<R0, R1, R2, R3>,
const PassLaunchFn kTable[] = {HARTREE_PLANS(HARTREE_ENTRY)};
#undef HARTREE_ENTRY
template <int R0, int R1, int R2, int R3, int CP>
hipError_t launch_fixed(int grid, size_t lds, hipStream_t s, const PassArgs &a)
{
    return launch_pass(k_fft_a<double, R0, R1, R2, R3, CP>, grid, lds, s, a);
}
#define HARTREE_ENTRY(R0, R1, R2, R3) &launch_fixed<R0, R1, R2, R3, 4>,
const PassLaunchFn kFixed4[] = {HARTREE_PLANS(HARTREE_ENTRY)};
#undef HARTREE_ENTRY
#define HARTREE_ENTRY(R0, R1, R2, R3) &launch_fixed<R0, R1, R2, R3, 8>,
const PassLaunchFn kFixed8[] = {HARTREE_PLANS(HARTREE_ENTRY)};
#undef HARTREE_ENTRY
}  // namespace

hipError_t run_a_f64(int plan, int maxn, int grid, hipStream_t s, const PassArgs &a)
{
    const size_t lds = pass_lds_bytes<double>(a, maxn);
    if (plan == kMultiPlan) return hipErrorInvalidValue;  // multi-plan launches are FP32 only
    if (plan < 0 || plan >= int(sizeof(kTable) / sizeof(kTable[0])))
        return launch_a_rt<double>(plan == kRuntimeWide, maxn, grid, s, a);
    // the compiled tiles address their pencils with 32-bit lane offsets
    if (a.pad == 0 && lane_offsets_fit<double>(a)) {
        if (a.p_log2 == 2) return kFixed4[plan](grid, lds, s, a);
        if (a.p_log2 == 3) return kFixed8[plan](grid, lds, s, a);
    }
    return kTable[plan](grid, lds, s, a);
}
}  // namespace hartree

// Device helpers shared by the splat kernels (binning, VALU and MFMA forms).
#pragma once

#include "fft_core.hpp"
#include "kernels.hpp"

namespace hartree {

// The last p < n whose start(p) is at or below v, for starts that do not
// decrease with p and start(0) <= v: the number of q in [1, n) with
// start(q) <= v.  v is the same in every lane and every lane is active:
// lane l compares start(q) for q = 1 + l, 65 + l, ..., so the lookup costs
// one load per 64 problems instead of a chain of dependent loads.
template <class Start>
__device__ __forceinline__ int wave_find(int n, int64_t v, Start start)
{
    const int lane = threadIdx.x & 63;
    int p = 0;
    for (int q0 = 1; q0 < n; q0 += 64) {
        const int q = q0 + lane;
        const bool le = q < n && start(q) <= v;
        p += __popcll(__ballot(le));
    }
    return __builtin_amdgcn_readfirstlane(p);
}

// the problem of an atom (atom_off ascending); callers hold the atom index
// in every lane with the whole wavefront active
__device__ __forceinline__ int find_prob_atom(const SplatArgs &a, int atom)
{
    return wave_find(a.nprob, atom, [&](int q) { return int64_t(a.atom_off[q]); });
}

__device__ __forceinline__ int wrapi(int i, int n)
{
    int r = i % n;
    return r < 0 ? r + n : r;
}

// bricks touched along one axis: circular range [start, start + count) mod nb
__device__ __forceinline__ void axis_bricks(int lo, int hi, int n, int bsz, int nb, int &start, int &count)
{
    if (hi < lo) {  // invalid atom: touches nothing
        start = 0;
        count = 0;
        return;
    }
    if (hi - lo + 1 >= n) {
        start = 0;
        count = nb;
        return;
    }
    const int s = wrapi(lo, n), e = wrapi(hi, n);
    const int bs = s / bsz, be = e / bsz;
    start = bs;
    if (s <= e)
        count = be - bs + 1;
    else
        count = (be >= bs) ? nb : (nb - bs) + be + 1;
}

// bricks touched by an atom along each axis
__device__ __forceinline__ void atom_bricks(const AtomInfo &in, const ProbDesc &d, int *st, int *ct)
{
    for (int x = 0; x < 3; ++x) axis_bricks(in.lo[x], in.hi[x], d.dims[x], d.bsz[x], d.nbricks[x], st[x], ct[x]);
}

// the problem of a brick (brick_off ascending), by bisection over the
// problems: a chain of scalar loads, which the scalar cache serves to every
// wavefront of the long splat kernels
__device__ __forceinline__ int brick_prob(const SplatArgs &a, int64_t b)
{
    int lo = 0, hi = a.nprob - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (b >= a.desc[mid].brick_off) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// the same by one vector load and a ballot, for the short binning kernels
// whose wavefronts are load chains; callers hold the brick index in every
// lane with the whole wavefront active
__device__ __forceinline__ int brick_prob_wave(const SplatArgs &a, int64_t b)
{
    return wave_find(a.nprob, b, [&](int q) { return a.desc[q].brick_off; });
}

// brick index of this workgroup: from the binning's work order where there
// is one (batched plans: bricks by descending atom count), else with
// consecutive bricks (which share cache lines at their edges along c) kept
// on one XCD
__device__ __forceinline__ int64_t brick_of_block(const SplatArgs &a)
{
    if (a.order) return a.order[blockIdx.x];
    return xcd_remap(blockIdx.x, gridDim.x);
}

// A brick's position (brick index per axis), kept in registers
struct BrickPos {
    int b0, b1, b2;
};

__device__ __forceinline__ BrickPos brick_pos(const ProbDesc &d, int64_t b)
{
    const int lb = int(b - d.brick_off);  // bricks of one problem fit 32 bits
    BrickPos p;
    p.b2 = lb % d.nbricks[2];
    const int bij = lb / d.nbricks[2];
    p.b1 = bij % d.nbricks[1];
    p.b0 = bij / d.nbricks[1];
    return p;
}

// exp(x): x = n ln 2 + r, |r| <= ln 2 / 2, exp(r) by its Taylor series to
// r^13 / 13! (the next term is 4e-18).  Without the library's range checks and
// branches: 2^n underflows to 0 and overflows by itself.  The coefficients are
// read from memory, so that they stay in scalar registers; ln 2 is split in
// 2^-40 floor(2^40 ln 2 + 1/2) and the rest, so that n times the first is exact.
static __constant__ double kExp[17] = {
    1.0 / 0.69314718055994530942, -762123384786.0 / 1099511627776.0, 1.7239444525614835e-13,
    1.0 / 6227020800.0, 1.0 / 479001600.0, 1.0 / 39916800.0, 1.0 / 3628800.0, 1.0 / 362880.0, 1.0 / 40320.0,
    1.0 / 5040.0, 1.0 / 720.0, 1.0 / 120.0, 1.0 / 24.0, 1.0 / 6.0, 0.5, 1.0, 1.0};
// The exponent as the instruction converts it: saturated, so that 2^n is 0 and
// infinity for any x (a conversion of the language's is undefined beyond 2^31, from
// |x| = 1.5e9 on, cutoffs of 5.5e4 sigmas; this costs 0.5 %, a bound on x 1.4 % of the
// FP64 splat and adjoint).
__device__ __forceinline__ int exponent64(double n)
{
    int i;
    asm("v_cvt_i32_f64 %0, %1" : "=v"(i) : "v"(n));
    return i;
}
__device__ __forceinline__ double exp64(double x)
{
    const double n = __builtin_rint(x * kExp[0]);
    const double r = __builtin_fma(n, kExp[2], __builtin_fma(n, kExp[1], x));
    double e = kExp[3];
#pragma unroll
    for (int k = 4; k < 17; ++k) e = __builtin_fma(e, r, kExp[k]);
    return __builtin_ldexp(e, exponent64(n));
}
// exp(x) and exp(-x): one reduction, and the series' even and odd terms once
__device__ __forceinline__ void exp64_pair(double x, double &plus, double &minus)
{
    const double n = __builtin_rint(x * kExp[0]);
    const double r = __builtin_fma(n, kExp[2], __builtin_fma(n, kExp[1], x));
    const double r2 = r * r;
    double odd = kExp[3], even = kExp[4];
#pragma unroll
    for (int k = 5; k < 17; k += 2) {
        odd = __builtin_fma(odd, r2, kExp[k]);
        even = __builtin_fma(even, r2, kExp[k + 1]);
    }
    plus = __builtin_ldexp(__builtin_fma(r, odd, even), exponent64(n));
    minus = __builtin_ldexp(__builtin_fma(-r, odd, even), exponent64(-n));
}

}  // namespace hartree

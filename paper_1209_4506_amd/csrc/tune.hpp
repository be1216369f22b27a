// What hartree_plan_tune may choose among.
//
// In FP32 the radix plans of a length round differently, and so do some tile
// shapes of one plan: the compiler orders the sums of each kernel's
// butterflies by itself.  Timings repeat to a few per cent only, so if they
// decided between such choices, tuning a plan again could give other values
// (as timed, 360 along a took 12 x 5 x 6 in 14 of 18 tunings and 12 x 6 x 5 in
// 4; E_H 2e-7 apart).  The tuner therefore times, per axis and length, only
// choices that give the same values bit for bit: one radix plan, and of its
// tiles those that agree with the ones it takes on most grids.  (In FP64
// they differ by 1e-16; every choice is timed.)  Host code without HIP.
#pragma once

namespace hartree {

// The FP32 radix plan (index in HARTREE_PLANS) of the lengths that have
// several, along axis x (0 = a, 1 = b, 2 = c); -1: the length's only one.
// Measured (us, the best of 4 to 16 pencils; b forward + inverse, c r2c + c2r;
// the other two lengths 240, beside 180 180): 48 a 1 13.7, 41 14.6 (48^3 7.3,
// 6.9); c 28.7, 23.4.  128 a 8 19.3, 42 19.9; b 28.5, 29.1; c 41.3, 33.4.
// 160 a 10 22.8, 43 24.5; b 34.0, 36.5; c 50.7, 46.6.  180 a 11 19.1, 39 18.7,
// 40 18.8; b 27.7, 27.4, 26.0; c 33.0, 29.2, 29.9.  360: 44 and 45 are within
// 1 % along a, 44 is the fastest along b and 38 along c.
constexpr int tuned_plan(int x, int n)
{
    switch (n) {
    case 48: return 41;
    case 128: return x == 2 ? 42 : 8;
    case 160: return x == 2 ? 43 : 10;
    case 180: return x == 2 ? 39 : 40;
    case 360: return x == 2 ? 38 : 44;
    default: return -1;
    }
}

// The FP32 tiles (2^p_log2 pencils, pitch pad) of a compiled radix plan.
// Along a and b up to 256 the kernels with 8 and 16 pencils compiled in,
// which are the fastest or within 3 % of it; they differ from the general kernel
// at 32, 48, 64, 72, 90, 96, 120, 128, 160 and 256, and from each other at 96
// along a.  Above 256 all but those with 4 at 320 and 512 and 16 at 512.  Along c
// all up to 256; 8 pencils differ at 288, 320, 360, 400 and 420 (2 and 4 are
// faster there), and 4 from 2 from 512 on.
constexpr bool tuned_tile(int x, int n, int p_log2, int pad)
{
    if (x == 2) {
        if (n >= 576) return p_log2 == 1;
        if (n == 512) return p_log2 == 2 || p_log2 == 3;
        return n <= 256 || p_log2 != 3 || n == 300 || n == 384 || n == 480;
    }
    if (n <= 256) return pad == 0 && (p_log2 == 3 || (p_log2 == 4 && !(x == 0 && n == 96)));
    const bool four = p_log2 == 2 && pad == 0 && (n == 320 || n == 512);
    return !four && !(p_log2 == 4 && pad == 0 && n == 512);
}

// whether the tuner times a choice (plan: index in HARTREE_PLANS, or -1 for
// the run-time radix kernels, which give the same values in every tile)
constexpr bool tune_times(int fp64, int x, int n, int plan, int p_log2, int pad)
{
    if (fp64 || plan < 0) return true;
    return (tuned_plan(x, n) < 0 || tuned_plan(x, n) == plan) && tuned_tile(x, n, p_log2, pad);
}

// Multi-plan launches (FP32 batches): lengths at which the tiles sized per
// length (32 and 64 pencils along c and 64 along a) or the fixed ones differ
// from the others.  A batch that holds one of them takes the sized tiles,
// which are the fastest for most mixes of lengths.
constexpr bool multi_sized_only(int x, int n)
{
    return x == 2 ? n == 60 || n == 64 || n == 128 : x == 0 && (n == 64 || n == 96);
}

}  // namespace hartree

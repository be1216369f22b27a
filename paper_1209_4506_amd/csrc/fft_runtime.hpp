// The grid passes with the stage radices taken at run time: the kernels of
// every length that has no compiled plan.
//
// The LDS holds the tile twice: each stage reads one copy and writes the
// other, one butterfly at a time, so a stage needs one barrier and the
// registers of one butterfly (plans with a radix-16 stage have kernels of
// their own, WIDE, so that the others need 64 to 110 registers in FP32).  A
// single copy instead needs every value of a stage in registers between its
// reads and its writes, whatever the radices: 256 registers, two wavefronts
// per SIMD.  135 x 168 x 189 FP32: r2c 71 -> 12, b 21 -> 8, a 46 -> 18, inverse b
// 26 -> 12, c2r 66 -> 9 us; the solve 252 -> 74 us.
//
// Along c the butterflies of all pencils of a tile are dealt to the threads
// together (short pencils leave no lane idle between them); along a and b a
// thread keeps one pencil, so that a wavefront moves whole runs of P
// consecutive values.
#pragma once

#include "fft_passes.hpp"

namespace hartree {

// The rounding of the transforms is part of the library's results: which
// product of a complex multiplication is rounded before the sum is fused
// would otherwise be the compiler's choice, made anew for each kernel.  The
// constant multiplications inside a first stage's butterflies (radices 8, 9
// and 16) therefore spell it out, and a stage's inputs are settled: opaque
// to the compiler, so that it contracts nothing across them.

// a (c - i s), the products of a.x rounded (Y_ROUNDED: in the imaginary part that of a.y)
template <typename T, bool Y_ROUNDED = false>
__device__ __forceinline__ Cx<T> turn(Cx<T> a, T c, T s)
{
    return Cx<T>{__builtin_fma(a.y, s, a.x * c), Y_ROUNDED ? __builtin_fma(-a.x, s, a.y * c) : __builtin_fma(a.y, c, -(a.x * s))};
}
template <>
__device__ __forceinline__ Cx<float> turn<float, false>(Cx<float> a, float c, float s)
{
    return Cx<float>{__builtin_fmaf(a.y, s, a.x * c), __builtin_fmaf(a.y, c, -(a.x * s))};
}
template <>
__device__ __forceinline__ Cx<float> turn<float, true>(Cx<float> a, float c, float s)
{
    return Cx<float>{__builtin_fmaf(a.y, s, a.x * c), __builtin_fmaf(-a.x, s, a.y * c)};
}

// radix A B (see dft_product)
template <typename T, int A, int B>
__device__ __forceinline__ void first_product(Cx<T> *x)
{
    constexpr int R = A * B;
    Cx<T> y[R];
#pragma unroll
    for (int n2 = 0; n2 < B; ++n2) {
        Cx<T> t[A];
#pragma unroll
        for (int n1 = 0; n1 < A; ++n1) t[n1] = x[B * n1 + n2];
        butterfly<T, A, false>(t);
#pragma unroll
        for (int k1 = 0; k1 < A; ++k1) {
            const int e = n2 * k1;
            const T c = T(unit_cos(R, e)), s = T(unit_sin(R, e));
            if (e == 0) y[k1 * B + n2] = t[k1];
            else if (R == 16 && e == 9) y[k1 * B + n2] = turn<T, true>(t[k1], c, s);
            else y[k1 * B + n2] = turn<T>(t[k1], c, s);
        }
    }
#pragma unroll
    for (int k1 = 0; k1 < A; ++k1) {
        Cx<T> t[B];
#pragma unroll
        for (int n2 = 0; n2 < B; ++n2) t[n2] = y[k1 * B + n2];
        butterfly<T, B, false>(t);
#pragma unroll
        for (int k2 = 0; k2 < B; ++k2) x[k1 + A * k2] = t[k2];
    }
}

// which stage a butterfly belongs to: its constant multiplications round as
// written for a first one, as the compiler contracts them for the others, and
// the radix-8 ones of the last stage along c (C2R) round every product of the
// imaginary part
enum RtForm { RT_FIRST, RT_MID, RT_LAST_C2R };

template <typename T, bool FUSED>
__device__ __forceinline__ Cx<T> turn8(Cx<T> a, T c, T s)
{
    if constexpr (FUSED) {
        return turn<T>(a, c, s);
    } else {
        T yc = a.y * c, xs = a.x * s, ys = a.y * s;
        asm("" : "+v"(yc), "+v"(xs), "+v"(ys));
        if constexpr (sizeof(T) == 4) return Cx<T>{__builtin_fmaf(a.x, c, ys), yc - xs};
        else return Cx<T>{__builtin_fma(a.x, c, ys), yc - xs};
    }
}

template <typename T, int R, RtForm FORM>
__device__ __forceinline__ void rt_dft(Cx<T> *a)
{
    if constexpr (FORM == RT_MID || (FORM == RT_LAST_C2R && R != 8)) {
        butterfly<T, R, false>(a);
    } else if constexpr (R == 8) {
        constexpr bool FUSED = FORM == RT_FIRST;
        constexpr T h = T(0.7071067811865475244008443621048490392848);
        Cx<T> e[4], f[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            e[q] = cadd(a[q], a[q + 4]);
            f[q] = csub(a[q], a[q + 4]);
        }
        f[1] = turn8<T, FUSED>(f[1], h, h);
        f[2] = rot<T, false>(f[2]);
        f[3] = turn8<T, FUSED>(f[3], -h, h);
        dft4<T, false>(e[0], e[1], e[2], e[3]);
        dft4<T, false>(f[0], f[1], f[2], f[3]);
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            a[2 * m] = e[m];
            a[2 * m + 1] = f[m];
        }
    } else if constexpr (R == 9) {
        first_product<T, 3, 3>(a);
    } else if constexpr (R == 16) {
        first_product<T, 4, 4>(a);
    } else {
        butterfly<T, R, false>(a);
    }
}

template <typename T>
__device__ __forceinline__ void settle(Cx<T> &v)
{
    asm("" : "+v"(v.x), "+v"(v.y));
}

// Butterfly j of a stage of radix R: src(i) loads element i of the pencil,
// dst(i, v) stores it.  ns: product of the earlier radices; ins: 1 / ns.
template <typename T, int R, RtForm FORM, typename Src, typename Dst>
__device__ __forceinline__ void rt_butterfly(const Src &src, const Dst &dst, const Cx<T> *tw, int j, int nb, int ns,
                                             float ins, int tws)
{
    Cx<T> v[R];
#pragma unroll
    for (int q = 0; q < R; ++q) v[q] = src(j + q * nb);
#pragma unroll
    for (int q = 0; q < R; ++q) settle(v[q]);
    int base = j * R;
    if constexpr (FORM != RT_FIRST) {
        // j / ns, exact: j < 4096 and the half keeps the quotient clear of whole numbers
        const int jd = int((float(j) + 0.5f) * ins);
        const int k = j - __mul24(jd, ns);
        const int step = __mul24(k, tws);
        int at = step;
#pragma unroll
        for (int q = 1; q < R; ++q, at += step) v[q] = cmul(v[q], tw[at]);
        base = __mul24(jd, ns * R) + k;
    }
    rt_dft<T, R, FORM>(v);
#pragma unroll
    for (int q = 0; q < R; ++q) dst(base + q * ns, v[q]);
}

// how a tile's butterflies are dealt to the 256 threads: f(pencil, butterfly)
struct RtStrided {
    int p, tip, tpp;
    template <typename F>
    __device__ __forceinline__ void each(int nb, F &&f) const
    {
#pragma unroll 1
        for (int j = tip; j < nb; j += tpp) f(p, j);
    }
};
struct RtRows {
    int pencils;
    template <typename F>
    __device__ __forceinline__ void each(int nb, F &&f) const
    {
        const float inb = 1.0f / float(nb);
#pragma unroll 1
        for (int e = threadIdx.x; e < pencils * nb; e += kPassThreads) {
            const int p = int((float(e) + 0.5f) * inb);  // exact: e < 2^16
            f(p, e - __mul24(p, nb));
        }
    }
};

// stage s of the plan: src(p, i) to dst(p, i, v)
template <typename T, bool WIDE, RtForm FORM, typename It, typename Src, typename Dst>
__device__ __forceinline__ void rt_stage(const It &it, const AxisPlan &ap, int s, const Cx<T> *tw, const Src &src,
                                         const Dst &dst)
{
    const int r = ap.radix[s], ns = int(ap.ns[s].d), tws = ap.twstride[s];
    const float ins = 1.0f / float(ns);
#define HARTREE_STAGE(RR)                                                                                        \
    case RR: {                                                                                                   \
        const int nb = ap.n / RR;                                                                                \
        it.each(nb, [&](int p, int j) {                                                                          \
            rt_butterfly<T, RR, FORM>([&](int i) { return src(p, i); }, [&](int i, Cx<T> v) { dst(p, i, v); }, \
                                       tw, j, nb, ns, ins, tws);                                                 \
        });                                                                                                      \
        break;                                                                                                   \
    }
    switch (r) {
        HARTREE_STAGE(2)
        HARTREE_STAGE(3)
        HARTREE_STAGE(4)
        HARTREE_STAGE(5)
        HARTREE_STAGE(7)
        HARTREE_STAGE(8)
        HARTREE_STAGE(9)
        HARTREE_STAGE(10)
    case 16:
        if constexpr (WIDE) {
            const int nb = ap.n / 16;
            it.each(nb, [&](int p, int j) {
                rt_butterfly<T, 16, FORM>([&](int i) { return src(p, i); }, [&](int i, Cx<T> v) { dst(p, i, v); }, tw, j,
                                          nb, ns, ins, tws);
            });
        }
        break;
    default: break;  // not produced by the plan search
    }
#undef HARTREE_STAGE
}

// The forward transform of a tile (conjugating src and dst make it the
// inverse): stage s writes copy (first + s) & 1 of the tile, the last one
// dst.  at(p, i): offset of element i of pencil p within a copy.  On return
// every thread has written its share; the caller synchronizes.
template <typename T, bool WIDE, RtForm LAST = RT_MID, typename It, typename At, typename Src, typename Dst>
__device__ __forceinline__ void rt_fft(const It &it, const AxisPlan &ap, const Cx<T> *tw, Cx<T> *tile, int copy, int first,
                                       const At &at, const Src &src, const Dst &dst)
{
    const int S = ap.nstages;
    if (S == 1) {
        rt_stage<T, WIDE, RT_FIRST>(it, ap, 0, tw, src, dst);
        return;
    }
    Cx<T> *to = tile + (first & 1) * copy, *from = tile + (~first & 1) * copy;
    rt_stage<T, WIDE, RT_FIRST>(it, ap, 0, tw, src, [&](int p, int i, Cx<T> v) { to[at(p, i)] = v; });
    __syncthreads();
    for (int s = 1; s + 1 < S; ++s) {
        Cx<T> *x = to;
        to = from;
        from = x;
        rt_stage<T, WIDE, RT_MID>(
            it, ap, s, tw, [&](int p, int i) { return from[at(p, i)]; }, [&](int p, int i, Cx<T> v) { to[at(p, i)] = v; });
        __syncthreads();
    }
    rt_stage<T, WIDE, LAST>(it, ap, S - 1, tw, [&](int p, int i) { return to[at(p, i)]; }, dst);
}

// the twiddle table: in LDS after the two copies, or (TWG: the copies fill
// the LDS) read from global memory
template <typename T, bool TWG>
__device__ __forceinline__ const Cx<T> *rt_twiddles(const PassArgs &a, const AxisPlan &ap, Cx<T> *lds, int tid)
{
    const Cx<T> *g = reinterpret_cast<const Cx<T> *>(a.tw) + ap.tw_off;
    if constexpr (TWG) {
        return g;
    } else {
        load_twiddles(lds, g, ap.n, tid, kPassThreads);
        __syncthreads();
        return lds;
    }
}

// 1, hidden from the compiler: the row weights of the accessors along c
// enter as products (the bits of the transforms depend on how the compiler
// contracts them with the first stage's sums)
template <typename T>
__device__ __forceinline__ T opaque_one()
{
    T one = T(1);
    asm("" : "+v"(one));
    return one;
}

template <typename T>
__device__ __forceinline__ Cx<T> conj_of(Cx<T> v)
{
    return Cx<T>{v.x, -v.y};
}

// ---------------------------------------------------------------- P1
template <typename T, int MODE, bool WIDE, bool TWG>
__global__ __launch_bounds__(256) void k_r2c_rt(PassArgs a)
{
    extern __shared__ __align__(16) unsigned char smem[];
    int prob, tile;
    find_item(a.tl, xcd_remap(blockIdx.x, gridDim.x), prob, tile);
    const ProbDesc &d = a.desc[prob];
    const AxisPlan &ap = d.ax[2];
    const int n = d.dims[2], nh = d.dims[3], P = 1 << a.p_log2, ldp = row_pitch(n), tid = threadIdx.x;
    const int64_t nrows = int64_t(d.dims[0]) * d.dims[1];
    const int64_t row0 = int64_t(tile) * 2 * P;
    const int rows = int((nrows - row0) < 2 * P ? (nrows - row0) : 2 * P);
    Cx<T> *buf = reinterpret_cast<Cx<T> *>(smem);
    const Cx<T> *tw = rt_twiddles<T, TWG>(a, ap, buf + 2 * P * ldp, tid);
    const T scale = MODE == 0 ? T(0) : T(a.grad_e[prob] * d.dv);
    const T *x = reinterpret_cast<const T *>(a.in) + d.grid_off + row0 * n;
    const T *h = reinterpret_cast<const T *>(a.in2) + d.grid_off + row0 * n;
    const int pencils = (rows + 1) >> 1;
    const RtRows it{pencils};
    const T one = opaque_one<T>();
    auto at = [&](int p, int i) { return p * ldp + i; };
    // the pair of rows 2 p, 2 p + 1; the last pair of an odd number of rows
    // is completed by the first one's zero-weighted double
    auto in = [&](int p, int i) {
        const bool v1 = 2 * p + 1 < rows;
        const int64_t e = int64_t(2 * p) * n, o = v1 ? e + n : e;
        RealPairIn<T, MODE> r;
        r.r0 = x + e;
        r.r1 = x + o;
        r.h0 = h + e;
        r.h1 = h + o;
        r.w0 = one;
        r.w1 = v1 ? one : T(0);
        r.s0 = scale * r.w0;
        r.s1 = scale * r.w1;
        return r.load(i);
    };
    Cx<T> *z = buf;
    if (ap.nstages > 0) {
        z = buf + ((ap.nstages - 1) & 1) * P * ldp;
        rt_fft<T, WIDE>(it, ap, tw, buf, P * ldp, 0, at, in, [&](int p, int i, Cx<T> v) { z[at(p, i)] = v; });
    } else if (tid < pencils) {
        z[at(tid, 0)] = in(tid, 0);
    }
    __syncthreads();
    // X[k] = (Z[k] + conj Z[n-k]) / 2,  Y[k] = (Z[k] - conj Z[n-k]) / (2i)
    Cx<T> *dst = reinterpret_cast<Cx<T> *>(a.spec) + d.spec_off + row0 * nh;
    const int totalh = rows * nh;
    for (int e = tid; e < totalh; e += kPassThreads) {
        const int row = int(fdiv(uint32_t(e), d.div_nh));
        const int k = e - row * nh;
        const Cx<T> *zr = z + (row >> 1) * ldp;
        const Cx<T> A = zr[k];
        const Cx<T> B = zr[k == 0 ? 0 : n - k];
        Cx<T> X;
        if ((row & 1) == 0)
            X = {T(0.5) * (A.x + B.x), T(0.5) * (A.y - B.y)};
        else
            X = {T(0.5) * (A.y + B.y), T(0.5) * (B.x - A.x)};
        dst[e] = X;
    }
}

// ---------------------------------------------------------------- P5
template <typename T, bool WIDE, bool TWG>
__global__ __launch_bounds__(256) void k_c2r_rt(PassArgs a)
{
    extern __shared__ __align__(16) unsigned char smem[];
    int prob, tile;
    find_item(a.tl, xcd_remap(blockIdx.x, gridDim.x), prob, tile);
    const ProbDesc &d = a.desc[prob];
    const AxisPlan &ap = d.ax[2];
    const int n = d.dims[2], nh = d.dims[3], P = 1 << a.p_log2, ldp = row_pitch(n), tid = threadIdx.x;
    const int64_t nrows = int64_t(d.dims[0]) * d.dims[1];
    const int64_t row0 = int64_t(tile) * 2 * P;
    const int rows = int((nrows - row0) < 2 * P ? (nrows - row0) : 2 * P);
    Cx<T> *buf = reinterpret_cast<Cx<T> *>(smem);
    const Cx<T> *tw = rt_twiddles<T, TWG>(a, ap, buf + 2 * P * ldp, tid);
    const Cx<T> *spec = reinterpret_cast<const Cx<T> *>(a.spec) + d.spec_off + row0 * nh;
    T *o = reinterpret_cast<T *>(a.out) + d.grid_off + row0 * n;
    const int pencils = (rows + 1) >> 1;
    const RtRows it{pencils};
    const T one = opaque_one<T>();
    auto in = [&](int p, int i) {
        const bool v1 = 2 * p + 1 < rows;
        HermitianPairIn<T> r;
        r.x0 = spec + 2 * p * nh;
        r.x1 = v1 ? r.x0 + nh : r.x0;
        r.n = n;
        r.nh = nh;
        r.w0 = one;
        r.w1 = v1 ? one : T(0);
        return r.load(i);
    };
    auto out = [&](int p, int i, Cx<T> v) {
        RealPairOut<T> r;
        r.o0 = o + int64_t(2 * p) * n;
        r.o1 = r.o0 + n;
        r.v0 = true;
        r.v1 = 2 * p + 1 < rows;
        r.store(i, v);
    };
    if (ap.nstages > 0)
        rt_fft<T, WIDE, RT_LAST_C2R>(it, ap, tw, buf, P * ldp, 0, [&](int p, int i) { return p * ldp + i; }, in, out);
    else if (tid < pencils)
        out(tid, 0, in(tid, 0));
}

// ---------------------------------------------------------------- P2 / P4
template <typename T, bool WIDE, bool TWG>
__global__ __launch_bounds__(256) void k_fft_b_rt(PassArgs a)
{
    extern __shared__ __align__(16) unsigned char smem[];
    int prob, tile;
    find_item(a.tl, xcd_remap(blockIdx.x, gridDim.x), prob, tile);
    const ProbDesc &d = a.desc[prob];
    const AxisPlan &ap = d.ax[1];
    if (ap.nstages == 0) return;  // a length-1 axis: identity
    const int n = d.dims[1], nh = d.dims[3], P = 1 << a.p_log2, PP = P + a.pad, tid = threadIdx.x;
    const int tpo = (nh + P - 1) >> a.p_log2;
    const int outer = tile / tpo;
    const int h0 = (tile - outer * tpo) * P;
    const int valid = (nh - h0) < P ? (nh - h0) : P;
    Cx<T> *buf = reinterpret_cast<Cx<T> *>(smem);
    const Cx<T> *tw = rt_twiddles<T, TWG>(a, ap, buf + 2 * n * PP, tid);
    const int p0 = tid & (P - 1);
    const RtStrided it{p0, tid >> a.p_log2, kPassThreads >> a.p_log2};
    const bool inv = a.inv != 0, ok = p0 < valid;
    // a pencil beyond the tile edge loads a valid one and stores nothing
    Cx<T> *g = reinterpret_cast<Cx<T> *>(a.spec) + d.spec_off + int64_t(outer) * n * nh + h0 + (ok ? p0 : 0);
    rt_fft<T, WIDE>(
        it, ap, tw, buf, n * PP, 0, [&](int p, int i) { return i * PP + p; },
        [&](int, int i) {
            Cx<T> v = g[int64_t(i) * nh];
            return inv ? conj_of(v) : v;
        },
        [&](int, int i, Cx<T> v) {
            if (ok) g[int64_t(i) * nh] = inv ? conj_of(v) : v;
        });
}

// ---------------------------------------------------------------- P3
template <typename T, bool WIDE, bool TWG>
__global__ __launch_bounds__(256) void k_fft_a_rt(PassArgs a)
{
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ double red[kPassThreads / 64];
    int prob, tile;
    find_item(a.tl, xcd_remap(blockIdx.x, gridDim.x), prob, tile);
    const ProbDesc &d = a.desc[prob];
    const AxisPlan &ap = d.ax[0];
    const int mode = a.mode;
    const bool energy = mode != 1;
    const int n = d.dims[0], nh = d.dims[3], Nc = d.dims[2], P = 1 << a.p_log2, PP = P + a.pad, tid = threadIdx.x;
    const int ncol = d.dims[1] * nh;
    const int col0 = tile * P;
    const int valid = (ncol - col0) < P ? (ncol - col0) : P;
    Cx<T> *buf = reinterpret_cast<Cx<T> *>(smem);
    const Cx<T> *tw = rt_twiddles<T, TWG>(a, ap, buf + 2 * n * PP, tid);
    const int p0 = tid & (P - 1);
    const RtStrided it{p0, tid >> a.p_log2, kPassThreads >> a.p_log2};
    const bool ok = p0 < valid;
    const int col = col0 + (ok ? p0 : 0);
    const int mb = int(fdiv(uint32_t(col), d.div_nh));
    const int mc = col - mb * nh;
    Cx<T> *g = reinterpret_cast<Cx<T> *>(a.spec) + d.spec_off + col;
    // (a single stage leaves most threads idle, one butterfly per pencil: its
    // result goes to the other copy first, and the multiply is dealt out to all
    // of them; 16 x 40 x 48 FP32 20 -> 9 us, 8 x 40 x 48 13 -> 8)
    const int S = ap.nstages, copy = n * PP, result = S > 1 ? (S - 1) & 1 : S;
    auto at = [&](int p, int i) { return i * PP + p; };
    KernelMultiply<T> km{buf + result * copy, PP, p0, &d, mb, mc, energy, T(d.inv_n),
                         ok ? ((mc == 0 || 2 * mc == Nc) ? 1.0 : 2.0) : 0.0, 0.0};
    km.init();
    auto from_global = [&](int, int i) { return g[int64_t(i) * ncol]; };
    if (S == 0) {
        // length-1 axis: the multiply alone
        if (it.tip == 0) km.store(0, g[0]);
    } else if (S == 1) {
        rt_fft<T, WIDE>(it, ap, tw, buf, copy, 0, at, from_global, [&](int p, int i, Cx<T> v) { buf[at(p, i)] = v; });
        __syncthreads();
        for (int i = it.tip; i < n; i += it.tpp) km.store(i, buf[at(p0, i)]);
    } else {
        rt_fft<T, WIDE>(it, ap, tw, buf, copy, 0, at, from_global, [&](int, int i, Cx<T> v) { km.store(i, v); });
    }
    __syncthreads();
    if (energy) {
        const double acc = wave_sum(km.acc);
        if ((tid & 63) == 0) red[tid >> 6] = acc;
        __syncthreads();
        if (tid == 0) {
            double s = 0.0;
            for (int w = 0; w < kPassThreads / 64; ++w) s += red[w];
            a.partials[d.part_off + tile] = s;
        }
    }
    if (mode == 2) return;
    // inverse along a: the forward stages on conjugated data, from the copy
    // that holds the product into the other one first
    const Cx<T> *from = buf + result * copy;
    if (S == 0) {
        if (it.tip == 0 && ok) g[0] = from[at(p0, 0)];
    } else {
        rt_fft<T, WIDE>(
            it, ap, tw, buf, copy, result + 1, at, [&](int p, int i) { return conj_of(from[at(p, i)]); },
            [&](int, int i, Cx<T> v) {
                if (ok) g[int64_t(i) * ncol] = conj_of(v);
            });
    }
}

// ------------------------------------------------------------- launchers
// wide: a plan of the launch has a radix-16 stage (kRuntimeWide)

#define HARTREE_RT_PICK(...)                                                               \
    do {                                                                                   \
        if constexpr (sizeof(T) == 8)                                                      \
            if (twg) return launch_pass(__VA_ARGS__ true, true>, grid, lds, s, a);        \
        if (wide) return launch_pass(__VA_ARGS__ true, false>, grid, lds, s, a);          \
        return launch_pass(__VA_ARGS__ false, false>, grid, lds, s, a);                   \
    } while (0)

template <typename T>
hipError_t launch_r2c_rt(bool wide, int maxn, int grid, hipStream_t s, const PassArgs &a)
{
    bool twg;
    const size_t lds = runtime_lds(sizeof(T) == 8, 2, maxn, a.p_log2, 0, twg);
    if (a.mode == 0 || a.grad_e == nullptr) HARTREE_RT_PICK(k_r2c_rt<T, 0, );
    if (a.in != nullptr) HARTREE_RT_PICK(k_r2c_rt<T, 1, );
    HARTREE_RT_PICK(k_r2c_rt<T, 2, );
}
template <typename T>
hipError_t launch_c2r_rt(bool wide, int maxn, int grid, hipStream_t s, const PassArgs &a)
{
    bool twg;
    const size_t lds = runtime_lds(sizeof(T) == 8, 2, maxn, a.p_log2, 0, twg);
    HARTREE_RT_PICK(k_c2r_rt<T, );
}
template <typename T>
hipError_t launch_b_rt(bool wide, int maxn, int grid, hipStream_t s, const PassArgs &a)
{
    bool twg;
    const size_t lds = runtime_lds(sizeof(T) == 8, 1, maxn, a.p_log2, a.pad, twg);
    HARTREE_RT_PICK(k_fft_b_rt<T, );
}
template <typename T>
hipError_t launch_a_rt(bool wide, int maxn, int grid, hipStream_t s, const PassArgs &a)
{
    bool twg;
    const size_t lds = runtime_lds(sizeof(T) == 8, 0, maxn, a.p_log2, a.pad, twg);
    HARTREE_RT_PICK(k_fft_a_rt<T, );
}
#undef HARTREE_RT_PICK

}  // namespace hartree

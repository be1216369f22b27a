// Splat and splat adjoint in any periodic cell (the vector-unit path for
// cells that are not diagonal; diagonal cells use the separable kernels).
//
// In a general cell a Gaussian is not a product of per-axis factors, so each
// (grid point, atom image) pair is evaluated directly, inside the cutoff
// sphere |d| <= cutoff sigma (the truncation of the CPU reference as well).
// Most points of a listed brick lie outside the sphere (at 160^3 in the
// diamond FCC cell 78%), so both precisions first place each atom image's
// sphere in the problem's triangular frame (GenDesc tri: the third axis along
// the cell row c, the second in the plane of b and c, where the points of a
// run of grid indices lie in a box) and pass over whole runs of points that
// the sphere does not reach.  A wavefront takes 64 points at a time, its sums
// (splat) in registers, a brick's grad_rho (adjoint) in LDS; it reads the
// brick's sorted list 64 entries at a time, one entry per lane, and takes the
// entries whose spheres reach its points one by one, broadcast from their
// lane's registers.
//
// Bound by vector and exponential issue over the points near the spheres.
// Diamond FCC cell, 160^3, 1,024 atoms, FP32: splat 896 -> 134 us, adjoint
// 1,492 -> 163 us; sheared cell, 72 x 80 x 90, 108 atoms, FP64: 450 -> 50 and
// 624 -> 75 us (before: every point of every listed brick, with the wrapped
// index arithmetic per pair, and one pass over LDS per atom).
#include "splat_common.hpp"

namespace hartree {

// smallest |x| over [lo, hi]
__device__ __forceinline__ double gap(double lo, double hi)
{
    return lo > 0.0 ? lo : (hi < 0.0 ? -hi : 0.0);
}

__device__ __forceinline__ int lane_value(int x, int q) { return __builtin_amdgcn_readlane(x, q); }
__device__ __forceinline__ float lane_value(float x, int q)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), q));
}
__device__ __forceinline__ double lane_value(double x, int q)
{
    const uint64_t b = __double_as_longlong(x);
    const uint32_t l = __builtin_amdgcn_readlane(int(uint32_t(b)), q), h = __builtin_amdgcn_readlane(int(uint32_t(b >> 32)), q);
    return __longlong_as_double(int64_t((uint64_t(h) << 32) | l));
}

// x plus its value moved across lanes by a data-parallel move (lanes without
// a source, or outside the row mask, add zero)
template <int CTRL, int ROWS>
__device__ __forceinline__ float dpp_plus(float x)
{
    return x + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, ROWS, 0xf, false));
}
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_plus(double x)
{
    const uint64_t b = __double_as_longlong(x);
    const uint32_t l = __builtin_amdgcn_update_dpp(0, int(uint32_t(b)), CTRL, ROWS, 0xf, false);
    const uint32_t h = __builtin_amdgcn_update_dpp(0, int(uint32_t(b >> 32)), CTRL, ROWS, 0xf, false);
    return x + __longlong_as_double(int64_t((uint64_t(h) << 32) | l));
}

// An atom's periodic images over one brick.  Unwrapped indices are counted from
// the atom's window start lo: the brick's first point g0 lies at u = g0 - lo +
// m N for image m (per axis), and the images whose points meet the window are
// numbered 0 .. count - 1, axis a slowest, from u0 on.  r: the atom relative to
// the window start, in the triangular frame (formed from the small Cartesian
// difference rb, which keeps the projection's rounding below that of rb).
// CENTRED (FP64): indices are counted from the middle of the window instead, at
// most a grid step or two from the atom, and rb is formed without rounding but
// its last: what a point's displacement is off by is then relative to the
// displacement, not to the window or the cell.  (72 x 80 x 90, 108 atoms, error
// of the density's norm: from the window start 1.9e-15, so 1.3e-15, nearly all of
// it from wrapping the positions; 1 to 2 us of 50 and 75.)
struct GenImages {
    double r[3];
    int u0[3], mc[3];
    int count;
};

// hi + lo -= f a (hi takes the rounded difference, lo what it leaves)
__device__ __forceinline__ void minus_product(double &hi, double &lo, double f, double a)
{
    double p = f * a;
    asm("" : "+v"(p));  // (not fused into the difference, whose remainder is taken)
    const double s = hi - p, b = s - hi;
    lo += ((hi - (s - b)) - (p + b)) - fma(f, a, -p);
    hi = s;
}

template <bool CENTRED>
__device__ __forceinline__ GenImages gen_images(const AtomInfo &in, const ProbDesc &d, const GenDesc &gd, const int g0[3], double rb[3])
{
    GenImages im;
    im.count = 1;
    for (int c = 0; c < 3; ++c) rb[c] = in.X[c];
    double rest[3] = {0.0, 0.0, 0.0};
    for (int x = 0; x < 3; ++x) {
        const int half = CENTRED ? (in.hi[x] - in.lo[x]) / 2 : 0;
        if constexpr (CENTRED) {
            const double u = in.lo[x] + half, per = 1.0 / d.dims[x];
            const double f = u * per, fl = fma(-f, double(d.dims[x]), u) * per;
            for (int c = 0; c < 3; ++c) {
                minus_product(rb[c], rest[c], f, d.A[3 * x + c]);
                rest[c] -= fl * d.A[3 * x + c];
            }
        } else {
            const double f = double(in.lo[x]) / d.dims[x];
            for (int c = 0; c < 3; ++c) rb[c] -= f * d.A[3 * x + c];
        }
        // u in [1 - bsz, hi - lo], in steps of N
        const int n = d.dims[x], first = 1 - d.bsz[x];
        im.u0[x] = first + wrapi(g0[x] - in.lo[x] - first, n);
        im.mc[x] = im.u0[x] <= in.hi[x] - in.lo[x] ? (in.hi[x] - in.lo[x] - im.u0[x]) / n + 1 : 0;
        im.count *= im.mc[x];
        im.u0[x] -= half;
    }
    if constexpr (CENTRED)
        for (int c = 0; c < 3; ++c) rb[c] += rest[c];
    for (int x = 0; x < 3; ++x) im.r[x] = rb[0] * gd.frame[3 * x] + rb[1] * gd.frame[3 * x + 1] + rb[2] * gd.frame[3 * x + 2];
    return im;
}

__device__ __forceinline__ GenImages no_images()
{
    GenImages im;
    for (int x = 0; x < 3; ++x) {
        im.r[x] = 0.0;
        im.u0[x] = 0;
        im.mc[x] = 1;
    }
    im.count = 0;
    return im;
}

// image i of an atom: the offset u of the brick's first point from the window
// start (or middle), and the displacement p, in the triangular frame, of the
// point k0 further along c
struct GenShift {
    int u[3];
    double p[3];
};
__device__ __forceinline__ GenShift gen_shift(const GenImages &im, const ProbDesc &d, const GenDesc &gd, int i, int k0 = 0)
{
    GenShift s;
    for (int x = 0; x < 3; ++x) s.u[x] = im.u0[x];
    if (i > 0) {
        const int uv = i / im.mc[2], u = uv / im.mc[1];
        s.u[2] += (i - uv * im.mc[2]) * d.dims[2];
        s.u[1] += (uv - u * im.mc[1]) * d.dims[1];
        s.u[0] += u * d.dims[0];
    }
    const double ga = s.u[0], gb = s.u[1], gc = s.u[2] + k0;
    s.p[0] = ga * gd.tri[0] - im.r[0];
    s.p[1] = ga * gd.tri[1] + gb * gd.tri[3] - im.r[1];
    s.p[2] = ga * gd.tri[2] + gb * gd.tri[4] + gc * gd.tri[5] - im.r[2];
    return s;
}

// squared distance from the atom to the box (in the triangular frame) that
// holds the points at offsets o .. o + e (inclusive, per axis) from the
// brick's first point
__device__ __forceinline__ double box_distance2(const GenDesc &gd, const double p[3], const int o[3], double ea, double eb,
                                                double ec)
{
    const double *t = gd.tri;
    const double oa = o[0], ob = o[1], oc = o[2];
    const double b1 = p[0] + oa * t[0], b2 = p[1] + oa * t[1] + ob * t[3], b3 = p[2] + oa * t[2] + ob * t[4] + oc * t[5];
    const double g1 = gap(b1, b1 + ea * t[0]);
    const double g2 = gap(b2 + fmin(ea * t[1], 0.0), b2 + fmax(ea * t[1], 0.0) + eb * t[3]);
    const double g3 = gap(b3 + fmin(ea * t[2], 0.0) + fmin(eb * t[4], 0.0),
                          b3 + fmax(ea * t[2], 0.0) + fmax(eb * t[4], 0.0) + ec * t[5]);
    return g1 * g1 + g2 * g2 + g3 * g3;
}
// margin of the box tests over the rounding of box_distance2 and of rc^2
constexpr double kBoxMargin = 1.0001;

// ---------------------------------------------------------------- FP32
// Every point is evaluated in Cartesian components, each formed with one
// rounding of the large terms (an fma chain) plus the small remainder terms,
// in this fixed order of operations, which the FP32 results' bits depend on:
//   d_c = fma(ua, a_c, fma(ub, b_c, fma(uc, c_c, -rb_c)))
//         + (fma(uc, cl_c, fma(ub, bl_c, ua al_c)) - rbl_c)
// with u_x the point's unwrapped offset from the window start lo_x, a_c, al_c
// ... the grid steps and their rounding remainders, and rb = R - sum_x (lo_x /
// N_x) x-th cell row (formed in double, small) carried as rb + rbl.
// A wavefront's 64 points are 8 (j) x 8 (k) at one i: the terms of ub and uc
// are formed once per atom, and the sphere of 6 sigma fills 64% of the 64
// points it reaches on average (45% of 2 x 32, 22% of whole bricks).

// The grid steps and their remainders, held in vector registers: left to
// itself the compiler reads them from the descriptor again for every point
// and waits for the scalar loads (adjoint 194 us instead of 161 at 160^3).
struct GenSteps {
    float e[9], l[9];
};
__device__ __forceinline__ GenSteps gen_steps(const GenDesc &gd)
{
    GenSteps g;
#pragma unroll
    for (int k = 0; k < 9; ++k) {
        g.e[k] = gd.step[k];
        g.l[k] = gd.stepl[k];
        asm volatile("" : "+v"(g.e[k]), "+v"(g.l[k]));
    }
    return g;
}

// one list entry per lane
struct GenAtom32 {
    GenImages im;
    float rb[3], rbl[3], inv2s2, w, rc2;
};
__device__ __forceinline__ GenAtom32 gen_atom32(const SplatArgs &a, const ProbDesc &d, const GenDesc &gd, const int g0[3], int64_t e,
                                                bool use)
{
    GenAtom32 g;
    g.im = no_images();
    for (int x = 0; x < 3; ++x) g.rb[x] = g.rbl[x] = 0.0f;
    g.inv2s2 = g.w = g.rc2 = 0.0f;
    if (!use) return g;
    const AtomInfo in = a.info[a.list_sorted[e]];
    double rb[3];
    g.im = gen_images<false>(in, d, gd, g0, rb);
    for (int c = 0; c < 3; ++c) {
        g.rb[c] = float(rb[c]);
        g.rbl[c] = float(rb[c] - double(g.rb[c]));
    }
    g.inv2s2 = float(in.inv2s2);
    g.w = float(in.w);
    const double rc = a.cutoff * sqrt(0.5 / in.inv2s2);
    g.rc2 = float(rc * rc);
    return g;
}

// the entry of lane q in every lane
__device__ __forceinline__ GenAtom32 lane_atom(const GenAtom32 &g, int q)
{
    GenAtom32 o;
    for (int x = 0; x < 3; ++x) {
        o.im.r[x] = lane_value(g.im.r[x], q);
        o.im.u0[x] = lane_value(g.im.u0[x], q);
        o.im.mc[x] = lane_value(g.im.mc[x], q);
        o.rb[x] = lane_value(g.rb[x], q);
        o.rbl[x] = lane_value(g.rbl[x], q);
    }
    o.im.count = lane_value(g.im.count, q);
    o.inv2s2 = lane_value(g.inv2s2, q);
    o.w = lane_value(g.w, q);
    o.rc2 = lane_value(g.rc2, q);
    return o;
}

// The images of the lane's entry that reach the box of points o .. o + e: bit
// i for image i < 32; with more images all of them (bit 31 stands for the
// images from 31 on).
__device__ __forceinline__ uint32_t gen_hits(const GenAtom32 &g, const ProbDesc &d, const GenDesc &gd, const int o[3],
                                             double ea, double eb, double ec)
{
    uint32_t hits = 0;
    for (int i = 0; __any(i < g.im.count && i < 32); ++i) {
        if (i >= g.im.count) continue;
        const GenShift s = gen_shift(g.im, d, gd, i);
        if (box_distance2(gd, s.p, o, ea, eb, ec) <= kBoxMargin * double(g.rc2)) hits |= 1u << i;
    }
    return g.im.count > 32 ? 0xffffffffu : hits;
}

// displacement terms of ub and uc of one lane's column (see above)
struct GenColumn {
    float h[3], ub, uc;
};
__device__ __forceinline__ GenColumn gen_column(const GenSteps &st, const GenAtom32 &at, int ub, int uc)
{
    GenColumn c;
    c.ub = float(ub);
    c.uc = float(uc);
#pragma unroll
    for (int x = 0; x < 3; ++x)
        c.h[x] = __builtin_fmaf(c.ub, st.e[3 + x], __builtin_fmaf(c.uc, st.e[6 + x], -at.rb[x]));
    return c;
}
// displacement at ua; returns |d|^2
__device__ __forceinline__ float gen_point(const GenSteps &st, const GenAtom32 &at, const GenColumn &c, float ua, float dv[3])
{
#pragma unroll
    for (int x = 0; x < 3; ++x) {
        const float lo = __builtin_fmaf(c.uc, st.l[6 + x], __builtin_fmaf(c.ub, st.l[3 + x], ua * st.l[x])) - at.rbl[x];
        dv[x] = __builtin_fmaf(ua, st.e[x], c.h[x]) + lo;
    }
    return __builtin_fmaf(dv[2], dv[2], __builtin_fmaf(dv[0], dv[0], dv[1] * dv[1]));
}

// NS: planes i per wavefront
template <int NS>
__global__ __launch_bounds__(256) void k_splat_general32(SplatArgs a)
{
    constexpr int UI = kMI / NS, UNITS = UI * (kMJ / 8) * (kMK / 8);
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6)), lane = threadIdx.x & 63;
    const int item = xcd_remap(blockIdx.x, gridDim.x) * 4 + wave;
    const int64_t b = item / UNITS;
    const int unit = item % UNITS;
    const int prob = brick_prob(a, b);
    const ProbDesc &d = a.desc[prob];
    const GenDesc &gd = a.gen[prob];
    const BrickPos p = brick_pos(d, b);
    const int g0[3] = {p.b0 * kMI, p.b1 * kMJ, p.b2 * kMK};
    const int o[3] = {NS * (unit % UI), 8 * ((unit / UI) % (kMJ / 8)), 8 * (unit / (UI * (kMJ / 8)))};
    if (g0[0] + o[0] >= d.dims[0] || g0[1] + o[1] >= d.dims[1] || g0[2] + o[2] >= d.dims[2]) return;
    const int lj = lane >> 3, lk = lane & 7;
    const GenSteps st = gen_steps(gd);
    const int64_t off = a.offsets[b];
    const int cnt = int(a.ends[b] - off);
    float acc[NS];
#pragma unroll
    for (int i = 0; i < NS; ++i) acc[i] = 0.0f;
    for (int c0 = 0; c0 < cnt; c0 += 64) {
        const GenAtom32 mine = gen_atom32(a, d, gd, g0, off + c0 + lane, c0 + lane < cnt);
        const uint32_t hits = gen_hits(mine, d, gd, o, NS - 1, 7.0, 7.0);
        uint64_t todo = __ballot(hits != 0u);
        while (todo) {
            const int q = __builtin_ctzll(todo);
            todo &= todo - 1;
            const uint32_t hq = lane_value(int(hits), q);
            const GenAtom32 at = lane_atom(mine, q);
            for (int im = 0; im < at.im.count; ++im) {
                if (!((hq >> (im < 31 ? im : 31)) & 1u)) continue;
                const GenShift s = gen_shift(at.im, d, gd, im);
                // planes the sphere reaches: lane l tests plane l
                const int ol[3] = {o[0] + (lane & (NS - 1)), o[1], o[2]};
                const uint32_t mask =
                    uint32_t(__ballot(box_distance2(gd, s.p, ol, 0.0, 7.0, 7.0) <= kBoxMargin * double(at.rc2)));
                const int u0 = s.u[0] + o[0];
                const GenColumn col = gen_column(st, at, s.u[1] + o[1] + lj, s.u[2] + o[2] + lk);
#pragma unroll
                for (int i = 0; i < NS; ++i) {
                    if (!((mask >> i) & 1u)) continue;
                    float dv[3];
                    const float d2 = gen_point(st, at, col, float(u0 + i), dv);
                    const float e = expf(-d2 * at.inv2s2);
                    const float next = __builtin_fmaf(at.w, e, acc[i]);
                    acc[i] = d2 <= at.rc2 ? next : acc[i];
                }
            }
        }
    }
    const int j = g0[1] + o[1] + lj, k = g0[2] + o[2] + lk;
    if (j >= d.dims[1] || k >= d.dims[2]) return;
    const float bg = a.subtract_background ? float(a.qsum[prob] / (d.dv * double(d.npts))) : 0.0f;
    float *out = reinterpret_cast<float *>(a.rho) + d.grid_off;
#pragma unroll
    for (int i = 0; i < NS; ++i) {
        const int ia = g0[0] + o[0] + i;
        if (ia < d.dims[0]) out[(int64_t(ia) * d.dims[1] + j) * d.dims[2] + k] = acc[i] - bg;
    }
}

// below this many bricks (with one wavefront per 8 x 8 columns, fewer than
// two per SIMD) each brick's work is cut into more, smaller pieces
constexpr int kFewBricks = 256;

// grad_rho of the brick's points of one kb (zero outside the grid) to LDS
__device__ __forceinline__ void load_grad32(const SplatArgs &a, const ProbDesc &d, const int g0[3], int kb, int lane,
                                            float (*gr)[64])
{
    const float *src = reinterpret_cast<const float *>(a.grad_rho) + d.grid_off;
    const int k = g0[2] + 8 * kb + (lane & 7);
#pragma unroll
    for (int i = 0; i < kMI; ++i)
#pragma unroll
        for (int jb = 0; jb < 2; ++jb) {
            const int ia = g0[0] + i, j = g0[1] + 8 * jb + (lane >> 3);
            const bool in = ia < d.dims[0] && j < d.dims[1] && k < d.dims[2];
            gr[2 * i + jb][lane] = *(in ? src + (int64_t(ia) * d.dims[1] + j) * d.dims[2] + k : a.zeros);
        }
}

// the end of a sum over 8 x 8 lanes (j0, k mod 8) whose rows j0 and j0 ^ 1 are
// added: over k ^ 4, 2, 1 (shifts within rows of 16 lanes), then over the four
// pairs of j0 in double
__device__ __forceinline__ double sum_pairs32(float z)
{
    float w = dpp_plus<0x104, 0xf>(z);
    w = dpp_plus<0x102, 0xf>(w);
    w = dpp_plus<0x101, 0xf>(w);
    double v = 0.0;
#pragma unroll
    for (int r = 0; r < 4; ++r) v += double(lane_value(w, 16 * r));
    return v;
}

// one point of the adjoint: d and grad_rho exp(-|d|^2 / (2 sigma^2)) into the sums
__device__ __forceinline__ void adjoint_point(const GenSteps &st, const GenAtom32 &at, const GenColumn &col, float ua, float g,
                                              float (&f)[3])
{
    float dv[3];
    const float d2 = gen_point(st, at, col, ua, dv);
    const float e = expf(-d2 * at.inv2s2);
    // (selected after the product: a non-finite grad_rho beyond the sphere
    // does not reach the atom)
    const float t = d2 <= at.rc2 ? g * e : 0.0f;
#pragma unroll
    for (int x = 0; x < 3; ++x) f[x] = __builtin_fmaf(dv[x], t, f[x]);
}

// An entry of which several images reach the brick, over the points of one kb
// (gr: their grad_rho, k0 = 8 kb): run by run, the images in order, 64 of them
// tested against a run at once, one per lane.
__device__ __forceinline__ void adjoint_images(const GenSteps &st, const ProbDesc &d, const GenDesc &gd, const GenAtom32 &at,
                                               double reach, const float (*gr)[64], int k0, int lane, float (&f)[3])
{
    const int lj = lane >> 3, lk = lane & 7, count = at.im.count;
    GenShift s = gen_shift(at.im, d, gd, lane < count ? lane : 0);
#pragma unroll 1
    for (int i = 0; i < 2 * kMI; ++i) {
        const float g = gr[i][lane];
        const int o[3] = {i >> 1, 8 * (i & 1), k0};
#pragma unroll 1
        for (int im = 0; im < count; im += 64) {
            if (count > 64) s = gen_shift(at.im, d, gd, im + lane < count ? im + lane : 0);
            uint64_t m = __ballot(im + lane < count && box_distance2(gd, s.p, o, 0.0, 7.0, 7.0) <= reach);
            while (m) {
                const int l = __builtin_ctzll(m);
                m &= m - 1;
                const int ua = lane_value(s.u[0], l) + o[0], ub = lane_value(s.u[1], l) + o[1] + lj,
                          uc = lane_value(s.u[2], l) + o[2] + lk;
                adjoint_point(st, at, gen_column(st, at, ub, uc), float(ua), g, f);
            }
        }
    }
}

// Adjoint: per list slot the partial sum over the brick's points of grad_rho
// exp(-|d|^2 / (2 sigma^2)) d (the caller scales by w / sigma^2).  grad_rho of
// the brick lies in LDS; each wavefront takes list entries of its own (the
// `split` workgroups of a brick and their four wavefronts in turn) and walks
// the whole brick for one, so that nothing waits between entries: a wavefront
// per 8 points of k with the partial sums combined over LDS every 16 entries
// measured 225 us at 160^3 (193 us every 8), the vector issue being 143 us.
// The sum over a brick's points keeps one order (the bits of the forces
// depend on it): per lane (j0, k mod 8) and kb = k / 8 over i with j0 before
// j0 + 8, then over j0 and j0 ^ 1, over k ^ 16, 8, 4, 2, 1, and over the four
// pairs of j0 in double.
// MANY: several images of one atom may reach one run of points (known on the
// host from the cell and the cutoff).
template <bool MANY>
__global__ __launch_bounds__(256) void k_adjoint_general32(SplatArgs a, int split)
{
    __shared__ float gr[4][2 * kMI][64];  // [kb][2 i + j / 8][lane (j0, k mod 8)]
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6)), lane = threadIdx.x & 63;
    const int64_t b = blockIdx.x / split;
    const int share = blockIdx.x - int(b) * split;
    const int prob = brick_prob(a, b);
    const ProbDesc &d = a.desc[prob];
    const GenDesc &gd = a.gen[prob];
    const int64_t off = a.offsets[b];
    const int cnt = int(a.ends[b] - off);
    const int ways = 4 * split, way = 4 * share + wave;  // entries way, way + ways, ... are this wavefront's
    if (4 * share >= cnt) return;
    const BrickPos p = brick_pos(d, b);
    const int g0[3] = {p.b0 * kMI, p.b1 * kMJ, p.b2 * kMK};
    const int lj = lane >> 3, lk = lane & 7;
    load_grad32(a, d, g0, wave, lane, gr[wave]);
    __syncthreads();
    const GenSteps st = gen_steps(gd);
    const int whole[3] = {0, 0, 0};
    for (int c0 = 0; c0 < cnt; c0 += 64 * ways) {
        const int mye = c0 + lane * ways + way;
        const GenAtom32 mine = gen_atom32(a, d, gd, g0, off + mye, mye < cnt);
        const uint32_t hits = gen_hits(mine, d, gd, whole, kMI - 1, kMJ - 1, kMK - 1);
        for (int q = 0; q < 64 && c0 + q * ways + way < cnt; ++q) {
            const uint32_t hq = lane_value(int(hits), q);
            double v[3] = {0.0, 0.0, 0.0};
            if (hq) {
                const GenAtom32 at = lane_atom(mine, q);
                const double reach = kBoxMargin * double(at.rc2);
                // runs of points the sphere of an image reaches, 32 per kb
                // (bit 2 i + j / 8), two kb at a time: lane l tests run l
                auto runs = [&](const GenShift &s, int kb) {
                    const int ol[3] = {(lane & 31) >> 1, 8 * (lane & 1), 8 * (kb + (lane >> 5))};
                    return uint64_t(__ballot(box_distance2(gd, s.p, ol, 0.0, 7.0, 7.0) <= reach));
                };
                auto column = [&](const GenShift &s, int kb, int jb) {
                    return gen_column(st, at, s.u[1] + 8 * jb + lj, s.u[2] + 8 * kb + lk);
                };
                float z[3] = {0.0f, 0.0f, 0.0f}, y[3];
                const bool one = !MANY || ((hq & (hq - 1)) == 0u && at.im.count <= 32);
                const GenShift s1 = gen_shift(at.im, d, gd, one ? __builtin_ctz(hq) : 0);
                const uint64_t m01 = one ? runs(s1, 0) : 0, m23 = one ? runs(s1, 2) : 0;
#pragma unroll 1
                for (int turn = 0; turn < 4; ++turn) {
                    const int kb = ((turn & 1) << 1) | (turn >> 1);  // 0, 2, 1, 3
                    float f[3] = {0.0f, 0.0f, 0.0f};
                    if (one) {
                        uint32_t m = uint32_t((kb & 2 ? m23 : m01) >> (32 * (kb & 1)));
                        const int u0 = s1.u[0];
                        const GenColumn col0 = column(s1, kb, 0), col1 = column(s1, kb, 1);
                        while (m) {
                            const int i = __builtin_ctz(m) >> 1;
                            const uint32_t two = m >> (2 * i);
                            m &= ~(3u << (2 * i));
                            const float ua = float(u0 + i);
                            const float ga = gr[kb][2 * i][lane], gb = gr[kb][2 * i + 1][lane];
                            if (two & 1u) adjoint_point(st, at, col0, ua, ga, f);
                            if (two & 2u) adjoint_point(st, at, col1, ua, gb, f);
                        }
                    } else {
                        adjoint_images(st, d, gd, at, reach, gr[kb], 8 * kb, lane, f);
                    }
#pragma unroll
                    for (int x = 0; x < 3; ++x) {
                        // j0 and j0 ^ 1 (a rotation by 8 within rows of 16 lanes)
                        const float w = dpp_plus<0x128, 0xf>(f[x]);
                        if (turn == 0) z[x] = w;
                        else if (turn == 1) z[x] += w;
                        else if (turn == 2) y[x] = w;
                        else z[x] += y[x] + w;
                    }
                }
#pragma unroll
                for (int x = 0; x < 3; ++x) v[x] = sum_pairs32(z[x]);
            }
            const int64_t slot = off + c0 + q * ways + way;
            if (lane < 3 && slot < a.capacity) a.bpart[slot * 3 + lane] = lane == 0 ? v[0] : (lane == 1 ? v[1] : v[2]);
        }
    }
}

// The same for plans of few bricks whose atoms may have several images over one:
// few entries to go round, and up to hundreds of images each.  The workgroup
// takes an entry together, a wavefront per kb, and the wavefronts in turn
// combine an entry's four sums, in the order above.
// (us; one wavefront per entry, before 64 images were tested at once / this: 2
// atoms, 343 and more images each, on 16^3 3,684 / 177; 6 on 20^3 1,928 / 115; 60 on
// 80^3 121 / 59; 200 on 108^3, 196 bricks, 110 / 106; 400 on 128^3, 256 bricks, 157 / 165)
__global__ __launch_bounds__(256) void k_adjoint_images32(SplatArgs a, int split)
{
    __shared__ float gr[4][2 * kMI][64];  // [kb][2 i + j / 8][lane (j0, k mod 8)]
    __shared__ float part[2][4][3][64];   // [entry parity][kb][x][lane]
    const int kb = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6)), lane = threadIdx.x & 63;
    const int64_t b = blockIdx.x / split;
    const int share = blockIdx.x - int(b) * split;
    const int prob = brick_prob(a, b);
    const ProbDesc &d = a.desc[prob];
    const GenDesc &gd = a.gen[prob];
    const int64_t off = a.offsets[b];
    const int cnt = int(a.ends[b] - off);
    if (share >= cnt) return;  // entries share, share + split, ... are this workgroup's
    const BrickPos p = brick_pos(d, b);
    const int g0[3] = {p.b0 * kMI, p.b1 * kMJ, p.b2 * kMK};
    const int lj = lane >> 3, lk = lane & 7;
    load_grad32(a, d, g0, kb, lane, gr[kb]);
    __syncthreads();
    const GenSteps st = gen_steps(gd);
    const int whole[3] = {0, 0, 0};
    int turn = 0;  // entries with an image in reach so far
    for (int c0 = 0; c0 < cnt; c0 += 64 * split) {
        const int mye = c0 + lane * split + share;
        const GenAtom32 mine = gen_atom32(a, d, gd, g0, off + mye, mye < cnt);
        const uint32_t hits = gen_hits(mine, d, gd, whole, kMI - 1, kMJ - 1, kMK - 1);
        for (int q = 0; q < 64 && c0 + q * split + share < cnt; ++q) {
            const uint32_t hq = lane_value(int(hits), q);
            const int64_t slot = off + c0 + q * split + share;
            double v[3] = {0.0, 0.0, 0.0};
            if (hq) {
                const GenAtom32 at = lane_atom(mine, q);
                const double reach = kBoxMargin * double(at.rc2);
                float f[3] = {0.0f, 0.0f, 0.0f};
                if ((hq & (hq - 1)) == 0u && at.im.count <= 32) {
                    // one image: lane l < 32 tests run l of this kb
                    const GenShift s = gen_shift(at.im, d, gd, __builtin_ctz(hq));
                    const int ol[3] = {(lane & 31) >> 1, 8 * (lane & 1), 8 * kb};
                    uint32_t m = uint32_t(__ballot(box_distance2(gd, s.p, ol, 0.0, 7.0, 7.0) <= reach));
                    const GenColumn col0 = gen_column(st, at, s.u[1] + lj, s.u[2] + 8 * kb + lk),
                                    col1 = gen_column(st, at, s.u[1] + 8 + lj, s.u[2] + 8 * kb + lk);
                    while (m) {
                        const int i = __builtin_ctz(m);
                        m &= m - 1;
                        adjoint_point(st, at, i & 1 ? col1 : col0, float(s.u[0] + (i >> 1)), gr[kb][i][lane], f);
                    }
                } else {
                    adjoint_images(st, d, gd, at, reach, gr[kb], 8 * kb, lane, f);
                }
                // (the wavefront that combines entry n has read part[n & 1]
                // when it comes to the barrier of entry n + 1, and entry n + 2
                // is written there after that)
                float (&pt)[4][3][64] = part[turn & 1];
#pragma unroll
                for (int x = 0; x < 3; ++x) pt[kb][x][lane] = dpp_plus<0x128, 0xf>(f[x]);
                __syncthreads();
                if ((turn++ & 3) != kb) continue;
#pragma unroll
                for (int x = 0; x < 3; ++x) {
                    float z = pt[0][x][lane] + pt[2][x][lane];
                    z += pt[1][x][lane] + pt[3][x][lane];
                    v[x] = sum_pairs32(z);
                }
            } else if (kb != 0) {
                continue;
            }
            if (lane < 3 && slot < a.capacity) a.bpart[slot * 3 + lane] = lane == 0 ? v[0] : (lane == 1 ? v[1] : v[2]);
        }
    }
}

// ---------------------------------------------------------------- FP64
// Lane (i, j) holds the rows along c of a kBI x kBJ brick, kRun consecutive
// points of each at a time.  In the triangular frame such a row has fixed d1
// and d2: with s = (d1^2 + d2^2) / (2 sigma^2) and t = d3 / (sqrt(2) sigma) a
// point's exponent is s + t^2, and t advances by a constant c along the row.
// Both kernels deal a brick's list out to several wavefronts (four per run of
// points in the splat, summed over LDS at the end; four or eight per brick in
// the adjoint): with one wavefront per run of points 270 bricks left most
// SIMDs a single wavefront, and some two (68 and 100 us in the sheared cell).
static_assert(kBI == 8 && kBJ == 8, "a wavefront's rows");
constexpr int kRun = 8;
constexpr int kSeg = kBK / kRun;  // runs per row
constexpr int kWays = 4;          // wavefronts per workgroup

struct GenRows {
    int g0[3];        // the brick's first point
    double r[3];      // (d1, d2, d3) of the lane's row start minus the brick's first point
    bool inside;      // the row lies inside the grid
    int64_t row;      // its first point in the grid
};

__device__ __forceinline__ GenRows gen_rows(const ProbDesc &d, const GenDesc &gd, const BrickPos &p, int lane)
{
    GenRows r;
    r.g0[0] = p.b0 * kBI;
    r.g0[1] = p.b1 * kBJ;
    r.g0[2] = p.b2 * kBK;
    const int li = lane >> 3, lj = lane & 7;
    r.r[0] = li * gd.tri[0];
    r.r[1] = li * gd.tri[1] + lj * gd.tri[3];
    r.r[2] = li * gd.tri[2] + lj * gd.tri[4];
    r.inside = r.g0[0] + li < d.dims[0] && r.g0[1] + lj < d.dims[1];
    r.row = (int64_t(r.g0[0] + li) * d.dims[1] + r.g0[1] + lj) * d.dims[2] + r.g0[2];
    return r;
}

// The run's eight exponentials, t_k = tm + k c for k = -4 .. 3: with x =
// exp(-2 tm c), exp(-(s + t_k^2)) = exp(-(s + tm^2)) x^k exp(-c^2 k^2), three
// exponentials (x^-1 = exp(2 tm c) and x from one reduction) and a few products
// instead of eight exponentials.  The error is
// that of the exponents' terms, eps (s + tm^2 + |2 tm c k| + c^2 k^2), a few
// ulps while 4 c is about a width or less; taken only for c <= 0.5 (grid
// spacing up to 0.7 sigma), otherwise the points are evaluated one by one
// (direct), which also keeps every factor in range.
struct GenRun {
    double c, k1, k2, k3, k4;  // step of t; exp(-c^2 k^2)
    bool direct;
};
__device__ __forceinline__ GenRun gen_run(double c, double qc)
{
    GenRun r;
    r.c = c;
    const double reach = sqrt(qc) + 4.0 * c;  // largest |tm| of a run inside the sphere
    r.direct = !(c <= 0.5 && qc + reach * reach < 600.0 && 8.0 * reach * c < 600.0);
    r.k1 = exp64(-c * c);
    r.k2 = exp64(-4.0 * c * c);
    r.k3 = exp64(-9.0 * c * c);
    r.k4 = exp64(-16.0 * c * c);
    return r;
}
__device__ __forceinline__ GenRun lane_run(const GenRun &r, int q)
{
    GenRun o;
    o.c = lane_value(r.c, q);
    o.k1 = lane_value(r.k1, q);
    o.k2 = lane_value(r.k2, q);
    o.k3 = lane_value(r.k3, q);
    o.k4 = lane_value(r.k4, q);
    o.direct = lane_value(r.direct ? 1 : 0, q) != 0;
    return o;
}
// in[k + 4]: point k lies inside the sphere; e is meaningful only there
__device__ __forceinline__ void gen_exps(const GenRun &r, double s, double tm, double qc, double (&t)[kRun], bool (&in)[kRun],
                                         double (&e)[kRun])
{
#pragma unroll
    for (int j = 0; j < kRun; ++j) {
        t[j] = fma(double(j - 4), r.c, tm);
        in[j] = fma(t[j], t[j], s) <= qc;
    }
    if (r.direct) {
#pragma unroll
        for (int j = 0; j < kRun; ++j) e[j] = exp64(-fma(t[j], t[j], s));
        return;
    }
    const double A = exp64(-fma(tm, tm, s));
    double x, y;
    exp64_pair(-2.0 * tm * r.c, x, y);
    const double x2 = x * x, y2 = y * y;
    const double A1 = A * r.k1, A2 = A * r.k2, A3 = A * r.k3;
    e[0] = (A * r.k4) * (y2 * y2);
    e[1] = A3 * (y2 * y);
    e[2] = A2 * y2;
    e[3] = A1 * y;
    e[4] = A;
    e[5] = A1 * x;
    e[6] = A2 * x2;
    e[7] = A3 * (x2 * x);
}

// One list entry per lane: its images, sc = 1 / (sqrt(2) sigma), the weight
// and the constants of its runs.
struct GenAtom64 {
    GenImages im;
    double sc, w;
    GenRun run;
};
__device__ __forceinline__ GenAtom64 gen_atom64(const SplatArgs &a, const ProbDesc &d, const GenDesc &gd, const int g0[3], int64_t e,
                                                bool use, double qc)
{
    GenAtom64 g;
    g.im = no_images();
    g.sc = 1.0;
    g.w = 0.0;
    if (use) {
        const AtomInfo &in = a.info[a.list_sorted[e]];
        double rb[3];
        g.im = gen_images<true>(in, d, gd, g0, rb);
        g.sc = sqrt(in.inv2s2);
        g.w = in.w;
    }
    g.run = gen_run(gd.tri[5] * g.sc, qc);
    return g;
}

// s of the lane's row and tm of its run at offset ok, for an image of a
// displacement p; false when the image reaches none of the wavefront's points
__device__ __forceinline__ bool gen_row(const GenDesc &gd, const GenRows &rows, const double p[3], double sc, double c, int ok,
                                        double qc, double &d1, double &d2, double &s, double &tm)
{
    d1 = p[0] + rows.r[0];
    d2 = p[1] + rows.r[1];
    const double u1 = d1 * sc, u2 = d2 * sc;
    s = rows.inside ? u1 * u1 + u2 * u2 : HUGE_VAL;
    tm = (p[2] + rows.r[2] + (ok + 4) * gd.tri[5]) * sc;
    const double far = fmax(fabs(tm) - 4.0 * c, 0.0);
    return __any(fma(far, far, s) <= qc);
}

// splat: one workgroup per brick and run of points, its wavefronts taking the
// list's entries in turn; their sums are added in a fixed order
__global__ __launch_bounds__(64 * kWays) void k_splat_general64(SplatArgs a)
{
    __shared__ double part[kWays - 1][kRun][64];
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6)), lane = threadIdx.x & 63;
    const int item = xcd_remap(blockIdx.x, gridDim.x);
    const int64_t b = item / kSeg;
    const int prob = brick_prob(a, b);
    const ProbDesc &d = a.desc[prob];
    const GenDesc &gd = a.gen[prob];
    const GenRows rows = gen_rows(d, gd, brick_pos(d, b), lane);
    const int k0 = kRun * (item % kSeg), o[3] = {0, 0, -4};  // (displacements at the run's middle)
    if (rows.g0[2] + k0 >= d.dims[2]) return;
    const int64_t off = a.offsets[b];
    const int cnt = int(a.ends[b] - off);
    const double qc = 0.5 * a.cutoff * a.cutoff;
    double acc[kRun];
#pragma unroll
    for (int k = 0; k < kRun; ++k) acc[k] = 0.0;
    for (int c0 = 0; c0 < cnt; c0 += 64 * kWays) {
        const int mye = c0 + lane * kWays + wave;
        const GenAtom64 mine = gen_atom64(a, d, gd, rows.g0, off + mye, mye < cnt, qc);
        for (int i = 0; __any(i < mine.im.count); ++i) {
            GenShift sh;
            bool hit = false;
            if (i < mine.im.count) {
                sh = gen_shift(mine.im, d, gd, i, k0 + 4);
                hit = box_distance2(gd, sh.p, o, 7.0, 7.0, kRun - 1) * mine.sc * mine.sc <= kBoxMargin * qc;
            }
            uint64_t todo = __ballot(hit);
            while (todo) {
                const int q = __builtin_ctzll(todo);
                todo &= todo - 1;
                const double p[3] = {lane_value(sh.p[0], q), lane_value(sh.p[1], q), lane_value(sh.p[2], q)};
                const GenRun rn = lane_run(mine.run, q);
                double d1, d2, s, tm;
                if (!gen_row(gd, rows, p, lane_value(mine.sc, q), rn.c, o[2], qc, d1, d2, s, tm)) continue;
                double t[kRun], e[kRun];
                bool in[kRun];
                gen_exps(rn, s, tm, qc, t, in, e);
                const double w = lane_value(mine.w, q);
#pragma unroll
                for (int j = 0; j < kRun; ++j) acc[j] = in[j] ? fma(w, e[j], acc[j]) : acc[j];
            }
        }
    }
    if (wave > 0)
#pragma unroll
        for (int k = 0; k < kRun; ++k) part[wave - 1][k][lane] = acc[k];
    __syncthreads();
    if (wave > 0 || !rows.inside) return;
    const double bg = a.subtract_background ? a.qsum[prob] / (d.dv * double(d.npts)) : 0.0;
    double *out = reinterpret_cast<double *>(a.rho) + d.grid_off + rows.row + k0;
    const int kn = d.dims[2] - rows.g0[2] - k0;
#pragma unroll
    for (int k = 0; k < kRun; ++k) {
        double v = acc[k];
        for (int w = 0; w < kWays - 1; ++w) v += part[w][k][lane];
        if (k < kn) out[k] = v - bg;
    }
}

// the wavefront's sum, in lane 63 (every lane active; a fixed order): within
// rows of 16 lanes (row shifts by 1, 2, 4, 8), then across the rows (row
// broadcasts of lanes 15 and 31)
__device__ __forceinline__ double wave_sum63(double x)
{
    x = dpp_plus<0x111, 0xf>(x);
    x = dpp_plus<0x112, 0xf>(x);
    x = dpp_plus<0x114, 0xf>(x);
    x = dpp_plus<0x118, 0xf>(x);
    x = dpp_plus<0x142, 0xa>(x);
    x = dpp_plus<0x143, 0xc>(x);
    return x;
}

// adjoint: as in FP32, grad_rho of the brick in LDS and each wavefront with
// list entries of its own; the sums, in the triangular frame, are turned to
// Cartesian axes at the end
__global__ __launch_bounds__(64 * kWays) void k_adjoint_general64(SplatArgs a, int split)
{
    __shared__ double gr[kSeg][kRun][64];
    static_assert(kSeg == kWays, "one wavefront loads each run");
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6)), lane = threadIdx.x & 63;
    const int64_t b = blockIdx.x / split;
    const int share = blockIdx.x - int(b) * split;
    const int prob = brick_prob(a, b);
    const ProbDesc &d = a.desc[prob];
    const GenDesc &gd = a.gen[prob];
    const GenRows rows = gen_rows(d, gd, brick_pos(d, b), lane);
    const int64_t off = a.offsets[b];
    const int cnt = int(a.ends[b] - off);
    const int ways = kWays * split, way = kWays * share + wave;
    if (kWays * share >= cnt) return;
    {
        // zero outside the grid
        const int k0 = kRun * wave;
        const double *src = reinterpret_cast<const double *>(a.grad_rho) + d.grid_off + (rows.inside ? rows.row : 0);
#pragma unroll
        for (int k = 0; k < kRun; ++k)
            gr[wave][k][lane] = rows.inside && rows.g0[2] + k0 + k < d.dims[2] ? src[k0 + k] : 0.0;
    }
    __syncthreads();
    const double qc = 0.5 * a.cutoff * a.cutoff;
    for (int c0 = 0; c0 < cnt; c0 += 64 * ways) {
        const int mye = c0 + lane * ways + way;
        const GenAtom64 mine = gen_atom64(a, d, gd, rows.g0, off + mye, mye < cnt, qc);
        for (int q = 0; q < 64 && c0 + q * ways + way < cnt; ++q) {
            const GenRun rn = lane_run(mine.run, q);
            const double sc = lane_value(mine.sc, q);
            GenImages im;
            im.count = lane_value(mine.im.count, q);
            for (int x = 0; x < 3; ++x) {
                im.r[x] = lane_value(mine.im.r[x], q);
                im.u0[x] = lane_value(mine.im.u0[x], q);
                im.mc[x] = lane_value(mine.im.mc[x], q);
            }
            double f1 = 0.0, f2 = 0.0, f3 = 0.0;
            for (int i = 0; i < im.count; ++i) {
                const GenShift sh = gen_shift(im, d, gd, i, kBK / 2);  // (the brick's middle)
                // runs the sphere reaches: lane l < kSeg tests run l
                const int ol[3] = {0, 0, kRun * (lane & (kSeg - 1)) - kBK / 2};
                const uint32_t reach =
                    uint32_t(__ballot(box_distance2(gd, sh.p, ol, 7.0, 7.0, kRun - 1) * sc * sc <= kBoxMargin * qc));
#pragma unroll 1
                for (int seg = 0; seg < kSeg; ++seg) {
                    if (!((reach >> seg) & 1u) || rows.g0[2] + kRun * seg >= d.dims[2]) continue;
                    double d1, d2, s, tm;
                    if (!gen_row(gd, rows, sh.p, sc, rn.c, kRun * seg - kBK / 2, qc, d1, d2, s, tm)) continue;
                    double t[kRun], e[kRun];
                    bool in[kRun];
                    gen_exps(rn, s, tm, qc, t, in, e);
                    double fs = 0.0;
#pragma unroll
                    for (int j = 0; j < kRun; ++j) {
                        // (selected after the product: a non-finite grad_rho
                        // beyond the sphere does not reach the atom)
                        const double g = in[j] ? gr[seg][j][lane] * e[j] : 0.0;
                        fs += g;
                        f3 += g * t[j];
                    }
                    f1 += fs * d1;
                    f2 += fs * d2;
                }
            }
            f1 = wave_sum63(f1);
            f2 = wave_sum63(f2);
            f3 = wave_sum63(f3) / sc;
            const int64_t slot = off + c0 + q * ways + way;
            if (lane == 63 && slot < a.capacity)
                for (int x = 0; x < 3; ++x)
                    a.bpart[slot * 3 + x] = f1 * gd.frame[x] + f2 * gd.frame[3 + x] + f3 * gd.frame[6 + x];
        }
    }
}

hipError_t run_gather_general(const SplatArgs &a, hipStream_t s)
{
    const int nb = int(a.nbricks_total);
    if (a.fp64)
        hipLaunchKernelGGL(k_splat_general64, dim3(nb * kSeg), dim3(64 * kWays), 0, s, a);
    else if (nb < kFewBricks)
        hipLaunchKernelGGL(k_splat_general32<4>, dim3(nb * 8), dim3(256), 0, s, a);
    else
        hipLaunchKernelGGL(k_splat_general32<16>, dim3(nb * 2), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t run_adjoint_general(const SplatArgs &a, hipStream_t s)
{
    const int nb = int(a.nbricks_total);
    int split = nb < kFewBricks ? 8 : 2;
    if (a.fp64) {
        // More shares fill the chip and repeat a brick's culling.  us with the
        // binning, 1 / 2 / 4 / 8 shares, bricks of 8 x 8 x 32 and atoms as given:
        // 72 and 88: 221 / 136 / 89 / 74    300 and 409: 328 / 218 / 193 / 187
        // 784 and 1,123: 614 / 498 / 465 / 472    1,024 and 335: 167 / 160 / 170 / 200
        // 2,000 and 655: 279 / 276 / 302 / 365    7,200 and 11,059: 3,674 / 3,744 / 3,802 / 4,014
        if (nb >= kFewBricks && nb < 4 * kFewBricks) split = 4;
        hipLaunchKernelGGL(k_adjoint_general64, dim3(nb * split), dim3(64 * kWays), 0, s, a, split);
    } else {
        if (a.many && nb < kFewBricks)
            hipLaunchKernelGGL(k_adjoint_images32, dim3(nb * split), dim3(256), 0, s, a, split);
        else if (a.many)
            hipLaunchKernelGGL(k_adjoint_general32<true>, dim3(nb * split), dim3(256), 0, s, a, split);
        else
            hipLaunchKernelGGL(k_adjoint_general32<false>, dim3(nb * split), dim3(256), 0, s, a, split);
    }
    return hipGetLastError();
}

}  // namespace hartree

// FP64 splat and splat adjoint on the matrix cores (v_mfma_f64_16x16x4f64).
//
// The same bricks (16 x 16 columns (i, j) by 32 points along c) and the same
// two contractions per brick as the FP32 kernels:
//
//   splat    rho[c][k]  = sum_a  W_a gx_a(i_c) gy_a(j_c)  *  gz_a(k)
//   adjoint  S[c][a, f] = sum_k  grho[c][k]  *  gz_a(k) (f = 0) or gdz_a(k) (f = 1),
//            F_a = sum_c [gdx gy S0, gx gdy S0, gx gy S1]
//
// here with FP64 operands, FP64 factors (displacements and exponentials in
// double) and FP64 accumulation.  The matrix cores run FP64 at the vector
// units' rate; what they add is the operand reuse of a dense product.
//
// Operand layout of v_mfma_f64_16x16x4f64 (D = A B + C, A 16x4, B 4x16):
// lane l supplies A[l % 16][l / 16] and B[l / 16][l % 16]; after the call
// lane l holds D[4 r + l / 16][l % 16] in its accumulator element r = 0..3
// (rows interleaved across the lane groups, unlike the FP32 layouts).
// A 16-row tile is one i with its 16 j (row = j); wavefront w owns
// i = 4w .. 4w + 3.  Which reduction index sits in which K slot is free as
// long as A and B agree: the splat puts atom 4 m + l / 16 of a step in slot
// l / 16 of its product m; the adjoint puts points 8 m + 2 (l / 16) and the
// next in slot l / 16 of its products 2 m and 2 m + 1, so that each pair of
// products covers 8 consecutive points.
//
// Bound by the FP64 units, which the matrix products (64 cycles each) and the
// vector instructions of the factors share; an atom's window covers about half
// of the bricks it touches, and the products of the other half add zeros.  So
// the staged atoms are ordered by the part of the brick that their windows
// cover along c, then a, and products in which no atom of the step has a point
// are left out.  360^3, 4,096 atoms, 637,006 (atom, brick) pairs: splat 262 ->
// 228 us, adjoint 640 -> 446 us (of which the rows' pitch in LDS, which had set
// eight lanes on one bank in the fold: 120 us).
#include "splat_common.hpp"

namespace hartree {

typedef double doublex4 __attribute__((ext_vector_type(4)));

constexpr int kDThreads = 256;  // four wavefronts per brick
constexpr int kDStage = 128;    // records staged at once (whole lists, almost always)
constexpr int kDSub = 8;        // atoms per splat step: two K = 4 products per tile
constexpr int kDGroup = 8;      // atoms per adjoint group: 16 columns (g, gd)
static_assert(kDStage % kDSub == 0 && kDStage % kDGroup == 0 && kDStage <= kDThreads, "record staging");
static_assert(kMI + kMJ + kMK == 64, "one factor entry per lane");
static_assert(kMI == 16 && kMJ == 16 && kMK == 32, "the tiling below");

// What lane q (0 .. 63) of a wavefront evaluates for every atom: entry q of
// the atom's factor row over this brick (q < 16 along a, q < 32 along b, the
// rest along c): the axis, the point's offset within the brick, the axis
// length, whether the grid has the point, and the spacing h.
struct LaneAxis64 {
    int x, qq, n;
    int beyond;  // 2^30 where the point lies past the grid's end (no window is that wide), else 0
    double h;
};

__device__ __forceinline__ LaneAxis64 lane_axis64(const ProbDesc &d, const BrickPos &p, int q)
{
    LaneAxis64 la;
    la.x = q < kMI ? 0 : (q < kMI + kMJ ? 1 : 2);
    la.qq = q - (la.x == 0 ? 0 : (la.x == 1 ? kMI : kMI + kMJ));
    const int b = la.x == 0 ? p.b0 * kMI : (la.x == 1 ? p.b1 * kMJ : p.b2 * kMK);
    la.n = d.dims[la.x];
    la.beyond = b + la.qq < la.n ? 0 : 1 << 30;
    la.h = d.h[la.x];
    return la;
}

constexpr double kExpZero = -2000.0;  // exp64 gives 0

struct Entry64 {
    double g, gd;  // factor and displacement-weighted factor
    bool more;     // the window holds further images of this point
};

// This lane's entry of one staged atom: the unwrapped offsets r, r + n, ...
// inside the window width wl have grid index lo + r and displacement
// d = (lo + r) h - X; g = sum of exp(-d^2 / (2 sigma^2)), gd = the same
// weighted by d.  entry64 takes the first image; more_images64 adds the
// others (windows wider than the cell only).
__device__ __forceinline__ Entry64 entry64(const LaneAxis64 &la, const SlotAtom64 &at)
{
    const SlotAxis64 ax = at.ax[la.x];
    int r = ax.r0 + la.qq;
    r = r >= la.n ? r - la.n : r;
    const double d = double(ax.lo + r) * la.h - ax.X;
    // (chosen before the exponential, not after, so that it has no branch)
    const double e = exp64((r | la.beyond) < ax.wl ? -(d * d) * at.inv2s2 : kExpZero);
    return Entry64{e, e * d, ((r + la.n) | la.beyond) < ax.wl};
}

__device__ __forceinline__ void more_images64(const LaneAxis64 &la, const SlotAtom64 &at, double &gs, double &gds)
{
    const SlotAxis64 ax = at.ax[la.x];
    int r = ax.r0 + la.qq;
    r = r >= la.n ? r - la.n : r;
    for (r += la.n; (r | la.beyond) < ax.wl; r += la.n) {
        const double d = double(ax.lo + r) * la.h - ax.X;
        const double e = exp64(-(d * d) * at.inv2s2);
        gs += e;
        gds += e * d;
    }
}

// bit c: the window holds one of the points c len .. (c + 1) len - 1 of the brick
__device__ __forceinline__ int covered(const SlotAxis64 &ax, int n, int len)
{
    int m = 0;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const int q = n - ax.r0;  // the point where the next image's window begins
        const bool in = c * len < ax.wl - ax.r0 || (ax.wl > 0 && (c + 1) * len > q && c * len < q + ax.wl);
        m |= in ? 1 << c : 0;
    }
    return m;
}

// an order of the masks in which neighbours differ little: those from the
// brick's start by length, the whole brick, those up to its end
__device__ __forceinline__ int cover_key(int m) { return m & 1 ? __popc(m) : (m & 8 ? 8 - __popc(m) : 4); }

// A block of staged records: threads t < kDStage copy list entries c0 + t
// (empty records past nc) to LDS, each 64 of them in the order of what their
// windows cover; mask: bits 0 .. 3 the eights of points along c, bits 4 .. 7
// the wavefronts' planes.  The order within a key is the list's, so that the
// sums stay in a fixed order.
struct Stage64 {
    SlotAtom64 recs[kDStage];
    alignas(8) uint8_t mask[kDStage];
};
__device__ __forceinline__ void stage64(Stage64 &st, const SplatArgs &a, const ProbDesc &d, int64_t off, int c0, int nc,
                                        int t)
{
    if (t >= kDStage) return;
    SlotAtom64 r = a.rec64[off + c0 + (t < nc ? t : 0)];
    int key = 63, m = 0;
    if (t >= nc) {
#pragma unroll
        for (int x = 0; x < 3; ++x) r.ax[x].wl = 0;
    } else {
        const int mz = covered(r.ax[2], d.dims[2], kMK / 4), mx = covered(r.ax[0], d.dims[0], kMI / 4);
        const int kz = cover_key(mz), kx = cover_key(mx);
        m = mz | mx << 4;
        key = kz << 3 | (kz & 1 ? 8 - kx : kx);
    }
    uint64_t same = ~uint64_t(0);
    int rank = 0;
#pragma unroll
    for (int bit = 5; bit >= 0; --bit) {
        const bool one = (key >> bit) & 1;
        const uint64_t ones = __ballot(one);
        rank += one ? __popcll(same & ~ones) : 0;
        same &= one ? ones : ~ones;
    }
    const int lane = t & 63;
    rank += __popcll(same & ((uint64_t(1) << lane) - 1));
    const int to = (t & ~63) + rank;
    st.recs[to] = r;
    st.mask[to] = uint8_t(m);
}

// the masks of staged atoms s0 .. s0 + N - 1 together (N = 4 or 8)
template <int N>
__device__ __forceinline__ int group_mask(const Stage64 &st, int s0)
{
    uint32_t w = *reinterpret_cast<const uint32_t *>(st.mask + s0);
    if constexpr (N == 8) w |= *reinterpret_cast<const uint32_t *>(st.mask + s0 + 4);
    w = __builtin_amdgcn_readfirstlane(w);
    w |= w >> 16;
    return int((w | w >> 8) & 255);
}

__device__ __forceinline__ bool brick_inside(const ProbDesc &d, const BrickPos &p)
{
    return (p.b0 + 1) * kMI <= d.dims[0] && (p.b1 + 1) * kMJ <= d.dims[1] && (p.b2 + 1) * kMK <= d.dims[2];
}

// ---------------------------------------------------------------- splat

// One step's factors: row s holds entry q of staged atom s of the step (W gx
// along a, then gy, then gz).  The pitch sets the rows that half a wavefront
// reads together on different banks.
constexpr int kFacPitch = 80;
struct SplatBuf64 {
    double f[kDSub][kFacPitch];
};

// factors of staged atoms s0 .. s0 + kDSub - 1 into buf: wavefront w evaluates
// atoms w and w + 4 of the step, lane q entry q
template <bool WIDE>
__device__ __forceinline__ void splat_factors64(SplatBuf64 &buf, const SlotAtom64 *recs, const LaneAxis64 &la,
                                                int wave, int lane)
{
    constexpr int R = kDSub / 4;
    double v[R];
    bool more = false;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const Entry64 e = entry64(la, recs[wave + 4 * r]);
        v[r] = e.g;
        more = more || e.more;
    }
    if constexpr (WIDE) {
        if (__any(more)) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                double gd = 0.0;
                more_images64(la, recs[wave + 4 * r], v[r], gd);
            }
        }
    }
#pragma unroll
    for (int r = 0; r < R; ++r)
        buf.f[wave + 4 * r][lane] = v[r] * (la.x == 0 ? recs[wave + 4 * r].w : 1.0);
}

// products of one step: acc[u][c] is the tile of i = 4 wave + u and points
// k = 16 c .. 16 c + 15
__device__ __forceinline__ void splat_products64(const SplatBuf64 &buf, const Stage64 &st, int s0, int wave, int lane,
                                                 doublex4 (&acc)[4][2])
{
    const int jj = lane & 15, kq = lane >> 4;
#pragma unroll
    for (int m = 0; m < kDSub / 4; ++m) {
        const int mask = group_mask<4>(st, s0 + 4 * m);
        if (!((mask >> (4 + wave)) & 1)) continue;
        const double *f = buf.f[4 * m + kq];
        const double y = f[kMI + jj];
        double av[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) av[u] = f[4 * wave + u] * y;
        if (mask & 3) {
            const double b = f[kMI + kMJ + jj];
#pragma unroll
            for (int u = 0; u < 4; ++u) acc[u][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[u], b, acc[u][0], 0, 0, 0);
        }
        if (mask & 12) {
            const double b = f[kMI + kMJ + 16 + jj];
#pragma unroll
            for (int u = 0; u < 4; ++u) acc[u][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[u], b, acc[u][1], 0, 0, 0);
        }
    }
}

template <bool WIDE>
__global__ __launch_bounds__(kDThreads) void k_splat_mfma64(SplatArgs a)
{
    __shared__ Stage64 st;
    __shared__ SplatBuf64 fac[2];  // double buffer of pipeline steps
    const int64_t b = brick_of_block(a);
    const int prob = brick_prob(a, b);
    const ProbDesc &d = a.desc[prob];
    const BrickPos p = brick_pos(d, b);
    const int t = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63;
    const int64_t off = a.offsets[b];
    const int cnt = int(a.ends[b] - off);
    const LaneAxis64 la = lane_axis64(d, p, lane);

    // the accumulators start at the background -Q / Omega
    const double bg = a.subtract_background ? a.qsum[prob] / (d.L[0] * d.L[1] * d.L[2]) : 0.0;
    doublex4 acc[4][2];
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int c = 0; c < 2; ++c) acc[u][c] = doublex4{-bg, -bg, -bg, -bg};

    for (int blk = 0; blk < cnt; blk += kDStage) {
        const int nb = (cnt - blk) < kDStage ? (cnt - blk) : kDStage;
        stage64(st, a, d, off, blk, nb, t);
        __syncthreads();
        const int nsub = (nb + kDSub - 1) / kDSub;
        splat_factors64<WIDE>(fac[0], st.recs, la, wave, lane);
        __syncthreads();
        for (int c = 0; c + 1 < nsub; ++c) {
            splat_factors64<WIDE>(fac[(c + 1) & 1], st.recs + (c + 1) * kDSub, la, wave, lane);
            splat_products64(fac[c & 1], st, c * kDSub, wave, lane, acc);
            __syncthreads();
        }
        splat_products64(fac[(nsub - 1) & 1], st, (nsub - 1) * kDSub, wave, lane, acc);
        __syncthreads();  // st and fac are reused by the next block
    }
    // lane l holds rows j = 4 r + l / 16 at point k = 16 c + l % 16
    double *out = reinterpret_cast<double *>(a.rho) + d.grid_off;
    const int64_t sb = d.dims[2], sa = int64_t(d.dims[1]) * d.dims[2];  // row strides along b and a
    const int kq = lane >> 4, kl = lane & 15;
    if (brick_inside(d, p)) {
        // a wavefront-uniform base plus a 32-bit lane offset
        double *base = out + (int64_t(p.b0 * kMI + 4 * wave) * d.dims[1] + p.b1 * kMJ) * sb + p.b2 * kMK;
        const uint32_t loff = uint32_t(kq * d.dims[2] + kl);
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                double *row = base + (u * sa + 4 * r * sb);
                row[loff] = acc[u][0][r];
                row[loff + 16] = acc[u][1][r];
            }
        return;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int ia = p.b0 * kMI + 4 * wave + u;
        if (ia >= d.dims[0]) continue;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int j = p.b1 * kMJ + 4 * r + kq;
            if (j >= d.dims[1]) continue;
            double *row = out + (int64_t(ia) * d.dims[1] + j) * sb;
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const int k = p.b2 * kMK + 16 * c + kl;
                if (k < d.dims[2]) row[k] = acc[u][c][r];
            }
        }
    }
}

// ---------------------------------------------------------------- adjoint

// One group's factors: xy[s][q] = gx (q < 16) or gy (16 <= q < 32) of staged
// atom s of the group, xy[8 + s] the displacement-weighted ones; bz[n][k]:
// matrix column n < 8 is gz of atom n, n >= 8 gdz of atom n - 8.  The pitches
// keep the lanes' reads of a row element each (xy: eight atoms and four j; bz:
// 16 columns) in different banks.
constexpr int kXyPitch = kMI + kMJ + 4, kBzPitch = kMK + 2;
struct AdjBuf64 {
    double xy[2 * kDGroup][kXyPitch];
    double bz[2 * kDGroup][kBzPitch];
};

// factors of staged atoms s0 .. s0 + kDGroup - 1 into buf: wavefront w
// evaluates atoms w and w + 4 of the group, lane q entry q
template <bool WIDE>
__device__ __forceinline__ void adjoint_factors64(AdjBuf64 &buf, const SlotAtom64 *recs, const LaneAxis64 &la,
                                                  int wave, int lane)
{
    constexpr int R = kDGroup / 4;
    Entry64 v[R];
    bool more = false;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        v[r] = entry64(la, recs[wave + 4 * r]);
        more = more || v[r].more;
    }
    if constexpr (WIDE) {
        if (__any(more)) {
#pragma unroll
            for (int r = 0; r < R; ++r) more_images64(la, recs[wave + 4 * r], v[r].g, v[r].gd);
        }
    }
    // (one address per lane for both kinds of row)
    const bool z = lane >= kMI + kMJ;
    double *row = z ? &buf.bz[0][la.qq] : &buf.xy[0][lane];
    const int pitch = z ? kBzPitch : kXyPitch;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        row[(wave + 4 * r) * pitch] = v[r].g;
        row[(wave + 4 * r + kDGroup) * pitch] = v[r].gd;
    }
}

// One group's products over the eights M0 .. M1 - 1 of the brick's points along
// c: acc[u] is S of the tile i = 4 wave + u, columns n = lane % 16, rows
// j = 4 r + lane / 16
template <int M0, int M1>
__device__ __forceinline__ void adjoint_products64(const AdjBuf64 &buf, const double (&g)[4][8], int lane,
                                                   doublex4 (&acc)[4])
{
    const int n = lane & 15, kq = lane >> 4;
    const double *bcol = &buf.bz[n][2 * kq];
#pragma unroll
    for (int u = 0; u < 4; ++u) acc[u] = doublex4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int m = M0; m < M1; ++m) {
        const double2 bv = *reinterpret_cast<const double2 *>(bcol + 8 * m);
#pragma unroll
        for (int u = 0; u < 4; ++u) acc[u] = __builtin_amdgcn_mfma_f64_16x16x4f64(g[u][2 * m], bv.x, acc[u], 0, 0, 0);
#pragma unroll
        for (int u = 0; u < 4; ++u)
            acc[u] = __builtin_amdgcn_mfma_f64_16x16x4f64(g[u][2 * m + 1], bv.y, acc[u], 0, 0, 0);
    }
}

// the sum of v over the four lane groups: ((0 + 1) + (2 + 3)), in every lane
__device__ __forceinline__ double sum_groups(double v)
{
    auto swapped = [](double x, auto swap) {
        const uint64_t q = __double_as_longlong(x);
        const auto lo = swap(uint32_t(q)), hi = swap(uint32_t(q >> 32));
        return __longlong_as_double(uint64_t(hi[0]) << 32 | lo[0]) + __longlong_as_double(uint64_t(hi[1]) << 32 | lo[1]);
    };
    v = swapped(v, [](uint32_t w) { return __builtin_amdgcn_permlane16_swap(w, w, false, false); });
    return swapped(v, [](uint32_t w) { return __builtin_amdgcn_permlane32_swap(w, w, false, false); });
}

// The fold with the transverse factors, then the sum over the four lane
// groups (fixed butterfly); lanes n < 16 write the wavefront's partials to
// red[n][0 .. 1]: [0] the x component (f = 0) or the z component (f = 1),
// [1] the y component (f = 0; f = 1 lanes compute a value nobody reads,
// which keeps the fold free of branches).
__device__ __forceinline__ void adjoint_fold64(const AdjBuf64 &buf, const doublex4 (&acc)[4], int wave, int lane,
                                               double (*red)[2])
{
    const int n = lane & 15, kq = lane >> 4;
    const int f = n >> 3, sl = n & 7;
    const double *gxy = buf.xy[sl], *gdxy = buf.xy[kDGroup + sl];
    const double *cx = f == 0 ? gdxy : gxy;
    double ax = 0.0, ay = 0.0;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        double sy = 0.0, sdy = 0.0;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int j = kMI + 4 * r + kq;
            sy += gxy[j] * acc[u][r];
            sdy += gdxy[j] * acc[u][r];
        }
        const int i = 4 * wave + u;
        ax += cx[i] * sy;
        ay += gxy[i] * sdy;
    }
    ax = sum_groups(ax);
    ay = sum_groups(ay);
    if (kq == 0) {
        red[n][0] = ax;
        red[n][1] = ay;
    }
}

// fixed-order sum over the 4 wavefronts of the partials of staged atoms
// s0 .. s0 + kDGroup - 1 (below nb), stored under (atom, touched brick)
// from their records: threads t < 24
__device__ __forceinline__ void adjoint_reduce64(const SplatArgs &a, const double (*red)[2 * kDGroup][2],
                                                 const SlotAtom64 *recs, int s0, int nb, int t)
{
    if (t < 3 * kDGroup) {
        const int st = t / 3, x = t - 3 * st;
        const int nn = x == 2 ? kDGroup + st : st;
        const int comp = x == 1 ? 1 : 0;
        double v = 0.0;
        for (int w = 0; w < 4; ++w) v += red[w][nn][comp];
        if (s0 + st < nb) {
            const SlotAtom64 &r = recs[s0 + st];
            a.bpart[(int64_t(r.atom) * a.cap_pa + r.touch) * 3 + x] = v;
        }
    }
}

// One group of the adjoint with products over the eights M0 .. M1 - 1 only
// (whole bodies per range, not branches around products: the accumulators
// then stay in place, and the next group's factors are evaluated while the
// products run)
template <bool WIDE, int M0, int M1>
__device__ __forceinline__ void adjoint_group64(const AdjBuf64 &buf, AdjBuf64 &nbuf, const SlotAtom64 *next,
                                                const LaneAxis64 &la, const double (&g)[4][8], int wave, int lane,
                                                double (*red)[2])
{
    doublex4 acc[4];
    adjoint_products64<M0, M1>(buf, g, lane, acc);
    if (next) adjoint_factors64<WIDE>(nbuf, next, la, wave, lane);
    adjoint_fold64(buf, acc, wave, lane, red);
}

// adjoint: wave w holds grad_rho of its four row tiles in registers; per
// group of 8 staged atoms it forms S for them (16 columns n = 8 f + atom)
// and folds the transverse factors in.  The products of a group are issued
// first, the next group's factors are evaluated while they run, then the
// fold; the previous group's partials are reduced at the top.
template <bool WIDE>
__global__ __launch_bounds__(kDThreads) __attribute__((amdgpu_waves_per_eu(3))) void k_adjoint_mfma64(SplatArgs a)
{
    __shared__ Stage64 st;
    __shared__ AdjBuf64 buf[2];
    __shared__ double red[2][4][2 * kDGroup][2];  // [group parity][wave][n][component]
    const int64_t b = brick_of_block(a);
    const int prob = brick_prob(a, b);
    const ProbDesc &d = a.desc[prob];
    const BrickPos p = brick_pos(d, b);
    const int t = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63;
    const int64_t off = a.offsets[b];
    const int cnt = int(a.ends[b] - off);
    if (cnt == 0) return;
    const LaneAxis64 la = lane_axis64(d, p, lane);

    // grad_rho of this lane's A rows: tile u (i = 4 wave + u), row j = lane
    // % 16, points k = 8 m + 2 (lane / 16) + e in g[u][2 m + e].  Loads outside
    // the grid read the workspace's zero block.
    double g[4][8];
    const double *src = reinterpret_cast<const double *>(a.grad_rho) + d.grid_off;
    const int jj = lane & 15, kq = lane >> 4;
    const int64_t sb = d.dims[2], sa = int64_t(d.dims[1]) * d.dims[2];
    if (a.grad_rows_vec16 && brick_inside(d, p) && (d.dims[2] & 1) == 0 && (d.grid_off & 1) == 0) {
        // a wavefront-uniform base plus a 32-bit lane offset, 16-byte loads
        const double *base = src + (int64_t(p.b0 * kMI + 4 * wave) * d.dims[1] + p.b1 * kMJ) * sb + p.b2 * kMK;
        const uint32_t loff = uint32_t(jj * d.dims[2] + 2 * kq);
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int ks = 0; ks < 8; ks += 2) {
                const double2 v = *reinterpret_cast<const double2 *>(base + u * sa + loff + 4 * ks);
                g[u][ks] = v.x;
                g[u][ks + 1] = v.y;
            }
    } else {
        const double *zeros = reinterpret_cast<const double *>(a.zeros);
        const int j = p.b1 * kMJ + jj;
        const int k0 = p.b2 * kMK + 2 * kq;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int ia = p.b0 * kMI + 4 * wave + u;
            const bool in = ia < d.dims[0] && j < d.dims[1];
            const double *row = src + (in ? (int64_t(ia) * d.dims[1] + j) * sb + k0 : 0);
#pragma unroll
            for (int ks = 0; ks < 8; ++ks) {
                const int k = 8 * (ks / 2) + ks % 2;
                g[u][ks] = *(in && k0 + k < d.dims[2] ? row + k : zeros);
            }
        }
    }

    for (int blk = 0; blk < cnt; blk += kDStage) {
        const int nb = (cnt - blk) < kDStage ? (cnt - blk) : kDStage;
        stage64(st, a, d, off, blk, nb, t);
        __syncthreads();
        const int ngroup = (nb + kDGroup - 1) / kDGroup;
        adjoint_factors64<WIDE>(buf[0], st.recs, la, wave, lane);
        __syncthreads();
        for (int gi = 0; gi < ngroup; ++gi) {
            if (gi > 0) adjoint_reduce64(a, red[(gi - 1) & 1], st.recs, (gi - 1) * kDGroup, nb, t);
            const int mask = group_mask<8>(st, gi * kDGroup);
            const SlotAtom64 *next = gi + 1 < ngroup ? st.recs + (gi + 1) * kDGroup : nullptr;
            AdjBuf64 &cur = buf[gi & 1], &nxt = buf[(gi + 1) & 1];
            double (*rw)[2] = red[gi & 1][wave];
            if (!((mask >> (4 + wave)) & 1)) {
                if (next) adjoint_factors64<WIDE>(nxt, next, la, wave, lane);
                if (lane < 2 * kDGroup) rw[lane][0] = rw[lane][1] = 0.0;
            } else if ((mask & 12) == 0) {
                adjoint_group64<WIDE, 0, 2>(cur, nxt, next, la, g, wave, lane, rw);
            } else if ((mask & 3) == 0) {
                adjoint_group64<WIDE, 2, 4>(cur, nxt, next, la, g, wave, lane, rw);
            } else if ((mask & 8) == 0) {
                adjoint_group64<WIDE, 0, 3>(cur, nxt, next, la, g, wave, lane, rw);
            } else if ((mask & 1) == 0) {
                adjoint_group64<WIDE, 1, 4>(cur, nxt, next, la, g, wave, lane, rw);
            } else {
                adjoint_group64<WIDE, 0, 4>(cur, nxt, next, la, g, wave, lane, rw);
            }
            __syncthreads();
        }
        adjoint_reduce64(a, red[(ngroup - 1) & 1], st.recs, (ngroup - 1) * kDGroup, nb, t);
        __syncthreads();  // st, buf and red are reused by the next block
    }
}

hipError_t run_gather_mfma64(const SplatArgs &a, hipStream_t s)
{
    const dim3 grid(int(a.nbricks_total)), block(kDThreads);
    if (a.wide)
        hipLaunchKernelGGL(k_splat_mfma64<true>, grid, block, 0, s, a);
    else
        hipLaunchKernelGGL(k_splat_mfma64<false>, grid, block, 0, s, a);
    return hipGetLastError();
}

hipError_t run_adjoint_mfma64(const SplatArgs &a, hipStream_t s)
{
    const dim3 grid(int(a.nbricks_total)), block(kDThreads);
    if (a.wide)
        hipLaunchKernelGGL(k_adjoint_mfma64<true>, grid, block, 0, s, a);
    else
        hipLaunchKernelGGL(k_adjoint_mfma64<false>, grid, block, 0, s, a);
    return hipGetLastError();
}

}  // namespace hartree

// Host-side dispatch of the grid passes and the E_H finalize kernel.
#include "fft_passes.hpp"

namespace hartree {

hipError_t run_r2c_f32(int, int, int, hipStream_t, const PassArgs &);
hipError_t run_r2c_f64(int, int, int, hipStream_t, const PassArgs &);
hipError_t run_c2r_f32(int, int, int, hipStream_t, const PassArgs &);
hipError_t run_c2r_f64(int, int, int, hipStream_t, const PassArgs &);
hipError_t run_b_f32(int, int, int, hipStream_t, const PassArgs &);
hipError_t run_b_f64(int, int, int, hipStream_t, const PassArgs &);
hipError_t run_a_f32(int, int, int, hipStream_t, const PassArgs &);
hipError_t run_a_f64(int, int, int, hipStream_t, const PassArgs &);

// ---------------------------------------------------------------- E_H
// one workgroup per problem: fixed-order sum of that problem's partials
// one workgroup per problem: each thread sums its strided share of the
// partials in four independent chains (the loads issue together), then a
// fixed butterfly per wavefront and a fixed-order sum over the wavefronts
constexpr int kFinThreads = 1024;

__global__ __launch_bounds__(kFinThreads) void k_finalize(const ProbDesc *desc, const double *partials, double *e_h)
{
    __shared__ double red[kFinThreads / 64];
    const ProbDesc &d = desc[blockIdx.x];
    const double *pp = partials + d.part_off;
    const int t = threadIdx.x;
    double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
    int i = t;
    for (; i + 3 * kFinThreads < d.nparts; i += 4 * kFinThreads) {
        s0 += pp[i];
        s1 += pp[i + kFinThreads];
        s2 += pp[i + 2 * kFinThreads];
        s3 += pp[i + 3 * kFinThreads];
    }
    for (; i < d.nparts; i += kFinThreads) s0 += pp[i];
    double s = (s0 + s1) + (s2 + s3);
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off, 64);
    if ((t & 63) == 0) red[t >> 6] = s;
    __syncthreads();
    if (t == 0) {
        double tot = 0.0;
        for (int w = 0; w < kFinThreads / 64; ++w) tot += red[w];
        e_h[blockIdx.x] = d.eh_scale * tot;
    }
}

// Pencils per workgroup for a length and its stage radices (log2; -1 if the
// length does not fit): enough threads per pencil that every stage's
// butterflies fit the registers, at most 64 pencils, and a tile that leaves
// room for two workgroups per CU.
int pass_min_tpp(int fp64, int n, const int *radix, int nstages)
{
    int tpp = 1;
    for (int s = 0; s < nstages; ++s) {
        const int nb = n / radix[s];
        const int mb = fp64 ? stage_maxb<double>(radix[s]) : stage_maxb<float>(radix[s]);
        const int need = (nb + mb - 1) / mb;
        while (tpp < need) tpp <<= 1;
    }
    return tpp;
}

size_t pass_tile_lds(int fp64, int n, int p_log2, int pad)
{
    const size_t P = size_t(1) << p_log2, cx = fp64 ? 16 : 8;
    const size_t strided = (P + size_t(pad)) * n, rows = P * (n + 31);
    return cx * ((strided > rows ? strided : rows) + n);
}

// Bank-conflict model of the strided tiles (element (i, p) at i (P + pad) + p):
// for every LDS access of every stage, the passes a wavefront needs on 64
// banks of 4 bytes, relative to the conflict-free count.
static double strided_lds_cost(int fp64, int n, const int *radix, int nstages, int p_log2, int pad)
{
    const int P = 1 << p_log2, tpp = kPassThreads >> p_log2, pitch = P + pad, wpe = fp64 ? 4 : 2;
    double total = 0.0, ideal = 0.0;
    int ns = 1;
    int count[64];
    for (int st = 0; st < nstages; ++st) {
        const int R = radix[st], nb = n / R, maxb = (nb + tpp - 1) / tpp;
        for (int wave = 0; wave < kPassThreads / 64; ++wave)
            for (int m = 0; m < maxb; ++m)
                for (int dir = 0; dir < 2; ++dir)
                    for (int q = 0; q < R; ++q) {
                        for (int b = 0; b < 64; ++b) count[b] = 0;
                        int lanes = 0;
                        for (int l = 0; l < 64; ++l) {
                            const int tid = wave * 64 + l, p = tid & (P - 1), tip = tid >> p_log2;
                            const int j = tip + m * tpp;
                            if (j >= nb) continue;
                            const int i = dir == 0 ? j + q * nb : (j / ns) * ns * R + j % ns + q * ns;
                            const long w0 = long(i * pitch + p) * wpe;
                            for (int k = 0; k < wpe; ++k) count[(w0 + k) & 63] += 1;
                            ++lanes;
                        }
                        if (!lanes) continue;
                        int mx = 0;
                        for (int b = 0; b < 64; ++b) mx = count[b] > mx ? count[b] : mx;
                        total += mx;
                        ideal += (lanes * wpe + 63) / 64;
                    }
        ns *= R;
    }
    return ideal > 0.0 ? total / ideal : 1.0;
}

// the LDS pitch pad with the fewest modelled bank conflicts
static int modelled_pad(int fp64, int n, const int *radix, int nstages, int p_log2)
{
    int best = 1;
    double cbest = 0.0;
    for (int pad = 0; pad <= 3; ++pad) {
        const double c = strided_lds_cost(fp64, n, radix, nstages, p_log2, pad);
        if (pad == 0 || c < cbest - 1e-9) {
            cbest = c;
            best = pad;
        }
    }
    return best;
}

int pass_p_log2(int fp64, int n, const int *radix, int nstages, int max_p)
{
    const int tpp = pass_min_tpp(fp64, n, radix, nstages);
    if (tpp > kPassThreads) return -1;
    int P = kPassThreads / tpp;
    if (P > max_p) P = max_p;
    const size_t cx = fp64 ? 16 : 8;
    while (P > 1 && size_t(row_pitch(n) > n + 1 ? row_pitch(n) : n + 1) * (P + 1) * cx > 80 * 1024) P >>= 1;
    int l = 0;
    while ((1 << l) < P) ++l;
    return l;
}

// a CU's LDS, less what the kernels hold beside the tile
constexpr size_t kCuLds = 160 * 1024 - 256;

size_t runtime_lds(int fp64, int x, int n, int p_log2, int pad, bool &twg)
{
    const size_t cx = fp64 ? 16 : 8, P = size_t(1) << p_log2;
    const size_t copy = x == 2 ? P * size_t(row_pitch(n)) : (P + size_t(pad)) * size_t(n);
    twg = cx * (2 * copy + size_t(n)) > kCuLds;
    return cx * (2 * copy + (twg ? 0 : size_t(n)));
}

// the tile a run-time radix pass takes for a requested one: the pad, then
// pencils, given up until two copies and the twiddles fit (a single pencil of
// the longest lengths in double reads its twiddles from global memory)
void runtime_tile(int fp64, int x, int n, int &p_log2, int &pad)
{
    bool twg;
    while (runtime_lds(fp64, x, n, p_log2, pad, twg) > kCuLds || twg) {
        if (pad > 0) pad = 0;
        else if (p_log2 > 0) --p_log2;
        else break;
    }
}

// Default pencils per tile of the run-time radix passes.  Long lengths: as many as
// leave a CU room for two to four such workgroups, as its kernel's registers
// allow, and no more than pay.  Measured (us, FP32 unless noted):
//   a  n = 75: 8 34.8, 16 26.0, 32 22.8; n = 252: 4 82, 8 62, 16 75 (past a third
//      of the LDS); FP64, two wavefronts per SIMD: n = 135: 8 42, 16 34, 32 39
//   b  n = 168: 4 15.1, 8 12.6, 16 16.7; n = 625: 2 20.4, 4 18.9, 8 27.5
//   c  n = 189: 4 16.9, 8 16.4, 16 21.4; n = 280: 2 64, 4 47, 8 57 (past a fourth)
// Along a and b a short length has few butterflies to a pencil, and only wide
// tiles occupy the 256 threads: up to 256, 3,072 points (2,048 along b) in at most
// 64 pencils, and fewer where that leaves less than 384 tiles (256 along a in
// FP64) or half of each empty.  (Not in a batch, whose problems share a launch
// where their tiles have one width.)
//   a  n = 16 of 16 x 64 x 2048: 16 34.1, 32 22.4, 64 18.2; of 16 x 40 x 48: 4 to 32 9 to 10, 64 11.5;
//      n = 35 of 35 x 192 x 192 (291 tiles of 64, 582 of 32): 32 14.4, 64 18.7
//      FP64 n = 4 of 4 x 360 x 360: 16 33.4, 64 12.9; n = 144 of 144 x 360 x 360: 4 284, 16 158
//   b  n = 16 of 64 x 16 x 2048: 8 43.5, 64 19.0; FP64 n = 9 of 360 x 9 x 360: 8 39.0, 64 19.7
static int runtime_default_p_log2(int fp64, int x, int n, const TileGrid &g)
{
    bool twg;
    const bool wide = x < 2 && n <= 256 && !g.batch;
    int lp = wide ? 6 : (x == 0 ? (fp64 ? 4 : 5) : 3);
    const size_t most = kCuLds / (x == 0 ? (fp64 ? 2 : 3) : (x == 1 || fp64 ? 3 : 4));
    const int points = x == 0 ? 3072 : 2048;
    while (lp > 0 && (runtime_lds(fp64, x, n, lp, 0, twg) > most || twg || (wide && n << lp > points))) --lp;
    const int least = x == 0 && fp64 ? 256 : 384;
    while (wide && lp > 3 && !g.enough(lp, least)) --lp;
    return lp;
}

#define HARTREE_ROW(R0, R1, R2, R3) {R0, R1, R2, R3},
static const int kPlanTable[][4] = {HARTREE_PLANS(HARTREE_ROW)};
#undef HARTREE_ROW

int plan_table_size() { return int(sizeof(kPlanTable) / sizeof(kPlanTable[0])); }

int plan_table_row(int id, int *radix)
{
    int ns = 0;
    for (int s = 0; s < 4; ++s) {
        radix[s] = kPlanTable[id][s];
        if (radix[s] > 0) ns = s + 1;
    }
    return ns;
}

// index of a radix sequence in HARTREE_PLANS, or -1
int find_plan(const int *radix, int nstages)
{
    const auto &plans = kPlanTable;
    const int np = plan_table_size();
    for (int i = 0; i < np; ++i) {
        bool same = true;
        for (int s = 0; s < 4; ++s) same = same && plans[i][s] == (s < nstages ? radix[s] : 0);
        if (same && nstages <= 4) return i;
    }
    return -1;
}

// Default pencils per tile of the compiled passes.  A wide strided tile reads
// long contiguous segments, a narrow one leaves a CU room for more workgroups
// and cuts a short grid into more of them; 64 KB and more of LDS for a tile
// (64 pencils up to n = 150, 32 up to 256, 16 up to 512) leaves two per CU.
// Measured (us; a forward / with E_H, b forward / inverse, c r2c / c2r; n^3):
//   FP32 a  n = 96: 16 10.8 / 9.4, 64 15.6 / 15.9; 180: 16 18.9 / 18.4, 32 21.8 / 21.3; 192: 8 18.8 / 17.8,
//           16 23.4 / 18.6, 32 28.7 / 28.2; 360: 8 82 / 79, 16 93 / 91; 256: 8 47.9, 16 34.7, 32 42.2 (rows a
//           power of two apart share few cache sets: the wide tile's longer segments win, so too at 512)
//   FP32 b  n = 120: 16 8.0 / 10.4, 64 11.6 / 14.1; 192: 8 13.7 / 16.4, 32 19.1 / 20.2; 360: 8 66 / 67, 16 70 / 71
//   FP64 a  n = 120: 8 16.1, 16 18.1, 32 19.6; 192: 4 32.6, 8 29.4, 16 38.4; 300: 4 98, 8 90; 420: 4 316, 8 379 (the
//           kernels of 4 and 8 without pad are compiled for them); 256: 8 74, 16 60; 512: 4 572, 8 535
//   FP64 b  n = 150: 16 12.2, 32 19.2; 192: 8 23.3, 16 26.9
//   c       FP32 n = 128: 4 11.3 / 14.5, 8 9.7 / 10.5; 192: 4 19.9 / 16.6, 8 17.8 / 11.6; 180: 4 19.9 / 16.9,
//           8 14.8 / 20.5; 288: 4 41 / 42, 8 38 / 54 (half-wavefronts on two rows: no conflict where n is a
//           multiple of 16); FP64 n = 128: 4 20.9 / 17.7, 8 14.6 / 12.2; 300: 97 / 80, 84 / 85; 360: 142 / 161, 168 / 169
// FP32 tiles of 16 take a pitch pad of one, so that the kernels are the ones
// of every other width: those with 16 compiled in round some lengths'
// butterflies in another order and are 0 to 10 % faster.
// On grids other than cubes (both passes):
//   short lengths, where plans of two stages leave the threads of a narrow
//   tile without a butterfly (n = 64: 8 a pencil), once there are tiles enough
//   of a width that some run more than half fills:
//     FP32 a  32 x 360 x 360: 16 29.3, 32 20.5, 64 18.2; 64 x 64 x 2048: 16 41.6, 32 30.3, 64 32.6
//     FP32 b  64 x 32 x 2048: 16 31.9, 64 25.7; 400 x 48 x 20 (400 tiles): 16 13.2, 64 15.4
//     FP64 a  64 x 100 x 300: 8 26.9, 16 25.1, 32 20.9; 64 x 400 x 20 (138 tiles of 32): 8 14.5, 16 16.5, 32 15.2;
//             72 x 360 x 360: 8 73.9, 16 64.9, 32 58.9; 160 x 16 x 4096: 8 70.0, 16 61.8; 60 (three stages) of
//             60 x 192 x 192: 8 22.1, 32 29.4
//     FP64 b  192 x 32 x 192: 16 19.7, 32 18.7; 400 x 256 x 20: 8 29.3, 16 25.7
//   long pencils along c in FP64 with less than 256 tiles: 12 x 10 x 200: 4 13.8, 8 16.4; 48 x 40 x 288: 4 15.9, 8 19.4
void default_tile(int fp64, int x, int n, const int *radix, int nstages, const TileGrid &g, int &p_log2, int &pad)
{
    const int widest = pass_p_log2(fp64, n, radix, nstages, 64);
    p_log2 = widest;
    pad = 0;
    if (widest < 0) return;
    if (find_plan(radix, nstages) < 0) {  // (no more pencils than set_config accepts)
        p_log2 = std::min(widest, runtime_default_p_log2(fp64, x, n, g));
        return;
    }
    if (x == 2) {
        const bool eight = fp64 ? n <= 300 && (n < 160 || g.tiles(3) >= 256) : n <= 160 || (n <= 256 && n % 16 == 0);
        p_log2 = std::min(widest, eight ? 3 : 2);
        return;
    }
    const bool pow2 = (n & (n - 1)) == 0;
    if (fp64) {
        const bool two = nstages == 2 && n <= 256;
        const int wide = x == 0 ? 96 : 48;  // the longest such length that 32 pencils still pay for
        if (two && n <= wide && widest >= 5 && g.enough(5, 256)) {
            p_log2 = 5;
            return;
        }
        if (two && (x == 0 || n == 256) && widest >= 4 && g.enough(4, x == 0 ? 512 : 256)) {
            p_log2 = 4;
            return;
        }
        if (x == 0 && n != 256) {
            p_log2 = std::min(widest, n <= 320 || pow2 ? 3 : 2);
            return;
        }
        p_log2 = std::min(widest, x == 0 || n <= 160 ? 4 : 3);
        // (among those no larger in LDS than a pad of one)
        pad = modelled_pad(fp64, n, radix, nstages, p_log2);
        if (pass_tile_lds(fp64, n, p_log2, pad) > pass_tile_lds(fp64, n, p_log2, 1)) pad = 1;
        return;
    }
    for (int lp = n <= 48 ? 6 : 5; lp >= 5 && n <= 64; --lp)
        if (widest >= lp && g.enough(lp, 512)) {
            p_log2 = lp;
            pad = 1;  // (in a batch no multi-plan tile, which would round otherwise)
            return;
        }
    p_log2 = std::min(widest, n <= 180 || pow2 ? 4 : 3);
    pad = p_log2 == 4 && n < 512 ? 1 : 0;
}

hipError_t run_pass(int fp64, PassKind kind, int plan, int p_log2, int pad, int maxn, int grid, hipStream_t s,
                    const PassArgs &a0)
{
    PassArgs a = a0;
    a.mode = 0;
    a.inv = 0;
    a.p_log2 = p_log2;
    a.pad = pad;
    switch (kind) {
    case PASS_R2C_FWD: return fp64 ? run_r2c_f64(plan, maxn, grid, s, a) : run_r2c_f32(plan, maxn, grid, s, a);
    case PASS_R2C_BWD:
        a.mode = 1;
        return fp64 ? run_r2c_f64(plan, maxn, grid, s, a) : run_r2c_f32(plan, maxn, grid, s, a);
    case PASS_C2R: return fp64 ? run_c2r_f64(plan, maxn, grid, s, a) : run_c2r_f32(plan, maxn, grid, s, a);
    case PASS_B_FWD: return fp64 ? run_b_f64(plan, maxn, grid, s, a) : run_b_f32(plan, maxn, grid, s, a);
    case PASS_B_INV:
        a.inv = 1;
        return fp64 ? run_b_f64(plan, maxn, grid, s, a) : run_b_f32(plan, maxn, grid, s, a);
    case PASS_A_FULL: return fp64 ? run_a_f64(plan, maxn, grid, s, a) : run_a_f32(plan, maxn, grid, s, a);
    case PASS_A_NOENERGY:
        a.mode = 1;
        return fp64 ? run_a_f64(plan, maxn, grid, s, a) : run_a_f32(plan, maxn, grid, s, a);
    default:
        a.mode = 2;
        return fp64 ? run_a_f64(plan, maxn, grid, s, a) : run_a_f32(plan, maxn, grid, s, a);
    }
}

__global__ void k_zero_bytes(uint32_t *p, size_t nwords)
{
    for (size_t i = blockIdx.x * size_t(blockDim.x) + threadIdx.x; i < nwords; i += size_t(gridDim.x) * blockDim.x)
        p[i] = 0u;
}

// zero a device array (byte count a multiple of 4) with a kernel
hipError_t run_zero(void *p, size_t bytes, hipStream_t s)
{
    hipLaunchKernelGGL(k_zero_bytes, dim3(2048), dim3(256), 0, s, static_cast<uint32_t *>(p), bytes / 4);
    return hipGetLastError();
}

hipError_t run_finalize(const ProbDesc *desc, const double *partials, double *e_h, int nprob, hipStream_t s)
{
    hipLaunchKernelGGL(k_finalize, dim3(nprob), dim3(kFinThreads), 0, s, desc, partials, e_h);
    return hipGetLastError();
}

}  // namespace hartree

// The paper's schemes with a rest population: D1Q3Q2 (Sec. 2) and D2Q5Q4Q4
// (Sec. 3), rest weight a >= 0, relaxed in moment space with one rate per
// non-conserved moment (eq. 2-relaxation, MRT).
//
// Equilibria (derivatives of the potentials h_j^* with K = 1/(2g),
// theta = g h - |u|^2/2, c = 1/(2 lambda)):
//   f_0 = a K theta,
//   1D: f_+- = (h - f_0)/2 +- q c,             g_+- = q/2 +- (q u + p) c
//   2D: f_{1,3} = (h - f_0)/4 +- qx c,         f_{2,4} = (h - f_0)/4 +- qy c,
//       gx / gy as in the a = 0 scheme (the rest potential does not depend on u).
// Moments (Sec. 2, Sec. 3):
//   1D: rho = f_0 + f_+ + f_-, J = lambda (f_+ - f_-), eps = lambda^2 (f_+ + f_- - 2 f_0),
//       q = g_+ + g_-, J_q = lambda (g_+ - g_-)
//   2D: rho, J_x = lambda (f_1 - f_3), J_y = lambda (f_2 - f_4),
//       eps = f_1 + f_2 + f_3 + f_4 - 4 f_0, XX = f_1 - f_2 + f_3 - f_4;
//       per momentum family: q, lambda (g_1 - g_3), lambda (g_2 - g_4),
//       g_1 - g_2 + g_3 - g_4.
// Equilibrium moments: J^eq = q; 1D eps^eq = lambda^2 (rho - 3 a K theta),
//   J_q^eq = q u + p; 2D eps^eq = (1 - 5a/2) rho + (5a/4)(u^2 + v^2)/g (the factor a
//   of the second term restored), XX^eq = 0, f_xx^eq = rho u^2 + p,
//   f_xy^eq = f_yx^eq = rho u v, f_yy^eq = rho v^2 + p.
// Plane order: rest population first, then the a = 0 order.
#include <algorithm>
#include <type_traits>

#include "internal.h"
#include "rest_device.h"
#include "xk_wave.h"
#include "multistep.h"
#include "strip_device.h"

namespace lbm {

// ---- pulls (rest plane 0 does not move) ---------------------------------------------
// An inflow face takes the equilibrium of its prescribed state, evaluated here in
// registers.  (Returning a value loaded from a precomputed table in the default
// case of the face switch made the compiler's control-flow structurizer drop the
// table address on one of the paths into that case, so the load went through an
// unassigned register.)
template <typename T>
__device__ double pull_rest_face2d(const T *__restrict__ src, const Geo &G, const Mrt &M, int pl,
                                   int face, int x, int y, int sx, int sy)
{
    switch (G.bc[face]) {
    case BC_PERIODIC:
        sx = sx < 0 ? sx + G.nx : (sx >= G.nx ? sx - G.nx : sx);
        sy = sy < 0 ? sy + G.ny : (sy >= G.ny ? sy - G.ny : sy);
        return ld(src + pl * G.ps + (long)sy * G.nx + sx);
    case BC_NEUMANN:
        return ld(src + pl * G.ps + (long)y * G.nx + x);
    case BC_WALL: {
        const int k = (pl - 1) >> 2, j = (pl - 1) & 3;
        const int opp = 1 + ((k << 2) | ((j + 2) & 3));
        const double v = ld(src + opp * G.ps + (long)y * G.nx + x);
        return k == (face < 2 ? 1 : 2) ? -v : v;
    }
    default: {
        double e[13];
        feq_rest2d(G.win[face][0], G.win[face][1], G.win[face][2], M, e);
        return e[pl];
    }
    }
}

template <typename T>
__device__ __forceinline__ void pull_rest2d(const T *__restrict__ src, const Geo &G, const Mrt &M,
                                            bool allper, int x, int y, double *f)
{
    const int nx = G.nx, ny = G.ny;
    const long ps = G.ps, row = (long)y * nx;
    f[0] = ld(src + row + x);
    const bool interior = x > 0 && x < nx - 1 && y > 0 && y < ny - 1;
    if (allper || interior) {
        const int xm = x == 0 ? nx - 1 : x - 1;
        const int xp = x == nx - 1 ? 0 : x + 1;
        const long rm = y == 0 ? (long)(ny - 1) * nx : row - nx;
        const long rp = y == ny - 1 ? 0 : row + nx;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const T *b = src + (1 + 4 * k) * ps;
            f[1 + 4 * k] = ld(b + row + xm);
            f[2 + 4 * k] = ld(b + ps + rm + x);
            f[3 + 4 * k] = ld(b + 2 * ps + row + xp);
            f[4 + 4 * k] = ld(b + 3 * ps + rp + x);
        }
        return;
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const int p1 = 1 + 4 * k;
        f[p1] = x > 0 ? ld(src + p1 * ps + row + x - 1)
                      : pull_rest_face2d(src, G, M, p1, 0, x, y, x - 1, y);
        f[p1 + 1] = y > 0 ? ld(src + (p1 + 1) * ps + row - nx + x)
                          : pull_rest_face2d(src, G, M, p1 + 1, 2, x, y, x, y - 1);
        f[p1 + 2] = x < nx - 1 ? ld(src + (p1 + 2) * ps + row + x + 1)
                               : pull_rest_face2d(src, G, M, p1 + 2, 1, x, y, x + 1, y);
        f[p1 + 3] = y < ny - 1 ? ld(src + (p1 + 3) * ps + row + nx + x)
                               : pull_rest_face2d(src, G, M, p1 + 3, 3, x, y, x, y + 1);
    }
}

template <typename T>
__device__ double pull_rest_face1d(const T *__restrict__ src, const Geo &G, const Mrt &M, int pl,
                                   int face, int x)
{
    switch (G.bc[face]) {
    case BC_PERIODIC:
        return ld(src + pl * G.ps + (face == 0 ? G.nx - 1 : 0));
    case BC_NEUMANN:
        return ld(src + pl * G.ps + x);
    case BC_WALL: {
        const int opp = pl == 1 ? 2 : pl == 2 ? 1 : pl == 3 ? 4 : 3;
        const double v = ld(src + opp * G.ps + x);
        return pl >= 3 ? -v : v;
    }
    default: {
        double e[5];
        feq_rest1d(G.win[face][0], G.win[face][1], M, e);
        return e[pl];
    }
    }
}

// ---- kernels -------------------------------------------------------------------------
// WIDE: any heights and g (rest_device.h).
template <typename T, bool WIDE>
__global__ void __launch_bounds__(256) k_step_rest2d(const T *__restrict__ src, T *__restrict__ dst,
                                                     Geo G, Mrt M, int tiles_x, int allper)
{
    const int t = blockIdx.x;
    const int y = t / tiles_x;
    const int x = (t - y * tiles_x) * 256 + threadIdx.x;
    if (x >= G.nx) return;
    double f[13];
    pull_rest2d(src, G, M, allper != 0, x, y, f);
    collide_mrt2d<WIDE>(f, M);
    T *o = dst + (long)y * G.nx + x;
#pragma unroll
    for (int pl = 0; pl < 13; ++pl) sth<2>(o + pl * G.ps, f[pl]);
}

template <typename T, bool WIDE>
__global__ void __launch_bounds__(256) k_step_rest1d(const T *__restrict__ src, T *__restrict__ dst,
                                                     Geo G, Mrt M)
{
    const int x = blockIdx.x * 256 + threadIdx.x;
    if (x >= G.nx) return;
    const long ps = G.ps;
    double f[5];
    f[0] = ld(src + x);
    if (x > 0) {
        f[1] = ld(src + ps + x - 1);
        f[3] = ld(src + 3 * ps + x - 1);
    } else {
        f[1] = pull_rest_face1d(src, G, M, 1, 0, x);
        f[3] = pull_rest_face1d(src, G, M, 3, 0, x);
    }
    if (x < G.nx - 1) {
        f[2] = ld(src + 2 * ps + x + 1);
        f[4] = ld(src + 4 * ps + x + 1);
    } else {
        f[2] = pull_rest_face1d(src, G, M, 2, 1, x);
        f[4] = pull_rest_face1d(src, G, M, 4, 1, x);
    }
    collide_mrt1d<WIDE>(f, M);
#pragma unroll
    for (int pl = 0; pl < 5; ++pl) sth<2>(dst + pl * ps + x, f[pl]);
}

// ---- D2Q5Q4Q4, K steps per launch on all-periodic grids ----------------------------
// One wavefront per column strip of 64 lanes, walking up a segment of rows, four
// neighbouring strips to a workgroup.  Iteration j computes level 1 of row
// i = y0 - (K - 1) + j from the level-n pulls of that row (loaded one iteration
// ahead), then level k + 1 of row i - k from level k for k = 1 .. K - 1, so the
// levels are skewed one row apart and only level K leaves the wavefront (row
// i - (K - 1), stored when it lies in the segment).  Level k + 1 of row r pulls
// from level k: e1 / e3 of row r from lanes l - 1 / l + 1 (kept from the previous
// iteration, DPP), e2 of row r - 1 (kept two iterations, two arrays used
// alternately), e4 of row r + 1 (just computed), and the rest population of row r
// (kept one iteration).  Every level is rounded to the storage type, as the
// one-step kernel's store and load round it, and the collision is the same
// function, so the result equals K single steps bit for bit.  The K - 1 lanes at
// each strip edge take values from outside the valid range and are not stored; the
// first 2 (K - 1) iterations store nothing and skip the collisions of the levels
// that have no row yet.
//   A strip owns whole 64-byte (FP32: 16-byte) pieces of a row (rest2k_out).  All planes share one
// buffer descriptor where they lie below 2 GiB together (else BIG: one per plane);
// accesses that must not happen carry an offset the hardware drops, so the loop has
// no branch and the loads of the next row stay in flight.  Bound by the issue of FP64
// operations on small grids and by the state through memory from about 2048^2 on.  Two
// wavefronts fit a SIMD up to K = 5 FP64 (230 registers) and 7 FP32; with 64-bit
// addresses, permutes and a second row buffer it was one (268): 1024^2 FP64, K = 5, 14.6
// us a step, 9.9 now, 4096^2 FP32 135, 107 at K = 7; 4096^2 FP64 160 either way (4.4 TB/s).
// FP64 K = 6 spills at two wavefronts and takes one (2048^2 48.3 us a step and 34.8).
// Columns a strip owns: as many as the halo lanes leave, in whole pieces of a row.  FP32
// pieces of 16 columns lose up to a fifth of the lanes (48 of 64 at every K from 2 to 7; in
// fours 60, 60, 56, 56, 52, 52): us a step 7 steps 2048^2 32.5 and 30.1, 1024^2 11.5 and 10.3,
// 100000 x 16 20.6 and 14.2.  FP64 ones of 8 cost less (56 or 48) than parts of lines.
template <typename T, int K>
constexpr int rest2k_out()
{
    constexpr int piece = sizeof(T) == 4 ? 4 : 8;
    return (64 - 2 * (K - 1)) / piece * piece;
}

template <typename T, int K, bool BIG>
__global__ void __launch_bounds__(256, sizeof(T) == 8 && K > 5 ? 1 : 2)
    k_step_rest2d_k(const T *__restrict__ src, T *__restrict__ dst, Geo G, Mrt M, int nstrips,
                    int seg)
{
    constexpr int WO = rest2k_out<T, K>(), H = (64 - WO) / 2;
    const int nx = G.nx, ny = G.ny;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));  // uniform
    const int ngroups = (nstrips + 3) / 4;
    const int tile = xk_tile(blockIdx.x, ngroups * ((ny + seg - 1) / seg), true);
    const int strip = tile % ngroups * 4 + wave;
    if (strip >= nstrips) return;  // whole wavefront; nothing here waits on others
    const int y0 = tile / ngroups * seg, y1 = min(y0 + seg, ny);
    const int xc = strip * WO - H + lane;
    const int xw = ((xc % nx) + nx) % nx;
    const int xm = xw == 0 ? nx - 1 : xw - 1, xp = xw == nx - 1 ? 0 : xw + 1;
    const bool olane = lane >= H && lane < H + WO && xc < nx;
    const unsigned sT = sizeof(T), pT = BIG ? 0 : (unsigned)G.ps * sT;  // bytes of a plane
    auto rsrc = [&](const T *p, int pl) __attribute__((always_inline)) {
        return __builtin_amdgcn_make_buffer_rsrc(
            const_cast<T *>(BIG ? p + pl * G.ps : p), 0,
            (int)(BIG ? (unsigned)nx * (unsigned)ny * sT : 13 * pT), 0x00020000);
    };
    auto load = [&](int r, T(&b)[13]) __attribute__((always_inline)) {
        const unsigned row = (unsigned)r * nx, rm = (unsigned)(r == 0 ? ny - 1 : r - 1) * nx,
                       rp = (unsigned)(r == ny - 1 ? 0 : r + 1) * nx;
        const unsigned o[4] = {(row + xm) * sT, (rm + xw) * sT, (row + xp) * sT, (rp + xw) * sT};
        pair_load(rsrc(src, 0), (row + xw) * sT, 0, b[0]);
#pragma unroll
        for (int pl = 0; pl < 12; ++pl)
            pair_load(rsrc(src, 1 + pl), o[pl & 3], (1 + pl) * pT, b[1 + pl]);
    };
    T e2[2][K - 1][3], e1[K - 1][3], e3[K - 1][3], r0[K - 1];
#pragma unroll
    for (int k = 0; k < K - 1; ++k) {
        r0[k] = (T)1;
#pragma unroll
        for (int c = 0; c < 3; ++c) e2[0][k][c] = e2[1][k][c] = e1[k][c] = e3[k][c] = (T)0;
    }
    T buf[13];
    int rl = (((y0 - (K - 1)) % ny) + ny) % ny;  // row of the last load, wrapped
    load(rl, buf);
    auto row = [&](int j, auto uc, auto wc) __attribute__((always_inline)) {
        constexpr int u = decltype(uc)::value;
        constexpr bool WARM = decltype(wc)::value;
        double v[13];
#pragma unroll
        for (int pl = 0; pl < 13; ++pl) v[pl] = (double)buf[pl];
        __builtin_amdgcn_sched_barrier(0);
        rl = rl == ny - 1 ? 0 : rl + 1;
        load(rl, buf);
        collide_mrt2d(v, M);  // level 1
#pragma unroll
        for (int k = 1; k < K; ++k) {
            double o[13];
            o[0] = (double)r0[k - 1];
            r0[k - 1] = (T)v[0];
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const int b = 1 + 4 * c;
                o[b + 0] = (double)pair_shr(e1[k - 1][c]);
                o[b + 1] = (double)e2[u][k - 1][c];
                o[b + 2] = (double)pair_shl(e3[k - 1][c]);
                o[b + 3] = (double)(T)v[b + 3];
                e1[k - 1][c] = (T)v[b + 0];
                e2[u][k - 1][c] = (T)v[b + 1];
                e3[k - 1][c] = (T)v[b + 2];
            }
            if constexpr (WARM) {
                // rounded here, not sunk past the branch with twice the registers
                __asm__ __volatile__("" : "+v"(r0[k - 1]));
#pragma unroll
                for (int c = 0; c < 3; ++c)
                    __asm__ __volatile__("" : "+v"(e1[k - 1][c]), "+v"(e2[u][k - 1][c]),
                                         "+v"(e3[k - 1][c]));
            }
            __builtin_amdgcn_sched_barrier(0);
            if (!WARM || j >= 2 * k) collide_mrt2d(o, M);  // (uniform)
#pragma unroll
            for (int pl = 0; pl < 13; ++pl) v[pl] = o[pl];
        }
        if constexpr (!WARM) {
            const int r = y0 - 2 * (K - 1) + j;
            const unsigned o = olane && r < y1 ? ((unsigned)r * nx + xc) * sT : kPairDrop;
#pragma unroll
            for (int pl = 0; pl < 13; ++pl) pair_store(rsrc(dst, pl), o, pl * pT, (T)v[pl]);
        }
    };
    using std::integral_constant;
    int j = 0;
    for (; j < 2 * (K - 1); j += 2) {
        row(j, integral_constant<int, 0>{}, std::true_type{});
        row(j + 1, integral_constant<int, 1>{}, std::true_type{});
    }
    for (const int n = (y1 - y0) + 2 * (K - 1); j < n; j += 2) {
        row(j, integral_constant<int, 0>{}, std::false_type{});
        row(j + 1, integral_constant<int, 1>{}, std::false_type{});
    }
}

template <typename T, int K>
static int rest2k_resident()
{
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_step_rest2d_k<T, K, false>, 256, 0) !=
        hipSuccess)
        return 0;
    return nb;
}

#define LBM_REST_KS(F) F(2) F(3) F(4) F(5) F(6)  // either storage; FP32 7 as well
// Output columns of a strip.
static int rest2k_wo(bool f32, int K)
{
    switch (K) {
#define LBM_REST_WO(KK) case KK: return f32 ? rest2k_out<float, KK>() : rest2k_out<double, KK>();
        LBM_REST_KS(LBM_REST_WO)
#undef LBM_REST_WO
    case 7: return rest2k_out<float, 7>();
    default: return 0;
    }
}

// Workgroups of the K-step launch resident per compute unit, compute units (0: unknown).
static int rest2k_per_cu(bool f32, int K, int *ncu)
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        return 0;
    switch (K) {
#define LBM_REST_OCC(KK) \
    case KK: return f32 ? rest2k_resident<float, KK>() : rest2k_resident<double, KK>();
        LBM_REST_KS(LBM_REST_OCC)
#undef LBM_REST_OCC
    case 7: return f32 ? rest2k_resident<float, 7>() : 0;
    default: return 0;
    }
}

int rest2k_depth(const Geo &G, bool f32)
{
    return f32 ? kDeepRest2dF32 : (long)G.nx * G.ny < 3000000 ? 5 : 6;
}

long rest2k_cols(const Geo &G, bool f32, int K)
{
    const long wo = rest2k_wo(f32, K);
    return ((G.nx + wo - 1) / wo + 3) / 4 * 4 * wo;
}

bool rest2k_fills(const Geo &G, bool f32)
{
    int ncu = 0;
    if (rest2k_per_cu(f32, 5, &ncu) <= 0) return false;
    int nseg = 1;  // most segments of at least 16 rows
    for (int n = 2; n <= G.ny; ++n) {
        const int sg = (G.ny + n - 1) / n;
        if (sg < 16) break;
        if ((G.ny + sg - 1) / sg == n) nseg = n;
    }
    return 3L * (((G.nx + 55) / 56 + 3) / 4) * nseg >= (f32 ? 2L : 1L) * ncu;
}

// Rows per segment: an iteration of two
// workgroups on a compute unit takes 1.97 times that of one (4096^2 FP64, 5 steps: 4.95
// and 2.47 us), so a second one only shortens the tail; the start of a segment costs 1.3
// iterations per level.  1024^2 FP64, 5 steps: 49 segments of 21 rows (one workgroup
// each) 9.9 us a step, 64 of 16 (two on some) 13.0.  Choosing them by whole rounds of resident
// workgroups instead: 4096^2 FP64, 5 steps, 849 us a launch, 770 so; 1024^2 FP32, 6 steps, 83,
// 61.
int rest2k_rows(const Geo &G, bool f32, int K, long *slots)
{
    int ncu = 0;
    const int resident = rest2k_per_cu(f32, K, &ncu), per = std::min(resident, 2);
    if (slots) *slots = (long)ncu * resident;
    if (per <= 0) return 0;
    const int WO = rest2k_wo(f32, K);
    const long ngroups = ((G.nx + WO - 1) / WO + 3) / 4;
    static const double kIter[3] = {0.0, 1.0, 1.97};
    int best = 0;
    double best_cost = 0.0;
    for (int nseg = 1; nseg <= G.ny; ++nseg) {
        const int sg = (G.ny + nseg - 1) / nseg;
        if (sg < 8 && nseg > 1) break;
        if ((G.ny + sg - 1) / sg != nseg) continue;
        const long n = (ngroups * nseg + ncu - 1) / ncu;
        const double cost =
            ((double)(n / per) * kIter[per] + kIter[n % per]) * (sg + 1.3 * K);
        if (best == 0 || cost < best_cost) {
            best = sg;
            best_cost = cost;
        }
    }
    return best;
}

static long rest2k_blocks(const Geo &G, bool f32, int K, int seg)
{
    const int WO = rest2k_wo(f32, K);
    return (long)(((G.nx + WO - 1) / WO + 3) / 4) * ((G.ny + seg - 1) / seg);
}

template <typename T, int K>
static hipError_t rest2k_launch(const void *src, void *dst, const Geo &G, const Mrt &M, int seg,
                                hipStream_t st)
{
    constexpr int WO = rest2k_out<T, K>();
    const int ns = (G.nx + WO - 1) / WO;
    const dim3 grid((unsigned)rest2k_blocks(G, sizeof(T) == 4, K, seg)), block(256);
    if (13L * G.ps * (long)sizeof(T) < (1L << 31))
        hipLaunchKernelGGL((k_step_rest2d_k<T, K, false>), grid, block, 0, st, (const T *)src,
                           (T *)dst, G, M, ns, seg);
    else
        hipLaunchKernelGGL((k_step_rest2d_k<T, K, true>), grid, block, 0, st, (const T *)src,
                           (T *)dst, G, M, ns, seg);
    return hipGetLastError();
}

hipError_t launch_step_rest2k(bool f32, const void *src, void *dst, const Geo &G, const Mrt &M,
                              int K, int seg, hipStream_t st)
{
    if (seg <= 0) return hipErrorInvalidValue;
    switch (K) {
#define LBM_REST_K(KK)                                                                       \
    case KK:                                                                                 \
        return f32 ? rest2k_launch<float, KK>(src, dst, G, M, seg, st)                       \
                   : rest2k_launch<double, KK>(src, dst, G, M, seg, st);
        LBM_REST_KS(LBM_REST_K)
#undef LBM_REST_K
    case 7: return f32 ? rest2k_launch<float, 7>(src, dst, G, M, seg, st) : hipErrorInvalidValue;
    default:
        return hipErrorInvalidValue;
    }
}

// f*(0) = C(f^eq(W0)).  bad: bit 0 for a field that is refused, bit 1 for a height outside
// kRestRange.
template <typename T>
__global__ void __launch_bounds__(256) k_init_rest(int dim, T *__restrict__ dst,
                                                   const double *__restrict__ h0,
                                                   const double *__restrict__ qx0,
                                                   const double *__restrict__ qy0, Geo G, Mrt M,
                                                   unsigned long long *speed_bits, int *bad)
{
    const long n = (long)G.nx * G.ny;
    const long i = (long)blockIdx.x * 256 + threadIdx.x;
    const bool in = i < n;
    const double h = in ? h0[i] : 1.0;
    const double qx = in && qx0 ? qx0[i] : 0.0;
    const double qy = in && dim == 2 && qy0 ? qy0[i] : 0.0;
    const bool good = h > 0.0 && isfinite(h) && isfinite(qx) && isfinite(qy);
    if (!good) atomicOr(bad, 1);
    if (!(h > 1.0 / kRestRange && h < kRestRange)) atomicOr(bad, 2);
    const double u = fabs(qx / h), v = fabs(qy / h);
    block_raise(in && good ? (u > v ? u : v) + sqrt(M.g * h) : 0.0, speed_bits);
    if (!in || !good) return;
    if (dim == 1) {
        double f[5];
        feq_rest1d(h, qx, M, f);
        collide_mrt1d<true>(f, M);
#pragma unroll
        for (int pl = 0; pl < 5; ++pl) st(dst + pl * G.ps + i, f[pl]);
    } else {
        double f[13];
        feq_rest2d(h, qx, qy, M, f);
        collide_mrt2d<true>(f, M);
#pragma unroll
        for (int pl = 0; pl < 13; ++pl) st(dst + pl * G.ps + i, f[pl]);
    }
}

// Conserved fields, per-block partial sums (fixed order) and the divergence flag.
template <typename T>
__global__ void __launch_bounds__(256) k_moments_rest(int dim, const T *__restrict__ state,
                                                      double *__restrict__ h,
                                                      double *__restrict__ qx,
                                                      double *__restrict__ qy,
                                                      double *__restrict__ partials, int *flag,
                                                      Geo G)
{
    __shared__ double sh[3][256];
    const long n = (long)G.nx * G.ny;
    const long i = (long)blockIdx.x * 256 + threadIdx.x;
    double w[3] = {0.0, 0.0, 0.0};
    if (i < n) {
        const long ps = G.ps;
        if (dim == 1) {
            w[0] = ld(state + i) + (ld(state + ps + i) + ld(state + 2 * ps + i));
            w[1] = ld(state + 3 * ps + i) + ld(state + 4 * ps + i);
        } else {
            double f[13];
#pragma unroll
            for (int pl = 0; pl < 13; ++pl) f[pl] = ld(state + pl * ps + i);
            w[0] = f[0] + ((f[1] + f[3]) + (f[2] + f[4]));
            w[1] = (f[5] + f[7]) + (f[6] + f[8]);
            w[2] = (f[9] + f[11]) + (f[10] + f[12]);
        }
        if (h) h[i] = w[0];
        if (qx) qx[i] = w[1];
        if (qy && dim == 2) qy[i] = w[2];
        if (flag && (!(w[0] > 0.0) || !isfinite(w[0]) || !isfinite(w[1]) || !isfinite(w[2])))
            atomicOr(flag, 1);
    }
    if (partials) {
        const int t = threadIdx.x;
        for (int c = 0; c < 3; ++c) sh[c][t] = w[c];
        __syncthreads();
        for (int s = 128; s > 0; s >>= 1) {
            if (t < s)
                for (int c = 0; c < 3; ++c) sh[c][t] = sh[c][t] + sh[c][t + s];
            __syncthreads();
        }
        if (t == 0)
            for (int c = 0; c < 3; ++c) partials[(long)blockIdx.x * 3 + c] = sh[c][0];
    }
}

// ---- launchers -----------------------------------------------------------------------------
hipError_t launch_init_rest(int dim, bool f32, void *dst, const double *h0, const double *qx0,
                            const double *qy0, const Geo &G, const Mrt &M,
                            unsigned long long *speed_bits, int *bad, hipStream_t st)
{
    const int nb = (int)(((long)G.nx * G.ny + 255) / 256);
    if (f32)
        hipLaunchKernelGGL(k_init_rest<float>, dim3(nb), dim3(256), 0, st, dim, (float *)dst, h0,
                           qx0, qy0, G, M, speed_bits, bad);
    else
        hipLaunchKernelGGL(k_init_rest<double>, dim3(nb), dim3(256), 0, st, dim, (double *)dst,
                           h0, qx0, qy0, G, M, speed_bits, bad);
    return hipGetLastError();
}

template <typename T, bool WIDE>
static void step_rest(int dim, const void *src, void *dst, const Geo &G, const Mrt &M,
                      hipStream_t st)
{
    const int tiles_x = (G.nx + 255) / 256;
    const int allper = G.bc[0] == BC_PERIODIC && G.bc[1] == BC_PERIODIC &&
                       G.bc[2] == BC_PERIODIC && G.bc[3] == BC_PERIODIC;
    if (dim == 2)
        hipLaunchKernelGGL((k_step_rest2d<T, WIDE>), dim3(tiles_x * G.ny), dim3(256), 0, st,
                           (const T *)src, (T *)dst, G, M, tiles_x, allper);
    else
        hipLaunchKernelGGL((k_step_rest1d<T, WIDE>), dim3(tiles_x), dim3(256), 0, st,
                           (const T *)src, (T *)dst, G, M);
}

hipError_t launch_step_rest(int dim, bool f32, bool wide, const void *src, void *dst,
                            const Geo &G, const Mrt &M, hipStream_t st)
{
    if (f32)
        wide ? step_rest<float, true>(dim, src, dst, G, M, st)
             : step_rest<float, false>(dim, src, dst, G, M, st);
    else
        wide ? step_rest<double, true>(dim, src, dst, G, M, st)
             : step_rest<double, false>(dim, src, dst, G, M, st);
    return hipGetLastError();
}

hipError_t launch_moments_rest(int dim, bool f32, const void *state, double *h, double *qx,
                               double *qy, double *partials, int *flag, const Geo &G,
                               hipStream_t st, int *nblocks_out)
{
    const int nb = (int)(((long)G.nx * G.ny + 255) / 256);
    if (nblocks_out) *nblocks_out = nb;
    if (f32)
        hipLaunchKernelGGL(k_moments_rest<float>, dim3(nb), dim3(256), 0, st, dim,
                           (const float *)state, h, qx, qy, partials, flag, G);
    else
        hipLaunchKernelGGL(k_moments_rest<double>, dim3(nb), dim3(256), 0, st, dim,
                           (const double *)state, h, qx, qy, partials, flag, G);
    return hipGetLastError();
}

} // namespace lbm

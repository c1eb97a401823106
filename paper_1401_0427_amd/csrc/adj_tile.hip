// Several steps of the discrete adjoint per launch on all-periodic 2D grids.
//
// The one-step kernel moves 36 values per node and step (u^n, lambda^{n+1} read,
// lambda^n written) and is bound by them on large grids; on small ones a launch costs
// 4.8 us whatever it does.
//   k_adj2d_levels (small grids): a workgroup keeps a tile of lambda in registers over up
//     to five steps and reads the stored levels' pulls as it goes.
//   k_adj2d_strip (larger grids): a wavefront marches up a column strip and applies two
//     steps from u^n and lambda^{n+2}, computing u^{n+1} itself: 36 values per node for
//     two steps.
//   k_levels_strip (larger grids): the forward steps that store every level for these,
//     several per launch.
// The transposed stream moves values as the tile kernels of the forward steps do (DPP
// along x, rows of the thread and LDS along y); the last step pushes to memory.  Every
// level of u and lambda is rounded to its storage type and dL/ds is summed in the same
// groups and order as by the one-step kernel, so the result is bitwise that of one-step
// launches over every level.
#include <type_traits>

#include "adj_device.h"
#include "multistep.h"
#include "strip_device.h"

namespace lbm {

// Values that cross between rows of threads: `up` from a thread's last row to the row
// above, `down` from its first row to the row below (a row of padding at either end).
template <typename T, int N>
struct PairRows {
    T up[3][N], down[3][N];
};

// The transposed stream: l <- e1 from x + 1, e2 from y + 1, e3 from x - 1, e4 from y - 1.
template <typename T, int TX, int R, int N>
__device__ __forceinline__ void pair_push(T (&l)[R][12], PairRows<T, N> &B, int t)
{
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        B.up[c][TX + t] = l[R - 1][4 * c + 3];
        B.down[c][t] = l[0][4 * c + 1];
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        T below = B.up[c][t];
        const T above = B.down[c][TX + t];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const T own = l[r][4 * c + 3];
            l[r][4 * c + 0] = pair_shl(l[r][4 * c + 0]);
            l[r][4 * c + 1] = r + 1 < R ? l[r + 1][4 * c + 1] : above;
            l[r][4 * c + 2] = pair_shr(l[r][4 * c + 2]);
            l[r][4 * c + 3] = below;
            below = own;
        }
    }
}

// K steps over stored levels, by tiles of TX x (TY R) nodes (R rows of one column per
// thread): v^{n+j} is read from level n + j (level n at `first`, level n + j at next +
// (j - 1) * stride), lambda stays in registers.  A step loses one more row and column at
// the tile's edges; nodes at least 4 columns and K - 1 rows inside are exact and owned.
// Bound by the latency of a launch and of a step's chain of operations: 96 x 64 FP64
// 1.8 us a step against 4.2 for one step per launch, 256^2 4.4 against 6.1.
template <typename T, typename TA, int TX, int TY, int R>
__global__ void __launch_bounds__(TX * TY)
    k_adj2d_levels(const T *__restrict__ first, const T *__restrict__ next, long stride,
                   const TA *__restrict__ lamK, TA *__restrict__ lam0,
                   double *__restrict__ partials, Geo G, Phys P, int K, int ntx)
{
    constexpr int NT = TX * TY, HX = 4;
    static_assert(64 % TX == 0 && NT % 64 == 0, "whole rows of lanes per wavefront");
    static_assert(HX % kAdjGroup == 0 && TX % kAdjGroup == 0, "whole groups of columns");
    __shared__ PairRows<TA, NT + TX> B[2];
    const int nx = G.nx, ny = G.ny, HY = K - 1;
    const long ps = G.ps;
    const int t = threadIdx.x, tx = t % TX, ty = t / TX;
    const int bx = (int)blockIdx.x % ntx, by = (int)blockIdx.x / ntx;
    const int x = bx * (TX - 2 * HX) - HX + tx;           // this thread's column, unwrapped
    const int y0 = by * (TY * R - 2 * HY) - HY + ty * R;  // its first row
    const int xw = ((x % nx) + nx) % nx;
    const int xm = xw == 0 ? nx - 1 : xw - 1, xp = xw == nx - 1 ? 0 : xw + 1;
    const int yw0 = ((y0 % ny) + ny) % ny;
    auto load_v = [&](const T *un, T(&v)[R][12]) __attribute__((always_inline)) {
        int yw = yw0;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const long row = (long)yw * nx;
            const long rm = yw == 0 ? (long)(ny - 1) * nx : row - nx;
            const long rp = yw == ny - 1 ? 0 : row + nx;
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const T *b = un + (4 * c) * ps;
                v[r][4 * c + 0] = b[row + xm];
                v[r][4 * c + 1] = b[ps + rm + xw];
                v[r][4 * c + 2] = b[2 * ps + row + xp];
                v[r][4 * c + 3] = b[3 * ps + rp + xw];
            }
            yw = yw == ny - 1 ? 0 : yw + 1;
        }
    };
    TA l[R][12];
    T vn[R][12];
    double acc[R];
    const bool ox = tx >= HX && tx < TX - HX && x < nx;
    {
        int yw = yw0;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const long i = (long)yw * nx + xw;
#pragma unroll
            for (int pl = 0; pl < 12; ++pl) l[r][pl] = lamK[pl * ps + i];
            yw = yw == ny - 1 ? 0 : yw + 1;
        }
    }
    load_v(K > 1 ? next + (K - 2) * stride : first, vn);
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int y = y0 + r, i = ty * R + r;
        acc[r] = ox && i >= HY && i < TY * R - HY && y < ny ? partials[adj_slot(nx, x, y)] : 0.0;
    }
    for (int j = K - 1; j >= 0; --j) {
        // v^{n+j}; the next one's loads run under this one's arithmetic
        T vc[R][12];
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int pl = 0; pl < 12; ++pl) vc[r][pl] = vn[r][pl];
        if (j > 0) load_v(j > 1 ? next + (j - 2) * stride : first, vn);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            double v[12], w[12];
#pragma unroll
            for (int pl = 0; pl < 12; ++pl) {
                v[pl] = (double)vc[r][pl];
                w[pl] = (double)l[r][pl];
            }
            const double a = adj_node2d<T>(v, w, P);
            acc[r] = acc[r] + group_sum(ox ? a : 0.0);
#pragma unroll
            for (int pl = 0; pl < 12; ++pl) l[r][pl] = (TA)w[pl];
        }
        if (j > 0) pair_push<TA, TX, R>(l, B[j & 1], t);
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int y = y0 + r, i = ty * R + r;
        if (ox && i >= HY && i < TY * R - HY && y < ny) {
            const long row = (long)y * nx;
            const long rm = y == 0 ? (long)(ny - 1) * nx : row - nx;
            const long rp = y == ny - 1 ? 0 : row + nx;
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                TA *b = lam0 + (4 * k) * ps;
                b[row + xm] = l[r][4 * k + 0];
                b[ps + rm + x] = l[r][4 * k + 1];
                b[2 * ps + row + xp] = l[r][4 * k + 2];
                b[3 * ps + rp + x] = l[r][4 * k + 3];
            }
            if (tx % kAdjGroup == 0) partials[adj_slot(nx, x, y)] = acc[r];
        }
    }
}

// ---- larger grids: two steps, wavefronts marching up column strips -----------------------
// A wavefront takes a strip of 64 columns, owns the inner 56, and marches up a segment
// of rows with the two levels skewed: in iteration i it loads v^n of row i and computes
// u^{n+1} there, applies step n + 1's adjoint at row i - 1 and step n's at row i - 2.
// Columns cost 64 / 56 and a segment 4 rows more than it owns (a tile of 64 x 16 nodes
// per workgroup, 1.8 times the nodes: 36 us a step at 1024^2 FP32), and the loads of the
// next row overlap the arithmetic of this one.  Between iterations a lane keeps the e1,
// e3 and (two rows) e2 planes of u^{n+1}, the e1, e3 and (two rows) e4 planes of
// vt^{n+1}, and in LDS its own v^n of the last three rows.  The first iterations run only
// the stages that have rows (two of four, then two of two more: 10 % of a segment of 20
// rows).  Stores and partial sums are
// buffer accesses whose non-owned lanes carry a dropped offset, so the loop has no
// branch, and a row's partial sums are read one iteration ahead like its planes: read
// in the iteration that needs them, behind the next row's loads, they made it wait for
// those (1024^2 FP32 28.4 us a step, 24.5 ahead).  Stages are kept apart by scheduling
// barriers so that two wavefronts fit a SIMD without spills (FP64 82 us a step spilling,
// 40 without), and all planes share one buffer descriptor (a descriptor and a base per
// plane spilled 38 scalar registers).  At 1024^2 19.3 us a step FP32 (one-step kernel
// 31.2), FP64 34.6 (60.0); 2048^2 77 (123) and 145 (229): u^n, lambda and their halos at
// 4.0 TB/s.  48 owned columns, whole 64-byte pieces, lose at 1024^2 (8 %) what they gain
// at 2048^2 (1 %).
constexpr int kPairWaves = 4;  // wavefronts (neighbouring strips) per workgroup
constexpr int kPairOut = 56;   // columns a strip owns

template <typename T, typename TA>
__global__ void __launch_bounds__(64 * kPairWaves, 2)
    k_adj2d_strip(const T *__restrict__ un, const TA *__restrict__ lam2, TA *__restrict__ lam0,
                  double *__restrict__ partials, Geo G, Phys P, int nstrips, int seg)
{
    __shared__ T hist[kPairWaves][3][12][64];
    const int nx = G.nx, ny = G.ny;
    const long ps = G.ps;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));  // uniform
    const int w0 = (int)blockIdx.x * kPairWaves + wave, strip = w0 % nstrips;
    const int y0 = w0 / nstrips * seg, y1 = min(y0 + seg, ny);
    if (y0 >= ny) return;  // whole wavefront; nothing here waits on others
    const int x = strip * kPairOut - 4 + lane;
    const int xw = ((x % nx) + nx) % nx;
    const int xm = xw == 0 ? nx - 1 : xw - 1, xp = xw == nx - 1 ? 0 : xw + 1;
    const bool ox = lane >= 4 && lane < 4 + kPairOut && x < nx;
    const bool lead = ox && lane % kAdjGroup == 0;
    T(*H)[12][64] = hist[wave];
    const unsigned sT = sizeof(T), sA = sizeof(TA);
    const unsigned pT = (unsigned)ps * sT, pA = (unsigned)ps * sA;  // bytes of a plane
    const auto rsrc = [](const void *p, unsigned bytes) __attribute__((always_inline)) {
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)bytes, 0x00020000);
    };
    const __amdgpu_buffer_rsrc_t ru_ = rsrc(un, 12 * pT), rl_ = rsrc(lam2, 12 * pA),
                                 rs = rsrc(lam0, 12 * pA);

    // loads of v^n of row r and of lambda^{n+2} of row r (wrapped row indices)
    auto load_u = [&](int r, T(&b)[12]) __attribute__((always_inline)) {
        const unsigned row = (unsigned)r * nx, rm = (unsigned)(r == 0 ? ny - 1 : r - 1) * nx,
                       rp = (unsigned)(r == ny - 1 ? 0 : r + 1) * nx;
        const unsigned o[4] = {(row + xm) * sT, (rm + xw) * sT, (row + xp) * sT, (rp + xw) * sT};
#pragma unroll
        for (int pl = 0; pl < 12; ++pl) pair_load(ru_, o[pl & 3], pl * pT, b[pl]);
    };
    auto load_l = [&](int r, TA(&b)[12]) __attribute__((always_inline)) {
        const unsigned o = ((unsigned)r * nx + xw) * sA;
#pragma unroll
        for (int pl = 0; pl < 12; ++pl) pair_load(rl_, o, pl * pA, b[pl]);
    };
    auto wrap = [ny](int r) { return ((r % ny) + ny) % ny; };
    T u1e1[3], u1e3[3], u1e2[2][3];
    TA te1[3], te3[3], te4[2][3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        u1e1[c] = u1e3[c] = u1e2[0][c] = u1e2[1][c] = (T)0;
        te1[c] = te3[c] = te4[0][c] = te4[1][c] = (TA)0;
    }
#pragma unroll
    for (int p = 0; p < 3; ++p)
#pragma unroll
        for (int pl = 0; pl < 12; ++pl) H[p][pl][lane] = (T)1;
    const __amdgpu_buffer_rsrc_t rp = rsrc(partials, (unsigned)adj_slots_row(nx) * (unsigned)ny * 8u);
    const unsigned prow = (unsigned)adj_slots_row(nx) * 8u, pcol = (unsigned)(x / kAdjGroup) * 8u;
    // Rows are loaded one iteration ahead, into the registers the current row was just
    // read from; a row's partial sums likewise.
    T ub[12];
    TA lb[12];
    double pnext = 0.0;
    int ru = wrap(y0 - 2), rl = wrap(y0 - 1);  // rows of the last loads
    load_u(ru, ub);
    load_l(rl, lb);
    int h0 = 0;  // slot of v^n of row i
    double sprev = 0.0;
    // Iteration j in stages: u^{n+1} at row i; step n + 1 at row i - 1, which has no row
    // that anything needs before j = 2; step n at row i - 2, none before j = 4.
    auto row = [&](int j, auto qc, auto stages) __attribute__((always_inline)) {
        constexpr int q = decltype(qc)::value, S = decltype(stages)::value;
        const int i = y0 - 2 + j;  // row of v^n
        const int r0 = i - 2;      // row of step n
        const bool out = ox && r0 < y1;
        const double pold = pnext;
        const unsigned po = lead && r0 < y1 ? (unsigned)r0 * prow + pcol : kPairDrop;
        // level n at row i: u^{n+1}
        double v[12];
#pragma unroll
        for (int pl = 0; pl < 12; ++pl) {
            v[pl] = (double)ub[pl];
            H[h0][pl][lane] = ub[pl];
        }
        __builtin_amdgcn_sched_barrier(0);
        ru = ru == ny - 1 ? 0 : ru + 1;
        load_u(ru, ub);
        pair_load(rp,
                  lead && r0 + 1 >= y0 && r0 + 1 < y1 ? (unsigned)(r0 + 1) * prow + pcol : kPairDrop,
                  0, pnext);
        collide2d<T>(v, P);
        // v^{n+1} at row i - 1
        double w[12];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            w[4 * c + 0] = (double)pair_shr(u1e1[c]);
            w[4 * c + 1] = (double)u1e2[q][c];
            w[4 * c + 2] = (double)pair_shl(u1e3[c]);
            w[4 * c + 3] = (double)(T)v[4 * c + 3];
            u1e1[c] = (T)v[4 * c + 0];
            u1e2[q][c] = (T)v[4 * c + 1];
            u1e3[c] = (T)v[4 * c + 2];
        }
        h0 = h0 == 2 ? 0 : h0 + 1;  // also the slot of row i - 2
        if constexpr (S >= 2) {
            double l[12];
#pragma unroll
            for (int pl = 0; pl < 12; ++pl) l[pl] = (double)lb[pl];
            __builtin_amdgcn_sched_barrier(0);
            rl = rl == ny - 1 ? 0 : rl + 1;
            load_l(rl, lb);
            const double a1 = adj_node2d<T>(w, l, P);
            const double s1 = group_sum(ox ? a1 : 0.0);
            // lambda^{n+1} at row i - 2, v^n there
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const TA n1 = (TA)l[4 * c + 0], n2 = (TA)l[4 * c + 1], n3 = (TA)l[4 * c + 2],
                         n4 = (TA)l[4 * c + 3];
                l[4 * c + 0] = (double)pair_shl(te1[c]);
                l[4 * c + 1] = (double)n2;
                l[4 * c + 2] = (double)pair_shr(te3[c]);
                l[4 * c + 3] = (double)te4[q][c];
                te1[c] = n1;
                te3[c] = n3;
                te4[q][c] = n4;
            }
            if constexpr (S >= 3) {
#pragma unroll
                for (int pl = 0; pl < 12; ++pl) w[pl] = (double)H[h0][pl][lane];
                __builtin_amdgcn_sched_barrier(0);
                const double a0 = adj_node2d<T>(w, l, P);
                const double s0 = group_sum(ox ? a0 : 0.0);
                const unsigned row = (unsigned)r0 * nx;
                const unsigned rm = (unsigned)(r0 == 0 ? ny - 1 : r0 - 1) * nx;
                const unsigned rq = (unsigned)(r0 == ny - 1 ? 0 : r0 + 1) * nx;
                const unsigned o1 = out ? (row + xm) * sA : kPairDrop;
                const unsigned o2 = out ? (rm + xw) * sA : kPairDrop;
                const unsigned o3 = out ? (row + xp) * sA : kPairDrop;
                const unsigned o4 = out ? (rq + xw) * sA : kPairDrop;
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    pair_store(rs, o1, (4 * c + 0) * pA, (TA)l[4 * c + 0]);
                    pair_store(rs, o2, (4 * c + 1) * pA, (TA)l[4 * c + 1]);
                    pair_store(rs, o3, (4 * c + 2) * pA, (TA)l[4 * c + 2]);
                    pair_store(rs, o4, (4 * c + 3) * pA, (TA)l[4 * c + 3]);
                }
                pair_store(rp, po, 0, (pold + sprev) + s0);
            }
            sprev = s1;
        }
    };
    using std::integral_constant;
    const integral_constant<int, 0> even{};
    const integral_constant<int, 1> odd{};
    row(0, even, integral_constant<int, 1>{});
    row(1, odd, integral_constant<int, 1>{});
    row(2, even, integral_constant<int, 2>{});
    row(3, odd, integral_constant<int, 2>{});
    for (int j = 4, n = (y1 - y0) + 4; j < n; j += 2) {
        row(j, even, integral_constant<int, 3>{});
        row(j + 1, odd, integral_constant<int, 3>{});
    }
}

// Rows per segment: a wavefront runs seg rows and `extra` iterations more (its start), an
// iteration taking 1.92 times as long with two workgroups on a compute unit as with one
// (1024^2 FP32: 2.8 and 1.6 us, 2048^2 4.0 and 1.9), in rounds of these; the shortest such
// time.  A few workgroups beyond a round cost it whole: 260 instead of 245 at 1024^2 took
// 47 us a launch instead of 43.
static int strip_seg(const Geo &G, int nstrips, int extra)
{
    int best = G.ny;
    double cost = 1e30;
    for (int seg = 4; seg <= 128; seg += 2) {
        const long waves = (long)nstrips * ((G.ny + seg - 1) / seg);
        const long blocks = (waves + kPairWaves - 1) / kPairWaves;
        const double it = seg + extra;
        const double t = blocks <= 256 ? it : 1.92 * it * (double)((blocks + 511) / 512);
        if (t < cost) {
            cost = t;
            best = seg;
        }
    }
    return best;
}

template <typename T, typename TA>
static hipError_t strip_launch(const void *un, const void *lam2, void *lam0, double *partials,
                               const Geo &G, const Phys &P, hipStream_t st)
{
    const int ns = (G.nx + kPairOut - 1) / kPairOut;
    const int seg = adjoint_pair_rows(G);
    const long waves = (long)ns * ((G.ny + seg - 1) / seg);
    hipLaunchKernelGGL((k_adj2d_strip<T, TA>), dim3((waves + kPairWaves - 1) / kPairWaves),
                       dim3(64 * kPairWaves), 0, st, (const T *)un, (const TA *)lam2, (TA *)lam0,
                       partials, G, P, ns, seg);
    return hipGetLastError();
}

// The strip kernel addresses whole buffers with 32-bit byte offsets, of which the upper
// half marks dropped accesses.  Flat grids below kPairNodes take single steps (20000 x 3 FP64
// 4.9 us, in strips 6.5; 50000 x 2 8.3 and 5.4).
constexpr long kPairNodes = 75000;
bool adjoint_pairs(const Geo &G, bool f32, bool a32)
{
    if ((long)G.nx * G.ny < kPairNodes) return false;
    const long bytes = 12L * G.ps * (f32 && a32 ? 4 : 8);
    const long slots = adj_slots_row(G.nx) * (long)G.ny * 8;
    return bytes < (1L << 31) && slots < (1L << 31);
}

int adjoint_pair_rows(const Geo &G) { return strip_seg(G, (G.nx + kPairOut - 1) / kPairOut, 4); }

hipError_t launch_adjoint_pair(bool f32, bool a32, const void *un, const void *lam2, void *lam0,
                               double *partials, const Geo &G, const Phys &P, hipStream_t st)
{
    if (f32 && a32) return strip_launch<float, float>(un, lam2, lam0, partials, G, P, st);
    if (f32) return strip_launch<float, double>(un, lam2, lam0, partials, G, P, st);
    return strip_launch<double, double>(un, lam2, lam0, partials, G, P, st);
}

// Shape and steps per launch over stored levels: the smallest tiles and the most steps whose
// tiles all run at once, one per compute unit (16^2 ones, which share it, in nodes), -1 where
// none do: two-step launches from every second level are faster there, or single steps.  Us
// a step FP32 / FP64 in tiles of 32 x 16 with 5 and 3 steps, 32 x 32 with 5, and strips: 200^2
// (225 tiles of the first) 2.3 / 2.9, 2.6 / 3.1, 3.4 / 4.0, 5.4 / 6.6; 200 x 225 (261) 3.1 / 4.1,
// 2.7 / 3.4, 3.5 / 4.0, 5.5 / 6.7; 256^2 4.0 / 5.1, 3.5 / 4.5, 3.7 / 4.6, 5.8 / 6.7; 128 x 512 (258
// tiles of the second) 4.1 / 5.4, 4.5 / 5.6, 3.7 / 4.7, 5.8 / 6.7; 400^2 (289 of the third) 6.5 /
// 10.2, 6.5 / 10.2, - / 9.5, 6.0 / 8.3.  Narrow grids fill few lanes of anything but 16^2 tiles
// (3 x 100000 FP64 27 us a step, strips 77, single ones 130).
static long levels_tiles(const Geo &G, int shape, int K)
{
    int tx, rows;
    adjoint_levels_dims(shape, &tx, &rows);
    const int wo = tx - 8, ho = rows - 2 * (K - 1);
    return (long)((G.nx + wo - 1) / wo) * ((G.ny + ho - 1) / ho);
}
int adjoint_levels_plan(const Geo &G, int *K)
{
    const long nodes = (long)G.nx * G.ny;
    *K = 5;
    if (nodes <= 2000 || (nodes <= 12000 && G.ny > 8)) return 0;
    if (G.nx <= 8) {
        *K = 3;
        return 0;
    }
    if (levels_tiles(G, 1, 5) <= 256) return 1;
    if (levels_tiles(G, 1, 3) <= 256) {
        *K = 3;
        return 1;
    }
    return levels_tiles(G, 2, 5) <= 256 ? 2 : -1;
}
void adjoint_levels_dims(int shape, int *cols, int *rows)
{
    *cols = shape == 0 ? 16 : 32;
    *rows = shape < 2 ? 16 : 32;
}

template <typename T, typename TA, int TX, int TY, int R>
static hipError_t levels_launch(const void *first, const void *next, long stride,
                                const void *lamK, void *lam0, double *partials, const Geo &G,
                                const Phys &P, int K, hipStream_t st)
{
    const int wo = TX - 8, ho = TY * R - 2 * (K - 1);
    if (K < 1 || K > 5 || ho < 1) return hipErrorInvalidValue;  // 4 halo columns
    const int ntx = (G.nx + wo - 1) / wo, nty = (G.ny + ho - 1) / ho;
    hipLaunchKernelGGL((k_adj2d_levels<T, TA, TX, TY, R>), dim3(ntx * nty), dim3(TX * TY), 0, st,
                       (const T *)first, (const T *)next, stride, (const TA *)lamK, (TA *)lam0,
                       partials, G, P, K, ntx);
    return hipGetLastError();
}

template <typename T, typename TA>
static hipError_t levels_any(int shape, const void *first, const void *next, long stride,
                             const void *lamK, void *lam0, double *partials, const Geo &G,
                             const Phys &P, int K, hipStream_t st)
{
    switch (shape) {
    case 0:
        return levels_launch<T, TA, 16, 16, 1>(first, next, stride, lamK, lam0, partials, G, P, K,
                                               st);
    case 1:
        return levels_launch<T, TA, 32, 16, 1>(first, next, stride, lamK, lam0, partials, G, P, K,
                                               st);
    case 2:
        return levels_launch<T, TA, 32, 16, 2>(first, next, stride, lamK, lam0, partials, G, P, K,
                                               st);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_adjoint_levels(bool f32, bool a32, int shape, const void *first,
                                 const void *next, long stride, const void *lamK, void *lam0,
                                 double *partials, const Geo &G, const Phys &P, int K,
                                 hipStream_t st)
{
    const auto run = f32 && a32 ? levels_any<float, float>
                     : f32      ? levels_any<float, double>
                                : levels_any<double, double>;
    return run(shape, first, next, stride, lamK, lam0, partials, G, P, K, st);
}

// ---- every level stored, larger grids ----------------------------------------------------
// K forward steps per launch in strips as above, level k + 1 of row i - k computed and
// stored in iteration i: 12 values read per node for K times 12 written, where single
// steps read and write 12 each and are bound by that.  A strip owns 48 columns: its rows
// then start and end on 64 bytes in either type, and with most of the traffic being
// stores, parts of lines cost more than halo columns (us a step with 56 / 48 / 32 owned:
// 1024^2 FP32 19.2 / 16.8 / 16.7, FP64 34.1 / 29.7 / 32.3, 2048^2 79 / 71 / 61 and 133 /
// 108 / 113; single steps 20.5, 41.4, 76.5, 149).
constexpr int kLevelOut = 48;
static_assert(64 - kLevelOut >= 2 * kLevelStripMost, "halo columns");
template <typename T, int K>
__global__ void __launch_bounds__(64 * kPairWaves, 2)
    k_levels_strip(const T *__restrict__ src, T *__restrict__ dst, long stride, Geo G, Phys P,
                   int nstrips, int seg)
{
    constexpr int HX = (64 - kLevelOut) / 2;  // halo columns on either side
    const int nx = G.nx, ny = G.ny;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));  // uniform
    const int w0 = (int)blockIdx.x * kPairWaves + wave, strip = w0 % nstrips;
    const int y0 = w0 / nstrips * seg, y1 = min(y0 + seg, ny);
    if (y0 >= ny) return;  // whole wavefront; nothing here waits on others
    const int x = strip * kLevelOut - HX + lane;
    const int xw = ((x % nx) + nx) % nx;
    const int xm = xw == 0 ? nx - 1 : xw - 1, xp = xw == nx - 1 ? 0 : xw + 1;
    const bool ox = lane >= HX && lane < HX + kLevelOut && x < nx;
    const unsigned sT = sizeof(T), pT = (unsigned)G.ps * sT;  // bytes of a plane
    const auto rsrc = [pT](const T *p) __attribute__((always_inline)) {
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<T *>(p), 0, (int)(12 * pT), 0x00020000);
    };
    const __amdgpu_buffer_rsrc_t rs = rsrc(src);
    auto load = [&](int r, T(&b)[12]) __attribute__((always_inline)) {
        const unsigned row = (unsigned)r * nx, rm = (unsigned)(r == 0 ? ny - 1 : r - 1) * nx,
                       rp = (unsigned)(r == ny - 1 ? 0 : r + 1) * nx;
        const unsigned o[4] = {(row + xm) * sT, (rm + xw) * sT, (row + xp) * sT, (rp + xw) * sT};
#pragma unroll
        for (int pl = 0; pl < 12; ++pl) pair_load(rs, o[pl & 3], pl * pT, b[pl]);
    };
    // of each level but the last: e1, e3 of its newest row, e2 of its two newest
    T e1[K - 1][3], e3[K - 1][3], e2[K - 1][2][3];
#pragma unroll
    for (int k = 0; k < K - 1; ++k)
#pragma unroll
        for (int c = 0; c < 3; ++c) e1[k][c] = e3[k][c] = e2[k][0][c] = e2[k][1][c] = (T)1;
    T ub[12];
    int ru = (((y0 - (K - 1)) % ny) + ny) % ny;  // row of the last load
    load(ru, ub);
    const int niter = (y1 - y0) + 2 * (K - 1);
    for (int j = 0; j < niter; j += 2) {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int i = y0 - (K - 1) + j + q;
            double v[12];
#pragma unroll
            for (int pl = 0; pl < 12; ++pl) v[pl] = (double)ub[pl];
            __builtin_amdgcn_sched_barrier(0);
            ru = ru == ny - 1 ? 0 : ru + 1;
            load(ru, ub);
#pragma unroll
            for (int k = 0; k < K; ++k) {  // level k + 1 at row i - k
                collide2d<T>(v, P);
                const int r = i - k;
                const unsigned o = ox && r >= y0 && r < y1 ? ((unsigned)r * nx + x) * sT : kPairDrop;
                const __amdgpu_buffer_rsrc_t rd = rsrc(dst + k * stride);
#pragma unroll
                for (int pl = 0; pl < 12; ++pl) pair_store(rd, o, pl * pT, (T)v[pl]);
                if (k == K - 1) break;
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    const T n1 = (T)v[4 * c + 0], n2 = (T)v[4 * c + 1], n3 = (T)v[4 * c + 2];
                    v[4 * c + 0] = (double)pair_shr(e1[k][c]);
                    v[4 * c + 1] = (double)e2[k][q][c];
                    v[4 * c + 2] = (double)pair_shl(e3[k][c]);
                    v[4 * c + 3] = (double)(T)v[4 * c + 3];
                    e1[k][c] = n1;
                    e2[k][q][c] = n2;
                    e3[k][c] = n3;
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
}

template <typename T, int K>
static hipError_t levels_strip(const void *src, void *dst, long stride, const Geo &G,
                               const Phys &P, hipStream_t st)
{
    const int ns = (G.nx + kLevelOut - 1) / kLevelOut;
    const int seg = levels_strip_rows(G, K);
    const long waves = (long)ns * ((G.ny + seg - 1) / seg);
    hipLaunchKernelGGL((k_levels_strip<T, K>), dim3((waves + kPairWaves - 1) / kPairWaves),
                       dim3(64 * kPairWaves), 0, st, (const T *)src, (T *)dst, stride, G, P, ns,
                       seg);
    return hipGetLastError();
}

// Steps per launch (us a step for K = 2 / 3 / 4 at 1024^2 and 2048^2: FP32 16.8 / 18.0 /
// 19.7 and 76 / 73 / 71, FP64 35.1 / 32.3 / 29.7 and 124 / 114 / 108); 0 where the
// buffers are beyond 32-bit byte offsets, and on flat grids, where a segment's start is not
// made up for (1000000 x 3 FP32 64 us a step, single ones 53; 100000 x 16 33.8 and 28.7).
int levels_strip_steps(const Geo &G, bool f32)
{
    if (G.ny <= (f32 ? 16 : 8)) return 0;
    if (12L * G.ps * (f32 ? 4 : 8) >= (1L << 31)) return 0;
    return f32 && (long)G.nx * G.ny < 2000000 ? 2 : kLevelStripMost;
}
int levels_strip_rows(const Geo &G, int K)
{
    return strip_seg(G, (G.nx + kLevelOut - 1) / kLevelOut, 2 * K);
}
hipError_t launch_levels_strip(bool f32, const void *src, void *dst, long stride, const Geo &G,
                               const Phys &P, int K, hipStream_t st)
{
    switch (K) {
    case 2: return f32 ? levels_strip<float, 2>(src, dst, stride, G, P, st)
                       : levels_strip<double, 2>(src, dst, stride, G, P, st);
    case 3: return f32 ? levels_strip<float, 3>(src, dst, stride, G, P, st)
                       : levels_strip<double, 3>(src, dst, stride, G, P, st);
    case 4: return f32 ? levels_strip<float, 4>(src, dst, stride, G, P, st)
                       : levels_strip<double, 4>(src, dst, stride, G, P, st);
    default: return hipErrorInvalidValue;
    }
}

} // namespace lbm

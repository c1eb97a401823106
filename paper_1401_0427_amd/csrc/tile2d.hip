// 2D steps on small grids: a tile of the grid in the registers of one workgroup,
// many steps per launch (D2Q4 per component and D2Q5Q4Q4, any faces).
//
// One step per launch costs 3.3 - 5.5 us whatever the grid's size up to about 10^5
// nodes (its start, one round trip to memory, its end), and the wave-strip kernels
// need long columns to be worth their warm-up.  Here a workgroup of TX x TY threads
// takes a tile of TX x (TY R) nodes, a thread R rows of one column, loads it once,
// advances it K steps and stores the nodes at least K away from the tile's edges
// inside the grid (each step invalidates one more row and column there).  A step
// pulls e1 / e3 from the neighbour lanes (DPP wave shifts; a wavefront holds 64 / TX
// rows of threads, and what crosses from one row of lanes to the next arrives at the
// tile's edge), e2 / e4 from the thread's own registers between its rows, and from
// LDS across threads (six values per thread, two buffers, one barrier per step).
// The face rules are the one-step kernel's, applied to the boundary node's own
// previous-level values by selects, in the wavefronts that hold boundary nodes.
// Every level is rounded to the storage type: K steps in one launch equal K single
// steps bit for bit.
#include <type_traits>

#include "internal.h"
#include "rest_device.h"
#include "multistep.h"

namespace lbm {

template <typename PH>
constexpr bool kTileRest = std::is_same<PH, Mrt>::value;

template <int CTRL>
__device__ __forceinline__ double tile_dpp(double v)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(b & 0xffffffffLL), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xf, 0xf, true);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
template <int CTRL>
__device__ __forceinline__ float tile_dpp(float v)
{
    return __int_as_float(
        __builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
template <typename T>
__device__ __forceinline__ T tile_shr(T v) { return tile_dpp<0x138>(v); }  // from lane l - 1
template <typename T>
__device__ __forceinline__ T tile_shl(T v) { return tile_dpp<0x130>(v); }  // from lane l + 1

template <typename T>
__device__ __forceinline__ void tile_collide(double, double *f, double *, const Phys &P)
{
    collide2d<T>(f, P);
}
template <typename T>
__device__ __forceinline__ void tile_collide(double r0, double *f, double *o0, const Mrt &M)
{
    double g[13];
    g[0] = r0;
#pragma unroll
    for (int i = 0; i < 12; ++i) g[1 + i] = f[i];
    collide_mrt2d(g, M);
    *o0 = g[0];
#pragma unroll
    for (int i = 0; i < 12; ++i) f[i] = g[1 + i];
}
template <typename T>
__device__ __forceinline__ void tile_inflow(const double *w, const Phys &P, double *e)
{
    feq2d<T>(w[0], w[1], w[2], P, e);
}
template <typename T>
__device__ __forceinline__ void tile_inflow(const double *w, const Mrt &M, double *e)
{
    double g[13];
    feq_rest2d(w[0], w[1], w[2], M, g);
#pragma unroll
    for (int i = 0; i < 12; ++i) e[i] = g[1 + i];
}

// One face for one node of this lane: which rule (if any) replaces the pull of the
// populations that cross it, and their inflow values.
struct TileFace {
    bool neumann, wall, inflow;
    double w[3];
};
// The direction (0 e1, 1 e2, 2 e3, 3 e4) pulled through each face.
constexpr int tile_face_dir(int face) { return face == 0 ? 0 : face == 1 ? 2 : face == 2 ? 1 : 3; }

// Pulls p[3] (components h, qx, qy) of direction j through face `face`, from the
// node's own previous values own[12].
template <typename T>
__device__ __forceinline__ void tile_pull(const TileFace &F, int face, const T *own, double *p)
{
    const int j = tile_face_dir(face), opp = (j + 2) & 3, normal = face < 2 ? 1 : 2;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const double a = (double)own[4 * c + j], b = (double)own[4 * c + opp];
        p[c] = F.neumann ? a : p[c];
        p[c] = F.wall ? (c == normal ? -b : b) : p[c];
        p[c] = F.inflow ? F.w[c] : p[c];
    }
}

// LEVELS: every level is stored, level k + 1 of the launch at dst + k * stride (else only
// the last, at dst).
template <typename T, typename PH, bool BND, bool LEVELS, int TX, int TY, int R>
__global__ void __launch_bounds__(TX * TY)
    k_tile2d(const T *__restrict__ src, T *__restrict__ dst, long stride, Geo G, PH P, int K,
             int ntx)
{
    constexpr int NR = kTileRest<PH> ? 1 : 0;
    constexpr int NT = TX * TY;
    static_assert(64 % TX == 0 && NT % 64 == 0, "whole rows of lanes per wavefront");
    // rows handed up (e2 of a thread's last row) and down (e4 of its first), with a row
    // of threads of padding at either end
    __shared__ T up[2][3][NT + TX], down[2][3][NT + TX];
    const int nx = G.nx, ny = G.ny;
    const long ps = G.ps;
    const int t = threadIdx.x, tx = t % TX, ty = t / TX;
    const int bx = (int)blockIdx.x % ntx, by = (int)blockIdx.x / ntx;
    const int x = bx * (TX - 2 * K) - K + tx;             // this thread's column, unwrapped
    const int y0 = by * (TY * R - 2 * K) - K + ty * R;    // its first row
    const bool perx = !BND || G.bc[0] == BC_PERIODIC, pery = !BND || G.bc[2] == BC_PERIODIC;
    const int xw = perx ? ((x % nx) + nx) % nx : min(max(x, 0), nx - 1);

    T f[R][12], r0[kTileRest<PH> ? R : 1];
    {
        int yw = pery ? ((y0 % ny) + ny) % ny : 0;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (!pery) yw = min(max(y0 + r, 0), ny - 1);
            const T *s = src + (long)yw * nx + xw;
            if constexpr (kTileRest<PH>) r0[r] = s[0];
#pragma unroll
            for (int pl = 0; pl < 12; ++pl) f[r][pl] = s[(NR + pl) * ps];
            if (pery) yw = yw == ny - 1 ? 0 : yw + 1;
        }
    }

    const bool ox = tx >= K && tx < TX - K && x < nx;
    auto store = [&](T *out) __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int y = y0 + r, i = ty * R + r;
            if (ox && i >= K && i < TY * R - K && y < ny) {
                T *d = out + (long)y * nx + x;
                if constexpr (kTileRest<PH>) d[0] = r0[r];
#pragma unroll
                for (int pl = 0; pl < 12; ++pl) d[(NR + pl) * ps] = f[r][pl];
            }
        }
    };
    auto steps = [&](auto xc, auto yc) __attribute__((always_inline)) {
        constexpr bool XF = decltype(xc)::value, YF = decltype(yc)::value;
        TileFace F[4]{};
        if constexpr (XF || YF) {
#pragma unroll
            for (int face = 0; face < 4; ++face) {
                const int bc = G.bc[face];
                if ((face < 2 && XF) || (face >= 2 && YF)) {
                    const bool here = face == 0 ? x == 0 : face == 1 ? x == nx - 1 : true;
                    F[face].neumann = here && bc == BC_NEUMANN;
                    F[face].wall = here && bc == BC_WALL;
                    F[face].inflow = here && bc == BC_INFLOW;
                    double e[12] = {};
                    if (bc == BC_INFLOW) tile_inflow<T>(G.win[face], P, e);
#pragma unroll
                    for (int c = 0; c < 3; ++c) F[face].w[c] = e[4 * c + tile_face_dir(face)];
                }
            }
        }
        for (int k = 0; k < K; ++k) {
            const int b = k & 1;
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                up[b][c][TX + t] = f[R - 1][4 * c + 1];
                down[b][c][t] = f[0][4 * c + 3];
            }
            __syncthreads();
            // (a buffer is written again two steps later, after the next barrier)
            T below[3], above[3];
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                below[c] = up[b][c][t];
                above[c] = down[b][c][TX + t];
            }
#pragma unroll
            for (int r = 0; r < R; ++r) {
                double v[12];
                T own[12];
#pragma unroll
                for (int pl = 0; pl < 12; ++pl) own[pl] = f[r][pl];
                double p1[3], p2[3], p3[3], p4[3];
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    p1[c] = (double)tile_shr(own[4 * c + 0]);
                    p2[c] = (double)below[c];
                    p3[c] = (double)tile_shl(own[4 * c + 2]);
                    p4[c] = (double)(r + 1 < R ? f[r + 1][4 * c + 3] : above[c]);
                    below[c] = own[4 * c + 1];
                }
                if constexpr (XF) {
                    tile_pull(F[0], 0, own, p1);
                    tile_pull(F[1], 1, own, p3);
                }
                if constexpr (YF) {
                    const bool lo = y0 + r == 0, hi = y0 + r == ny - 1;
                    TileFace A = F[2], B = F[3];
                    A.neumann = A.neumann && lo;
                    A.wall = A.wall && lo;
                    A.inflow = A.inflow && lo;
                    B.neumann = B.neumann && hi;
                    B.wall = B.wall && hi;
                    B.inflow = B.inflow && hi;
                    tile_pull(A, 2, own, p2);
                    tile_pull(B, 3, own, p4);
                }
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    v[4 * c + 0] = p1[c];
                    v[4 * c + 1] = p2[c];
                    v[4 * c + 2] = p3[c];
                    v[4 * c + 3] = p4[c];
                }
                double o0 = 0.0;
                tile_collide<T>((double)r0[kTileRest<PH> ? r : 0], v, &o0, P);
                if constexpr (kTileRest<PH>) r0[r] = (T)o0;
#pragma unroll
                for (int pl = 0; pl < 12; ++pl) f[r][pl] = (T)v[pl];
            }
            if constexpr (LEVELS) store(dst + k * stride);
        }
    };
    if constexpr (BND) {
        // uniform per wavefront: does it hold nodes of an x face, of a y face?
        const bool xf = !perx && __any(x == 0 || x == nx - 1);
        const bool yf = !pery && __any((y0 <= 0 && y0 + R > 0) || (y0 < ny && y0 + R >= ny));
        if (xf && yf)
            steps(std::true_type{}, std::true_type{});
        else if (xf)
            steps(std::true_type{}, std::false_type{});
        else if (yf)
            steps(std::false_type{}, std::true_type{});
        else
            steps(std::false_type{}, std::false_type{});
    } else {
        steps(std::false_type{}, std::false_type{});
    }

    if constexpr (!LEVELS) store(dst);
}

// ---- launchers -----------------------------------------------------------------------
// Tile shapes: threads TX x TY, R rows per thread.  Small tiles spread a small grid over
// the compute units (the step time is then that of one tile: a chain of dependent FP64
// operations, LDS and a barrier, 0.3 - 0.5 us); larger ones waste less on halos.
struct TileShape {
    int tx, ty, R;
    int resident;  // tiles per compute unit (registers)
};
static const TileShape kTileShapes[] = {
    {16, 16, 1, 8}, {32, 16, 1, 4}, {32, 16, 2, 2}, {64, 8, 3, 1}, {64, 8, 4, 1}, {32, 8, 4, 3}};
enum { kTile16 = 0, kTile32x16, kTile32, kTile64x24, kTile64x32, kTile32Tall };

// Microseconds per step of a K-step launch: its fixed cost, the state through the
// caches, and K steps of either one tile's latency or the issue of the tiles that share
// a compute unit (about 112 FP64 operations per node of a = 0, 160 of the MRT scheme, a
// quarter more where faces are selected).  Used to choose K for a given shape.
static double tile_cost(const Geo &G, bool rest, bool f32, bool bnd, const TileShape &S, int K)
{
    const int wo = S.tx - 2 * K, ho = S.ty * S.R - 2 * K;
    const long n = (long)((G.nx + wo - 1) / wo) * ((G.ny + ho - 1) / ho);
    const double waves = S.tx * S.ty / 64.0, es = (f32 ? 4.0 : 8.0) * (rest ? 13 : 12);
    const double c = (rest ? 0.29 : 0.2) * (f32 ? 0.9 : 1.0) * (bnd ? 1.25 : 1.0);
    const long cap = 256L * S.resident;
    const double per = n <= cap ? (double)((n + 255) / 256)
                     : n < 3 * cap ? (double)((n + cap - 1) / cap * S.resident)
                                   : (double)n / 256.0;
    const double lat = 0.06 + 0.32 * S.R * c + 0.02 * waves, issue = per * waves / 4.0 * S.R * c;
    const double mem = ((double)n * S.tx * S.ty * S.R + (double)G.nx * G.ny) * es / 8e6;
    return (4.2 + mem + K * (lat > issue ? lat : issue)) / K;
}

// Grids at most kShortSide nodes high (flat) or wide (narrow).  Tiles of the shapes below,
// chosen for grids of their area, are mostly empty there: 200000 x 2 MRT with faces FP32
// took 44.8 us a step in them, 15.6 in single steps; 20000 x 2 MRT periodic FP32 5.7, in
// tiles of 32 x 16 3.3, in strips 2.5.  Narrow grids: tiles of 16 x 16 (4 x 50000 FP64 6.6 us,
// single steps and strips, which fill few lanes, 38 and 20).  Flat ones: tiles of 32 x 16,
// six steps per launch while four rows are enough and all tiles are resident, else four;
// strips or single steps where they are cheaper.  The costs are fits to 14 flat grids of
// 32000 to 3 M nodes x 8 kinds, the choice within 15 % of the fastest: a tile has its share
// of a launch and its issue; a strip an iteration per row and level or its share of issue
// and memory per node.  Few rows leave little to share a strip's start, so it runs few
// steps: FP64 1000000 x 3 in 4, 5, 7, 9 steps 43.5, 43.2, 48.3, 54.7 us a step, FP32 in 2,
// 4, 8 34.4, 26.2, 39.6.
constexpr int kShortSide = 8;
static int short_plan(const Geo &G, bool rest, bool f32, bool bnd, bool strips, int *K)
{
    if (G.ny > kShortSide) {
        *K = 3;
        return kTile16;
    }
    const double nodes = (double)G.nx * G.ny, ny = G.ny;
    const bool six = G.ny <= 4 && (G.nx + 19) / 20 <= 256 * kTileShapes[kTile32x16].resident;
    const double each =  // us per tile and step
        (rest ? 2.6e-3 : f32 ? 1.7e-3 : 2.0e-3) * (bnd ? 1.12 : 1.0);
    const double tile = six ? 0.9 + 0.8 * each * ((G.nx + 19) / 20) : 1.4 + each * ((G.nx + 23) / 24);
    *K = six ? 6 : 4;
    if (strips) {
        const double lat = bnd ? 3.3 + 0.52 * ny : 1.8 + 0.34 * ny;
        const double node = bnd    ? (f32 ? 6.5 + 20 / ny : 11 + 22 / ny)
                            : rest ? (f32 ? 8.5 + 20 / ny : 10 + 19 / ny)
                                   : (f32 ? 5 + 13 / ny : 8.5 + 17 / ny);
        const double all = node * nodes * 1e-6;
        if ((lat > all ? lat : all) < tile) {
            *K = f32 ? (rest || G.ny < 4 ? 3 : 4) : (bnd || G.ny < 3 ? 4 : 5);
            return kRunStrips;
        }
    } else if (rest && bnd) {
        if ((f32 ? 4.2 + 23e-6 * nodes : 4.5 + 37e-6 * nodes) < tile) return kRunSteps;
    }
    return kTile32x16;
}

// Shape by the number of nodes; the limits are from grids of 7 : 4 (measured fastest, us per
// step FP64 a = 0 with inflow / wall / Neumann faces against one step per launch, at 35 x 20,
// 70 x 40, 140 x 80, 280 x 160, 560 x 320: 0.94 / 4.75, 1.03 / 4.2, 1.34 / 4.3, 2.1 / 5.6,
// 3.9 / 8.9; all periodic 0.80 / 2.7, 0.93 / 2.9, 1.2 / 3.1, 1.9 / 4.4, 3.4 / 8.9).  What
// decides is how many tiles fall on the fullest compute unit, which on such grids goes by the
// nodes: 400 x 300 with faces in tiles of 64 x 24 FP64 2.7, FP32 2.5, of 64 x 32 (at a smaller
// depth) 3.3, 3.0; 160 x 140 in 32 x 16 1.5, in 32 x 32 1.9; 640 x 600 in 32 x 32 tall 6.1, in
// 64 x 32 7.1.  A long grid of as many nodes makes more tiles and would change shape at other
// sizes (FP64 periodic, this shape / the fastest of the six at any depth / single steps:
// 1500 x 16 1.60 / 1.60 / 3.8, 1200 x 24 1.75 / 1.75 / 3.5, 40 x 2500 2.59 / 2.30 / 6.2,
// 1000 x 100 2.49 / 2.35 / 5.4, 4000 x 60 3.75 / 3.74 / 11.0, 60 x 4000 5.9 / 4.2 / 11.9; of
// 96 such runs in all kinds half are within 5 %, all but 7 within 20 %, the worst 51 %).
//   On larger grids the wave-strip launches take over (us a step tile / strips on square
// grids: periodic FP64 250 000 nodes 4.2 / 4.6, 302 000 5.3 / 4.6, 577 000 8.4 / 5.6; FP32
// 360 000 4.4 / 4.7, 462 000 5.2 / 4.8, 883 000 8.2 / 6.9; with faces FP64 462 000 7.7 / 8.5,
// 722 000 11.0 / 10.8, FP32 1.05 M 11.0 / 11.9, 1.7 M 15.6 / 12.7; MRT periodic FP64 202 000
// 4.4 / 4.8, 302 000 6.2 / 4.9, 722 000 12.0 / 7.1, FP32 360 000 6.2 / 6.4, 577 000 9.0 /
// 7.1).  MRT with faces has no strip launch: tiles throughout (4.2 M nodes FP64 71 us against
// 163 for one step per launch).  These limits count the nodes of whole output tiles, and grow
// with the columns that whole strips cover beyond the grid's (200 x 2000 FP64: 5.9 / 6.5;
// 2000 x 200: 6.0 / 5.1).  strip_cols: those columns, 0 where no strip launch runs.
int tile2d_plan(const Geo &G, bool rest, bool f32, long strip_cols, int *K)
{
    const bool bnd = G.bc[0] != BC_PERIODIC || G.bc[2] != BC_PERIODIC;
    const long nodes = (long)G.nx * G.ny;
    int shape, lo = 2, hi = 10;
    if (nodes >= 5000 && (G.nx <= kShortSide || G.ny <= kShortSide))
        return short_plan(G, rest, f32, bnd, strip_cols > 0, K);
    if (nodes < 5000) {
        shape = kTile16;
    } else if (nodes < (bnd || rest ? 30000 : 23500)) {
        shape = kTile32x16;
    } else if (nodes < (f32 && !rest && bnd ? 108000 : 90000)) {
        shape = kTile32;
    } else if (nodes < 150000 && !(f32 && !rest && !bnd && nodes < 112000)) {
        shape = kTile64x24;
    } else if (nodes < (!bnd ? 400000 : f32 ? 300000 : rest ? 400000 : 330000)) {
        shape = kTile64x32;
    } else if (f32) {
        shape = bnd ? kTile32 : kTile64x32;
        lo = hi = bnd ? 4 : 5;
    } else {
        shape = bnd && rest ? kTile64x32 : kTile32Tall;
        lo = hi = bnd && rest ? 7 : 6;
    }
    const TileShape &S = kTileShapes[shape];
    const int side = S.tx < S.ty * S.R ? S.tx : S.ty * S.R;
    double best = 1e30;
    for (int k = lo; k <= hi && side - 2 * k >= 2; ++k) {
        const double t = tile_cost(G, rest, f32, bnd, S, k);
        if (t < best) {
            best = t;
            *K = k;
        }
    }
    if (strip_cols > 0) {
        const long wo = S.tx - 2 * *K, ho = S.ty * S.R - 2 * *K;
        const long covered = (G.nx + wo - 1) / wo * wo * ((G.ny + ho - 1) / ho * ho);
        const long limit = rest ? (f32 ? 520000 : 270000)
                           : bnd ? (f32 ? 1500000 : 640000)
                                 : (f32 ? 450000 : 300000);
        if ((double)covered > (double)limit * strip_cols / (1.1 * G.nx)) {
            *K = 0;
            return kRunStrips;
        }
    }
    return shape;
}

template <typename T, typename PH, bool LEVELS, int TX, int TY, int R>
static hipError_t tile_launch(const void *src, void *dst, long stride, const Geo &G, const PH &P,
                              int K, hipStream_t st)
{
    const int wo = TX - 2 * K, ho = TY * R - 2 * K;
    if (K < 1 || wo < 1 || ho < 1) return hipErrorInvalidValue;
    const int ntx = (G.nx + wo - 1) / wo, nty = (G.ny + ho - 1) / ho;
    if ((long)ntx * nty > 0x7fffffffL) return hipErrorInvalidValue;
    const bool bnd = G.bc[0] != BC_PERIODIC || G.bc[2] != BC_PERIODIC;
    if (bnd)
        hipLaunchKernelGGL((k_tile2d<T, PH, true, LEVELS, TX, TY, R>), dim3(ntx * nty),
                           dim3(TX * TY), 0, st, (const T *)src, (T *)dst, stride, G, P, K, ntx);
    else
        hipLaunchKernelGGL((k_tile2d<T, PH, false, LEVELS, TX, TY, R>), dim3(ntx * nty),
                           dim3(TX * TY), 0, st, (const T *)src, (T *)dst, stride, G, P, K, ntx);
    return hipGetLastError();
}

template <typename T, typename PH>
static hipError_t tile_any(int shape, const void *src, void *dst, const Geo &G, const PH &P,
                           int K, hipStream_t st)
{
    switch (shape) {
    case kTile16: return tile_launch<T, PH, false, 16, 16, 1>(src, dst, 0, G, P, K, st);
    case kTile32x16: return tile_launch<T, PH, false, 32, 16, 1>(src, dst, 0, G, P, K, st);
    case kTile32: return tile_launch<T, PH, false, 32, 16, 2>(src, dst, 0, G, P, K, st);
    case kTile64x24: return tile_launch<T, PH, false, 64, 8, 3>(src, dst, 0, G, P, K, st);
    case kTile64x32: return tile_launch<T, PH, false, 64, 8, 4>(src, dst, 0, G, P, K, st);
    case kTile32Tall:
        if constexpr (sizeof(T) == 8)
            return tile_launch<T, PH, false, 32, 8, 4>(src, dst, 0, G, P, K, st);
        break;
    default: break;
    }
    return hipErrorInvalidValue;
}

hipError_t launch_tile2d(bool f32, int shape, const void *src, void *dst, const Geo &G,
                         const Phys &P, int K, hipStream_t st)
{
    return f32 ? tile_any<float>(shape, src, dst, G, P, K, st)
               : tile_any<double>(shape, src, dst, G, P, K, st);
}
hipError_t launch_tile2d_rest(bool f32, int shape, const void *src, void *dst, const Geo &G,
                              const Mrt &M, int K, hipStream_t st)
{
    return f32 ? tile_any<float>(shape, src, dst, G, M, K, st)
               : tile_any<double>(shape, src, dst, G, M, K, st);
}
// Shapes and depths of launches that store every level.  By nodes up to 120 000 (us per level
// FP32 / FP64 against single steps, at 96 x 64, 160^2, 256^2: 1.1 / 1.2 against 3.0, 1.4 / 1.7
// against 3.1, 2.3 / 2.9 against 3.3 / 4.1); beyond, the one of two shapes that computes fewer
// nodes for the grid (512^2 4.4 / 7.1 against 6.6 / 11.8 in 64 x 32, 64 x 4096 5.8 / 8.1 against
// 6.6 / 11.0 in 32 x 32).  FP64 with faces spills registers in 64 x 32 tiles (512^2 17.6 against
// 11.3, 700^2 34 against 22): 32 x 32 there (8.1, 15.7).  Beyond the last size the strips that
// store every level take over on all-periodic grids (724^2 FP32 10.7, 1024^2 FP64 29.7 against
// 35.4), single steps with faces (1024^2 FP32 20.6 against 21.4).
//   Flat grids take tiles of 32 x 16 where all are resident, or are not three times as many
// nodes as the grid, else single steps (20000 x 3 FP64 3.3 against 3.8, but 300000 x 2 57 in 64
// x 32 tiles, 33 in 32 x 16, 24 in strips, 25.8 in single steps; with faces 170, 37 and 20);
// narrow ones 16 x 16 (3 x 100000 FP64 15.7 against 81).
static const struct {
    long nodes;  // at most
    int shape, K;
} kLevelShapes[] = {{12000, kTile16, 5}, {50000, kTile32x16, 5}, {120000, kTile32x16, 4}};

// Tiles of a launch (owned nodes wo x ho), and the nodes they compute.
static double tile_nodes(const Geo &G, int shape, int K, long *tiles)
{
    const TileShape &S = kTileShapes[shape];
    const int wo = S.tx - 2 * K, ho = S.ty * S.R - 2 * K;
    const long n = (long)((G.nx + wo - 1) / wo) * ((G.ny + ho - 1) / ho);
    if (tiles) *tiles = n;
    return (double)n * S.tx * S.ty * S.R;
}

int tile2d_levels_plan(const Geo &G, bool f32, int *K)
{
    const long nodes = (long)G.nx * G.ny;
    const bool bnd = G.bc[0] != BC_PERIODIC || G.bc[2] != BC_PERIODIC;
    *K = 4;
    if (nodes > 5000 && G.ny <= kShortSide) {
        long n;
        const double all = tile_nodes(G, kTile32x16, 4, &n);
        return n <= 256 * kTileShapes[kTile32x16].resident || all <= 3.0 * nodes ? kTile32x16 : -1;
    }
    if (nodes > 12000 && G.nx <= kShortSide) return kTile16;
    for (const auto &s : kLevelShapes)
        if (nodes <= s.nodes) {
            *K = s.K;
            return s.shape;
        }
    if (nodes > (bnd && !f32 ? 900000 : 700000)) return -1;
    const double small = tile_nodes(G, kTile32, 4, nullptr);
    const double large = tile_nodes(G, kTile64x32, 4, nullptr);
    const bool wide = large < small && !(bnd && !f32);
    return (wide ? large : small) <= 3.0 * nodes ? (wide ? kTile64x32 : kTile32) : -1;
}

template <typename T>
static hipError_t levels_any(int shape, const void *src, void *dst, long stride, const Geo &G,
                             const Phys &P, int K, hipStream_t st)
{
    switch (shape) {
    case kTile16: return tile_launch<T, Phys, true, 16, 16, 1>(src, dst, stride, G, P, K, st);
    case kTile32x16: return tile_launch<T, Phys, true, 32, 16, 1>(src, dst, stride, G, P, K, st);
    case kTile32: return tile_launch<T, Phys, true, 32, 16, 2>(src, dst, stride, G, P, K, st);
    case kTile64x32: return tile_launch<T, Phys, true, 64, 8, 4>(src, dst, stride, G, P, K, st);
    default: return hipErrorInvalidValue;
    }
}
hipError_t launch_tile2d_levels(bool f32, int shape, const void *src, void *dst, long stride,
                                const Geo &G, const Phys &P, int K, hipStream_t st)
{
    return f32 ? levels_any<float>(shape, src, dst, stride, G, P, K, st)
               : levels_any<double>(shape, src, dst, stride, G, P, K, st);
}

void tile2d_dims(int shape, int *cols, int *rows)
{
    *cols = kTileShapes[shape].tx;
    *rows = kTileShapes[shape].ty * kTileShapes[shape].R;
}

} // namespace lbm

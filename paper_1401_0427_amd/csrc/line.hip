// 1D steps, many per launch, with the nodes in registers (D1Q2 per component and
// D1Q3Q2).
//
// A lane holds R consecutive nodes, a wavefront 64 R, and a step moves values
// between registers: f+ / g+ of node r come from node r - 1 of the same lane, f- /
// g- from node r + 1, and only the lane's end nodes exchange with the neighbour
// lanes (DPP wave shifts: eight moves per lane and step, however large R).  No LDS
// and no barrier in the step loop, so the FP64 issue rate bounds it (at 2^20 nodes;
// on small domains the chain of about 25 dependent FP64 operations of one step).
// Against one node per thread of a 1024-thread workgroup with the planes in LDS and a
// barrier per step, us a step FP64: 2^20 nodes 1.63 (2.5 before), 2^18 0.61 (1.0), 2000 to
// 30000 0.23 - 0.25 (0.5 - 0.55), 1000 with ends 0.25 (0.51), 80 with a rest population 0.37
// (0.73); one step per launch 15.9, 3.7, 2.3 - 2.5, 2.2, 1.9.
//   k_line: the domain is cut into tiles of `nout` output nodes, one wavefront each,
//     with K nodes of halo per side inside the domain (each step invalidates one more
//     node at either end).  Tiles start at multiples of R, so the domain's first node
//     is always node 0 of its lane and its last one node (nx - 1) % R.
//   k_line_whole: a domain with non-periodic ends of at most kK1Threads nodes in one
//     workgroup of W wavefronts, nothing lost at the ends, any K; neighbouring
//     wavefronts exchange their end values through LDS, one barrier per step (none
//     when W = 1).
// The face rules are those of the one-step kernel, applied to the end node's own
// previous-level values, and every level is rounded to the storage type, so K steps
// in one launch equal K single steps bit for bit.
#include <type_traits>

#include "internal.h"
#include "line_plan.h"
#include "rest_device.h"
#include "xk_wave.h"
#include "multistep.h"

namespace lbm {

// Value of lane l - 1 / l + 1 (the end lanes receive 0; they are halo lanes, or the
// face rule replaces what they pulled).
template <int CTRL>
__device__ __forceinline__ double line_dpp(double v)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(b & 0xffffffffLL), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xf, 0xf, true);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
__device__ __forceinline__ double line_shr(double v) { return line_dpp<0x138>(v); }
__device__ __forceinline__ double line_shl(double v) { return line_dpp<0x130>(v); }

// Planes of a node in registers: 4 moving ones (f+, f-, g+, g-), after the rest
// population where there is one.
template <typename PH>
constexpr bool kRest = std::is_same<PH, Mrt>::value;

template <typename T>
__device__ __forceinline__ void line_collide(double r0, const double *m, const Phys &P, double *o0,
                                             double *o)
{
    double f[4] = {m[0], m[1], m[2], m[3]};
    collide1d<T>(f, P);
#pragma unroll
    for (int i = 0; i < 4; ++i) o[i] = f[i];
    *o0 = r0;
}
template <typename T>
__device__ __forceinline__ void line_collide(double r0, const double *m, const Mrt &M, double *o0,
                                             double *o)
{
    double f[5] = {r0, m[0], m[1], m[2], m[3]};
    collide_mrt1d(f, M);
    *o0 = f[0];
#pragma unroll
    for (int i = 0; i < 4; ++i) o[i] = f[1 + i];
}

// Moving planes of the equilibrium of an inflow face's state.
template <typename T>
__device__ __forceinline__ void line_inflow(const double *w, const Phys &P, double *e)
{
    feq1d<T>(w[0], w[1], P, e);
}
template <typename T>
__device__ __forceinline__ void line_inflow(const double *w, const Mrt &M, double *e)
{
    double f[5];
    feq_rest1d(w[0], w[1], M, f);
#pragma unroll
    for (int i = 0; i < 4; ++i) e[i] = f[1 + i];
}

// Face rule of one end for this lane: which of the three replaces the end node's
// pulls through the face (none: the lane does not hold the node), and the inflow
// values.  Applied by selects, so a wavefront that holds a domain end runs the same
// straight code as the others: as branches around the end nodes the rules kept the
// compiler from overlapping the nodes' arithmetic, and the two end tiles, being the
// slowest, set the time of a launch with one or two wavefronts per SIMD.
struct LineFace {
    bool neumann, wall, inflow;
    double f, g;  // inflow values of the h and q planes
};
// Face 0 (x-) takes planes 0, 2 (f+, g+); face 1 (x+) planes 1, 3.
template <typename T, typename PH>
__device__ __forceinline__ LineFace line_face(const Geo &G, const PH &P, int face, bool here)
{
    LineFace F;
    const int bc = G.bc[face];
    F.neumann = here && bc == BC_NEUMANN;
    F.wall = here && bc == BC_WALL;
    F.inflow = here && bc == BC_INFLOW;
    double w[4] = {0.0, 0.0, 0.0, 0.0};
    if (bc == BC_INFLOW) line_inflow<T>(G.win[face], P, w);
    F.f = w[face];
    F.g = w[2 + face];
    return F;
}
__device__ __forceinline__ void line_pull(const LineFace &F, int face, const double *own, double *p)
{
    const int a = face, b = 2 + face;
    p[a] = F.neumann ? own[a] : p[a];
    p[b] = F.neumann ? own[b] : p[b];
    p[a] = F.wall ? own[a ^ 1] : p[a];
    p[b] = F.wall ? -own[b ^ 1] : p[b];
    p[a] = F.inflow ? F.f : p[a];
    p[b] = F.inflow ? F.g : p[b];
}

// The lane's nodes.
template <int R, typename PH>
struct LineNodes {
    double m[4][R];
    double r0[kRest<PH> ? R : 1];
};

// One step of the lane's R nodes.  in[]: f+, g+ of the node before the lane's first
// and f-, g- of the node after its last (previous level).  LEFT / RIGHT: the
// wavefront holds that end of the domain; f0 applies to node 0, f1[] to the last
// node (ANYR: to whichever node holds the end).
template <typename T, int R, bool LEFT, bool RIGHT, bool ANYR, typename PH>
__device__ __forceinline__ void line_step(LineNodes<R, PH> &N, const double *in, const PH &P,
                                          const LineFace &f0, const LineFace *f1)
{
    double pf = in[0], pg = in[1];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        double p[4] = {pf, r + 1 < R ? N.m[1][r + 1] : in[2], pg,
                       r + 1 < R ? N.m[3][r + 1] : in[3]};
        const double own[4] = {N.m[0][r], N.m[1][r], N.m[2][r], N.m[3][r]};
        if constexpr (LEFT)
            if (r == 0) line_pull(f0, 0, own, p);
        if constexpr (RIGHT)
            if (ANYR || r == R - 1) line_pull(f1[ANYR ? r : 0], 1, own, p);
        pf = own[0];
        pg = own[2];
        double o[4], o0;
        line_collide<T>(N.r0[kRest<PH> ? r : 0], p, P, &o0, o);
#pragma unroll
        for (int i = 0; i < 4; ++i) N.m[i][r] = (double)(T)o[i];
        if constexpr (kRest<PH>) N.r0[r] = (double)(T)o0;
    }
}

// Wavefront-private LDS for turning coalesced memory rows into R nodes per lane and
// back, one plane at a time.  Element e sits at e + e / 16, which spreads the
// accesses at a stride of R elements over the banks.
__device__ __forceinline__ int line_slot(int e) { return e + (e >> 4); }

// The rows of one plane as they lie in memory, and turned into the lane's nodes.  All planes
// are read before the first is turned, so their loads are in flight together (two steps of
// 1000 nodes FP32 one plane after the other 4.5 us a launch, MRT 5.2, together 3.9 and 4.4).
template <typename T, int R>
__device__ __forceinline__ void line_read(const T *__restrict__ p, int lane, int base, int nx,
                                          bool per, T *raw)
{
    int x = base + lane, s = 64;
    if (per) {
        x = ((x % nx) + nx) % nx;
        s = 64 % nx;
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        raw[r] = p[per ? x : min(max(x, 0), nx - 1)];
        x += s;
        if (per && x >= nx) x -= nx;
    }
}
template <typename T, int R>
__device__ __forceinline__ void line_turn(const T *raw, T *lds, int lane, double *v)
{
#pragma unroll
    for (int r = 0; r < R; ++r) lds[line_slot(r * 64 + lane)] = raw[r];
    __asm__ __volatile__("" ::: "memory");
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = (double)lds[line_slot(lane * R + r)];
    __asm__ __volatile__("" ::: "memory");
}

template <typename T, int R>
__device__ __forceinline__ void line_store(T *__restrict__ p, T *lds, int lane, int base, int ob,
                                           int oe, const double *v)
{
#pragma unroll
    for (int r = 0; r < R; ++r) lds[line_slot(lane * R + r)] = (T)v[r];
    __asm__ __volatile__("" ::: "memory");
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int x = base + r * 64 + lane;
        const T o = lds[line_slot(r * 64 + lane)];
        if (x >= ob && x < oe) p[x] = o;
    }
    __asm__ __volatile__("" ::: "memory");
}

constexpr int kLineWaves = 4;  // wavefronts (independent tiles) per workgroup

// K steps of output nodes [i nout, (i + 1) nout) by wavefront i; hl: halo nodes
// before the outputs (K rounded up to a multiple of R).
template <typename T, int R, typename PH>
__global__ void __launch_bounds__(64 * kLineWaves, 2)
    k_line(const T *__restrict__ src, T *__restrict__ dst, Geo G, PH P, int K, int nout, int hl,
           int ntiles)
{
    constexpr int NR = kRest<PH> ? 1 : 0;
    __shared__ T turn[kLineWaves][64 * R + 4 * R];
    const int wave = (int)(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int tile = (int)blockIdx.x * kLineWaves + wave;
    if (tile >= ntiles) return;  // whole wavefront; nothing here waits on others
    T *lds = turn[wave];
    const int nx = G.nx;
    const long ps = G.ps;
    const bool per = G.bc[0] == BC_PERIODIC;  // the two 1D faces are periodic together
    const int ob = tile * nout;
    const int oe = nx - ob < nout ? nx : ob + nout;
    // The wavefront's first node, unwrapped: node 0 of its lane is a multiple of R, so
    // the domain's first node is node 0 of its lane; a tile that reaches the domain's
    // end starts up to R - 1 nodes earlier, so that the last node is node R - 1.
    int base = ob - hl;
    const bool right = !per && base + 64 * R >= nx, left = !per && !right && base <= 0;
    if (right) base -= (R - (nx - base) % R) % R;
    LineNodes<R, PH> N;
    const int first = base + lane * R;
    if constexpr (R == 2) {  // a lane's two nodes, unturned: these launches 3.5 and 3.8 us
        int x0 = first, x1 = first + 1;
        if (per) {
            x0 = ((x0 % nx) + nx) % nx;
            x1 = x0 == nx - 1 ? 0 : x0 + 1;
        } else {
            x0 = min(max(x0, 0), nx - 1);
            x1 = min(max(x1, 0), nx - 1);
        }
        if constexpr (kRest<PH>) {
            N.r0[0] = ld(src + x0);
            N.r0[1] = ld(src + x1);
        }
#pragma unroll
        for (int pl = 0; pl < 4; ++pl) {
            N.m[pl][0] = ld(src + (NR + pl) * ps + x0);
            N.m[pl][1] = ld(src + (NR + pl) * ps + x1);
        }
    } else {
        T raw[4 + NR][R];
#pragma unroll
        for (int pl = 0; pl < 4 + NR; ++pl)
            line_read<T, R>(src + pl * ps, lane, base, nx, per, raw[pl]);
        if constexpr (kRest<PH>) line_turn<T, R>(raw[0], lds, lane, N.r0);
#pragma unroll
        for (int pl = 0; pl < 4; ++pl) line_turn<T, R>(raw[NR + pl], lds, lane, N.m[pl]);
    }
    auto steps = [&](auto lc, auto rc) __attribute__((always_inline)) {
        constexpr bool LEFT = decltype(lc)::value, RIGHT = decltype(rc)::value;
        LineFace f0{}, f1{};
        if constexpr (LEFT) f0 = line_face<T>(G, P, 0, first == 0);
        if constexpr (RIGHT) f1 = line_face<T>(G, P, 1, first + R == nx);
        for (int k = 0; k < K; ++k) {
            const double in[4] = {line_shr(N.m[0][R - 1]), line_shr(N.m[2][R - 1]),
                                  line_shl(N.m[1][0]), line_shl(N.m[3][0])};
            line_step<T, R, LEFT, RIGHT, false>(N, in, P, f0, &f1);
        }
    };
    if (right)
        steps(std::false_type{}, std::true_type{});
    else if (left)
        steps(std::true_type{}, std::false_type{});
    else
        steps(std::false_type{}, std::false_type{});
    if constexpr (R == 2) {
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const int x = first + r;
            if (x >= ob && x < oe) {
                if constexpr (kRest<PH>) st(dst + x, N.r0[r]);
#pragma unroll
                for (int pl = 0; pl < 4; ++pl) st(dst + (NR + pl) * ps + x, N.m[pl][r]);
            }
        }
    } else {
        if constexpr (kRest<PH>) line_store<T, R>(dst, lds, lane, base, ob, oe, N.r0);
#pragma unroll
        for (int pl = 0; pl < 4; ++pl)
            line_store<T, R>(dst + (NR + pl) * ps, lds, lane, base, ob, oe, N.m[pl]);
    }
}

// A whole domain with non-periodic ends of at most 64 R W nodes, K steps.
template <typename T, int R, int W, typename PH>
__global__ void __launch_bounds__(64 * W)
    k_line_whole(const T *__restrict__ src, T *__restrict__ dst, Geo G, PH P, int K)
{
    constexpr int NR = kRest<PH> ? 1 : 0;
    __shared__ double edge[2][W + 2][4];  // [parity][wavefront + 1][f+, g+, f-, g-]
    const int wave = (int)(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int nx = G.nx;
    const long ps = G.ps;
    const int first = (int)threadIdx.x * R;
    LineNodes<R, PH> N;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int x = first + r < nx ? first + r : nx - 1;
        if constexpr (kRest<PH>) N.r0[r] = ld(src + x);
#pragma unroll
        for (int pl = 0; pl < 4; ++pl) N.m[pl][r] = ld(src + (NR + pl) * ps + x);
    }
    auto steps = [&](auto lc, auto rc) __attribute__((always_inline)) {
        constexpr bool LEFT = decltype(lc)::value, RIGHT = decltype(rc)::value;
        LineFace f0{}, f1[R]{};
        if constexpr (LEFT) f0 = line_face<T>(G, P, 0, first == 0);
        if constexpr (RIGHT) {
#pragma unroll
            for (int r = 0; r < R; ++r) f1[r] = line_face<T>(G, P, 1, first + r == nx - 1);
        }
        for (int k = 0; k < K; ++k) {
            double in[4] = {line_shr(N.m[0][R - 1]), line_shr(N.m[2][R - 1]),
                            line_shl(N.m[1][0]), line_shl(N.m[3][0])};
            if constexpr (W > 1) {
                double(*e)[4] = edge[k & 1];
                if (lane == 63) {
                    e[wave + 1][0] = N.m[0][R - 1];
                    e[wave + 1][1] = N.m[2][R - 1];
                }
                if (lane == 0) {
                    e[wave + 1][2] = N.m[1][0];
                    e[wave + 1][3] = N.m[3][0];
                }
                __syncthreads();
                // (slots of this parity are written again two steps later, after the
                // next step's barrier)
                if (lane == 0) {
                    in[0] = e[wave][0];
                    in[1] = e[wave][1];
                }
                if (lane == 63) {
                    in[2] = e[wave + 2][2];
                    in[3] = e[wave + 2][3];
                }
            }
            line_step<T, R, LEFT, RIGHT, true>(N, in, P, f0, f1);
        }
    };
    // every wavefront runs K steps (and meets K barriers) in its own copy of the loop
    const bool left = wave == 0, right = wave == (nx - 1) / (64 * R);
    if (W == 1 || (left && right))
        steps(std::true_type{}, std::true_type{});
    else if (left)
        steps(std::true_type{}, std::false_type{});
    else if (right)
        steps(std::false_type{}, std::true_type{});
    else
        steps(std::false_type{}, std::false_type{});
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int x = first + r;
        if (x < nx) {
            if constexpr (kRest<PH>) st(dst + x, N.r0[r]);
#pragma unroll
            for (int pl = 0; pl < 4; ++pl) st(dst + (NR + pl) * ps + x, N.m[pl][r]);
        }
    }
}

// ---- launchers (shapes and depths: line_plan.h) ---------------------------------------
int line_steps(const Geo &G, bool rest, bool f32)
{
    if (step1k_whole(G) && G.nx <= kLineWholeNodes) return 0;
    return line_depth(G.nx, G.bc[0] == BC_PERIODIC, rest, f32);
}

template <typename T, int R, typename PH>
static void tile_launch(const void *src, void *dst, const Geo &G, const PH &P, int K,
                        hipStream_t st)
{
    const int nout = line_out(K, R), hl = (K + R - 1) / R * R;
    const int ntiles = (G.nx + nout - 1) / nout;
    hipLaunchKernelGGL((k_line<T, R, PH>), dim3((ntiles + kLineWaves - 1) / kLineWaves),
                       dim3(64 * kLineWaves), 0, st, (const T *)src, (T *)dst, G, P, K, nout, hl,
                       ntiles);
}

template <typename T, int R, int W, typename PH>
static void whole_launch(const void *src, void *dst, const Geo &G, const PH &P, int K,
                         hipStream_t st)
{
    hipLaunchKernelGGL((k_line_whole<T, R, W, PH>), dim3(1), dim3(64 * W), 0, st, (const T *)src,
                       (T *)dst, G, P, K);
}

// Whether a K-step launch takes the whole domain in one workgroup.
static bool line_one_group(const Geo &G, int K)
{
    return step1k_whole(G) && (G.nx <= kLineWholeNodes || K > kLineMaxK);
}
int line_tile(const Geo &G, bool rest, bool f32, int K)
{
    if (line_one_group(G, K)) return G.nx;
    return 64 * line_shape(G.nx, G.bc[0] == BC_PERIODIC, rest, f32, K, nullptr);
}

template <typename T, typename PH>
static hipError_t line_launch(const void *src, void *dst, const Geo &G, const PH &P, int K,
                              hipStream_t st)
{
    if (K < 1) return hipErrorInvalidValue;
    if (line_one_group(G, K)) {
        if (G.nx <= 64)
            whole_launch<T, 1, 1>(src, dst, G, P, K, st);
        else if (G.nx <= 128)
            whole_launch<T, 2, 1>(src, dst, G, P, K, st);
        else if (G.nx <= 256)
            whole_launch<T, 1, 4>(src, dst, G, P, K, st);
        else if (G.nx <= 512)  // (16 wavefronts: 400 steps of 257 nodes FP32 220 us, 168 so)
            whole_launch<T, 1, 8>(src, dst, G, P, K, st);
        else
            whole_launch<T, 1, 16>(src, dst, G, P, K, st);
        return hipGetLastError();
    }
    switch (line_shape(G.nx, G.bc[0] == BC_PERIODIC, kRest<PH>, sizeof(T) == 4, K, nullptr)) {
    case 2: tile_launch<T, 2>(src, dst, G, P, K, st); break;
    case 3: tile_launch<T, 3>(src, dst, G, P, K, st); break;
    case 4: tile_launch<T, 4>(src, dst, G, P, K, st); break;
    case 6: tile_launch<T, 6>(src, dst, G, P, K, st); break;
    case 7: tile_launch<T, 7>(src, dst, G, P, K, st); break;
    case 10: tile_launch<T, 10>(src, dst, G, P, K, st); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_line(bool f32, const void *src, void *dst, const Geo &G, const Phys &P, int K,
                       hipStream_t st)
{
    return f32 ? line_launch<float>(src, dst, G, P, K, st)
               : line_launch<double>(src, dst, G, P, K, st);
}
hipError_t launch_line_rest(bool f32, const void *src, void *dst, const Geo &G, const Mrt &M,
                            int K, hipStream_t st)
{
    return f32 ? line_launch<float>(src, dst, G, M, K, st)
               : line_launch<double>(src, dst, G, M, K, st);
}

} // namespace lbm

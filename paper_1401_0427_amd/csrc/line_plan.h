// Which tiles a 1D launch takes (line.hip): plain host arithmetic.
#pragma once

namespace lbm {

// Output nodes per tile of a K-step launch with R nodes per lane (a multiple of R;
// <= 0: the halo does not leave any).
inline int line_out(int K, int R) { return (64 * R - (K + R - 1) / R * R - K) / R * R; }

// Nodes per lane the tiled launch is built for, and the wavefronts per SIMD resident
// with each (registers).
struct LineShape {
    int R, waves;
};
constexpr LineShape kLineShapes[] = {{2, 6}, {3, 4}, {4, 4}, {6, 3}, {7, 3}, {10, 2}};

// Whether a tile of R nodes per lane can take the domain: k_line applies one face rule per
// tile, so where the ends are not periodic a tile must never reach both of them.
inline bool line_fits(int nx, bool per, int R) { return per || 64 * R < nx; }

// Microseconds per step of a K-step tiled launch.  A launch costs about 4.5 us (its
// start, and the load and store phases of one tile) plus the state at 5 TB/s, which
// nothing overlaps: all wavefronts load, step and store together.  A step takes a
// wavefront a + b R on its own (the chain of dependent FP64 operations of a node,
// then issue), or c R per wavefront on its SIMD once these fill it.  a, b, c fitted to
// 8 shapes x 7 depths at 7 sizes from 2000 to 2^20 nodes: the shape and depth it picks
// were the fastest measured, or within 2 % of it, at each size.
inline double line_cost(int nx, bool rest, bool f32, int K, int R, int waves)
{
    const int nout = line_out(K, R);
    if (nout <= 0) return 1e30;
    const long tiles = (nx + nout - 1) / nout;
    long w = (tiles + 1023) / 1024;  // wavefronts per SIMD (256 CUs x 4 SIMDs)
    if (w > waves) w = (tiles + 1024L * waves - 1) / (1024L * waves) * waves;  // rounds
    const double a = rest ? 0.08 : 0.09, b = rest ? 0.117 : 0.065, c = rest ? 0.117 : 0.070;
    const double one = a + b * R, all = (double)w * c * R;
    const double bytes = (double)nx * (rest ? 10 : 8) * (f32 ? 4 : 8);
    return (4.5 + bytes / 5e6 + K * (one > all ? one : all)) / K;
}

// Nodes per lane of a K-step tiled launch (0: none fits).
inline int line_shape(int nx, bool per, bool rest, bool f32, int K, double *cost)
{
    int R = 0;
    double best = 1e30;
    for (const LineShape &s : kLineShapes) {
        if (!line_fits(nx, per, s.R)) continue;
        const double t = line_cost(nx, rest, f32, K, s.R, s.waves);
        if (t < best) {
            best = t;
            R = s.R;
        }
    }
    if (cost) *cost = best;
    return R;
}

// At most this many steps per tiled launch (beyond it halos outgrow the tiles: no
// size measured faster at 128 than at 96).
constexpr int kLineMaxK = 96;
// A domain with non-periodic ends of at most this many nodes runs in one workgroup
// for any number of steps: one wavefront takes 0.16 / 0.26 us a step with 1 / 2 nodes
// per lane, four 0.33 us, against 0.31 us (0.41 with a rest population) for 48-step
// launches of tiles; sixteen wavefronts (1024 nodes on one compute unit) 0.52 us.
constexpr int kLineWholeNodes = 256;

// Steps per tiled launch that are fastest on the domain.
inline int line_depth(int nx, bool per, bool rest, bool f32)
{
    int K = 16;
    double best = 1e30, t;
    for (int k = 16; k <= kLineMaxK; k += 16) {
        line_shape(nx, per, rest, f32, k, &t);
        if (t < best) {
            best = t;
            K = k;
        }
    }
    return K;
}

} // namespace lbm

// Multi-step launches beside the wave strips of the a = 0 scheme (tblock.hip): 1D in
// registers, register tiles, the rest-population strips and the adjoint sweeps.
#pragma once
#include "internal.h"

namespace lbm {

// D2Q5Q4Q4 on all-periodic grids, K = 2 .. kMaxFuseRest2d steps per launch
// (one wavefront per 64-column strip, four to a 256-thread workgroup, segments of
// `seg` rows; bitwise equal to K single steps).  rest2k_rows: the segment length (0 if
// the device cannot be queried), *slots (may be NULL) the resident workgroups; rest2k_fills:
// whether default plans take it, segments of 16 rows giving a third of a workgroup (FP32: two
// thirds) per compute unit.
constexpr int kMaxFuseRest2d = 6;
// Depth of the regrouped launches of default plans: FP32 7 (us a step at 2048^2 and 4096^2 for
// 5, 6, 7 steps: 29.9, 30.0, 29.9 and 115, 107, 105); FP64 5, from 3 M nodes on 6 (one wavefront
// per SIMD; 5 and 6 steps at 1024^2 9.5 and 10.4, 2048^2 39.4 and 34.8, 4096^2 154 and 135).
constexpr int kDeepRest2dF32 = 7;
int rest2k_depth(const Geo &G, bool f32);
int rest2k_rows(const Geo &G, bool f32, int K, long *slots);
long rest2k_cols(const Geo &G, bool f32, int K);  // columns their whole strips cover
bool rest2k_fills(const Geo &G, bool f32);
hipError_t launch_step_rest2k(bool f32, const void *src, void *dst, const Geo &G, const Mrt &M,
                              int K, int seg, hipStream_t st);
// 1D (D1Q2 per component; D1Q3Q2), K steps per launch with the nodes in registers
// (csrc/line.hip), any faces; bitwise equal to K single steps.  K at most 96, or
// anything on a domain for which step1k_whole holds.
hipError_t launch_line(bool f32, const void *src, void *dst, const Geo &G, const Phys &P, int K,
                       hipStream_t st);
hipError_t launch_line_rest(bool f32, const void *src, void *dst, const Geo &G, const Mrt &M,
                            int K, hipStream_t st);
// Steps per kernel launch that are fastest on the domain (0: the whole run in one).
int line_steps(const Geo &G, bool rest, bool f32);

// 2D grids, K steps per launch of register tiles (csrc/tile2d.hip), any faces; bitwise
// equal to K single steps.  tile2d_plan: the tile shape and the steps per launch for a
// grid; kRunStrips where the wave-strip launches, whose whole strips cover strip_cols
// columns (0: there are none), are faster, *K then their depth (0: the grid's own);
// kRunSteps where one step per launch is.
constexpr int kRunStrips = -1, kRunSteps = -2;
int tile2d_plan(const Geo &G, bool rest, bool f32, long strip_cols, int *K);
hipError_t launch_tile2d(bool f32, int shape, const void *src, void *dst, const Geo &G,
                         const Phys &P, int K, hipStream_t st);
hipError_t launch_tile2d_rest(bool f32, int shape, const void *src, void *dst, const Geo &G,
                              const Mrt &M, int K, hipStream_t st);

// Two adjoint steps in one launch on an all-periodic 2D grid (csrc/adj_tile.hip): from
// u^n and lambda^{n+2} to lambda^n and the dL/ds partials of both; bitwise equal to
// the two one-step launches.
bool adjoint_pairs(const Geo &G, bool f32, bool a32);  // whether the grid can run them
hipError_t launch_adjoint_pair(bool f32, bool a32, const void *un, const void *lam2, void *lam0,
                               double *partials, const Geo &G, const Phys &P, hipStream_t st);
// Every level of K steps in one launch on larger all-periodic grids (csrc/adj_tile.hip):
// level k + 1 at dst + k * stride elements, K up to kLevelStripMost.  levels_strip_steps:
// the K of a grid, 0 where single steps have to do.
constexpr int kLevelStripMost = 4;
int levels_strip_steps(const Geo &G, bool f32);
hipError_t launch_levels_strip(bool f32, const void *src, void *dst, long stride, const Geo &G,
                               const Phys &P, int K, hipStream_t st);
// Small 2D grids: K steps in one launch that stores every level (level k + 1 at dst + k *
// stride elements; any faces), and K adjoint steps over stored levels (all-periodic;
// level 0 at first, level j > 0 at next + (j - 1) * stride).  *_plan: the tile shape and
// the K of the grid, -1 where strips or single steps are faster.
int tile2d_levels_plan(const Geo &G, bool f32, int *K);
hipError_t launch_tile2d_levels(bool f32, int shape, const void *src, void *dst, long stride,
                                const Geo &G, const Phys &P, int K, hipStream_t st);
int adjoint_levels_plan(const Geo &G, int *K);
hipError_t launch_adjoint_levels(bool f32, bool a32, int shape, const void *first,
                                 const void *next, long stride, const void *lamK, void *lam0,
                                 double *partials, const Geo &G, const Phys &P, int K,
                                 hipStream_t st);
// What a launch consists of: nodes of a tile, rows of a strip's segment.
void tile2d_dims(int shape, int *cols, int *rows);
void adjoint_levels_dims(int shape, int *cols, int *rows);
int adjoint_pair_rows(const Geo &G);
int levels_strip_rows(const Geo &G, int K);
int line_tile(const Geo &G, bool rest, bool f32, int K);

// Deterministic sum of n doubles into *out, n large: two launches, through kLongSum
// doubles of scratch (csrc/adjoint.hip).
constexpr int kLongSum = 256;
hipError_t launch_sum_long(const double *in, long n, double *scratch, double *out,
                           hipStream_t st);

} // namespace lbm

// gwn_far.h -- the far part of the boundary sum on grids.
//
// An edge's term 2 atan2(N, D) is an analytic function of the query away from the
// edge and the vertical curtain below it, so on a block of samples whose x/y
// distance from a chunk of the boundary is a few block widths the chunk's sum is
// a polynomial to rounding.  The grid is cut into blocks of b^3 samples (level 0),
// 2b (level 1), ...; a chunk is summed at the n^3 Chebyshev nodes of the coarsest
// blocks it is far from (far: at least kappa block half-widths away in x or in y,
// whatever its z), the node values are interpolated down the levels, and a sample
// sums only the chunks near its level-0 block itself.  On the 512^3 grid of the
// 1.05M-triangle soup that leaves 1.5% of the (sample, edge) pairs, and node values for
// about as many again: 397 -> 23.5 ms.
//
// Interpolation error.  The terms' singularities lie outside the Bernstein ellipse of
// parameter kappa + sqrt(kappa^2 + 1) in every axis: 5.2 at kappa = 2.5 (FP32), 6.2 at 3
// (FP64).  An edge at the closest allowed distance errs by 2e-7 of its largest |term| on
// the block at most with n = 10 and kappa = 2.5, 4e-8 RMS (a term's own rounding in FP32:
// 6e-8), by 6e-13 and 9e-14 RMS with n = 16 and kappa = 3; edges farther away far less.
// Measured against the sum over all chunks: FP64 3e-16 RMS and 7e-15 at most on a
// 120 x 97 x 121 grid of 30,000 triangles (n = 14: 7e-15 and 1.4e-13); FP32 RMS error
// against FP64 3.35e-8 all chunks, 3.37e-8 with the far part.
//
// Nodes have the samples' kind of coordinates (w: quantised x and y, z in cells in
// the type; the gradient, whose samples are not quantised: all in cells in the type),
// and the interpolation uses the nodes' and samples' actual
// positions, so rounding them costs no accuracy.  Sums stay in FP64 throughout.
#pragma once

#include <hip/hip_runtime.h>

#include "gwn_kernels.h"
#include "gwn_mesh.h"

namespace gwn {

constexpr int kFarLevels = 6;
constexpr int kFarMaxNodes = 16;                  // nodes per block and axis: 10 in FP32, 16 in FP64
constexpr double kFarKappa32 = 2.5, kFarKappa64 = 3.0;
constexpr size_t kFarMaxBytes = size_t(16) << 30;   // larger workspaces: larger blocks instead

// One level: blocks of b samples per axis (the last may hold fewer; b itself may exceed
// the axis), nc blocks and nn = nc * nodes node positions per axis.
struct FarLevel {
    int b[3], nc[3], nn[3];
    int thr;                     // kappa half-widths, in cells
    int2 *cx, *cy;               // per block: quantised range
    double* pos[3];              // node positions in cells
    double* w[3];                // [nn][nodes]: interpolation from the next coarser level's nodes
    double* T;                   // [C][nn x][nn y][nn z]: sums at the nodes
};

// C: values per sample (1: w, 3: the gradient)
struct FarPlan {
    int levels = 0;              // 0: no far part
    int C = 1;
    int nodes[3] = {0, 0, 0};    // per axis: n, or all the samples of an axis that has no more
    int ns[3] = {0, 0, 0};       // samples per axis
    FarLevel lv[kFarLevels];
    double* s[3];                // [ns][nodes]: interpolation from level 0's nodes to the samples
    double* U;                   // [C][nn x][ns y][nn z]: level 0's sums interpolated in y
    size_t bytes = 0;
    double cost = 0.0;           // expected time of the boundary sum, s, with or without a far part
    double t[kFarMaxNodes];      // Chebyshev nodes of [-1, 1], ascending
};

// The samples first ... last that block c of a level reaches over along an axis.  A block
// with room for more samples than are left reaches one step past the grid, so that a
// single sample has a range too.  Blocks of the next level hold two of this one's, so the
// ranges nest: first is the parent's or later, and last, the smaller of two ends of which
// the parent has the same or a later one, lies within the parent's.  A chunk far from a
// block's parent is then far from the block (the distances do not fall with the level),
// which is what makes the levels' shares of the chunks disjoint.
struct FarRange {
    long long first, last;
};

__host__ __device__ inline FarRange far_range(const FarPlan& p, const FarLevel& l, int axis, long long c) {
    FarRange r{c * l.b[axis], (c + 1) * l.b[axis] - 1};
    if (r.last > p.ns[axis]) r.last = p.ns[axis];
    return r;
}

// The crossings of a grid's columns (k_raster in grid.hip).
constexpr int kCrossings = 32;

struct ColCrossings {
    int* count;        // per column; null: no lists
    int* list;         // [kCrossings][ncols]: samples below the crossing * 2 + (sign < 0)
    long long ncols;
};

// Lays out a far part for the grid, or none (levels = 0) where the direct sum is
// expected to be as fast or the grid's form does not allow one.
FarPlan far_plan(const gwn_mesh_s* m, const GridArgs& ga, int prec, int C);

// Points the plan into ws (plan.bytes) and enqueues the node positions and
// interpolation weights.
gwn_status far_setup(FarPlan& p, const gwn_mesh_s* m, const GridArgs& ga, int prec, void* ws, hipStream_t st);

// After the node sums: down the levels, then level 0's interpolation in y.
gwn_status far_transfer(const FarPlan& p, hipStream_t st);

// Boxes of samples (boxes.hip) instead of the columns of plan p: whether, and how many.
bool want_boxes(const gwn_mesh_s* m, const GridArgs& ga, const FarPlan& p, long long* boxes);
gwn_status launch_boxes(const gwn_mesh_s* m, const GridArgs& ga, long long boxes, const ColCrossings& cc, float* w,
                        int32_t* chi_out, hipStream_t st);

// What the column kernels take: level 0 and the samples' weights.
struct FarView {
    int on;
    int nodes[3];
    int bx, by, bz, thr;
    int nnx, nnz, ny;
    const int2 *cx, *cy;
    const double *sx, *sz, *U;
    size_t ustep;                // doubles per value in U
};

inline FarView far_view(const FarPlan& p) {
    FarView v{};
    v.on = p.levels > 0;
    if (!v.on) return v;
    const FarLevel& l = p.lv[0];
    for (int a = 0; a < 3; ++a) v.nodes[a] = p.nodes[a];
    v.bx = l.b[0];
    v.by = l.b[1];
    v.bz = l.b[2];
    v.thr = l.thr;
    v.nnx = l.nn[0];
    v.nnz = l.nn[2];
    v.ny = p.ns[1];
    v.cx = l.cx;
    v.cy = l.cy;
    v.sx = p.s[0];
    v.sz = p.s[2];
    v.U = p.U;
    v.ustep = (size_t)l.nn[0] * p.ns[1] * l.nn[2];
    return v;
}

// The blocks of one level for its node columns.
struct FarNodes {
    int nodes[3], nn[3];
    int thr, pthr;               // pthr < 0: the coarsest level
    const int2 *cx, *cy, *pcx, *pcy;
    const double *px, *py, *pz;
    double* T;
    size_t tstep;                // doubles per value in T
};

inline FarNodes far_nodes(const FarPlan& p, int l) {
    FarNodes f{};
    const FarLevel& v = p.lv[l];
    for (int a = 0; a < 3; ++a) {
        f.nodes[a] = p.nodes[a];
        f.nn[a] = v.nn[a];
    }
    f.thr = v.thr;
    f.pthr = -1;
    if (l + 1 < p.levels) {
        f.pthr = p.lv[l + 1].thr;
        f.pcx = p.lv[l + 1].cx;
        f.pcy = p.lv[l + 1].cy;
    }
    f.cx = v.cx;
    f.cy = v.cy;
    f.px = v.pos[0];
    f.py = v.pos[1];
    f.pz = v.pos[2];
    f.T = v.T;
    f.tstep = (size_t)v.nn[0] * v.nn[1] * v.nn[2];
    return f;
}

// A stream that may be under capture takes no far part: its workspace would belong to
// the graph.
inline bool stream_captures(hipStream_t st) {
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(st, &cap) == hipSuccess) return cap != hipStreamCaptureStatusNone;
    (void)hipGetLastError();
    return true;
}

namespace {

// the chunks of node column (ci, cj): far from its block, not from the block's parent
__device__ __forceinline__ ChunkFilter far_filter(const FarNodes& f, int ci, int cj) {
    const int bx = ci / f.nodes[0], by = cj / f.nodes[1];
    ChunkFilter flt{};
    flt.mode = ChunkFilter::kRing;
    flt.x = f.cx[bx];
    flt.y = f.cy[by];
    flt.thr = f.thr;
    flt.pthr = f.pthr;
    if (f.pthr >= 0) {
        flt.px = f.pcx[bx / 2];
        flt.py = f.pcy[by / 2];
    }
    return flt;
}

constexpr int kFarV = 320;   // node values of 64 samples in LDS: at most 64 / 8 + 2 blocks

// Adds the far part to the samples of a wave's column (ci, cj): level 0's values
// in y are contracted in x for the z nodes of 64 samples at a time (one node per
// lane), then in z per sample.  V: the wave's LDS, kFarV doubles.
template <int ZB>
__device__ __forceinline__ void far_add(const FarView& f, int ci, int cj, int k0, int nz, int value, double* S,
                                        double* V) {
    const int lane = (int)(threadIdx.x & 63);
    const int n0 = f.nodes[0], n2 = f.nodes[2];
    const double* __restrict__ wx = f.sx + (size_t)ci * n0;
    const double* __restrict__ U = f.U + value * f.ustep + ((size_t)(ci / f.bx) * n0 * f.ny + cj) * f.nnz;
    const size_t ustep = (size_t)f.ny * f.nnz;
#pragma unroll
    for (int r = 0; r < ZB; ++r) {
        const int ka = k0 + 64 * r;
        if (ka < nz) {
            const int c0 = ka / f.bz, c1 = min(ka + 63, nz - 1) / f.bz;
            const int nv = (c1 - c0 + 1) * n2;
            for (int i = lane; i < nv; i += 64) {
                double v = 0.0;
                for (int j = 0; j < n0; ++j) v = fma(wx[j], U[j * ustep + c0 * n2 + i], v);
                V[i] = v;
            }
            wave_lds_sync();
            const int k = min(ka + lane, nz - 1);
            const double* __restrict__ wz = f.sz + (size_t)k * n2;
            const double* v = V + (k / f.bz - c0) * n2;
            double a = 0.0;
            for (int j = 0; j < n2; ++j) a = fma(wz[j], v[j], a);
            S[r] += a;
            wave_lds_sync();
        }
    }
}

}  // namespace
}  // namespace gwn

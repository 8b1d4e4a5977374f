// grid.hip -- w on a regular grid with one ray per (x, y) column (Sec. 4.3.1,
// ray reuse): the triangles are rasterised onto the columns once and every
// crossing is classified against a column's samples (k_raster); the boundary term
// shares the column's x/y work (gwn_kernels.h), and where it pays its far part is
// summed at nodes and interpolated (gwn_far.h).
//
// Built on its own with the max-ILP machine scheduler: the column kernels issue the
// same instructions under either scheduler, in an order that runs 2-5% faster
// (160 x 160 x 64 grid of the torus soup 15.8 and 16.1 ms, 512^3 of the 1.05M-triangle
// soup 26.7 and 27.5), while that scheduler costs the FP64 point kernels half their
// occupancy -- hence the separate source.
#include <cmath>
#include <cstdlib>

#include <algorithm>

#include "gwn_alloc.h"
#include "gwn_far.h"
#include "gwn_kernels.h"
#include "gwn_mesh.h"

namespace gwn {
namespace {

// Crossings of a grid's columns by rasterisation: every triangle visits the columns
// under its x/y box, applies the exact x/y test and turns a hit into the number of
// the column's samples below the triangle (a crossing is above the samples up to a
// height, so that number and the sign settle it for all of them).  The column sums
// read the short list.  A walk of the BVH per column is a chain of dependent
// loads, here every load is independent: of the 512^3 grid of the 1.05M-triangle
// soup 9.2 ms were that walk with 8 exact tests per lane and crossing.  A column of
// more than kCrossings crossings is left to its wave.

// column indices whose quantised coordinate may lie in [lo, hi] (rising coordinates;
// slack: rounding of a coordinate, in columns)
__device__ __forceinline__ void col_range(const GridArgs& ga, const QGrid& g, int axis, double slack, int n, int lo,
                                          int hi, int& i0, int& i1) {
    const double a = ((double)lo / g.scale + g.lo[axis] - ga.o[axis]) / ga.s[axis] - 0.5;
    const double b = ((double)hi / g.scale + g.lo[axis] - ga.o[axis]) / ga.s[axis] - 0.5;
    i0 = (int)fmin(fmax(ceil(a - slack), 0.0), (double)n);
    i1 = (int)fmin(fmax(floor(b + slack), -1.0), (double)(n - 1));
}

__device__ __forceinline__ void raster_hit(const GridArgs& ga, const QGrid& g, const ColCrossings& cc, const TriQ& tr,
                                           int ci, int cj) {
    const QPoint q = quantize_point(grid_coord(ga.o[0], ga.s[0], ci), grid_coord(ga.o[1], ga.s[1], cj), 0.0f, g);
    if (!q.inbox) return;
    const int s = tri_xy_sign(tr, q.x, q.y);
    if (s == 0) return;
    const int nz = (int)ga.nz;
    const PlaneQ pl = plane_of(tr, q.x, q.y);
    auto above = [&](int k) {
        const double z = qround(grid_coord(ga.o[2], ga.s[2], k), g.lo[2], g.scale);
        return plane_above(pl, (int)fmin(fmax(z, -1.0), (double)(kQMax + 1)));
    };
    // an estimate from the plane's height, checked by the exact test at the two
    // samples around it; else a bisection by that test
    const double f0 = (double)pl.nx * (tr.a.x - q.x) + (double)pl.ny * (tr.a.y - q.y) + (double)pl.nz * tr.a.z;
    const double est = ceil(((f0 / (double)pl.nz / g.scale + g.lo[2]) - ga.o[2]) / ga.s[2] - 0.5);
    int k = (int)fmin(fmax(est, 0.0), (double)nz);
    if (!((k == 0 || above(k - 1)) && (k == nz || !above(k)))) {
        int lo = 0, hi = nz;   // above(i) for i < lo, not for i >= hi
        while (lo < hi) {
            const int m = (lo + hi) >> 1;
            if (above(m)) lo = m + 1;
            else hi = m;
        }
        k = lo;
    }
    if (k == 0) return;
    const long long col = (long long)ci * ga.ny + cj;
    const int n = atomicAdd(cc.count + col, 1);   // the order of a column's list does not matter: a sum of integers
    if (n < kCrossings) cc.list[n * cc.ncols + col] = 2 * k + (s < 0);
}

// One triangle per lane, blockIdx.y: every gridDim.y-th column in x (few triangles
// against many columns).  A lane with more than 32 columns hands them to its wave.
__global__ __launch_bounds__(256) void k_raster(MeshView mv, GridArgs ga, ColCrossings cc, double slack_x,
                                                double slack_y) {
    const int t = blockIdx.x * 256 + threadIdx.x, lane = threadIdx.x & 63, step = gridDim.y;
    const bool valid = t < mv.nf;
    int i0 = 0, ni = 0, j0 = 0, nj = 0;
    TriQ tr = mv.tris[valid ? t : 0];
    if (valid) {
        int i1, j1;
        col_range(ga, mv.g, 0, slack_x, (int)ga.nx, min(tr.a.x, min(tr.b.x, tr.c.x)), max(tr.a.x, max(tr.b.x, tr.c.x)),
                  i0, i1);
        col_range(ga, mv.g, 1, slack_y, (int)ga.ny, min(tr.a.y, min(tr.b.y, tr.c.y)), max(tr.a.y, max(tr.b.y, tr.c.y)),
                  j0, j1);
        i0 += ((int)blockIdx.y + step - i0 % step) % step;   // the first of this stripe
        ni = i1 >= i0 ? (i1 - i0) / step + 1 : 0;
        nj = max(j1 - j0 + 1, 0);
    }
    const bool big = (long long)ni * nj > 32;
    if (!big)
        for (int e = 0; e < ni * nj; ++e) raster_hit(ga, mv.g, cc, tr, i0 + e / nj * step, j0 + e % nj);
    for (unsigned long long m = __builtin_amdgcn_ballot_w64(big); m; m &= m - 1) {
        const int l = __builtin_ctzll(m);
        tr = mv.tris[__builtin_amdgcn_readlane(t, l)];
        const int a0 = __builtin_amdgcn_readlane(i0, l), an = __builtin_amdgcn_readlane(ni, l);
        const int b0 = __builtin_amdgcn_readlane(j0, l), bn = __builtin_amdgcn_readlane(nj, l);
        for (long long e = lane; e < (long long)an * bn; e += 64)
            raster_hit(ga, mv.g, cc, tr, a0 + (int)(e / bn) * step, b0 + (int)(e % bn));
    }
}

// Waves per SIMD that the column kernels' registers are held to.  FP32: one more than
// the compiler's own choice at 2 samples per lane and above (512^3 grid: 25.7 ms, 27.5
// without); FP64: three, the rare path's arctangent alone would take 200 registers.
template <class T, int ZB>
constexpr int col_waves = sizeof(T) == 8 ? 3 : ZB >= 4 ? 4 : ZB == 3 ? 5 : ZB == 2 ? 6 : 1;

// One wave owns one (x, y) column and a chunk of 64*ZB consecutive z samples;
// lane l holds samples l, l+64, ..., l+64(ZB-1) of the chunk.  The column's crossings
// come from its list, or (no list, or too many) from one walk of the BVH that all
// lanes take together, each crossing classified against every sample with the exact
// plane predicate (Sec. 4.3.1, ray reuse).  They ride in the boundary sums, which
// start at 2 pi chi, so no register holds them through the loops.
//
// Bound by VALU issue: a trip of four chained vertices (col_quad) is about 90
// instructions per sample, 12 of them square roots and reciprocals at a quarter of
// the rate; all chunks of 512^3 x 10,904 vertices run at 3.3e12 vertices/s.
//
// SPLIT: a workgroup of kSplitWaves waves takes one column and shares out the
// chunks, the partial sums added in LDS in a fixed order; the waves' other work is
// repeated.  For grids of too few columns to fill the chip one wave each.
template <class T, int ZB, bool SPLIT>
__global__ __launch_bounds__(64 * (SPLIT ? kSplitWaves : kGridWaves))
__attribute__((amdgpu_waves_per_eu(col_waves<T, ZB>))) void k_grid(MeshView mv, GridArgs ga, FarView far, ColCrossings cc,
                                                          int* __restrict__ chi_out, T* __restrict__ w) {
    constexpr int W = SPLIT ? kSplitWaves : kGridWaves;
    __shared__ int wstack[W][kLdsStack];
    __shared__ ColBuf<T> buf[W];
    __shared__ double farv[SPLIT ? 1 : W][kFarV];
    __shared__ double part[SPLIT ? W : 1][SPLIT ? 64 * ZB : 1];
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lane = threadIdx.x & 63;
    const long long gw = ga.wave0 + (SPLIT ? (long long)blockIdx.x : (long long)blockIdx.x * W + wave);
    if (gw >= ga.nwaves) return;
    // column (ci, cj) and z chunk of this wave: every grid axis has at most 2^20
    // points, so they are 32-bit and wave-uniform (scalar registers)
    const long long col = gw / ga.nchunks;
    const int chunk = __builtin_amdgcn_readfirstlane((int)(gw - col * ga.nchunks));
    const int ci = __builtin_amdgcn_readfirstlane((int)(col / ga.ny));
    const int cj = __builtin_amdgcn_readfirstlane((int)(col - (long long)ci * ga.ny));
    const float px = grid_coord(ga.o[0], ga.s[0], ci);
    const float py = grid_coord(ga.o[1], ga.s[1], cj);
    const int nz = (int)ga.nz;
    const int k0 = chunk * 64 * ZB + lane;   // sample r is k0 + 64 r

    float pz[ZB];
    int qzr[ZB];
    int chi[ZB];
    const QPoint q0 = quantize_point(px, py, 0.0f, mv.g);
#pragma unroll
    for (int r = 0; r < ZB; ++r) {
        pz[r] = grid_coord(ga.o[2], ga.s[2], min(k0 + 64 * r, nz - 1));
        qzr[r] = quantize_point(px, py, pz[r], mv.g).z;
        chi[r] = 0;
    }

    // ---- crossings along the column's vertical line, classified per sample
    int nc = cc.count ? __builtin_amdgcn_readfirstlane(cc.count[col]) : kCrossings + 1;
    if (nc <= kCrossings) {
        const int e = lane < nc ? cc.list[lane * cc.ncols + col] : 0;   // one crossing per lane
        for (int i = 0; i < nc; ++i) {
            const int x = __builtin_amdgcn_readlane(e, i), s = (x & 1) ? -1 : 1;
#pragma unroll
            for (int r = 0; r < ZB; ++r) chi[r] += k0 + 64 * r < (x >> 1) ? s : 0;
        }
    } else if (q0.inbox && mv.root != kNoRoot) {
        int* stk = wstack[wave];
        int node = mv.root;
        int sp = 0;
        const bool leaf_only = node < 0;
        while (true) {
            // up to two leaves reached at this node (the triangles to test); -1 = none
            int leaf0 = -1, leaf1 = -1;
            if (leaf_only) {
                leaf0 = ~node;
            } else {
                const Node nd = mv.nodes[node];
                bool hl = box_has_xy(nd.lxy.x, nd.lxy.y, nd.lxy.z, nd.lxy.w, q0.x, q0.y);
                bool hr = box_has_xy(nd.rxy.x, nd.rxy.y, nd.rxy.z, nd.rxy.w, q0.x, q0.y);
                const int L = nd.link.x, R = nd.link.y;
                if (hl && L < 0) { leaf0 = ~L; hl = false; }
                if (hr && R < 0) { leaf1 = ~R; hr = false; }
                if (hl && hr) { stk[sp++] = R; node = L; }
                else if (hl) node = L;
                else if (hr) node = R;
                else node = -1;
            }
            for (int h = 0; h < 2; ++h) {
                const int leaf = h == 0 ? leaf0 : leaf1;
                if (leaf < 0) continue;
                const TriQ t = mv.tris[leaf];
                const int s = tri_xy_sign(t, q0.x, q0.y);
                if (s == 0) continue;
                const PlaneQ pl = plane_of(t, q0.x, q0.y);
#pragma unroll
                for (int r = 0; r < ZB; ++r) chi[r] += plane_above(pl, qzr[r]) ? s : 0;
            }
            if (leaf_only) break;
            if (node < 0) {
                if (sp == 0) break;
                node = stk[--sp];
            }
        }
    }

    // The crossing counts are final here: store them, and start each sample's
    // boundary sum at 2 pi chi (w = S / 2 pi), so that no register holds the
    // counts through the boundary loops.
    if (chi_out && (!SPLIT || wave == 0)) {
        const long long base = (long long)ci * ga.st[0] + (long long)cj * ga.st[1];
#pragma unroll
        for (int r = 0; r < ZB; ++r) {
            const int k = k0 + 64 * r;
            if (k < nz) chi_out[base + (long long)k * ga.st[2]] = chi[r];
        }
    }

    // ---- boundary term
    T pzs[ZB];
    double S[ZB];
    if (q0.inbox) {
        const T sc = (T)mv.g.scale;
        bool near = true, quad = true;
#pragma unroll
        for (int r = 0; r < ZB; ++r) {
            pzs[r] = (T)pz[r] * sc;
            S[r] = (double)chi[r] * k2Pi;
            near &= near_z(pz[r], mv.g);
            quad &= quad_z(pz[r], mv.g);
        }
        near = __builtin_amdgcn_ballot_w64(!near) == 0ull;   // one choice for the whole column
        quad = __builtin_amdgcn_ballot_w64(!quad) == 0ull;
        ChunkFilter flt{};
        flt.mode = ChunkFilter::kAll;
        if (far.on) {
            flt.mode = ChunkFilter::kNear;
            flt.x = far.cx[ci / far.bx];
            flt.y = far.cy[cj / far.by];
            flt.thr = far.thr;
        }
        if (SPLIT && wave > 0) {
#pragma unroll
            for (int r = 0; r < ZB; ++r) S[r] = 0.0;
        }
        column_chunks<T, ZB>(mv, flt, q0.x, q0.y, pzs, S, near, quad, SPLIT ? wave : 0, SPLIT ? W : 1, buf[wave]);
        if constexpr (SPLIT) {   // (the column is in the box or not for the whole workgroup)
            split_sum<ZB, W>(wave, lane, S, part);
            if (wave > 0) return;
        }
        if (far.on) far_add<ZB>(far, ci, cj, chunk * 64 * ZB, nz, 0, S, farv[SPLIT ? 0 : wave]);
    } else {
        if (SPLIT && wave > 0) return;
        float pzm = 0.f;
#pragma unroll
        for (int r = 0; r < ZB; ++r) pzm = fmaxf(pzm, fabsf(pz[r]));
        const FarScale<T> fs = far_scale<T>(px, py, pzm, mv.g.scale);
#pragma unroll
        for (int r = 0; r < ZB; ++r) {
            pzs[r] = (T)pz[r] * fs.scf;
            S[r] = (double)chi[r] * k2Pi;
        }
        boundary_loops_far<T, ZB>(mv, (T)px * fs.scf, (T)py * fs.scf, pzs, S, fs.f);
    }

    // output positions from the wave-uniform column and the lane, recomputed
    // here rather than kept through the boundary loops
    const long long base = (long long)ci * ga.st[0] + (long long)cj * ga.st[1];
    const int k1 = chunk * 64 * ZB + (int)(threadIdx.x & 63);
#pragma unroll
    for (int r = 0; r < ZB; ++r) {
        const int k = k1 + 64 * r;
        if (k < nz) w[base + (long long)k * ga.st[2]] = (T)(S[r] * kInv2Pi);
    }
}

// The sums at one level's nodes (gwn_far.h): one wave per node column and chunk of
// 64 ZB node heights, the same column sums as the grid's, over the chunks that are
// far from the column's block and near its parent.
template <class T, int ZB, bool SPLIT>
__global__ __launch_bounds__(64 * (SPLIT ? kSplitWaves : kGridWaves)) __attribute__((amdgpu_waves_per_eu(col_waves<T, ZB>))) void k_far_columns(MeshView mv, FarNodes f, int nchunks, long long wave0,
                                                                 long long nwaves) {
    constexpr int W = SPLIT ? kSplitWaves : kGridWaves;
    __shared__ ColBuf<T> buf[W];
    __shared__ double part[SPLIT ? W : 1][SPLIT ? 64 * ZB : 1];
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lane = threadIdx.x & 63;
    const long long gw = wave0 + (SPLIT ? (long long)blockIdx.x : (long long)blockIdx.x * W + wave);
    if (gw >= nwaves) return;
    const long long col = gw / nchunks;
    const int chunk = __builtin_amdgcn_readfirstlane((int)(gw - col * nchunks));
    const int ci = __builtin_amdgcn_readfirstlane((int)(col / f.nn[1]));
    const int cj = __builtin_amdgcn_readfirstlane((int)(col - (long long)ci * f.nn[1]));
    const int k0 = chunk * 64 * ZB + lane;
    T pzs[ZB];
    double S[ZB];
#pragma unroll
    for (int r = 0; r < ZB; ++r) {
        pzs[r] = (T)f.pz[min(k0 + 64 * r, f.nn[2] - 1)];
        S[r] = 0.0;
    }
    column_chunks<T, ZB>(mv, far_filter(f, ci, cj), (int)f.px[ci], (int)f.py[cj], pzs, S, true, true, SPLIT ? wave : 0, SPLIT ? W : 1, buf[wave]);
    if constexpr (SPLIT) {
        split_sum<ZB, W>(wave, lane, S, part);
        if (wave > 0) return;
    }
    double* out = f.T + ((size_t)ci * f.nn[1] + cj) * f.nn[2];
    const int k1 = chunk * 64 * ZB + (int)(threadIdx.x & 63);
#pragma unroll
    for (int r = 0; r < ZB; ++r)
        if (k1 + 64 * r < f.nn[2]) out[k1 + 64 * r] = S[r];
}

template <class T, int ZB, bool SPLIT = false>
gwn_status launch_far_zb(const gwn_mesh_s* m, const FarNodes& f, hipStream_t st) {
    const int nchunks = (f.nn[2] + 64 * ZB - 1) / (64 * ZB);
    const long long nwaves = (long long)f.nn[0] * f.nn[1] * nchunks, most = max_launch_queries() / 64;
    for (long long w0 = 0; w0 < nwaves; w0 += most) {
        const long long n = std::min(most, nwaves - w0), blocks = SPLIT ? n : (n + kGridWaves - 1) / kGridWaves;
        k_far_columns<T, ZB, SPLIT><<<(unsigned)blocks, 64 * (SPLIT ? kSplitWaves : kGridWaves), 0, st>>>(m->view(), f, nchunks, w0,
                                                                          std::min(nwaves, w0 + most));
        GWN_HIP_TRY(hipGetLastError());
    }
    return GWN_OK;
}

// node heights per lane: the number of 64-node blocks that a column fills with the
// fewest idle ones, up to 5 (FP64: 3)
template <class T>
gwn_status launch_far(const gwn_mesh_s* m, const FarNodes& f, hipStream_t st) {
    const int blocks = (f.nn[2] + 63) / 64;
    if ((long long)f.nn[0] * f.nn[1] * blocks < kFewWaves) return launch_far_zb<T, 1, true>(m, f, st);
    if (blocks == 1) return launch_far_zb<T, 1>(m, f, st);
    if (blocks == 2) return launch_far_zb<T, 2>(m, f, st);
    if constexpr (sizeof(T) == 4)
        if (blocks % 5 == 0 || blocks > 9) return launch_far_zb<T, 5>(m, f, st);
    if (blocks == 4) return launch_far_zb<T, 2>(m, f, st);
    return launch_far_zb<T, 3>(m, f, st);
}

template <class T, int ZB, bool SPLIT = false>
gwn_status launch_grid_zb(const gwn_mesh_s* m, GridArgs ga, const FarView& far, const ColCrossings& cc, T* w, int32_t* chi_out,
                          hipStream_t st) {
    ga.nchunks = (ga.nz + 64 * ZB - 1) / (64 * ZB);
    ga.nwaves = ga.nx * ga.ny * ga.nchunks;
    // at most 2^24 waves per launch
    const long long kMaxWaves = max_launch_queries() / 64;
    for (long long w0 = 0; w0 < ga.nwaves; w0 += kMaxWaves) {
        ga.wave0 = w0;
        const long long n = std::min(kMaxWaves, ga.nwaves - w0), blocks = SPLIT ? n : (n + kGridWaves - 1) / kGridWaves;
        k_grid<T, ZB, SPLIT><<<(unsigned)blocks, 64 * (SPLIT ? kSplitWaves : kGridWaves), 0, st>>>(m->view(), ga, far, cc, chi_out, w);
        GWN_HIP_TRY(hipGetLastError());
    }
    return GWN_OK;
}

// Samples per lane: more share a column's records, trips and crossings, fewer leave
// registers for more resident waves and fill short columns.  Measured (far part on,
// ms at 1, 2, 4): 512^3 33.8, 25.8, 24.1; 256^3 10.0, 9.1, 9.8; 120 x 97 x 121 3.1, 3.0,
// 5.2; 160 x 160 x 64 15.8, 21.0, 33.3; FP64 120 x 97 x 121 13.7, 13.7 (4: registers spill).
// So 4 (FP64: 2) from 8 blocks of 64 samples on, 2 where the blocks fill it, else 1; with
// hardly any boundary a wave is all prologue: 160^3 samples of one triangle 57 us at 1.
// GWN_GRID_SAMPLES_PER_LANE (1, 2, 4 or 8) overrides everything; then the mesh's tuning
// for the precision (gwn_mesh_set_tuning, gwn_mesh_autotune); larger values take the
// largest of 4 (FP64: 2).
constexpr int kFewChunks = 4;

template <class T>
gwn_status launch_columns(const gwn_mesh_s* m, GridArgs ga, const FarView& far, const ColCrossings& cc, T* w, int32_t* chi_out,
                          hipStream_t st) {
    int zb = 0;
    if (const char* e = std::getenv("GWN_GRID_SAMPLES_PER_LANE")) zb = std::atoi(e);
    if (zb == 0) zb = m->grid_zb[sizeof(T) == 8 ? GWN_PREC_FP64 : GWN_PREC_FP32];
    const long long blocks = (ga.nz + 63) / 64;
    if (zb == 0) {
        if (split_columns(ga.nx * ga.ny, blocks, m->nchunk, sizeof(T) == 8)) return launch_grid_zb<T, 1, true>(m, ga, far, cc, w, chi_out, st);
        zb = blocks >= 8 ? 4 : blocks == 2 || blocks >= 4 ? 2 : 1;
        if (m->nchunk < kFewChunks && blocks == 3) zb = 4;   // the fewest waves
    }
    if constexpr (sizeof(T) == 4)
        if (zb >= 4) return launch_grid_zb<T, 4>(m, ga, far, cc, w, chi_out, st);
    if (zb >= 2) return launch_grid_zb<T, 2>(m, ga, far, cc, w, chi_out, st);
    return launch_grid_zb<T, 1>(m, ga, far, cc, w, chi_out, st);
}

// Crossing lists (132 bytes per column, at most 4 GiB) where the columns' x, y rise by
// steps well above a float's rounding, so that a triangle's columns follow from its
// box, and z rises, so that a crossing is one number; and where they pay.  Lists cost 22 us
// whatever the grid: an allocation, a clear and a launch.  Without them each column's wave
// walks the BVH, about 0.1 us log2(triangles)^2 for up to 3,000 waves at once, half as much
// again on a soup (us, lists / walk: 320 closed triangles 32^3 samples 37 / 14, 100^3 42 / 39,
// 160^3 83 / 207; 5,120 32^3 36 / 24, 64^3 36 / 35, 100^3 36 / 57; 20,480 48^3 35 / 33, 64^3
// 35 / 45; four open spheres of 1,329 48^3 38 / 35, 64^3 41 / 46); soups of many chunks of
// boundary are as many shells, whose walk is longer (770 triangles in 36 chunks 32^3 40 / 59).
bool want_crossings(const gwn_mesh_s* m, const GridArgs& ga, double* slack) {
    if (m->nf < 1 || ga.nx * ga.ny > (1ll << 25) || !(ga.s[2] > 0.0)) return false;
    if (m->nchunk < 16) {
        const double waves = (double)ga.nx * (double)ga.ny * std::ceil((double)ga.nz / 64.0), depth = std::log2((double)m->nf);
        if ((m->nb > 0 ? 0.16 : 0.1) * depth * depth * std::max(1.0, waves / 3000.0) < 22.0) return false;
    }
    const long long n[2] = {ga.nx, ga.ny};
    for (int a = 0; a < 2; ++a) {
        const double big = std::max(std::fabs(ga.o[a]), std::fabs(ga.o[a] + (double)n[a] * ga.s[a]));
        if (!(ga.s[a] > 0.0) || !(ga.s[a] >= 0x1p-20 * big)) return false;
        // a float's rounding and the quantisation's, in columns, and the estimate's own
        slack[a] = (0x1p-23 * big + 1.0 / m->g.scale) / ga.s[a] + 1e-3;
    }
    return std::isfinite(slack[0]) && std::isfinite(slack[1]);
}

// Stripes of columns per triangle so that a soup of few triangles fills the chip too.
gwn_status launch_crossings(const gwn_mesh_s* m, const GridArgs& ga, const ColCrossings& cc, const double* slack,
                            hipStream_t st) {
    GWN_HIP_TRY(hipMemsetAsync(cc.count, 0, sizeof(int) * (size_t)cc.ncols, st));
    const long long stripes = std::min<long long>({ga.nx, 1024, std::max<long long>(1, 65536 / m->nf)});
    k_raster<<<dim3((unsigned)((m->nf + 255) / 256), (unsigned)stripes), 256, 0, st>>>(m->view(), ga, cc, slack[0],
                                                                                     slack[1]);
    GWN_HIP_TRY(hipGetLastError());
    return GWN_OK;
}

// With a far part where far_plan() expects one to pay: its node sums and their
// interpolation first, in a stream-ordered workspace.  A stream that is being
// captured and a workspace that cannot be had take the sum over all chunks instead.  FP32
// grids of few samples take boxes (boxes.hip), captured or not; without crossing lists
// these walk the BVH per sample.
template <class T>
gwn_status launch_grid(const gwn_mesh_s* m, GridArgs ga, T* w, int32_t* chi_out, hipStream_t st) {
    constexpr int prec = sizeof(T) == 8 ? GWN_PREC_FP64 : GWN_PREC_FP32;
    FarPlan p;
    ColCrossings cc{};
    const long long ncols = ga.nx * ga.ny;
    void* ws = nullptr;
    size_t clist = 0;
    double slack[2];
    long long boxes = 0;
    bool box = false;
    p = far_plan(m, ga, prec, 1);
    if constexpr (sizeof(T) == 4) box = want_boxes(m, ga, p, &boxes);
    const bool captures = stream_captures(st);
    if (box || captures) p.levels = 0;
    if (!captures) {
        if (want_crossings(m, ga, slack)) clist = sizeof(int) * (size_t)(kCrossings + 1) * (size_t)ncols;
        const size_t far_bytes = p.levels > 0 ? p.bytes : 0;
        if (far_bytes + clist > 0) {
            if (gwn::dmalloc_async(&ws, far_bytes + clist, st) != hipSuccess) {
                (void)hipGetLastError();
                p.levels = 0;
            } else if (clist > 0) {
                cc.count = (int*)((char*)ws + far_bytes);
                cc.list = cc.count + ncols;
                cc.ncols = ncols;
            }
        }
    }
    gwn_status s = GWN_OK;
    if (cc.count) s = launch_crossings(m, ga, cc, slack, st);
    if (p.levels > 0) {
        if (s == GWN_OK) s = far_setup(p, m, ga, prec, ws, st);
        for (int l = 0; l < p.levels && s == GWN_OK; ++l) s = launch_far<T>(m, far_nodes(p, l), st);
        if (s == GWN_OK) s = far_transfer(p, st);
    }
    if constexpr (sizeof(T) == 4)
        if (s == GWN_OK && box) s = launch_boxes(m, ga, boxes, cc, w, chi_out, st);
    if (s == GWN_OK && !box) s = launch_columns<T>(m, ga, far_view(p), cc, w, chi_out, st);
    if (ws) (void)hipFreeAsync(ws, st);
    return s;
}

}  // namespace

gwn_status query_grid(const gwn_mesh_s* m, const double* origin, const double* spacing, const int64_t* dims, int prec,
                      void* w, int32_t* chi_out, hipStream_t st) {
    GridArgs ga = frame_grid(m->axis, origin, spacing, dims);
    if (ga.nx == 0 || ga.ny == 0 || ga.nz == 0) return GWN_OK;
    if (prec == GWN_PREC_FP64) return launch_grid<double>(m, ga, (double*)w, chi_out, st);
    return launch_grid<float>(m, ga, (float*)w, chi_out, st);
}

}  // namespace gwn

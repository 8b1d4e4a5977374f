// far.hip -- the far part of the boundary sum on grids (gwn_far.h): the choice of
// its blocks and levels, node positions and interpolation weights, and the
// interpolation from coarse to fine levels.  The sums at the nodes are the grid
// kernels' own column sums (grid.hip, grad.hip).
#include <algorithm>
#include <cmath>
#include <cstdlib>

#include "../../include/gwn_test.h"
#include "gwn_far.h"

namespace gwn {
namespace {

// sample i of an axis in the mesh frame, as the column kernels place it: x, y
// quantised for w (C = 1), else in cells
__device__ __forceinline__ double far_sample(const GridArgs& ga, const QGrid& g, bool f32, int C, int axis, long long i) {
    const float p = grid_coord(ga.o[axis], ga.s[axis], i);
    if (C == 1 && axis < 2) return qround(p, g.lo[axis], g.scale);
    return f32 ? (double)(p * (float)g.scale) : (double)p * g.scale;
}

// blockIdx.y: axis, blockIdx.z: level; one thread per block of samples
__global__ void k_far_nodes(FarPlan p, GridArgs ga, QGrid g, bool f32) {
    const int axis = blockIdx.y;
    const FarLevel& l = p.lv[blockIdx.z];
    const int c = blockIdx.x * 64 + threadIdx.x, n = p.nodes[axis];
    if (c >= l.nc[axis]) return;
    const FarRange i = far_range(p, l, axis, c);
    const double a = far_sample(ga, g, f32, p.C, axis, i.first), b = far_sample(ga, g, f32, p.C, axis, i.last);
    if (axis < 2) {
        const double qa = far_sample(ga, g, f32, 1, axis, i.first), qb = far_sample(ga, g, f32, 1, axis, i.last);
        (axis == 0 ? l.cx : l.cy)[c] = make_int2((int)fmin(qa, qb), (int)fmax(qa, qb));
    }
    for (int j = 0; j < n; ++j) {
        double x;
        if (n == p.ns[axis]) x = far_sample(ga, g, f32, p.C, axis, j);   // the samples themselves (one block)
        else x = 0.5 * (a + b) + 0.5 * (b - a) * p.t[j];                 // in the samples' direction
        l.pos[axis][c * n + j] = p.C == 1 && axis < 2 ? rint(x) : f32 ? (double)(float)x : x;
    }
}

// Lagrange weights at x of the n nodes xs
__device__ void lagrange(double x, const double* xs, int n, double* w) {
    for (int j = 0; j < n; ++j) {
        double num = 1.0, den = 1.0;
        for (int m = 0; m < n; ++m)
            if (m != j) {
                num *= x - xs[m];
                den *= xs[j] - xs[m];
            }
        w[j] = num / den;
    }
}

// blockIdx.z < levels - 1: weights of level z's nodes from level z + 1's; the last:
// weights of the samples from level 0's nodes
__global__ void k_far_weights(FarPlan p, GridArgs ga, QGrid g, bool f32) {
    const int axis = blockIdx.y, lev = blockIdx.z, n = p.nodes[axis];
    const int i = blockIdx.x * 64 + threadIdx.x;
    const bool sample = lev == p.levels - 1;
    const FarLevel& from = p.lv[sample ? 0 : lev + 1];
    int c;
    double x;
    double* w;
    if (sample) {
        if (i >= p.ns[axis]) return;
        x = far_sample(ga, g, f32, p.C, axis, i);
        c = i / from.b[axis];
        w = p.s[axis];
    } else {
        const FarLevel& l = p.lv[lev];
        if (i >= l.nn[axis]) return;
        x = l.pos[axis][i];
        c = min(i / n / 2, from.nc[axis] - 1);
        w = l.w[axis];
    }
    lagrange(x, from.pos[axis] + (size_t)c * n, n, w + (size_t)i * n);
}

// Adds the parent level's sums, interpolated, to a block's nodes: one workgroup per
// block of the finer level, the three axes in turn through LDS.
__global__ __launch_bounds__(256) void k_far_down(FarPlan p, int lev, int value) {
    extern __shared__ double sm[];
    const int n0 = p.nodes[0], n1 = p.nodes[1], n2 = p.nodes[2], nt = n0 * n1 * n2;
    double *A = sm, *B = sm + nt;
    const FarLevel &l = p.lv[lev], &up = p.lv[lev + 1];
    const int bz = blockIdx.x % l.nc[2], by = (blockIdx.x / l.nc[2]) % l.nc[1], bx = blockIdx.x / l.nc[2] / l.nc[1];
    const int ux = min(bx / 2, up.nc[0] - 1), uy = min(by / 2, up.nc[1] - 1), uz = min(bz / 2, up.nc[2] - 1);
    const double* T = up.T + value * (size_t)up.nn[0] * up.nn[1] * up.nn[2];
    for (int e = threadIdx.x; e < nt; e += 256) {
        const int k = e % n2, j = (e / n2) % n1, i = e / n2 / n1;
        A[e] = T[((size_t)(ux * n0 + i) * up.nn[1] + uy * n1 + j) * up.nn[2] + uz * n2 + k];
    }
    __syncthreads();
    for (int e = threadIdx.x; e < nt; e += 256) {   // z
        const int k = e % n2, ij = e / n2;
        const double* w = l.w[2] + (size_t)(bz * n2 + k) * n2;
        double s = 0.0;
        for (int m = 0; m < n2; ++m) s = fma(w[m], A[ij * n2 + m], s);
        B[e] = s;
    }
    __syncthreads();
    for (int e = threadIdx.x; e < nt; e += 256) {   // y
        const int k = e % n2, j = (e / n2) % n1, i = e / n2 / n1;
        const double* w = l.w[1] + (size_t)(by * n1 + j) * n1;
        double s = 0.0;
        for (int m = 0; m < n1; ++m) s = fma(w[m], B[(i * n1 + m) * n2 + k], s);
        A[e] = s;
    }
    __syncthreads();
    double* O = l.T + value * (size_t)l.nn[0] * l.nn[1] * l.nn[2];
    for (int e = threadIdx.x; e < nt; e += 256) {   // x
        const int k = e % n2, j = (e / n2) % n1, i = e / n2 / n1;
        const double* w = l.w[0] + (size_t)(bx * n0 + i) * n0;
        double s = 0.0;
        for (int m = 0; m < n0; ++m) s = fma(w[m], A[(m * n1 + j) * n2 + k], s);
        O[((size_t)(bx * n0 + i) * l.nn[1] + by * n1 + j) * l.nn[2] + bz * n2 + k] += s;
    }
}

// Level 0's sums at (x node, sample in y, z node): a thread keeps the nodes of one
// block in y and writes all of its samples.  N: nodes in y (0: any number).
template <int N>
__global__ __launch_bounds__(256) void k_far_y(FarPlan p, int value) {
    const FarLevel& l = p.lv[0];
    const int n = N ? N : p.nodes[1];
    const long long id = blockIdx.x * 256ll + threadIdx.x;
    if (id >= (long long)l.nn[0] * l.nc[1] * l.nn[2]) return;
    const int z = (int)(id % l.nn[2]), c = (int)(id / l.nn[2] % l.nc[1]), x = (int)(id / l.nn[2] / l.nc[1]);
    const double* T = l.T + ((size_t)value * l.nn[0] + x) * l.nn[1] * l.nn[2] + (size_t)c * n * l.nn[2] + z;
    double* U = p.U + ((size_t)value * l.nn[0] + x) * p.ns[1] * l.nn[2] + z;
    double t[N ? N : 1];
    if constexpr (N > 0) {
#pragma unroll
        for (int j = 0; j < N; ++j) t[j] = T[(size_t)j * l.nn[2]];
    }
    const int k1 = min((c + 1) * l.b[1], p.ns[1]);
    for (int k = c * l.b[1]; k < k1; ++k) {
        const double* w = p.s[1] + (size_t)k * n;
        double s = 0.0;
        if constexpr (N > 0) {
#pragma unroll
            for (int j = 0; j < N; ++j) s = fma(w[j], t[j], s);
        } else {
            for (int j = 0; j < n; ++j) s = fma(w[j], T[(size_t)j * l.nn[2]], s);
        }
        U[(size_t)k * l.nn[2]] = s;
    }
}

// node positions per axis and the workspace a plan needs; with base, its pointers
size_t far_layout(FarPlan& p, char* base) {
    size_t o = 0;
    auto take = [&](size_t bytes) {
        char* q = base ? base + o : nullptr;
        o += (bytes + 255) & ~(size_t)255;
        return q;
    };
    for (int i = 0; i < p.levels; ++i) {
        FarLevel& l = p.lv[i];
        l.cx = (int2*)take(sizeof(int2) * l.nc[0]);
        l.cy = (int2*)take(sizeof(int2) * l.nc[1]);
        for (int a = 0; a < 3; ++a) l.pos[a] = (double*)take(sizeof(double) * l.nn[a]);
        for (int a = 0; a < 3; ++a) l.w[a] = (double*)take(sizeof(double) * (size_t)l.nn[a] * p.nodes[a]);
        l.T = (double*)take(sizeof(double) * (size_t)p.C * l.nn[0] * l.nn[1] * l.nn[2]);
    }
    for (int a = 0; a < 3; ++a) p.s[a] = (double*)take(sizeof(double) * (size_t)p.ns[a] * p.nodes[a]);
    p.U = (double*)take(sizeof(double) * (size_t)p.C * p.lv[0].nn[0] * p.ns[1] * p.lv[0].nn[2]);
    return o;
}

}  // namespace

FarPlan far_plan(const gwn_mesh_s* m, const GridArgs& ga, int prec, int C) {
    FarPlan none;
    const long long N[3] = {ga.nx, ga.ny, ga.nz};
    // Expected time in seconds.  Chained vertices per second, measured: all chunks 3.0e12
    // (FP64 8.3e11), near chunks alone 2.4e12 (8e11; their edges look wider), node columns
    // 2.1e12 (9e11); interpolation per sample and node value; launches.
    // The gradient's rates likewise, for its three sums together.
    const bool f32 = prec != GWN_PREC_FP64;
    const double rate = f32 ? 3.0e12 : 0.83e12, near_rate = f32 ? 2.4e12 : 0.8e12, node_rate = f32 ? 2.1e12 : 0.9e12;
    const double B = (double)m->nchunk * kChunk * (C == 3 ? 1.3 : 1.0), all = (double)N[0] * N[1] * N[2];
    auto padded = [](double z) { return std::ceil(z / 64.0) * 64.0; };
    const double columns = (double)N[0] * N[1] * padded((double)N[2]), direct = columns * B / rate;
    none.cost = direct;
    // GWN_GRID_FAR: 0 never; 8 to 96 blocks of that many samples wherever the form allows
    int forced = 0;
    if (const char* e = std::getenv("GWN_GRID_FAR")) {
        forced = std::atoi(e);
        if (forced <= 0) return none;
    }
    const int n = f32 ? 10 : 16;
    if (m->nchunk < 1) return none;
    // every sample inside the fixed-point box in x and y, and no farther than its
    // size in z; rising or falling coordinates
    double step[3];   // cells per sample
    const double scale = m->g.scale;
    for (int a = 0; a < 3; ++a) {
        const double p0 = ((ga.o[a] + 0.5 * ga.s[a]) - m->g.lo[a]) * scale;
        const double p1 = ((ga.o[a] + ((double)N[a] + 0.5) * ga.s[a]) - m->g.lo[a]) * scale;   // one past the last
        step[a] = std::fabs(ga.s[a]) * scale;
        const double lo = a < 2 ? 0x1p20 : -0x1p30, hi = a < 2 ? (double)kQMax - 0x1p20 : 0x1p31;
        if (!(p0 >= lo && p0 <= hi && p1 >= lo && p1 <= hi)) return none;
        if (N[a] > 1 && !(step[a] >= 0x1p14)) return none;
        // distinct FP32 node positions: a step of at least 2^8 ulps of the largest coordinate
        if ((a == 2 || C == 3) && N[a] > 1 && !(step[a] >= 0x1p-15 * scale * std::max(std::fabs(ga.o[a]), std::fabs(ga.o[a] + (double)N[a] * ga.s[a]))))
            return none;
    }
    // the gradient's offsets in units of 2^18 cells, no other scale (far_scale)
    if (C == 3)
        for (int a = 0; a < 3; ++a)
            if (!(scale * std::max(std::fabs(ga.o[a]), std::fabs(ga.o[a] + ((double)N[a] + 1.0) * ga.s[a])) <= 0x1p39)) return none;
    double ext[2];   // the boundary's x and y extent is taken for the mesh's
    for (int a = 0; a < 2; ++a) ext[a] = std::max((m->bbox[3 + a] - m->bbox[a]) * scale, 1.0);

    FarPlan best, p;
    for (int j = 0; j < n; ++j) p.t[j] = -std::cos((2 * j + 1) * M_PI / (2 * n));
    p.C = C;
    for (int a = 0; a < 3; ++a) {
        p.ns[a] = (int)N[a];
        p.nodes[a] = (int)std::min<long long>(n, N[a]);
    }
    double smin = 0.0;   // finest step of the axes that have more samples than nodes
    for (int a = 0; a < 3; ++a)
        if (N[a] > n) smin = smin > 0.0 ? std::min(smin, step[a]) : step[a];
    if (!(smin > 0.0)) return none;
    double cost = forced > 0 ? 1e30 : 0.9 * direct;
    for (int bs : {8, 10, 12, 14, 16, 20, 24, 28, 32, 40, 48, 56, 64, 80, 96}) {
        if (forced > 0) bs = forced;
        const double h = bs * smin;
        FarPlan q = p;
        q.levels = 0;
        double near_up = 1.0, t = 2e-5;
        double nodes_t = 0.0;
        // levels from fine to coarse until a level's blocks span the grid
        for (int l = 0; l < kFarLevels; ++l) {
            FarLevel& v = q.lv[l];
            double half = 0.0;
            bool one = true;
            for (int a = 0; a < 3; ++a) {
                long long b = l == 0 ? std::max<long long>(8, (long long)std::llround(h / step[a])) : 2ll * q.lv[l - 1].b[a];
                if (N[a] <= n) b = N[a];
                v.b[a] = (int)b;
                v.nc[a] = (int)((N[a] + b - 1) / b);
                v.nn[a] = v.nc[a] * q.nodes[a];
                if (N[a] > n) half = std::max(half, 0.5 * (double)far_range(q, v, a, 0).last * step[a]);
                one &= v.nc[a] == 1;
            }
            const double thr = std::ceil((f32 ? kFarKappa32 : kFarKappa64) * half) + 4.0;
            if (!(thr < 0x1p30)) break;
            v.thr = (int)thr;
            q.levels = l + 1;
            if (one) break;
        }
        if (q.levels == 0) continue;
        // expected share of the boundary near a block, averaged over the blocks
        auto share = [&](const FarLevel& v) {
            double f = 1.0;
            for (int a = 0; a < 2; ++a) {
                const double len = (double)N[a] * step[a], w = std::min((double)v.b[a] * step[a], len), reach = (double)v.thr + 0.5 * m->chunk_w;
                // blocks over the grid's length; the boundary over ext in its middle
                double s = 0.0;
                for (int c = 0; c < v.nc[a]; ++c) {
                    const double lo = std::max((double)c * w - reach, 0.5 * (len - ext[a]));
                    const double hi = std::min((double)(c + 1) * w + reach, 0.5 * (len + ext[a]));
                    s += std::min(1.0, std::max(0.0, hi - lo) / ext[a]);
                }
                f *= s / v.nc[a];
            }
            return f;
        };
        double sh[kFarLevels];
        for (int l = 0; l < q.levels; ++l) sh[l] = share(q.lv[l]);
        // drop coarse levels that would hold less than a tenth of the boundary
        while (q.levels > 1 && sh[q.levels - 1] > 0.9) --q.levels;
        for (int l = 0; l < q.levels; ++l) {
            const FarLevel& v = q.lv[l];
            near_up = l + 1 < q.levels ? sh[l + 1] : 1.0;
            const double nv = (double)v.nn[0] * v.nn[1] * padded((double)v.nn[2]);
            // a launch of few columns takes as long as one of its columns
            nodes_t += nv * B * (near_up - sh[l]) / node_rate + 2e-5;
            nodes_t += C * (double)v.nn[0] * v.nn[1] * v.nn[2] * 2e-11;
        }
        t += nodes_t + sh[0] * columns * B / near_rate + C * all * 2e-11 + C * (double)q.lv[0].nn[0] * N[1] * q.lv[0].nn[2] * 6e-12;
        if (far_layout(q, nullptr) > kFarMaxBytes) continue;
        if (t < cost) {
            cost = t;
            best = q;
            best.cost = t;
        }
    }
    if (best.levels == 0) return none;
    best.bytes = far_layout(best, nullptr);
    return best;
}

gwn_status far_setup(FarPlan& p, const gwn_mesh_s* m, const GridArgs& ga, int prec, void* ws, hipStream_t st) {
    far_layout(p, (char*)ws);
    const bool f32 = prec != GWN_PREC_FP64;
    int nc = 1, nt = 1;
    for (int a = 0; a < 3; ++a) {
        nc = std::max(nc, p.lv[0].nc[a]);
        nt = std::max({nt, p.lv[0].nn[a], p.ns[a]});
    }
    k_far_nodes<<<dim3((nc + 63) / 64, 3, p.levels), 64, 0, st>>>(p, ga, m->g, f32);
    GWN_HIP_TRY(hipGetLastError());
    k_far_weights<<<dim3((nt + 63) / 64, 3, p.levels), 64, 0, st>>>(p, ga, m->g, f32);
    GWN_HIP_TRY(hipGetLastError());
    return GWN_OK;
}

gwn_status far_transfer(const FarPlan& p, hipStream_t st) {
    const size_t lds = sizeof(double) * 2 * p.nodes[0] * p.nodes[1] * p.nodes[2];
    for (int v = 0; v < p.C; ++v) {
        for (int l = p.levels - 2; l >= 0; --l) {
            const FarLevel& f = p.lv[l];
            k_far_down<<<(unsigned)((long long)f.nc[0] * f.nc[1] * f.nc[2]), 256, lds, st>>>(p, l, v);
            GWN_HIP_TRY(hipGetLastError());
        }
        const FarLevel& f = p.lv[0];
        const unsigned blocks = (unsigned)(((long long)f.nn[0] * f.nc[1] * f.nn[2] + 255) / 256);
        if (p.nodes[1] == 10) k_far_y<10><<<blocks, 256, 0, st>>>(p, v);
        else if (p.nodes[1] == 16) k_far_y<16><<<blocks, 256, 0, st>>>(p, v);
        else k_far_y<0><<<blocks, 256, 0, st>>>(p, v);
        GWN_HIP_TRY(hipGetLastError());
    }
    return GWN_OK;
}

}  // namespace gwn

extern "C" int64_t gwn_test_far_plan(const double* bbox, int64_t nchunk, double chunk_w, const double* origin,
                                     const double* spacing, const int64_t* dims, int32_t prec, int32_t values,
                                     int64_t* out, int64_t cap) {
    gwn_mesh_s m;
    std::copy(bbox, bbox + 6, m.bbox);
    m.g = gwn::make_qgrid(bbox);
    m.nchunk = nchunk;
    m.chunk_w = chunk_w;
    const gwn::FarPlan p = gwn::far_plan(&m, gwn::frame_grid(0, origin, spacing, dims), prec, values);
    int64_t n = 0;
    auto put = [&](int64_t v) {
        if (n < cap) out[n] = v;
        ++n;
    };
    put(p.levels);
    for (int l = 0; l < p.levels; ++l) {
        put(p.lv[l].thr);
        for (int a = 0; a < 2; ++a) {
            put(p.lv[l].nc[a]);
            for (int c = 0; c < p.lv[l].nc[a]; ++c) {
                const gwn::FarRange r = gwn::far_range(p, p.lv[l], a, c);
                put(r.first);
                put(r.last);
            }
        }
    }
    return n <= cap ? n : -1;
}

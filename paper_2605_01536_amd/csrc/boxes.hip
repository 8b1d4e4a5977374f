// boxes.hip -- w on grids of few samples against a ragged boundary, where sharing a
// column's x/y work among its samples (grid.hip) saves less than sharing the boundary's far
// clusters among a box of them.  Built apart from grid.hip, whose scheduler costs the point
// routines a third of their resident waves.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdlib>

#include <algorithm>

#include "../../include/gwn_test.h"
#include "gwn_far.h"
#include "gwn_kernels.h"
#include "gwn_mesh.h"

namespace gwn {
namespace {

// A workgroup of PARTS waves takes a box of 64 samples, one per lane, and walks the
// clusters that serve scattered points (point_clusters): the samples of a box have the same
// clusters near and far, and the waves share the top level out.  A sample's w has the bits
// of a query at its position.
//
// Bound by VALU issue of expansions and near edges, as the points are; few boxes by the
// chain of clusters that a wave walks, hence more waves per box for fewer boxes (us at 16,
// 8, 4 waves: 125 boxes 399, 462, 610; 1,040 boxes 974, 666, 604; 4,096 boxes 3033, 1828,
// 1191, all on a torus of loops of 25 k edges).  The box is the nearest to a cube that the
// spacing and the grid allow (20 x 150 x 30 samples over a cube, us: 4 x 4 x 4 703, 2 x 16 x 2
// 548).
struct Boxes {
    int l[3];   // log2 of a box's samples along each axis, 6 in all
    int n[3];   // boxes along each axis
};

template <int PARTS>
__global__ __launch_bounds__(64 * PARTS) void k_grid_boxes(MeshView mv, GridArgs ga, Boxes nb, int box0,
                                                           ColCrossings cc, int* __restrict__ chi_out,
                                                           float* __restrict__ w) {
    __shared__ int stack[kLdsStack * kChiBlock];
    __shared__ double part[PARTS][64];
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    int lane = threadIdx.x & 63;
    // the lane's sample; beyond the grid's end the last one
    const int box = box0 + (int)blockIdx.x;
    const int bz = box % nb.n[2], bxy = box / nb.n[2], bx = bxy / nb.n[1], by = bxy - bx * nb.n[1];
    auto sample = [&](int& i, int& j, int& k) {
        i = (bx << nb.l[0]) + (lane >> (nb.l[1] + nb.l[2]));
        j = (by << nb.l[1]) + ((lane >> nb.l[2]) & ((1 << nb.l[1]) - 1));
        k = (bz << nb.l[2]) + (lane & ((1 << nb.l[2]) - 1));
        const bool in = i < ga.nx && j < ga.ny && k < ga.nz;
        i = min(i, (int)ga.nx - 1);
        j = min(j, (int)ga.ny - 1);
        k = min(k, (int)ga.nz - 1);
        return in;
    };
    int i, j, k;
    sample(i, j, k);
    const float px = grid_coord(ga.o[0], ga.s[0], i), py = grid_coord(ga.o[1], ga.s[1], j),
                pz = grid_coord(ga.o[2], ga.s[2], k);
    const QPoint q = quantize_point(px, py, pz, mv.g);
    const int unit = point_unit(px, py, pz, q.inbox, mv.g);
    double S = 0.0;
    if (!q.inbox) {
        outside_sum<float>(mv, px, py, pz, wave, PARTS, unit, S);
    } else {
        const float sc = mv.g.scalef;
        S = point_clusters(mv, {q.x, q.y, px * sc, py * sc, pz * sc, quad_z(pz, mv.g), unit}, wave, PARTS);
    }
    part[wave][lane] = S;
    __syncthreads();
    if (wave > 0) return;
    for (int v = 1; v < PARTS; ++v) S += part[v][lane];

    // the sample's place again rather than kept through the sum
    asm volatile("" : "+v"(lane));
    const bool in = sample(i, j, k);
    int chi = 0;
    if (q.inbox) {
        const long long col = (long long)i * ga.ny + j;
        const int nc = cc.count ? cc.count[col] : kCrossings + 1;
        if (nc <= kCrossings) {
            for (int c = 0; c < nc; ++c) {
                const int x = cc.list[c * cc.ncols + col];
                chi += k < (x >> 1) ? (x & 1) ? -1 : 1 : 0;
            }
        } else {
            chi = chi_up(mv, quantize_point(grid_coord(ga.o[0], ga.s[0], i), grid_coord(ga.o[1], ga.s[1], j),
                                            grid_coord(ga.o[2], ga.s[2], k), mv.g), stack + lane);
        }
    }
    if (!in) return;
    const long long o = (long long)i * ga.st[0] + (long long)j * ga.st[1] + (long long)k * ga.st[2];
    if (chi_out) chi_out[o] = chi;
    w[o] = (float)((double)chi + point_total<float>(S, unit) * kInv2Pi);
}

// The box nearest to a cube: its shortest side doubled six times, no side beyond the grid's.
Boxes box_shape(const GridArgs& ga) {
    const long long N[3] = {ga.nx, ga.ny, ga.nz};
    Boxes b{};
    for (int k = 0; k < 6; ++k) {
        int best = -1;
        double len = 0.0;
        for (int a = 0; a < 3; ++a) {
            const double side = std::fabs(ga.s[a]) * (double)(1 << b.l[a]);
            if ((1ll << b.l[a]) < N[a] && (best < 0 || side < len)) {
                best = a;
                len = side;
            }
        }
        ++b.l[best < 0 ? 0 : best];
    }
    for (int a = 0; a < 3; ++a) b.n[a] = (int)((N[a] + (1 << b.l[a]) - 1) >> b.l[a]);
    return b;
}

int box_waves(long long boxes) { return boxes <= 256 ? 16 : boxes <= 1024 ? 8 : 4; }

}  // namespace

// By the expected time, on meshes of short loops (at most 8 edges on average: clusters of
// few long loops are near most boxes; 64 loops of 160 edges: 37 x 50 x 29 samples 1.1 ms in
// boxes, 0.7 in columns).  Boxes: per sample the far clusters, whose number goes with
// the root of the edges' number B until the levels of the tree take over, and the edges
// near the box, which go with B times the square of its side over the mesh's until most are
// near; and a wave's walk.  Columns: far_plan's estimate with what it leaves out, the part
// of a column's wave that does not go with the boundary, and a column's length where there
// are few; 15% less with a far part, whose estimate is the looser one.  Measured, us, columns / boxes: B = 1,001 (ellipsoids) 37 x 50 x 29
// 124 / 98, 64^3 254 / 217, 100^3 634 / 614, 130^3 949 / 1342; B = 2,538 (torus) 20^3 88 / 97,
// 64^3 524 / 371, 100^3 929 / 1126; B = 25,229 20^3 517 / 399, 64^3 3720 / 1191, 100^3 5735 /
// 3264, 160^3 9143 / 11738; B = 53,776 (ellipsoids) 64^3 7668 / 1473,
// 160^3 27478 / 12323, slices 512 x 512 x 1 29489 / 1191, 1 x 256 x 256 1236 / 636.
// GWN_GRID_BOXES: 0 never, 1 wherever the mesh has clusters; a choice of column form
// by GWN_GRID_FAR or GWN_GRID_SAMPLES_PER_LANE is a choice of columns, as is the tuner's
// timing of the samples per lane (columns_only).
bool want_boxes(const gwn_mesh_s* m, const GridArgs& ga, const FarPlan& p, long long* boxes) {
    const Boxes b = box_shape(ga);
    const long long N[3] = {ga.nx, ga.ny, ga.nz};
    double n = 1.0, side = 0.0, ext = 0.0;
    for (int a = 0; a < 3; ++a) {
        const double h = N[a] > 1 ? (double)(1 << b.l[a]) * ga.s[a] : 0.0;
        n *= (double)b.n[a];
        side += h * h;
        ext += (m->bbox[3 + a] - m->bbox[a]) * (m->bbox[3 + a] - m->bbox[a]);
    }
    if (m->nclusters < kFewClusters || !(n < 0x1p31)) return false;
    *boxes = (long long)n;
    if (const char* e = std::getenv("GWN_GRID_BOXES")) return std::atoi(e) != 0;
    if (std::getenv("GWN_GRID_FAR") || std::getenv("GWN_GRID_SAMPLES_PER_LANE") || m->columns_only) return false;
    if (m->nb > 8 * m->nloops) return false;
    const double B = (double)m->nb, x = B * side / ext;
    const double share = std::min(2.4, 0.018 * std::sqrt(B)) + 0.02 * x / (1.0 + x / 400.0);   // ns
    const double t = 64e-9 * n * share + 1e-6 * std::sqrt(B);
    const double waves = (double)ga.nx * (double)ga.ny * std::ceil((double)ga.nz / 64.0);
    const double columns = p.levels > 0 ? 0.85 * p.cost : std::max(1.4 * p.cost, 1.4e-8 * B);
    return t < columns + 2e-9 * waves + 2.5e-5;
}

gwn_status launch_boxes(const gwn_mesh_s* m, const GridArgs& ga, long long boxes, const ColCrossings& cc, float* w,
                        int32_t* chi_out, hipStream_t st) {
    const Boxes nb = box_shape(ga);
    const int parts = box_waves(boxes);
    hipError_t e = hipSuccess;
    launch_slices(boxes, 64 * parts, [&](int64_t b, int64_t n) {   // 1,021^3 samples: 2^32 work-items and more
        auto go = [&](auto kernel) { kernel<<<(unsigned)n, 64 * parts, 0, st>>>(m->view(), ga, nb, (int)b, cc, chi_out, w); };
        if (parts == 16) go(k_grid_boxes<16>);
        else if (parts == 8) go(k_grid_boxes<8>);
        else go(k_grid_boxes<4>);
        if (e == hipSuccess) e = hipGetLastError();
    });
    GWN_HIP_TRY(e);
    return GWN_OK;
}

}  // namespace gwn

extern "C" int64_t gwn_test_boxes(const double* bbox, int64_t nchunk, double chunk_w, int64_t nb, int64_t nloops,
                                  int64_t nclusters, const double* origin, const double* spacing, const int64_t* dims,
                                  int64_t* work_items) {
    gwn_mesh_s m;
    std::copy(bbox, bbox + 6, m.bbox);
    m.g = gwn::make_qgrid(bbox);
    m.nchunk = nchunk;
    m.chunk_w = chunk_w;
    m.nb = nb;
    m.nloops = nloops;
    m.nclusters = nclusters;
    const gwn::GridArgs ga = gwn::frame_grid(0, origin, spacing, dims);
    long long boxes = 0;
    *work_items = 0;
    if (!gwn::want_boxes(&m, ga, gwn::far_plan(&m, ga, GWN_PREC_FP32, 1), &boxes)) return 0;
    const int threads = 64 * gwn::box_waves(boxes);
    gwn::launch_slices(boxes, threads, [&](int64_t, int64_t n) { *work_items = std::max(*work_items, n * threads); });
    return boxes;
}

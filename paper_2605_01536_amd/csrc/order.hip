// order.hip -- a traversal order for batches of arbitrary points.
//
// Lanes of one wave that trace nearby vertical lines visit the same BVH nodes.
// Visiting the points in Morton order of their quantised x, y (the ray is
// vertical: z does not matter) lets a wave walk the tree once, uniformly, for
// all its lanes (k_chi_wave).  The boundary sum's clusters depend on z too: there
// the points are taken along a Hilbert curve.  The order only permutes which lane handles which
// point; every result is written to the point's own slot.
#include <cstdlib>

#include "gwn_alloc.h"
#include "gwn_internal.h"
#include "gwn_mesh.h"
#include "gwn_sort.h"

namespace gwn {
namespace {

__global__ void k_order_keys(const float* __restrict__ qx, const float* __restrict__ qy, const float* __restrict__ qz,
                             long long qs, long long n, QGrid g, bool space, uint32_t* __restrict__ key,
                             int* __restrict__ idx) {
    const long long i = blockIdx.x * 256ll + threadIdx.x;
    if (i >= n) return;
    key[i] = point_key(quantize_point(qx[i * qs], qy[i * qs], qz[i * qs], g), space);
    idx[i] = (int)i;
}

}  // namespace

// Worth it when the points are dense enough that a wave's 64 neighbours in
// Morton order trace nearly the same path: measured on the 1.05M-triangle soup,
// 2^20 random grid points go 3.4x faster, 2^16 (16x sparser) 25% slower.
bool want_xy_order(const gwn_mesh_s* m, int64_t n) {
    if (const char* e = std::getenv("GWN_ORDER_QUERIES")) return std::atoi(e) != 0 && n > 1;
    if (m->order_min != 0) return m->order_min > 0 && n >= m->order_min && n > 1;
    return n >= (1 << 18) && m->nf >= (1 << 15);
}

// The boundary sum with clusters, a point per lane: a wave's lanes should see the same
// clusters as near, or it sums nearly every cluster's chunks (85 k triangles with 63 k
// edges, 8 k points in no order 11.9 ms, 33 k in order 2.7).  The sort is about 25 launches
// (0.1 ms); on few clusters there is nothing to skip, and on few edges little (us in order /
// not: 131 k points on 1,026 edges 529 / 468, on 1,272 404 / 384, 262 k 766 / 797 and 583 / 681;
// 33 k on 3,073 edges 514 / 527, on 7,827 700 / 872).
bool want_space_order(const gwn_mesh_s* m, int64_t n, int prec) {
    if (prec == GWN_PREC_FP64 || m->nclusters < 16 || n < 2) return false;
    if (const char* e = std::getenv("GWN_ORDER_QUERIES")) return std::atoi(e) != 0;
    if (m->order_min != 0) return m->order_min > 0 && n >= m->order_min;
    return n >= 16384 && (double)n * (double)m->nb >= (m->nb < 2048 ? 2.2e8 : 1e8);
}

size_t xy_order_temp_bytes(int64_t n) {
    const size_t keys = (sizeof(uint32_t) * (size_t)n + 255) & ~(size_t)255;
    const size_t idx = (sizeof(int) * (size_t)n + 255) & ~(size_t)255;
    return 2 * keys + idx + sort_temp_bytes(n, 4, true);
}

gwn_status xy_order_into(const gwn_mesh_s* m, const float* qx, const float* qy, const float* qz, int64_t qs, int64_t n,
                         bool space, int* perm, void* temp, hipStream_t st) {
    const size_t keys = (sizeof(uint32_t) * (size_t)n + 255) & ~(size_t)255;
    const size_t idx = (sizeof(int) * (size_t)n + 255) & ~(size_t)255;
    char* p = (char*)temp;
    uint32_t* k0 = (uint32_t*)p;
    uint32_t* k1 = (uint32_t*)(p + keys);
    int* i0 = (int*)(p + 2 * keys);
    void* stmp = p + 2 * keys + idx;
    k_order_keys<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(qx, qy, qz, qs, n, m->g, space, k0, i0);
    GWN_HIP_TRY(hipGetLastError());
    GWN_HIP_TRY(radix_sort_u32(k0, k1, i0, perm, n, 0, space ? 30 : 32, stmp, st));
    return GWN_OK;
}

gwn_status xy_order(const gwn_mesh_s* m, const float* qx, const float* qy, const float* qz, int64_t qs, int64_t n,
                    bool space, int** perm_out, hipStream_t st) {
    *perm_out = nullptr;
    int* perm = nullptr;
    void* tmp = nullptr;
    hipError_t e = gwn::dmalloc_async((void**)&perm, sizeof(int) * (size_t)n, st);
    if (e == hipSuccess) e = gwn::dmalloc_async(&tmp, xy_order_temp_bytes(n), st);
    if (e != hipSuccess) {
        if (perm) (void)hipFreeAsync(perm, st);
        GWN_HIP_TRY(e);
    }
    const gwn_status s = xy_order_into(m, qx, qy, qz, qs, n, space, perm, tmp, st);
    (void)hipFreeAsync(tmp, st);
    if (s != GWN_OK) {
        (void)hipFreeAsync(perm, st);
        return s;
    }
    *perm_out = perm;
    return GWN_OK;
}

}  // namespace gwn

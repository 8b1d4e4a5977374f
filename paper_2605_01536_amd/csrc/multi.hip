// multi.hip -- many meshes with uneven sizes and query counts in one captured
// HIP graph: [reset work counters] -> [crossing counts for every query of every
// mesh] -> [persistent boundary-term kernels].  The persistent kernels keep
// waves resident and hand out (mesh, query tile) work items through an atomic
// counter, largest estimated cost first, so meshes whose cost spans orders of
// magnitude share the GPU without a long tail.  The schedule (tile size, item
// order, resident waves) is chosen by timing candidates (autotune) and can be
// cached in a JSON-lines file keyed by device and problem size.  Meshes with
// many queries take them 64 neighbours to a wave, in orders (index
// permutations) made once at creation from the query values then; the others as
// they come, a few queries per wave or a query per lane (see plan_forms).
#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <string>
#include <vector>

#include "../../include/gwn_test.h"
#include "gwn_alloc.h"
#include "gwn_kernels.h"
#include "gwn_mesh.h"
#include "gwn_sort.h"

namespace gwn {
namespace {

struct alignas(16) Item {
    long long q0;   // first query (global index)
    int mesh;
    int nq;         // queries in this item
};

__global__ void k_reset_counter(int* c) {
    if (threadIdx.x < 2 && blockIdx.x == 0) c[threadIdx.x] = 0;
}

// Crossing counts along +z for every query, one wave per work item: the item's
// queries (in Morton order within their mesh when perm is given, as the
// boundary-term kernel takes them) walk the mesh's BVH together
// (chi_wave_walk), so a wave follows about one path.  Out-of-box queries get 0.
__global__ __launch_bounds__(64 * kGridWaves) void k_chi_items(const MeshView* __restrict__ table,
                                                              const Item* __restrict__ items, int nitems,
                                                              const float* __restrict__ qx,
                                                              const float* __restrict__ qy,
                                                              const float* __restrict__ qz, long long qs,
                                                              const int* __restrict__ perm, int* __restrict__ chi) {
    __shared__ int wstack[kGridWaves][kLdsStack];
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
    const long long it = (long long)blockIdx.x * kGridWaves + wave;
    if (it >= nitems) return;   // the whole wave
    const Item I = items[it];
    const MeshView mv = table[I.mesh];
    const float *x = qx, *y = qy, *z = qz;
    axis_ptrs(mv.axis, x, y, z);   // the mesh's frame
    for (int sub = 0; sub < I.nq; sub += 64) {
        const int k = sub + lane;
        const long long i0 = I.q0 + min(k, I.nq - 1);
        const long long i = perm ? (long long)perm[i0] : i0;
        const QPoint q = quantize_point(x[i * qs], y[i * qs], z[i * qs], mv.g);
        int u, d;
        chi_wave_walk<true>(mv, q, k < I.nq && q.inbox, wstack[wave], u, d);
        if (k < I.nq) chi[i] = u;
    }
}

// the same for queries in no order, a wave per query (chi_up_wave): kChiParts workgroups
// share an item's queries
constexpr int kChiParts = 4;

__global__ __launch_bounds__(64 * kGridWaves) void k_chi_items_point(const MeshView* __restrict__ table,
                                                                    const Item* __restrict__ items, int nitems,
                                                                    const float* __restrict__ qx,
                                                                    const float* __restrict__ qy,
                                                                    const float* __restrict__ qz, long long qs,
                                                                    int* __restrict__ chi) {
    __shared__ ChiLists lists[kGridWaves];
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int it = (int)(blockIdx.x / kChiParts), part = (int)(blockIdx.x % kChiParts) * kGridWaves + wave;
    if (it >= nitems) return;
    const Item I = items[it];
    const MeshView mv = table[I.mesh];
    const float *x = qx, *y = qy, *z = qz;
    axis_ptrs(mv.axis, x, y, z);   // the mesh's frame
    for (int k = part; k < I.nq; k += kChiParts * kGridWaves) {
        const long long i = I.q0 + k;
        const QPoint q = quantize_point(x[i * qs], y[i * qs], z[i * qs], mv.g);
        const int c = q.inbox ? chi_up_wave(mv, q, lists[wave]) : 0;
        if ((threadIdx.x & 63) == 0) chi[i] = c;
    }
}

// the same for queries in no order, a lane per query (chi_up): a workgroup of one wave per 64
// queries, `claims` of them per item
__global__ __launch_bounds__(kChiBlock) void k_chi_items_lane(const MeshView* __restrict__ table,
                                                             const Item* __restrict__ items, int claims,
                                                             const float* __restrict__ qx,
                                                             const float* __restrict__ qy,
                                                             const float* __restrict__ qz, long long qs,
                                                             int* __restrict__ chi) {
    __shared__ int stk[kLdsStack * kChiBlock];
    const Item I = items[blockIdx.x / claims];
    const int k = (int)(blockIdx.x % claims) * kChiBlock + threadIdx.x;
    if (k >= I.nq) return;
    const MeshView mv = table[I.mesh];
    const float *x = qx, *y = qy, *z = qz;
    axis_ptrs(mv.axis, x, y, z);   // the mesh's frame
    const long long i = I.q0 + k;
    const QPoint q = quantize_point(x[i * qs], y[i * qs], z[i * qs], mv.g);
    chi[i] = q.inbox ? chi_up(mv, q, stk + threadIdx.x) : 0;
}

// sort keys of all queries: the mesh, then (items [0, nkeyed)) the query's place in the order
__global__ void k_plan_keys(const MeshView* __restrict__ table, const Item* __restrict__ items, int nkeyed,
                            const float* __restrict__ qx, const float* __restrict__ qy, const float* __restrict__ qz,
                            long long qs, bool space, uint64_t* __restrict__ key, int* __restrict__ idx) {
    const Item I = items[blockIdx.x];   // items, nkeyed: from the launch's first item on
    const QGrid g = table[I.mesh].g;
    const float *x = qx, *y = qy, *z = qz;
    axis_ptrs(table[I.mesh].axis, x, y, z);
    for (int k = threadIdx.x; k < I.nq; k += blockDim.x) {
        const long long i = I.q0 + k;
        uint32_t c = 0;
        if ((int)blockIdx.x < nkeyed) c = point_key(quantize_point(x[i * qs], y[i * qs], z[i * qs], g), space);
        key[i] = ((uint64_t)I.mesh << 32) | c;
        idx[i] = (int)i;
    }
}

// Persistent boundary-term kernel: every wave claims a share of an item at a time, `claims` to
// an item, and takes its queries 64 at once, one per lane, until none are left (the counter
// only grows, so every wave reaches the exit).
// perm (nullable): in items [0, nperm) position i of the work list is query perm[i], a
// permutation within each mesh.  T is the geometry precision; per query the sums have the batch kernels' terms, so
// the results are the same bits.
// The mesh's data are read by scalar loads (see uniform_load): 7.2 ms instead of 10.3 for
// 3.2 M queries on 48 soups; claims of 64 queries instead of 128 shorten the last wave's
// way (a wave's way through the largest soup takes 2.5 ms).  Where queries take little, the
// claims themselves do, some 12 ns each at their one address: there a claim is an item (ITEM; 1 M
// queries on soups of a triangle 301 us at 64 queries a claim, 208 at 128).
template <class T, bool ITEM>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 8 ? 4 : 1))) void k_bdry_persistent(const MeshView* __restrict__ table,
                                                        const Item* __restrict__ items, int nitems, int claims,
                                                        int* __restrict__ counter, const float* __restrict__ qx,
                                                        const float* __restrict__ qy, const float* __restrict__ qz,
                                                        long long qs, const int* __restrict__ perm, int nperm,
                                                        const int* __restrict__ chi, T* __restrict__ w) {
    const int lane = threadIdx.x & 63;
    while (true) {
        int t = 0;
        if (lane == 0) t = atomicAdd(counter, 1);
        t = __builtin_amdgcn_readfirstlane(__shfl(t, 0));
        const int it = ITEM ? t : t / claims, first = ITEM ? 0 : (t - it * claims) * 64;
        if (it >= nitems) break;
        const Item I = uniform_load(items + it);
        if (first >= I.nq) continue;
        const MeshView mv = uniform_load(table + I.mesh);
        const float *x = qx, *y = qy, *z = qz;
        axis_ptrs(mv.axis, x, y, z);   // the mesh's frame
        for (int sub = first; sub < (ITEM ? I.nq : first + 1); sub += 64) {
            const int k = sub + lane;
            const long long i0 = I.q0 + min(k, I.nq - 1);
            const long long i = perm && it < nperm ? (long long)perm[i0] : i0;
            const float px = x[i * qs], py = y[i * qs], pz = z[i * qs];
            const QPoint q = quantize_point(px, py, pz, mv.g);
            const int unit = sizeof(T) == 4 ? point_unit(px, py, pz, q.inbox, mv.g) : 0;
            double S = 0.0;
            if (!q.inbox) {
                outside_sum<T>(mv, px, py, pz, 0, 1, unit, S);
            } else if constexpr (sizeof(T) == 4) {
                const float sc = mv.g.scalef;
                S = point_clusters(mv, {q.x, q.y, px * sc, py * sc, pz * sc, quad_z(pz, mv.g), unit}, 0, 1);
            } else {
                point_chunks<T, true>(mv, 0, mv.nchunk, 1, q.x, q.y, (T)pz * (T)mv.g.scale, quad_z(pz, mv.g), unit, S);
            }
            if (k < I.nq) w[i] = (T)((double)chi[i] + point_total<T>(S, unit) * kInv2Pi);
        }
    }
}

// FP32 boundary term, groups of kPlanGroup queries per wave (see point_group): a wave claims
// kPlanClaim queries of an item at a time.
constexpr int kPlanGroup = 4, kPlanClaim = 16;

__global__ __launch_bounds__(256) void k_group_persistent(const MeshView* __restrict__ table,
                                                         const Item* __restrict__ items, int nitems, int claims,
                                                         int* __restrict__ counter, const float* __restrict__ qx,
                                                         const float* __restrict__ qy, const float* __restrict__ qz,
                                                         long long qs, const int* __restrict__ perm, int stack_ints,
                                                         const int* __restrict__ chi, float* __restrict__ w) {
    __shared__ PointLists<kPlanGroup> lists[4];
    extern __shared__ int stacks[];
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
    while (true) {
        int t = 0;
        if (lane == 0) t = atomicAdd(counter, 1);
        t = __builtin_amdgcn_readfirstlane(__shfl(t, 0));
        const int it = t / claims, k0 = (t - it * claims) * kPlanClaim;
        if (it >= nitems) break;
        const Item I = uniform_load(items + it);
        if (k0 >= I.nq) continue;
        const MeshView mv = uniform_load(table + I.mesh);
        const float *x = qx, *y = qy, *z = qz;
        axis_ptrs(mv.axis, x, y, z);   // the mesh's frame
        for (int k = k0; k < min(I.nq, k0 + kPlanClaim); k += kPlanGroup)
            point_group_out<kPlanGroup>(mv, x, y, z, qs, I.q0 + k, min(kPlanGroup, I.nq - k), perm,
                                        stacks + (size_t)wave * stack_ints, stack_ints, lists[wave], chi, w);
    }
}

// Meshes of at least this many queries take them in orders.  48 soups of 0.5 to 11 k edges,
// queries per soup on average, ms in order against in groups: 67 k 5.9 / 19.6, 34 k 4.4 / 10.0,
// 17 k 4.2 / 5.1, 8 k 4.0 / 2.7, 4 k 3.6 / 1.5.
constexpr long long kDenseQueries = 16384;

// How a mesh's queries are taken, in the order of the items' ranges: crossings by a walk that a
// wave's queries take together, in order or not, by a lane or by a wave per query; FP32 sums by a
// lane per query, ordered or not, or in groups.
enum { kChiOrdered, kChiTogether, kChiLane, kChiPoint, kSumOrdered = 0, kSumLane, kSumGroup };
struct Form {
    int chi, sum;
};

struct Schedule {
    int item_queries = 128;   // multiple of 64
    int waves_per_simd = 8;   // resident persistent waves per SIMD
    int order = 0;            // bit 0: mesh order (else largest cost first); bit 1: queries in Morton order
};

constexpr int kOrderMesh = 1, kOrderSorted = 2;

}  // namespace
}  // namespace gwn

struct gwn_multi_s {
    int device = 0;
    int nmesh = 0;
    long long nq = 0;
    double est_pairs = 0.0;
    gwn::Schedule sched;
    bool tuned = false;
    double tuned_ms = 0.0;
    std::vector<gwn_mesh_s*> meshes;
    std::vector<long long> qoff_h;
    const float *qx = nullptr, *qy = nullptr, *qz = nullptr;
    long long qs = 1;
    int prec = GWN_PREC_FP32;
    void* w = nullptr;   // float (GWN_PREC_FP32) or double (GWN_PREC_FP64)
    int* chi = nullptr;
    bool own_chi = false;
    gwn::MeshView* table = nullptr;
    std::vector<gwn::Form> forms;   // per mesh
    // the work items twice: by the form of their crossings, and of their sums; and where each
    // form's items end
    gwn::Item *citems = nullptr, *items = nullptr;
    int nitems = 0;
    int cend[4] = {}, send[3] = {};
    // each mesh's queries in an order: Morton order of x and y (for the crossing walk, and what a
    // schedule asks for), and a space-filling curve's (FP32 boundary term)
    int *perm = nullptr, *sperm = nullptr;
    int sorted = 0;           // perm holds: 0 nothing, 1 the ordered meshes' queries, 2 all
    int* counter = nullptr;   // two
    int grid = 0;
    hipStream_t cap = nullptr;
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
};

namespace gwn {
namespace {

void drop_graph(gwn_multi_s* p) {
    if (p->exec) (void)hipGraphExecDestroy(p->exec);
    if (p->graph) (void)hipGraphDestroy(p->graph);
    p->exec = nullptr;
    p->graph = nullptr;
}

void release(gwn_multi_s* p) {
    if (!p) return;
    drop_graph(p);
    if (p->cap) (void)hipStreamDestroy(p->cap);
    (void)hipFree(p->table);
    (void)hipFree(p->citems);
    (void)hipFree(p->items);
    (void)hipFree(p->perm);
    (void)hipFree(p->sperm);
    (void)hipFree(p->counter);
    if (p->own_chi) (void)hipFree(p->chi);
    delete p;
}

// The forms by expected time.
//
// Meshes with at least kDenseQueries queries take them in order, 64 neighbours to a wave, for
// the crossing walk and the boundary term; with fewer than 64 triangles or 32 boundary edges
// there is less to share than reading through the order costs (64 x 20,000 queries on a
// triangle 231 us, in order 377; on 320 closed triangles 479 in order, 990 without, 1,107 if the
// queries are not those that the order was made from).
//
// The others' queries lie too far apart for an order.  Crossings by a wave per query, or, on
// closed meshes and on few triangles, by a lane where queries enough, over all such meshes, hide
// its longer way (us, waves / lanes at 64 k, 256 k and 800 k queries on meshes of 320 closed triangles 87 /
// 81, 296 / 158, 882 / 416; 5,120 closed 121 / 134, 400 / 243, 1,164 / 649; 1,329 of four open
// spheres 95 / 195, 287 / 300, 829 / 684; 3,434 of soups 102 / 217, 318 / 393, 904 / 944; 35,000
// 132 / 331, 384 / 611, 1,090 / 1,379).
//
// FP32 sums in groups of queries or by a lane per query, the boundaries of least edges first,
// as many as the expected time asks for.  A lane takes 0.25 us per edge, and with work
// enough 1.2 ps per edge and query; a group 3.5 us sqrt(edges), and 0.1 ns sqrt(edges) a query.
// Groups / lanes, us: 16 k queries on boundaries of 61 edges 43 / 29, of 216 73 / 69, of 1,046
// 175 / 281, of 3,036 285 / 721, of 10,660 459 / 2,654; 256 k 315 / 115, 440 / 164, 1,100 / 552,
// 1,913 / 1,366, 2,801 / 3,880.  (Queries in order come before a lane's, the smallest boundaries
// last, and hide little of a lane's way.)
std::vector<Form> plan_forms(const std::vector<gwn_mesh_s*>& meshes, const std::vector<long long>& off) {
    const int n = (int)meshes.size();
    const bool order = off[n] <= 0x7fffffffll;   // the permutations hold 32-bit indices
    auto queries = [&](int m) { return off[m + 1] - off[m]; };
    auto edges = [&](int m) { return (double)meshes[m]->nb; };
    auto lane = [&](int m) { return (double)queries(m) * (0.18e-9 + 1.2e-12 * edges(m)); };
    auto group = [&](int m) { return (double)queries(m) * (0.5e-9 + 0.1e-9 * std::sqrt(edges(m))); };
    auto walks = [&](int m) { return meshes[m]->nb == 0 ? 4 : meshes[m]->nf < 2048 ? 1 : 0; };
    std::vector<Form> f(n);
    std::vector<int> loose;    // whose sums a lane or a group may take
    long long walked = 0;      // queries that a lane may walk for, closed meshes' four times
    double lanes = 0.0, groups = 0.0;   // seconds
    for (int m = 0; m < n; ++m) {
        const bool dense = order && queries(m) >= kDenseQueries;
        f[m].chi = meshes[m]->nf < 64 ? kChiTogether : dense ? kChiOrdered : kChiLane;
        f[m].sum = dense && meshes[m]->nb >= 32 ? kSumOrdered : kSumLane;
        if (f[m].chi == kChiLane) walked += walks(m) * queries(m);
        if (f[m].sum == kSumOrdered) continue;
        if (meshes[m]->wide_edges()) lanes += lane(m);
        else if (queries(m) > 0) {
            loose.push_back(m);
            groups += group(m);
        }
    }
    for (int m = 0; m < n; ++m)
        if (f[m].chi == kChiLane && (walked <= 1 << 18 || walks(m) == 0)) f[m].chi = kChiPoint;
    std::stable_sort(loose.begin(), loose.end(), [&](int a, int b) { return edges(a) < edges(b); });
    size_t best = 0;
    double least = INFINITY;
    for (size_t k = 0; k <= loose.size(); ++k) {   // the first k by lanes
        if (k > 0) {
            lanes += lane(loose[k - 1]);
            groups -= group(loose[k - 1]);
        }
        const double way = k > 0 ? 0.25e-6 * edges(loose[k - 1]) : 0.0;
        const double t = std::max(lanes, way) + (k < loose.size() ? groups + 3.5e-6 * std::sqrt(edges(loose.back())) : 0.0);
        if (t < least) {
            least = t;
            best = k;
        }
    }
    for (size_t k = best; k < loose.size(); ++k) f[loose[k]].sum = kSumGroup;
    return f;
}

// work-items per item; 2^31 queries in items of 128 at 1,024 each exceed a launch's 2^32
constexpr int kKeyThreads = 128, kWalkThreads = 64, kPointThreads = kChiParts * 64 * kGridWaves;   // (a lane per query: its queries)

// Work list for a schedule: tiles of item_queries queries, ordered by estimated
// cost (queries x (boundary edges + a traversal allowance)) or by mesh.
gwn_status build_items(gwn_multi_s* p, const Schedule& s, hipStream_t st) {
    std::vector<Item> h;
    std::vector<double> cost;
    for (int m = 0; m < p->nmesh; ++m) {
        const long long q0 = p->qoff_h[m], q1 = p->qoff_h[m + 1];
        const double per_q = (double)p->meshes[m]->nb + 16.0;
        for (long long a = q0; a < q1; a += s.item_queries) {
            Item it;
            it.q0 = a;
            it.mesh = m;
            it.nq = (int)std::min<long long>(s.item_queries, q1 - a);
            h.push_back(it);
            cost.push_back(per_q * it.nq);
        }
    }
    if (!(s.order & kOrderMesh)) {
        std::vector<size_t> idx(h.size());
        for (size_t i = 0; i < idx.size(); ++i) idx[i] = i;
        std::stable_sort(idx.begin(), idx.end(), [&](size_t a, size_t b) { return cost[a] > cost[b]; });
        std::vector<Item> s2(h.size());
        for (size_t i = 0; i < idx.size(); ++i) s2[i] = h[idx[i]];
        h.swap(s2);
    }
    (void)hipFree(p->items);
    (void)hipFree(p->citems);
    p->items = p->citems = nullptr;
    p->nitems = (int)h.size();
    std::vector<Item> c(h);
    auto by_form = [&](std::vector<Item>& v, int Form::*which, int n, int* end) {
        auto it = v.begin();
        for (int k = 0; k < n; ++k) {
            it = std::stable_partition(it, v.end(), [&](const Item& i) { return p->forms[i.mesh].*which == k; });
            end[k] = (int)(it - v.begin());
        }
    };
    by_form(h, &Form::sum, 3, p->send);
    by_form(c, &Form::chi, 4, p->cend);
    const size_t bytes = sizeof(Item) * std::max<size_t>(1, h.size());
    GWN_HIP_TRY(gwn::dmalloc((void**)&p->items, bytes));
    GWN_HIP_TRY(gwn::dmalloc((void**)&p->citems, bytes));
    if (!h.empty()) {
        GWN_HIP_TRY(hipMemcpyAsync(p->items, h.data(), sizeof(Item) * h.size(), hipMemcpyHostToDevice, st));
        GWN_HIP_TRY(hipMemcpyAsync(p->citems, c.data(), sizeof(Item) * c.size(), hipMemcpyHostToDevice, st));
    }
    GWN_HIP_TRY(hipStreamSynchronize(st));
    return GWN_OK;
}

// Each mesh's queries in Morton order of their quantised x, y in the mesh's frame, or along
// the space-filling curve (the batch path's traversal orders), as one permutation of all
// queries; keyed: the first items that take an order, the others' queries stay as they are.
// One sort for all meshes: with a sort each, 48 meshes of 67 k queries took 10 ms per order.
gwn_status build_perm(gwn_multi_s* p, bool space, const Item* items, int keyed, int** perm, hipStream_t st) {
    const int64_t n = p->nq;
    if (n <= 0) return GWN_OK;
    if (!*perm) GWN_HIP_TRY(gwn::dmalloc((void**)perm, sizeof(int) * (size_t)n));
    int bits = 32;
    while ((1ll << (bits - 32)) < p->nmesh) ++bits;
    const size_t kb = ((size_t)n * 8 + 255) & ~(size_t)255, ib = ((size_t)n * 4 + 255) & ~(size_t)255;
    unsigned char* tmp = nullptr;
    GWN_HIP_TRY(gwn::dmalloc((void**)&tmp, 2 * kb + ib + sort_temp_bytes(n, 8, true)));
    uint64_t *k0 = (uint64_t*)tmp, *k1 = (uint64_t*)(tmp + kb);
    int* i0 = (int*)(tmp + 2 * kb);
    hipError_t e = hipSuccess;
    launch_slices(p->nitems, kKeyThreads, [&](int64_t i, int64_t ni) {
        k_plan_keys<<<(unsigned)ni, kKeyThreads, 0, st>>>(p->table, items + i, (int)(keyed - i), p->qx, p->qy, p->qz, p->qs,
                                                         space, k0, i0);
        if (e == hipSuccess) e = hipGetLastError();
    });
    if (e == hipSuccess) e = radix_sort_u64(k0, k1, i0, *perm, n, 0, bits, tmp + 2 * kb + ib, st);
    const hipError_t e2 = hipStreamSynchronize(st);
    (void)hipFree(tmp);
    GWN_HIP_TRY(e);
    GWN_HIP_TRY(e2);
    return GWN_OK;
}

gwn_status capture(gwn_multi_s* p, const Schedule& s) {
    drop_graph(p);
    int ncu = 0;
    GWN_HIP_TRY(hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, p->device));
    const long long waves = (long long)ncu * 4 * s.waves_per_simd;
    const int claims = (s.item_queries + kPlanClaim - 1) / kPlanClaim, lanes = (s.item_queries + 63) / 64;
    const bool f32 = p->prec != GWN_PREC_FP64;
    const int nlane = f32 ? p->send[kSumLane] : p->nitems, ngroup = p->nitems - nlane;
    double edges = 0.0, queries = 0.0;   // of the lanes' items
    for (int m = 0; m < p->nmesh; ++m)
        if (!f32 || p->forms[m].sum != kSumGroup) {
            queries += (double)(p->qoff_h[m + 1] - p->qoff_h[m]);
            edges += (double)(p->qoff_h[m + 1] - p->qoff_h[m]) * (double)p->meshes[m]->nb;
        }
    // claims per item
    const int sums = edges < 256.0 * queries && (long long)nlane * lanes > waves ? 1 : lanes;
    // no more waves than claims
    const long long need = std::max((long long)nlane * sums, (long long)ngroup * claims) / 4 + 1;
    p->grid = (int)std::max<long long>(1, std::min<long long>(waves / 4, need));
    GWN_HIP_TRY(hipStreamBeginCapture(p->cap, hipStreamCaptureModeThreadLocal));
    hipError_t le = hipSuccess;   // of the first launch that was refused
    auto launched = [&] {
        const hipError_t e = hipGetLastError();
        if (le == hipSuccess) le = e;
    };
    k_reset_counter<<<1, 64, 0, p->cap>>>(p->counter);
    launched();
    if (p->nq > 0) {
        const int* c = p->cend;
        auto walk = [&](int first, int end, const int* perm) {
            launch_slices(end - first, kWalkThreads, [&](int64_t i, int64_t n) {
                k_chi_items<<<(unsigned)((n + kGridWaves - 1) / kGridWaves), 64 * kGridWaves, 0, p->cap>>>(
                    p->table, p->citems + first + i, (int)n, p->qx, p->qy, p->qz, p->qs, perm, p->chi);
                launched();
            });
        };
        walk(0, c[kChiOrdered], p->perm);
        walk(c[kChiOrdered], c[kChiTogether], nullptr);
        launch_slices(c[kChiLane] - c[kChiTogether], lanes * kChiBlock, [&](int64_t i, int64_t n) {
            k_chi_items_lane<<<(unsigned)(n * lanes), kChiBlock, 0, p->cap>>>(p->table, p->citems + c[kChiTogether] + i, lanes,
                                                                              p->qx, p->qy, p->qz, p->qs, p->chi);
            launched();
        });
        launch_slices(p->nitems - c[kChiLane], kPointThreads, [&](int64_t i, int64_t n) {
            k_chi_items_point<<<(unsigned)n * kChiParts, 64 * kGridWaves, 0, p->cap>>>(
                p->table, p->citems + c[kChiLane] + i, (int)n, p->qx, p->qy, p->qz, p->qs, p->chi);
            launched();
        });
        auto lanes_sum = [&](auto kernel, auto* w, int n, const int* perm, int nperm) {
            kernel<<<p->grid, 256, 0, p->cap>>>(p->table, p->items, n, sums, p->counter, p->qx, p->qy, p->qz, p->qs, perm, nperm,
                                                p->chi, w);
            launched();
        };
        if (!f32) {
            const int* perm = (s.order & kOrderSorted) ? p->perm : nullptr;
            if (sums == 1) lanes_sum(k_bdry_persistent<double, true>, (double*)p->w, p->nitems, perm, p->nitems);
            else lanes_sum(k_bdry_persistent<double, false>, (double*)p->w, p->nitems, perm, p->nitems);
        } else {
            const int nperm = p->send[kSumOrdered];
            if (nlane > 0 && sums == 1) lanes_sum(k_bdry_persistent<float, true>, (float*)p->w, nlane, p->sperm, nperm);
            else if (nlane > 0) lanes_sum(k_bdry_persistent<float, false>, (float*)p->w, nlane, p->sperm, nperm);
            if (ngroup > 0) {
                int top = 0;
                for (const gwn_mesh_s* m : p->meshes) top = std::max(top, m->cluster_top);
                const size_t ints = point_stack_ints<kPlanGroup>(top);
                k_group_persistent<<<p->grid, 256, 4 * ints * sizeof(int), p->cap>>>(
                    p->table, p->items + nlane, ngroup, claims, p->counter + 1, p->qx, p->qy, p->qz, p->qs, nullptr, (int)ints,
                    p->chi, (float*)p->w);
                launched();
            }
        }
    }
    const hipError_t e = hipStreamEndCapture(p->cap, &p->graph);
    GWN_HIP_TRY(le);
    GWN_HIP_TRY(e);
    GWN_HIP_TRY(hipGraphInstantiate(&p->exec, p->graph, nullptr, nullptr, 0));
    return GWN_OK;
}

gwn_status apply(gwn_multi_s* p, Schedule s, hipStream_t st) {
    if (p->nq > 0x7fffffffll) s.order &= ~kOrderSorted;   // the permutation holds 32-bit indices
    gwn_status r = build_items(p, s, st);
    if (r != GWN_OK) return r;
    const bool all = (s.order & kOrderSorted) != 0;
    const bool walk = p->cend[kChiOrdered] > 0, sums = p->prec != GWN_PREC_FP64 && p->send[kSumOrdered] > 0;
    if (all ? p->sorted < 2 : (walk || sums) && p->sorted < 1) {
        r = GWN_OK;
        if (all || walk) r = build_perm(p, false, p->citems, all ? p->nitems : p->cend[kChiOrdered], &p->perm, st);
        if (r == GWN_OK && sums && !p->sperm) r = build_perm(p, true, p->items, p->send[kSumOrdered], &p->sperm, st);
        if (r == GWN_E_OOM && !all) {   // no memory for orders that nobody asked for: none
            clear_error();
            (void)hipGetLastError();
            (void)hipFree(p->perm);
            (void)hipFree(p->sperm);
            p->perm = p->sperm = nullptr;
        } else if (r != GWN_OK) {
            return r;
        } else {
            p->sorted = all ? 2 : 1;
        }
    }
    r = capture(p, s);
    if (r != GWN_OK) return r;
    p->sched = s;
    return GWN_OK;
}

gwn_status time_replay(gwn_multi_s* p, hipStream_t st, double* ms) {
    hipEvent_t a, b;
    GWN_HIP_TRY(hipEventCreate(&a));
    GWN_HIP_TRY(hipEventCreate(&b));
    GWN_HIP_TRY(hipGraphLaunch(p->exec, st));           // warm-up
    GWN_HIP_TRY(hipEventRecord(a, st));
    GWN_HIP_TRY(hipGraphLaunch(p->exec, st));
    GWN_HIP_TRY(hipEventRecord(b, st));
    GWN_HIP_TRY(hipEventSynchronize(b));
    float f = 0.f;
    GWN_HIP_TRY(hipEventElapsedTime(&f, a, b));
    (void)hipEventDestroy(a);
    (void)hipEventDestroy(b);
    *ms = f;
    return GWN_OK;
}

// plan2: schedules timed before the kernels over clusters are not used
std::string cache_key(const gwn_multi_s* p) {
    hipDeviceProp_t prop;
    std::string arch = "gpu";
    if (hipGetDeviceProperties(&prop, p->device) == hipSuccess) arch = prop.gcnArchName;
    const size_t colon = arch.find(':');
    if (colon != std::string::npos) arch = arch.substr(0, colon);
    char buf[256];
    std::snprintf(buf, sizeof(buf), "%s|%s|plan2|meshes=%d|q=2^%d|pairs=2^%d", arch.c_str(),
                  p->prec == GWN_PREC_FP64 ? "fp64" : "fp32", p->nmesh,
                  (int)std::lround(std::log2(std::max(1.0, (double)p->nq))),
                  (int)std::lround(std::log2(std::max(1.0, p->est_pairs))));
    return buf;
}

bool cache_lookup(const char* path, const std::string& key, Schedule* s) {
    if (!path) return false;
    FILE* f = std::fopen(path, "r");
    if (!f) return false;
    char line[512];
    bool found = false;
    while (std::fgets(line, sizeof(line), f)) {
        char k[256];
        Schedule t;
        if (std::sscanf(line, " {\"key\": \"%255[^\"]\", \"item_queries\": %d, \"waves_per_simd\": %d, \"order\": %d",
                        k, &t.item_queries, &t.waves_per_simd, &t.order) == 4 &&
            key == k && t.item_queries >= 64 && t.item_queries % 64 == 0 && t.waves_per_simd >= 1 &&
            t.waves_per_simd <= 8 && t.order >= 0 && t.order <= 3) {
            *s = t;
            found = true;   // the last matching line wins
        }
    }
    std::fclose(f);
    return found;
}

void cache_store(const char* path, const std::string& key, const Schedule& s, double ms) {
    if (!path) return;
    FILE* f = std::fopen(path, "a");
    if (!f) return;
    std::fprintf(f, "{\"key\": \"%s\", \"item_queries\": %d, \"waves_per_simd\": %d, \"order\": %d, \"ms\": %.4f}\n",
                 key.c_str(), s.item_queries, s.waves_per_simd, s.order, ms);
    std::fclose(f);
}

}  // namespace

gwn_status multi_create(const gwn_mesh* meshes, int nmesh, const float* qx, const float* qy, const float* qz,
                        int64_t qs, const int64_t* q_offsets, int prec, void* w_out, int32_t* chi_out,
                        const gwn_multi_opts* opts, hipStream_t st, gwn_multi_s** out) {
    gwn_multi_s* p = new (std::nothrow) gwn_multi_s();
    if (!p) return GWN_E_OOM;
    struct Guard {
        gwn_multi_s* p;
        ~Guard() { if (p) release(p); }
    } guard{p};
    GWN_HIP_TRY(hipGetDevice(&p->device));
    p->nmesh = nmesh;
    p->meshes.assign(meshes, meshes + nmesh);
    p->qoff_h.assign(q_offsets, q_offsets + nmesh + 1);
    p->nq = p->qoff_h[nmesh];
    for (int m = 0; m < nmesh; ++m)
        p->est_pairs += (double)(p->qoff_h[m + 1] - p->qoff_h[m]) * (double)p->meshes[m]->nb;
    p->qx = qx;
    p->qy = qy;
    p->qz = qz;
    p->qs = qs;
    p->prec = prec;
    p->w = w_out;
    p->chi = chi_out;
    if (!p->chi) {
        GWN_HIP_TRY(gwn::dmalloc((void**)&p->chi, sizeof(int) * (size_t)std::max<long long>(1, p->nq)));
        p->own_chi = true;
    }
    p->forms = plan_forms(p->meshes, p->qoff_h);
    std::vector<MeshView> tab(nmesh);
    for (int m = 0; m < nmesh; ++m) tab[m] = p->meshes[m]->view();
    GWN_HIP_TRY(gwn::dmalloc((void**)&p->table, sizeof(MeshView) * (size_t)nmesh));
    GWN_HIP_TRY(gwn::dmalloc((void**)&p->counter, 2 * sizeof(int)));
    GWN_HIP_TRY(hipMemcpyAsync(p->table, tab.data(), sizeof(MeshView) * nmesh, hipMemcpyHostToDevice, st));
    GWN_HIP_TRY(hipStreamSynchronize(st));
    GWN_HIP_TRY(hipStreamCreateWithFlags(&p->cap, hipStreamNonBlocking));

    Schedule s;
    const bool explicit_sched = opts && (opts->item_queries > 0 || opts->waves_per_simd > 0 || opts->order > 0);
    if (opts && opts->item_queries > 0) s.item_queries = ((opts->item_queries + 63) / 64) * 64;
    if (opts && opts->waves_per_simd > 0) s.waves_per_simd = std::min(8, opts->waves_per_simd);
    if (opts && opts->order > 0) s.order = opts->order & 3;
    const char* cache = opts ? opts->tune_cache : nullptr;
    const std::string key = cache_key(p);
    Schedule cached;
    if (!explicit_sched && cache_lookup(cache, key, &cached)) {
        s = cached;
        p->tuned = true;
    } else if (!explicit_sched && opts && opts->autotune && p->nq > 0) {
        static const int tiles[] = {64, 128, 256, 512};
        static const int wps[] = {4, 8};
        static const int orders[] = {0, 1};
        double best = 1e300;
        Schedule bs = s;
        for (int o : orders)
            for (int wv : wps)
                for (int t : tiles) {
                    Schedule c;
                    c.item_queries = t;
                    c.waves_per_simd = wv;
                    c.order = o;
                    gwn_status r = apply(p, c, st);
                    if (r != GWN_OK) return r;
                    double ms = 0.0;
                    r = time_replay(p, st, &ms);
                    if (r != GWN_OK) return r;
                    if (ms < best) {
                        best = ms;
                        bs = c;
                    }
                }
        // the best schedule again with each mesh's queries in Morton order
        Schedule c = bs;
        c.order |= kOrderSorted;
        gwn_status r = apply(p, c, st);
        if (r != GWN_OK) return r;
        double ms = 0.0;
        r = time_replay(p, st, &ms);
        if (r != GWN_OK) return r;
        if (ms < best) {
            best = ms;
            bs = c;
        }
        s = bs;
        p->tuned = true;
        p->tuned_ms = best;
        cache_store(cache, key, s, best);
    }
    gwn_status r = apply(p, s, st);
    if (r != GWN_OK) return r;
    guard.p = nullptr;
    *out = p;
    return GWN_OK;
}

gwn_status multi_run(gwn_multi_s* p, hipStream_t st) {
    GWN_HIP_TRY(hipGraphLaunch(p->exec, st));
    return GWN_OK;
}

void multi_destroy(gwn_multi_s* p) { release(p); }

void multi_info(const gwn_multi_s* p, gwn_multi_info* o) {
    o->nmesh = p->nmesh;
    o->nqueries = p->nq;
    o->nitems = p->nitems;
    o->item_queries = p->sched.item_queries;
    o->waves_per_simd = p->sched.waves_per_simd;
    o->order = p->sched.order;
    o->grid_blocks = p->grid;
    o->tuned = p->tuned ? 1 : 0;
    o->est_pairs = p->est_pairs;
    o->tuned_ms = p->tuned_ms;
}

}  // namespace gwn

extern "C" int64_t gwn_test_plan_launches(int64_t nitems, int32_t kernel, int64_t* work_items) {
    const int threads = kernel == 0 ? gwn::kKeyThreads : kernel == 1 ? gwn::kWalkThreads : kernel == 2 ? gwn::kPointThreads : 512;
    int64_t launches = 0, next = 0;
    *work_items = 0;
    gwn::launch_slices(nitems, threads, [&](int64_t i, int64_t n) {
        launches += i == next;   // the slices follow each other
        next = i + n;
        *work_items = std::max(*work_items, n * threads);
    });
    return next == nitems ? launches : -1;
}

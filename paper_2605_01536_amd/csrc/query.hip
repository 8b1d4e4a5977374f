// query.hip -- single-mesh query kernels for arbitrary points: crossing counts
// and the boundary term per point (the arithmetic lives in gwn_kernels.h; the
// grid kernel with one ray per column is in grid.hip).
#include <cmath>
#include <cstdlib>
#include <type_traits>

#include <algorithm>

#include "gwn_alloc.h"
#include "gwn_kernels.h"
#include "gwn_mesh.h"

namespace gwn {
namespace {

// Where the crossing kernels' results go.  A mesh without boundary has w = chi: then they
// write w (wf or wd) too, and there is no second kernel and, unless the caller wants the
// counts, no array for them (1,000 points on a closed mesh of 1,280 triangles: 32 -> 9 us
// a call).
struct ChiOut {
    int* chi;
    float* wf;
    double* wd;
    __device__ __forceinline__ void put(long long i, int c) const {
        if (chi) chi[i] = c;
        if (wf) wf[i] = (float)c;
        if (wd) wd[i] = (double)c;
    }
};

// crossing counts of arbitrary points (per-lane LDS traversal stack)
__global__ __launch_bounds__(kChiBlock) void k_chi_batch(MeshView mv, const float* __restrict__ qx,
                                                         const float* __restrict__ qy, const float* __restrict__ qz,
                                                         long long qs, long long nq, ChiOut out) {
    __shared__ int stk[kLdsStack * kChiBlock];
    const long long i = blockIdx.x * (long long)kChiBlock + threadIdx.x;
    if (i >= nq) return;
    const QPoint q = quantize_point(qx[i * qs], qy[i * qs], qz[i * qs], mv.g);
    out.put(i, q.inbox ? chi_up(mv, q, stk + threadIdx.x) : 0);
}

// the same for few points, a wave per point
__global__ __launch_bounds__(64 * kGridWaves) void k_chi_point(MeshView mv, const float* __restrict__ qx,
                                                              const float* __restrict__ qy,
                                                              const float* __restrict__ qz, long long qs, long long nq,
                                                              ChiOut out) {
    __shared__ ChiLists lists[kGridWaves];
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const long long i = (long long)blockIdx.x * kGridWaves + wave;
    if (i >= nq) return;   // the whole wave
    const QPoint q = quantize_point(qx[i * qs], qy[i * qs], qz[i * qs], mv.g);
    const int c = q.inbox ? chi_up_wave(mv, q, lists[wave]) : 0;
    if ((threadIdx.x & 63) == 0) out.put(i, c);
}

// Crossing counts of Morton-ordered points, one wave-uniform traversal per wave
// (chi_wave_walk): neighbouring lines share almost their whole path, so the
// wave walks about one path instead of 64 divergent ones.  UP: the +z ray only
// (z-pruned); otherwise both directions of the whole line.
template <bool UP>
__global__ __launch_bounds__(64 * kGridWaves) void k_chi_wave(MeshView mv, const float* __restrict__ qx,
                                                             const float* __restrict__ qy,
                                                             const float* __restrict__ qz, long long qs, long long nq,
                                                             const int* __restrict__ perm, ChiOut up,
                                                             int* __restrict__ down) {
    __shared__ int wstack[kGridWaves][kLdsStack];
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const long long j = ((long long)blockIdx.x * kGridWaves + wave) * 64 + (threadIdx.x & 63);
    if ((long long)(blockIdx.x * kGridWaves + wave) * 64 >= nq) return;   // whole wave past the end
    const bool valid = j < nq;
    const long long i = perm[valid ? j : nq - 1];
    const QPoint q = quantize_point(qx[i * qs], qy[i * qs], qz[i * qs], mv.g);
    const bool act = valid && q.inbox;
    int u, d;
    chi_wave_walk<UP>(mv, q, act, wstack[wave], u, d);
    if (valid) {
        up.put(i, u);
        if (down) down[i] = d;
    }
}

// both crossing counts of arbitrary points (the whole vertical line)
__global__ __launch_bounds__(kChiBlock) void k_chi_line(MeshView mv, const float* __restrict__ qx,
                                                        const float* __restrict__ qy, const float* __restrict__ qz,
                                                        long long qs, long long nq, int* __restrict__ up,
                                                        int* __restrict__ down) {
    __shared__ int stk[kLdsStack * kChiBlock];
    const long long i = blockIdx.x * (long long)kChiBlock + threadIdx.x;
    if (i >= nq) return;
    const QPoint q = quantize_point(qx[i * qs], qy[i * qs], qz[i * qs], mv.g);
    int u = 0, d = 0;
    if (q.inbox) chi_line(mv, q, stk + threadIdx.x, u, d);
    if (up) up[i] = u;
    if (down) down[i] = d;
}

// ---------------------------------------------------------------- boundary, batch

// PARTS > 1: that many waves share 64 points, in FP32 each with a part of the clusters, the
// sums added in LDS; in FP64 in turn with a chunk each, whose sums the first wave adds in the
// chunks' order, so that the bits are those of a lane alone.
template <class T, int PARTS>
__global__ __launch_bounds__(PARTS > 4 ? 64 * PARTS : 256) void k_bdry_batch(MeshView mv, const float* __restrict__ qx, const float* __restrict__ qy,
                                                    const float* __restrict__ qz, long long qs, long long nq,
                                                    const int* __restrict__ perm, const int* __restrict__ chi,
                                                    T* __restrict__ w) {
    static_assert(PARTS == 1 || PARTS == 4 || (PARTS == 16 && sizeof(T) == 4), "256 threads, FP32 also 1,024");
    const int wave = PARTS == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const long long j = (long long)blockIdx.x * (PARTS == 1 ? 256 : 64) + (PARTS == 1 ? threadIdx.x : threadIdx.x & 63);
    const long long jj = j < nq ? j : nq - 1;
    // with a traversal order, lane j takes point perm[j]: the lanes of a wave are
    // neighbours, with the same clusters near and far
    const long long i = j < nq ? (perm ? (long long)perm[j] : j) : nq;
    const long long ii = perm ? (long long)perm[jj] : jj;
    const float px = qx[ii * qs], py = qy[ii * qs], pz = qz[ii * qs];
    const QPoint q = quantize_point(px, py, pz, mv.g);
    const int unit = sizeof(T) == 4 ? point_unit(px, py, pz, q.inbox, mv.g) : 0;
    double S = 0.0;
    if constexpr (sizeof(T) == 8 && PARTS > 1) {
        __shared__ double part[2][PARTS][64];
        const int lane = threadIdx.x & 63;
        const T pzs = (T)pz * (T)mv.g.scale;
        const bool quads = quad_z(pz, mv.g);
        PVert<T> last;
        for (int c0 = 0, b = 0; c0 < mv.nchunk; c0 += PARTS, b ^= 1) {
            if (q.inbox && c0 + wave < mv.nchunk)
                part[b][wave][lane] = point_chunk<T, true>(mv.chain + (size_t)(c0 + wave) * kChunk, q.x, q.y, pzs, quads, last, false);
            __syncthreads();   // one a step: the other half is written meanwhile
            if (wave == 0 && q.inbox)
                for (int v = 0; v < min(PARTS, mv.nchunk - c0); ++v) S += part[b][v][lane];
        }
        if (wave > 0) return;
        if (!q.inbox) outside_sum<T>(mv, px, py, pz, 0, 1, unit, S);
    } else if (!q.inbox) {   // rare: raw offsets, edge by edge
        outside_sum<T>(mv, px, py, pz, wave, PARTS, unit, S);
    } else if constexpr (sizeof(T) == 4) {
        const float sc = mv.g.scalef;
        S = point_clusters(mv, {q.x, q.y, px * sc, py * sc, pz * sc, quad_z(pz, mv.g), unit}, wave, PARTS);
    } else {
        point_chunks<T, true>(mv, 0, mv.nchunk, 1, q.x, q.y, (T)pz * (T)mv.g.scale, quad_z(pz, mv.g), unit, S);
    }
    if constexpr (PARTS > 1 && sizeof(T) == 4) {
        __shared__ double part[PARTS][64];
        const int lane = threadIdx.x & 63;
        part[wave][lane] = S;
        __syncthreads();
        if (wave > 0) return;
        for (int v = 1; v < PARTS; ++v) S += part[v][lane];
    }
    if (i < nq) w[i] = (T)((double)chi[i] + point_total<T>(S, unit) * kInv2Pi);
}

// ---------------------------------------------------------------- boundary, few points
// FP32: G points per wave (see point_group).
constexpr int kPointWaves = 4;

template <int G>
__global__ __launch_bounds__(64 * kPointWaves) void k_bdry_group(MeshView mv, const float* __restrict__ qx,
                                                                const float* __restrict__ qy,
                                                                const float* __restrict__ qz, long long qs,
                                                                long long nq, const int* __restrict__ perm,
                                                                int stack_ints, const int* __restrict__ chi,
                                                                float* __restrict__ w) {
    __shared__ PointLists<G> lists[kPointWaves];
    extern __shared__ int stacks[];
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const long long j0 = ((long long)blockIdx.x * kPointWaves + wave) * G;
    if (j0 >= nq) return;   // the whole wave
    point_group_out<G>(mv, qx, qy, qz, qs, j0, (int)min((long long)G, nq - j0), perm, stacks + (size_t)wave * stack_ints,
                       stack_ints, lists[wave], chi, w);
}

// FP32, so few points that a wave each leaves most of the chip idle: a workgroup per point
// (a point on a loop of 200,002 edges 1.11 -> 0.46 ms, 0.58 edge by edge; 200 points on 63 k
// edges 67 -> 47 us).
__global__ __launch_bounds__(64 * kPointWaves) void k_bdry_point(MeshView mv, const float* __restrict__ qx,
                                                                const float* __restrict__ qy,
                                                                const float* __restrict__ qz, long long qs,
                                                                int stack_ints, const int* __restrict__ chi,
                                                                float* __restrict__ w) {
    __shared__ PointLists<1> lists[kPointWaves];
    __shared__ double part[kPointWaves];
    extern __shared__ int stacks[];
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
    const long long i = blockIdx.x;
    const float px = qx[i * qs], py = qy[i * qs], pz = qz[i * qs];
    const QPoint q = quantize_point(px, py, pz, mv.g);
    const float sc = mv.g.scalef;
    const int unit = point_unit(px, py, pz, q.inbox, mv.g);
    double S = 0.0;
    if (q.inbox) {
        if (lane == 0) lists[wave].p[0] = {q.x, q.y, px * sc, py * sc, pz * sc, quad_z(pz, mv.g), unit};
        wave_lds_sync();
        S = point_group<1>(mv, 1u, stacks + (size_t)wave * stack_ints, stack_ints, lists[wave], wave, kPointWaves);
    } else {
        outside_sum<float>(mv, px, py, pz, (int)threadIdx.x, 64 * kPointWaves, unit, S);
        for (int o = 32; o > 0; o >>= 1) S += __shfl_xor(S, o);
    }
    if (lane == 0) part[wave] = S;
    __syncthreads();
    if (threadIdx.x > 0) return;
    for (int v = 1; v < kPointWaves; ++v) S += part[v];
    w[i] = (float)((double)chi[i] + point_total<float>(S, unit) * kInv2Pi);
}

// FP64, few points against many boundary edges: one workgroup per point, the chunks dealt
// out to its lanes, the partial sums reduced across the wave by shuffles and across the
// workgroup in LDS, in a fixed order.
constexpr int kSplitThreads = 256;

__global__ __launch_bounds__(kSplitThreads) void k_bdry_split(MeshView mv, const float* __restrict__ qx,
                                                             const float* __restrict__ qy,
                                                             const float* __restrict__ qz, long long qs, long long nq,
                                                             const int* __restrict__ chi, double* __restrict__ w) {
    __shared__ double red[kSplitThreads / 64];
    const long long i = blockIdx.x;   // one point per workgroup
    if (i >= nq) return;
    const float px = qx[i * qs], py = qy[i * qs], pz = qz[i * qs];
    const QPoint q = quantize_point(px, py, pz, mv.g);
    double S = 0.0;
    if (q.inbox)
        point_chunks<double, false>(mv, (int)threadIdx.x, mv.nchunk, kSplitThreads, q.x, q.y, (double)pz * mv.g.scale,
                             quad_z(pz, mv.g), 0, S);
    else
        outside_sum<double>(mv, px, py, pz, (int)threadIdx.x, kSplitThreads, 0, S);
    for (int o = 32; o > 0; o >>= 1) S += __shfl_xor(S, o);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = S;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int k = 0; k < kSplitThreads / 64; ++k) t += red[k];
        w[i] = (double)chi[i] + t * kInv2Pi;
    }
}

// ws (nullable): caller memory for the temporaries -- a crossing-count buffer
// when chi_out is null, the traversal order and its sort's scratch -- for at
// most one launch's worth of points; without it they are stream-ordered
// allocations.
template <class T>
gwn_status launch_batch(const gwn_mesh_s* m, const float* qx, const float* qy, const float* qz, int64_t qs, int64_t nq,
                        T* w, int32_t* chi_out, const BatchWorkspace* ws, hipStream_t st) {
    int* chi = chi_out;
    const bool closed = m->nb == 0;
    if (!chi && !closed) {
        if (ws) chi = ws->chi;
        else GWN_HIP_TRY(gwn::dmalloc_async((void**)&chi, sizeof(int) * (size_t)nq, st));
    }
    const bool own_chi = !chi_out && !ws && !closed;
    const MeshView mv = m->view();
    constexpr int kPrec = sizeof(T) == 8 ? GWN_PREC_FP64 : GWN_PREC_FP32;
    hipError_t e = hipSuccess;
    // one launch covers at most max_launch_queries() points (the 32-bit grid size)
    const int64_t chunk = max_launch_queries();
    for (int64_t o = 0; o < nq && e == hipSuccess; o += chunk) {
        const int64_t n = std::min<int64_t>(chunk, nq - o);
        const float *x = qx + o * qs, *y = qy + o * qs, *z = qz + o * qs;
        // a traversal order for either pass (with ws in the same memory, one after the other)
        int* perm = nullptr;
        auto order = [&](bool space) {
            if (!ws) return xy_order(m, x, y, z, qs, n, space, &perm, st);
            perm = ws->perm;
            return xy_order_into(m, x, y, z, qs, n, space, ws->perm, ws->order_temp, st);
        };
        auto drop = [&] {
            if (perm && !ws) (void)hipFreeAsync(perm, st);
            perm = nullptr;
        };
        ChiOut out{chi ? chi + o : nullptr, nullptr, nullptr};
        if (closed) {
            if constexpr (sizeof(T) == 4) out.wf = w + o;
            else out.wd = w + o;
        }
        gwn_status so = want_xy_order(m, n) ? order(false) : GWN_OK;
        if (so == GWN_OK) {
            if (perm) {
                k_chi_wave<true><<<(unsigned)((n + 64 * kGridWaves - 1) / (64 * kGridWaves)), 64 * kGridWaves, 0, st>>>(
                    mv, x, y, z, qs, n, perm, out, nullptr);
            } else if (want_chi_point(m, n)) {
                k_chi_point<<<(unsigned)((n + kGridWaves - 1) / kGridWaves), 64 * kGridWaves, 0, st>>>(mv, x, y, z, qs, n,
                                                                                                            out);
            } else {
                k_chi_batch<<<(unsigned)((n + kChiBlock - 1) / kChiBlock), kChiBlock, 0, st>>>(mv, x, y, z, qs, n, out);
            }
            e = hipGetLastError();
        }
        const bool few = want_split(m, n, kPrec) && !(sizeof(T) == 4 && m->wide_edges());
        if (so == GWN_OK && e == hipSuccess && !closed && !few && want_space_order(m, n, kPrec)) {
            drop();
            so = order(true);
            if (so == GWN_E_OOM && !ws && !want_xy_order(m, n)) {   // unordered instead: the same bits, later
                clear_error();
                (void)hipGetLastError();
                perm = nullptr;
                so = GWN_OK;
            }
        }
        if (so != GWN_OK) {
            if (own_chi) (void)hipFreeAsync(chi, st);
            return so;   // the order has set the message
        }
        if (e == hipSuccess && !closed) {
            if (!few) {
                const bool parts = want_parts(m, n, kPrec);
                const bool many = sizeof(T) == 4 && parts && m->wide_edges() && n <= kManyParts;
                if constexpr (sizeof(T) == 4)
                    if (many) k_bdry_batch<T, 16><<<(unsigned)((n + 63) / 64), 1024, 0, st>>>(mv, x, y, z, qs, n, perm, chi + o, w + o);
                if (parts && !many)
                    k_bdry_batch<T, 4><<<(unsigned)((n + 63) / 64), 256, 0, st>>>(mv, x, y, z, qs, n, perm, chi + o, w + o);
                if (!parts)
                    k_bdry_batch<T, 1><<<(unsigned)((n + 255) / 256), 256, 0, st>>>(mv, x, y, z, qs, n, perm, chi + o, w + o);
            } else if constexpr (sizeof(T) == 4) {
                auto go = [&](auto G) {
                    constexpr int kG = decltype(G)::value;
                    const size_t ints = point_stack_ints<kG>(m->cluster_top);
                    const long long groups = (n + kG - 1) / kG;
                    k_bdry_group<kG><<<(unsigned)((groups + kPointWaves - 1) / kPointWaves), 64 * kPointWaves,
                                       kPointWaves * ints * sizeof(int), st>>>(mv, x, y, z, qs, n, perm, (int)ints,
                                                                               chi + o, w + o);
                };
                const bool single = m->cluster_top <= kSingleTop;
                if (n <= kFewPoints && single) {
                    const size_t ints = point_stack_ints<1>(m->cluster_top);
                    k_bdry_point<<<(unsigned)n, 64 * kPointWaves, kPointWaves * ints * sizeof(int), st>>>(
                        mv, x, y, z, qs, (int)ints, chi + o, w + o);
                } else if (n <= kSinglePoints && single) go(std::integral_constant<int, 1>{});
                else go(std::integral_constant<int, 4>{});
            } else {
                k_bdry_split<<<(unsigned)n, kSplitThreads, 0, st>>>(mv, x, y, z, qs, n, chi + o, w + o);
            }
            e = hipGetLastError();
        }
        drop();
    }
    if (own_chi) (void)hipFreeAsync(chi, st);
    GWN_HIP_TRY(e);
    return GWN_OK;
}

}  // namespace

gwn_status query_crossings(const gwn_mesh_s* m, const float* qx, const float* qy, const float* qz, int64_t qs,
                           int64_t nq, int32_t* up, int32_t* down, hipStream_t st) {
    axis_ptrs(m->axis, qx, qy, qz);
    const MeshView mv = m->view();
    const int64_t chunk = max_launch_queries();
    for (int64_t o = 0; o < nq; o += chunk) {
        const int64_t n = std::min<int64_t>(chunk, nq - o);
        const float *x = qx + o * qs, *y = qy + o * qs, *z = qz + o * qs;
        int* perm = nullptr;
        if (want_xy_order(m, n)) {
            const gwn_status so = xy_order(m, x, y, z, qs, n, false, &perm, st);
            if (so != GWN_OK) return so;
        }
        if (perm) {
            k_chi_wave<false><<<(unsigned)((n + 64 * kGridWaves - 1) / (64 * kGridWaves)), 64 * kGridWaves, 0, st>>>(
                mv, x, y, z, qs, n, perm, ChiOut{up ? up + o : nullptr, nullptr, nullptr}, down ? down + o : nullptr);
        } else {
            k_chi_line<<<(unsigned)((n + kChiBlock - 1) / kChiBlock), kChiBlock, 0, st>>>(
                mv, x, y, z, qs, n, up ? up + o : nullptr, down ? down + o : nullptr);
        }
        const hipError_t e = hipGetLastError();
        if (perm) (void)hipFreeAsync(perm, st);
        GWN_HIP_TRY(e);
    }
    return GWN_OK;
}

bool want_chi_point(const gwn_mesh_s* m, int64_t n) {
    return n <= (m->nf >= (1 << 15) ? (1 << 18) : m->nf >= 1024 ? 32768 : 8192);
}

bool want_split(const gwn_mesh_s* m, int64_t n, int prec) {
    if (const char* e = std::getenv("GWN_SPLIT_BOUNDARY")) return std::atoi(e) != 0 && m->nb > 0;
    if (prec >= 0 && prec < 2 && m->split_max[prec] != 0) return m->split_max[prec] > 0 && n <= m->split_max[prec] && m->nb > 0;
    if (prec == GWN_PREC_FP32) return n < kDensePoints && m->nb >= (n <= 16384 ? 64 : kGroupEdges);
    return n <= 8192 && m->nb >= 16 * 256;
}

bool want_parts(const gwn_mesh_s* m, int64_t n, int prec) {
    if (prec == GWN_PREC_FP64) return n <= (m->nchunk < 64 ? 4 * kSharedPoints64 : kSharedPoints64) && m->nchunk >= 8;
    return n <= kSharedPoints && m->nchunk >= 8;
}

int64_t max_launch_queries() {
    int64_t n = int64_t(1) << 30;
    if (const char* e = std::getenv("GWN_MAX_LAUNCH_QUERIES")) {
        const long long v = std::atoll(e);
        if (v >= 256 && v < n && v % 256 == 0) n = v;
    }
    return n;
}

gwn_status query_batch(const gwn_mesh_s* m, const float* qx, const float* qy, const float* qz, int64_t qs, int64_t nq,
                       int prec, void* w, int32_t* chi_out, hipStream_t st) {
    return query_batch_ws(m, qx, qy, qz, qs, nq, prec, w, chi_out, nullptr, st);
}

gwn_status query_batch_ws(const gwn_mesh_s* m, const float* qx, const float* qy, const float* qz, int64_t qs,
                          int64_t nq, int prec, void* w, int32_t* chi_out, const BatchWorkspace* ws, hipStream_t st) {
    if (nq == 0) return GWN_OK;
    if (ws && nq > max_launch_queries()) {
        set_error("query_batch: a workspace covers one launch of at most %lld points", (long long)max_launch_queries());
        return GWN_E_INVALID;
    }
    axis_ptrs(m->axis, qx, qy, qz);
    if (prec == GWN_PREC_FP64) return launch_batch<double>(m, qx, qy, qz, qs, nq, (double*)w, chi_out, ws, st);
    return launch_batch<float>(m, qx, qy, qz, qs, nq, (float*)w, chi_out, ws, st);
}

}  // namespace gwn

// build.hip -- device-side mesh ingest (gwn_build_mesh):
//   vertex statistics and validation, fixed-point quantisation, Morton-ordered
//   LBVH with integer boxes (Karras-style split search, bottom-up refit), and
//   the directed boundary chain of the soup (Sec. 4.1: interior edges cancel),
//   chained into closed loops so that the query kernels visit every boundary
//   vertex once.  Sorting and scans use the library's radix sort and scan
//   (sort.hip); everything else is below.

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstring>
#include <vector>

#include "gwn_alloc.h"
#include "gwn_mesh.h"
#include "gwn_sort.h"

namespace gwn {
namespace {

constexpr int kThreads = 256;

inline int nblocks(int64_t n, int t = kThreads) {
    int64_t b = (n + t - 1) / t;
    return (int)std::max<int64_t>(1, std::min<int64_t>(b, 1 << 20));
}

// ------------------------------------------------------------------ helpers

// Build temporaries: slices of a few large blocks, released when the build
// returns -- also on an error path, where kernels enqueued before the failure may
// still be running: the stream is drained first.  A block each for the 66
// temporaries of a welded build cost more than its kernels (a hipFree takes about
// 90 us, a hipMalloc 15: 7 of 12.6 ms for 312,000 triangles).
struct Scratch {
    std::vector<void*> blocks;
    char* cur = nullptr;
    size_t left = 0;
    size_t first = size_t(1) << 20;   // bytes of the first block; the others as large as asked, at least 1/8 of it
    hipStream_t st = nullptr;
    ~Scratch() {
        if (!blocks.empty()) (void)hipStreamSynchronize(st);
        for (void* p : blocks) (void)hipFree(p);
    }
    hipError_t block(size_t want) {
        void* q = nullptr;
        const hipError_t e = gwn::dmalloc(&q, want);
        if (e != hipSuccess) return e;
        blocks.push_back(q);
        cur = (char*)q;
        left = want;
        return hipSuccess;
    }
    // one block for slices of `bytes` in all, if they do not fit the current one
    hipError_t reserve(size_t bytes) { return bytes > left ? block(bytes) : hipSuccess; }
    template <class T>
    hipError_t alloc(T** p, int64_t n) {
        *p = nullptr;
        const size_t bytes = (sizeof(T) * (size_t)std::max<int64_t>(n, 1) + 255) & ~(size_t)255;
        if (bytes > left) {
            const hipError_t e = block(std::max(bytes, blocks.empty() ? first : first / 8));
            if (e != hipSuccess) return e;
        }
        *p = (T*)cur;
        cur += bytes;
        left -= bytes;
        return hipSuccess;
    }
};

// ------------------------------------------------------------------ kernels

__global__ void k_vertex_stats(const float* __restrict__ vx, const float* __restrict__ vy, const float* __restrict__ vz,
                               int64_t vs, int64_t nv, float* __restrict__ part, int* __restrict__ flags) {
    __shared__ float sm[6][kThreads];
    float mn[3] = {INFINITY, INFINITY, INFINITY}, mx[3] = {-INFINITY, -INFINITY, -INFINITY};
    bool bad = false;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < nv; i += (int64_t)gridDim.x * blockDim.x) {
        float p[3] = {vx[i * vs], vy[i * vs], vz[i * vs]};
        for (int a = 0; a < 3; ++a) {
            bad |= !isfinite(p[a]);
            mn[a] = fminf(mn[a], p[a]);
            mx[a] = fmaxf(mx[a], p[a]);
        }
    }
    if (bad) atomicOr(flags, 1);
    for (int a = 0; a < 3; ++a) {
        sm[a][threadIdx.x] = mn[a];
        sm[3 + a][threadIdx.x] = mx[a];
    }
    __syncthreads();
    for (int s = kThreads / 2; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) {
            for (int a = 0; a < 3; ++a) {
                sm[a][threadIdx.x] = fminf(sm[a][threadIdx.x], sm[a][threadIdx.x + s]);
                sm[3 + a][threadIdx.x] = fmaxf(sm[3 + a][threadIdx.x], sm[3 + a][threadIdx.x + s]);
            }
        }
        __syncthreads();
    }
    if (threadIdx.x == 0)
        for (int a = 0; a < 6; ++a) part[blockIdx.x * 6 + a] = sm[a][0];
}

__global__ void k_tri_check(const int32_t* __restrict__ tri, int64_t n3, int64_t nv, int* __restrict__ flags) {
    bool bad = false;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n3; i += (int64_t)gridDim.x * blockDim.x) {
        int32_t v = tri[i];
        bad |= (v < 0) | ((int64_t)v >= nv);
    }
    if (bad) atomicOr(flags, 2);
}

__global__ void k_quantize_vertices(const float* __restrict__ vx, const float* __restrict__ vy,
                                    const float* __restrict__ vz, int64_t vs, int64_t nv, QGrid g,
                                    int4* __restrict__ qv) {
    int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= nv) return;
    int4 q;
    q.x = (int)qround(vx[i * vs], g.lo[0], g.scale);
    q.y = (int)qround(vy[i * vs], g.lo[1], g.scale);
    q.z = (int)qround(vz[i * vs], g.lo[2], g.scale);
    q.w = 0;
    qv[i] = q;
}

__device__ __forceinline__ uint32_t spread10(uint32_t v) {
    v &= 1023u;
    v = (v | (v << 16)) & 0x030000FFu;
    v = (v | (v << 8)) & 0x0300F00Fu;
    v = (v | (v << 4)) & 0x030C30C3u;
    v = (v | (v << 2)) & 0x09249249u;
    return v;
}

__global__ void k_tri_setup(const int32_t* __restrict__ tri, int64_t nf, const int4* __restrict__ qv, int4 qlo,
                            int4 qspan, TriQ* __restrict__ tq, uint64_t* __restrict__ keys) {
    int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (t >= nf) return;
    int4 a = qv[tri[3 * t]], b = qv[tri[3 * t + 1]], c = qv[tri[3 * t + 2]];
    TriQ r;
    r.a = a;
    r.b = b;
    r.c = c;
    tq[t] = r;
    long long cx = ((long long)a.x + b.x + c.x) / 3 - qlo.x;
    long long cy = ((long long)a.y + b.y + c.y) / 3 - qlo.y;
    long long cz = ((long long)a.z + b.z + c.z) / 3 - qlo.z;
    uint32_t mx = (uint32_t)((cx * 1024) / ((long long)qspan.x + 1));
    uint32_t my = (uint32_t)((cy * 1024) / ((long long)qspan.y + 1));
    uint32_t mz = (uint32_t)((cz * 1024) / ((long long)qspan.z + 1));
    uint32_t m = (spread10(mx) << 2) | (spread10(my) << 1) | spread10(mz);
    keys[t] = ((uint64_t)m << 32) | (uint64_t)t;
}

__global__ void k_permute_tris(const uint64_t* __restrict__ keys, int64_t nf, const TriQ* __restrict__ src,
                               TriQ* __restrict__ dst, const int32_t* __restrict__ tri, const float* __restrict__ vx,
                               const float* __restrict__ vy, const float* __restrict__ vz, int64_t vs,
                               float4* __restrict__ trif) {
    int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= nf) return;
    const int64_t t = (int64_t)(keys[i] & 0xffffffffull);
    dst[i] = src[t];
    for (int c = 0; c < 3; ++c) {
        const int64_t v = tri[3 * t + c];
        trif[3 * i + c] = make_float4(vx[v * vs], vy[v * vs], vz[v * vs], 0.f);
    }
}

__device__ __forceinline__ int prefix_len(const uint64_t* __restrict__ keys, int n, int i, int j) {
    if (j < 0 || j >= n) return -1;
    return __clzll((long long)(keys[i] ^ keys[j]));   // keys are unique (index in the low bits)
}

// Karras (2012) radix-tree construction over the sorted unique keys: node i
// spans a key range found by exponential + binary search on the common-prefix
// length; its split is where the prefix length drops.
__global__ void k_karras(const uint64_t* __restrict__ keys, int n, Node* __restrict__ nodes, int* __restrict__ leaf_parent) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n - 1) return;
    int d = (prefix_len(keys, n, i, i + 1) - prefix_len(keys, n, i, i - 1)) >= 0 ? 1 : -1;
    int dmin = prefix_len(keys, n, i, i - d);
    int lmax = 2;
    while (prefix_len(keys, n, i, i + lmax * d) > dmin) lmax <<= 1;
    int l = 0;
    for (int t = lmax >> 1; t >= 1; t >>= 1)
        if (prefix_len(keys, n, i, i + (l + t) * d) > dmin) l += t;
    int j = i + l * d;
    int dnode = prefix_len(keys, n, i, j);
    int s = 0, t = l;
    do {
        t = (t + 1) >> 1;
        if (prefix_len(keys, n, i, i + (s + t) * d) > dnode) s += t;
    } while (t > 1);
    int gamma = i + s * d + min(d, 0);
    int left = (min(i, j) == gamma) ? ~gamma : gamma;
    int right = (max(i, j) == gamma + 1) ? ~(gamma + 1) : gamma + 1;
    nodes[i].link.x = left;
    nodes[i].link.y = right;
    nodes[i].link.w = j;   // the other end of the node's leaf range (i is one)
    if (left >= 0) nodes[left].link.z = i;
    else leaf_parent[~left] = i;
    if (right >= 0) nodes[right].link.z = i;
    else leaf_parent[~right] = i;
}

__device__ __forceinline__ int ld_acq(const int* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ void write_slot(Node* nodes, int parent, int child, const int b[6]) {
    Node* p = nodes + parent;
    if (p->link.x == child) {
        p->lxy = make_int4(b[0], b[1], b[2], b[3]);
        p->z.x = b[4];
        p->z.y = b[5];
    } else {
        p->rxy = make_int4(b[0], b[1], b[2], b[3]);
        p->z.z = b[4];
        p->z.w = b[5];
    }
}

// Bottom-up refit: each leaf writes its box into its parent's child slot; the
// second thread to reach a node merges both slots and continues upward.  A node
// whose leaves all belong to one workgroup (all but about 1 in 200) is settled there:
// its arrival count is in LDS and its boxes pass through the workgroup's own cache.
// Only the nodes above cross workgroups and need fences of the whole device, which
// write back and invalidate an XCD's L2: with those at every node the refit took
// 2.2 ms for 312,000 triangles (7.7 ms for 1.05M).
constexpr int kRefitThreads = 1024, kRefitLeaves = 4096;

__device__ __forceinline__ void refit_leaf(const TriQ* __restrict__ tris, int n, Node* nodes,
                                           const int* __restrict__ leaf_parent, int* flags, int t, int t0, int t1,
                                           int* inside) {
    TriQ q = tris[t];
    int b[6] = {min(q.a.x, min(q.b.x, q.c.x)), max(q.a.x, max(q.b.x, q.c.x)),
                min(q.a.y, min(q.b.y, q.c.y)), max(q.a.y, max(q.b.y, q.c.y)),
                min(q.a.z, min(q.b.z, q.c.z)), max(q.a.z, max(q.b.z, q.c.z))};
    int child = ~t;
    int parent = leaf_parent[t];
    for (int guard = 0; parent >= 0; ++guard) {
        if (guard > 70) {           // a radix tree over 62-bit keys is at most 63 deep
            atomicOr(flags + n, 4);
            return;
        }
        write_slot(nodes, parent, child, b);
        const int other = nodes[parent].link.w;   // written before this kernel
        const bool local = min(parent, other) >= t0 && max(parent, other) < t1;
        if (local) {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
            const int before = __hip_atomic_fetch_add(&inside[parent - t0], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            if (before == 0) return;
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
        } else {
            __threadfence();
            if (atomicAdd(flags + parent, 1) == 0) return;
            __threadfence();
        }
        const int* L = &nodes[parent].lxy.x;
        const int* R = &nodes[parent].rxy.x;
        const int* Z = &nodes[parent].z.x;
        if (local) {
            const int4 l = *(const int4*)L, r = *(const int4*)R, z = *(const int4*)Z;
            b[0] = min(l.x, r.x);
            b[1] = max(l.y, r.y);
            b[2] = min(l.z, r.z);
            b[3] = max(l.w, r.w);
            b[4] = min(z.x, z.z);
            b[5] = max(z.y, z.w);
        } else {
            b[0] = min(ld_acq(L + 0), ld_acq(R + 0));
            b[1] = max(ld_acq(L + 1), ld_acq(R + 1));
            b[2] = min(ld_acq(L + 2), ld_acq(R + 2));
            b[3] = max(ld_acq(L + 3), ld_acq(R + 3));
            b[4] = min(ld_acq(Z + 0), ld_acq(Z + 2));
            b[5] = max(ld_acq(Z + 1), ld_acq(Z + 3));
        }
        child = parent;
        parent = ld_acq(&nodes[parent].link.z);
    }
}

__global__ __launch_bounds__(kRefitThreads) void k_refit(const TriQ* __restrict__ tris, int n, Node* nodes,
                                                        const int* __restrict__ leaf_parent, int* flags) {
    __shared__ int inside[kRefitLeaves];   // arrivals at node t0 + k, for nodes within the workgroup's leaves
    if (n < 2) return;
    const int t0 = blockIdx.x * kRefitLeaves, t1 = min(t0 + kRefitLeaves, n);
    for (int k = threadIdx.x; k < kRefitLeaves; k += kRefitThreads) inside[k] = 0;
    __syncthreads();
    for (int t = t0 + (int)threadIdx.x; t < t1; t += kRefitThreads)
        refit_leaf(tris, n, nodes, leaf_parent, flags, t, t0, t1, inside);
}

__global__ void k_depth(int n, const Node* __restrict__ nodes, const int* __restrict__ leaf_parent, int* depth) {
    int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n || n < 2) return;
    int d = 0;
    for (int p = leaf_parent[t]; p >= 0 && d < 1000; p = nodes[p].link.z) ++d;
    atomicMax(depth, d);
}

// ---- boundary chain

// Both vertices of an edge in 2 bits bits (the smaller above), so that the sort has passes
// for those only.  Degenerate edges have all bits set: their low bits (twice the same vertex)
// are no edge's either.
__global__ void k_edge_keys(const int32_t* __restrict__ tri, int64_t nf, int bits, uint64_t* __restrict__ keys,
                            int* __restrict__ sgn) {
    int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= 3 * nf) return;
    int64_t t = i / 3;
    int c = (int)(i - 3 * t);
    uint32_t u = (uint32_t)tri[3 * t + c];
    uint32_t v = (uint32_t)tri[3 * t + (c + 1) % 3];
    if (u == v) {
        keys[i] = ~0ull;
        sgn[i] = 0;
    } else {
        keys[i] = ((uint64_t)min(u, v) << bits) | (uint64_t)max(u, v);
        sgn[i] = u < v ? 1 : -1;
    }
}

// net multiplicity per unordered vertex pair, stored at the first entry of its run
__global__ void k_edge_runs(const uint64_t* __restrict__ keys, const int* __restrict__ sgn, int64_t n,
                            int* __restrict__ net, int* __restrict__ cnt) {
    int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n) return;
    uint64_t k = keys[i];
    bool head = (k != ~0ull) && (i == 0 || keys[i - 1] != k);
    int m = 0;
    if (head)
        for (int64_t j = i; j < n && keys[j] == k; ++j) m += sgn[j];
    net[i] = m;
    cnt[i] = head ? abs(m) : 0;
}

__global__ void k_edge_emit(const uint64_t* __restrict__ keys, const int* __restrict__ net, const int* __restrict__ cnt,
                            const int* __restrict__ off, int64_t n, int bits, int* __restrict__ efrom, int* __restrict__ eto) {
    int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n || cnt[i] == 0) return;
    int lo = (int)(keys[i] >> bits), hi = (int)(keys[i] & ((1ull << bits) - 1ull));
    int m = net[i];
    for (int r = 0; r < cnt[i]; ++r) {
        efrom[off[i] + r] = m > 0 ? lo : hi;
        eto[off[i] + r] = m > 0 ? hi : lo;
    }
}

__global__ void k_iota(int* __restrict__ a, int64_t n) {
    int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i < n) a[i] = (int)i;
}

// in-degree == out-degree at every vertex, so the k-th edge sorted by target
// and the k-th edge sorted by source meet at the same vertex
__global__ void k_link(const int* __restrict__ in_by_to, const int* __restrict__ out_by_from, int64_t n,
                       int* __restrict__ succ) {
    int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (k < n) succ[in_by_to[k]] = out_by_from[k];
}

// Pointer doubling, twice per launch: of 85 k edges 17 rounds of two launches each are 0.2 ms
// of launches, whatever the loops' lengths.
__global__ void k_rep_round(const int* __restrict__ rep, const int* __restrict__ jmp, int64_t n, int* __restrict__ rep2,
                            int* __restrict__ jmp2) {
    int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int j = jmp[i], k = jmp[j], l = jmp[k];
    rep2[i] = min(min(rep[i], rep[j]), min(rep[k], rep[l]));
    jmp2[i] = jmp[l];
}

__global__ void k_rank_init(const int* __restrict__ succ, const int* __restrict__ rep, int64_t n, int* __restrict__ nxt,
                            int* __restrict__ dist) {
    int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n) return;
    int s = succ[i];
    nxt[i] = (s == rep[i]) ? -1 : s;
    dist[i] = (s == rep[i]) ? 0 : 1;
}

__global__ void k_rank_round(const int* __restrict__ nxt, const int* __restrict__ dist, int64_t n, int* __restrict__ nxt2,
                             int* __restrict__ dist2) {
    int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n) return;
    int j = nxt[i], d = dist[i];
    for (int k = 0; k < 3 && j >= 0; ++k) {
        d += dist[j];
        j = nxt[j];
    }
    nxt2[i] = j;
    dist2[i] = d;
}

// Representatives, ranks and both scans for few edges in one workgroup, in LDS: the rounds
// are two launches a power of two otherwise, 26 for 7 k edges.
constexpr int kFewEdges = 8192, kRankThreads = 1024, kRankPer = kFewEdges / kRankThreads;

__global__ __launch_bounds__(kRankThreads) void k_rank_loops(const int* __restrict__ succ, int nb, int rounds,
                                                            int* __restrict__ rep_out, int* __restrict__ dist_out,
                                                            int* __restrict__ voff, int* __restrict__ lid,
                                                            int* __restrict__ nloops) {
    __shared__ int A[kFewEdges], B[kFewEdges];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    int rep[kRankPer], jmp[kRankPer], dist[kRankPer];
    // element k of thread t: t * kRankPer + k, so that scans go in order
#pragma unroll
    for (int k = 0; k < kRankPer; ++k) {
        const int i = t * kRankPer + k;
        rep[k] = i;
        jmp[k] = i < nb ? succ[i] : i;
        A[i] = rep[k];
        B[i] = jmp[k];
    }
    __syncthreads();
    for (int r = 0; r < rounds; ++r) {   // the smallest edge of the cycle
#pragma unroll
        for (int k = 0; k < kRankPer; ++k) {
            const int j = jmp[k];
            rep[k] = min(rep[k], A[j]);
            jmp[k] = B[j];
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kRankPer; ++k) {
            A[t * kRankPer + k] = rep[k];
            B[t * kRankPer + k] = jmp[k];
        }
        __syncthreads();
    }
#pragma unroll
    for (int k = 0; k < kRankPer; ++k) {   // the distance to the cycle's end, opened there
        const int i = t * kRankPer + k, s = i < nb ? succ[i] : i;
        const bool end = s == rep[k];
        jmp[k] = end ? -1 : s;
        dist[k] = end ? 0 : 1;
        A[i] = jmp[k];
        B[i] = dist[k];
    }
    __syncthreads();
    for (int r = 0; r < rounds; ++r) {
#pragma unroll
        for (int k = 0; k < kRankPer; ++k) {
            const int j = jmp[k];
            if (j >= 0) {
                dist[k] += B[j];
                jmp[k] = A[j];
            }
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kRankPer; ++k) {
            A[t * kRankPer + k] = jmp[k];
            B[t * kRankPer + k] = dist[k];
        }
        __syncthreads();
    }
    // exclusive sums over the representatives: loop lengths, loops
    int len = 0, heads = 0;
#pragma unroll
    for (int k = 0; k < kRankPer; ++k) {
        const int i = t * kRankPer + k;
        if (i < nb && rep[k] == i) {
            len += dist[k] + 1;
            ++heads;
        }
    }
    int pl = len, ph = heads;
    for (int d = 1; d < 64; d <<= 1) {
        const int a = __shfl_up(pl, d), b = __shfl_up(ph, d);
        if (lane >= d) {
            pl += a;
            ph += b;
        }
    }
    if (lane == 63) {
        A[wave] = pl;
        B[wave] = ph;
    }
    __syncthreads();
    pl -= len;
    ph -= heads;
    for (int w = 0; w < wave; ++w) {
        pl += A[w];
        ph += B[w];
    }
#pragma unroll
    for (int k = 0; k < kRankPer; ++k) {
        const int i = t * kRankPer + k;
        if (i >= nb) continue;
        rep_out[i] = rep[k];
        dist_out[i] = dist[k];
        voff[i] = pl;
        lid[i] = ph;
        if (rep[k] == i) {
            pl += dist[k] + 1;
            ++ph;
        }
    }
    if (t == kRankThreads - 1) *nloops = ph;
}

__global__ void k_loop_counts(const int* __restrict__ rep, const int* __restrict__ dist, int64_t n, int* __restrict__ len,
                              int* __restrict__ head) {
    int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n) return;
    bool h = rep[i] == (int)i;
    len[i] = h ? dist[i] + 1 : 0;
    head[i] = h ? 1 : 0;
}

__global__ void k_emit_loops(const int* __restrict__ efrom, const int* __restrict__ rep, const int* __restrict__ dist,
                             const int* __restrict__ voff, const int* __restrict__ lid, int64_t n, const float* __restrict__ vx,
                             const float* __restrict__ vy, const float* __restrict__ vz, int64_t vs,
                             const int4* __restrict__ qv, float scalef, BVert* __restrict__ bv, int* __restrict__ loop_off) {
    int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n) return;
    int r = rep[i];
    int pos = dist[r] - dist[i];
    int slot = voff[r] + pos;
    if (r < 0 || r >= n || pos < 0 || slot < 0 || slot >= n) return;   // unreachable for a balanced chain
    int v = efrom[i];
    BVert b;
    b.x = vx[(int64_t)v * vs] * scalef;
    b.y = vy[(int64_t)v * vs] * scalef;
    b.z = vz[(int64_t)v * vs] * scalef;
    int4 q = qv[v];
    b.qx = q.x;
    b.qy = q.y;
    b.pad0 = v;
    b.pad1 = 0;
    b.loop = lid[r];   // lid is the loop index at each loop's representative only
    bv[slot] = b;
    if (r == (int)i) loop_off[lid[i]] = voff[i];
}

// ---------------------------------------------------------------- boundary chunks
// The grid kernels decide per chunk of the boundary whether it is near a block of
// columns, so a chunk should be compact: loops are taken along a Hilbert curve
// by their first vertex, and a chunk holds kChunk = 8 chained vertices (7 edges).
// Fewer vertices per chunk cost more repeated end vertices (8/7 of the vertex work,
// 4/3 at four), more make the chunks wide: on the 64 loops of the 1.05M-triangle
// opened spheres a chunk of 16 has 2.1 times the edges near a block that single
// edges would have, one of 8 1.5 times.  A loop of m edges is m / 7 whole chunks
// and a rest of m % 7 edges: a chunk of its own, or half a chunk if at most three
// (a missing triangle's loop exactly fills a half).

__device__ __forceinline__ uint32_t loop_key(const BVert& b, const QGrid& g) {
    const double z = fmin(fmax((double)b.z - g.lo[2] * g.scale, 0.0), (double)kQMax);
    return hilbert_key((uint32_t)b.qx >> 20, (uint32_t)b.qy >> 20, (uint32_t)z >> 20);
}

__global__ void k_loop_keys(const BVert* __restrict__ bv, const int* __restrict__ loop_off, int64_t nl, QGrid g,
                            uint32_t* __restrict__ key, int* __restrict__ idx) {
    int64_t l = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (l >= nl) return;
    key[l] = loop_key(bv[loop_off[l]], g);
    idx[l] = (int)l;
}

// per loop, in that order: whole chunks (piece[i]), halves (piece[nl + i]) and edges
// (piece[2 nl + i]); one scan makes prefix sums of all three, off
__global__ void k_loop_pieces(const int* __restrict__ loop_off, const int* __restrict__ order, int64_t nl,
                              int* __restrict__ rank, int* __restrict__ piece) {
    int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i > nl) return;
    if (i == nl) {
        piece[3 * nl] = 0;   // its prefix sum is the total
        return;
    }
    const int l = order[i], m = loop_off[l + 1] - loop_off[l], r = m % (kChunk - 1);
    rank[l] = (int)i;
    piece[i] = m / (kChunk - 1) + (r > 3);
    piece[nl + i] = r >= 1 && r <= 3;
    piece[2 * nl + i] = m;
}

// Edges per lowest cluster: about what two expansions cost.  2 M points against 63 k edges
// (torus of small loops) 7.6 ms, with 14 edges 7.9, 42 8.0, 60 9.9.
constexpr int kLeafEdges = 28;

// Clusters: loops whose first edge falls into the same `size` edges of the order.
__global__ void k_cluster_heads(const int* __restrict__ off, int64_t nl, int size, int* __restrict__ head) {
    int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i > nl) return;
    const int64_t e0 = off[2 * nl];
    head[i] = i < nl && (i == 0 || (off[2 * nl + i] - e0) / size != (off[2 * nl + i - 1] - e0) / size);
}

// hid: exclusive prefix sums of head; first[c]: rank of cluster c's first loop
__global__ void k_cluster_first(const int* __restrict__ head, const int* __restrict__ hid, int64_t nl, int most,
                                int* __restrict__ cid, int* __restrict__ first) {
    int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= nl) return;
    const int c = hid[i] + head[i] - 1;
    cid[i] = c;
    if (head[i] && c >= 0 && c < most) first[c] = (int)i;
}

// chunks per cluster (0 past the last)
__global__ void k_cluster_chunks(const int* __restrict__ hid, const int* __restrict__ first, const int* __restrict__ off,
                                 int64_t nl, int most, int* __restrict__ count, int* __restrict__ clusters) {
    int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c > most) return;
    const int n = hid[nl];
    if (c == most) *clusters = n;
    int k = 0;
    if (c < n && c < most) {
        const int64_t r0 = first[c], r1 = c + 1 < n ? first[c + 1] : nl;
        k = off[r1] - off[r0] + (off[nl + r1] - off[nl + r0] + 1) / 2;
    }
    count[c] = k;
}

// All of the above for few loops in one workgroup: sorted in LDS, scanned by waves, with
// the same results.  The launches it saves (25) cost as much as the rest of a small mesh's
// boundary.
constexpr int kFewLoops = 2048, kPlanThreads = 1024;

// exclusive prefix sums of a pair of values per thread over the workgroup, and the total
__device__ int plan_scan(int a, int b, int* first, int* second) {
    __shared__ int wsum[kPlanThreads / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int t = a + b;
    for (int d = 1; d < 64; d <<= 1) {
        const int o = __shfl_up(t, d);
        if (lane >= d) t += o;
    }
    __syncthreads();   // wsum may still be read from the call before
    if (lane == 63) wsum[wave] = t;
    __syncthreads();
    int before = 0, total = 0;
    for (int k = 0; k < kPlanThreads / 64; ++k) {
        if (k < wave) before += wsum[k];
        total += wsum[k];
    }
    *first = before + t - a - b;
    *second = *first + a;
    return total;
}

__global__ __launch_bounds__(kPlanThreads) void k_plan_loops(const BVert* __restrict__ bv, const int* __restrict__ loop_off,
                                                            int nl, QGrid g, int size, int most, int* __restrict__ order,
                                                            int* __restrict__ rank, int* __restrict__ off,
                                                            int* __restrict__ cid, int* __restrict__ first,
                                                            int* __restrict__ count, int* __restrict__ base) {
    __shared__ uint64_t key[kFewLoops];
    __shared__ int start[kFewLoops + 1], whole[kFewLoops + 1], half[kFewLoops + 1];   // by cluster, and by rank
    const int t = threadIdx.x;
    int n2 = 2;
    while (n2 < nl) n2 *= 2;
    for (int l = t; l < n2; l += kPlanThreads)
        key[l] = l < nl ? ((uint64_t)loop_key(bv[loop_off[l]], g) << 32) | (unsigned)l : ~0ull;
    for (int k = 2; k <= n2; k *= 2) {
        for (int j = k / 2; j > 0; j /= 2) {
            __syncthreads();
            for (int p = t; p < n2 / 2; p += kPlanThreads) {
                const int a = 2 * p - (p & (j - 1)), b = a + j;   // pairs j apart
                const uint64_t x = key[a], y = key[b];
                if ((x > y) == ((a & k) == 0)) {
                    key[a] = y;
                    key[b] = x;
                }
            }
        }
    }
    __syncthreads();
    // thread t: loops of rank 2t and 2t + 1
    int w[2] = {0, 0}, h[2] = {0, 0}, e[2] = {0, 0};
    for (int s = 0; s < 2; ++s) {
        const int i = 2 * t + s;
        if (i >= nl) continue;
        const int l = (int)(unsigned)key[i], m = loop_off[l + 1] - loop_off[l], r = m % (kChunk - 1);
        order[i] = l;
        rank[l] = i;
        w[s] = m / (kChunk - 1) + (r > 3);
        h[s] = r >= 1 && r <= 3;
        e[s] = m;
    }
    int pw[2], ph[2], pe[2], pc[2];
    const int tw = plan_scan(w[0], w[1], pw, pw + 1), th = plan_scan(h[0], h[1], ph, ph + 1);
    plan_scan(e[0], e[1], pe, pe + 1);
    int head[2] = {0, 0};
    for (int s = 0; s < 2; ++s) {
        const int i = 2 * t + s;
        if (i >= nl) continue;
        off[i] = pw[s];
        off[nl + i] = tw + ph[s];
        off[2 * nl + i] = tw + th + pe[s];
        whole[i] = pw[s];
        half[i] = ph[s];
        int before = 0;   // edges of the loop before
        if (i > 0) {
            const int l = (int)(unsigned)key[i - 1];
            before = loop_off[l + 1] - loop_off[l];
        }
        head[s] = i == 0 || pe[s] / size != (pe[s] - before) / size;
    }
    if (t == 0) {
        off[3 * nl] = tw + th + loop_off[nl];
        whole[nl] = tw;
        half[nl] = th;
    }
    const int n = plan_scan(head[0], head[1], pc, pc + 1);
    for (int s = 0; s < 2; ++s) {
        const int i = 2 * t + s;
        if (i >= nl) continue;
        const int c = pc[s] + head[s] - 1;
        cid[i] = c;
        if (head[s] && c < most) {
            first[c] = i;
            start[c] = i;
        }
    }
    __syncthreads();
    int cn[2] = {0, 0}, pb[2];
    for (int s = 0; s < 2; ++s) {
        const int c = 2 * t + s;
        if (c >= n || c >= most) continue;
        const int r0 = start[c], r1 = c + 1 < n ? start[c + 1] : nl;
        cn[s] = whole[r1] - whole[r0] + (half[r1] - half[r0] + 1) / 2;
        count[c] = cn[s];
    }
    const int total = plan_scan(cn[0], cn[1], pb, pb + 1);
    for (int s = 0; s < 2; ++s)
        if (2 * t + s < most) base[2 * t + s] = pb[s];
    if (t == 0) {
        base[most] = total;
        base[most + 1] = n;
    }
}

// entry of path position k of the loop of rank i (k / 7-th piece), in its cluster's chunks:
// the whole ones first, then the halves
struct ChainPlan {
    const int *rank, *cid, *first, *off, *base;
    int64_t nl;
    int n;   // clusters
};

__device__ __forceinline__ int64_t chain_slot(const ChainPlan& p, int64_t i, int m, int k) {
    const int s = k / (kChunk - 1), whole = m / (kChunk - 1), r = m % (kChunk - 1);
    const int c = p.cid[i];
    const int64_t r0 = p.first[c], r1 = c + 1 < p.n ? p.first[c + 1] : p.nl;
    if (s < whole || r > 3) return ((int64_t)p.base[c] + p.off[i] - p.off[r0] + s) * kChunk;
    return ((int64_t)p.base[c] + p.off[r1] - p.off[r0]) * kChunk +
           ((int64_t)p.off[p.nl + i] - p.off[p.nl + r0]) * (kChunk / 2);
}

__global__ void k_emit_chain(const BVert* __restrict__ bv, const int* __restrict__ loop_off, ChainPlan p, int64_t nb,
                             int64_t nentry, CVert* __restrict__ chain, GVertex* __restrict__ gchain) {
    int64_t j = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (j >= nb) return;
    BVert b = bv[j];
    const int l = b.loop, b0 = loop_off[l], m = loop_off[l + 1] - b0, k = (int)(j - b0);
    const int64_t i = p.rank[l];
    auto put = [&](int64_t e, const BVert& v, int flags) {
        if (e < 0 || e >= nentry) return;
        CVert w;
        w.z = v.z;
        w.qx = v.qx;
        w.qy = v.qy;
        w.ex = w.ey = 0.f;   // with the chunk's next vertex, below
        w.m = 0.f;
        w.flags = flags;
        w.none = (flags & kChainEdge) ? 0.f : 0x1p27f;
        chain[e] = w;
        gchain[e] = {v.x, v.y, v.z, w.flags};
    };
    const int64_t base = chain_slot(p, i, m, k);
    const int s = k % (kChunk - 1);
    const int64_t before = s == 0 && k > 0 ? chain_slot(p, i, m, k - 1) : -1;   // the piece before
    put(base + s, b, kChainEdge | kChainValid | (m == 3 && k == 0 ? kChainTri : 0) |
                         (before >= 0 && before + kChunk == base ? kChainCont : 0));
    if (before >= 0) put(before + kChunk - 1, b, kChainValid);   // its end
    if (k == m - 1) {   // the closing vertex, and the rest of its piece
        const int r = m % (kChunk - 1);
        const int end = r == 0 ? kChunk : (r > 3 ? kChunk : kChunk / 2);
        const BVert c = bv[b0];
        for (int e = s + 1; e < end; ++e) put(base + e, c, kChainValid | (e == s + 1 && k == s && m >= 3 ? kChainClose : 0));
    }
}

// boxes of the chunks and their edges; entries that no piece filled (half of a cluster's
// last chunk) repeat the chunk's first vertex
__global__ void k_chunk_boxes(int64_t nchunk, CVert* __restrict__ chain, GVertex* __restrict__ gchain,
                              int4* __restrict__ box, unsigned long long* __restrict__ width) {
    int64_t c = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (c >= nchunk) return;
    CVert* v = chain + c * kChunk;
    GVertex* gv = gchain + c * kChunk;
    CVert f = v[0];
    f.ex = f.ey = f.m = 0.f;
    f.flags = kChainValid;
    f.none = 0x1p27f;
    GVertex gf = gv[0];
    gf.flags = f.flags;
    int4 b = make_int4(f.qx, f.qx, f.qy, f.qy);
    for (int e = 1; e < kChunk; ++e) {
        if (!(v[e].flags & kChainValid)) {
            v[e] = f;
            gv[e] = gf;
            continue;
        }
        b.x = min(b.x, v[e].qx);
        b.y = max(b.y, v[e].qx);
        b.z = min(b.z, v[e].qy);
        b.w = max(b.w, v[e].qy);
        if (v[e - 1].flags & kChainEdge) {
            const float ex = (float)(v[e].qx - v[e - 1].qx) * 0x1p-18f, ey = (float)(v[e].qy - v[e - 1].qy) * 0x1p-18f;
            v[e - 1].ex = ex;
            v[e - 1].ey = ey;
            v[e - 1].m = fmaxf(0x1p-20f, ex * ex + ey * ey);
        }
    }
    box[c] = b;
    atomicAdd(width, (unsigned long long)(b.y - b.x) + (unsigned long long)(b.w - b.z));
}

// ---------------------------------------------------------------- cluster expansions
// Away from its loops, and where the vertical ray misses a surface spanned by them, a
// cluster's boundary sum is half the loops' solid angle, a harmonic function of the
// query.  With p = (query - centre) / radius and u = p / |p|^2 it is
//
//     S = |u| sum_{l=1..10} sum_{m=0..l}  Re( conj(W_lm) Q_lm(u) ),
//     W_lm = -c_lm / 2  oint  -(x cross grad Q_lm) / (l + 1) . dx,
//
// Q_lm = q_lm(z, r^2) (x + i y)^m the solid harmonics with q_mm = 1, q_{m+1,m} = z and
// q_{l+1,m} = z q_lm - (l^2 - m^2)/(4 l^2 - 1) r^2 q_{l-1,m}, and
// c_lm = (2 - [m = 0]) ((2l - 1)!!)^2 / ((l + m)! (l - m)!) the weights of 1/|x - p|'s
// expansion.  (The line integral is the surface integral of n . grad Q_lm: the curl of
// x cross grad Q is -(l + 1) grad Q for a harmonic Q of degree l.)  Their gradients are
// solid harmonics of a degree less, with g the value of q on the axis (g_{m,m} = 1):
//     d/dz Q_lm = (l - m) g_lm / g_{l-1,m} Q_{l-1,m},
//     (d/dx + i d/dy) Q_lm = -(l - m)(l - m - 1) / (2 (m + 1)) g_lm / g_{l-1,m+1} Q_{l-1,m+1},
//     (d/dx - i d/dy) Q_lm = 2 m g_lm / g_{l-1,m-1} Q_{l-1,m-1}   (m > 0).
//
// Truncation at degree P, with A the area of triangle fans spanning the loops, a the
// radius and t = a / distance:  at most  A / a^2 (P + 1) t^(P+2) / (1 - t)^2 / 2.  The
// distances from which a degree is taken are those where that bound is kPoleBound.  Errors
// there, as parts of the bound at degree 10, 6 and 4 (worst of some hundred points around
// clusters of 27 edges, series and solid angle in FP64 on the host): triangles of one
// orientation on a disc 1/57, 1/16, 1/8; random ones 1/24, 1/9, 1/6; all at two opposite
// ends of the cluster 1/12, 1/3, 1/2, the most found: 2.4e-6, 1.7e-6 and 4.4e-7 of solid
// angle, in w the 4 pi-th part.  The bound scales with the area, so a pile of duplicated
// triangles only moves dmin out.
// For degree kPoles, kPolesMid, kPolesLow: so that FP32 results are nearer to FP64 than the sum
// of all edges with an arctangent each was (relative: 48 ellipsoid soups 8.3e-8 against 1.2e-7,
// torus of 63 k edges 1.1e-7 against 3.5e-7; largest 5e-7 against 7e-7).  With 1e-4, 1e-5, 3e-6
// 2 M points take 7.6 ms instead of 8.4, but the soups' error is 1.4e-7.
constexpr double kPoleBound[3] = {3e-5, 5e-6, 1e-6};
constexpr int kPairs = kPoles * (kPoles + 3) / 2;   // (l, m) with l >= 1
constexpr int kSmallCluster = 16, kHugeCluster = 4096;   // chunks

// the factors above by (l, m), made by the compiler
struct PoleTable {
    double z[kPoles + 1][kPoles + 1], up[kPoles + 1][kPoles + 1], down[kPoles + 1][kPoles + 1];   // of the gradients
    double b[kPoles + 1][kPoles + 1];   // (l^2 - m^2) / (4 l^2 - 1)
    double f[kPoles + 1][kPoles + 1];   // (2l - 1)!! / ((l - m)! (l + m)!)
    double w[kPoles + 1][kPoles + 1];   // -c_lm / (2 (l + 1))
    double s[kPoles + 1][kPoles + 1];   // -(2 - [m = 0]) (2l - 1)!! / 2

    constexpr PoleTable() : z(), up(), down(), b(), f(), w(), s() {
        double g[kPoles + 1][kPoles + 2] = {};
        double odd = 1.0, fact[2 * kPoles + 1] = {1.0};
        for (int k = 1; k <= 2 * kPoles; ++k) fact[k] = fact[k - 1] * k;
        for (int l = 0; l <= kPoles; ++l) {
            if (l > 0) odd *= 2 * l - 1;
            for (int m = 0; m <= l; ++m) {
                const double eps = m == 0 ? 1.0 : 2.0;
                b[l][m] = (double)(l * l - m * m) / (double)(4 * l * l - 1);
                g[l][m] = l - m < 2 ? 1.0 : g[l - 1][m] - b[l - 1][m] * g[l - 2][m];
                f[l][m] = odd / (fact[l - m] * fact[l + m]);
                w[l][m] = -0.5 / (l + 1) * eps * odd * f[l][m];
                s[l][m] = -0.5 * eps * odd;
                if (m < l) z[l][m] = (l - m) * g[l][m] / g[l - 1][m];
                if (m + 1 < l) up[l][m] = -0.5 * (l - m) * (l - m - 1) / (m + 1) * g[l][m] / g[l - 1][m + 1];
                if (m > 0) down[l][m] = 2.0 * m * g[l][m] / g[l - 1][m - 1];
            }
        }
    }
};
constexpr PoleTable kPole;

struct Cplx {
    double re, im;
};

__device__ __forceinline__ Cplx operator*(const Cplx& a, const Cplx& b) {
    return {fma(a.re, b.re, -(a.im * b.im)), fma(a.re, b.im, a.im * b.re)};
}

// position of (l, m) among the pairs, m outermost as in the moments
__host__ __device__ constexpr int pole_pair(int l, int m) {
    int o = 0;
    for (int k = 0; k < m; ++k) o += kPoles - (k > 1 ? k : 1) + 1;
    return o + l - (m > 1 ? m : 1);
}

// position of W_lm's real (part 0) or imaginary part in a cluster's moments
__host__ __device__ constexpr int pole_slot(int l, int m, int part) {
    return l * l - 1 + (m == 0 ? 0 : 2 * m - 1 + part);
}

// The distances that are tried, in radii: from 2 up by 2% to a million.
constexpr int kReaches = 664;
struct ReachTable {
    double d[kReaches];
    constexpr ReachTable() : d() {
        d[0] = 2.0;
        for (int i = 1; i < kReaches; ++i) d[i] = d[i - 1] * 1.02;
    }
};
constexpr ReachTable kReach;
static_assert(kReach.d[kReaches - 2] < 1e6 && kReach.d[kReaches - 1] >= 1e6, "the last distance is the first of a million");

// squared distances from which the truncation bound holds for each degree; never: none.  The
// bound falls with the distance: bisected (tried in turn, 150 to 300 of 60 FP64 operations
// each, this took 20 us of a cluster's 45).
__device__ void cluster_reach(double radius, double area, bool never, float* far2) {
    const double rel = area / (radius * radius);
    const int degree[3] = {kPoles, kPolesMid, kPolesLow};
    const double bound[3] = {kPoleBound[0], kPoleBound[1], kPoleBound[2]};
    int lo = 0;   // the least that is left to try
    for (int i = 0; i < 3; ++i) {
        const int P = degree[i];
        int hi = kReaches - 1;
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            const double t = 1.0 / kReach.d[mid];
            double b = 0.5 * rel * (P + 1) / ((1.0 - t) * (1.0 - t));
            for (int k = 0; k < P + 2; ++k) b *= t;
            if (b <= bound[i]) hi = mid;
            else lo = mid + 1;
        }
        const double d = kReach.d[lo];
        far2[i] = never ? INFINITY : (float)fmin(d * radius * d * radius, 1e38);
    }
}

__device__ __forceinline__ double wave_sum(double x) {
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o);
    return x;
}

struct Levels {
    int first[kLevels + 1];   // each level's first cluster, and the end of the last
};

// Clusters of the lowest level (and the level table behind all clusters): box, centre, radius and spanned area.  One wave each.
__global__ __launch_bounds__(64) void k_cluster_frames(const BVert* __restrict__ bv, const int* __restrict__ loop_off,
                                                      const int* __restrict__ order, ChainPlan p,
                                                      const int* __restrict__ count, Levels levels,
                                                      Cluster* __restrict__ out) {
    const int c = blockIdx.x, lane = threadIdx.x;
    if (c == 0 && lane <= kLevels) reinterpret_cast<int*>(out + levels.first[kLevels])[lane] = levels.first[lane];
    const int r0 = p.first[c], r1 = c + 1 < p.n ? p.first[c + 1] : (int)p.nl;
    // an overlong loop's moments would keep one workgroup busy too long: never far, and no frame
    // either (a million edges: two passes of 16,000 steps of one wave)
    if (count[c] > kHugeCluster || p.n < kFewClusters) {
        if (lane > 0) return;
        const BVert v = bv[loop_off[order[r0]]];
        Cluster k{};
        k.x = v.x;
        k.y = v.y;
        k.z = k.ztop = k.zlow = v.z;
        k.inva = 1.0f;
        k.far2[0] = k.far2[1] = k.far2[2] = INFINITY;
        k.xlo = k.xhi = v.qx;
        k.ylo = k.yhi = v.qy;
        k.first = p.base[c];
        k.count = -count[c];
        out[c] = k;
        return;
    }
    // a wave per loop, or of short loops one per lane
    const bool shorts = p.off[2 * p.nl + r1] - p.off[2 * p.nl + r0] <= 8 * (r1 - r0);
    const int rl = shorts ? lane : 0, rstep = shorts ? 64 : 1, jl = shorts ? 0 : lane, jstep = shorts ? 1 : 64;
    float lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
    int qlo[2] = {0x7fffffff, 0x7fffffff}, qhi[2] = {-1, -1};
    double area = 0.0;
    for (int r = r0 + rl; r < r1; r += rstep) {
        const int b0 = loop_off[order[r]], b1 = loop_off[order[r] + 1];
        const BVert o = bv[b0];
        for (int j = b0 + jl; j < b1; j += jstep) {
            const BVert v = bv[j], w = bv[j + 1 < b1 ? j + 1 : b0];
            const float q[3] = {v.x, v.y, v.z};
            for (int a = 0; a < 3; ++a) {
                lo[a] = fminf(lo[a], q[a]);
                hi[a] = fmaxf(hi[a], q[a]);
            }
            qlo[0] = min(qlo[0], v.qx);
            qhi[0] = max(qhi[0], v.qx);
            qlo[1] = min(qlo[1], v.qy);
            qhi[1] = max(qhi[1], v.qy);
            const double a0 = (double)v.x - o.x, a1 = (double)v.y - o.y, a2 = (double)v.z - o.z;
            const double e0 = (double)w.x - o.x, e1 = (double)w.y - o.y, e2 = (double)w.z - o.z;
            const double n0 = a1 * e2 - a2 * e1, n1 = a2 * e0 - a0 * e2, n2 = a0 * e1 - a1 * e0;
            area += 0.5 * sqrt(n0 * n0 + n1 * n1 + n2 * n2);
        }
    }
    for (int s = 32; s > 0; s >>= 1) {
        for (int a = 0; a < 3; ++a) {
            lo[a] = fminf(lo[a], __shfl_xor(lo[a], s));
            hi[a] = fmaxf(hi[a], __shfl_xor(hi[a], s));
        }
        for (int a = 0; a < 2; ++a) {
            qlo[a] = min(qlo[a], __shfl_xor(qlo[a], s));
            qhi[a] = max(qhi[a], __shfl_xor(qhi[a], s));
        }
    }
    area = wave_sum(area);
    const float cx = 0.5f * lo[0] + 0.5f * hi[0], cy = 0.5f * lo[1] + 0.5f * hi[1], cz = 0.5f * lo[2] + 0.5f * hi[2];
    double rad2 = 0.0;
    for (int r = r0 + rl; r < r1; r += rstep) {
        const int b0 = loop_off[order[r]], b1 = loop_off[order[r] + 1];
        for (int j = b0 + jl; j < b1; j += jstep) {
            const double x = (double)bv[j].x - cx, y = (double)bv[j].y - cy, z = (double)bv[j].z - cz;
            rad2 = fmax(rad2, x * x + y * y + z * z);
        }
    }
    for (int s = 32; s > 0; s >>= 1) rad2 = fmax(rad2, __shfl_xor(rad2, s));
    if (lane > 0) return;
    const double radius = fmax(sqrt(rad2) * (1.0 + 1e-6), 0.5);
    Cluster k;
    k.x = cx;
    k.y = cy;
    k.z = cz;
    k.inva = (float)(1.0 / radius);
    k.ztop = hi[2];
    k.zlow = lo[2];
    k.xlo = qlo[0];
    k.xhi = qhi[0];
    k.ylo = qlo[1];
    k.yhi = qhi[1];
    k.first = p.base[c];
    k.count = -count[c];
    k.area = (float)area;
    cluster_reach(radius, area, false, k.far2);
    out[c] = k;
}

// Their moments.  Lanes take (edge, Gauss point) samples (six points integrate the
// polynomial exactly) and keep all coefficients in registers: about 14 operations per
// sample and coefficient, against some 300 for a lane that forms one coefficient's
// harmonics anew.  One wave per small cluster, a workgroup of eight per larger one, each
// for orders M0 to M1 (all of them at once take 240 registers for the sums alone).
template <int WAVES, int M0, int M1>
__device__ __forceinline__ void cluster_moments(const GVertex* __restrict__ gchain, const Cluster& K, int nch,
                                                float* __restrict__ out, double (*part)[kMoments]) {
    const int t0 = threadIdx.x;
    constexpr int kFirst = pole_pair(M0 > 0 ? M0 : 1, M0), kCount = pole_pair(kPoles, M1) + 1 - kFirst;
    const double gx[3] = {0.2386191860831969, 0.6612093864662645, 0.9324695142031521};
    const double gw[3] = {0.4679139345726910, 0.3607615730481386, 0.1713244923791704};
    double re[kCount], im[kCount];
#pragma unroll
    for (int i = 0; i < kCount; ++i) re[i] = im[i] = 0.0;
    constexpr int kSamples = 6 * (kChunk - 1);
    const int total = nch * kSamples;   // at most kHugeCluster chunks
    for (int base = 0; base < total; base += 64 * WAVES) {
        const int t = min(base + t0, total - 1), ch = t / kSamples, r = t % kSamples, e = r / 6, g = r % 6;
        const GVertex v = gchain[(size_t)(K.first + ch) * kChunk + e], w = gchain[(size_t)(K.first + ch) * kChunk + e + 1];
        const double ia = (double)K.inva;
        const double gn = g % 3 == 0 ? gx[0] : g % 3 == 1 ? gx[1] : gx[2], s = 0.5 + 0.5 * (g < 3 ? gn : -gn);
        // no edge, or no sample: no weight
        const double wt = (v.flags & kChainEdge) && base + t0 < total
                              ? 0.5 * (g % 3 == 0 ? gw[0] : g % 3 == 1 ? gw[1] : gw[2]) : 0.0;
        const double ex = ((double)w.x - v.x) * ia, ey = ((double)w.y - v.y) * ia, ez = ((double)w.z - v.z) * ia;
        const double x = fma(s, ex, ((double)v.x - K.x) * ia), y = fma(s, ey, ((double)v.y - K.y) * ia);
        const double z = fma(s, ez, ((double)v.z - K.z) * ia), r2 = fma(x, x, fma(y, y, z * z));
        // wt (x cross e): -(x cross grad) . e = grad . (x cross e)
        const Cplx V = {wt * fma(y, ez, -(z * ey)), wt * fma(z, ex, -(x * ez))}, Vc = {V.re, -V.im};
        const double vz = wt * fma(x, ey, -(y * ex));
        Cplx q[kPoles], qp[kPoles];   // Q_{l-1,m} and Q_{l-2,m}
        Cplx xy = {1.0, 0.0};         // (x + i y)^{l-1}
#pragma unroll
        for (int l = 1; l <= kPoles; ++l) {
            // to degree l - 1
#pragma unroll
            for (int m = 0; m < l; ++m) {
                if (m == l - 1) {
                    q[m] = xy;
                    qp[m] = {0.0, 0.0};
                } else {
                    const int k = l - 2;
                    const double b = k > m ? kPole.b[k > 0 ? k : 0][m] * r2 : 0.0;
                    const Cplx n = {fma(z, q[m].re, -(b * qp[m].re)), fma(z, q[m].im, -(b * qp[m].im))};
                    qp[m] = q[m];
                    q[m] = n;
                }
            }
            xy = xy * Cplx{x, y};
#pragma unroll
            for (int m = M0; m <= (l < M1 ? l : M1); ++m) {
                const int i = pole_pair(l, m) - kFirst;
                const double o = m == 0 ? 1.0 : 0.5;
                if (m < l) {
                    const double f = kPole.z[l][m];
                    re[i] = fma(f * vz, q[m].re, re[i]);
                    if (m > 0) im[i] = fma(f * vz, q[m].im, im[i]);
                }
                if (m + 1 < l) {
                    const double f = o * kPole.up[l][m];
                    const Cplx a = q[m + 1] * Vc;
                    re[i] = fma(f, a.re, re[i]);
                    if (m > 0) im[i] = fma(f, a.im, im[i]);
                }
                if (m > 0) {
                    const double f = 0.5 * kPole.down[l][m];
                    const Cplx a = q[m - 1] * V;
                    re[i] = fma(f, a.re, re[i]);
                    im[i] = fma(f, a.im, im[i]);
                }
            }
        }
    }
    const int lane = t0 & 63, wave = t0 >> 6;
#pragma unroll
    for (int m = M0; m <= M1; ++m) {
#pragma unroll
        for (int l = m > 1 ? m : 1; l <= kPoles; ++l) {
            const double f = kPole.w[l][m];
            const int i = pole_pair(l, m) - kFirst;
            const double a = f * wave_sum(re[i]), b = m > 0 ? f * wave_sum(im[i]) : 0.0;
            if (lane == 0) {
                part[wave][pole_slot(l, m, 0)] = a;
                if (m > 0) part[wave][pole_slot(l, m, 1)] = b;
            }
        }
    }
    __syncthreads();
    for (int j = t0; j < kMoments; j += 64 * WAVES) {
        int l = 1;
        while (l * (l + 2) <= j) ++l;
        const int m = (j - l * l + 2) / 2;   // order of slot j
        if (m < M0 || m > M1) continue;
        double s = 0.0;
        for (int k = 0; k < WAVES; ++k) s += part[k][j];
        out[j] = (float)s;
    }
}

template <int WAVES>
__global__ __launch_bounds__(64 * WAVES) void k_cluster_moments(const GVertex* __restrict__ gchain,
                                                               const Cluster* __restrict__ clusters,
                                                               float* __restrict__ moments) {
    __shared__ double part[WAVES][kMoments];
    const Cluster K = clusters[blockIdx.x];
    const int nch = -K.count;
    if ((nch <= kSmallCluster) != (WAVES == 1) || nch > kHugeCluster) return;
    float* out = moments + (size_t)blockIdx.x * kMoments;
    if (blockIdx.y == 0) cluster_moments<WAVES, 0, 2>(gchain, K, nch, out, part);
    else cluster_moments<WAVES, 3, kPoles>(gchain, K, nch, out, part);
}


// A level from the one below: the children's expansions moved to the parent's centre.
// With S_lm = f_lm Q_lm the translation is S_lm(x + t) = sum S_l'm'(x) S_{l-l',m-m'}(t)
// (m' from -l' to l', S_l,-m = (-1)^m conj S_lm), and W_lm = -(2 - [m = 0]) (2l - 1)!! / 2
// times the surface integral of n . grad S_lm, which scales with radius^(l + 1).
// One workgroup per parent, a thread per coefficient and child.
constexpr int kMergeThreads = (kFan * kPairs + 63) / 64 * 64;

__global__ __launch_bounds__(kMergeThreads) void k_cluster_merge(int first, int count, int child_first, int child_count,
                                                               double ox, double oy, Cluster* __restrict__ clusters,
                                                               float* __restrict__ moments) {
    __shared__ Cplx mu[kFan][kPairs];
    __shared__ Cplx sh[kFan][kPoles * (kPoles + 1) / 2];   // S_lm(t), l < kPoles
    __shared__ double rho[kFan][kPoles + 2];
    __shared__ Cplx part[kFan][kPairs];
    const int P = blockIdx.x, t = threadIdx.x;
    if (P >= count) return;
    const int c0 = child_first + P * kFan, n = min(kFan, child_count - P * kFan);
    Cluster K = clusters[c0];
    for (int c = 1; c < n; ++c) {
        const Cluster k = clusters[c0 + c];
        K.xlo = min(K.xlo, k.xlo);
        K.xhi = max(K.xhi, k.xhi);
        K.ylo = min(K.ylo, k.ylo);
        K.yhi = max(K.yhi, k.yhi);
        K.zlow = fminf(K.zlow, k.zlow);
        K.ztop = fmaxf(K.ztop, k.ztop);
        K.area += k.area;
        K.far2[0] = fmaxf(K.far2[0], k.far2[0]);
    }
    const bool never = K.far2[0] == INFINITY;
    // centre and radius from the box; the children's spheres if those end sooner
    K.x = (float)(0.5 * ((double)K.xlo + K.xhi) + ox);
    K.y = (float)(0.5 * ((double)K.ylo + K.yhi) + oy);
    K.z = (float)(0.5 * ((double)K.zlow + K.ztop));
    double ra = 0.0;
    for (int c = 0; c < n; ++c) {
        const Cluster k = clusters[c0 + c];
        const double x = (double)k.x - K.x, y = (double)k.y - K.y, z = (double)k.z - K.z;
        ra = fmax(ra, sqrt(x * x + y * y + z * z) + 1.0 / k.inva);
    }
    {
        // the stored centre is rounded to FP32 (2^-24 of the coordinate)
        const double x = 0.5 * ((double)K.xhi - K.xlo) + 1.0 + 1e-7 * fabs((double)K.x);
        const double y = 0.5 * ((double)K.yhi - K.ylo) + 1.0 + 1e-7 * fabs((double)K.y);
        const double z = 0.5 * ((double)K.ztop - K.zlow) + 1.0 + 1e-7 * fabs((double)K.z);
        ra = fmax(fmin(ra, sqrt(x * x + y * y + z * z)) * (1.0 + 1e-6), 0.5);
    }
    K.inva = (float)(1.0 / ra);
    cluster_reach(ra, K.area, never, K.far2);
    K.first = c0;
    K.count = n;
    if (t == 0) clusters[first + P] = K;
    if (never) return;
    for (int j = t; j < n * kPairs; j += kMergeThreads) {
        const int c = j / kPairs, i = j % kPairs;
        int m = 0, l = i + 1;
        while (l > kPoles) {   // pairs by m
            l -= kPoles - (m > 1 ? m : 1) + 1;
            ++m;
            l += (m > 1 ? m : 1) - (m > 2 ? m - 1 : 1);
        }
        const float* W = moments + (size_t)(c0 + c) * kMoments;
        const double f = 1.0 / kPole.s[l][m];
        mu[c][i] = {f * W[pole_slot(l, m, 0)], m > 0 ? f * W[pole_slot(l, m, 1)] : 0.0};
    }
    const double ia = (double)K.inva;
    for (int j = t; j < n * kPoles; j += kMergeThreads) {   // child, m
        const int c = j / kPoles, m = j % kPoles;
        const Cluster k = clusters[c0 + c];
        const double x = ((double)k.x - K.x) * ia, y = ((double)k.y - K.y) * ia, z = ((double)k.z - K.z) * ia;
        const double r2 = x * x + y * y + z * z;
        Cplx e = {1.0, 0.0};
        for (int i = 0; i < m; ++i) e = e * Cplx{x, y};
        double q0 = 0.0, q1 = 1.0;
        for (int l = m; l < kPoles; ++l) {
            const double f = kPole.f[l][m] * q1;
            sh[c][l * (l + 1) / 2 + m] = {f * e.re, f * e.im};
            const double nq = z * q1 - (l > m ? kPole.b[l][m] * r2 * q0 : 0.0);
            q0 = q1;
            q1 = nq;
        }
        if (m == 0) {
            const double h = ia / (double)k.inva;   // the child's radius in the parent's
            double pw = h;
            for (int l = 0; l <= kPoles; ++l) {
                rho[c][l] = pw;
                pw *= h;
            }
        }
    }
    __syncthreads();
    const int c = t / kPairs, i = t % kPairs;
    int m = 0, l = i + 1;
    while (l > kPoles) {
        l -= kPoles - (m > 1 ? m : 1) + 1;
        ++m;
        l += (m > 1 ? m : 1) - (m > 2 ? m - 1 : 1);
    }
    if (c < n) {
        Cplx sum = {0.0, 0.0};
        int row = 0;   // pole_pair(a, b) - a for the b at hand
        for (int b = 0; b <= l; ++b) {   // orders b and -b of the child
            row = b < 2 ? b * kPoles - 1 : row + kPoles - b + 1;
            for (int a = b > 1 ? b : 1; a <= l; ++a) {
                const Cplx u = mu[c][row + a];
                const double r = rho[c][a];
                for (int s = b == 0 ? 1 : 0; s < 2; ++s) {   // s = 1: order b, s = 0: -b
                    const int d = s ? m - b : m + b, ad = d < 0 ? -d : d;
                    if (ad > l - a) continue;
                    Cplx x = u, v = sh[c][(l - a) * (l - a + 1) / 2 + ad];
                    if (!s) x = {(b & 1) ? -u.re : u.re, (b & 1) ? u.im : -u.im};
                    if (d < 0) v = {(ad & 1) ? -v.re : v.re, (ad & 1) ? v.im : -v.im};
                    const Cplx w = x * v;
                    sum.re = fma(r, w.re, sum.re);
                    sum.im = fma(r, w.im, sum.im);
                }
            }
        }
        part[c][i] = sum;
    }
    __syncthreads();
    if (c > 0) return;
    Cplx sum = part[0][i];
    for (int k = 1; k < n; ++k) {
        sum.re += part[k][i].re;
        sum.im += part[k][i].im;
    }
    const double f = kPole.s[l][m];
    float* W = moments + (size_t)(first + P) * kMoments;
    W[pole_slot(l, m, 0)] = (float)(f * sum.re);
    if (m > 0) W[pole_slot(l, m, 1)] = (float)(f * sum.im);
}

// ---------------------------------------------------------------- ray axis
// Twice the triangles' total |projected area| on the planes normal to x, y, z:
// the expected number of crossings of a random line along that axis scales
// with it.  Per-block partial sums, written by one lane each.
__global__ __launch_bounds__(kThreads) void k_proj_area(const float* __restrict__ vx, const float* __restrict__ vy,
                                                         const float* __restrict__ vz, int64_t vs,
                                                         const int32_t* __restrict__ tri, int64_t nf,
                                                         double* __restrict__ part) {
    __shared__ double sm[3][kThreads];
    double acc[3] = {0.0, 0.0, 0.0};
    for (int64_t t = blockIdx.x * (int64_t)kThreads + threadIdx.x; t < nf; t += (int64_t)gridDim.x * kThreads) {
        double p[3][3];
        for (int c = 0; c < 3; ++c) {
            const int64_t v = tri[3 * t + c];
            p[c][0] = vx[v * vs];
            p[c][1] = vy[v * vs];
            p[c][2] = vz[v * vs];
        }
        const double ux = p[1][0] - p[0][0], uy = p[1][1] - p[0][1], uz = p[1][2] - p[0][2];
        const double wx = p[2][0] - p[0][0], wy = p[2][1] - p[0][1], wz = p[2][2] - p[0][2];
        acc[0] += fabs(uy * wz - uz * wy);
        acc[1] += fabs(uz * wx - ux * wz);
        acc[2] += fabs(ux * wy - uy * wx);
    }
    for (int a = 0; a < 3; ++a) sm[a][threadIdx.x] = acc[a];
    __syncthreads();
    for (int s = kThreads / 2; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s)
            for (int a = 0; a < 3; ++a) sm[a][threadIdx.x] += sm[a][threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0)
        for (int a = 0; a < 3; ++a) part[blockIdx.x * 3 + a] = sm[a][0];
}

// ---------------------------------------------------------------- welding
// Vertices with equal float coordinates (+0 and -0 equal) become one index, the
// smallest: sort by a hash of the position (stable), find runs, map.

__device__ __forceinline__ uint32_t weld_bits(float f) {
    const uint32_t b = __float_as_uint(f);
    return (b & 0x7fffffffu) == 0u ? 0u : b;
}

// Equal positions have equal hashes; a sort by the hash (four passes; the three coordinates
// themselves take twelve) brings them together.
__global__ void k_weld_keys(const float* __restrict__ vx, const float* __restrict__ vy, const float* __restrict__ vz,
                            int64_t vs, int64_t nv, uint32_t* __restrict__ key, int* __restrict__ idx) {
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= nv) return;
    uint64_t h = ((uint64_t)weld_bits(vx[i * vs]) << 32) | weld_bits(vy[i * vs]);
    h = (h ^ (h >> 33)) * 0xff51afd7ed558ccdull;
    h ^= (uint64_t)weld_bits(vz[i * vs]) * 0x9e3779b97f4a7c15ull;
    h = (h ^ (h >> 33)) * 0xc4ceb9fe1a85ec53ull;
    key[i] = (uint32_t)(h >> 32);
    idx[i] = (int)i;
}

// start of each sorted hash's run (0 where it continues one)
__global__ void k_weld_heads(int64_t nv, const uint32_t* __restrict__ key, int* __restrict__ head) {
    const int64_t j = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (j >= nv) return;
    head[j] = j == 0 || key[j] != key[j - 1] ? (int)j : 0;
}

// A vertex goes to the first of its run with its position: the smallest index (the sort is
// stable).  That is the run's first but for two positions of one hash.
__global__ __launch_bounds__(kThreads) void k_weld_map(const float* __restrict__ vx, const float* __restrict__ vy,
                                                      const float* __restrict__ vz, int64_t vs,
                                                      const int* __restrict__ idx, const int* __restrict__ start,
                                                      int64_t nv, int* __restrict__ remap, int* __restrict__ nunique) {
    int heads = 0;
    for (int64_t j0 = blockIdx.x * (int64_t)kThreads; j0 < nv; j0 += (int64_t)gridDim.x * kThreads) {
        const int64_t j = j0 + threadIdx.x;
        bool own = false;
        if (j < nv) {
            const int v = idx[j];
            const uint32_t x = weld_bits(vx[v * vs]), y = weld_bits(vy[v * vs]), z = weld_bits(vz[v * vs]);
            int64_t k = start[j];
            int u = idx[k];
            while (k < j && (weld_bits(vx[u * vs]) != x || weld_bits(vy[u * vs]) != y || weld_bits(vz[u * vs]) != z))
                u = idx[++k];
            remap[v] = u;
            own = u == v;
        }
        heads += __syncthreads_count(own);
    }
    if (threadIdx.x == 0) atomicAdd(nunique, heads);   // one per workgroup: they all meet at one address
}

__global__ void k_weld_tris(const int32_t* __restrict__ tri, int64_t n3, const int* __restrict__ remap,
                            int32_t* __restrict__ out) {
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n3) return;
    out[i] = remap[tri[i]];
}

// runs f(temp) with `bytes` of build scratch
template <class F>
hipError_t with_temp(Scratch& S, size_t bytes, F&& f) {
    char* tmp = nullptr;
    hipError_t e = S.alloc(&tmp, (int64_t)bytes);
    if (e != hipSuccess) return e;
    return f((void*)tmp);
}

int bits_for(int64_t n) {
    int b = 1;
    while ((1ll << b) < n) ++b;
    return b;
}

}  // namespace

QGrid make_qgrid(const double bbox[6]) {
    QGrid g;
    double e = 0.0;
    for (int a = 0; a < 3; ++a) e = std::max(e, bbox[3 + a] - bbox[a]);
    if (!(e > 0.0)) e = 1.0;
    for (int a = 0; a < 3; ++a) g.lo[a] = bbox[a] - 0.75 * e;
    const double ext = 2.5 * e;
    const double qmax = (double)kQMax;
    int k = 0;
    if (std::ldexp(ext, 0) <= qmax) {
        while (std::ldexp(ext, k + 1) <= qmax) ++k;
    } else {
        while (std::ldexp(ext, k) > qmax) --k;
    }
    g.k = k;
    g.scale = std::ldexp(1.0, k);
    g.scalef = std::ldexp(1.0f, k);
    return g;
}

gwn_status build_mesh(const float* vx, const float* vy, const float* vz, int64_t vs, int64_t nv, const int32_t* tri,
                      int64_t nf, bool weld, int axis, hipStream_t st, gwn_mesh_s* m) {
    auto t0 = std::chrono::steady_clock::now();
    Scratch S;
    S.st = st;
    // what the build slices off: about 70 bytes per vertex with welding (16 without) and
    // 260 per triangle, and the boundary's, which is usually small against those
    S.first += (size_t)nv * (weld ? 96 : 24) + (size_t)nf * 288;
    int loop_tail = 0;
    unsigned long long *chunk_width = nullptr, width = 0;   // function scope: copied at the end
    m->nv = nv;
    m->nf = nf;
    GWN_HIP_TRY(hipGetDevice(&m->device));

    // ---- vertex statistics and validation
    int* flags = nullptr;
    GWN_HIP_TRY(S.alloc(&flags, 1));
    GWN_HIP_TRY(hipMemsetAsync(flags, 0, sizeof(int), st));
    const int sb = 256;
    float* part = nullptr;
    GWN_HIP_TRY(S.alloc(&part, sb * 6));
    if (nv > 0) {
        k_vertex_stats<<<sb, kThreads, 0, st>>>(vx, vy, vz, vs, nv, part, flags);
        GWN_HIP_TRY(hipGetLastError());
    }
    if (nf > 0) {
        k_tri_check<<<std::min(nblocks(3 * nf), 4096), kThreads, 0, st>>>(tri, 3 * nf, nv, flags);
        GWN_HIP_TRY(hipGetLastError());
    }
    std::vector<float> hpart(sb * 6);
    int hflags = 0;
    if (nv > 0) GWN_HIP_TRY(hipMemcpyAsync(hpart.data(), part, sizeof(float) * sb * 6, hipMemcpyDeviceToHost, st));
    GWN_HIP_TRY(hipMemcpyAsync(&hflags, flags, sizeof(int), hipMemcpyDeviceToHost, st));
    GWN_HIP_TRY(hipStreamSynchronize(st));
    if (hflags & 1) {
        set_error("gwn_build_mesh: non-finite vertex coordinate");
        return GWN_E_INVALID;
    }
    if (hflags & 2) {
        set_error("gwn_build_mesh: triangle index outside [0, %lld)", (long long)nv);
        return GWN_E_INVALID;
    }
    // ---- ray axis: least total projected area (fewest expected crossings) when asked
    if (axis < 0) {
        axis = 0;
        if (nf > 0) {
            const int pb = 256;
            double* pa = nullptr;
            GWN_HIP_TRY(S.alloc(&pa, 3 * pb));
            k_proj_area<<<pb, kThreads, 0, st>>>(vx, vy, vz, vs, tri, nf, pa);
            GWN_HIP_TRY(hipGetLastError());
            std::vector<double> h(3 * pb);
            GWN_HIP_TRY(hipMemcpyAsync(h.data(), pa, sizeof(double) * 3 * pb, hipMemcpyDeviceToHost, st));
            GWN_HIP_TRY(hipStreamSynchronize(st));
            double A[3] = {0, 0, 0};
            for (int b = 0; b < pb; ++b)
                for (int a = 0; a < 3; ++a) A[a] += h[3 * b + a];
            // world x, y, z -> axis codes 1, 2, 0; z wins ties
            if (A[0] < A[2] && A[0] <= A[1]) axis = 1;
            else if (A[1] < A[2] && A[1] < A[0]) axis = 2;
            m->proj_area[0] = A[0];
            m->proj_area[1] = A[1];
            m->proj_area[2] = A[2];
        }
    }
    m->axis = axis;
    axis_ptrs(axis, vx, vy, vz);   // from here on every coordinate is in the mesh frame

    // ---- optional welding of equal positions (the boundary is extracted by index)
    m->nunique = nv;
    if (weld && nv > 1 && nf > 0) {
        uint32_t *key = nullptr, *key2 = nullptr;
        int *idx = nullptr, *idx2 = nullptr, *head = nullptr, *start = nullptr, *remap = nullptr, *nuq = nullptr;
        int32_t* triw = nullptr;
        GWN_HIP_TRY(S.alloc(&key, nv));
        GWN_HIP_TRY(S.alloc(&key2, nv));
        GWN_HIP_TRY(S.alloc(&idx, nv));
        GWN_HIP_TRY(S.alloc(&idx2, nv));
        GWN_HIP_TRY(S.alloc(&head, nv));
        GWN_HIP_TRY(S.alloc(&start, nv));
        GWN_HIP_TRY(S.alloc(&remap, nv));
        GWN_HIP_TRY(S.alloc(&nuq, 1));
        GWN_HIP_TRY(S.alloc(&triw, 3 * nf));
        GWN_HIP_TRY(hipMemsetAsync(nuq, 0, sizeof(int), st));
        k_weld_keys<<<nblocks(nv), kThreads, 0, st>>>(vx, vy, vz, vs, nv, key, idx);
        GWN_HIP_TRY(hipGetLastError());
        GWN_HIP_TRY(with_temp(S, sort_temp_bytes(nv, 4, true), [&](void* tmp) {
            return radix_sort_u32(key, key2, idx, idx2, nv, 0, 32, tmp, st);
        }));
        k_weld_heads<<<nblocks(nv), kThreads, 0, st>>>(nv, key2, head);
        GWN_HIP_TRY(hipGetLastError());
        GWN_HIP_TRY(with_temp(S, scan_temp_bytes(nv), [&](void* tmp) {
            return scan_inclusive_max(head, start, nv, tmp, st);
        }));
        k_weld_map<<<std::min(nblocks(nv), 1024), kThreads, 0, st>>>(vx, vy, vz, vs, idx2, start, nv, remap, nuq);
        GWN_HIP_TRY(hipGetLastError());
        k_weld_tris<<<nblocks(3 * nf), kThreads, 0, st>>>(tri, 3 * nf, remap, triw);
        GWN_HIP_TRY(hipGetLastError());
        int hn = 0;
        GWN_HIP_TRY(hipMemcpyAsync(&hn, nuq, sizeof(int), hipMemcpyDeviceToHost, st));
        GWN_HIP_TRY(hipStreamSynchronize(st));
        m->nunique = hn;
        tri = triw;   // the rest of the build sees welded indices
    }

    double bbox[6] = {0, 0, 0, 0, 0, 0};
    if (nv > 0) {
        for (int a = 0; a < 3; ++a) {
            float mn = INFINITY, mx = -INFINITY;
            for (int b = 0; b < sb; ++b) {
                mn = std::min(mn, hpart[b * 6 + a]);
                mx = std::max(mx, hpart[b * 6 + 3 + a]);
            }
            bbox[a] = (double)mn;
            bbox[3 + a] = (double)mx;
        }
        // the statistics ran on the world axes: frame component c is world (c + axis) % 3
        double bw[6];
        std::memcpy(bw, bbox, sizeof(bw));
        for (int c = 0; c < 3; ++c) {
            bbox[c] = bw[(c + axis) % 3];
            bbox[3 + c] = bw[3 + (c + axis) % 3];
        }
    }
    std::memcpy(m->bbox, bbox, sizeof(bbox));
    m->g = make_qgrid(bbox);
    const QGrid g = m->g;

    int4* qv = nullptr;
    GWN_HIP_TRY(S.alloc(&qv, nv));
    if (nv > 0) {
        k_quantize_vertices<<<nblocks(nv), kThreads, 0, st>>>(vx, vy, vz, vs, nv, g, qv);
        GWN_HIP_TRY(hipGetLastError());
    }

    // ---- triangles, Morton order, LBVH
    if (nf > 0) {
        int4 qlo, qspan;
        auto qc = [&](double x, int a) { return (int)std::rint((x - g.lo[a]) * g.scale); };
        qlo = make_int4(qc(bbox[0], 0), qc(bbox[1], 1), qc(bbox[2], 2), 0);
        qspan = make_int4(qc(bbox[3], 0) - qlo.x, qc(bbox[4], 1) - qlo.y, qc(bbox[5], 2) - qlo.z, 0);
        TriQ* tq = nullptr;
        uint64_t *keys = nullptr, *keys2 = nullptr;
        GWN_HIP_TRY(S.alloc(&tq, nf));
        GWN_HIP_TRY(S.alloc(&keys, nf));
        GWN_HIP_TRY(S.alloc(&keys2, nf));
        k_tri_setup<<<nblocks(nf), kThreads, 0, st>>>(tri, nf, qv, qlo, qspan, tq, keys);
        GWN_HIP_TRY(hipGetLastError());
        // the low 32 bits of a key are its triangle's index, i.e. its input
        // position: a stable sort by the Morton code (bits 32..61) alone gives
        // the order of a sort by the whole key
        GWN_HIP_TRY(with_temp(S, sort_temp_bytes(nf, 8, false), [&](void* tmp) {
            return radix_sort_u64(keys, keys2, nullptr, nullptr, nf, 32, 62, tmp, st);
        }));
        GWN_HIP_TRY(gwn::dmalloc((void**)&m->tris, sizeof(TriQ) * (size_t)nf));
        GWN_HIP_TRY(gwn::dmalloc((void**)&m->trif, sizeof(float4) * 3 * (size_t)nf));
        k_permute_tris<<<nblocks(nf), kThreads, 0, st>>>(keys2, nf, tq, m->tris, tri, vx, vy, vz, vs, m->trif);
        GWN_HIP_TRY(hipGetLastError());
        if (nf >= 2) {
            m->nnodes = nf - 1;
            GWN_HIP_TRY(gwn::dmalloc((void**)&m->nodes, sizeof(Node) * (size_t)(nf - 1)));
            GWN_HIP_TRY(hipMemsetAsync(m->nodes, 0xff, sizeof(Node) * (size_t)(nf - 1), st));
            int *leaf_parent = nullptr, *rflags = nullptr, *depth = nullptr;
            GWN_HIP_TRY(S.alloc(&leaf_parent, nf));
            GWN_HIP_TRY(S.alloc(&rflags, nf + 1));
            GWN_HIP_TRY(S.alloc(&depth, 1));
            GWN_HIP_TRY(hipMemsetAsync(rflags, 0, sizeof(int) * (size_t)(nf + 1), st));
            GWN_HIP_TRY(hipMemsetAsync(depth, 0, sizeof(int), st));
            k_karras<<<nblocks(nf - 1), kThreads, 0, st>>>(keys2, (int)nf, m->nodes, leaf_parent);
            GWN_HIP_TRY(hipGetLastError());
            k_refit<<<(unsigned)((nf + kRefitLeaves - 1) / kRefitLeaves), kRefitThreads, 0, st>>>(m->tris, (int)nf, m->nodes, leaf_parent, rflags);
            GWN_HIP_TRY(hipGetLastError());
            k_depth<<<nblocks(nf), kThreads, 0, st>>>((int)nf, m->nodes, leaf_parent, depth);
            GWN_HIP_TRY(hipGetLastError());
            int hd = 0, rf = 0;
            GWN_HIP_TRY(hipMemcpyAsync(&hd, depth, sizeof(int), hipMemcpyDeviceToHost, st));
            GWN_HIP_TRY(hipMemcpyAsync(&rf, rflags + nf, sizeof(int), hipMemcpyDeviceToHost, st));
            GWN_HIP_TRY(hipStreamSynchronize(st));
            if (rf != 0) {
                set_error("gwn_build_mesh: malformed BVH (refit did not reach the root)");
                return GWN_E_HIP;
            }
            m->depth = hd;
            m->root = 0;
        } else {
            m->root = ~0;
            m->depth = 0;
        }
    }

    // ---- boundary chain
    if (nf > 0) {
        const int64_t ne = 3 * nf;
        uint64_t *ek = nullptr, *ek2 = nullptr;
        int *es = nullptr, *es2 = nullptr, *net = nullptr, *cnt = nullptr, *off = nullptr;
        GWN_HIP_TRY(S.alloc(&ek, ne));
        GWN_HIP_TRY(S.alloc(&ek2, ne));
        GWN_HIP_TRY(S.alloc(&es, ne));
        GWN_HIP_TRY(S.alloc(&es2, ne));
        GWN_HIP_TRY(S.alloc(&net, ne));
        GWN_HIP_TRY(S.alloc(&cnt, ne));
        GWN_HIP_TRY(S.alloc(&off, ne));
        const int vb = bits_for(nv);
        k_edge_keys<<<nblocks(ne), kThreads, 0, st>>>(tri, nf, vb, ek, es);
        GWN_HIP_TRY(hipGetLastError());
        GWN_HIP_TRY(with_temp(S, sort_temp_bytes(ne, 8, true), [&](void* tmp) {
            return radix_sort_u64(ek, ek2, es, es2, ne, 0, 2 * vb, tmp, st);
        }));
        k_edge_runs<<<nblocks(ne), kThreads, 0, st>>>(ek2, es2, ne, net, cnt);
        GWN_HIP_TRY(hipGetLastError());
        GWN_HIP_TRY(with_temp(S, scan_temp_bytes(ne), [&](void* tmp) {
            return scan_exclusive_sum(cnt, off, ne, tmp, st);
        }));
        int last_off = 0, last_cnt = 0;
        GWN_HIP_TRY(hipMemcpyAsync(&last_off, off + ne - 1, sizeof(int), hipMemcpyDeviceToHost, st));
        GWN_HIP_TRY(hipMemcpyAsync(&last_cnt, cnt + ne - 1, sizeof(int), hipMemcpyDeviceToHost, st));
        GWN_HIP_TRY(hipStreamSynchronize(st));
        const int64_t nb = (int64_t)last_off + last_cnt;
        m->nb = nb;
        if (nb > 0) {
            int *efrom = nullptr, *eto = nullptr, *ids = nullptr, *kk = nullptr, *in_by_to = nullptr,
                *out_by_from = nullptr, *succ = nullptr;
            int *repA = nullptr, *repB = nullptr, *jA = nullptr, *jB = nullptr, *dA = nullptr, *dB = nullptr;
            int *len = nullptr, *head = nullptr, *voff = nullptr, *lid = nullptr;
            // the boundary's temporaries: 17 numbers per edge and (at most nb / 2 loops) 18 per loop,
            // the sorts' and scans'; of an unwelded soup as much as the triangles' (85 k of them: nine
            // blocks of an eighth, a third of 3.2 ms)
            GWN_HIP_TRY(S.reserve((size_t)nb * 4 * (17 + 9) + 2 * sort_temp_bytes(nb, 4, true) + sort_temp_bytes(nb / 2 + 1, 4, true) +
                                  4 * scan_temp_bytes(2 * nb) + 64 * 256));
            for (int** p : {&efrom, &eto, &ids, &kk, &in_by_to, &out_by_from, &succ, &repA, &repB, &jA, &jB, &dA, &dB,
                            &len, &head, &voff, &lid})
                GWN_HIP_TRY(S.alloc(p, nb));
            k_edge_emit<<<nblocks(ne), kThreads, 0, st>>>(ek2, net, cnt, off, ne, vb, efrom, eto);
            GWN_HIP_TRY(hipGetLastError());
            k_iota<<<nblocks(nb), kThreads, 0, st>>>(ids, nb);
            GWN_HIP_TRY(with_temp(S, sort_temp_bytes(nb, 4, true), [&](void* tmp) {
                return radix_sort_u32((const uint32_t*)eto, (uint32_t*)kk, ids, in_by_to, nb, 0, vb, tmp, st);
            }));
            GWN_HIP_TRY(with_temp(S, sort_temp_bytes(nb, 4, true), [&](void* tmp) {
                return radix_sort_u32((const uint32_t*)efrom, (uint32_t*)kk, ids, out_by_from, nb, 0, vb, tmp, st);
            }));
            k_link<<<nblocks(nb), kThreads, 0, st>>>(in_by_to, out_by_from, nb, succ);
            GWN_HIP_TRY(hipGetLastError());
            if (nb <= kFewEdges) {
                k_rank_loops<<<1, kRankThreads, 0, st>>>(succ, (int)nb, bits_for(nb) + 1, repA, dA, voff, lid, head);
                GWN_HIP_TRY(hipGetLastError());
                int loops = 0;
                GWN_HIP_TRY(hipMemcpyAsync(&loops, head, sizeof(int), hipMemcpyDeviceToHost, st));
                GWN_HIP_TRY(hipStreamSynchronize(st));
                m->nloops = loops;
            } else {
                // cycle representative = smallest edge id on the cycle (pointer jumping)
                GWN_HIP_TRY(hipMemcpyAsync(jA, succ, sizeof(int) * nb, hipMemcpyDeviceToDevice, st));
                k_iota<<<nblocks(nb), kThreads, 0, st>>>(repA, nb);
                const int rounds = (bits_for(nb) + 2) / 2;   // of two doublings
                for (int r = 0; r < rounds; ++r) {
                    k_rep_round<<<nblocks(nb), kThreads, 0, st>>>(repA, jA, nb, repB, jB);
                    std::swap(repA, repB);
                    std::swap(jA, jB);
                }
                GWN_HIP_TRY(hipGetLastError());
                // distance to the end of the cycle opened at its representative (list ranking)
                k_rank_init<<<nblocks(nb), kThreads, 0, st>>>(succ, repA, nb, jA, dA);
                for (int r = 0; r < rounds; ++r) {
                    k_rank_round<<<nblocks(nb), kThreads, 0, st>>>(jA, dA, nb, jB, dB);
                    std::swap(jA, jB);
                    std::swap(dA, dB);
                }
                GWN_HIP_TRY(hipGetLastError());
                k_loop_counts<<<nblocks(nb), kThreads, 0, st>>>(repA, dA, nb, len, head);
                GWN_HIP_TRY(with_temp(S, scan_temp_bytes(nb), [&](void* tmp) {
                    return scan_exclusive_sum(len, voff, nb, tmp, st);
                }));
                GWN_HIP_TRY(with_temp(S, scan_temp_bytes(nb), [&](void* tmp) {
                    return scan_exclusive_sum(head, lid, nb, tmp, st);
                }));
                int last[2] = {0, 0};
                GWN_HIP_TRY(hipMemcpyAsync(&last[0], lid + nb - 1, sizeof(int), hipMemcpyDeviceToHost, st));
                GWN_HIP_TRY(hipMemcpyAsync(&last[1], head + nb - 1, sizeof(int), hipMemcpyDeviceToHost, st));
                GWN_HIP_TRY(hipStreamSynchronize(st));
                m->nloops = (int64_t)last[0] + last[1];
            }
            GWN_HIP_TRY(gwn::dmalloc((void**)&m->bverts, sizeof(BVert) * (size_t)nb));
            GWN_HIP_TRY(gwn::dmalloc((void**)&m->loop_off, sizeof(int) * (size_t)(m->nloops + 1)));
            k_emit_loops<<<nblocks(nb), kThreads, 0, st>>>(efrom, repA, dA, voff, lid, nb, vx, vy, vz, vs, qv, g.scalef,
                                                          m->bverts, m->loop_off);
            GWN_HIP_TRY(hipGetLastError());
            loop_tail = (int)nb;   // function scope: the copy reads it after this block
            GWN_HIP_TRY(hipMemcpyAsync(m->loop_off + m->nloops, &loop_tail, sizeof(int), hipMemcpyHostToDevice, st));

            // the boundary in chunks, loops along a Hilbert curve and in clusters
            const int64_t nl = m->nloops;
            const int csize = kLeafEdges;
            const int most = (int)std::min<int64_t>(nl, nb / csize + 1);
            uint32_t *lk = nullptr, *lk2 = nullptr;
            int *li = nullptr, *lord = nullptr, *rank = nullptr, *piece = nullptr, *poff = nullptr;
            int *heads = nullptr, *hid = nullptr, *cid = nullptr, *cfirst = nullptr, *ccount = nullptr, *cbase = nullptr;
            GWN_HIP_TRY(S.alloc(&lk, nl));
            GWN_HIP_TRY(S.alloc(&lk2, nl));
            GWN_HIP_TRY(S.alloc(&li, nl));
            GWN_HIP_TRY(S.alloc(&lord, nl));
            GWN_HIP_TRY(S.alloc(&rank, nl));
            GWN_HIP_TRY(S.alloc(&piece, 3 * nl + 1));
            GWN_HIP_TRY(S.alloc(&poff, 3 * nl + 1));
            GWN_HIP_TRY(S.alloc(&heads, nl + 1));
            GWN_HIP_TRY(S.alloc(&hid, nl + 1));
            GWN_HIP_TRY(S.alloc(&cid, nl));
            GWN_HIP_TRY(S.alloc(&cfirst, most));
            GWN_HIP_TRY(S.alloc(&ccount, most + 1));
            GWN_HIP_TRY(S.alloc(&cbase, most + 2));
            GWN_HIP_TRY(S.alloc(&chunk_width, 1));
            if (nl <= kFewLoops) {
                k_plan_loops<<<1, kPlanThreads, 0, st>>>(m->bverts, m->loop_off, (int)nl, g, csize, most, lord, rank, poff,
                                                         cid, cfirst, ccount, cbase);
                GWN_HIP_TRY(hipGetLastError());
            } else {
                k_loop_keys<<<nblocks(nl), kThreads, 0, st>>>(m->bverts, m->loop_off, nl, g, lk, li);
                GWN_HIP_TRY(hipGetLastError());
                GWN_HIP_TRY(with_temp(S, sort_temp_bytes(nl, 4, true), [&](void* tmp) {
                    return radix_sort_u32(lk, lk2, li, lord, nl, 0, 30, tmp, st);
                }));
                k_loop_pieces<<<nblocks(nl + 1), kThreads, 0, st>>>(m->loop_off, lord, nl, rank, piece);
                GWN_HIP_TRY(hipGetLastError());
                GWN_HIP_TRY(with_temp(S, scan_temp_bytes(3 * nl + 1), [&](void* tmp) {
                    return scan_exclusive_sum(piece, poff, 3 * nl + 1, tmp, st);
                }));
                k_cluster_heads<<<nblocks(nl + 1), kThreads, 0, st>>>(poff, nl, csize, heads);
                GWN_HIP_TRY(hipGetLastError());
                GWN_HIP_TRY(with_temp(S, scan_temp_bytes(nl + 1), [&](void* tmp) {
                    return scan_exclusive_sum(heads, hid, nl + 1, tmp, st);
                }));
                k_cluster_first<<<nblocks(nl), kThreads, 0, st>>>(heads, hid, nl, most, cid, cfirst);
                GWN_HIP_TRY(hipGetLastError());
                k_cluster_chunks<<<nblocks(most + 1), kThreads, 0, st>>>(hid, cfirst, poff, nl, most, ccount, cbase + most + 1);
                GWN_HIP_TRY(hipGetLastError());
                GWN_HIP_TRY(with_temp(S, scan_temp_bytes(most + 1), [&](void* tmp) {
                    return scan_exclusive_sum(ccount, cbase, most + 1, tmp, st);
                }));
            }
            int totals[2] = {0, 0};   // chunks, clusters
            GWN_HIP_TRY(hipMemcpyAsync(totals, cbase + most, sizeof(totals), hipMemcpyDeviceToHost, st));
            GWN_HIP_TRY(hipStreamSynchronize(st));
            const int hchunks = totals[0], hclusters = totals[1];
            if (hclusters < 1 || hclusters > most || hchunks < 1) {
                set_error("gwn_build_mesh: malformed boundary clusters");
                return GWN_E_HIP;
            }
            m->nchunk = hchunks;
            m->nclusters = hclusters;
            const size_t nent = kChunk * (size_t)m->nchunk;
            // levels: kFan clusters of one make one of the next, until at most kRoots are left
            int nlev = 0, total = 0;
            for (int c = hclusters;; c = (c + kFan - 1) / kFan) {
                m->cluster_level[nlev++] = total;
                total += c;
                if (c <= kRoots || nlev == kLevels) break;
            }
            m->cluster_top = nlev - 1;
            for (int l = nlev; l <= kLevels; ++l) m->cluster_level[l] = total;
            Levels levels;
            std::copy(m->cluster_level, m->cluster_level + kLevels + 1, levels.first);
            static_assert(sizeof(m->cluster_level) <= sizeof(Cluster), "the level table follows the clusters");
            // one block for all of it: a hipMalloc and a hipFree each cost as much as a kernel
            const size_t bytes[5] = {sizeof(CVert) * nent, sizeof(GVertex) * nent, sizeof(int4) * (size_t)m->nchunk,
                                     sizeof(Cluster) * ((size_t)total + 1), sizeof(float) * kMoments * (size_t)total};
            void** dst[5] = {(void**)&m->chain, (void**)&m->gchain, (void**)&m->cbox, (void**)&m->clusters, (void**)&m->moments};
            size_t all = 0;
            for (size_t b : bytes) all += (b + 255) & ~(size_t)255;
            char* at = nullptr;
            GWN_HIP_TRY(gwn::dmalloc((void**)&at, all));
            for (int k = 0; k < 5; ++k) {
                *dst[k] = at;
                at += (bytes[k] + 255) & ~(size_t)255;
            }
            GWN_HIP_TRY(hipMemsetAsync(m->chain, 0, sizeof(CVert) * nent, st));
            GWN_HIP_TRY(hipMemsetAsync(chunk_width, 0, sizeof(unsigned long long), st));
            const ChainPlan cp{rank, cid, cfirst, poff, cbase, nl, hclusters};
            k_emit_chain<<<nblocks(nb), kThreads, 0, st>>>(m->bverts, m->loop_off, cp, nb, (int64_t)nent, m->chain,
                                                          m->gchain);
            GWN_HIP_TRY(hipGetLastError());
            k_chunk_boxes<<<nblocks(m->nchunk), kThreads, 0, st>>>(m->nchunk, m->chain, m->gchain, m->cbox, chunk_width);
            GWN_HIP_TRY(hipGetLastError());
            k_cluster_frames<<<(unsigned)hclusters, 64, 0, st>>>(m->bverts, m->loop_off, lord, cp, ccount, levels,
                                                                   m->clusters);
            GWN_HIP_TRY(hipGetLastError());
            if (hclusters >= kFewClusters) {
                k_cluster_moments<1><<<dim3((unsigned)hclusters, 2), 64, 0, st>>>(m->gchain, m->clusters, m->moments);
                GWN_HIP_TRY(hipGetLastError());
                k_cluster_moments<8><<<dim3((unsigned)hclusters, 2), 512, 0, st>>>(m->gchain, m->clusters, m->moments);
                GWN_HIP_TRY(hipGetLastError());
                for (int l = 1; l < nlev; ++l) {
                    const int* o = m->cluster_level;
                    k_cluster_merge<<<(unsigned)(o[l + 1] - o[l]), kMergeThreads, 0, st>>>(
                        o[l], o[l + 1] - o[l], o[l - 1], o[l] - o[l - 1], g.lo[0] * g.scale, g.lo[1] * g.scale, m->clusters,
                        m->moments);
                    GWN_HIP_TRY(hipGetLastError());
                }
            }
            GWN_HIP_TRY(hipMemcpyAsync(&width, chunk_width, sizeof(width), hipMemcpyDeviceToHost, st));
        }
    }
    if (!m->loop_off) {
        GWN_HIP_TRY(gwn::dmalloc((void**)&m->loop_off, sizeof(int)));
        GWN_HIP_TRY(hipMemsetAsync(m->loop_off, 0, sizeof(int), st));
    }
    GWN_HIP_TRY(hipStreamSynchronize(st));
    if (m->nchunk > 0) m->chunk_w = (double)width / (2.0 * (double)m->nchunk);
    m->build_ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
    return GWN_OK;
}

}  // namespace gwn

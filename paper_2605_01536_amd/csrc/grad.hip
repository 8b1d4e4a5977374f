// grad.hip -- gradient of w with respect to the query point (Supp. Sec. 4).
//
// The crossing count is locally constant, so only the boundary term has a gradient,
// and the gradient of a loop's solid angle is a line integral along the loop that
// needs no auxiliary direction (the Biot-Savart field of the loop).  Per directed
// boundary edge (a, b), with r0 = a - p, r1 = b - p and l = |r|:
//
//     grad = c (l0 + l1) / (l0 l1 (l0 l1 + r0.r1)),   c = r0 x r1 = r0 x (b - a),
//
// 4 pi grad w being the sum.  Alg. 3 sums the derivative of 2 atan2(N, D) for an axis
// x0 instead: the same total, per edge twice the work (l, s, and two quotients), and
// 0/0 for a query whose line along x0 meets a boundary vertex, which then has to be
// summed again for another axis.  The form here is singular on the edge alone.
//
// Where r0.r1 < 0 the bracket cancels next to the edge; there it is
// |c|^2 / (l0 l1 - r0.r1), exactly the same, and c, from the edge's own vector, is
// rounded once, so the term keeps its digits up to the edge.
// FP32 offsets are in units of 2^18 cells (times 2^e for far queries, see far_scale):
// an offset stays below 2^23 and the products below 2^118.
//
// Grids share a column's x/y terms among its samples as for w, and sum the chunks far
// from a block of columns at its nodes (gwn_far.h).
#include <algorithm>

#include "gwn_alloc.h"
#include "gwn_far.h"
#include "gwn_kernels.h"
#include "gwn_mesh.h"

namespace gwn {
namespace {

// cells per offset unit
template <class T>
constexpr float kGradUnit = sizeof(T) == 4 ? 0x1p18f : 1.0f;

// x y - z w, correctly rounded to about an ulp however far it cancels
template <class T>
__device__ __forceinline__ T diff_of_products(T x, T y, T z, T w) {
    const T p = z * w;
    return fma(x, y, -p) + fma(-z, w, p);
}

// One edge's term added to g, given c, the dot product, h = |e|^2 / 2 and the two
// lengths.  A lane with dot < h (the edge as long as its distance, or longer) takes c
// from exact(), without cancellation, and with dot < 0 the other form of the bracket;
// the wave looks for one first, and each lane's result is its own.
template <class T, class F>
__device__ __forceinline__ void grad_term(T cx, T cy, T cz, T dot, T h, T la, T lb, F&& exact, bool general, T* g) {
    const T ll = la * lb;
    T den = ll * (ll + dot), num = la + lb;
    if (general) {
        const bool near = dot < h, neg = dot < (T)0;
        T x, y, z;
        exact(x, y, z);
        cx = near ? x : cx;
        cy = near ? y : cy;
        cz = near ? z : cz;
        den = neg ? ll * fma(x, x, fma(y, y, z * z)) : den;
        num = neg ? num * (ll - dot) : num;
    }
    const T f = num * Arith<T>::rcp(den);
    g[0] = fma(cx, f, g[0]);
    g[1] = fma(cy, f, g[1]);
    g[2] = fma(cz, f, g[2]);
}

// ---------------------------------------------------------------- points

template <class T>
struct GVert {
    T x, y, z, l;   // offset and length
};

template <class T>
__device__ __forceinline__ GVert<T> grad_vert(const GVertex& b, T px, T py, T pz, T f) {
    GVert<T> v;
    v.x = fma((T)b.x, f, -px);
    v.y = fma((T)b.y, f, -py);
    v.z = fma((T)b.z, f, -pz);
    v.l = Arith<T>::sqrt(fma(v.x, v.x, fma(v.y, v.y, v.z * v.z)));
    return v;
}

// Sum over chunks c0, c0 + step, ..., < nchunk for one point; FP32 partials are flushed to
// FP64 every 4 chunks.
template <class T>
__device__ __forceinline__ void grad_chunks_point(const GVertex* __restrict__ gchain, int nchunk, int c0, int step, T px, T py,
                                                  T pz, T f, double* G) {
    G[0] = G[1] = G[2] = 0.0;
    T acc[3] = {(T)0, (T)0, (T)0};
    int left = 4;
    for (int c = c0; c < nchunk; c += step) {
        const GVertex* __restrict__ v = gchain + (size_t)c * kChunk;
        GVertex a = v[0];
        GVert<T> ra = grad_vert<T>(a, px, py, pz, f);
#pragma unroll
        for (int e = 1; e < kChunk; ++e) {
            const GVertex b = v[e];
            const GVert<T> rb = grad_vert<T>(b, px, py, pz, f);
            if (a.flags & kChainEdge) {
                const T ex = ((T)b.x - (T)a.x) * f, ey = ((T)b.y - (T)a.y) * f, ez = ((T)b.z - (T)a.z) * f;
                const T dot = fma(ra.x, rb.x, fma(ra.y, rb.y, ra.z * rb.z));
                const T h = (T)0.5 * fma(ex, ex, fma(ey, ey, ez * ez));
                grad_term<T>(
                    fma(ra.y, ez, -(ra.z * ey)), fma(ra.z, ex, -(ra.x * ez)), fma(ra.x, ey, -(ra.y * ex)), dot, h, ra.l,
                    rb.l,
                    [&](T& x, T& y, T& z) {
                        x = diff_of_products(ra.y, ez, ra.z, ey);
                        y = diff_of_products(ra.z, ex, ra.x, ez);
                        z = diff_of_products(ra.x, ey, ra.y, ex);
                    },
                    __builtin_amdgcn_ballot_w64(dot < h) != 0ull, acc);
            }
            a = b;
            ra = rb;
        }
        if (--left == 0) {
            for (int k = 0; k < 3; ++k) {
                G[k] += (double)acc[k];
                acc[k] = (T)0;
            }
            left = 4;
        }
    }
    for (int k = 0; k < 3; ++k) G[k] += (double)acc[k];
}

// a point's offsets' scale and its coordinates in offset units
template <class T>
struct GPoint {
    T f, x, y, z;
    double out;   // the sum's factor: 1 / (4 pi) and the chain rule through the units
};

template <class T>
__device__ __forceinline__ GPoint<T> grad_point(const QGrid& g, float px, float py, float pz, float pzmax) {
    constexpr T u = (T)1 / (T)kGradUnit<T>;
    const FarScale<T> fs = far_scale<T>(px, py, pzmax, g.scale);
    GPoint<T> p;
    p.f = fs.f * u;
    const T s = fs.scf * u;
    p.x = (T)px * s;
    p.y = (T)py * s;
    p.z = (T)pz * s;
    p.out = 0.5 * kInv2Pi * (double)s;
    return p;
}

// A point whose FP32 sum is not finite, again in FP64: next to a vertex the products of a
// term leave FP32's range (from about 1e-18 of the mesh's size; where floats are that fine,
// near the origin).  Rare, and out of line so that its registers do not count.
struct Grad3 {
    double g[3];
};

__device__ __attribute__((noinline)) Grad3 grad_again(const GVertex* gchain, int nentry, float scale, float px, float py, float pz) {
    Grad3 r = {};
#pragma unroll 1
    for (const GVertex* v = gchain; v + 1 < gchain + nentry; ++v) {   // (a chunk's last entry has no edge)
        if (!(v->flags & kChainEdge)) continue;
        const double ax = v->x - (double)px * scale, ay = v->y - (double)py * scale, az = v->z - (double)pz * scale;
        const double ex = (double)v[1].x - v->x, ey = (double)v[1].y - v->y, ez = (double)v[1].z - v->z;
        const double bx = v[1].x - (double)px * scale, by = v[1].y - (double)py * scale, bz = v[1].z - (double)pz * scale;
        const double dot = fma(ax, bx, fma(ay, by, az * bz));
        const double lb = Arith<double>::sqrt(fma(bx, bx, fma(by, by, bz * bz)));
        __builtin_amdgcn_sched_barrier(0);   // (few registers rather than speed)
        const double la = Arith<double>::sqrt(fma(ax, ax, fma(ay, ay, az * az))), ll = la * lb;
        const double cx = diff_of_products(ay, ez, az, ey), cy = diff_of_products(az, ex, ax, ez), cz = diff_of_products(ax, ey, ay, ex);
        __builtin_amdgcn_sched_barrier(0);
        const bool neg = dot < 0.0;
        double f = (la + lb) * Arith<double>::rcp(ll) * (neg ? ll - dot : 1.0);
        f *= Arith<double>::rcp(neg ? fma(cx, cx, fma(cy, cy, cz * cz)) : ll + dot);
        r.g[0] = fma(cx, f, r.g[0]);
        r.g[1] = fma(cy, f, r.g[1]);
        r.g[2] = fma(cz, f, r.g[2]);
    }
    for (int c = 0; c < 3; ++c) r.g[c] *= 0.5 * kInv2Pi * scale;
    return r;
}

template <class T>
__device__ __forceinline__ void grad_out(const MeshView& mv, float px, float py, float pz, double g0, double g1, double g2, int axis,
                                         T* __restrict__ g) {
    Grad3 r = {{g0, g1, g2}};
    if (sizeof(T) == 4 && !(fabs(g0) + fabs(g1) + fabs(g2) < 1e300)) r = grad_again(mv.gchain, mv.nchunk * kChunk, mv.g.scalef, px, py, pz);
    for (int c = 0; c < 3; ++c) g[(c + axis) % 3] = (T)r.g[c];   // frame component c is world component (c + axis) % 3
}

// AGAIN: with grad_again's call, which costs the loop 5%; without, k_grad_again follows, which
// costs a launch.
template <class T, bool AGAIN>
__global__ __launch_bounds__(256) void k_grad_batch(MeshView mv, const float* __restrict__ qx,
                                                    const float* __restrict__ qy, const float* __restrict__ qz,
                                                    long long qs, long long nq, int axis, T* __restrict__ g) {
    const long long i = blockIdx.x * 256ll + threadIdx.x;
    if (blockIdx.x * 256ll >= nq) return;
    const long long ii = i < nq ? i : nq - 1;
    const float px = qx[ii * qs], py = qy[ii * qs], pz = qz[ii * qs];
    const GPoint<T> p = grad_point<T>(mv.g, px, py, pz, fabsf(pz));
    double G[3];
    grad_chunks_point<T>(mv.gchain, mv.nchunk, 0, 1, p.x, p.y, p.z, p.f, G);
    if (i >= nq) return;
    if constexpr (AGAIN) {
        grad_out<T>(mv, px, py, pz, G[0] * p.out, G[1] * p.out, G[2] * p.out, axis, g + 3 * i);
    } else {
        for (int c = 0; c < 3; ++c) g[3 * i + (c + axis) % 3] = (T)(G[c] * p.out);
    }
}

__global__ __launch_bounds__(256) void k_grad_again(MeshView mv, const float* __restrict__ qx, const float* __restrict__ qy,
                                                    const float* __restrict__ qz, long long qs, long long nq, int axis,
                                                    float* __restrict__ g) {
    const long long i = blockIdx.x * 256ll + threadIdx.x;
    if (i >= nq) return;
    const double s = (double)fabsf(g[3 * i]) + (double)fabsf(g[3 * i + 1]) + (double)fabsf(g[3 * i + 2]);
    if (!(s < 1e300)) grad_out<float>(mv, qx[i * qs], qy[i * qs], qz[i * qs], s, s, s, axis, g + 3 * i);
}

// Few points against many boundary edges: one workgroup per point, the chunks dealt
// out to its lanes, reduced by wave shuffles and LDS in a fixed order.
constexpr int kSplitThreads = 256;

template <class T>
__global__ __launch_bounds__(kSplitThreads) void k_grad_split(MeshView mv, const float* __restrict__ qx,
                                                             const float* __restrict__ qy,
                                                             const float* __restrict__ qz, long long qs, long long nq,
                                                             int axis, T* __restrict__ g) {
    __shared__ double red[kSplitThreads / 64][3];
    const long long i = blockIdx.x;   // one point per workgroup
    if (i >= nq) return;
    const float px = qx[i * qs], py = qy[i * qs], pz = qz[i * qs];
    const GPoint<T> p = grad_point<T>(mv.g, px, py, pz, fabsf(pz));
    double G[3];
    grad_chunks_point<T>(mv.gchain, mv.nchunk, (int)threadIdx.x, kSplitThreads, p.x, p.y, p.z, p.f, G);
    for (int c = 0; c < 3; ++c)
        for (int o = 32; o > 0; o >>= 1) G[c] += __shfl_xor(G[c], o);
    if ((threadIdx.x & 63) == 0)
        for (int c = 0; c < 3; ++c) red[threadIdx.x >> 6][c] = G[c];
    __syncthreads();
    if (threadIdx.x == 0) {
        double t[3] = {0.0, 0.0, 0.0};
        for (int k = 0; k < kSplitThreads / 64; ++k)
            for (int c = 0; c < 3; ++c) t[c] += red[k][c];
        grad_out<T>(mv, px, py, pz, t[0] * p.out, t[1] * p.out, t[2] * p.out, axis, g + 3 * i);
    }
}

// ---------------------------------------------------------------- grid columns
// Records of 64 chained vertices in LDS, one per lane, as for w: the vertex's z and
// x/y distance and everything about its outgoing edge that the column's samples share.
template <class T>
struct alignas(4 * sizeof(T)) GRec {
    T zu, rho2, ex, ey;   // vertex z, r_x^2 + r_y^2; the edge's x, y
};

template <class T>
struct alignas(4 * sizeof(T)) GEdge {
    T a, b, cz, dot;      // r_y e_z, r_x e_z, c_z and the x/y dot
};

template <class T>
struct GAux {             // beside the edge only
    T rx, ry, ez;
};

template <class T>
struct GBuf {
    GRec<T> v[kColRecs];
    GEdge<T> e[kColRecs];
    GAux<T> x[kColRecs];
    T h[kColRecs];        // |e|^2 / 2 (no edge: 0)
    int queue[64 + kColChunks];
};

template <class T>
__device__ __forceinline__ void grad_fill(const MeshView& mv, const int* queue, int n, T px, T py, T f, GBuf<T>& buf) {
    int lane = (int)(threadIdx.x & 63);
    asm volatile("" : "+v"(lane));   // addresses formed per fill (see col_fill)
    const int c = lane >> 3, en = lane & 7;
    if (c < n) {
        const GVertex* v = mv.gchain + (size_t)queue[c] * kChunk;
        const GVertex a = v[en], b = v[min(en + 1, kChunk - 1)];
        const bool edge = (a.flags & kChainEdge) != 0;
        const T ax = fma((T)a.x, f, -px), ay = fma((T)a.y, f, -py);
        const T bx = fma((T)b.x, f, -px), by = fma((T)b.y, f, -py);
        const T ex = edge ? ((T)b.x - (T)a.x) * f : (T)0, ey = edge ? ((T)b.y - (T)a.y) * f : (T)0;
        const T ez = edge ? ((T)b.z - (T)a.z) * f : (T)0;
        // between two pieces no edge: c = 0, and a large dot product keeps the bracket positive
        buf.v[lane] = {(T)a.z * f, ax * ax + ay * ay, ex, ey};
        buf.x[lane] = {ax, ay, ez};
        buf.h[lane] = (T)0.5 * fma(ex, ex, fma(ey, ey, ez * ez));
        buf.e[lane] = {ay * ez, ax * ez, fma(ax, ey, -(ay * ex)), edge ? ax * bx + ay * by : (T)1e30};
    }
    wave_lds_sync();
}

// Sum over the chunks that `flt` keeps, added to S[c * ZB + r] (component c, sample r),
// for the ZB samples of each lane of a column; px, py, pz in offset units.  FP32
// partials are flushed to FP64 every 32 edges.
template <class T, int ZB>
__device__ __forceinline__ void grad_column(const MeshView& mv, const ChunkFilter& flt, T px, T py, const T* pz, T f,
                                            double* S, int part, int parts, GBuf<T>& buf) {
    T rza[ZB], la[ZB];
    GRec<T> va = {(T)0, (T)0, (T)0, (T)0};   // the vertex before the current one: none yet
    GEdge<T> ea = {(T)0, (T)0, (T)0, (T)1e30};
    T ha = (T)0;
#pragma unroll
    for (int r = 0; r < ZB; ++r) {
        rza[r] = (T)0;
        la[r] = (T)1;
    }
    ChunkQueue q(mv, part, parts, buf.queue);
    while (true) {
        const int n = q.next(mv, flt);
        if (n == 0) break;
        grad_fill<T>(mv, q.ids(n), n, px, py, f, buf);
        for (int k = 0; k < n * kChunk;) {
            const int ke = min(n * kChunk, k + 32);
            T acc[ZB][3];
#pragma unroll
            for (int r = 0; r < ZB; ++r) acc[r][0] = acc[r][1] = acc[r][2] = (T)0;
#pragma unroll 4
            for (; k < ke; ++k) {
                const GRec<T> vb = buf.v[k];
                const GEdge<T> eb = buf.e[k];
                const T hb = buf.h[k];
                T rzb[ZB], lb[ZB], dot[ZB];
                bool near = false;
#pragma unroll
                for (int r = 0; r < ZB; ++r) {
                    rzb[r] = vb.zu - pz[r];
                    lb[r] = Arith<T>::sqrt(fma(rzb[r], rzb[r], vb.rho2));
                    dot[r] = fma(rza[r], rzb[r], ea.dot);
                    near |= dot[r] < ha;
                }
                const bool general = __builtin_amdgcn_ballot_w64(near) != 0ull;
#pragma unroll
                for (int r = 0; r < ZB; ++r) {
                    grad_term<T>(
                        fma(-rza[r], va.ey, ea.a), fma(rza[r], va.ex, -ea.b), ea.cz, dot[r], ha, la[r], lb[r],
                        [&](T& x, T& y, T& z) {
                            const GAux<T> a = buf.x[k > 0 ? k - 1 : 0];   // (record 0 is entered by no edge)
                            x = diff_of_products(a.ry, a.ez, rza[r], va.ey);
                            y = diff_of_products(rza[r], va.ex, a.rx, a.ez);
                            z = diff_of_products(a.rx, va.ey, a.ry, va.ex);
                        },
                        general, acc[r]);
                    rza[r] = rzb[r];
                    la[r] = lb[r];
                }
                va = vb;
                ea = eb;
                ha = hb;
            }
#pragma unroll
            for (int r = 0; r < ZB; ++r)
#pragma unroll
                for (int c = 0; c < 3; ++c) S[c * ZB + r] += (double)acc[r][c];
        }
    }
}

// Gradient on a grid: one wave per (column, z-chunk) as for w, ZB samples per lane
// (lane l holds samples l + 64 r of the chunk); SPLIT as for w.  AGAIN as for points: the call
// costs up to 4% (35 x 80 x 100 samples on a torus soup 8.3 ms, 7.95 without), the kernel behind
// 5 us and, at 512^3, 1%.
template <class T, int ZB, bool SPLIT, bool AGAIN>
__global__ __launch_bounds__(64 * (SPLIT ? kSplitWaves : kGridWaves)) void k_grad_grid(MeshView mv, GridArgs ga, FarView far,
                                                                                      int axis, T* __restrict__ g) {
    constexpr int W = SPLIT ? kSplitWaves : kGridWaves;
    __shared__ GBuf<T> buf[W];
    __shared__ double farv[SPLIT ? 1 : W][kFarV];
    __shared__ double part[SPLIT ? W : 1][SPLIT ? 64 * 3 * ZB : 1];
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lane = threadIdx.x & 63;
    const long long gw = ga.wave0 + (SPLIT ? (long long)blockIdx.x : (long long)blockIdx.x * W + wave);
    if (gw >= ga.nwaves) return;
    const long long col = gw / ga.nchunks;
    const int chunk = __builtin_amdgcn_readfirstlane((int)(gw - col * ga.nchunks));
    const int ci = __builtin_amdgcn_readfirstlane((int)(col / ga.ny));
    const int cj = __builtin_amdgcn_readfirstlane((int)(col - (long long)ci * ga.ny));
    const float px = grid_coord(ga.o[0], ga.s[0], ci);
    const float py = grid_coord(ga.o[1], ga.s[1], cj);
    const int nz = (int)ga.nz, k0 = chunk * 64 * ZB + lane;   // sample r is k0 + 64 r
    float pz[ZB], pzm = 0.f;
#pragma unroll
    for (int r = 0; r < ZB; ++r) {
        pz[r] = grid_coord(ga.o[2], ga.s[2], min(k0 + 64 * r, nz - 1));
        pzm = fmaxf(pzm, fabsf(pz[r]));
    }
    // one scale for the column: its lanes share the records
    for (int o = 32; o > 0; o >>= 1) pzm = fmaxf(pzm, __shfl_xor(pzm, o));
    const GPoint<T> p = grad_point<T>(mv.g, px, py, 0.f, pzm);
    constexpr T u = (T)1 / (T)kGradUnit<T>;
    const T s = far_scale<T>(px, py, pzm, mv.g.scale).scf * u;
    T pzs[ZB];
    double S[3 * ZB];
#pragma unroll
    for (int r = 0; r < ZB; ++r) {
        pzs[r] = (T)pz[r] * s;
        S[r] = S[ZB + r] = S[2 * ZB + r] = 0.0;
    }
    ChunkFilter flt{};
    flt.mode = ChunkFilter::kAll;
    if (far.on) {
        flt.mode = ChunkFilter::kNear;
        flt.x = far.cx[ci / far.bx];
        flt.y = far.cy[cj / far.by];
        flt.thr = far.thr;
    }
    grad_column<T, ZB>(mv, flt, p.x, p.y, pzs, p.f, S, SPLIT ? wave : 0, SPLIT ? W : 1, buf[wave]);
    if constexpr (SPLIT) {
        split_sum<3 * ZB, W>(wave, lane, S, part);
        if (wave > 0) return;
    }
    if (far.on)
        for (int c = 0; c < 3; ++c)
            far_add<ZB>(far, ci, cj, chunk * 64 * ZB, nz, c, S + c * ZB, farv[SPLIT ? 0 : wave]);
    const long long base = (long long)ci * ga.st[0] + (long long)cj * ga.st[1];
#pragma unroll
    for (int r = 0; r < ZB; ++r) {
        const int k = k0 + 64 * r;
        if (k >= nz) continue;
        T* out = g + 3 * (base + (long long)k * ga.st[2]);
        if constexpr (AGAIN) {
            grad_out<T>(mv, px, py, pz[r], S[r] * p.out, S[ZB + r] * p.out, S[2 * ZB + r] * p.out, axis, out);
        } else {
            for (int c = 0; c < 3; ++c) out[(c + axis) % 3] = (T)(S[c * ZB + r] * p.out);
        }
    }
}

__global__ __launch_bounds__(256) void k_grad_grid_again(MeshView mv, GridArgs ga, long long o0, long long n, int axis,
                                                         float* __restrict__ g) {
    const long long t = blockIdx.x * 256ll + threadIdx.x, o = o0 + t;   // in the output's order
    if (t >= n) return;
    const double s = (double)fabsf(g[3 * o]) + (double)fabsf(g[3 * o + 1]) + (double)fabsf(g[3 * o + 2]);
    if (s < 1e300) return;
    const float px = grid_coord(ga.o[0], ga.s[0], o / ga.st[0] % ga.nx);
    const float py = grid_coord(ga.o[1], ga.s[1], o / ga.st[1] % ga.ny);
    const float pz = grid_coord(ga.o[2], ga.s[2], o / ga.st[2] % ga.nz);
    grad_out<float>(mv, px, py, pz, s, s, s, axis, g + 3 * o);
}

// the sums at one level's nodes (gwn_far.h; see k_far_columns)
template <class T, int ZB, bool SPLIT>
__global__ __launch_bounds__(64 * (SPLIT ? kSplitWaves : kGridWaves)) void k_grad_far(MeshView mv, FarNodes f, int nchunks,
                                                                                     long long wave0, long long nwaves) {
    constexpr int W = SPLIT ? kSplitWaves : kGridWaves;
    __shared__ GBuf<T> buf[W];
    __shared__ double part[SPLIT ? W : 1][SPLIT ? 64 * 3 * ZB : 1];
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lane = threadIdx.x & 63;
    const long long gw = wave0 + (SPLIT ? (long long)blockIdx.x : (long long)blockIdx.x * W + wave);
    if (gw >= nwaves) return;
    const long long col = gw / nchunks;
    const int chunk = __builtin_amdgcn_readfirstlane((int)(gw - col * nchunks));
    const int ci = __builtin_amdgcn_readfirstlane((int)(col / f.nn[1]));
    const int cj = __builtin_amdgcn_readfirstlane((int)(col - (long long)ci * f.nn[1]));
    const int k0 = chunk * 64 * ZB + lane;
    constexpr T u = (T)1 / (T)kGradUnit<T>;
    T pzs[ZB];
    double S[3 * ZB];
#pragma unroll
    for (int r = 0; r < ZB; ++r) {
        pzs[r] = (T)f.pz[min(k0 + 64 * r, f.nn[2] - 1)] * u;
        S[r] = S[ZB + r] = S[2 * ZB + r] = 0.0;
    }
    grad_column<T, ZB>(mv, far_filter(f, ci, cj), (T)f.px[ci] * u, (T)f.py[cj] * u, pzs, u, S, SPLIT ? wave : 0,
                       SPLIT ? W : 1, buf[wave]);
    if constexpr (SPLIT) {
        split_sum<3 * ZB, W>(wave, lane, S, part);
        if (wave > 0) return;
    }
    double* out = f.T + ((size_t)ci * f.nn[1] + cj) * f.nn[2];
#pragma unroll
    for (int r = 0; r < ZB; ++r)
        if (k0 + 64 * r < f.nn[2])
            for (int c = 0; c < 3; ++c) out[c * f.tstep + k0 + 64 * r] = S[c * ZB + r];
}

template <class T, int ZB, bool SPLIT>
gwn_status launch_grad_far(const gwn_mesh_s* m, const FarNodes& f, hipStream_t st) {
    const int nchunks = (f.nn[2] + 64 * ZB - 1) / (64 * ZB);
    const long long nwaves = (long long)f.nn[0] * f.nn[1] * nchunks, most = max_launch_queries() / 64;
    for (long long w0 = 0; w0 < nwaves; w0 += most) {
        const long long n = std::min(most, nwaves - w0), blocks = SPLIT ? n : (n + kGridWaves - 1) / kGridWaves;
        k_grad_far<T, ZB, SPLIT><<<(unsigned)blocks, 64 * (SPLIT ? kSplitWaves : kGridWaves), 0, st>>>(
            m->view(), f, nchunks, w0, std::min(nwaves, w0 + most));
        GWN_HIP_TRY(hipGetLastError());
    }
    return GWN_OK;
}

template <class T, int ZB, bool SPLIT>
gwn_status launch_grad_columns(const gwn_mesh_s* m, GridArgs ga, const FarView& far, T* g, hipStream_t st) {
    ga.nchunks = (ga.nz + 64 * ZB - 1) / (64 * ZB);
    ga.nwaves = ga.nx * ga.ny * ga.nchunks;
    const long long kMaxWaves = max_launch_queries() / 64;
    constexpr bool kSingle = sizeof(T) == 4;   // (FP64 has nothing to take again)
    const bool again = kSingle && (SPLIT || m->nb < 512);
    for (long long w0 = 0; w0 < ga.nwaves; w0 += kMaxWaves) {
        ga.wave0 = w0;
        const long long n = std::min(kMaxWaves, ga.nwaves - w0), blocks = SPLIT ? n : (n + kGridWaves - 1) / kGridWaves;
        const int threads = 64 * (SPLIT ? kSplitWaves : kGridWaves);
        if (again) k_grad_grid<T, ZB, SPLIT, kSingle><<<(unsigned)blocks, threads, 0, st>>>(m->view(), ga, far, m->axis, g);
        else k_grad_grid<T, ZB, SPLIT, kSingle && SPLIT><<<(unsigned)blocks, threads, 0, st>>>(m->view(), ga, far, m->axis, g);
        GWN_HIP_TRY(hipGetLastError());
    }
    if constexpr (kSingle)
        if (!again) {
            launch_slices(ga.nx * ga.ny * ga.nz, 1, [&](int64_t o, int64_t n) {
                k_grad_grid_again<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(m->view(), ga, o, n, m->axis, g);
            });
            GWN_HIP_TRY(hipGetLastError());
        }
    return GWN_OK;
}

// The far part under the same conditions as for w (see launch_grid in grid.hip).
template <class T>
gwn_status launch_grad_grid(const gwn_mesh_s* m, const GridArgs& ga, T* g, hipStream_t st) {
    constexpr int prec = sizeof(T) == 8 ? GWN_PREC_FP64 : GWN_PREC_FP32;
    constexpr int ZB = 2;
    FarPlan p;
    void* ws = nullptr;
    if (!stream_captures(st)) p = far_plan(m, ga, prec, 3);
    if (p.levels > 0 && gwn::dmalloc_async(&ws, p.bytes, st) != hipSuccess) {
        (void)hipGetLastError();
        p.levels = 0;
    }
    gwn_status s = GWN_OK;
    if (p.levels > 0) {
        s = far_setup(p, m, ga, prec, ws, st);
        for (int l = 0; l < p.levels && s == GWN_OK; ++l) {
            const FarNodes f = far_nodes(p, l);
            const long long blocks = (f.nn[2] + 63) / 64;
            if ((long long)f.nn[0] * f.nn[1] * blocks < kFewWaves) s = launch_grad_far<T, 1, true>(m, f, st);
            else if (blocks == 1) s = launch_grad_far<T, 1, false>(m, f, st);
            else s = launch_grad_far<T, ZB, false>(m, f, st);
        }
        if (s == GWN_OK) s = far_transfer(p, st);
    }
    if (s == GWN_OK) {
        const FarView far = far_view(p);
        const long long blocks = (ga.nz + 63) / 64;
        if (split_gradient(ga.nx * ga.ny, blocks, m->nchunk, sizeof(T) == 8)) s = launch_grad_columns<T, 1, true>(m, ga, far, g, st);
        else if (blocks == 1) s = launch_grad_columns<T, 1, false>(m, ga, far, g, st);
        else s = launch_grad_columns<T, ZB, false>(m, ga, far, g, st);
    }
    if (ws) (void)hipFreeAsync(ws, st);
    return s;
}

}  // namespace

gwn_status query_grid_gradient(const gwn_mesh_s* m, const double* origin, const double* spacing, const int64_t* dims,
                               int prec, void* g, hipStream_t st) {
    GridArgs ga = frame_grid(m->axis, origin, spacing, dims);
    if (ga.nx == 0 || ga.ny == 0 || ga.nz == 0) return GWN_OK;
    if (prec == GWN_PREC_FP64) return launch_grad_grid<double>(m, ga, (double*)g, st);
    return launch_grad_grid<float>(m, ga, (float*)g, st);
}

gwn_status query_gradient(const gwn_mesh_s* m, const float* qx, const float* qy, const float* qz, int64_t qs,
                          int64_t nq, int prec, void* g, hipStream_t st) {
    const MeshView mv = m->view();
    axis_ptrs(m->axis, qx, qy, qz);
    const int64_t chunk = max_launch_queries();
    for (int64_t o = 0; o < nq; o += chunk) {
        const int64_t n = std::min<int64_t>(chunk, nq - o);
        const unsigned blocks = (unsigned)((n + 255) / 256);
        const float *x = qx + o * qs, *y = qy + o * qs, *z = qz + o * qs;
        if (want_split(m, n, -1)) {   // few points, many edges: a workgroup per point
            if (prec == GWN_PREC_FP64)
                k_grad_split<double><<<(unsigned)n, kSplitThreads, 0, st>>>(mv, x, y, z, qs, n, m->axis,
                                                                             (double*)g + 3 * o);
            else
                k_grad_split<float><<<(unsigned)n, kSplitThreads, 0, st>>>(mv, x, y, z, qs, n, m->axis,
                                                                            (float*)g + 3 * o);
        } else if (prec == GWN_PREC_FP64) {
            k_grad_batch<double, false><<<blocks, 256, 0, st>>>(mv, x, y, z, qs, n, m->axis, (double*)g + 3 * o);
        } else if (m->nb < 512) {
            k_grad_batch<float, true><<<blocks, 256, 0, st>>>(mv, x, y, z, qs, n, m->axis, (float*)g + 3 * o);
        } else {
            k_grad_batch<float, false><<<blocks, 256, 0, st>>>(mv, x, y, z, qs, n, m->axis, (float*)g + 3 * o);
            GWN_HIP_TRY(hipGetLastError());
            k_grad_again<<<blocks, 256, 0, st>>>(mv, x, y, z, qs, n, m->axis, (float*)g + 3 * o);
        }
        GWN_HIP_TRY(hipGetLastError());
    }
    return GWN_OK;
}

}  // namespace gwn

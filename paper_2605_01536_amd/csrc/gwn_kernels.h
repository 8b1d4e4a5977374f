// gwn_kernels.h -- device routines of the query path shared by the single-mesh
// kernels (query.hip) and the persistent multi-mesh kernel (multi.hip).
//
// Boundary term of the antipodal method (Eq. 10, Alg. 1):
//
//   w(p) = chi(+z) + (1/2pi) * sum over boundary edges (a,b) of atan2(N, D)
//
// where, with r = v - p, rho^2 = r_x^2 + r_y^2, l = |r| and
// s = l - r_z = rho^2 / (l + r_z) (the second form for r_z > 0),
//
//   N = r_a,y r_b,x - r_a,x r_b,y          (= l_a l_b  A . (B x x1))
//   D = s_a s_b + r_a,x r_b,x + r_a,y r_b,y (= l_a l_b (1 + A.B + A.x1 + B.x1))
//
// for x1 = -z.  Scaling both atan2 arguments by l_a l_b > 0 and writing D
// through s (an exact algebraic rearrangement) keeps FP32 accurate when a
// boundary vertex is close to the ray above the query.  Offsets are in
// fixed-point cell units: x and y from the quantised grid (exact integers),
// z from the input scaled by 2^k.  The atan2 branch where an edge passes over
// the ray (D <= 0) takes the sign of N from the exact perturbed predicate
// that also decides ray crossings (Supp. Sec. 2.1), so the integer jumps of
// chi and of the boundary sum coincide.
#pragma once

#include <algorithm>
#include <cmath>
#include <type_traits>

#include "gwn_internal.h"

namespace gwn {
namespace {

constexpr double kInv2Pi = 0.15915494309189533576888376337251;  // 1 / (2 pi)
constexpr double k2Pi = 6.283185307179586476925286766559;         // 2 pi

// atan(t) for |t| <= 1 as t + t x Q(x), x = t^2, Q of degree 7 fitted by the
// Remez exchange for minimax relative error (gen_atan_poly.py: 1.7e-8 in exact
// arithmetic, 9.2e-8 max / 2e-9 mean signed when evaluated in float32).
constexpr float kAtanQ[8] = {0.002920693f, -0.01636793f, 0.043211866f, -0.07552215f,
                             0.106660046f, -0.14211056f, 0.19993773f, -0.33333153f};
// atan(t) for |t| <= tan(pi/8) in double: Q of degree 9 interpolated at the
// Chebyshev nodes of [0, tan^2(pi/8)] (gen_atan_poly.py 9 double: |Q - h| <=
// 1e-15, relative error of atan <= 2e-16).
constexpr double kAtanQd[10] = {0.02277211404923737,  -0.044850509519182694, 0.05736903901999104,
                                -0.06649717364503759, 0.0769106629901103,    -0.09090853283150221,
                                0.11111109664858296,  -0.14285714266729652,  0.19999999999905727,
                                -0.33333333333333276};
// For |t| <= tan(pi/8) (the edge-pair path) atan(t) = t P(t^2), P of degree 4
// fitted to atan(sqrt x)/sqrt x by the Remez exchange (gen_atan_poly.py 4 pform:
// 1.8e-8 relative in exact arithmetic, 1.2e-7 max when evaluated in float32),
// so that a pair's arctangent accumulates in its final FMA.
constexpr float kAtanP[5] = {0.07986737f, -0.13852088f, 0.1997447f, -0.33332798f, 1.0f};
constexpr float kPi = 3.14159265358979f;
constexpr float kPi2 = 1.57079632679490f;

__device__ __forceinline__ float atan_unit(float t) {
    const float x = t * t;
    float q = kAtanQ[0];
#pragma unroll
    for (int k = 1; k < 8; ++k) q = fmaf(q, x, kAtanQ[k]);
    return fmaf(t * x, q, t);
}

// acc + atan(t) for |t| <= tan(pi/8) as fma(t, P(t^2), acc)
__device__ __forceinline__ float atan_pair_acc(float t, float acc) {
    const float x = t * t;
    float p = kAtanP[0];
#pragma unroll
    for (int k = 1; k < 5; ++k) p = fmaf(p, x, kAtanP[k]);
    return fmaf(t, p, acc);
}

// full-range atan2 built on atan_unit (octant reduction by min/max)
__device__ __forceinline__ float atan2_full(float y, float x) {
    const float ay = fabsf(y), ax = fabsf(x);
    const float mx = fmaxf(ay, ax), mn = fminf(ay, ax);
    const float t = mx > 0.f ? mn * __builtin_amdgcn_rcpf(mx) : 0.f;
    float a = atan_unit(t);
    a = ay > ax ? kPi2 - a : a;
    a = x < 0.f ? kPi - a : a;
    return copysignf(a, y);
}

// Arithmetic of the boundary loop per type.  kFast bounds |N|/D on the fast
// path (the range of the small-argument arctangent).
template <class T>
struct Arith;

template <>
struct Arith<float> {
    static constexpr float kFast = 1.0f;
    static __device__ __forceinline__ float sqrt(float x) { return __builtin_amdgcn_sqrtf(x); }
    static __device__ __forceinline__ float rcp(float x) { return __builtin_amdgcn_rcpf(x); }
    static __device__ __forceinline__ float atan_small(float t) { return atan_unit(t); }
    static __device__ __forceinline__ float atan2(float y, float x) { return atan2_full(y, x); }
};

template <>
struct Arith<double> {
    static constexpr double kFast = 0.41421356237;   // just below tan(pi/8)
    // hardware reciprocal square root, then one coupled Goldschmidt step on
    // (y ~ sqrt x, h ~ 1/(2 sqrt x)) and a final correction: correctly rounded on
    // 2^20 log-uniform arguments in [1e-12, 1e12], about half the cost of the
    // library square root; x = 0 gives 0
    static __device__ __forceinline__ double sqrt(double x) {
        const double r = __builtin_amdgcn_rsq(x);
        const double y0 = x * r, h0 = 0.5 * r;
        const double g = fma(-y0, h0, 0.5);
        const double y = fma(y0, g, y0), h = fma(h0, g, h0);
        const double s = fma(fma(-y, y, x), h, y);
        return x > 0.0 ? s : 0.0;
    }
    // hardware reciprocal refined by two Newton steps
    static __device__ __forceinline__ double rcp(double x) {
        double r = __builtin_amdgcn_rcp(x);
        double e = fma(-x, r, 1.0);
        r = fma(r, e, r);
        e = fma(-x, r, 1.0);
        return fma(r, e, r);
    }
    static __device__ __forceinline__ double atan_small(double t) {
        const double x = t * t;
        double q = kAtanQd[0];
#pragma unroll
        for (int k = 1; k < 10; ++k) q = fma(q, x, kAtanQd[k]);
        return fma(t * x, q, t);
    }
    // where the fast path would apply, its own expression, so that a lane gets
    // the same bits whichever path its wave takes (the FP32 full-range atan2
    // reduces to the same polynomial by construction)
    static __device__ __forceinline__ double atan2(double y, double x) {
        if (x > 0.0 && fabs(y) < kFast * x) return atan_small(y * rcp(x));
        return ::atan2(y, x);
    }
};

// ---------------------------------------------------------------- boundary loop
// x/y quantities of one boundary vertex relative to the query column (shared by
// all samples of a grid column; per lane in the batch kernels).
template <class T>
struct ColV {
    int dx, dy;
    T rx, ry, rho2;
};

// Offsets of a query outside the fixed-point box are taken in units of 2^e
// cells, e >= 0 chosen per query so that they stay below about 2^41: atan2(N, D)
// does not change under a common positive scale of all offsets, and FP32 would
// otherwise overflow N, D and rho^2 for queries ~1e10 mesh sizes away.  f = 2^-e
// scales the boundary vertices (exactly), scf = 2^(k-e) the query.
template <class T>
struct FarScale {
    T scf, f;
};

template <class T>
__device__ __forceinline__ FarScale<T> far_scale(float px, float py, float pz_abs_max, double scale) {
    const double M = fmax(fmax(fabs((double)px), fabs((double)py)), (double)pz_abs_max) * scale;
    const int e = M > 0x1p40 ? ilogb(M) - 40 : 0;
    FarScale<T> s;
    s.scf = (T)ldexp(scale, -e);
    s.f = (T)ldexp(1.0, -e);
    return s;
}

// value of x in lane l (uniform result)
template <class T>
__device__ __forceinline__ T wave_lane(T x, int l) {
    if constexpr (sizeof(T) == 4) {
        return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), l));
    } else {
        const long long v = __double_as_longlong(x);
        const int lo = __builtin_amdgcn_readlane((int)(v & 0xffffffffll), l);
        const int hi = __builtin_amdgcn_readlane((int)(v >> 32), l);
        return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
    }
}

// Edge pairs.  Inside the fixed-point box two consecutive edges with
// |N| < tan(pi/16) D each (a wave-uniform test) are summed by one arctangent:
// (D1 + i N1)(D2 + i N2) has argument atan(N1/D1) + atan(N2/D2) in
// (-pi/8, pi/8), so its real part is positive and atan(Im/Re) needs no branch
// fix-up and only the short-range polynomial.  Where ZB samples share one
// column's x/y (grids), N1 N2 is the column's and the product costs three
// operations per sample instead of a second reciprocal and arctangent.  FP32
// offsets are in units of 2^18 cells (an exact scale), and D <= 2^-50 of those
// units takes the single-edge path (products stay normal).
//
// On grids four edges with |N| < tan(pi/32) D each, decided by the column's x/y
// terms alone, take one arctangent likewise: the product of two pairs costs four
// more operations per sample and saves a reciprocal and a polynomial (ten).  That
// needs D^4 in FP32's range: with the samples within 2^32 cells of the box in z
// (quad_z) an offset is below 2^15 units and D below 2^30, and the x/y bound
// D > dot > kQuadDot = 2^-20 keeps the product above 2^-80.
template <class T, int ZB, bool FAR>
struct EdgePairs {
    static constexpr bool on = !FAR;
    static constexpr bool f32 = std::is_same<T, float>::value;
    static constexpr float kUnit = on && f32 ? 0x1p-18f : 1.0f;   // cell units per offset unit
    static constexpr float kInvTan = 5.02734f;                     // 1 / tan(pi/16), rounded up
    static constexpr float kInvTan4 = 10.15318f;                   // 1 / tan(pi/32), rounded up
    static constexpr float kMinD = 0x1p-50f;
    static constexpr float kQuadDot = 0x1p-20f;
    static constexpr float kTan8 = 0.41421354f;                    // just below tan(pi/8)
};

template <class T, int ZB, bool FAR, class V>
__device__ __forceinline__ ColV<T> col_vtx(const V& b, int qqx, int qqy, T pxs, T pys, T f) {
    ColV<T> c;
    c.dx = b.qx - qqx;
    c.dy = b.qy - qqy;
    if constexpr (FAR) {
        c.rx = fma((T)b.x, f, -pxs);
        c.ry = fma((T)b.y, f, -pys);
    } else {
        c.rx = (T)c.dx * (T)EdgePairs<T, ZB, FAR>::kUnit;
        c.ry = (T)c.dy * (T)EdgePairs<T, ZB, FAR>::kUnit;
    }
    c.rho2 = c.rx * c.rx + c.ry * c.ry;
    return c;
}

// a chained edge's x or y in offset units: as kept in FP32, from the integers in FP64
template <class T>
__device__ __forceinline__ T edge_e(float e, int d) {
    if constexpr (sizeof(T) == 4) return e;
    else return (T)d;
}

// N = r_a,y r_b,x - r_a,x r_b,y of the edge a -> b through the edge's own x, y (exact
// integers): r x e is the same for either endpoint's r, and with the nearer one its error
// goes with that distance times the edge's length, not with the product of the two
// distances.
template <class T>
__device__ __forceinline__ T edge_N(const ColV<T>& a, const ColV<T>& b, T ex, T ey) {
    const bool na = a.rho2 <= b.rho2;
    const T rx = na ? a.rx : b.rx, ry = na ? a.ry : b.ry;
    return ry * ex - rx * ey;
}

// s = l - r_z without cancellation
template <class T>
__device__ __forceinline__ T samp_s(T rho2, T rz) {
    const T l = Arith<T>::sqrt(rz * rz + rho2);
    const T t = l + fabs(rz);
    return rz > (T)0 ? rho2 * Arith<T>::rcp(t) : t;
}

// Rare path of one (sample, edge): exact atan2 branch where D <= 0 (sign of N from
// the perturbed predicate, or the perturbation limit for an endpoint on the ray),
// then the full-range atan2.  An endpoint on the sample's vertical line
// (dx = dy = 0, so rho = 0 exactly) lies on the ray above it exactly when its
// s = rho^2 / (l + r_z) is 0 (below it s = 2 |r_z| > 0); s = 0 with r_z = 0 is a
// vertex at the sample itself, on the surface, where w is undefined.
// CALL: FP64's arctangent by a call, see point_wide_call.
__device__ __attribute__((noinline)) double atan2_call(double y, double x) { return Arith<double>::atan2(y, x); }

template <class T, bool CALL = false>
__device__ __forceinline__ T edge_slow(const ColV<T>& a, const ColV<T>& b, T sa, T sb, T N, T D, bool exact) {
    if (exact && D <= (T)0) {
        const bool aon = (a.dx == 0) & (a.dy == 0) & (sa == (T)0);
        const bool bon = (b.dx == 0) & (b.dy == 0) & (sb == (T)0);
        if (aon && bon) {
            N = (T)0;
            D = (T)1;
        } else if (aon) {        // N ~ e1 rb_y - e2 rb_x,  D ~ -e1 rb_x - e2 rb_y
            if (b.ry != (T)0) { N = b.ry; D = -b.rx; }
            else if (b.rx > (T)0) { N = -(T)0; D = (T)-1; }
            else { N = (T)0; D = (T)1; }
        } else if (bon) {        // N ~ -e1 ra_y + e2 ra_x, D ~ -e1 ra_x - e2 ra_y
            if (a.ry != (T)0) { N = -a.ry; D = -a.rx; }
            else if (a.rx > (T)0) { N = (T)0; D = (T)-1; }
            else { N = (T)0; D = (T)1; }
        } else {
            const int o = orient_sos(a.dx, a.dy, b.dx, b.dy);   // N = -orient2d(a, b, q_eps)
            if (o > 0) N = -fabs(N);
            else if (o < 0) N = fabs(N);
        }
    }
    if constexpr (CALL && sizeof(T) == 8) return atan2_call(N, D);
    else return Arith<T>::atan2(N, D);
}

// One boundary edge for ZB samples given N and D.  Fast path (wave-uniform):
// every sample has |N| < kFast D, so atan2(N, D) = atan(N/D) with no branch
// fix-up.
template <class T, int ZB, bool FAR>
__device__ __forceinline__ void edge_finish(const ColV<T>& a, const ColV<T>& b, const T* sa, const T* sb, T N,
                                            const T* D, T* acc) {
    const T aN = fabs(N);
    bool slow = false;
#pragma unroll
    for (int r = 0; r < ZB; ++r) slow |= !(aN < Arith<T>::kFast * D[r]);
    if (__builtin_amdgcn_ballot_w64(slow) == 0ull) {
#pragma unroll
        for (int r = 0; r < ZB; ++r) acc[r] += Arith<T>::atan_small(N * Arith<T>::rcp(D[r]));
    } else {
#pragma unroll
        for (int r = 0; r < ZB; ++r) acc[r] += edge_slow<T, FAR>(a, b, sa[r], sb[r], N, D[r], !FAR);
    }
}

template <class T, int ZB, bool FAR>
__device__ __forceinline__ void edge_step(const ColV<T>& a, const ColV<T>& b, const T* sa, const T* sb, T* acc) {
    const T N = a.ry * b.rx - a.rx * b.ry;
    const T dot = a.rx * b.rx + a.ry * b.ry;
    T D[ZB];
#pragma unroll
    for (int r = 0; r < ZB; ++r) D[r] = sa[r] * sb[r] + dot;
    edge_finish<T, ZB, FAR>(a, b, sa, sb, N, D, acc);
}

// Inside the box x and y are within 2^31 cells of every boundary vertex but z
// is not bounded: a sample more than 2^40 cells above or below the box takes
// single edges (its offsets may even be infinite in FP32, which the single-edge
// form turns into the right limit), so an edge pair's product stays below 2^101
// in its units.
__device__ __forceinline__ bool near_z(float pz, const QGrid& g) {
    return fabs(((double)pz - g.lo[2]) * g.scale) <= 0x1p40;
}

__device__ __forceinline__ bool quad_z(float pz, const QGrid& g) {
    return fabs(((double)pz - g.lo[2]) * g.scale) <= 0x1p32;
}

// s of a vertex for ZB samples of a query outside the box (pzs in units of 2^e cells)
template <class T, int ZB>
__device__ __forceinline__ void load_vertex(const BVert& b, T pxs, T pys, const T* pzs, T f, ColV<T>& c, T* sv) {
    c = col_vtx<T, ZB, true>(b, 0, 0, pxs, pys, f);
#pragma unroll
    for (int r = 0; r < ZB; ++r) sv[r] = samp_s<T>(c.rho2, fma((T)b.z, f, -pzs[r]));
}

// Boundary sum S = sum of atan2 over the chained loops for ZB samples sharing one
// (x, y) outside the fixed-point box, raw offsets in units of 2^e cells, edge by edge.
// FP32 partials are flushed into the FP64 sum every 32 edges.
template <class T, int ZB>
__device__ __forceinline__ void boundary_loops_far(const MeshView& mv, T pxs, T pys, const T* pzs, double* S, T f) {
    const BVert* __restrict__ bv = mv.bverts;
    for (int l = 0; l < mv.nloops; ++l) {
        const int b0 = mv.loop_off[l], b1 = mv.loop_off[l + 1];
        ColV<T> cp, cq;
        T sp[ZB], sq[ZB];
        load_vertex<T, ZB>(bv[b0], pxs, pys, pzs, f, cp, sp);
        for (int j = b0 + 1; j <= b1;) {   // j = b1 closes the loop
            const int je = min(b1 + 1, j + 32);
            T acc[ZB];
#pragma unroll
            for (int r = 0; r < ZB; ++r) acc[r] = (T)0;
            for (; j < je; ++j) {
                load_vertex<T, ZB>(bv[j < b1 ? j : b0], pxs, pys, pzs, f, cq, sq);
                edge_step<T, ZB, true>(cp, cq, sp, sq, acc);
                cp = cq;
#pragma unroll
                for (int r = 0; r < ZB; ++r) sp[r] = sq[r];
            }
#pragma unroll
            for (int r = 0; r < ZB; ++r) S[r] += (double)acc[r];
        }
    }
}

// ---------------------------------------------------------------- grid columns
// In a grid column every sample shares x and y, so a boundary vertex's x/y
// terms (rho^2, and N, the x/y dot and the pair bound of its outgoing edge) are
// the same for the whole wave.  They are computed for 64 chained vertices (8
// chunks of the boundary) at a time, one vertex per lane, into records in LDS
// that every lane then reads at the same address (a broadcast): a wave
// instruction's worth of x/y work per vertex becomes one lane's.  What the x/y terms
// settle for all samples at once becomes bits of wave masks: whether the outgoing
// edge can share an arctangent, and whether the vertex is in the FARV case:
// every sample below it has r_z^2 <= 3 rho^2, where s = l - r_z = t - 2 max(r_z, 0)
// loses at most ~16 ulps to cancellation (its rounding error is ~2 u l, and
// s = rho^2 / (l + r_z) >= l / 8 there) and needs no reciprocal.  Between two chunks, and past a piece's end, stands an edge
// with N = 0 and x/y dot 1 (offset units squared): its D is positive whatever its
// vertices, so it adds an angle of 0 through the same instructions as any edge.
template <class T>
struct alignas(4 * sizeof(T)) ColRec {
    T zu;     // vertex z in offset units
    T rho2;   // r_x^2 + r_y^2 from the column
    T N;      // N of the outgoing edge (to the next vertex of the chunk)
    T dot;    // r_a,x r_b,x + r_a,y r_b,y of the outgoing edge
};

template <class T>
struct ColAux {   // read on the rare paths only
    T m;          // pair bound of the outgoing edge, max(|N| / tan(pi/16), kMinD)
    T rx, ry;
    int dx, dy;
};

constexpr int kColChunks = 8;   // chunks per fill
constexpr int kColRecs = kColChunks * kChunk;
static_assert(kColRecs == 64, "one lane per record");

template <class T>
struct ColBuf {
    ColRec<T> rec[kColRecs];
    ColAux<T> aux[kColRecs];
    int queue[64 + kColChunks];   // chunks waiting for a fill
};

// Which chunks a column sums (see gwn_far.h): all of them, those near its block
// of columns, or those far from the block but not from the block's parent.  Far
// from a block: the chunk's box and the block are at least thr cells apart in x
// or in y.
struct ChunkFilter {
    enum Mode { kAll, kNear, kRing } mode;
    int2 x, y;        // the block's quantised x and y ranges
    int thr;
    int2 px, py;      // its parent's (kRing; pthr < 0: no parent)
    int pthr;
};

__device__ __forceinline__ bool chunk_far(const int4& b, const int2& x, const int2& y, int thr) {
    return max(max(b.x - x.y, x.x - b.y), max(b.z - y.y, y.x - b.w)) >= thr;
}

__device__ __forceinline__ bool chunk_kept(const int4& b, const ChunkFilter& f) {
    const bool far = chunk_far(b, f.x, f.y, f.thr);
    if (f.mode == ChunkFilter::kNear) return !far;
    return far && !(f.pthr >= 0 && chunk_far(b, f.px, f.py, f.pthr));
}

// the wave reads what its own lanes wrote; LDS operations of a wave complete in order
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// A wave's way through the chunks that a filter keeps, 64 looked at a time, up to 8
// handed out at a time (every lane of the wave calls together).  parts > 1: only the
// part-th of `parts` shares of the chunks, dealt out in eights.
struct ChunkQueue {
    int* queue;   // the wave's LDS, 64 + kColChunks ints
    int base = 0, head = 0, have = 0, share, part, parts;

    __device__ __forceinline__ ChunkQueue(const MeshView& mv, int part_, int parts_, int* queue_)
        : queue(queue_), share((mv.nchunk + 8 * parts_ - 1) / (8 * parts_) * 8), part(part_), parts(parts_) {}

    // the number of chunks to take next (0: done); ids(n) are theirs
    __device__ __forceinline__ int next(const MeshView& mv, const ChunkFilter& flt) {
        const int lane = (int)(threadIdx.x & 63);
        if (have < kColChunks && base < share) {
            if (head > 0) {   // the rest to the front: fewer than 8 chunks
                const int t = lane < have ? queue[head + lane] : 0;
                wave_lds_sync();
                if (lane < have) queue[lane] = t;
                head = 0;
            }
            while (have < kColChunks && base < share) {
                const int j = base + lane, id = parts == 1 ? j : (j >> 3) * 8 * parts + part * 8 + (j & 7);
                const bool keep = j < share && id < mv.nchunk && (flt.mode == ChunkFilter::kAll || chunk_kept(mv.cbox[id], flt));
                const unsigned long long m = __builtin_amdgcn_ballot_w64(keep);
                if (keep)
                    queue[have + __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32),
                                                           __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u))] = id;
                have += __builtin_popcountll(m);
                base += 64;
            }
            wave_lds_sync();
        }
        return min(have, kColChunks);
    }
    __device__ __forceinline__ const int* ids(int n) {
        const int* q = queue + head;
        head += n;
        have -= n;
        return q;
    }
};

// Records of the chunks queue[0 .. n) (n <= 8), record k = 8 c + e for entry e of
// chunk c.  zmin: the samples' smallest z in offset units.  Bit k of m2 (m4): the edge
// leaving record k can be one of a pair (of four) on its x/y terms alone; of mf: its
// vertex is in the FARV case; of mt: it starts a loop of three edges.
template <class T, int ZB>
__device__ __forceinline__ void col_fill(const MeshView& mv, const int* queue, int n, int qqx, int qqy, T zmin,
                                         bool pairs, bool quads, ColBuf<T>& buf, unsigned long long& m2,
                                         unsigned long long& m4, unsigned long long& mf, unsigned long long& mt) {
    using P = EdgePairs<T, ZB, false>;
    constexpr T u = (T)P::kUnit;
    int lane = (int)(threadIdx.x & 63);
    // Opaque to the optimiser (no instruction is emitted): the record addresses
    // derived from the lane are then formed here, once per fill, instead of
    // being hoisted out of the boundary loops and held (or spilled) throughout.
    asm volatile("" : "+v"(lane));
    const int c = lane >> 3, en = lane & 7;
    bool e = false, e4 = false, ef = false, et = false;
    if (c < n) {
        const CVert* v = mv.chain + (size_t)queue[c] * kChunk;
        const CVert a = v[en], b = v[min(en + 1, kChunk - 1)];
        const ColV<T> ca = col_vtx<T, ZB, false>(a, qqx, qqy, (T)0, (T)0, (T)1);
        const ColV<T> cb = col_vtx<T, ZB, false>(b, qqx, qqy, (T)0, (T)0, (T)1);
        const bool edge = (a.flags & kChainEdge) != 0;
        et = (a.flags & kChainTri) != 0;
        ColRec<T> rc;
        rc.zu = u == (T)1 ? (T)a.z : (T)a.z * u;   // exact (u is a power of two)
        rc.rho2 = ca.rho2;
        rc.N = edge ? edge_N<T>(ca, cb, edge_e<T>(a.ex, b.qx - a.qx), edge_e<T>(a.ey, b.qy - a.qy)) : (T)0;
        rc.dot = edge ? ca.rx * cb.rx + ca.ry * cb.ry : (T)1;
        ColAux<T> ax;
        ax.m = fmax(fabs(rc.N) * (T)P::kInvTan, (T)P::kMinD);
        ax.rx = ca.rx;
        ax.ry = ca.ry;
        ax.dx = ca.dx;
        ax.dy = ca.dy;
        e = ax.m < rc.dot;
        e4 = fmax(fabs(rc.N) * (T)P::kInvTan4, (T)P::kQuadDot) < rc.dot;
        buf.rec[lane] = rc;
        buf.aux[lane] = ax;
        const T zr = u == (T)1 ? (T)a.z - zmin : fma((T)a.z, u, -zmin);   // the largest r_z
        ef = !((zr > (T)0) & (zr * zr > (T)3 * rc.rho2));
    }
    m2 = __builtin_amdgcn_ballot_w64(e && pairs);
    m4 = __builtin_amdgcn_ballot_w64(e4 && quads);
    mf = __builtin_amdgcn_ballot_w64(ef);
    mt = __builtin_amdgcn_ballot_w64(et);
    wave_lds_sync();
}

// s of a vertex for the lane's ZB samples (pz in offset units), and its
// outgoing edge's N and x/y dot
template <class T, int ZB, bool FARV = false>
__device__ __forceinline__ void col_vertex(const ColRec<T>& c, const T* pz, T* sv, T& N, T& dot) {
#pragma unroll
    for (int r = 0; r < ZB; ++r) {
        const T rz = c.zu - pz[r];
        const T t = Arith<T>::sqrt(rz * rz + c.rho2) + fabs(rz);
        if constexpr (FARV) sv[r] = fma((T)-2, fmax(rz, (T)0), t);
        else sv[r] = rz > (T)0 ? c.rho2 * Arith<T>::rcp(t) : t;
    }
    N = c.N;
    dot = c.dot;
}

template <class T>
__device__ __forceinline__ ColV<T> col_aux(const ColBuf<T>& buf, int k) {
    const ColAux<T> a = buf.aux[k];
    ColV<T> c;
    c.dx = a.dx;
    c.dy = a.dy;
    c.rx = a.rx;
    c.ry = a.ry;
    c.rho2 = (T)0;   // not used by edge_slow
    return c;
}

// One edge (record ka to record kb) given its D per sample: the fast form where
// every sample allows it, else the exact and full-range forms (edge_slow).
template <class T, int ZB>
__device__ __forceinline__ void col_finish(const ColBuf<T>& buf, int ka, int kb, const T* sa, const T* sb, T N,
                                           const T* D, T* acc) {
    const T aN = fabs(N);
    bool slow = false;
#pragma unroll
    for (int r = 0; r < ZB; ++r) slow |= !(aN < Arith<T>::kFast * D[r]);
    if (__builtin_amdgcn_ballot_w64(slow) == 0ull) {
#pragma unroll
        for (int r = 0; r < ZB; ++r) acc[r] += Arith<T>::atan_small(N * Arith<T>::rcp(D[r]));
    } else {
        const ColV<T> a = col_aux<T>(buf, ka), b = col_aux<T>(buf, kb);
#pragma unroll
        for (int r = 0; r < ZB; ++r) acc[r] += edge_slow<T>(a, b, sa[r], sb[r], N, D[r], true);
    }
}

// Two edges, record ka -> kb -> kc, given their D per sample: one arctangent for the
// pair where every sample of the wave allows it (known when ok), else one by one.
template <class T, int ZB>
__device__ __forceinline__ void col_pair(const ColBuf<T>& buf, int ka, int kb, int kc, T N1, T N2, T m1, bool ok,
                                         bool pairs, const T* sa, const T* sb, const T* sc, const T* D1, const T* D2,
                                         T* acc) {
    using P = EdgePairs<T, ZB, false>;
    bool pair = ok;
    if (!ok && pairs) {
        const T m2 = buf.aux[kb].m;
        bool slow = false;
#pragma unroll
        for (int r = 0; r < ZB; ++r) slow |= !(m1 < D1[r]) | !(m2 < D2[r]);
        pair = __builtin_amdgcn_ballot_w64(slow) == 0ull;
    }
    if (pair) {
        const T N12 = N1 * N2;
#pragma unroll
        for (int r = 0; r < ZB; ++r) {
            const T re = fma(D1[r], D2[r], -N12);
            const T im = fma(D1[r], N2, N1 * D2[r]);
            const T t = im * Arith<T>::rcp(re);
            if constexpr (P::f32) acc[r] = atan_pair_acc(t, acc[r]);
            else acc[r] += Arith<T>::atan_small(t);   // |t| < tan(pi/8)
        }
    } else {
        col_finish<T, ZB>(buf, ka, kb, sa, sb, N1, D1, acc);
        col_finish<T, ZB>(buf, kb, kc, sb, sc, N2, D2, acc);
    }
}

// Edges a -> b -> c -> d -> e known to take one arctangent on their x/y terms.
template <class T>
struct Pair {
    T re, im;
};

template <class T>
__device__ __forceinline__ Pair<T> edge_product(T N1, T D1, T N2, T D2) {
    return {fma(D1, D2, -(N1 * N2)), fma(D1, N2, N1 * D2)};
}

template <class T>
__device__ __forceinline__ Pair<T> edge_product(const Pair<T>& a, const Pair<T>& b) {
    return {fma(a.re, b.re, -(a.im * b.im)), fma(a.re, b.im, a.im * b.re)};
}

template <class T>
__device__ __forceinline__ T pair_acc(const Pair<T>& a, T acc) {
    const T t = a.im * Arith<T>::rcp(a.re);   // |t| < tan(pi/8)
    if constexpr (std::is_same<T, float>::value) return atan_pair_acc(t, acc);
    else return acc + Arith<T>::atan_small(t);
}

// Edges p -> k -> k + 1 -> k + 2 -> k + 3 (records), p's s, N and dot in sp, Np,
// dotp and replaced by record k + 3's.  FARV: all four vertices are in that case.
// TRI: the records are a loop of three edges (entered by an edge of no angle),
// whose last vertex, its first again, is not computed twice.
template <class T, int ZB, bool FARV, bool TRI>
__device__ __forceinline__ void col_quad(const ColBuf<T>& buf, int k, const T* pz, T* sp, T& Np, T& dotp, T* acc) {
    const ColRec<T> c0 = buf.rec[k], c1 = buf.rec[k + 1], c2 = buf.rec[k + 2];
    T sq[ZB], sr[ZB], N0, dot0, N1, dot1;
    Pair<T> g[ZB];
    if constexpr (TRI) {
        T N2, dot2;
        col_vertex<T, ZB, FARV>(c0, pz, sp, N0, dot0);
        col_vertex<T, ZB, FARV>(c1, pz, sq, N1, dot1);
        col_vertex<T, ZB, FARV>(c2, pz, sr, N2, dot2);
#pragma unroll
        for (int r = 0; r < ZB; ++r) {
            g[r] = edge_product<T>(N0, fma(sp[r], sq[r], dot0), N1, fma(sq[r], sr[r], dot1));
            acc[r] = pair_acc<T>(edge_product<T>(g[r], {fma(sr[r], sp[r], dot2), N2}), acc[r]);
        }
        Np = (T)0;
        dotp = (T)1;
    } else {
        const ColRec<T> c3 = buf.rec[k + 3];
        col_vertex<T, ZB, FARV>(c0, pz, sq, N0, dot0);
        col_vertex<T, ZB, FARV>(c1, pz, sr, N1, dot1);
#pragma unroll
        for (int r = 0; r < ZB; ++r)
            g[r] = edge_product<T>(Np, fma(sp[r], sq[r], dotp), N0, fma(sq[r], sr[r], dot0));
        col_vertex<T, ZB, FARV>(c2, pz, sq, N0, dot0);
        col_vertex<T, ZB, FARV>(c3, pz, sp, Np, dotp);
#pragma unroll
        for (int r = 0; r < ZB; ++r)
            acc[r] = pair_acc<T>(
                edge_product<T>(g[r], edge_product<T>(N1, fma(sr[r], sq[r], dot1), N0, fma(sq[r], sp[r], dot0))), acc[r]);
    }
}

// The same four edges where their x/y terms alone do not settle it: one arctangent
// where for every sample each angle is below pi/4 (|N| < D), so that the sum is the
// product's argument without a turn, and the sum below pi/8 (a missing triangle's
// loop, one trip, turns by half its solid angle however wide its edges look); else
// pair by pair, else edge by edge.  Bit i of b: the i-th edge pairs on its x/y terms.
template <class T, int ZB>
__device__ __forceinline__ void col_trip(const ColBuf<T>& buf, int k, unsigned b, bool pairs, bool quads, const T* pz,
                                         T* sp, T& Np, T& dotp, T* acc) {
    using P = EdgePairs<T, ZB, false>;
    const ColRec<T> c0 = buf.rec[k], c1 = buf.rec[k + 1], c2 = buf.rec[k + 2], c3 = buf.rec[k + 3];
    T s0[ZB], s1[ZB], s2[ZB], s3[ZB], D0[ZB], D1[ZB], D2[ZB], D3[ZB], N0, N1, N2, N3, dot0, dot1, dot2, dot3;
    col_vertex<T, ZB>(c0, pz, s0, N0, dot0);
    col_vertex<T, ZB>(c1, pz, s1, N1, dot1);
    col_vertex<T, ZB>(c2, pz, s2, N2, dot2);
    col_vertex<T, ZB>(c3, pz, s3, N3, dot3);
    const T b0 = fmax(fabs(Np), (T)P::kQuadDot), b1 = fmax(fabs(N0), (T)P::kQuadDot);
    const T b2 = fmax(fabs(N1), (T)P::kQuadDot), b3 = fmax(fabs(N2), (T)P::kQuadDot);
    Pair<T> g[ZB];
    bool slow = !quads;
#pragma unroll
    for (int r = 0; r < ZB; ++r) {
        D0[r] = fma(sp[r], s0[r], dotp);
        D1[r] = fma(s0[r], s1[r], dot0);
        D2[r] = fma(s1[r], s2[r], dot1);
        D3[r] = fma(s2[r], s3[r], dot2);
        g[r] = edge_product<T>(edge_product<T>(Np, D0[r], N0, D1[r]), edge_product<T>(N1, D2[r], N2, D3[r]));
        slow |= !(b0 < D0[r]) | !(b1 < D1[r]) | !(b2 < D2[r]) | !(b3 < D3[r]) | !(fabs(g[r].im) < (T)P::kTan8 * g[r].re);
    }
    if (__builtin_amdgcn_ballot_w64(slow) == 0ull) {
#pragma unroll
        for (int r = 0; r < ZB; ++r) acc[r] = pair_acc<T>(g[r], acc[r]);
    } else {
        // record 0 is entered by an edge of no angle, which takes no rare path
        const int kp = k > 0 ? k - 1 : 0;
        const T mp = k > 0 ? buf.aux[kp].m : (T)P::kMinD;
        col_pair<T, ZB>(buf, kp, k, k + 1, Np, N0, mp, (b & 3u) == 3u, pairs, sp, s0, s1, D0, D1, acc);
        col_pair<T, ZB>(buf, k + 1, k + 2, k + 3, N1, N2, buf.aux[k + 1].m, (b >> 2) == 3u, pairs, s1, s2, s3, D2, D3,
                        acc);
    }
#pragma unroll
    for (int r = 0; r < ZB; ++r) sp[r] = s3[r];
    Np = N3;
    dotp = dot3;
}

// Boundary sum over the chunks that `flt` keeps, added to S, for the ZB samples of
// each lane of a column inside the fixed-point box (qqx, qqy: the column's
// quantised x, y; pzs: the samples' z in cells).  z is monotone in the lane.  pairs: edge pairs allowed
// (see near_z); quads: products of four too (see quad_z).  FP32 partials are
// flushed to FP64 every 32 edges.  parts > 1: only the part-th of `parts` shares of
// the chunks, dealt out in eights.
template <class T, int ZB>
__device__ __forceinline__ void column_chunks(const MeshView& mv, const ChunkFilter& flt, int qqx, int qqy,
                                              const T* pzs, double* S, bool pairs, bool quads, int part, int parts,
                                              ColBuf<T>& buf) {
    constexpr T u = (T)EdgePairs<T, ZB, false>::kUnit;
    T pz[ZB];
#pragma unroll
    for (int r = 0; r < ZB; ++r) pz[r] = pzs[r] * u;
    // the samples are monotone in the lane, so each register's smallest z is in lane 0 or 63
    T zmin = (T)INFINITY;
#pragma unroll
    for (int r = 0; r < ZB; ++r) zmin = fmin(zmin, fmin(wave_lane<T>(pz[r], 0), wave_lane<T>(pz[r], 63)));
    // the chained vertex before the current record: none yet, so an edge of no angle
    T sp[ZB], Np = (T)0, dotp = (T)1;
#pragma unroll
    for (int r = 0; r < ZB; ++r) sp[r] = (T)1;
    ChunkQueue q(mv, part, parts, buf.queue);
    while (true) {
        const int n = q.next(mv, flt);
        if (n == 0) break;
        unsigned long long ms, mq, mf, mt;
        col_fill<T, ZB>(mv, q.ids(n), n, qqx, qqy, zmin, pairs, quads, buf, ms, mq, mf, mt);
        // bit k from here on: the edge entering record k (record 0 is entered by an edge of no angle)
        ms = (ms << 1) | (pairs ? 1ull : 0ull);
        mq = (mq << 1) | (quads ? 1ull : 0ull);
        const int nt = n * (kChunk / 4);   // trips of four vertices (two edge pairs): p-q-r, then r-q-p
        int t = 0;
        while (t < nt) {
            const int te = min(nt, t + 8);
            T acc[ZB];
#pragma unroll
            for (int r = 0; r < ZB; ++r) acc[r] = (T)0;
            while (t < te) {
                // trips whose four edges take one arctangent on their x/y terms alone
                for (; t < te && ((unsigned)(mq >> (4 * t)) & 15u) == 15u; ++t) {
                    const bool f = ((unsigned)(mf >> (4 * t)) & 15u) == 15u;
                    if ((mt >> (4 * t)) & 1ull) {
                        if (f) col_quad<T, ZB, true, true>(buf, 4 * t, pz, sp, Np, dotp, acc);
                        else col_quad<T, ZB, false, true>(buf, 4 * t, pz, sp, Np, dotp, acc);
                    } else {
                        if (f) col_quad<T, ZB, true, false>(buf, 4 * t, pz, sp, Np, dotp, acc);
                        else col_quad<T, ZB, false, false>(buf, 4 * t, pz, sp, Np, dotp, acc);
                    }
                }
                if (t >= te) break;
                col_trip<T, ZB>(buf, 4 * t, (unsigned)(ms >> (4 * t)) & 15u, pairs, quads, pz, sp, Np, dotp, acc);
                ++t;
            }
#pragma unroll
            for (int r = 0; r < ZB; ++r) S[r] += (double)acc[r];
        }
    }
}

// ---------------------------------------------------------------- points
// Boundary sum of one point inside the fixed-point box over chunks (see kChunk).  As in
// the grid columns up to four edges take one arctangent, but each lane chooses for its
// own point, so that a point's result does not depend on which points share its wave.
// No contraction in these functions: their operations, and with them the results, are
// the same in every kernel that calls them.
// Per edge about 35 VALU slots: per vertex 23 (the integer offsets and their conversion
// 8, r_z, l, s with a square root and a reciprocal of four slots each), per edge N, the
// x/y dot and D 5, a share of the product, the tests and the arctangent.
// *p at a wave-uniform address of data that no kernel of the launch writes, by scalar loads
// (the compiler takes vector loads for it in a kernel with atomics or LDS lists)
template <class X>
__device__ __forceinline__ X uniform_load(const X* p) {
    using W = std::conditional_t<sizeof(X) % 16 == 0, unsigned __attribute__((ext_vector_type(4))), unsigned>;
    static_assert(sizeof(X) % sizeof(W) == 0, "whole words");
    const unsigned long long a = (unsigned long long)p;
    const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)a);
    const unsigned hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(a >> 32));
    const auto q = (const __attribute__((address_space(4))) W*)(((unsigned long long)hi << 32) | lo);
    struct Words {
        W w[sizeof(X) / sizeof(W)];
    } u;
#pragma unroll
    for (unsigned i = 0; i < sizeof(X) / sizeof(W); ++i) u.w[i] = q[i];
    return __builtin_bit_cast(X, u);
}

template <class T>
struct PVert {
    int dx, dy;
    T rx, ry, rho2, s;
};

template <class T>
__device__ __forceinline__ PVert<T> point_vertex(const CVert& b, int qqx, int qqy, T pz) {
#pragma clang fp contract(off)
    constexpr T u = (T)EdgePairs<T, 1, false>::kUnit;
    PVert<T> v;
    v.dx = b.qx - qqx;
    v.dy = b.qy - qqy;
    v.rx = (T)v.dx * u;
    v.ry = (T)v.dy * u;
    v.rho2 = fma(v.rx, v.rx, v.ry * v.ry);
    const T rz = fma((T)b.z, u, -pz);
    const T l = Arith<T>::sqrt(fma(rz, rz, v.rho2));
    const T t = l + fabs(rz);
    v.s = rz > (T)0 ? v.rho2 * Arith<T>::rcp(t) : t;   // l - r_z without cancellation
    return v;
}

// N and D of the edge from entry ba to bb.  Where ba leads nowhere N is 0 (FP64: nothing beside
// D) and D > 0, no angle.  FP32 forms N from one endpoint's offset and the edge's own x, y (exact integers,
// kept in offset units): from the nearer one (NEARER) its error goes with that distance
// times the edge's length, see edge_N.  FP64 has the digits for the product of both.
template <class T, bool NEARER>
__device__ __forceinline__ T point_N(const CVert& ba, const PVert<T>& a, const PVert<T>& b) {
    if constexpr (sizeof(T) == 4) {
        const bool nb = NEARER && !(a.rho2 <= b.rho2);
        return fma(nb ? b.ry : a.ry, ba.ex, -((nb ? b.rx : a.rx) * ba.ey));
    } else {
        return fma(a.ry, b.rx, -(a.rx * b.ry));   // without an edge b is a: below 2^8, against D's 2^200
    }
}

template <class T>
__device__ __forceinline__ T point_D(const CVert& ba, const PVert<T>& a, const PVert<T>& b) {
    const T k = sizeof(T) == 4 ? (T)ba.none : (ba.flags & kChainEdge) ? (T)0 : (T)0x1p200;
    return fma(a.s, b.s, fma(a.rx, b.rx, fma(a.ry, b.ry, k)));
}

// the edge from entry b[0] to b[1], of any angle
template <class T>
__device__ __forceinline__ T point_wide_edge(const CVert* b, int qqx, int qqy, T pz) {
#pragma clang fp contract(off)
    const PVert<T> a = point_vertex<T>(b[0], qqx, qqy, pz), c = point_vertex<T>(b[1], qqx, qqy, pz);
    return edge_slow<T>({a.dx, a.dy, a.rx, a.ry, a.rho2}, {c.dx, c.dy, c.rx, c.ry, c.rho2}, a.s, c.s,
                        point_N<T, true>(b[0], a, c), point_D<T>(b[0], a, c), true);
}

// In FP64 by a call: with the library's arctangent inline a point per lane takes 162 registers,
// three waves per SIMD, without it 115, four (1.1 M points on a loop of 2,002 edges 4.43 ->
// 4.33 ms, 530 k on 1,026 short-looped edges 2.25 -> 2.21; in plans 173 and 127, 800 k queries on
// 100 such soups 3.42 -> 3.07 ms).
__device__ __attribute__((noinline)) double point_wide_call(const CVert* b, int qqx, int qqy, double pz) {
    return point_wide_edge<double>(b, qqx, qqy, pz);
}

template <class T>
__device__ __forceinline__ T point_wide(const CVert* b, int qqx, int qqy, T pz) {
    if constexpr (sizeof(T) == 8) return point_wide_call(b, qqx, qqy, pz);
    else return point_wide_edge<T>(b, qqx, qqy, pz);
}

// acc + the angles of n (2, 3 or 4) consecutive edges v[0] -> ... -> v[n].  By one
// arctangent of the product of the D + i N where each D > m >= the edge's squared length (FP32: so N from the first endpoint is off by about
// two ulps of D at most; also D > 0, and D^4 is far from FP32's ends, see quad_z) and the
// sum's tangent is below tan(pi/8) (up to three angles below pi/2 are it themselves; of four,
// the first two must be below pi/2 together).  Else each by its own where |N| < kFast D; the
// others are left out and set their bits in odd.
// WIDE (FP32, meshes of few chunks): half of the runs have a lane in their wave for which that
// does not do, and both forms are executed.  N from the nearer endpoint serves any D, and the
// product's full-range arctangent any sum: with each pair below pi/2 the four are below pi.
// 1.1 M points on 216 edges: 435 VALU instructions per chunk -> 369, 375 us -> 310 with the
// rest of the call; on longer boundaries the nearer endpoint costs 4% and gains nothing.
template <class T, int n, bool WIDE>
__device__ __forceinline__ T point_run(const CVert* b, const PVert<T>* v, bool quads, T acc, unsigned& odd) {
#pragma clang fp contract(off)
    using P = EdgePairs<T, 1, false>;
    T N[n], D[n];
    bool ok = quads;
#pragma unroll
    for (int i = 0; i < n; ++i) {
        N[i] = point_N<T, WIDE>(b[i], v[i], v[i + 1]);
        D[i] = point_D<T>(b[i], v[i], v[i + 1]);
        ok &= D[i] > (WIDE ? (T)P::kQuadDot : sizeof(T) == 4 ? (T)b[i].m : (T)1);
    }
    T gr = fma(D[0], D[1], -(N[0] * N[1])), gi = fma(D[0], N[1], D[1] * N[0]);
    if constexpr (n > 2) {
        T r2 = D[2], i2 = N[2];
        if constexpr (n == 4) {
            r2 = fma(D[2], D[3], -(N[2] * N[3]));
            i2 = fma(D[2], N[3], D[3] * N[2]);
            if constexpr (WIDE) ok &= r2 > (T)0;
        }
        if constexpr (n == 4 || WIDE) ok &= gr > (T)0;
        const T re = gr;
        gr = fma(re, r2, -(gi * i2));
        gi = fma(re, i2, gi * r2);
    }
    if constexpr (!WIDE) ok &= fabs(gi) < (T)P::kTan8 * gr;
    odd = 0u;
    if (ok) {
        if constexpr (WIDE) return acc + atan2_full(gi, gr);
        else return pair_acc<T>({gr, gi}, acc);
    }
#pragma unroll
    for (int i = 0; i < n; ++i) {
        T t;
        bool own;
        if constexpr (WIDE) {
            own = D[i] > (T)0;
            t = atan2_full(N[i], D[i]);
        } else {
            const T Ni = point_N<T, true>(b[i], v[i], v[i + 1]);
            own = fabs(Ni) < Arith<T>::kFast * D[i];
            t = Arith<T>::atan_small(Ni * Arith<T>::rcp(D[i]));
        }
        acc += own ? t : (T)0;
        odd |= own ? 0u : 1u << i;
    }
    return acc;
}

// The edges of one chunk: four if that is all, else the first three, then the other four,
// or (two halves) three, or the last two of them.  A loop's closing vertex is its first.
// UNIFORM: the same chunk for the wave; last: the chunk's last vertex; with cont, on entry
// that of the chunk before it.
struct Chunk {
    CVert v[kChunk];
};

template <class T, bool UNIFORM, bool WIDE = false>
__device__ __forceinline__ T point_chunk(const CVert* __restrict__ chunk, int qqx, int qqy, T pz, bool quads,
                                         PVert<T>& last, bool cont) {
    const CVert* b = chunk;
    Chunk c;
    if constexpr (UNIFORM) {
        c = uniform_load((const Chunk*)chunk);
        b = c.v;
    }
    auto vertex = [&](int e) { return point_vertex<T>(b[e], qqx, qqy, pz); };
    PVert<T> v[kChunk];
    T acc = (T)0;
    unsigned odd, odd1;
    v[0] = cont && (b[0].flags & kChainCont) ? last : vertex(0);
    v[1] = vertex(1);
    v[2] = vertex(2);
    v[3] = b[3].flags & kChainClose ? v[0] : vertex(3);
    if (!(b[4].flags & kChainEdge)) {
        if (b[3].flags & kChainEdge) {
            v[4] = b[4].flags & kChainClose ? v[0] : vertex(4);
            acc = point_run<T, 4, WIDE>(b, v, quads, acc, odd);
        } else {
            acc = point_run<T, 3, WIDE>(b, v, quads, acc, odd);
        }
    } else {
        acc = point_run<T, 3, WIDE>(b, v, quads, acc, odd);
        v[4] = vertex(4);
        v[5] = b[5].flags & kChainClose ? v[0] : vertex(5);
        if ((b[5].flags | b[6].flags) & kChainEdge) {
            v[6] = b[6].flags & kChainClose ? v[0] : vertex(6);
            if (!(b[6].flags & kChainEdge)) v[7] = v[6];   // no edge: any vertex
            else if (!(b[7].flags & kChainClose)) v[7] = vertex(7);
            else if (b[4].flags & kChainTri) v[7] = v[4];
            else v[7] = v[0];
            last = v[7];
            if (b[3].flags & kChainEdge) {
                acc = point_run<T, 4, WIDE>(b + 3, v + 3, quads, acc, odd1);
            } else {   // two halves
                acc = point_run<T, 3, WIDE>(b + 4, v + 4, quads, acc, odd1);
                odd1 <<= 1;
            }
        } else {
            acc = point_run<T, 2, WIDE>(b + 3, v + 3, quads, acc, odd1);
        }
        odd |= odd1 << 3;
    }
    while (odd) {
        const int e = __ffs(odd) - 1;
        odd &= odd - 1u;
        acc += point_wide<T>(chunk + e, qqx, qqy, pz);
    }
    return acc;
}

// FP32 sums are kept in units of 2^-e: rounded to whole units, the FP64 additions are
// exact up to 2^(53 - e), so that the order of the chunks and clusters, which differs
// between the kernels, does not show.  FP64 sums are plain.  e is 36, more for a point so
// far away that its terms are small: above the box they go with the height's inverse
// square, outside with the inverse distance, from the box in x and y or above it.  Below
// the box they do not fall: each tends to the angle that its edge has in x and y.
constexpr int kSumUnit = 36;

template <class T>
__device__ __forceinline__ void point_add(double& S, T v, int e) {
    if constexpr (sizeof(T) == 4) S += rint(ldexp((double)v, e));
    else S += v;
}

template <class T>
__device__ __forceinline__ double point_total(double S, int e) {
    return sizeof(T) == 4 ? ldexp(S, -e) : S;
}

__device__ __forceinline__ int point_unit(float px, float py, float pz, bool inbox, const QGrid& g) {
    double h = ((double)pz - g.lo[2]) * g.scale;
    if (!inbox)
        h = fmax(h, fmax(fabs(((double)px - g.lo[0]) * g.scale - 0x1p29), fabs(((double)py - g.lo[1]) * g.scale - 0x1p29)));
    if (!(h > 0x1p32 && h < 1e300)) return kSumUnit;
    const int k = ilogb(h) - 32;
    return kSumUnit + min(inbox ? 2 * k : k, 400);
}

// the sum over chunks c0, c0 + step, ..., < c1.  pz: the point's z in offset units
template <class T, bool UNIFORM, bool WIDE = false>
__device__ __forceinline__ void point_chunks(const MeshView& mv, int c0, int c1, int step, int qqx, int qqy, T pz,
                                             bool quads, int unit, double& S) {
    PVert<T> last = {};
    for (int c = c0; c < c1; c += step)
        point_add<T>(S, point_chunk<T, UNIFORM, WIDE>(mv.chain + (size_t)c * kChunk, qqx, qqy, pz, quads,
                                                last, UNIFORM && step == 1 && c > c0), unit);
}

// A point outside the box: boundary vertices [a, e), edge j leading from vertex j to the
// next vertex of its loop, raw offsets in units of 2^e cells.
template <class T>
__device__ T outside_run(const MeshView& mv, int a, int e, T pxs, T pys, T pzs, T f) {
    const BVert* __restrict__ bv = mv.bverts;
    ColV<T> cp;
    T sp;
    load_vertex<T, 1>(bv[a], pxs, pys, &pzs, f, cp, &sp);
    T acc = (T)0;
    for (int j = a; j < e; ++j) {
        const int lp = min(max(bv[j].loop, 0), mv.nloops - 1);   // in range for any stored value
        const int nx = j + 1 < mv.loop_off[lp + 1] ? j + 1 : mv.loop_off[lp];
        ColV<T> cn;
        T sn;
        load_vertex<T, 1>(bv[nx], pxs, pys, &pzs, f, cn, &sn);
        edge_step<T, 1, true>(cp, cn, &sp, &sn, &acc);
        if (j + 1 < e) {
            if (nx == j + 1) {
                cp = cn;
                sp = sn;
            } else {   // the next edge starts a new loop
                load_vertex<T, 1>(bv[j + 1], pxs, pys, &pzs, f, cp, &sp);
            }
        }
    }
    return acc;
}

// its whole sum, runs of 32 edges part, part + parts, ...
template <class T>
__device__ void outside_sum(const MeshView& mv, float px, float py, float pz, int part, int parts, int unit,
                            double& S) {
    const int nb = mv.nloops > 0 ? mv.loop_off[mv.nloops] : 0;
    const FarScale<T> fs = far_scale<T>(px, py, fabsf(pz), mv.g.scale);
    for (int a = part * 32; a < nb; a += parts * 32)
        point_add<T>(S, outside_run<T>(mv, a, min(nb, a + 32), (T)px * fs.scf, (T)py * fs.scf, (T)pz * fs.scf, fs.f), unit);
}

// ---------------------------------------------------------------- points, clusters
// The boundary sum of a cluster's loops from its expansion to degree P (see
// k_cluster_moments in build.hip for the formula; p: the point's raw position in cells).
// About 430 VALU slots for degree 10, 200 for 6, 120 for 4: as much as 12, 6 or 4 edges.
template <int P, bool UNIFORM>
__device__ __forceinline__ float cluster_far(const Cluster& k, const float4* __restrict__ W, float px, float py, float pz) {
#pragma clang fp contract(off)
    const float x0 = (px - k.x) * k.inva, y0 = (py - k.y) * k.inva, z0 = (pz - k.z) * k.inva;
    const float i2 = Arith<float>::rcp(fmaf(x0, x0, fmaf(y0, y0, z0 * z0)));
    const float x = x0 * i2, y = y0 * i2, z = z0 * i2;   // u = p / |p|^2, |u|^2 = i2
    auto w = [&](int i) {
        const float4 t = UNIFORM ? uniform_load(W + (i >> 2)) : W[i >> 2];
        return (i & 3) == 0 ? t.x : (i & 3) == 1 ? t.y : (i & 3) == 2 ? t.z : t.w;
    };
    float c = 1.f, s = 0.f, sum = 0.f;
#pragma unroll
    for (int m = 0; m <= P; ++m) {
        float q0 = 0.f, q1 = 1.f, re = 0.f, im = 0.f;
#pragma unroll
        for (int l = m; l <= P; ++l) {
            if (l >= 1) {
                re = fmaf(w(l * l - 1 + (m > 0 ? 2 * m - 1 : 0)), q1, re);
                if (m > 0) im = fmaf(w(l * l - 1 + 2 * m), q1, im);
            }
            const float beta = (float)(l * l - m * m) / (float)(4 * l * l - 1);
            const float t = l == m ? z * q1 : fmaf(z, q1, -(beta * i2) * q0);
            q0 = q1;
            q1 = t;
        }
        sum = fmaf(c, re, sum);
        if (m > 0) sum = fmaf(s, im, sum);
        const float t = fmaf(c, x, -(s * y));
        s = fmaf(s, x, c * y);
        c = t;
    }
    return sum * Arith<float>::sqrt(i2);
}

// The degree class (index into far2) with which a cluster may stand for its loops at a
// point, -1: none.  Beyond the distance, the vertical ray up from the point must miss the
// loops' box (a surface spanned inside it has no crossing to be counted in chi).
__device__ __forceinline__ int cluster_class(const Cluster& k, int qqx, int qqy, float px, float py, float pz) {
#pragma clang fp contract(off)
    const float x = px - k.x, y = py - k.y, z = pz - k.z, d2 = fmaf(x, x, fmaf(y, y, z * z));
    const bool aside = (qqx < k.xlo) | (qqx > k.xhi) | (qqy < k.ylo) | (qqy > k.yhi);
    if (!(aside | (pz > k.ztop))) return -1;
    return d2 >= k.far2[2] ? 2 : d2 >= k.far2[1] ? 1 : d2 >= k.far2[0] ? 0 : -1;
}

struct PointPos {
    int qx, qy;
    float x, y, z;   // cells
    bool quads;
    int unit;        // see point_unit
};

// One point per lane: the clusters in depth-first order, every step the same for the
// wave; a lane that took a cluster as far sits out its children (skip: the first cluster
// of the lowest level that the lane has not yet got).  Of the top level only clusters part,
// part + parts, ...
__device__ __forceinline__ double point_clusters(const MeshView& mv, const PointPos& p, int part, int parts) {
    double S = 0.0;
    if (mv.nclusters < kFewClusters) {
        if (mv.nchunk < kWideChunks)
            point_chunks<float, true, true>(mv, part, mv.nchunk, parts, p.qx, p.qy, p.z * 0x1p-18f, p.quads, p.unit, S);
        else
            point_chunks<float, true>(mv, part, mv.nchunk, parts, p.qx, p.qy, p.z * 0x1p-18f, p.quads, p.unit, S);
        return S;
    }
    int L = mv.top, i = part, skip = 0;
    while (true) {
        const int base = uniform_load(mv.level + L), id = base + i;
        if (id >= uniform_load(mv.level + L + 1)) break;
        const Cluster k = uniform_load(mv.clusters + id);
        const bool act = (i << (kFanBits * L)) >= skip;
        const int cls = act && p.quads ? cluster_class(k, p.qx, p.qy, p.x, p.y, p.z) : -1;
        const float4* W = (const float4*)(mv.moments + (size_t)id * kMoments);
        if (cls >= 0) {
            float v;
            if (cls == 2) v = cluster_far<kPolesLow, true>(k, W, p.x, p.y, p.z);
            else if (cls == 1) v = cluster_far<kPolesMid, true>(k, W, p.x, p.y, p.z);
            else v = cluster_far<kPoles, true>(k, W, p.x, p.y, p.z);
            point_add<float>(S, v, p.unit);
            skip = (i + 1) << (kFanBits * L);
        }
        if (__ballot(act && cls < 0)) {
            if (L > 0) {
                --L;
                i <<= kFanBits;
                continue;
            }
            if (act && cls < 0) point_chunks<float, true>(mv, k.first, k.first - k.count, 1, p.qx, p.qy, p.z * 0x1p-18f, p.quads, p.unit, S);
        }
        ++i;
        while (L < mv.top && (i & (kFan - 1)) == 0) {
            i >>= kFanBits;
            ++L;
        }
        if (L == mv.top) i += parts - 1;
    }
    return S;
}

// (Meshes of at least kWideChunks chunks or kFewClusters clusters: see point_run's WIDE.)
// G points per wave: the lanes share out (cluster, point) pairs to be tested, far pairs
// and (chunk, point) pairs of near clusters, each kind from a list in LDS, 64 at a time.
// For few points, or points so far apart that those of a wave of one point per lane would
// have few clusters in common.  A lane's moments are its own loads here, 30 of 16 bytes,
// and what bounds it is their way through the cache's address unit (64 lines a load where
// every lane has another cluster): neighbouring points in a group share those lines.
template <int G>
struct PointLists {
    PointPos p[G];
    double S[G];
    int far[3][128], far_pt[3][128];   // by degree class
    int leaf[128], leaf_mask[128];
    int sum[64];
};

// of the cluster stack (ids, then masks of points).  A step pops up to 64 / G entries and
// pushes up to kFan children of each, one level down; an entry's siblings are popped with
// or before it, so a level has at most kFan * 64 / G entries, less 64 / G while it has
// descendants on the stack.
template <int G>
constexpr size_t point_stack_ints(int top) {
    return (G == 1 ? 1 : 2) * (kRoots + (size_t)(kFan - 1) * (64 / G) * top + 64);
}

// The highest level for which four waves' lists and stacks fit the 64 KB of LDS that a launch
// may ask for: with a point per wave 470 million edges are too many, groups of four always fit.
constexpr int kSingleTop = 6;
static_assert(4 * sizeof(PointLists<1>) + 16 * point_stack_ints<1>(kSingleTop) <= 65000, "a point per wave");
static_assert(4 * sizeof(PointLists<4>) + 16 * point_stack_ints<4>(kLevels - 1) <= 65000, "groups");

__device__ __forceinline__ int lane_rank(unsigned long long m) {
    return __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
}

// position of the k-th set bit (k from 0, fewer than G set bits before the end)
template <int G>
__device__ __forceinline__ int nth_bit(unsigned m, int k) {
#pragma unroll
    for (int i = 0; i < G - 1; ++i)
        if (i < k) m &= m - 1;
    return __ffs(m) - 1;
}

// sums of the points ls.p[g] with a bit in mask, in their units: of point lane % G.
// parts > 1 (G = 1): that many waves walk the clusters alike and share out what they find,
// far clusters and near chunks; the part-th share.
template <int G>
__device__ __forceinline__ double point_group(const MeshView& mv, unsigned mask, int* stack, int stack_ints,
                                              PointLists<G>& ls, int part = 0, int parts = 1) {
    constexpr int kEntries = 64 / G;
    constexpr unsigned kAll = (1u << G) - 1u;
    const int lane = threadIdx.x & 63, pt = lane % G, en = lane / G;
    int* const smask = stack + stack_ints / 2;
    const PointPos mine = ls.p[pt];
    double S = 0.0;   // G == 1
    auto add = [&](int g, int unit, float v) {
        if constexpr (G == 1) point_add<float>(S, v, unit);
        else __hip_atomic_fetch_add(&ls.S[g], rint(ldexp((double)v, unit)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    };
    if (lane < G) ls.S[lane] = 0.0;
    const int root = uniform_load(mv.level + mv.top);
    int n = uniform_load(mv.level + mv.top + 1) - root, nleaf = 0, nfar[3] = {0, 0, 0}, turn = 0;
    if (lane < n) {
        stack[lane] = root + lane;
        if (G > 1) smask[lane] = (int)mask;
    }
    wave_lds_sync();
    while (true) {
        bool some = false;
#pragma unroll
        for (int f = 0; f < 3; ++f) {
            if (nfar[f] < 64 && (n > 0 || nfar[f] == 0)) continue;
            const int m = min(nfar[f], 64);
            nfar[f] -= m;
            const bool ours = turn++ % parts == part;
            if (lane < m && ours) {
                const int id = ls.far[f][nfar[f] + lane], g = G == 1 ? 0 : ls.far_pt[f][nfar[f] + lane];
                const PointPos p = G == 1 ? mine : ls.p[g];
                const Cluster& k = mv.clusters[id];
                const float4* W = (const float4*)(mv.moments + (size_t)id * kMoments);
                add(g, p.unit, f == 0   ? cluster_far<kPoles, false>(k, W, p.x, p.y, p.z)
                       : f == 1 ? cluster_far<kPolesMid, false>(k, W, p.x, p.y, p.z)
                                : cluster_far<kPolesLow, false>(k, W, p.x, p.y, p.z));
            }
            some = true;
        }
        if (some) {
            wave_lds_sync();
            continue;
        }
        if (nleaf >= 64 || (n == 0 && nleaf > 0)) {
            const int m = min(nleaf, 64);
            nleaf -= m;
            int c0 = 0, cn = 0;
            unsigned lm = 1u;
            if (lane < m) {
                const Cluster& k = mv.clusters[ls.leaf[nleaf + lane]];
                lm = G == 1 ? 1u : (unsigned)ls.leaf_mask[nleaf + lane];
                c0 = k.first;
                cn = -k.count * (G == 1 ? 1 : __popc(lm));
            }
            int t = cn;   // inclusive sums
            for (int d = 1; d < 64; d <<= 1) {
                const int o = __shfl_up(t, d);
                if (lane >= d) t += o;
            }
            ls.sum[lane] = t;
            const int total = __shfl(t, 63), before = t - cn;
            wave_lds_sync();
            for (int j0 = 64 * part; j0 < total; j0 += 64 * parts) {
                const int j = min(j0 + lane, total - 1);
                int a = 0;   // the first range whose sum exceeds j
                for (int h = 32; h > 0; h >>= 1)
                    if (ls.sum[a + h - 1] <= j) a += h;
                int r = j - __shfl(before, a), g = 0;
                if constexpr (G > 1) {
                    const unsigned am = (unsigned)__shfl((int)lm, a);
                    const int np = __popc(am), q = r / np;
                    g = nth_bit<G>(am, r - q * np);
                    r = q;
                }
                const int c = __shfl(c0, a) + r;
                const PointPos p = G == 1 ? mine : ls.p[g];
                PVert<float> end;
                if (j0 + lane < total)
                    add(g, p.unit, point_chunk<float, false>(mv.chain + (size_t)c * kChunk, p.qx, p.qy, p.z * 0x1p-18f, p.quads, end, false));
            }
            wave_lds_sync();
            continue;
        }
        if (n == 0) break;
        const int m = min(n, kEntries);
        n -= m;
        int cls = -2, id = 0, first = 0, count = 0;   // -2: no pair
        if (en < m && (G == 1 || ((unsigned)smask[n + en] >> pt & 1u))) {
            id = stack[n + en];
            const Cluster& k = mv.clusters[id];
            cls = mine.quads ? cluster_class(k, mine.qx, mine.qy, mine.x, mine.y, mine.z) : -1;
            first = k.first;
            count = k.count;
        }
        wave_lds_sync();
        const bool near = cls == -1;
#pragma unroll
        for (int f = 0; f < 3; ++f) {
            const unsigned long long b = __ballot(cls == f);
            if (cls == f) {
                ls.far[f][nfar[f] + lane_rank(b)] = id;
                if (G > 1) ls.far_pt[f][nfar[f] + lane_rank(b)] = pt;
            }
            nfar[f] += __popcll(b);
        }
        // one lane per entry that is near for some point: its first such point's
        unsigned long long b = __ballot(near);
        const unsigned nm = G == 1 ? (near ? 1u : 0u) : (unsigned)(b >> (en * G)) & kAll;
        const bool lead = near && (G == 1 || (nm & ((1u << pt) - 1u)) == 0u);
        b = __ballot(lead && count <= 0);
        if (lead && count <= 0) {
            ls.leaf[nleaf + lane_rank(b)] = id;
            if (G > 1) ls.leaf_mask[nleaf + lane_rank(b)] = (int)nm;
        }
        nleaf += __popcll(b);
        if (!lead) count = 0;
        if (__ballot(count > 0)) {
#pragma unroll
            for (int c = 0; c < kFan; ++c) {
                b = __ballot(c < count);
                if (c < count) {
                    stack[n + lane_rank(b)] = first + c;
                    if (G > 1) smask[n + lane_rank(b)] = (int)nm;
                }
                n += __popcll(b);
            }
        }
        wave_lds_sync();
    }
    if constexpr (G == 1) {
        for (int o = 32; o > 0; o >>= 1) S += __shfl_xor(S, o);
        return S;
    } else {
        return ls.S[pt];
    }
}

// points j0 ... j0 + m - 1 of the order perm (nullable), m <= G: w from chi and the sums
template <int G>
__device__ __forceinline__ void point_group_out(const MeshView& mv, const float* __restrict__ qx,
                                                const float* __restrict__ qy, const float* __restrict__ qz,
                                                long long qs, long long j0, int m, const int* __restrict__ perm,
                                                int* stack, int stack_ints, PointLists<G>& ls,
                                                const int* __restrict__ chi, float* __restrict__ w) {
    const int lane = threadIdx.x & 63;
    const long long j = j0 + min(lane, m - 1), i = perm ? (long long)perm[j] : j;
    const float px = qx[i * qs], py = qy[i * qs], pz = qz[i * qs];
    const QPoint q = quantize_point(px, py, pz, mv.g);
    const float sc = mv.g.scalef;
    const int unit = point_unit(px, py, pz, q.inbox, mv.g);
    if (lane < G) ls.p[lane] = {q.x, q.y, px * sc, py * sc, pz * sc, quad_z(pz, mv.g), unit};
    const unsigned in = (unsigned)__ballot(lane < m && q.inbox), out = (unsigned)__ballot(lane < m && !q.inbox);
    wave_lds_sync();
    double S = in && mv.nclusters > 0 ? point_group<G>(mv, in, stack, stack_ints, ls) : 0.0;
    for (int g = 0; g < m; ++g) {   // rare: outside the box
        if (!(out >> g & 1u)) continue;
        double So = 0.0;
        outside_sum<float>(mv, __shfl(px, g), __shfl(py, g), __shfl(pz, g), lane, 64, __shfl(unit, g), So);
        for (int o = 32; o > 0; o >>= 1) So += __shfl_xor(So, o);
        if (lane == g) S = So;
    }
    if (lane < m) w[i] = (float)((double)chi[i] + point_total<float>(S, unit) * kInv2Pi);
    wave_lds_sync();
}

// ---------------------------------------------------------------- grids

constexpr int kGridWaves = 4;  // waves per block in the wave-per-task kernels

// The grid in the frame of a mesh built along `axis`: frame axis c is world
// axis (c + axis) % 3; the output keeps the world layout (x slowest, z fastest).
inline GridArgs frame_grid(int axis, const double* origin, const double* spacing, const int64_t* dims) {
    GridArgs ga;
    const long long wst[3] = {dims[1] * dims[2], dims[2], 1};
    long long n[3];
    for (int c = 0; c < 3; ++c) {
        const int a = (c + axis) % 3;
        ga.o[c] = origin[a];
        ga.s[c] = spacing[a];
        n[c] = dims[a];
        ga.st[c] = wst[a];
    }
    ga.nx = n[0];
    ga.ny = n[1];
    ga.nz = n[2];
    ga.nchunks = ga.nwaves = ga.wave0 = 0;
    return ga;
}

// grid coordinate origin + (i + 0.5) * spacing in FP64, the product and the
// sum each rounded (no fused multiply-add: the pragma keeps the compiler from
// contracting them, which near a float32 rounding tie moves the sample by an
// ulp), then rounded to float32
__device__ __forceinline__ float grid_coord(double o, double s, long long i) {
#pragma clang fp contract(off)
    const double t = ((double)i + 0.5) * s;
    return (float)(o + t);
}

// Grids of few columns take the split form of the column kernels: a workgroup of
// kSplitWaves waves per column, one sample per lane, each wave a share of the chunks, the
// partial sums added in a fixed order.
constexpr long long kFewWaves = 4096;
constexpr int kSplitWaves = 8;

// Whether columns of `blocks` blocks of 64 samples are few: up to four waves per SIMD, FP64's w,
// whose registers leave room for fewer, up to two and a half, from three (which would be four) up
// to three and a half (from two up to three where a lane would take two samples else), and fewer
// where a wave's share of the chunks does not pay for what every wave of the column repeats:
// for w the crossings and, FP64, much of the work per vertex.  us split / not: w, 10 chunks 1,024 waves 58 / 33 (FP64 95 / 38), 36 chunks 2,115 waves 60 / 65 (155 /
// 113), 2,880 in pairs 69 / 84, 70 chunks 2,970 waves 71 / 79 (211 / 156), 150 chunks FP64 2,115
// waves 346 / 364, 2,970 467 / 411, 2,880 in pairs 450 / 514, 2,500 chunks 2,544 waves 4,538 /
// 4,762, 3,000 5,345 / 4,821, 3,127 5,760 / 6,420, 3,720 6,658 / 6,418, 2,880 in pairs 5,313 /
// 6,034; gradient, 10 chunks 576 waves 13 /
// 14 (27 / 17), 1,024 22 / 15 (30 / 17), 36 chunks 2,115 waves 40 / 52 (88 / 100), 2,970 51 / 54
// (114 / 102), 2,880 in pairs 52 / 74 (113 / 128), 70 chunks 4,032 waves 100 / 104 (214 / 217),
// 2,500 chunks FP64 4,032 7,990 / 8,801.
inline bool split_columns(long long columns, long long blocks, int64_t nchunk, bool f64) {
    const bool pairs = blocks == 2 || blocks > 3;
    const long long waves = columns * blocks, pays = (f64 ? 24 : 64) * nchunk;
    const long long most = !f64 ? kFewWaves : pairs ? 3200 : waves <= 3072 ? 2540 : nchunk < 2048 ? 3300 : 3520;
    return waves < std::min(most, (f64 ? pairs : blocks > 1) ? pays + pays / 2 : pays);
}
inline bool split_gradient(long long columns, long long blocks, int64_t nchunk, bool f64) {
    const long long pays = f64 ? 80 * (nchunk - 6) : 100 * (nchunk - 4);
    return columns * blocks < std::min(kFewWaves, blocks > 1 ? pays + pays / 2 : pays);
}

// the first wave's NV values per lane plus the other waves', in order
template <int NV, int W>
__device__ __forceinline__ void split_sum(int wave, int lane, double* S, double (*part)[64 * NV]) {
    if (wave > 0) {
#pragma unroll
        for (int r = 0; r < NV; ++r) part[wave][64 * r + lane] = S[r];
    }
    __syncthreads();
    if (wave == 0) {
        for (int v = 1; v < W; ++v) {
#pragma unroll
            for (int r = 0; r < NV; ++r) S[r] += part[v][64 * r + lane];
        }
    }
}

// ---------------------------------------------------------------- chi, batch

constexpr int kChiBlock = 64;

__device__ __forceinline__ int leaf_up(const MeshView& mv, int t, const QPoint& q) {
    return ray_up_hit(mv.tris[t], q.x, q.y, q.z);
}

// signed crossings of the +z ray from q: depth-first over the BVH with a
// per-lane stack in LDS (the radix tree over 62-bit keys is at most 63 deep)
__device__ int chi_up(const MeshView& mv, const QPoint& q, int* stk) {
    int node = mv.root;
    if (node == kNoRoot) return 0;
    if (node < 0) return leaf_up(mv, ~node, q);
    int c = 0, sp = 0;
    while (true) {
        const Node nd = mv.nodes[node];
        bool hl = box_has_xy(nd.lxy.x, nd.lxy.y, nd.lxy.z, nd.lxy.w, q.x, q.y) & (q.z <= nd.z.y);
        bool hr = box_has_xy(nd.rxy.x, nd.rxy.y, nd.rxy.z, nd.rxy.w, q.x, q.y) & (q.z <= nd.z.w);
        const int L = nd.link.x, R = nd.link.y;
        if (hl && L < 0) {
            c += leaf_up(mv, ~L, q);
            hl = false;
        }
        if (hr && R < 0) {
            c += leaf_up(mv, ~R, q);
            hr = false;
        }
        if (hl && hr) {
            stk[sp * kChiBlock] = R;
            ++sp;
            node = L;
        } else if (hl) {
            node = L;
        } else if (hr) {
            node = R;
        } else {
            if (sp == 0) break;
            --sp;
            node = stk[sp * kChiBlock];
        }
    }
    return c;
}

// chi_up of one point by a whole wave: a stack of nodes in LDS, up to 64 popped at a
// time, hit leaves tested 64 at a time.  A lane's walk is a chain of dependent loads, one
// per node on the way (some hundred); this is about one per level of the tree.  Near the
// stack's end nodes are popped singly, in depth-first order: at most one more entry per
// level, for which 64 are kept back (kLdsStack bounds the depth).
constexpr int kFrontier = 384;
struct ChiLists {
    int node[kFrontier];
    int leaf[192];
};

__device__ __forceinline__ int chi_up_wave(const MeshView& mv, const QPoint& q, ChiLists& ls) {
    if (mv.root == kNoRoot) return 0;
    if (mv.root < 0) return leaf_up(mv, ~mv.root, q);
    const int lane = threadIdx.x & 63;
    int c = 0, n = 1, nleaf = 0;
    if (lane == 0) ls.node[0] = mv.root;
    wave_lds_sync();
    while (n > 0 || nleaf > 0) {
        if (nleaf >= 64 || n == 0) {
            const int m = min(nleaf, 64);
            nleaf -= m;
            if (lane < m) c += leaf_up(mv, ls.leaf[nleaf + lane], q);
            wave_lds_sync();
            continue;
        }
        const int m = min(n, max(1, min(64, kFrontier - kLdsStack - n)));
        n -= m;
        bool hl = false, hr = false;
        int L = 0, R = 0;
        if (lane < m) {
            const Node nd = mv.nodes[ls.node[n + lane]];
            hl = box_has_xy(nd.lxy.x, nd.lxy.y, nd.lxy.z, nd.lxy.w, q.x, q.y) & (q.z <= nd.z.y);
            hr = box_has_xy(nd.rxy.x, nd.rxy.y, nd.rxy.z, nd.rxy.w, q.x, q.y) & (q.z <= nd.z.w);
            L = nd.link.x;
            R = nd.link.y;
        }
        wave_lds_sync();
        auto put = [&](bool hit, int link) {
            unsigned long long b = __ballot(hit && link < 0);
            if (hit && link < 0) ls.leaf[nleaf + lane_rank(b)] = ~link;
            nleaf += __popcll(b);
            b = __ballot(hit && link >= 0);
            if (hit && link >= 0) ls.node[n + lane_rank(b)] = link;
            n += __popcll(b);
        };
        put(hl, L);
        put(hr, R);
        wave_lds_sync();
    }
    for (int o = 32; o > 0; o >>= 1) c += __shfl_xor(c, o);
    return c;
}

// Signed crossings of the whole vertical line through q, split at q: up = the
// sum of s over crossings above q (chi along +z), down = minus the sum over
// crossings below it (chi along -z).  Same traversal as chi_up without the
// z pruning.
__device__ void chi_line(const MeshView& mv, const QPoint& q, int* stk, int& up, int& down) {
    up = down = 0;
    int node = mv.root;
    if (node == kNoRoot) return;
    auto leaf = [&](int t) {
        const TriQ tr = mv.tris[t];
        const int s = tri_xy_sign(tr, q.x, q.y);
        if (s == 0) return;
        if (plane_above(plane_of(tr, q.x, q.y), q.z)) up += s;
        else down -= s;
    };
    if (node < 0) {
        leaf(~node);
        return;
    }
    int sp = 0;
    while (true) {
        const Node nd = mv.nodes[node];
        bool hl = box_has_xy(nd.lxy.x, nd.lxy.y, nd.lxy.z, nd.lxy.w, q.x, q.y);
        bool hr = box_has_xy(nd.rxy.x, nd.rxy.y, nd.rxy.z, nd.rxy.w, q.x, q.y);
        const int L = nd.link.x, R = nd.link.y;
        if (hl && L < 0) {
            leaf(~L);
            hl = false;
        }
        if (hr && R < 0) {
            leaf(~R);
            hr = false;
        }
        if (hl && hr) {
            stk[sp * kChiBlock] = R;
            ++sp;
            node = L;
        } else if (hl) {
            node = L;
        } else if (hr) {
            node = R;
        } else {
            if (sp == 0) break;
            --sp;
            node = stk[sp * kChiBlock];
        }
    }
}

// Signed crossings of the lines of a wave's lanes, the wave walking the BVH
// together: it descends into a child when the line of ANY active lane meets
// the child's box (ballot), nodes and triangles arrive by scalar loads, and each
// active lane applies its own exact leaf test (u: crossings above q, d: minus
// those below).  UP: the +z ray only, the walk pruned by z (d then holds only
// the leaves it visited); otherwise the whole line.  Every lane of the wave
// calls it together; stk is the wave's LDS stack of kLdsStack entries (a
// child is pushed only where both are taken, so it never holds more entries
// than the tree is deep).
template <bool UP>
__device__ __forceinline__ void chi_wave_walk(const MeshView& mv, const QPoint& q, bool act, int* stk, int& u,
                                              int& d) {
    u = d = 0;
    auto leaf = [&](int t) {
        const TriQ tr = mv.tris[t];
        const int s = tri_xy_sign(tr, q.x, q.y);
        if (s == 0) return;
        if (plane_above(plane_of(tr, q.x, q.y), q.z)) u += s;
        else d -= s;
    };
    int node = mv.root;
    if (__builtin_amdgcn_ballot_w64(act) == 0ull || node == kNoRoot) return;
    if (node < 0) {
        if (act) leaf(~node);
        return;
    }
    int sp = 0;
    while (true) {
        const Node nd = mv.nodes[node];
        const bool ml = act && box_has_xy(nd.lxy.x, nd.lxy.y, nd.lxy.z, nd.lxy.w, q.x, q.y) && (!UP || q.z <= nd.z.y);
        const bool mr = act && box_has_xy(nd.rxy.x, nd.rxy.y, nd.rxy.z, nd.rxy.w, q.x, q.y) && (!UP || q.z <= nd.z.w);
        bool hl = __builtin_amdgcn_ballot_w64(ml) != 0ull;
        bool hr = __builtin_amdgcn_ballot_w64(mr) != 0ull;
        const int L = nd.link.x, R = nd.link.y;
        if (hl && L < 0) {
            if (ml) leaf(~L);
            hl = false;
        }
        if (hr && R < 0) {
            if (mr) leaf(~R);
            hr = false;
        }
        if (hl && hr) {
            stk[sp++] = R;   // every lane stores the same value
            node = L;
        } else if (hl) {
            node = L;
        } else if (hr) {
            node = R;
        } else {
            if (sp == 0) break;
            --sp;
            node = stk[sp];
        }
        node = __builtin_amdgcn_readfirstlane(node);
    }
}

}  // namespace
}  // namespace gwn

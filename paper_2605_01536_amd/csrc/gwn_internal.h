// gwn_internal.h -- device data layouts and exact predicates shared by the
// library's HIP sources (not part of the public ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace gwn {

constexpr long long kQMax = (1LL << 30) - 1;   // fixed-point coordinates live in [0, 2^30)
constexpr int kLdsStack = 64;  // per-lane BVH stack depth in LDS (a radix tree over 62-bit keys is <= 63 deep)

// Internal BVH node: boxes of both children (integer, fixed-point coords)
// plus the child links, 64 bytes = one fetch per visited node.
// link.x/.y: child >= 0 internal node, child < 0 leaf ~t (sorted triangle t);
// link.z: parent (-1 at the root).
struct alignas(16) Node {
    int4 lxy;   // left child  xlo, xhi, ylo, yhi
    int4 rxy;   // right child xlo, xhi, ylo, yhi
    int4 z;     // left zlo, left zhi, right zlo, right zhi
    int4 link;  // left, right, parent, and the other end of the leaf range that begins or
                // ends with the node's own index (k_karras writes it, k_refit reads it)
};

// Quantised triangle corners in Morton order (w unused).
struct alignas(16) TriQ {
    int4 a, b, c;
};

// One boundary-loop vertex, 32 bytes so a wave can fetch it with one scalar load.
// x, y, z: the input position times 2^k (an exact power-of-two scaling), i.e. in
// fixed-point cell units; qx, qy: the quantised x and y; loop: the loop it
// belongs to (its edge leads to the next vertex, or back to the loop's first).
struct alignas(32) BVert {
    float x, y, z;
    int qx, qy;
    int pad0, pad1;
    int loop;
};

// The boundary again as chunks of kChunk chained vertices (see k_emit_chain in
// build.hip): entry e of a chunk leads to entry e + 1 where flags & kChainEdge.
// A long loop is cut every kChunk - 1 edges, loops (or their ends) of at most
// three edges share a chunk in pairs; loops follow each other along a Hilbert
// curve, so a chunk is small.  Entries past a piece's end repeat a vertex, without an edge.
constexpr int kChunk = 8;
constexpr int kChainEdge = 1, kChainValid = 2;
constexpr int kChainTri = 4;    // first vertex of a loop of three edges
constexpr int kChainCont = 8;   // first of a chunk: the vertex that the chunk before ends with
constexpr int kChainClose = 16; // closes a loop that its chunk holds whole: the loop's first vertex again
struct alignas(32) CVert {
    float z;          // as BVert
    int qx, qy;
    float ex, ey;     // the edge's quantised x, y in units of 2^18 cells (0 without one)
    float m;          // the smallest D (units squared) that lets it share an arctangent, see point_run
    int flags;
    float none;       // added to D: 2^27 where there is no edge (x/y dot products inside the box stay above -2^26), 0 else
};

// Raw positions of the chain's vertices (BVert's x, y, z) and the flags, for the gradient.
struct alignas(16) GVertex {
    float x, y, z;
    int flags;
};

// A cluster: consecutive whole loops and the multipole expansion of their solid angle
// (see cluster_far).  kFan clusters of one level (in order) make one of the next, up to a
// level of at most kRoots.
struct alignas(64) Cluster {
    float x, y, z;            // centre, as BVert
    float inva;               // 1 / radius of the sphere about it that holds the loops
    float far2[3];            // squared distances (cells) from which degree kPoles, kPolesMid, kPolesLow will do
    float ztop;               // the loops' largest z
    int xlo, xhi, ylo, yhi;   // their quantised box
    int first, count;         // children; on the lowest level chunks, and minus their number
    float zlow;               // the loops' smallest z
    float area;               // of triangle fans spanning the loops, cells squared
};

constexpr int kFanBits = 3, kFan = 1 << kFanBits, kRoots = 64, kLevels = 12;

// Meshes of fewer clusters sum all edges: little is far from such a mesh's points, and the
// lanes of a wave of unordered points differ in what is (171 edges in 7 clusters, 2 M
// points: 0.44 ms with the expansions).
constexpr int kFewClusters = 16;

// Of these, meshes of fewer chunks have edges that look wide from most of their points: the FP32
// sums of their chunks have a form of their own (WIDE, see point_run), by a lane per point always.
constexpr int kWideChunks = 64;

constexpr int kPoles = 10, kPolesMid = 6, kPolesLow = 4;       // degrees of the expansions
constexpr int kMoments = (kPoles + 1) * (kPoles + 1) - 1;    // real coefficients, degree 1 up (l^2 - 1: degree l's first)

// Fixed-point grid parameters: q = rint((x - lo) * scale), scale = 2^k.
struct QGrid {
    double lo[3];
    double scale;
    float scalef;  // 2^k as float (cell units for the boundary term)
    int k;
};

// Read-only view of a built mesh handed to query kernels.
struct alignas(16) MeshView {
    const Node* nodes;
    const TriQ* tris;
    const BVert* bverts;
    const int* loop_off;   // nloops + 1 offsets into bverts
    const CVert* chain;    // kChunk vertices per chunk
    const GVertex* gchain;
    const Cluster* clusters;
    const float* moments;  // kMoments per cluster
    int nclusters;         // on the lowest level
    int top;               // the highest level
    const int* level;      // first cluster of each level, and the end of the last
    const int4* cbox;      // per chunk: quantised xlo, xhi, ylo, yhi
    int nchunk;
    int nloops;
    int nf;
    int root;              // >= 0 internal node, < 0 leaf ~t, INT_MIN when nf == 0
    int axis;              // ray axis of the mesh frame: 0 = z, 1 = x, 2 = y (see axis_ptrs)
    QGrid g;
};

constexpr int kNoRoot = (int)0x80000000;

// A cell-centred grid in the mesh frame; one wave per (column, z-chunk).
struct GridArgs {
    double o[3], s[3];
    long long nx, ny, nz;
    long long nchunks;   // z-chunks per column
    long long nwaves;    // columns * nchunks
    long long wave0;     // first wave of this launch (large grids take several)
    long long st[3];     // output strides of the frame's x, y, z indices (world z fastest)
};

// A mesh built along axis a works in the frame (X, Y, Z) = (x, y, z), (y, z, x)
// or (z, x, y) for a = 0 (z), 1 (x), 2 (y): a cyclic permutation, i.e. a
// rotation, so orientations and w are unchanged and the ray +Z is the chosen
// world axis.  Frame component c is world component (c + a) % 3.
__host__ __device__ inline void axis_ptrs(int a, const float*& x, const float*& y, const float*& z) {
    const float* t = x;
    if (a == 1) {
        x = y;
        y = z;
        z = t;
    } else if (a == 2) {
        x = z;
        z = y;
        y = t;
    }
}

// Fixed-point coordinate of one input value, evaluated in FP64 exactly as the
// rule states: rint((x - lo) * 2^k).  The multiply by a power of two is exact,
// so no contraction can change the result.
__device__ __forceinline__ double qround(float x, double lo, double scale) {
    return rint(((double)x - lo) * scale);
}

struct QPoint {
    int x, y, z;   // x, y valid when inbox; z clamped to [-1, 2^30]
    bool inbox;
};

__device__ __forceinline__ QPoint quantize_point(float px, float py, float pz, const QGrid& g) {
    QPoint q;
    double tx = qround(px, g.lo[0], g.scale);
    double ty = qround(py, g.lo[1], g.scale);
    double tz = qround(pz, g.lo[2], g.scale);
    q.inbox = (tx >= 0.0) && (tx <= (double)kQMax) && (ty >= 0.0) && (ty <= (double)kQMax);
    q.x = q.inbox ? (int)tx : 0;
    q.y = q.inbox ? (int)ty : 0;
    tz = fmin(fmax(tz, -1.0), (double)(kQMax + 1));   // NaN -> -1 via fmax
    q.z = (int)tz;
    return q;
}

// Position of the cell (x, y, z), 10 bits each, along a Hilbert curve (Skilling's transform
// of the axes, "Programming the Hilbert curve", 2004).  Consecutive cells touch, so a run
// of points in this order is compact; in Morton order one in ten runs of 28 edges of a
// torus of loops spans a jump and has twice the radius.
__device__ __forceinline__ uint32_t hilbert_key(uint32_t x, uint32_t y, uint32_t z) {
    uint32_t v[3] = {x & 1023u, y & 1023u, z & 1023u};
    for (uint32_t q = 512u; q > 1u; q >>= 1) {
        const uint32_t low = q - 1u;
        for (int a = 0; a < 3; ++a) {
            const uint32_t t = (v[a] & q) ? 0u : (v[0] ^ v[a]) & low;   // exchange the low bits, or
            v[0] ^= (v[a] & q) ? low : t;                               // invert the first axis'
            v[a] ^= t;
        }
    }
    v[1] ^= v[0];
    v[2] ^= v[1];
    uint32_t t = 0u;
    for (uint32_t q = 512u; q > 1u; q >>= 1)
        if (v[2] & q) t ^= q - 1u;
    uint32_t key = 0u;
    for (int b = 9; b >= 0; --b)
        for (int a = 0; a < 3; ++a) key = (key << 1) | (((v[a] ^ t) >> b) & 1u);
    return key;
}

// The traversal orders' key of a point: Morton order of 16 bits of x and y each (the rays
// are vertical), or (space) the Hilbert curve; points outside the box come last.
__device__ __forceinline__ uint32_t spread16(uint32_t v) {
    v &= 0xffffu;
    v = (v | (v << 8)) & 0x00ff00ffu;
    v = (v | (v << 4)) & 0x0f0f0f0fu;
    v = (v | (v << 2)) & 0x33333333u;
    v = (v | (v << 1)) & 0x55555555u;
    return v;
}

__device__ __forceinline__ uint32_t point_key(const QPoint& q, bool space) {
    const uint32_t z = (uint32_t)min(max(q.z, 0), (int)kQMax);
    if (space) return q.inbox ? hilbert_key((uint32_t)q.x >> 20, (uint32_t)q.y >> 20, z >> 20) : 0x3fffffffu;
    return q.inbox ? (spread16((uint32_t)q.x >> 14) | (spread16((uint32_t)q.y >> 14) << 1)) : 0xffffffffu;
}

__device__ __forceinline__ int sgnll(long long v) { return (v > 0) - (v < 0); }
__device__ __forceinline__ int sgni(int v) { return (v > 0) - (v < 0); }

// Sign of orient2d(a, b, q_eps) = cross(a - q_eps, b - q_eps) with the query
// perturbed by (e1, e2), 0 < e2 << e1.  In offsets d = vertex - q the value is
// cross(da, db) + e1 (da.y - db.y) + e2 (db.x - da.x): exactly linear in e.
__device__ __forceinline__ int orient_sos(int dax, int day, int dbx, int dby) {
    long long o = (long long)dax * dby - (long long)day * dbx;
    if (o != 0) return sgnll(o);
    if (day != dby) return day > dby ? 1 : -1;
    return sgni(dbx - dax);
}

// x/y part of the crossing of the vertical line through q_eps with one
// quantised triangle: 0 for a miss, else the common sign s of the three
// perturbed edge tests (= sign of the projected area).
__device__ __forceinline__ int tri_xy_sign(const TriQ& t, int qx, int qy) {
    const int ax = t.a.x - qx, ay = t.a.y - qy;
    const int bx = t.b.x - qx, by = t.b.y - qy;
    const int cx = t.c.x - qx, cy = t.c.y - qy;
    const int e0 = orient_sos(ax, ay, bx, by);
    const int e1 = orient_sos(bx, by, cx, cy);
    const int e2 = orient_sos(cx, cy, ax, ay);
    return (e0 != 0 && e0 == e1 && e0 == e2) ? e0 : 0;
}

// Supporting plane of a quantised triangle, prepared for many queries on one
// vertical line: f(qz) = n . (a - q) = f0 - n_z qz with
// f0 = n . (a - (qx, qy, 0)), n = (b - a) x (c - a).
struct PlaneQ {
    __int128 f0;
    long long nx, ny, nz;
};

__device__ __forceinline__ PlaneQ plane_of(const TriQ& t, int qx, int qy) {
    const long long ux = t.b.x - t.a.x, uy = t.b.y - t.a.y, uz = t.b.z - t.a.z;
    const long long vx = t.c.x - t.a.x, vy = t.c.y - t.a.y, vz = t.c.z - t.a.z;
    PlaneQ p;
    p.nx = uy * vz - uz * vy;
    p.ny = uz * vx - ux * vz;
    p.nz = ux * vy - uy * vx;
    p.f0 = (__int128)p.nx * (long long)(t.a.x - qx) + (__int128)p.ny * (long long)(t.a.y - qy) +
           (__int128)p.nz * (long long)t.a.z;
    return p;
}

// Whether the crossing lies on the +z side of q_eps: the sign of
// f(q_eps) = f - n_x e1 - n_y e2 - n_z e3 (real part, then -n_x, -n_y, -n_z)
// equals the sign of n_z.
__device__ __forceinline__ bool plane_above(const PlaneQ& p, int qz) {
    const __int128 f = p.f0 - (__int128)p.nz * qz;
    int side;
    if (f != 0) side = f > 0 ? 1 : -1;
    else if (p.nx != 0) side = -sgnll(p.nx);
    else if (p.ny != 0) side = -sgnll(p.ny);
    else side = -sgnll(p.nz);
    return side == sgnll(p.nz);
}

// Signed crossing of the +z ray from q_eps with one triangle: 0 if the line
// misses it or the crossing is below the query, else s.
__device__ __forceinline__ int ray_up_hit(const TriQ& t, int qx, int qy, int qz) {
    const int s = tri_xy_sign(t, qx, qy);
    if (s == 0) return 0;
    return plane_above(plane_of(t, qx, qy), qz) ? s : 0;
}

__device__ __forceinline__ bool box_has_xy(int xlo, int xhi, int ylo, int yhi, int qx, int qy) {
    return (qx >= xlo) & (qx <= xhi) & (qy >= ylo) & (qy <= yhi);
}

}  // namespace gwn

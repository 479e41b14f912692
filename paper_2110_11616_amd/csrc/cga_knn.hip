// k-nearest-neighbour search, Eq. (7)-(8) generalised to k, over a sorted
// unique MORTON key array, and plain binary-search point lookup.
//
// In Morton order voxels that are near in the array are near in space, so the
// array itself is the leaf level of a bounding-volume hierarchy, with no
// pointers and no sizes to compute: leaf j is the keys [16 j, 16 j + 16),
// node j of every level above is the 16 consecutive nodes [16 j, 16 j + 16)
// of the level below.  A node's record (32 bytes) holds the axis-aligned box
// of its voxels and an oriented one: on a surface the voxels of a node fill a
// thin slab along their least-variance direction, so the oriented box bounds
// a far query's distance to them far more tightly.  The build is one launch
// over the keys (tiles of 4096 keys give the leaves and the two levels above
// them, their boxes fitted to the voxels) and, from 2^16 keys on, one block
// for the few nodes of the levels above.
//
// Queries: a team of 16 lanes (a DPP row) answers one query at a time, one
// lane per child or voxel.  A step of a team takes the nearest open child of
// its current node: an inner node's 16 records are one coalesced load, each
// lane bounding its child's distance; a leaf's 16 voxels are one coalesced
// load, each lane taking its voxel's distance.  Children whose bound is
// strictly beyond the team's k-th distance are never taken (so ties
// survive); a node with no child left is climbed out of.  The team keeps one
// candidate list, ordered by (squared distance, key index), spread over its
// lanes.  The teams of a wave do not wait for each other: each goes on with
// its next query.
//
// Why: an octree walked by one lane per subtree (the former search) entered a
// node per voxel or two where the voxels are sparse, computed the child
// bounds of each node on one lane, and grew a cube around the query until it
// held k voxels; its build took a launch or three per level.
#include <cstdlib>
#include <map>
#include <mutex>
#include <tuple>

#include "cga_common.h"
#include "cga_sort.h"

namespace cga {

constexpr int kKnnBlock = 256;
constexpr int kTeam = 16;       // lanes per query, keys per leaf, children per node
constexpr int kTeamBits = 4;
constexpr int kBvhTile = 4096;  // keys per block of the build: 16 x 16 x 16
constexpr int kBvhLevels = 7;   // 2^31 keys: 16^7 leaves under 16 roots
constexpr uint32_t kPackedDepth = 15;              // deepest grid with 32-bit squared distances
// Large query sets are answered in the order of the top kOrderBits of their
// Morton keys (a 3-pass sort of index << kOrderBits | key bits), so that
// teams in flight at one time search neighbouring regions: shared nodes.
constexpr int kOrderBits = 24;
constexpr int64_t kOrderMin = (int64_t)1 << 18;
constexpr int kLinearSortCtr = 8;  // tile counters of the LINEAR keys' re-key sort (up to 8 passes)
// Query counters of the search: group g of G of the blocks (blockIdx mod G)
// answers queries g, g + G, ... from its own counter, a cache line apart.
// Atomics on one word take about 10 ns each, so one counter for all teams set
// the time of near queries (400k beside a LiDAR surface, k = 8: 3.9 ms, 1.1
// with the groups' counters, 1.3 with a counter per block, whose work differs
// too much).
constexpr int kQueryGroups = 32;
constexpr int kQueryCtrStride = 32;  // words
// Groups of a grid: at least eight blocks each, so that one block more or
// less in a group hardly unbalances them.
__device__ __forceinline__ uint32_t query_groups(uint32_t blocks) {
    const uint32_t g = blocks / 8;
    return g < 1 ? 1 : (g < kQueryGroups ? g : kQueryGroups);
}
constexpr int kLeafTrips = 4;      // leaves a team may visit per trip of the search loop

template <typename K>
__device__ __forceinline__ int64_t lower_bound_dev(const K *keys, int64_t n, K q) {
    if (n <= 0) return 0;
    int64_t lo = 0, len = n;
    while (len > 1) {
        int64_t half = len >> 1;
        lo = keys[lo + half] < q ? lo + half : lo;
        len -= half;
    }
    return lo + (keys[lo] < q ? 1 : 0);
}

// Number of keys: the device count when given, never above the host bound.
__device__ __forceinline__ int64_t key_count(int64_t n_host, const int64_t *d_n) {
    const int64_t n = dev_count(n_host, d_n);
    return n < n_host ? n : n_host;
}

// ------------------------------------------------------------- hierarchy
// Nodes of level l (0 = leaves) over n keys.
__host__ __device__ __forceinline__ int64_t bvh_nodes(int64_t n, int l) {
    const int b = kTeamBits * (l + 1);
    return (n + ((int64_t)1 << b) - 1) >> b;
}

// Where each level's records start, and the top level: the first of at most
// 16 nodes for the host bound n (a device count can only leave it fewer).
struct BvhShape {
    uint32_t off[kBvhLevels];
    int top;
    int64_t records;
};

static BvhShape bvh_shape(int64_t n) {
    BvhShape S{};
    int64_t at = 0;
    for (S.top = 0;; ++S.top) {
        S.off[S.top] = (uint32_t)at;
        at += bvh_nodes(n, S.top);
        if (bvh_nodes(n, S.top) <= kTeam || S.top == kBvhLevels - 1) break;
    }
    S.records = at > 0 ? at : 1;
    return S;
}

// A node's record, 32 bytes: the low and the high corner of its voxels (x |
// y << 21 | z << 42 each), then four 32-bit words with
//   the oriented box's frame (3 x 14 bits), its range [lo, hi] along each of
//   the frame's axes (12 bits a bound) and the voxels' mean (3 x 4 bits):
//   0: qx 0-13, qy 14-27, mean x 28-31;    1: qz 0-13, lo0 14-25, hi2 low 26-29;
//   2: hi0 0-11, lo1 12-23, mean y 24-27, mean z 28-31;
//   3: hi1 0-11, lo2 12-23, hi2 high 24-31.
// The frame's axes are the principal axes of the voxel positions, up to order
// and sign: the rotation onto them of least angle (at most 63 degrees), as a
// unit quaternion whose real part, at least 0.85, follows from the others.
// Ranges are of the voxels' offsets from the centre of the axis-aligned box,
// in units of its longest edge / 2048, rounded outwards (an offset is at most
// sqrt(3) / 2 of that edge).  The mean, in 16ths of the axis-aligned box,
// only guides the order of visits.
typedef unsigned long long u64x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__host__ __device__ __forceinline__ uint64_t pack_vox(uint32_t x, uint32_t y, uint32_t z) {
    return (uint64_t)x | ((uint64_t)y << 21) | ((uint64_t)z << 42);
}
__device__ __forceinline__ Vox unpack_vox(uint64_t v) {
    return Vox{(uint32_t)v & 0x1FFFFFu, (uint32_t)(v >> 21) & 0x1FFFFFu, (uint32_t)(v >> 42)};
}

struct Frame {
    float a[3][3];  // rows: the box's axes
};
constexpr float kQuatStep = 0.53f / 8191.f;  // sin of half the greatest angle is 0.522

__device__ __forceinline__ float bits_s(uint32_t w, int at, int n) {
    return (float)(int)__builtin_amdgcn_sbfe((int)w, at, n);
}

__device__ __forceinline__ Frame frame_decode(uint32_t w0, uint32_t w1) {
    const float x = bits_s(w0, 0, 14) * kQuatStep, y = bits_s(w0, 14, 14) * kQuatStep,
                z = bits_s(w1, 0, 14) * kQuatStep;
    const float xx = x * x, yy = y * y, zz = z * z;
    const float w = __builtin_amdgcn_sqrtf(fmaxf(1.f - xx - yy - zz, 0.f));
    const float x2 = x + x, y2 = y + y, z2 = z + z;
    Frame f;
    f.a[0][0] = 1.f - 2.f * (yy + zz);
    f.a[0][1] = x2 * y - z2 * w;
    f.a[0][2] = x2 * z + y2 * w;
    f.a[1][0] = x2 * y + z2 * w;
    f.a[1][1] = 1.f - 2.f * (xx + zz);
    f.a[1][2] = y2 * z - x2 * w;
    f.a[2][0] = x2 * z - y2 * w;
    f.a[2][1] = y2 * z + x2 * w;
    f.a[2][2] = 1.f - 2.f * (xx + yy);
    return f;
}

// The quaternion bits (w0, w1 of the record) of the axes n, e1, e2 (an
// orthonormal right-handed frame), in the order and with the signs that make
// the rotation's angle least.
__device__ __forceinline__ void frame_encode(const float u[3][3], uint32_t &w0, uint32_t &w1) {
    float best = -4.f, r[3][3];
#pragma unroll
    for (int p = 0; p < 6; ++p) {
        const int i0 = p % 3, odd = p / 3, i1 = (i0 + 1 + odd) % 3, i2 = (i0 + 2 - odd) % 3;
        const float a = u[i0][0], b = u[i1][1], c = u[i2][2];
        const float m = fminf(fminf(fabsf(a), fabsf(b)), fabsf(c));
        const bool neg = ((a < 0.f) != (b < 0.f)) != ((c < 0.f) != (odd != 0));
        const float tr = fabsf(a) + fabsf(b) + fabsf(c) - (neg ? 2.f * m : 0.f);
        if (tr > best) {
            best = tr;
            // signs that make the diagonal positive, but for its least
            // element when the frame would otherwise be left-handed
            bool fa = a < 0.f, fb = b < 0.f, fc = c < 0.f;
            if (neg) {
                const bool la = fabsf(a) == m, lb = !la && fabsf(b) == m;
                fa ^= la;
                fb ^= lb;
                fc ^= !la && !lb;
            }
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                r[0][k] = fa ? -u[i0][k] : u[i0][k];
                r[1][k] = fb ? -u[i1][k] : u[i1][k];
                r[2][k] = fc ? -u[i2][k] : u[i2][k];
            }
        }
    }
    const float inv = 0.5f / sqrtf(fmaxf(1.f + best, 1.f)) / kQuatStep;  // 1 / (4 w) in steps
    int q[3];
    const float v[3] = {r[2][1] - r[1][2], r[0][2] - r[2][0], r[1][0] - r[0][1]};
#pragma unroll
    for (int k = 0; k < 3; ++k) q[k] = min(max((int)rintf(v[k] * inv), -8191), 8191);
    w0 = ((uint32_t)q[0] & 0x3FFFu) | (((uint32_t)q[1] & 0x3FFFu) << 14);
    w1 = (uint32_t)q[2] & 0x3FFFu;
}

struct Box {
    uint32_t lo[3], hi[3];
};
// Centre and longest edge (in voxels, at least 1) of a box: exact in float
// (halves of integers below 2^22).
__device__ __forceinline__ void box_centre(const Box &b, float c[3], float &edge) {
    uint32_t e = 0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        c[a] = 0.5f * (float)(b.lo[a] + b.hi[a]);
        e = max(e, b.hi[a] - b.lo[a]);
    }
    edge = (float)(e + 1u);
}

// The frame of m voxels with sums s and products S (xx, yy, zz, xy, xz, yz)
// about any one point, as record bits.  The least-variance axis n comes from
// inverse iteration on the covariance by its adjugate, whose largest column
// already is nearly along n on a slab (power iteration from the other end
// does not converge where a node's voxels lie in two clumps; its loose boxes
// cost 1M queries over 20M sphere points twice the visits).  Any orthonormal
// frame is a valid one; only tightness depends on it.
__device__ __forceinline__ void fit_frame(float m, const float s[3], const float S[6], uint32_t &w0,
                                          uint32_t &w1) {
    const float inv = 1.f / m;
    const float mu0 = s[0] * inv, mu1 = s[1] * inv, mu2 = s[2] * inv;
    float xx = S[0] * inv - mu0 * mu0, yy = S[1] * inv - mu1 * mu1, zz = S[2] * inv - mu2 * mu2;
    float xy = S[3] * inv - mu0 * mu1, xz = S[4] * inv - mu0 * mu2, yz = S[5] * inv - mu1 * mu2;
    const float tr = xx + yy + zz, r = tr > 0.f ? 1.f / tr : 0.f;
    xx = xx * r + 1e-5f;
    yy = yy * r + 1e-5f;
    zz = zz * r + 1e-5f;
    xy *= r;
    xz *= r;
    yz *= r;
    const float A = yy * zz - yz * yz, B = xx * zz - xz * xz, C = xx * yy - xy * xy;
    const float D = xz * yz - xy * zz, E = xy * yz - xz * yy, F = xy * xz - xx * yz;
    float n0, n1, n2;
    if (A >= B && A >= C) {
        n0 = A;
        n1 = D;
        n2 = E;
    } else if (B >= C) {
        n0 = D;
        n1 = B;
        n2 = F;
    } else {
        n0 = E;
        n1 = F;
        n2 = C;
    }
#pragma unroll
    for (int it = 0; it < 3; ++it) {
        const float q = 1.f / fmaxf(fmaxf(fabsf(n0), fabsf(n1)), fmaxf(fabsf(n2), 1e-30f));
        n0 *= q;
        n1 *= q;
        n2 *= q;
        const float v0 = A * n0 + D * n1 + E * n2, v1 = D * n0 + B * n1 + F * n2,
                    v2 = E * n0 + F * n1 + C * n2;
        n0 = v0;
        n1 = v1;
        n2 = v2;
    }
    const float big = fmaxf(fmaxf(fabsf(n0), fabsf(n1)), fabsf(n2));
    if (!(big > 1e-30f)) {
        n0 = 0.f;
        n1 = 0.f;
        n2 = 1.f;
    } else {
        const float q = 1.f / big;
        n0 *= q;
        n1 *= q;
        n2 *= q;
        const float l = rsqrtf(n0 * n0 + n1 * n1 + n2 * n2);
        n0 *= l;
        n1 *= l;
        n2 *= l;
    }
    // axes across n: n x (the unit axis along which n is smallest), and n x that
    float c0, c1, c2;
    if (fabsf(n0) <= fabsf(n1) && fabsf(n0) <= fabsf(n2)) {
        c0 = 0.f;
        c1 = n2;
        c2 = -n1;
    } else if (fabsf(n1) <= fabsf(n2)) {
        c0 = -n2;
        c1 = 0.f;
        c2 = n0;
    } else {
        c0 = n1;
        c1 = -n0;
        c2 = 0.f;
    }
    const float rc = rsqrtf(c0 * c0 + c1 * c1 + c2 * c2);
    c0 *= rc;
    c1 *= rc;
    c2 *= rc;
    const float e0 = n1 * c2 - n2 * c1, e1 = n2 * c0 - n0 * c2, e2 = n0 * c1 - n1 * c0;
    // turned onto the covariance's principal axes across n: half the angle
    // of (cc - ee, 2 ce)
    const float g0 = xx * c0 + xy * c1 + xz * c2, g1 = xy * c0 + yy * c1 + yz * c2,
                g2 = xz * c0 + yz * c1 + zz * c2;
    const float h0 = xx * e0 + xy * e1 + xz * e2, h1 = xy * e0 + yy * e1 + yz * e2,
                h2 = xz * e0 + yz * e1 + zz * e2;
    const float cc = c0 * g0 + c1 * g1 + c2 * g2, ce = e0 * g0 + e1 * g1 + e2 * g2,
                ee = e0 * h0 + e1 * h1 + e2 * h2;
    const float p = cc - ee, q = 2.f * ce, hyp = sqrtf(p * p + q * q);
    const float cos2 = hyp > 0.f ? p / hyp : 1.f;
    const float ct = sqrtf(fmaxf(0.5f * (1.f + cos2), 0.f));
    const float st = copysignf(sqrtf(fmaxf(0.5f * (1.f - cos2), 0.f)), q);
    const float u[3][3] = {{n0, n1, n2},
                           {ct * c0 + st * e0, ct * c1 + st * e1, ct * c2 + st * e2},
                           {ct * e0 - st * c0, ct * e1 - st * c1, ct * e2 - st * c2}};
    frame_encode(u, w0, w1);
}

__device__ __forceinline__ void write_record(uint64_t *__restrict__ r, const Box &b, float edge,
                                             uint32_t w0, uint32_t w1, const float tmin[3],
                                             const float tmax[3], const float mean[3]) {
    // the slack covers the rounding of the projections
    const float inv = 2048.f / edge, slack = 1.f / 16.f;
    uint32_t lo[3], hi[3], mc[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        lo[k] = (uint32_t)min(max((int)floorf(tmin[k] * inv - slack), -2048), 2047) & 0xFFFu;
        hi[k] = (uint32_t)min(max((int)ceilf(tmax[k] * inv + slack), -2048), 2047) & 0xFFFu;
        const float at = (mean[k] + 0.5f - (float)b.lo[k]) * 16.f / (float)(b.hi[k] - b.lo[k] + 1u);
        mc[k] = (uint32_t)min(max((int)at, 0), 15);
    }
    u64x2 c;
    c.x = pack_vox(b.lo[0], b.lo[1], b.lo[2]);
    c.y = pack_vox(b.hi[0], b.hi[1], b.hi[2]);
    u32x4 w;
    w.x = w0 | (mc[0] << 28);
    w.y = w1 | (lo[0] << 14) | ((hi[2] & 15u) << 26);
    w.z = hi[0] | (lo[1] << 12) | (mc[1] << 24) | (mc[2] << 28);
    w.w = hi[1] | (lo[2] << 12) | ((hi[2] >> 4) << 24);
    *(u64x2 *)r = c;
    *(u32x4 *)(r + 2) = w;
}

// All-reduce over the 16 lanes of a DPP row by rotations.
template <int ROR>
__device__ __forceinline__ uint32_t row_ror(uint32_t x) {
    return (uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)x, 0x120 | ROR, 0xF, 0xF, false);
}
__device__ __forceinline__ uint32_t row_min(uint32_t x) {
    x = min(x, row_ror<8>(x));
    x = min(x, row_ror<4>(x));
    x = min(x, row_ror<2>(x));
    return min(x, row_ror<1>(x));
}
__device__ __forceinline__ uint32_t row_max(uint32_t x) { return ~row_min(~x); }
template <int ROR>
__device__ __forceinline__ float row_rorf(float x) {
    return __uint_as_float(row_ror<ROR>(__float_as_uint(x)));
}
__device__ __forceinline__ float row_sum(float x) {
    x += row_rorf<8>(x);
    x += row_rorf<4>(x);
    x += row_rorf<2>(x);
    return x + row_rorf<1>(x);
}
__device__ __forceinline__ float row_minf(float x) {
    x = fminf(x, row_rorf<8>(x));
    x = fminf(x, row_rorf<4>(x));
    x = fminf(x, row_rorf<2>(x));
    return fminf(x, row_rorf<1>(x));
}
__device__ __forceinline__ float row_maxf(float x) { return -row_minf(-x); }

// Reductions of the low build: over the thread itself (SCOPE 0), its row of
// 16 threads (1) or the block's 256 (2, through 16 words of LDS).
template <int SCOPE, typename T, typename F>
__device__ __forceinline__ T scoped(T v, F row, T *s_red) {
    if constexpr (SCOPE >= 1) v = row(v);
    if constexpr (SCOPE == 2) {
        __syncthreads();
        if ((threadIdx.x & 15) == 0) s_red[threadIdx.x >> 4] = v;
        __syncthreads();
        v = row(s_red[threadIdx.x & 15]);
    }
    return v;
}

// The record of the node made of each thread's own m voxels (its leaf's, in
// LDS), its row's or its block's; every thread of the scope returns with it
// written once.  Sums (count, offsets and products about the box centre) go
// to mom (nullable) for the levels above.
template <int SCOPE>
__device__ __forceinline__ void fit_node(const uint64_t *__restrict__ s_own, int m,
                                         uint64_t *__restrict__ rec, float *__restrict__ mom,
                                         bool writer, uint32_t *s_u, float *s_f) {
    Box b;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        b.lo[a] = ~0u;
        b.hi[a] = 0u;
    }
    for (int i = 0; i < m; ++i) {
        const Vox v = unpack_vox(s_own[i]);
        const uint32_t c[3] = {v.x, v.y, v.z};
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            b.lo[a] = min(b.lo[a], c[a]);
            b.hi[a] = max(b.hi[a], c[a]);
        }
    }
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        b.lo[a] = scoped<SCOPE>(b.lo[a], row_min, s_u);
        b.hi[a] = scoped<SCOPE>(b.hi[a], row_max, s_u);
    }
    float c[3], edge;
    box_centre(b, c, edge);
    float cnt = (float)m, s[3] = {0.f, 0.f, 0.f}, S[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    for (int i = 0; i < m; ++i) {
        const Vox v = unpack_vox(s_own[i]);
        const float d0 = (float)v.x - c[0], d1 = (float)v.y - c[1], d2 = (float)v.z - c[2];
        s[0] += d0;
        s[1] += d1;
        s[2] += d2;
        S[0] += d0 * d0;
        S[1] += d1 * d1;
        S[2] += d2 * d2;
        S[3] += d0 * d1;
        S[4] += d0 * d2;
        S[5] += d1 * d2;
    }
    cnt = scoped<SCOPE>(cnt, row_sum, s_f);
#pragma unroll
    for (int e = 0; e < 3; ++e) s[e] = scoped<SCOPE>(s[e], row_sum, s_f);
#pragma unroll
    for (int e = 0; e < 6; ++e) S[e] = scoped<SCOPE>(S[e], row_sum, s_f);
    uint32_t w0, w1;
    fit_frame(cnt, s, S, w0, w1);
    const Frame f = frame_decode(w0, w1);
    float tmin[3] = {3e38f, 3e38f, 3e38f}, tmax[3] = {-3e38f, -3e38f, -3e38f};
    for (int i = 0; i < m; ++i) {
        const Vox v = unpack_vox(s_own[i]);
        const float d0 = (float)v.x - c[0], d1 = (float)v.y - c[1], d2 = (float)v.z - c[2];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const float t = f.a[k][0] * d0 + f.a[k][1] * d1 + f.a[k][2] * d2;
            tmin[k] = fminf(tmin[k], t);
            tmax[k] = fmaxf(tmax[k], t);
        }
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        tmin[k] = scoped<SCOPE>(tmin[k], row_minf, s_f);
        tmax[k] = scoped<SCOPE>(tmax[k], row_maxf, s_f);
    }
    if (writer && cnt > 0.f) {
        const float mean[3] = {c[0] + s[0] / cnt, c[1] + s[1] / cnt, c[2] + s[2] / cnt};
        write_record(rec, b, edge, w0, w1, tmin, tmax, mean);
        if (mom) {
            mom[0] = cnt;
#pragma unroll
            for (int e = 0; e < 3; ++e) mom[1 + e] = s[e];
#pragma unroll
            for (int e = 0; e < 6; ++e) mom[4 + e] = S[e];
        }
    }
}

// Build, low levels: one block per kBvhTile keys, a thread per leaf.  The
// keys are checked (sorted, unique, within the grid), decoded once into vox
// (what a leaf visit of the search reads) and kept in LDS, from which each
// thread fits its leaf, each row of 16 threads the node of its 16 leaves and
// the block the node of those.  Bound: VALU work (the three fits over the
// voxels), about 16 bytes moved per key beside it.
template <typename K>
__global__ __launch_bounds__(256) void k_bvh_low(const K *__restrict__ keys, int64_t n_host,
                                                 const int64_t *d_n, uint32_t depth, BvhShape S,
                                                 uint64_t *__restrict__ vox,
                                                 uint64_t *__restrict__ rec,
                                                 float *__restrict__ mom,
                                                 uint32_t *__restrict__ qctr, uint32_t *err) {
    constexpr int kStride = kTeam + 1;  // LDS words per leaf, off by one against bank conflicts
    __shared__ uint64_t s_v[256 * kStride];
    __shared__ uint32_t s_u[16];
    __shared__ float s_f[16];
    const int64_t n = key_count(n_host, d_n), base = (int64_t)blockIdx.x * kBvhTile;
    const int tid = threadIdx.x;
    if (blockIdx.x == 0)  // the search's query counters start at zero
        for (int i = tid; i < kQueryGroups * kQueryCtrStride; i += 256) qctr[i] = 0;
    if (base >= n) return;  // block-uniform
    bool bad = false;
#pragma unroll 4
    for (int r = 0; r < kBvhTile / 256; ++r) {
        const int li = r * 256 + tid;
        const int64_t i = base + li;
        if (i < n) {
            const K k = keys[i];
            // not a CGA of this grid: unsorted, repeated, or wider than 3 * depth bits
            bad |= (i > 0 && k <= keys[i - 1]) || ((uint64_t)k >> (3 * depth)) != 0;
            const Vox v = dec3((uint64_t)k, depth, false);
            const uint64_t w = pack_vox(v.x, v.y, v.z);
            vox[i] = w;
            s_v[(li >> kTeamBits) * kStride + (li & (kTeam - 1))] = w;
        }
    }
    if (bad) set_err(err, ERR_MISMATCH);
    __syncthreads();
    const int64_t first = base + (int64_t)tid * kTeam;
    const int m = first < n ? (n - first < kTeam ? (int)(n - first) : kTeam) : 0;
    const uint64_t *own = s_v + tid * kStride;
    const int64_t leaf = (int64_t)blockIdx.x * 256 + tid, mid = leaf >> kTeamBits, high = blockIdx.x;
    fit_node<0>(own, m, rec + 4 * (S.off[0] + leaf), nullptr, m > 0, s_u, s_f);
    if (S.top >= 1)
        fit_node<1>(own, m, rec + 4 * (S.off[1] + mid), nullptr, (tid & 15) == 0, s_u, s_f);
    if (S.top >= 2)
        fit_node<2>(own, m, rec + 4 * (S.off[2] + high), S.top >= 3 ? mom + 10 * high : nullptr,
                    tid == 0, s_u, s_f);
}

struct Obb {
    Frame f;
    float lo[3], hi[3];  // in voxels from the box centre
};
__device__ __forceinline__ Obb obb_decode(u32x4 w, float edge) {
    Obb o;
    o.f = frame_decode(w.x, w.y);
    const float u = edge * (1.f / 2048.f);
    o.lo[0] = bits_s(w.y, 14, 12) * u;
    o.hi[0] = bits_s(w.z, 0, 12) * u;
    o.lo[1] = bits_s(w.z, 12, 12) * u;
    o.hi[1] = bits_s(w.w, 0, 12) * u;
    o.lo[2] = bits_s(w.w, 12, 12) * u;
    o.hi[2] = (float)((((int)w.w >> 24) << 4) | (int)((w.y >> 26) & 15u)) * u;
    return o;
}
__device__ __forceinline__ Box rec_box(u64x2 w) {
    const Vox l = unpack_vox(w.x), h = unpack_vox(w.y);
    return Box{{l.x, l.y, l.z}, {h.x, h.y, h.z}};
}

// Build, the levels above the block nodes (from 2^16 keys on; a few hundred
// nodes for 20M keys): one block, a row of 16 lanes per node, a lane per
// child.  The direction comes from the children's sums, the ranges from the
// corners of their oriented boxes.
constexpr int kBvhHighBlock = 1024;

__global__ __launch_bounds__(kBvhHighBlock) void k_bvh_high(int64_t n_host, const int64_t *d_n,
                                                            BvhShape S, uint64_t *__restrict__ rec,
                                                            float *__restrict__ mom) {
    const int64_t n = key_count(n_host, d_n);
    const int row = threadIdx.x >> kTeamBits, tl = threadIdx.x & (kTeam - 1);
    for (int l = 3; l <= S.top; ++l) {
        const int64_t nodes = bvh_nodes(n, l), kids = bvh_nodes(n, l - 1);
        for (int64_t j = row; j < nodes; j += kBvhHighBlock / kTeam) {
            const int64_t c = j * kTeam + tl;
            const bool has = c < kids;
            const uint64_t *r = rec + 4 * ((int64_t)S.off[l - 1] + (has ? c : j * kTeam));
            const Box cb = rec_box(*(const u64x2 *)r);
            const u32x4 cw = *(const u32x4 *)(r + 2);
            Box b;
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                b.lo[a] = row_min(cb.lo[a]);  // a lane without a child repeats the first
                b.hi[a] = row_max(cb.hi[a]);
            }
            float pc[3], pe, cc[3], ce;
            box_centre(b, pc, pe);
            box_centre(cb, cc, ce);
            const float *cm = mom + 10 * ((int64_t)S.off[l - 1] - S.off[2] + (has ? c : j * kTeam));
            const float m = has ? cm[0] : 0.f;
            const float s0 = has ? cm[1] : 0.f, s1 = has ? cm[2] : 0.f, s2 = has ? cm[3] : 0.f;
            const float d0 = cc[0] - pc[0], d1 = cc[1] - pc[1], d2 = cc[2] - pc[2];
            float s[3] = {s0 + m * d0, s1 + m * d1, s2 + m * d2};
            float P[6] = {2.f * d0 * s0 + m * d0 * d0, 2.f * d1 * s1 + m * d1 * d1,
                          2.f * d2 * s2 + m * d2 * d2, d0 * s1 + d1 * s0 + m * d0 * d1,
                          d0 * s2 + d2 * s0 + m * d0 * d2, d1 * s2 + d2 * s1 + m * d1 * d2};
            const float cnt = row_sum(m);
#pragma unroll
            for (int e = 0; e < 3; ++e) s[e] = row_sum(s[e]);
#pragma unroll
            for (int e = 0; e < 6; ++e) P[e] = row_sum(P[e] + (has ? cm[4 + e] : 0.f));
            uint32_t w0, w1;
            fit_frame(cnt, s, P, w0, w1);
            const Frame f = frame_decode(w0, w1);
            const Obb o = obb_decode(cw, ce);
            float tmin[3] = {3e38f, 3e38f, 3e38f}, tmax[3] = {-3e38f, -3e38f, -3e38f};
#pragma unroll
            for (int corner = 0; corner < 8; ++corner) {
                const float t0 = (corner & 1) ? o.hi[0] : o.lo[0], t1 = (corner & 2) ? o.hi[1] : o.lo[1],
                            t2 = (corner & 4) ? o.hi[2] : o.lo[2];
                const float p0 = d0 + t0 * o.f.a[0][0] + t1 * o.f.a[1][0] + t2 * o.f.a[2][0];
                const float p1 = d1 + t0 * o.f.a[0][1] + t1 * o.f.a[1][1] + t2 * o.f.a[2][1];
                const float p2 = d2 + t0 * o.f.a[0][2] + t1 * o.f.a[1][2] + t2 * o.f.a[2][2];
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    const float t = f.a[k][0] * p0 + f.a[k][1] * p1 + f.a[k][2] * p2;
                    tmin[k] = fminf(tmin[k], t);
                    tmax[k] = fmaxf(tmax[k], t);
                }
            }
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                // never wider than the axis-aligned box's own extent along the axis
                const float sup = 0.5f * (fabsf(f.a[k][0]) * (float)(b.hi[0] - b.lo[0]) +
                                          fabsf(f.a[k][1]) * (float)(b.hi[1] - b.lo[1]) +
                                          fabsf(f.a[k][2]) * (float)(b.hi[2] - b.lo[2]));
                tmin[k] = fmaxf(row_minf(tmin[k]), -sup);
                tmax[k] = fminf(row_maxf(tmax[k]), sup);
            }
            if (tl == 0) {
                const float mean[3] = {pc[0] + s[0] / cnt, pc[1] + s[1] / cnt, pc[2] + s[2] / cnt};
                write_record(rec + 4 * ((int64_t)S.off[l] + j), b, pe, w0, w1, tmin, tmax, mean);
                float *pm = mom + 10 * ((int64_t)S.off[l] - S.off[2] + j);
                pm[0] = cnt;
#pragma unroll
                for (int e = 0; e < 3; ++e) pm[1 + e] = s[e];
#pragma unroll
                for (int e = 0; e < 6; ++e) pm[4 + e] = P[e];
            }
        }
        __syncthreads();  // this level's records, read by the next
    }
}

// ----------------------------------------------------------------- search
// Lower bound on the squared distance from a query voxel to a node's voxels,
// and the node's place in the order of visits (pri).  The bound is the
// greater of the distances to its two boxes.  The axis-aligned gaps are exact
// in float (halves of integers below 2^22), their scale covers the rounding
// of the squares and their sum; the oriented ones carry safety margins for
// the rounding of the projections and of the frame, so that neither exceeds
// the squared distance to any voxel of the node.  The order is the bound plus
// a share of the distance to the node's mean voxel: by the bound alone, boxes
// that hold or face the query alike come in any order (a third more leaves
// visited by queries beside a LiDAR surface).
__device__ __forceinline__ float node_bound(const Box &b, u32x4 w, const float q[3], float &pri) {
    float d[3], e[3], edge = 0.f, aabb = 0.f, mean = 0.f, l1 = 0.f;
    const uint32_t mc[3] = {w.x >> 28, (w.z >> 24) & 15u, w.z >> 28};
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        d[a] = q[a] - 0.5f * (float)(b.lo[a] + b.hi[a]);
        e[a] = (float)(b.hi[a] - b.lo[a]);
        edge = fmaxf(edge, e[a]);
        const float g = fmaxf(fabsf(d[a]) - 0.5f * e[a], 0.f);
        aabb += g * g;
        const float m = d[a] - ((float)mc[a] - 7.5f) * (1.f / 16.f) * e[a];
        mean += m * m;
        l1 += fabsf(d[a]);
    }
    const Obb o = obb_decode(w, edge + 1.f);
    const float margin = l1 * (1.f / 262144.f);
    float s = 0.f;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const float t = o.f.a[k][0] * d[0] + o.f.a[k][1] * d[1] + o.f.a[k][2] * d[2];
        const float g = fmaxf(fmaxf(o.lo[k] - t, t - o.hi[k]) - margin, 0.f);
        s += g * g;
    }
    const float lb = fmaxf(aabb * (1.f - 1.f / 1048576.f), s * (1.f - 1.f / 65536.f));
    pri = lb + 0.3f * mean;
    return lb;
}

// Team lane shifts for the shared candidate lists: a 64-bit value from the
// lane one below (DPP row shift; a team's lane 0 gets another team's value,
// which the caller discards), and one lane's value sent to every lane.
__device__ __forceinline__ uint32_t dpp_prev_u32(uint32_t x) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xF, 0xF, false);  // row_shr:1
}
__device__ __forceinline__ uint64_t dpp_prev_u64(uint64_t x) {
    return ((uint64_t)dpp_prev_u32((uint32_t)(x >> 32)) << 32) | dpp_prev_u32((uint32_t)x);
}
__device__ __forceinline__ uint64_t shfl_u64(uint64_t x, int src) {
    const uint32_t lo = (uint32_t)__shfl((int)(uint32_t)x, src, 64);
    const uint32_t hi = (uint32_t)__shfl((int)(uint32_t)(x >> 32), src, 64);
    return ((uint64_t)hi << 32) | lo;
}

// Candidate lists of one query, shared by its team of 16 lanes: ascending in
// (squared distance, key index) over the team, lane t holding positions
// t*E .. t*E + E - 1 in registers (every array below is indexed only inside
// unrolled loops).  A candidate offered by one lane is sent to the whole team
// and inserted with one shift by one position: the team then prunes with the
// k-th distance of every candidate it has found.  Insertions need every lane
// of the team active.
//
// Up to depth 15 a squared voxel distance is below 2^32 - 1, so a candidate
// packs into one word, distance above index, whose integer order is the
// candidate order; distances are 32-bit throughout.
template <int KT>
struct PackedList {
    using Dist = uint32_t;
    static constexpr int E = KT >= kTeam ? KT / kTeam : 1;  // entries per lane
    static constexpr uint64_t kNone = ~0ull;  // bound meaning "no k-th candidate yet"
    struct Cand {
        uint64_t v;
    };
    uint64_t e[E];
    __device__ __forceinline__ void clear() {
#pragma unroll
        for (int s = 0; s < E; ++s) e[s] = ~0ull;
    }
    __device__ static __forceinline__ Cand make(uint32_t d, int32_t i) {
        return Cand{((uint64_t)d << 32) | (uint32_t)i};
    }
    __device__ static __forceinline__ Cand bcast(Cand c, int src) { return Cand{shfl_u64(c.v, src)}; }
    // insert c (the same on every lane of the team); tl = lane within the team
    __device__ __forceinline__ void insert(Cand c, int tl) {
        const uint64_t v = c.v;
        const uint64_t p = dpp_prev_u64(e[E - 1]);
        const uint64_t below = tl == 0 ? 0ull : p;  // position t*E - 1 (none for lane 0)
#pragma unroll
        for (int s = E - 1; s > 0; --s) {
            const uint64_t lo = e[s - 1], cur = e[s];
            e[s] = v < lo ? lo : (v < cur ? v : cur);
        }
        e[0] = v < below ? below : (v < e[0] ? v : e[0]);
    }
    // insert what every lane offers (all ones: nothing) at once: the offers
    // are sorted downwards over the row by a bitonic network, the lesser of
    // each offer and the list's entry keeps the 16 smallest, and a last
    // merge orders them.  About 130 instructions (70 for a leaf's near
    // voxels) and no LDS, where an insert takes about 25 and the latency of
    // its broadcast; one entry per lane.
    static constexpr bool kBatch = E == 1;
    static constexpr int kBatchMin = 4;  // offers of one team from which the batch is used
    // Offers below 2^28 whose order by index is that of their lanes (a leaf's
    // voxels, from index `first` on) are sorted as distance << 4 | lane.  None
    // of them reads as "nothing": 2^28 - 1 is 7 mod 8, no sum of three squares.
    __device__ __forceinline__ void insert_leaf(uint32_t d, bool offered, uint32_t first, int tl) {
        uint32_t v = offered ? (d << 4) | (uint32_t)tl : ~0u;
        const bool b0 = tl & 1, b1 = tl & 2, b2 = tl & 4, b3 = tl & 8;
        v = exchange32<0xB1>(v, !b0);
        v = exchange32<0x1B>(v, !b1);
        v = exchange32<0xB1>(v, !b0);
        v = exchange32<0x141>(v, !b2);
        v = exchange32<0x4E>(v, !b1);
        v = exchange32<0xB1>(v, !b0);
        v = exchange32<0x140>(v, !b3);
        {
            const uint32_t y = dpp32<0x141>(dpp32<0x1B>(v));
            v = b2 ? min(v, y) : max(v, y);
        }
        v = exchange32<0x4E>(v, !b1);
        v = exchange32<0xB1>(v, !b0);
        merge_down(v == ~0u ? ~0ull : ((uint64_t)(v >> 4) << 32) | (first + (v & 15u)), tl);
    }
    __device__ __forceinline__ void insert_all(Cand c, int tl) {
        uint64_t v = c.v;
        const bool b0 = tl & 1, b1 = tl & 2, b2 = tl & 4, b3 = tl & 8;
        // exchange with the lane m away (or mirrored): the upper lane of a
        // pair keeps the lesser value here, the greater one in the merge
        v = exchange(v, xor1(v), !b0);
        v = exchange(v, xor3(v), !b1);
        v = exchange(v, xor1(v), !b0);
        v = exchange(v, xor7(v), !b2);
        v = exchange(v, xor2(v), !b1);
        v = exchange(v, xor1(v), !b0);
        v = exchange(v, xor15(v), !b3);
        v = exchange(v, xor7(xor3(v)), !b2);
        v = exchange(v, xor2(v), !b1);
        v = exchange(v, xor1(v), !b0);
        merge_down(v, tl);
    }
    // the 16 smallest of the list and 16 offers sorted downwards
    __device__ __forceinline__ void merge_down(uint64_t v, int tl) {
        const bool b0 = tl & 1, b1 = tl & 2, b2 = tl & 4, b3 = tl & 8;
        uint64_t a = e[0] < v ? e[0] : v;
        a = exchange(a, ror8(a), b3);
        a = exchange(a, xor7(xor3(a)), b2);
        a = exchange(a, xor2(a), b1);
        e[0] = exchange(a, xor1(a), b0);
    }
    template <int CTRL>
    __device__ static __forceinline__ uint32_t dpp32(uint32_t x) {
        return (uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)x, CTRL, 0xF, 0xF, false);
    }
    template <int CTRL>
    __device__ static __forceinline__ uint32_t exchange32(uint32_t x, bool greater) {
        const uint32_t y = dpp32<CTRL>(x);
        return greater ? max(x, y) : min(x, y);
    }
    template <int CTRL>
    __device__ static __forceinline__ uint64_t dpp64(uint64_t x) {
        return ((uint64_t)dpp32<CTRL>((uint32_t)(x >> 32)) << 32) | dpp32<CTRL>((uint32_t)x);
    }
    __device__ static __forceinline__ uint64_t xor1(uint64_t x) { return dpp64<0xB1>(x); }   // quad_perm 1,0,3,2
    __device__ static __forceinline__ uint64_t xor2(uint64_t x) { return dpp64<0x4E>(x); }   // quad_perm 2,3,0,1
    __device__ static __forceinline__ uint64_t xor3(uint64_t x) { return dpp64<0x1B>(x); }   // quad_perm 3,2,1,0
    __device__ static __forceinline__ uint64_t xor7(uint64_t x) { return dpp64<0x141>(x); }  // row_half_mirror
    __device__ static __forceinline__ uint64_t xor15(uint64_t x) { return dpp64<0x140>(x); } // row_mirror
    __device__ static __forceinline__ uint64_t ror8(uint64_t x) { return dpp64<0x128>(x); }  // row_ror:8
    __device__ static __forceinline__ uint64_t exchange(uint64_t x, uint64_t y, bool greater) {
        return (y < x) != greater ? y : x;
    }
    // the team's k-th distance, or kNone while it holds fewer than k; base =
    // the team's lane 0
    __device__ __forceinline__ uint64_t kth(int k, int base) const {
        const int pos = k - 1, slot = pos % E;
        uint32_t hi = (uint32_t)(e[0] >> 32);
#pragma unroll
        for (int s = 1; s < E; ++s) hi = s == slot ? (uint32_t)(e[s] >> 32) : hi;
        hi = (uint32_t)__shfl((int)hi, base + pos / E, 64);
        return hi == 0xFFFFFFFFu ? kNone : hi;
    }
    // this lane's entry s (team position tl*E + s)
    __device__ __forceinline__ void out(int s, int64_t &idx, uint64_t &d2) const {
        uint64_t v = e[0];
#pragma unroll
        for (int t = 1; t < E; ++t) v = t == s ? e[t] : v;
        idx = v == ~0ull ? -1 : (int64_t)(uint32_t)v;
        d2 = v == ~0ull ? ~0ull : (v >> 32);
    }
};

// Deeper grids: 64-bit distances beside the indexes, in two arrays (whole
// struct swaps would be lowered to memory copies).
template <int KT>
struct WideList {
    using Dist = uint64_t;
    static constexpr int E = KT >= kTeam ? KT / kTeam : 1;
    static constexpr uint64_t kNone = ~0ull;
    struct Cand {
        uint64_t d;
        int32_t i;
    };
    uint64_t d[E];
    int32_t i[E];
    static constexpr bool kBatch = false;
    __device__ static __forceinline__ bool less(uint64_t ad, int32_t ai, uint64_t bd, int32_t bi) {
        return ad < bd || (ad == bd && ai < bi);
    }
    __device__ __forceinline__ void clear() {
#pragma unroll
        for (int s = 0; s < E; ++s) {
            d[s] = ~0ull;
            i[s] = 0x7FFFFFFF;
        }
    }
    __device__ static __forceinline__ Cand make(uint64_t vd, int32_t vi) { return Cand{vd, vi}; }
    __device__ static __forceinline__ Cand bcast(Cand c, int src) {
        return Cand{shfl_u64(c.d, src), __shfl(c.i, src, 64)};
    }
    __device__ __forceinline__ void insert(Cand c, int tl) {
        const uint64_t vd = c.d;
        const int32_t vi = c.i;
        uint64_t bd = dpp_prev_u64(d[E - 1]);
        int32_t bi = (int32_t)dpp_prev_u32((uint32_t)i[E - 1]);
        if (tl == 0) {  // nothing below lane 0's first position
            bd = 0;
            bi = INT32_MIN;
        }
#pragma unroll
        for (int s = E - 1; s > 0; --s) {
            const bool sh = less(vd, vi, d[s - 1], i[s - 1]);
            const bool here = less(vd, vi, d[s], i[s]);
            const uint64_t nd = sh ? d[s - 1] : (here ? vd : d[s]);
            const int32_t ni = sh ? i[s - 1] : (here ? vi : i[s]);
            d[s] = nd;
            i[s] = ni;
        }
        const bool sh = less(vd, vi, bd, bi);
        const bool here = less(vd, vi, d[0], i[0]);
        const uint64_t nd = sh ? bd : (here ? vd : d[0]);
        const int32_t ni = sh ? bi : (here ? vi : i[0]);
        d[0] = nd;
        i[0] = ni;
    }
    __device__ __forceinline__ uint64_t kth(int k, int base) const {
        const int pos = k - 1, slot = pos % E;
        uint64_t m = d[0];
#pragma unroll
        for (int s = 1; s < E; ++s) m = s == slot ? d[s] : m;
        return shfl_u64(m, base + pos / E);
    }
    __device__ __forceinline__ void out(int s, int64_t &idx, uint64_t &d2) const {
        uint64_t vd = d[0];
        int32_t vi = i[0];
#pragma unroll
        for (int t = 1; t < E; ++t) {
            vd = t == s ? d[t] : vd;
            vi = t == s ? i[t] : vi;
        }
        idx = vd == ~0ull ? -1 : (int64_t)vi;
        d2 = vd;
    }
};

// One query at a time per team of 16 lanes: each team's first query by its
// place in the grid, the next ones from a counter: its group's (qctr, zero at
// launch) or, without them, the block's own in LDS over every grid-stride'th
// run of 16 queries.  LIST is PackedList (depth <= 15) or
// WideList; KT (16 or 32) its capacity.  The kernel is one loop whose every
// trip moves each team one step in its own query.  kCount (a measurement
// build, same results): node records and leaf voxels loaded, voxels offered
// to the list and steps, summed over lanes into work[0..3].
template <int KT, class LIST, bool kCount = false>
__global__ __launch_bounds__(kKnnBlock) void k_knn_bvh(
    const uint64_t *__restrict__ rec, const uint64_t *__restrict__ vox, BvhShape S, int64_t n_host,
    const int64_t *d_n, const float *__restrict__ q, int64_t nq,
    const uint64_t *__restrict__ order, float o0, float o1, float o2, float scale, uint32_t depth,
    int k, int64_t *__restrict__ idx_out, uint64_t *__restrict__ d2_out, uint32_t *err,
    uint32_t *qctr, const uint32_t *__restrict__ perm = nullptr,
    unsigned long long *work = nullptr) {
    uint32_t c_node = 0, c_vox = 0, c_offer = 0, c_step = 0;  // kCount only
    using Dist = typename LIST::Dist;
    using Cand = typename LIST::Cand;
    constexpr int kTeamsPerBlock = kKnnBlock / kTeam;
    // bounds of the open nodes' children, one column per thread: the levels
    // above the one being worked on
    __shared__ float s_lb[kBvhLevels][kKnnBlock], s_pri[kBvhLevels][kKnnBlock];
    __shared__ uint32_t s_off[kBvhLevels], s_next;
    const int tid = threadIdx.x, team = tid / kTeam, tl = tid % kTeam;
    const int tw = (tid & 63) / kTeam, tbase = (tid & 63) - tl;  // team within the wave, its lane 0
    if (tid < kBvhLevels) s_off[tid] = S.off[tid];
    if (tid == 0) s_next = 0;
    __syncthreads();  // the only block-wide barrier; teams run independently after it
    const int64_t n = key_count(n_host, d_n);
    const float o[3] = {o0, o1, o2};
    const int64_t stride = (int64_t)gridDim.x * kTeamsPerBlock;
    constexpr uint32_t kInf = 0x7F800000u;

    // ---- per query
    // group g's blocks are g, g + G, ...: their teams' first queries are the
    // group's first, and its counter goes on after them
    const uint32_t groups = qctr ? query_groups(gridDim.x) : 1;
    const uint32_t grp = blockIdx.x % groups;
    const int64_t ahead = (int64_t)((gridDim.x - grp + groups - 1) / groups) * kTeamsPerBlock;
    int64_t slot = qctr ? grp + (int64_t)groups * ((int64_t)(blockIdx.x / groups) * kTeamsPerBlock + team)
                        : (int64_t)blockIdx.x * kTeamsPerBlock + team;
    int64_t j = 0;
    if (qctr) qctr += grp * kQueryCtrStride;
    uint32_t nxt = 0;  // lane 0: the team's next query from the counter, taken one query ahead
    auto next_slot = [&]() __attribute__((always_inline)) -> int64_t {
        const int64_t i = (int64_t)(uint32_t)__shfl((int)nxt, tbase, 64);
        return qctr ? grp + groups * (ahead + i)
                    : (int64_t)blockIdx.x * kTeamsPerBlock + (i & (kTeamsPerBlock - 1)) + (i / kTeamsPerBlock + 1) * stride;
    };
    Vox qv{0, 0, 0};
    float qf[3] = {0.f, 0.f, 0.f};
    LIST list;
    list.clear();
    uint64_t kth = LIST::kNone;  // the team's k-th distance
    constexpr float kNoBound = 3e38f;  // no squared distance comes near it
    float kthf = kNoBound;             // at least the k-th distance, in float
    // ---- the open node: level of its children, the first of them, this
    // lane's bound on its child (infinite: none, or taken) and its place in
    // the order of visits
    int l = 0;
    uint32_t base = 0;
    float lb = 0.f, pri = 0.f;
    // The open child to visit next, its lane in the low four bits (kInf: no
    // child within the k-th distance).
    auto nearest = [&]() __attribute__((always_inline)) -> uint32_t {
        return row_min(lb <= kthf ? (__float_as_uint(pri) & ~15u) | (uint32_t)tl : kInf);
    };
    enum { kQuery, kWalk, kDone };
    int phase = kQuery;

    for (;;) {
        bool group = false;
        if (phase == kWalk) {
            // ---- the next child to open; nodes without one are climbed out
            // of.  Past the root every node within the k-th distance has been
            // searched, and the list is the answer.
            uint32_t m;
            for (;;) {
                m = nearest();
                if (m != kInf || l == S.top) break;
                ++l;
                base = (base >> kTeamBits) & ~15u;
                lb = s_lb[l][tid];
                pri = s_pri[l][tid];
            }
            if (m == kInf) {
#pragma unroll
                for (int s = 0; s < LIST::E; ++s) {
                    const int pos = tl * LIST::E + s;
                    if (pos < k) {
                        int64_t idx;
                        uint64_t d2;
                        list.out(s, idx, d2);
                        idx_out[j * k + pos] = idx;
                        d2_out[j * k + pos] = d2;
                    }
                }
                slot = next_slot();
                phase = kQuery;
            } else if (l > 0) {
                if (kCount && tl == 0) ++c_step;
                if ((m & 15u) == (uint32_t)tl) lb = __uint_as_float(kInf);
                s_lb[l][tid] = lb;
                s_pri[l][tid] = pri;
                --l;
                base = (base + (m & 15u)) << kTeamBits;
                group = true;
            }
        }
        if (phase == kQuery) {
            // ---- next query of the team: opens the root
            if (slot >= nq) {
                phase = kDone;
            } else {
                if (tl == 0) nxt = qctr ? atomicAdd(qctr, 1u) : atomicAdd(&s_next, 1u);
                j = order ? (int64_t)(order[slot] >> kOrderBits) : slot;  // query (and output row)
                const bool finite = quantize3(q[3 * j], q[3 * j + 1], q[3 * j + 2], o, scale, depth, qv);
                if (!finite && tl == 0) set_err(err, ERR_NONFINITE);
                if (!finite || n == 0) {
                    for (int s = tl; s < k; s += kTeam) {
                        idx_out[j * k + s] = -1;
                        d2_out[j * k + s] = ~0ull;
                    }
                    slot = next_slot();
                } else {
                    qf[0] = (float)qv.x;
                    qf[1] = (float)qv.y;
                    qf[2] = (float)qv.z;
                    list.clear();
                    kth = LIST::kNone;
                    kthf = kNoBound;
                    l = S.top;
                    base = 0;
                    group = true;
                    phase = kWalk;
                }
            }
        }
        if (group) {
            const int64_t i = (int64_t)base + tl;
            lb = __uint_as_float(kInf);
            if (i < bvh_nodes(n, l)) {
                const uint64_t *r = rec + 4 * ((int64_t)s_off[l] + i);
                const Box b = rec_box(*(const u64x2 *)r);
                const u32x4 w = *(const u32x4 *)(r + 2);
                if (kCount) ++c_node;
                lb = node_bound(b, w, qf, pri);
            }
        }
        // ---- leaves, nearest first: up to kLeafTrips of the open leaf group
        // per trip, the one just loaded included
#pragma unroll 1
        for (int visit = 0; visit < kLeafTrips; ++visit) {
            const uint32_t m = nearest();
            const bool go = phase == kWalk && l == 0 && m != kInf;
            if (!__ballot(go)) break;
            bool pend = false;  // this lane's voxel for the team's list, if any
            Cand cv = LIST::make((Dist)~(Dist)0, -1);
            const uint32_t first = (base + (m & 15u)) << kTeamBits;
            if (go) {
                if (kCount && tl == 0) ++c_step;
                if ((m & 15u) == (uint32_t)tl) lb = __uint_as_float(kInf);
                const int64_t i = (int64_t)first + tl;
                if (i < n) {
                    const Vox v = unpack_vox(vox[i]);
                    if (kCount) ++c_vox;
                    const Dist dx = v.x > qv.x ? v.x - qv.x : qv.x - v.x, dy = v.y > qv.y ? v.y - qv.y : qv.y - v.y,
                               dz = v.z > qv.z ? v.z - qv.z : qv.z - v.z;
                    const Dist d = dx * dx + dy * dy + dz * dz;
                    if ((uint64_t)d <= kth) {
                        // a voxel's position: in the key array, or through
                        // perm in the caller's LINEAR array (then ties go to
                        // the smaller LINEAR position, as there)
                        pend = true;
                        cv = LIST::make(d, perm ? (int32_t)perm[i] : (int32_t)i);
                        if (kCount) ++c_offer;
                    }
                }
            }
            // the team's list takes what its lanes offered; the team's k-th
            // distance follows (every lane of the wave is active here)
            const uint64_t b = __ballot(pend);
            if (!b) continue;
            uint32_t tm = (uint32_t)(b >> (kTeam * tw)) & 0xFFFFu;
            bool batched = false;
            if constexpr (LIST::kBatch) {
                if (__ballot(__popc(tm) >= LIST::kBatchMin)) {
                    if (!perm && !__ballot(pend && (uint32_t)(cv.v >> 32) >= (1u << 28)))
                        list.insert_leaf((uint32_t)(cv.v >> 32), pend, first, tl);
                    else
                        list.insert_all(cv, tl);
                    batched = true;
                }
            }
            if (!batched) {
                while (tm) {
                    const int src = __builtin_ctz(tm);
                    tm &= tm - 1;
                    list.insert(LIST::bcast(cv, tbase + src), tl);
                }
            }
            kth = list.kth(k, tbase);
            kthf = kth == LIST::kNone ? kNoBound : (float)kth * (1.f + 1.f / 1048576.f);
        }
        if (!__ballot(phase != kDone)) break;
    }
    if (kCount) {  // the team's sums, one atomic per counter per team
#pragma unroll
        for (int o2 = 1; o2 < kTeam; o2 <<= 1) {
            c_node += __shfl_xor(c_node, o2, 64);
            c_vox += __shfl_xor(c_vox, o2, 64);
            c_offer += __shfl_xor(c_offer, o2, 64);
            c_step += __shfl_xor(c_step, o2, 64);
        }
        if (tl == 0 && (c_node | c_vox | c_offer | c_step)) {
            atomicAdd(&work[0], (unsigned long long)c_node);
            atomicAdd(&work[1], (unsigned long long)c_vox);
            atomicAdd(&work[2], (unsigned long long)c_offer);
            atomicAdd(&work[3], (unsigned long long)c_step);
        }
    }
}

// LINEAR keys -> the Morton keys of the same voxels, with each key's position.
template <typename K>
__global__ __launch_bounds__(256) void k_linear_to_morton(const K *__restrict__ keys, int64_t n_host,
                                                          const int64_t *d_n, uint32_t depth,
                                                          K *__restrict__ mk, uint32_t *__restrict__ pos) {
    const int64_t n = key_count(n_host, d_n);
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const Vox v = dec3((uint64_t)keys[i], depth, true);
        mk[i] = (K)enc3(v.x, v.y, v.z, depth, false);
        pos[i] = (uint32_t)i;
    }
}

// Ordering code of every query: its index above the top kOrderBits of its
// Morton key, with the digit histogram of the three 8-bit passes.
__global__ __launch_bounds__(256) void k_knn_order(const float *__restrict__ q, int64_t nq, float o0,
                                                   float o1, float o2, float scale,
                                                   uint32_t depth, uint64_t *__restrict__ out,
                                                   uint32_t *hist) {
    constexpr int RB = 8, PASSES = kOrderBits / RB;
    __shared__ uint32_t s_h[PASSES << RB];
    for (int i = threadIdx.x; i < (PASSES << RB); i += blockDim.x) s_h[i] = 0;
    __syncthreads();
    const float o[3] = {o0, o1, o2};
    const int drop = 3 * (int)depth > kOrderBits ? 3 * (int)depth - kOrderBits : 0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nq;
         i += (int64_t)gridDim.x * blockDim.x) {
        Vox v;
        quantize3(q[3 * i], q[3 * i + 1], q[3 * i + 2], o, scale, depth, v);  // the search reports non-finite queries
        const uint64_t code = ((uint64_t)i << kOrderBits) | (enc3(v.x, v.y, v.z, depth, false) >> drop);
        out[i] = code;
        hist_add<RB>(s_h, code, PASSES);
    }
    __syncthreads();
    hist_flush<RB>(s_h, hist, PASSES);
}

// Launch knob (never changes results): CGA_KNN_ORDER = 1 / 0 forces the query
// ordering on / off; by default it is on from kOrderMin queries.
static bool knn_order(int64_t nq) {
    if (const char *e = getenv("CGA_KNN_ORDER")) return atoi(e) != 0 && nq > 0;
    return nq >= kOrderMin;
}

// Launch knob (never changes results): CGA_KNN_QUEUE = 0 takes the search's
// queries from counters of the blocks instead of the groups'.
static int knn_queue_knob() {
    if (const char *e = getenv("CGA_KNN_QUEUE")) return atoi(e) != 0 ? 1 : 0;
    return 1;
}

// Launch knob (never changes results): CGA_KNN_BLOCKS = n caps the search's
// grid at n blocks, so that every team answers many queries in turn.
static int knn_blocks_knob() {
    if (const char *e = getenv("CGA_KNN_BLOCKS")) return atoi(e);
    return 0;
}

struct KnnLayout {
    Control *ctl;
    SortWs sort;             // query ordering (when on)
    uint64_t *oa = nullptr, *ob = nullptr;
    // LINEAR keys only: their Morton re-keys (in, alternate, sorted) with
    // the key positions riding along, and the sort's workspace
    SortWs msort;
    void *mk[3] = {nullptr, nullptr, nullptr};
    uint32_t *pos[3] = {nullptr, nullptr, nullptr};
    const uint32_t *perm = nullptr;  // set per call: the sorted keys' LINEAR positions
    BvhShape shape;
    uint64_t *vox;  // the keys' voxels
    uint64_t *rec;  // node records, four words each
    float *mom;     // sums of the nodes from level 2 on, ten floats each (build only)
    uint32_t *qctr; // the search's query counters
    size_t bytes;
};

static KnnLayout knn_layout(void *ws, int64_t n, uint32_t depth, int64_t nq_order = 0,
                            bool linear = false) {
    KnnLayout L;
    Carve c(ws);
    L.shape = bvh_shape(n);
    const size_t m = (size_t)(n > 0 ? n : 1);
    L.ctl = c.take<Control>(1);
    if (linear) {  // LINEAR keys: re-keyed to Morton and sorted with their positions
        SortCfg cfg;
        cfg.radix_bits = 8;
        cfg.items = 16;
        sort_carve(c, L.msort, n, 3 * (int)depth, cfg);
        const size_t kb = wide_keys(depth) ? 8 : 4;
        for (int b = 0; b < 3; ++b) L.mk[b] = c.take<uint8_t>(m * kb);
        for (int b = 0; b < 3; ++b) L.pos[b] = c.take<uint32_t>(m);
    }
    if (nq_order > 0) {
        SortCfg cfg;
        cfg.radix_bits = 8;
        cfg.items = 16;
        sort_carve(c, L.sort, nq_order, kOrderBits, cfg);
        L.oa = c.take<uint64_t>((size_t)nq_order);
        L.ob = c.take<uint64_t>((size_t)nq_order);
    }
    L.vox = c.take<uint64_t>(m);
    L.rec = c.take<uint64_t>(4 * (size_t)L.shape.records);
    L.mom = c.take<float>(L.shape.top >= 3 ? 10 * (size_t)(L.shape.records - L.shape.off[2]) : 1);
    L.qctr = c.take<uint32_t>(kQueryGroups * kQueryCtrStride);
    L.bytes = c.size();
    return L;
}

template <typename K>
static void bvh_build(const KnnLayout &L, const K *keys, int64_t n, const int64_t *d_n,
                      uint32_t depth, hipStream_t s) {
    CGA_PROF("knn_tree", s);
    const int64_t blocks = n > 0 ? (n + kBvhTile - 1) / kBvhTile : 1;
    k_bvh_low<K><<<(unsigned)blocks, 256, 0, s>>>(keys, n, d_n, depth, L.shape, L.vox, L.rec, L.mom,
                                                  L.qctr, &L.ctl->err);
    if (L.shape.top >= 3)
        k_bvh_high<<<1, kBvhHighBlock, 0, s>>>(n, d_n, L.shape, L.rec, L.mom);
}

// Blocks of the search kernel resident on the whole GPU at once (occupancy
// per CU times the CU count; no cap if the runtime cannot say), cached per
// kernel and device.
template <int KT>
static int64_t knn_resident_blocks(bool packed, bool counting) {
    static std::mutex mu;
    static std::map<std::tuple<bool, bool, int>, int64_t> cache;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return INT64_MAX;
    std::lock_guard<std::mutex> lk(mu);
    const auto key = std::make_tuple(packed, counting, dev);
    const auto it = cache.find(key);
    if (it != cache.end()) return it->second;
    int per_cu = 0, cus = 0;
    hipError_t e;
    if (packed)
        e = counting ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_knn_bvh<KT, PackedList<KT>, true>, kKnnBlock, 0)
                     : hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_knn_bvh<KT, PackedList<KT>, false>, kKnnBlock, 0);
    else
        e = counting ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_knn_bvh<KT, WideList<KT>, true>, kKnnBlock, 0)
                     : hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_knn_bvh<KT, WideList<KT>, false>, kKnnBlock, 0);
    if (e != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        per_cu = cus = 0;
    const int64_t b = (int64_t)per_cu * cus;
    cache[key] = b > 0 ? b : INT64_MAX;
    return cache[key];
}

template <int KT, bool kCount = false>
static void knn_launch(const cga_grid *g, const KnnLayout &L, int64_t n, const int64_t *d_n,
                       const float *q, int64_t nq, int k, int64_t *idx, uint64_t *d2, hipStream_t s,
                       unsigned long long *work = nullptr) {
    CGA_PROF(kCount ? "knn_count" : "knn", s);
    // as many blocks as the GPU holds at once (each team then goes on from
    // query to query), fewer for small query sets
    constexpr int kTeamsPerBlock = kKnnBlock / kTeam;
    const int64_t want = (nq + kTeamsPerBlock - 1) / kTeamsPerBlock;
    int64_t cap = knn_resident_blocks<KT>(g->depth <= kPackedDepth, kCount);
    if (const int b = knn_blocks_knob(); b > 0 && b < cap) cap = b;
    const unsigned blocks = (unsigned)(want < cap ? want : cap);
    // Teams take their queries from their group's counter, so that a slow
    // query holds up only its own team.  The counters' 32 bits must not wrap.
    uint32_t *qctr = knn_queue_knob() != 0 && nq < (int64_t)1 << 31 ? L.qctr : nullptr;
    if (g->depth <= kPackedDepth)
        k_knn_bvh<KT, PackedList<KT>, kCount><<<blocks, kKnnBlock, 0, s>>>(
            L.rec, L.vox, L.shape, n, d_n, q, nq, L.ob, g->origin[0], g->origin[1], g->origin[2],
            g->scale, g->depth, k, idx, d2, &L.ctl->err, qctr, L.perm, work);
    else
        k_knn_bvh<KT, WideList<KT>, kCount><<<blocks, kKnnBlock, 0, s>>>(
            L.rec, L.vox, L.shape, n, d_n, q, nq, L.ob, g->origin[0], g->origin[1], g->origin[2],
            g->scale, g->depth, k, idx, d2, &L.ctl->err, qctr, L.perm, work);
}

template <bool kCount>
static void knn_dispatch(const cga_grid *g, const KnnLayout &L, int64_t n, const int64_t *d_n,
                         const float *q, int64_t nq, int k, int64_t *idx, uint64_t *d2,
                         hipStream_t s, unsigned long long *work) {
    if (k <= 16) knn_launch<16, kCount>(g, L, n, d_n, q, nq, k, idx, d2, s, work);
    else knn_launch<32, kCount>(g, L, n, d_n, q, nq, k, idx, d2, s, work);
}

// ---------------------------------------------------------- binary lookup
__global__ __launch_bounds__(256) void k_binary_lookup(const uint64_t *__restrict__ keys,
                                                       int64_t n_host, const int64_t *d_n,
                                                       const uint64_t *__restrict__ q, int64_t nq,
                                                       int64_t *__restrict__ rank,
                                                       uint8_t *__restrict__ found) {
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= nq) return;
    const int64_t n = dev_count(n_host, d_n);
    const uint64_t v = q[j];
    const int64_t r = lower_bound_dev(keys, n, v);
    rank[j] = r;
    if (found) found[j] = (uint8_t)(r < n && keys[r] == v);
}

// LINEAR keys: their Morton re-keys sorted with the key positions (an 8-bit
// key-value radix sort: mk[0] -> ... -> mk[2], pos likewise); the tree is
// built over mk[2] and the search reports positions through pos[2].
template <typename K>
static void linear_rekey(KnnLayout &L, const K *keys, int64_t n, const int64_t *d_n,
                         uint32_t depth, hipStream_t s) {
    int64_t blocks = (n + 255) / 256;
    blocks = blocks < 1 ? 1 : (blocks > 2048 ? 2048 : blocks);
    {
        CGA_PROF("knn_rekey", s);
        k_linear_to_morton<K><<<(unsigned)blocks, 256, 0, s>>>(keys, n, d_n, depth, (K *)L.mk[0],
                                                                L.pos[0]);
    }
    sort_launch_kv<K>(L.msort, (const K *)L.mk[0], (K *)L.mk[2], (K *)L.mk[1], (K *)L.mk[2],
                      L.pos[0], L.pos[2], L.pos[1], L.pos[2], n, d_n, false,
                      &L.ctl->tile_ctr[kLinearSortCtr], s);
    L.perm = L.pos[2];
}

}  // namespace cga

using namespace cga;

extern "C" {

size_t cga_knn_workspace_bytes(const cga_grid *g, int64_t n, int64_t nq) {
    if (!grid_valid(g) || n < 0 || nq < 0) return 0;
    return knn_layout(nullptr, n, g->depth, knn_order(nq) ? nq : 0,
                      g->key_mode == CGA_KEY_LINEAR).bytes;
}


static int knn_call(const cga_grid *g, const void *d_keys, int64_t n, const int64_t *d_n,
                    const float *d_q, int64_t nq, int k, int64_t *d_idx, uint64_t *d_d2, void *d_ws,
                    size_t ws_bytes, cga_stream stream, unsigned long long *work) {
    if (!grid_valid(g) || n < 0 || n > INT32_MAX || nq < 0 || k < 1 || k > 32 || !d_ws)
        return CGA_EINVAL;
    if (nq > 0 && (!d_q || !d_idx || !d_d2)) return CGA_EINVAL;
    if (n > 0 && !d_keys) return CGA_EINVAL;
    if (nq >= ((int64_t)1 << (64 - kOrderBits))) return CGA_EUNSUPPORTED;
    const bool ordered = knn_order(nq), linear = g->key_mode == CGA_KEY_LINEAR;
    KnnLayout L = knn_layout(d_ws, n, g->depth, ordered ? nq : 0, linear);
    if (ws_bytes < L.bytes) return CGA_EWORKSPACE;
    hipStream_t s = (hipStream_t)stream;
    CGA_TRY(launch_begin(L.ctl, ordered ? L.sort.hist : nullptr, ordered ? sort_zero_bytes(L.sort) : 0,
                         linear ? L.msort.hist : nullptr, linear ? sort_zero_bytes(L.msort) : 0,
                         nullptr, s));
    if (nq > 0) {
        if (ordered) {
            int64_t blocks = (nq + 256 * 8 - 1) / (256 * 8);
            blocks = blocks > 1024 ? 1024 : blocks;
            {
                CGA_PROF("knn_order", s);
                k_knn_order<<<(unsigned)blocks, 256, 0, s>>>(d_q, nq, g->origin[0], g->origin[1],
                                                              g->origin[2], g->scale, g->depth, L.oa,
                                                              L.sort.hist);
            }
            // three passes: oa -> ob -> oa -> ob
            sort_launch<uint64_t>(L.sort, L.oa, L.ob, L.oa, L.ob, nq, nullptr, true,
                                  L.ctl->tile_ctr, s);
        } else {
            L.ob = nullptr;
        }
        const void *tk = d_keys;  // the keys the tree is built over (Morton order)
        if (linear && n > 0) {
            if (wide_keys(g->depth))
                linear_rekey<uint64_t>(L, (const uint64_t *)d_keys, n, d_n, g->depth, s);
            else
                linear_rekey<uint32_t>(L, (const uint32_t *)d_keys, n, d_n, g->depth, s);
            tk = L.mk[2];
        }
        if (wide_keys(g->depth))
            bvh_build<uint64_t>(L, (const uint64_t *)tk, n, d_n, g->depth, s);
        else
            bvh_build<uint32_t>(L, (const uint32_t *)tk, n, d_n, g->depth, s);
        if (work) knn_dispatch<true>(g, L, n, d_n, d_q, nq, k, d_idx, d_d2, s, work);
        else knn_dispatch<false>(g, L, n, d_n, d_q, nq, k, d_idx, d_d2, s, nullptr);
        CGA_HIP(hipGetLastError());
    }
    return CGA_OK;
}

int cga_knn(const cga_grid *g, const void *d_keys, int64_t n, const int64_t *d_n, const float *d_q,
            int64_t nq, int k, int64_t *d_idx, uint64_t *d_d2, void *d_ws, size_t ws_bytes,
            cga_stream stream) {
    return knn_call(g, d_keys, n, d_n, d_q, nq, k, d_idx, d_d2, d_ws, ws_bytes, stream, nullptr);
}

int cga_knn_count(const cga_grid *g, const void *d_keys, int64_t n, const int64_t *d_n,
                  const float *d_q, int64_t nq, int k, int64_t *d_idx, uint64_t *d_d2,
                  uint64_t *d_work, void *d_ws, size_t ws_bytes, cga_stream stream) {
    if (!d_work) return CGA_EINVAL;
    return knn_call(g, d_keys, n, d_n, d_q, nq, k, d_idx, d_d2, d_ws, ws_bytes, stream,
                    (unsigned long long *)d_work);
}

int cga_binary_lookup(const uint64_t *d_keys, int64_t n, const int64_t *d_n, const uint64_t *d_q,
                      int64_t nq, int64_t *d_rank, uint8_t *d_found, cga_stream stream) {
    if (n < 0 || nq < 0) return CGA_EINVAL;
    if ((n > 0 && !d_keys) || (nq > 0 && (!d_q || !d_rank))) return CGA_EINVAL;
    if (nq == 0) return CGA_OK;
    hipStream_t s = (hipStream_t)stream;
    CGA_PROF("binary_lookup", s);
    k_binary_lookup<<<(unsigned)((nq + 255) / 256), 256, 0, s>>>(d_keys, n, d_n, d_q, nq, d_rank,
                                                                d_found);
    CGA_HIP(hipGetLastError());
    return CGA_OK;
}

}  // extern "C"

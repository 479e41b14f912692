// Temporal prediction of a frame from a reference frame, the inter-frame
// path of the CGA compression scheme (Section V-D), on two CGAs (sorted
// unique keys plus one packed 4 x 8-bit value per voxel):
//
// 1. clustering: k-means over each frame's voxels with eight centres started
//    at the corners of the frame's bounding box (corner i takes the maximum
//    of x when bit 2 of i is set, of y for bit 1, of z for bit 0, else the
//    minimum).  A pass assigns every voxel to its nearest centre (squared
//    distance in double precision, x + y + z terms summed in that order,
//    every operation separately rounded; ties to the lower cluster) while
//    summing coordinates per cluster in 64-bit integers; the run stops at
//    the first pass that changes no assignment or after max_iter passes, and
//    otherwise every non-empty cluster moves to its mean (one rounded
//    division), an empty one stays;
// 2. motion: cluster i of the two frames correspond (same starting corner);
//    its motion vector is the predicted centroid minus the reference one,
//    rounded half away from zero to whole voxels;
// 3. matching: every predicted voxel moved back by its cluster's vector is
//    matched to the reference voxel of least SAD over the four channels among
//    those within `window` voxels on each axis (ties: smaller L1 offset, then
//    smaller key), found by key searches;
// 4. residual: predicted minus matched channels (int16), or the voxel's own
//    channels with match -1 and SAD UINT32_MAX when it left the grid or found
//    no reference voxel.
//
// The passes run as a fixed sequence of launches that turn into no-ops once
// a frame has converged, so the whole call is asynchronous.
#include "cga_common.h"

namespace cga {

constexpr int kCl = 8;  // clusters (the bounding-box corners)
constexpr int kTemporalMaxWindow = 15;
constexpr int kTemporalMaxIter = 1000;

// Per-frame k-means state, zeroed at the start of a call.  Pass t assigns
// with the centres cent[t & 1] and sums into sum / cnt / changed [t % 3]; it
// computes its centres itself, in every block, from pass t - 1's sums (so
// no launch sits between passes), and clears slot (t + 1) % 3, which pass
// t - 1 finished reading.
// Each pass's sums are kept in kRep copies (block b adds to copy b % kRep),
// so that fewer blocks add to one word; the next pass adds the copies up.
// The sums are integers, so the copies change no result.
constexpr int kRep = 8;

struct KmState {
    double cent[2][kCl][3];
    unsigned long long sum[3][kRep][kCl][3];
    unsigned long long cnt[3][kRep][kCl];
    uint32_t changed[3];
    uint32_t lo_inv[3];  // ~min per axis (so that a zeroed block starts at "no voxel")
    uint32_t hi[3];
    uint32_t halt;       // the run has ended: later passes do nothing
    int32_t iters;       // passes run
};

template <typename K>
__device__ __forceinline__ int64_t lower_bound_k(const K *keys, int64_t n, uint64_t v) {
    int64_t lo = 0, len = n;
    while (len > 0) {
        const int64_t half = len >> 1;
        if ((uint64_t)keys[lo + half] < v) {
            lo += half + 1;
            len -= half + 1;
        } else {
            len = half;
        }
    }
    return lo;
}

// Frame f (blockIdx.y) of the two: keys, count.
template <typename K>
struct Frames {
    const K *keys[2];
    int64_t n[2];
    uint8_t *assign[2];
};

template <typename K>
__global__ __launch_bounds__(256) void k_km_bbox(Frames<K> F, uint32_t depth, bool linear, KmState *st) {
    const int f = blockIdx.y;
    uint32_t lo[3] = {~0u, ~0u, ~0u}, hi[3] = {0, 0, 0};
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < F.n[f];
         i += (int64_t)gridDim.x * blockDim.x) {
        const Vox v = dec3((uint64_t)F.keys[f][i], depth, linear);
        const uint32_t c[3] = {v.x, v.y, v.z};
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            lo[a] = c[a] < lo[a] ? c[a] : lo[a];
            hi[a] = c[a] > hi[a] ? c[a] : hi[a];
        }
    }
    // wave, then block, then one atomic per block and value
    __shared__ uint32_t s_m[6];
    if (threadIdx.x < 6) s_m[threadIdx.x] = 0;
    __syncthreads();
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        uint32_t l = ~lo[a], h = hi[a];
        for (int o = 32; o > 0; o >>= 1) {
            const uint32_t lo2 = __shfl_xor(l, o, 64), h2 = __shfl_xor(h, o, 64);
            l = lo2 > l ? lo2 : l;
            h = h2 > h ? h2 : h;
        }
        if ((threadIdx.x & 63) == 0) {
            atomicMax(&s_m[a], l);
            atomicMax(&s_m[3 + a], h);
        }
    }
    __syncthreads();
    if (threadIdx.x < 3) atomicMax(&st[f].lo_inv[threadIdx.x], s_m[threadIdx.x]);
    else if (threadIdx.x < 6) atomicMax(&st[f].hi[threadIdx.x - 3], s_m[threadIdx.x]);
}

__global__ void k_km_seed(KmState *st) {
    const int f = blockIdx.x, c = threadIdx.x;
    if (c < kCl) {
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            uint32_t lo = ~st[f].lo_inv[a], hi = st[f].hi[a];
            if (lo > hi) lo = hi = 0;  // an empty frame: every corner at the origin
            st[f].cent[0][c][a] = (double)(((c >> (2 - a)) & 1) ? hi : lo);
        }
    }
}

// Sum of a value over the wave (six adds along DPP rows), on every lane.
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp_add(uint32_t x) {
    return x + (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, ROWS, 0xF, false);
}
__device__ __forceinline__ uint32_t wave_sum(uint32_t x) {
    x = dpp_add<0x111, 0xF>(x);  // row_shr:1, 2, 4, 8
    x = dpp_add<0x112, 0xF>(x);
    x = dpp_add<0x114, 0xF>(x);
    x = dpp_add<0x118, 0xF>(x);
    x = dpp_add<0x142, 0xA>(x);  // row_bcast:15, 31
    x = dpp_add<0x143, 0xC>(x);
    return (uint32_t)__builtin_amdgcn_readlane((int)x, 63);
}

// One pass over both frames: stop if the previous pass changed nothing,
// else move to the previous pass's cluster means and assign every voxel.
//
// Bound: latency.  A pass over 2 x 0.5M voxels is a chain of loads (the state
// and last pass's sums, then the keys), the sums of its waves and the adds of
// its blocks, about 7 us beside the 2.5 us between launches.  So everything
// the start may need is loaded before the first branch, a wave loads its
// ROWS rows of keys at once, and it keeps per-lane sums of its rows' common
// cluster (neighbouring keys are neighbouring voxels) that it adds up over
// its lanes once; only voxels of other clusters take a sum of their own.
// 100 passes and the match, 2 x 0.5M voxels on LINEAR keys: 1.41 -> 1.06 ms.
// Frames of up to kKmSmall voxels take one row per wave: four waves of one
// row then end sooner than one of four (50k points at depth 8, 50 passes and
// the match: 359 against 462 us).
constexpr int64_t kKmSmall = (int64_t)1 << 18;

template <typename K, int kKmRows>
__global__ __launch_bounds__(256) void k_km_assign(Frames<K> F, uint32_t depth, bool linear, int pass,
                                                   KmState *st) {
    const int f = blockIdx.y;
    KmState &S = st[f];
    const int cur = pass % 3, prev = (pass + 2) % 3, next = (pass + 1) % 3;
    // pass 0 starts from the corners in cent[0]; pass t > 0 from the means
    // of pass t - 1's clusters, an empty cluster keeping pass t - 1's centre
    // (24 lanes divide, the block reads the results from LDS)
    const int ck = (int)threadIdx.x / 3, ca = (int)threadIdx.x % 3;
    const uint32_t halt = S.halt, moved = S.changed[prev];
    unsigned long long n = 0, sa = 0;
    double v0 = 0.0;
    if (threadIdx.x < kCl * 3) {
        v0 = S.cent[pass > 0 ? (pass + 1) & 1 : 0][ck][ca];
#pragma unroll
        for (int r = 0; r < kRep; ++r) {
            n += S.cnt[prev][r][ck];
            sa += S.sum[prev][r][ck][ca];
        }
    }
    if (halt) return;  // block-uniform: only ever set by a launch before
    if (pass > 0 && !moved) {  // the run ended with the previous pass
        if (blockIdx.x == 0 && threadIdx.x == 0) S.halt = 1;
        return;
    }
    __shared__ unsigned long long s_sum[kCl * 4];
    __shared__ uint32_t s_changed;
    for (int t = threadIdx.x; t < kCl * 4; t += blockDim.x) s_sum[t] = 0;
    if (threadIdx.x == 0) s_changed = 0;
    __shared__ double s_c[kCl * 3];
    if (threadIdx.x < kCl * 3) {
        const double v = pass > 0 && n > 0 ? __ddiv_rn((double)sa, (double)n) : v0;
        s_c[threadIdx.x] = v;
        // block 0 keeps this pass's centres (for the next pass's empty
        // clusters and for the result)
        if (blockIdx.x == 0 && pass > 0) S.cent[pass & 1][ck][ca] = v;
    }
    if (blockIdx.x == 0) {
        if (threadIdx.x == 0) S.iters = pass + 1;
        for (int t = threadIdx.x; t < kRep * kCl * 4; t += blockDim.x) {
            const int r = t / (kCl * 4), w = t % (kCl * 4);
            if ((w & 3) == 3) S.cnt[next][r][w >> 2] = 0;
            else S.sum[next][r][w >> 2][w & 3] = 0;
        }
        if (threadIdx.x == 0) S.changed[next] = 0;
    }
    __syncthreads();
    double c[kCl][3];
#pragma unroll
    for (int k = 0; k < kCl; ++k)
#pragma unroll
        for (int a = 0; a < 3; ++a) c[k][a] = s_c[k * 3 + a];
    bool changed = false;
    const int lane = threadIdx.x & 63;
    const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int64_t waves = ((int64_t)gridDim.x * blockDim.x) >> 6;
    for (int64_t base = wave * (64 * kKmRows); base < F.n[f]; base += waves * (64 * kKmRows)) {
        K key[kKmRows];
        int old[kKmRows];
#pragma unroll
        for (int r = 0; r < kKmRows; ++r) {
            const int64_t i = base + r * 64 + lane;
            key[r] = i < F.n[f] ? F.keys[f][i] : K(0);
            old[r] = pass > 0 && i < F.n[f] ? F.assign[f][i] : -1;
        }
        int common = 0;  // the cluster of the wave's first voxel
        uint32_t ax = 0, ay = 0, az = 0, an = 0;
#pragma unroll
        for (int r = 0; r < kKmRows; ++r) {
            const int64_t i = base + r * 64 + lane;
            const bool active = i < F.n[f];
            const Vox v = dec3((uint64_t)key[r], depth, linear);
            const double px = (double)v.x, py = (double)v.y, pz = (double)v.z;
            double bd = 0.0;
            int best = 0;
#pragma unroll
            for (int k = 0; k < kCl; ++k) {
                const double dx = __dsub_rn(px, c[k][0]), dy = __dsub_rn(py, c[k][1]),
                             dz = __dsub_rn(pz, c[k][2]);
                const double d = __dadd_rn(__dadd_rn(__dmul_rn(dx, dx), __dmul_rn(dy, dy)), __dmul_rn(dz, dz));
                if (k == 0 || d < bd) {
                    bd = d;
                    best = k;
                }
            }
            if (active && old[r] != best) {
                changed = true;
                F.assign[f][i] = (uint8_t)best;
            }
            if (r == 0) common = __builtin_amdgcn_readfirstlane(best);
            // at most 64 * kKmRows coordinates below 2^21: 32-bit sums are exact
            const bool with = active && best == common;
            ax += with ? v.x : 0u;
            ay += with ? v.y : 0u;
            az += with ? v.z : 0u;
            an += (uint32_t)__popcll(__ballot(with));
            uint64_t rem = __ballot(active && best != common);
            while (rem) {
                const int leader = __ffsll((unsigned long long)rem) - 1;
                const int k = __builtin_amdgcn_readlane(best, leader);
                const bool mine = active && best == k;
                const uint64_t m = __ballot(mine);
                const uint32_t sx = wave_sum(mine ? v.x : 0u), sy = wave_sum(mine ? v.y : 0u),
                               sz = wave_sum(mine ? v.z : 0u);
                if (lane < 4)
                    atomicAdd(&s_sum[k * 4 + lane], (unsigned long long)(lane == 0 ? sx : lane == 1 ? sy : lane == 2 ? sz : (uint32_t)__popcll(m)));
                rem &= ~m;
            }
        }
        ax = wave_sum(ax);
        ay = wave_sum(ay);
        az = wave_sum(az);
        if (lane < 4)
            atomicAdd(&s_sum[common * 4 + lane], (unsigned long long)(lane == 0 ? ax : lane == 1 ? ay : lane == 2 ? az : an));
    }
    if (__ballot(changed) && (threadIdx.x & 63) == 0) s_changed = 1;
    __syncthreads();
    for (int t = threadIdx.x; t < kCl * 4; t += blockDim.x) {
        const unsigned long long v = s_sum[t];
        const int r = blockIdx.x % kRep;
        if (v) atomicAdd((t & 3) == 3 ? &S.cnt[cur][r][t >> 2] : &S.sum[cur][r][t >> 2][t & 3], v);
    }
    if (threadIdx.x == 0 && s_changed) atomicOr(&S.changed[cur], 1u);
}

// Centroids, motion vectors and pass counts to the caller's arrays.
__global__ void k_motion(const KmState *st, double *centroids, int32_t *mv, int32_t *iters,
                         int32_t *mv_ws) {
    const int t = threadIdx.x;  // cluster * 3 + axis
    if (t < kCl * 3) {
        const int k = t / 3, a = t % 3;
        // the centres of each frame's last pass
        const double cr = st[0].cent[(st[0].iters + 1) & 1][k][a], cp = st[1].cent[(st[1].iters + 1) & 1][k][a];
        const int32_t m = (int32_t)round(__dsub_rn(cp, cr));
        mv_ws[t] = m;
        if (mv) mv[t] = m;
        if (centroids) {
            centroids[t] = cr;
            centroids[kCl * 3 + t] = cp;
        }
    }
    if (t < 2 && iters) iters[t] = st[t].iters;
}

__device__ __forceinline__ uint32_t chan_sad(uint32_t a, uint32_t b) {
    uint32_t s = 0;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const int32_t d = (int32_t)((a >> (8 * c)) & 0xFFu) - (int32_t)((b >> (8 * c)) & 0xFFu);
        s += (uint32_t)(d < 0 ? -d : d);
    }
    return s;
}

// First index in [lo, n) whose key is >= v, for one not far past lo: steps
// that double, then a search of the last one.
template <typename K>
__device__ __forceinline__ int64_t lower_bound_from(const K *keys, int64_t lo, int64_t n, uint64_t v) {
    int64_t step = 1;
    while (lo + step <= n && (uint64_t)keys[lo + step - 1] < v) {
        lo += step;
        step <<= 1;
    }
    int64_t len = lo + step <= n ? step - 1 : n - lo;
    while (len > 0) {
        const int64_t half = len >> 1;
        if ((uint64_t)keys[lo + half] < v) {
            lo += half + 1;
            len -= half + 1;
        } else {
            len = half;
        }
    }
    return lo;
}

// Matching, a thread per predicted voxel.  Bound: dependent key probes, so
// few searches start from the whole array: on LINEAR keys one per x of the
// window, the columns of further y then from where the one before ended; on
// MORTON keys one per aligned cell of at least the window's width (eight at
// most), whose keys are then taken in turn.  With a search of the whole
// array per (x, y) column, 0.5M voxels took 179 us on LINEAR keys (window 2),
// 127 now; with one per voxel of the window, whole calls on MORTON keys 3.4
// ms (depth 11, window 3, 20 passes), 0.96 now.
template <typename K>
__global__ __launch_bounds__(256) void k_match(const K *__restrict__ ref_keys,
                                               const uint32_t *__restrict__ ref_vals, int64_t n_ref,
                                               const K *__restrict__ pred_keys,
                                               const uint32_t *__restrict__ pred_vals, int64_t n_pred,
                                               const uint8_t *__restrict__ pred_assign,
                                               const int32_t *__restrict__ mv_ws, uint32_t depth,
                                               bool linear, int window, int64_t *__restrict__ match,
                                               uint32_t *__restrict__ sad, int16_t *__restrict__ residual) {
    __shared__ int32_t s_mv[kCl * 3];
    if (threadIdx.x < kCl * 3) s_mv[threadIdx.x] = mv_ws[threadIdx.x];
    __syncthreads();
    const int64_t top = (int64_t)1 << depth;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n_pred;
         i += (int64_t)gridDim.x * blockDim.x) {
        const Vox p = dec3((uint64_t)pred_keys[i], depth, linear);
        const int cl = pred_assign[i];
        const int64_t r[3] = {(int64_t)p.x - s_mv[cl * 3], (int64_t)p.y - s_mv[cl * 3 + 1],
                              (int64_t)p.z - s_mv[cl * 3 + 2]};
        const uint32_t pv = pred_vals[i];
        int64_t best = -1;
        uint32_t bs = 0xFFFFFFFFu, bl = 0;
        uint64_t bk = 0;
        auto consider = [&](int64_t j, uint32_t l1) __attribute__((always_inline)) {
            const uint32_t s = chan_sad(pv, ref_vals[j]);
            const uint64_t key = (uint64_t)ref_keys[j];
            if (best < 0 || s < bs || (s == bs && (l1 < bl || (l1 == bl && key < bk)))) {
                best = j;
                bs = s;
                bl = l1;
                bk = key;
            }
        };
        const bool inside = r[0] >= 0 && r[0] < top && r[1] >= 0 && r[1] < top && r[2] >= 0 && r[2] < top;
        if (inside && n_ref > 0) {
            const int64_t zlo = r[2] - window > 0 ? r[2] - window : 0;
            const int64_t zhi = r[2] + window < top - 1 ? r[2] + window : top - 1;
            const int64_t xlo = r[0] - window > 0 ? r[0] - window : 0;
            const int64_t xhi = r[0] + window < top - 1 ? r[0] + window : top - 1;
            const int64_t ylo = r[1] - window > 0 ? r[1] - window : 0;
            const int64_t yhi = r[1] + window < top - 1 ? r[1] + window : top - 1;
            auto off = [](int64_t a, int64_t b) { return (uint32_t)(a > b ? a - b : b - a); };
            if (linear) {
                for (int64_t x = xlo; x <= xhi; ++x) {
                    int64_t j = 0;
                    for (int64_t y = ylo; y <= yhi; ++y) {
                        const uint32_t lxy = off(x, r[0]) + off(y, r[1]);
                        // the column's z range is one run of LINEAR keys
                        const uint64_t k0 = enc3((uint32_t)x, (uint32_t)y, (uint32_t)zlo, depth, true);
                        const uint64_t k1 = enc3((uint32_t)x, (uint32_t)y, (uint32_t)zhi, depth, true);
                        j = y == ylo ? lower_bound_k(ref_keys, n_ref, k0) : lower_bound_from(ref_keys, j, n_ref, k0);
                        for (; j < n_ref && (uint64_t)ref_keys[j] <= k1; ++j)
                            consider(j, lxy + off((int64_t)((uint64_t)ref_keys[j] & (uint64_t)(top - 1)), r[2]));
                    }
                }
            } else {
                int lev = 0;
                while (((int64_t)1 << lev) < 2 * window + 1 && lev < (int)depth) ++lev;
                for (int64_t cx = xlo >> lev; cx <= xhi >> lev; ++cx)
                    for (int64_t cy = ylo >> lev; cy <= yhi >> lev; ++cy)
                        for (int64_t cz = zlo >> lev; cz <= zhi >> lev; ++cz) {
                            const uint64_t cell = enc3((uint32_t)cx, (uint32_t)cy, (uint32_t)cz, depth, false);
                            const uint64_t k0 = cell << (3 * lev), k1 = k0 + ((1ull << (3 * lev)) - 1);
                            for (int64_t j = lower_bound_k(ref_keys, n_ref, k0); j < n_ref; ++j) {
                                const uint64_t k = (uint64_t)ref_keys[j];
                                if (k > k1) break;
                                const Vox v = dec3(k, depth, false);
                                if (v.x >= xlo && v.x <= xhi && v.y >= ylo && v.y <= yhi && v.z >= zlo && v.z <= zhi)
                                    consider(j, off(v.x, r[0]) + off(v.y, r[1]) + off(v.z, r[2]));
                            }
                        }
            }
        }
        match[i] = best;
        sad[i] = best < 0 ? 0xFFFFFFFFu : bs;
        const uint32_t rv = best < 0 ? 0u : ref_vals[best];
#pragma unroll
        for (int c = 0; c < 4; ++c)
            residual[4 * i + c] = (int16_t)((int32_t)((pv >> (8 * c)) & 0xFFu) - (int32_t)((rv >> (8 * c)) & 0xFFu));
    }
}

static unsigned temporal_grid(int64_t n) {
    int64_t b = (n + 255) / 256;
    return (unsigned)(b < 1 ? 1 : (b > 4096 ? 4096 : b));
}

struct TemporalLayout {
    Control *ctl;
    KmState *st;
    int32_t *mv;
    size_t bytes;
};

static TemporalLayout temporal_layout(void *ws) {
    TemporalLayout L;
    Carve c(ws);
    L.ctl = c.take<Control>(1);
    L.st = c.take<KmState>(2);
    L.mv = c.take<int32_t>(kCl * 3);
    L.bytes = c.size();
    return L;
}

template <typename K>
static void temporal_launch(const cga_grid *g, const K *rk, const uint32_t *rv, int64_t nr,
                            const K *pk, const uint32_t *pv, int64_t np, int window, int max_iter,
                            uint8_t *ra, uint8_t *pa, double *cent, int32_t *mv, int32_t *iters,
                            int64_t *match, uint32_t *sad, int16_t *res, const TemporalLayout &L,
                            hipStream_t s) {
    const bool linear = g->key_mode == CGA_KEY_LINEAR;
    Frames<K> F{{rk, pk}, {nr, np}, {ra, pa}};
    // a few blocks per CU, striding over the frame: few global atomics per pass
    unsigned gb = temporal_grid(nr > np ? nr : np);
    gb = gb < 512 ? gb : 512;
    const dim3 grid(gb, 2);
    {
        CGA_PROF("temporal_kmeans", s);
        k_km_bbox<K><<<grid, 256, 0, s>>>(F, g->depth, linear, L.st);
        k_km_seed<<<2, 64, 0, s>>>(L.st);
        const bool small = (nr > np ? nr : np) <= kKmSmall;
        for (int pass = 0; pass < max_iter; ++pass) {
            if (small) k_km_assign<K, 1><<<grid, 256, 0, s>>>(F, g->depth, linear, pass, L.st);
            else k_km_assign<K, 4><<<grid, 256, 0, s>>>(F, g->depth, linear, pass, L.st);
        }
        k_motion<<<1, 64, 0, s>>>(L.st, cent, mv, iters, L.mv);
    }
    if (np > 0) {
        CGA_PROF("temporal_match", s);
        k_match<K><<<temporal_grid(np), 256, 0, s>>>(rk, rv, nr, pk, pv, np, pa, L.mv, g->depth, linear,
                                                     window, match, sad, res);
    }
}

}  // namespace cga

using namespace cga;

extern "C" {

size_t cga_temporal_workspace_bytes(void) { return temporal_layout(nullptr).bytes; }

int cga_temporal_predict(const cga_grid *g, const void *d_ref_keys, const uint32_t *d_ref_values,
                         int64_t n_ref, const void *d_pred_keys, const uint32_t *d_pred_values,
                         int64_t n_pred, int window, int max_iter, uint8_t *d_ref_assign,
                         uint8_t *d_pred_assign, double *d_centroids, int32_t *d_mv,
                         int32_t *d_iters, int64_t *d_match, uint32_t *d_sad, int16_t *d_residual,
                         void *d_ws, size_t ws_bytes, cga_stream stream) {
    if (!grid_valid(g) || n_ref < 0 || n_pred < 0 || !d_ws) return CGA_EINVAL;
    if (window < 0 || window > kTemporalMaxWindow || max_iter < 1 || max_iter > kTemporalMaxIter)
        return CGA_EINVAL;
    if (n_ref > 0 && (!d_ref_keys || !d_ref_values || !d_ref_assign)) return CGA_EINVAL;
    if (n_pred > 0 && (!d_pred_keys || !d_pred_values || !d_pred_assign || !d_match || !d_sad ||
                       !d_residual))
        return CGA_EINVAL;
    const TemporalLayout L = temporal_layout(d_ws);
    if (ws_bytes < L.bytes) return CGA_EWORKSPACE;
    hipStream_t s = (hipStream_t)stream;
    CGA_TRY(launch_begin(L.ctl, L.st, 2 * sizeof(KmState), nullptr, 0, nullptr, s));
    if (wide_keys(g->depth))
        temporal_launch<uint64_t>(g, (const uint64_t *)d_ref_keys, d_ref_values, n_ref,
                                  (const uint64_t *)d_pred_keys, d_pred_values, n_pred, window,
                                  max_iter, d_ref_assign, d_pred_assign, d_centroids, d_mv, d_iters,
                                  d_match, d_sad, d_residual, L, s);
    else
        temporal_launch<uint32_t>(g, (const uint32_t *)d_ref_keys, d_ref_values, n_ref,
                                  (const uint32_t *)d_pred_keys, d_pred_values, n_pred, window,
                                  max_iter, d_ref_assign, d_pred_assign, d_centroids, d_mv, d_iters,
                                  d_match, d_sad, d_residual, L, s);
    CGA_HIP(hipGetLastError());
    return CGA_OK;
}

}  // extern "C"

// Octree occupancy codes (Section II-E) of a sorted unique MORTON key array.
//
// In Morton order every octree cell is a contiguous run of keys: the
// level-L node j (L = 1 .. depth) is the j-th distinct prefix key >> 3L.  The
// nodes of every level are numbered from the keys alone (counts per tile, a
// scan per level, then each node's first child and octant), and one pass over
// all nodes of all levels writes their codes.
//
// Bound: launches and load latency (a LiDAR union of 0.6M voxels), then the
// key array read twice and 5 bytes per node written and read back.
#include "cga_common.h"

namespace cga {

constexpr int kMaxDepth = 21;
constexpr int kTreeRows = 4;                       // rows of 256 keys per build tile
constexpr int kTreeTile = kTreeRows * 256;         // keys per build tile

// Highest level at which key i starts a new cell: key 0 starts every cell up
// to the root (level depth); key i > 0 starts the cells of every level below
// the highest bit in which it differs from key i - 1.  -1 past the end (and
// for a repeated key, which valid input never has).
template <typename K>
__device__ __forceinline__ int head_level(const K *keys, int64_t i, int64_t n, uint32_t depth) {
    if (i >= n) return -1;
    if (i == 0) return (int)depth;
    const uint64_t x = (uint64_t)keys[i] ^ (uint64_t)keys[i - 1];
    return x ? (63 - __clzll(x)) / 3 : -1;
}

// Number of keys: the device count when given, never above the host bound.
__device__ __forceinline__ int64_t key_count(int64_t n_host, const int64_t *d_n) {
    const int64_t n = dev_count(n_host, d_n);
    return n < n_host ? n : n_host;
}

// The level table: lvl[L] = nodes at level L (lvl[0] = keys), lvl[kLvlBase +
// L] = first node of level L in the concatenated arrays (L = 1 .. depth + 1,
// the last being the total), and lvl[kLvlTotal] = the total, or -1 when it
// exceeds the arrays (a key array that is not a CGA of the grid can have
// more cells than the bound).
constexpr int kLvlBase = kMaxDepth + 2;
constexpr int kLvlTotal = 2 * kMaxDepth + 4;
constexpr int kLvlWords = 2 * kMaxDepth + 6;

__device__ __forceinline__ int64_t tree_total(const int64_t *lvl) { return lvl[kLvlTotal]; }

// The node bases and the total, from the level sizes (one thread).
__global__ void k_tree_bases(int64_t *__restrict__ lvl, uint32_t depth, int64_t nodes_max) {
    if (threadIdx.x != 0) return;
    int64_t b = 0;
    for (uint32_t L = 1; L <= depth; ++L) {
        lvl[kLvlBase + L] = b;
        b += lvl[L];
    }
    lvl[kLvlBase + depth + 1] = b;
    lvl[kLvlTotal] = b <= nodes_max ? b : -1;
}

__device__ __forceinline__ uint32_t mbcnt64(uint64_t m) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Pass 1: per tile of kTreeTile keys, the number of nodes each level starts
// in it (cnt[(L - 1) * tiles + tile]).
template <typename K>
__global__ __launch_bounds__(256) void k_tree_count(const K *__restrict__ keys, int64_t n_host,
                                                    const int64_t *d_n, uint32_t depth,
                                                    int64_t tiles, uint32_t *__restrict__ cnt,
                                                    uint32_t *err) {
    __shared__ uint32_t s_c[kMaxDepth + 1];
    const int64_t n = key_count(n_host, d_n);
    if (threadIdx.x <= kMaxDepth) s_c[threadIdx.x] = 0;
    __syncthreads();
    const int lane = threadIdx.x & 63;
    for (int r = 0; r < kTreeRows; ++r) {
        const int64_t i = (int64_t)blockIdx.x * kTreeTile + r * 256 + threadIdx.x;
        const int h = head_level(keys, i, n, depth);
        // not a CGA of this grid: unsorted, repeated, or wider than 3 * depth bits
        if (i < n && ((i > 0 && keys[i] <= keys[i - 1]) || ((uint64_t)keys[i] >> (3 * depth)) != 0))
            set_err(err, ERR_MISMATCH);
        for (uint32_t L = 1; L <= depth; ++L) {
            const uint64_t b = __ballot(h >= (int)L);
            if (!b) break;
            if (lane == 0) atomicAdd(&s_c[L], (uint32_t)__popcll(b));
        }
    }
    __syncthreads();
    if (threadIdx.x >= 1 && threadIdx.x <= depth)
        cnt[(int64_t)(threadIdx.x - 1) * tiles + blockIdx.x] = s_c[threadIdx.x];
}

// Pass 2: one block per level; exclusive scan of the tile counts in place,
// level size into lvl[L] (lvl[0] = number of keys).
__global__ __launch_bounds__(1024) void k_tree_scan(uint32_t *__restrict__ cnt, int64_t tiles,
                                                    int64_t n_host, const int64_t *d_n,
                                                    int64_t *__restrict__ lvl) {
    __shared__ uint32_t s_w[16];
    const int L = blockIdx.x + 1;
    uint32_t *c = cnt + (int64_t)(L - 1) * tiles;
    const int64_t per = (tiles + 1023) / 1024;
    const int64_t b0 = (int64_t)threadIdx.x * per;
    const int64_t b1 = b0 + per < tiles ? b0 + per : tiles;
    uint32_t sum = 0;
    for (int64_t t = b0; t < b1; ++t) sum += c[t];
    // block exclusive scan of the per-thread sums
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t incl = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t v = __shfl_up(incl, o, 64);
        if (lane >= o) incl += v;
    }
    if (lane == 63) s_w[wave] = incl;
    __syncthreads();
    uint32_t before = 0, total = 0;
    for (int w = 0; w < 16; ++w) {
        before += w < wave ? s_w[w] : 0;
        total += s_w[w];
    }
    uint32_t run = before + incl - sum;
    for (int64_t t = b0; t < b1; ++t) {
        const uint32_t v = c[t];
        c[t] = run;
        run += v;
    }
    if (threadIdx.x == 0) {
        lvl[L] = total;
        if (L == 1) lvl[0] = key_count(n_host, d_n);
    }
}

// Pass 3: node index of every cell each key starts, at every level; writes
// the first-child index and the octant of each node.  The node arrays of all
// levels are concatenated, level L starting at lvl[1] + ... + lvl[L - 1].
template <typename K>
__global__ __launch_bounds__(256) void k_tree_build(const K *__restrict__ keys, int64_t n_host,
                                                    const int64_t *d_n, uint32_t depth,
                                                    int64_t tiles, const uint32_t *__restrict__ cnt,
                                                    const int64_t *__restrict__ lvl,
                                                    uint32_t *__restrict__ first,
                                                    uint8_t *__restrict__ oct) {
    __shared__ uint32_t s_w[kTreeRows][4][kMaxDepth + 1];
    __shared__ int64_t s_base[kMaxDepth + 2];
    __shared__ uint32_t s_off[kMaxDepth + 1];
    __shared__ int s_max[4];
    if (tree_total(lvl) < 0) return;  // block-uniform
    const int64_t n = key_count(n_host, d_n);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (threadIdx.x >= 1 && threadIdx.x <= depth + 1) s_base[threadIdx.x] = lvl[kLvlBase + threadIdx.x];
    if (threadIdx.x >= 1 && threadIdx.x <= depth)
        s_off[threadIdx.x] = cnt[(int64_t)(threadIdx.x - 1) * tiles + blockIdx.x];
    int h[kTreeRows];
    int hmax = -1;
#pragma unroll
    for (int r = 0; r < kTreeRows; ++r) {
        h[r] = head_level(keys, (int64_t)blockIdx.x * kTreeTile + r * 256 + threadIdx.x, n, depth);
        hmax = h[r] > hmax ? h[r] : hmax;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const int v = __shfl_xor(hmax, o, 64);
        hmax = v > hmax ? v : hmax;
    }
    if (lane == 0) s_max[wave] = hmax;
    __syncthreads();
    int bmax = s_max[0];
    for (int w = 1; w < 4; ++w) bmax = s_max[w] > bmax ? s_max[w] : bmax;
    // wave counts of the nodes each level starts, per row
#pragma unroll
    for (int r = 0; r < kTreeRows; ++r)
        for (int L = 1; L <= bmax; ++L) {
            const uint64_t b = __ballot(h[r] >= L);
            if (lane == 0) s_w[r][wave][L] = (uint32_t)__popcll(b);
        }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kTreeRows; ++r) {
        const int64_t i = (int64_t)blockIdx.x * kTreeTile + r * 256 + threadIdx.x;
        int64_t child = i;  // this key's node one level down (the key itself at level 0)
        for (int L = 1; L <= bmax; ++L) {
            const uint64_t b = __ballot(h[r] >= L);
            if (!b) break;
            uint32_t before = s_off[L];
            for (int rr = 0; rr < r; ++rr)
                for (int w = 0; w < 4; ++w) before += s_w[rr][w][L];
            for (int w = 0; w < wave; ++w) before += s_w[r][w][L];
            if (h[r] >= L) {
                const int64_t j = (int64_t)before + mbcnt64(b);
                const int64_t t = s_base[L] + j;
                first[t] = (uint32_t)child;
                oct[t] = (uint8_t)(((uint64_t)keys[i] >> (3 * L)) & 7);
                child = j;
            }
        }
    }
}

// Pass 4: one thread per node of every level, its code from its children's
// octants.  Codes go to occ (nullable) root first, level by level, cells in
// key order (level L starts after the codes of levels depth .. L + 1); counts
// (nullable) gets the cells per level.  The levels do not depend on each
// other, so one launch covers them all (the k-NN search's boxes, which were
// built level by level, once came with it: 300 us for the 0.6M voxels of a
// LiDAR sweep pair where the codes alone take 40).
template <typename K>
__global__ __launch_bounds__(256) void k_tree_codes(const K *__restrict__ keys, uint32_t depth,
                                                    const int64_t *__restrict__ lvl,
                                                    const uint32_t *__restrict__ first,
                                                    const uint8_t *__restrict__ oct,
                                                    uint8_t *__restrict__ occ, int64_t occ_cap,
                                                    int64_t *__restrict__ counts, uint32_t *err) {
    __shared__ int64_t s_n[kMaxDepth + 2], s_base[kMaxDepth + 2];
    if (threadIdx.x <= depth + 1) {
        s_n[threadIdx.x] = lvl[threadIdx.x];
        s_base[threadIdx.x] = lvl[kLvlBase + threadIdx.x];
    }
    __syncthreads();
    const int64_t total = tree_total(lvl) > 0 ? tree_total(lvl) : 0;  // 0: nothing to do
    if (blockIdx.x == 0) {
        if (counts && threadIdx.x <= depth) counts[threadIdx.x] = s_n[threadIdx.x];
        if (threadIdx.x == 0 && occ && total > occ_cap) set_err(err, ERR_CAPACITY);
    }
    if (!occ) return;
    for (int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x; t < total; t += (int64_t)gridDim.x * 256) {
        uint32_t L = 1;
        while (L < depth && t >= s_base[L + 1]) ++L;
        const int64_t j = t - s_base[L];
        const int64_t f0 = first[t];
        int64_t f1 = j + 1 < s_n[L] ? (int64_t)first[t + 1] : s_n[L - 1];
        if (f1 > f0 + 8) f1 = f0 + 8;  // eight children at most (unique keys)
        uint32_t mask = 0;
        for (int64_t c = f0; c < f1; ++c)
            mask |= 1u << (L == 1 ? (uint32_t)((uint64_t)keys[c] & 7) : oct[s_base[L - 1] + c]);
        const int64_t o = total - s_base[L + 1] + j;  // codes of levels above L come first
        if (o < occ_cap) occ[o] = (uint8_t)mask;
    }
}

// Upper bound on the number of octree nodes of n unique keys: level L has at
// most min(n, 8^(depth - L)) nodes.
static int64_t tree_nodes_max(int64_t n, uint32_t depth) {
    int64_t t = 0;
    for (uint32_t L = 1; L <= depth; ++L) {
        const uint32_t e = 3 * (depth - L);
        const int64_t cap = e >= 62 ? INT64_MAX : (int64_t)1 << e;
        t += n < cap ? n : cap;
    }
    return t > 0 ? t : 1;
}

struct OccLayout {
    Control *ctl;
    uint32_t *cnt;
    int64_t *lvl;
    uint32_t *first;
    uint8_t *oct;
    int64_t tiles, nodes;
    size_t bytes;
};

static OccLayout occ_layout(void *ws, int64_t n, uint32_t depth) {
    OccLayout L;
    Carve c(ws);
    L.tiles = n > 0 ? (n + kTreeTile - 1) / kTreeTile : 1;
    L.nodes = tree_nodes_max(n, depth);
    L.ctl = c.take<Control>(1);
    L.lvl = c.take<int64_t>(kLvlWords);
    L.cnt = c.take<uint32_t>((size_t)L.tiles * depth);
    L.first = c.take<uint32_t>((size_t)L.nodes);
    L.oct = c.take<uint8_t>((size_t)L.nodes);
    L.bytes = c.size();
    return L;
}

template <typename K>
static void occupancy_enqueue(const OccLayout &L, const K *keys, int64_t n, const int64_t *d_n,
                              uint32_t depth, uint8_t *occ, int64_t occ_cap, int64_t *counts,
                              hipStream_t s) {
    CGA_PROF("occupancy", s);
    k_tree_count<K><<<(unsigned)L.tiles, 256, 0, s>>>(keys, n, d_n, depth, L.tiles, L.cnt,
                                                      &L.ctl->err);
    k_tree_scan<<<depth, 1024, 0, s>>>(L.cnt, L.tiles, n, d_n, L.lvl);
    k_tree_bases<<<1, 64, 0, s>>>(L.lvl, depth, L.nodes);
    k_tree_build<K><<<(unsigned)L.tiles, 256, 0, s>>>(keys, n, d_n, depth, L.tiles, L.cnt, L.lvl,
                                                      L.first, L.oct);
    // about n / 2 nodes on a surface; the threads stride over the real count
    int64_t blocks = (n + 511) / 512;
    blocks = blocks < 1 ? 1 : (blocks < 8192 ? blocks : 8192);
    k_tree_codes<K><<<(unsigned)blocks, 256, 0, s>>>(keys, depth, L.lvl, L.first, L.oct, occ,
                                                     occ_cap, counts, &L.ctl->err);
}

}  // namespace cga

using namespace cga;

extern "C" {

size_t cga_occupancy_workspace_bytes(const cga_grid *g, int64_t n) {
    if (!grid_valid(g) || n < 0) return 0;
    return occ_layout(nullptr, n, g->depth).bytes;
}

int cga_occupancy(const cga_grid *g, const void *d_keys, int64_t n, const int64_t *d_n,
                  uint8_t *d_occ, int64_t occ_cap, int64_t *d_counts, void *d_ws, size_t ws_bytes,
                  cga_stream stream) {
    if (!grid_valid(g) || n < 0 || n > INT32_MAX || occ_cap < 0 || !d_ws) return CGA_EINVAL;
    if ((n > 0 && !d_keys) || (occ_cap > 0 && !d_occ)) return CGA_EINVAL;
    if (g->key_mode != CGA_KEY_MORTON) return CGA_EUNSUPPORTED;
    OccLayout L = occ_layout(d_ws, n, g->depth);
    if (ws_bytes < L.bytes) return CGA_EWORKSPACE;
    hipStream_t s = (hipStream_t)stream;
    CGA_TRY(launch_begin(L.ctl, nullptr, 0, nullptr, 0, nullptr, s));
    if (wide_keys(g->depth))
        occupancy_enqueue<uint64_t>(L, (const uint64_t *)d_keys, n, d_n, g->depth, d_occ, occ_cap,
                                    d_counts, s);
    else
        occupancy_enqueue<uint32_t>(L, (const uint32_t *)d_keys, n, d_n, g->depth, d_occ, occ_cap,
                                    d_counts, s);
    CGA_HIP(hipGetLastError());
    return CGA_OK;
}

}  // extern "C"

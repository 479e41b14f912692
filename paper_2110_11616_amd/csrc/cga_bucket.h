// Sorted run-length compaction of encoded points by sampled buckets: instead
// of one pass over memory per digit, the keys are split once into buckets of
// a few thousand by splitters drawn from a sample of the input, and each
// bucket is sorted and compacted by one block in LDS.
//   1. sample: S = kBkOver * buckets points at hashed positions (one per
//      equal stretch of the input), encoded and sorted; every kBkOver-th is a
//      splitter.
//   2. encode: points -> keys, bin = 2 * (splitters below the key) + (key is
//      the next splitter), and the bins' counts.
//   3. scan: first slot of every bucket.
//   4. scatter: the keys to their buckets, in any order; keys that equal a
//      splitter are one run and are only counted.
//   5. sort: a block per bucket subtracts the bucket's lower bound, sorts the
//      differences in LDS and finds the runs.  A bucket over kBkCap keys, or
//      half of that where the difference takes more than 32 bits, is sorted
//      through global memory by its block, slowly.  With eight samples a bucket
//      (at hashed positions, repeated keys made splitters) one of 4096 keys on
//      average is over kBkCap with probability 3e-7, over the half with 3 %:
//      2M to 12M points of wide spans (a filled volume, or a surface of 14 bits
//      an axis and more in random order) have some tens of those and still gain
//      (filled volume of 63-bit keys, us of a sort against buckets: 2M 262 / 217,
//      4M 406 / 305, 8M 583 / 507).
//   6. emit: the buckets' runs to their places in the output.
// Measured, 10M points of a surface in random order, 42-bit keys (us): sample 31,
// encode 60, scan 7, scatter 96 (1.9 TB/s by its own bytes, but it writes 3.6 times
// those in lines that leave part-filled; 128 with a range per block instead of the
// shared cursors), sort 158 (LDS and barriers: its waves wait 59 % of their time;
// 392 with a look-back for the place of its output), emit 55 (4.4 TB/s); the call
// 447 against 514 by six radix passes and a compaction.  1M LiDAR points, 36 bits:
// 84 against 126.
#pragma once

#include "cga_common.h"

namespace cga {

constexpr int kBkBlock = 1024;
constexpr int kBkWaves = kBkBlock / 64;
constexpr int kBkItems = 15;                 // two blocks' LDS in a CU
constexpr int kBkCap = kBkBlock * kBkItems;  // keys that one block sorts in LDS
constexpr int kBkOver = 8;                   // samples per bucket
constexpr int kBkMax = 4096;                 // buckets: two tables in an encode block's LDS
constexpr int kBkOneSort = 4096;             // samples that are ranked at once
constexpr int kBkGroups = 64;                // parts of a larger sample
constexpr int kBkGroupCap = 2048;            // and the room of each
constexpr int kBkCoarse = 16;                // samples per part for their own splitters
constexpr int kBkGrid = 512;                 // encode and scatter blocks: two per CU
// Scatter blocks share a cursor per bucket with the blocks of their group, which
// are dealt to one XCD (block b to XCD b mod 8): all of an XCD's open ends fit its
// L2, so its lines fill there before they leave.
constexpr int kBkXcds = 8;

// Buckets for n points: 1024 points each while that is at most two per CU,
// then 4096.
inline int bk_buckets(int64_t n) {
    int64_t b = (n + 1023) / 1024;
    b = b < 512 ? b : 512;
    const int64_t c = (n + 4095) / 4096;
    b = b > c ? b : c;
    return (int)(b > kBkMax ? kBkMax : b);
}
inline int bk_blocks(int64_t n) {
    const int64_t b = (n + 4095) / 4096;
    return (int)(b < 1 ? 1 : (b > kBkGrid ? kBkGrid : b));
}

struct BkGrid {
    float o0, o1, o2, scale;
    uint32_t depth;
    int linear;
};

struct BkWs {
    int nb = 0, blocks = 0, samples = 0;
    uint32_t *zero = nullptr;    // zeroed region: gbin, gcount
    uint32_t *gbin = nullptr;    // per group 2 nb: points per bin
    uint32_t *bin = nullptr;     // 2 nb: their sums
    uint32_t *gcount = nullptr;  // kBkGroups
    uint32_t *uniq = nullptr;    // nb: runs of each bucket
    size_t zero_bytes = 0;
    void *split = nullptr;       // nb - 1 splitters
    void *coarse = nullptr;      // kBkGroups - 1
    void *groups = nullptr;      // kBkGroups * kBkGroupCap sample keys
    uint32_t *start = nullptr;   // nb: first slot of each bucket
    uint32_t *cursor = nullptr;  // per group nb: next slot of each bucket
    uint16_t *ids = nullptr;     // n bins
    void *a = nullptr, *b = nullptr;
};

inline void bk_carve(Carve &c, BkWs &w, int64_t n, size_t kb) {
    w.nb = bk_buckets(n);
    w.blocks = bk_blocks(n);
    w.samples = w.nb * kBkOver;
    w.gbin = c.take<uint32_t>((size_t)kBkXcds * 2 * w.nb);
    w.gcount = c.take<uint32_t>(kBkGroups);
    w.uniq = c.take<uint32_t>((size_t)w.nb);
    w.split = c.take<char>((size_t)w.nb * kb);
    w.zero = w.gbin;
    w.zero_bytes = (size_t)((char *)w.uniq - (char *)w.gbin);
    w.bin = c.take<uint32_t>((size_t)2 * w.nb);
    w.coarse = c.take<char>(kBkGroups * kb);
    w.groups = c.take<char>(w.samples > kBkOneSort ? (size_t)kBkGroups * kBkGroupCap * kb : kb);
    w.start = c.take<uint32_t>((size_t)w.nb);
    w.cursor = c.take<uint32_t>((size_t)kBkXcds * w.nb);
    w.ids = c.take<uint16_t>((size_t)(n > 0 ? n : 1));
    w.a = c.take<char>((size_t)(n > 0 ? n : 1) * kb);
    w.b = c.take<char>((size_t)(n > 0 ? n : 1) * kb);
}

// ---------------------------------------------------------------- sample
// Position of sample i of S over n points: hashed within its stretch (the mix is
// MurmurHash3's 32-bit finalizer, in the public domain), so that no regularity
// of the input meets the sampling.
__device__ __forceinline__ int64_t bk_sample_at(int64_t i, int64_t S, int64_t n, uint32_t seed) {
    const int64_t lo = i * n / S, hi = (i + 1) * n / S;
    uint32_t h = (uint32_t)i * 0x9E3779B9u + seed;
    h = (h ^ (h >> 16)) * 0x85EBCA6Bu;
    h = (h ^ (h >> 13)) * 0xC2B2AE35u;
    h ^= h >> 16;
    return hi > lo ? lo + (int64_t)(h % (uint32_t)(hi - lo)) : lo;
}

template <typename K>
__device__ __forceinline__ K bk_encode_at(const float *xyz, int64_t i, const BkGrid &g, bool *ok) {
    const float o[3] = {g.o0, g.o1, g.o2};
    Vox v;
    *ok = quantize3(xyz[3 * i], xyz[3 * i + 1], xyz[3 * i + 2], o, g.scale, g.depth, v);
    return (K)enc3(v.x, v.y, v.z, g.depth, g.linear != 0);
}

// Rank of `mine` (index tag) among the keys [j0, j1) in LDS, ties by index.  A
// sort of a few thousand samples by one block is a chain of barriers (18 us for
// 1024); counting by many threads is one pass over LDS.
template <typename K>
__device__ __forceinline__ uint32_t bk_count_below(const K *s_k, int j0, int j1, K mine, int tag) {
    uint32_t r = 0;
#pragma unroll 4
    for (int j = j0; j < j1; ++j) {
        const K x = s_k[j];
        r += x < mine || (x == mine && j < tag) ? 1u : 0u;
    }
    return r;
}

// S <= kBkOneSort samples; every step-th of their order goes to out[0..m).
// Every block encodes all of them and ranks 16, its 64 quarter waves a share of
// the comparisons each.
template <typename K>
__global__ __launch_bounds__(kBkBlock) void k_bk_sample(const float *__restrict__ xyz, int64_t n,
                                                        BkGrid g, int S, uint32_t seed, int step,
                                                        K *__restrict__ out, int m) {
    __shared__ K s_k[kBkOneSort];
    __shared__ uint32_t s_rank[16];
    for (int i = threadIdx.x; i < S; i += kBkBlock) {
        bool ok;
        s_k[i] = bk_encode_at<K>(xyz, bk_sample_at(i, S, n, seed), g, &ok);
    }
    if (threadIdx.x < 16) s_rank[threadIdx.x] = 0;
    __syncthreads();
    const int i = blockIdx.x * 16 + (int)(threadIdx.x & 15u), share = (int)(threadIdx.x >> 4);
    const K mine = i < S ? s_k[i] : K(0);
    const int per = (S + kBkBlock / 16 - 1) / (kBkBlock / 16);
    const int j0 = share * per, j1 = j0 + per < S ? j0 + per : S;
    atomicAdd(&s_rank[threadIdx.x & 15u], bk_count_below(s_k, j0, j1, mine, i));
    __syncthreads();
    if (threadIdx.x < 16 && i < S) {
        const int r = (int)s_rank[threadIdx.x];
        if (r > 0 && r % step == 0 && r / step <= m) out[r / step - 1] = mine;
    }
}

// Samples to the parts between the coarse splitters.  Copies of a coarse
// splitter are dropped but for one a block: as a splitter it needs one, and a
// key that fills much of the input would fill its part.
template <typename K>
__global__ __launch_bounds__(256) void k_bk_distribute(const float *__restrict__ xyz, int64_t n,
                                                       BkGrid g, int S,
                                                       const K *__restrict__ coarse,
                                                       uint32_t *gcount, K *__restrict__ groups) {
    __shared__ uint32_t s_cnt[kBkGroups], s_eq[kBkGroups], s_base[kBkGroups];
    if (threadIdx.x < kBkGroups) s_cnt[threadIdx.x] = s_eq[threadIdx.x] = 0;
    __syncthreads();
    const int i = blockIdx.x * 256 + threadIdx.x;
    K k = 0;
    int at = 0;
    uint32_t rank = 0;
    bool use = i < S;
    if (use) {
        bool ok;
        k = bk_encode_at<K>(xyz, bk_sample_at(i, S, n, 0u), g, &ok);
        for (int h = kBkGroups / 2; h; h >>= 1)
            if (coarse[at + h - 1] < k) at += h;
        if (at < kBkGroups - 1 && coarse[at] == k) use = atomicExch(&s_eq[at], 1u) == 0;
        if (use) rank = atomicAdd(&s_cnt[at], 1u);
    }
    __syncthreads();
    if (threadIdx.x < kBkGroups && s_cnt[threadIdx.x])
        s_base[threadIdx.x] = atomicAdd(&gcount[threadIdx.x], s_cnt[threadIdx.x]);
    __syncthreads();
    if (use && s_base[at] + rank < kBkGroupCap) groups[at * kBkGroupCap + s_base[at] + rank] = k;
}

// A block per part: its samples ranked, every kBkOver-th of the whole order a
// splitter; the last part's block gives the splitters that no sample is left
// for the value above all keys.
template <typename K>
__global__ __launch_bounds__(kBkBlock) void k_bk_group_rank(const uint32_t *__restrict__ gcount,
                                                            const K *__restrict__ groups,
                                                            K *__restrict__ split, int m) {
    __shared__ K s_k[kBkGroupCap];
    __shared__ int s_first, s_cnt;
    const int gi = blockIdx.x, wave = threadIdx.x >> 6;
    if (threadIdx.x < kBkGroups) {
        const uint32_t c = gcount[threadIdx.x], k = c < kBkGroupCap ? c : kBkGroupCap;
        const uint32_t upto = wave_incl_sum(k);
        if ((int)threadIdx.x == gi) {
            s_first = (int)(upto - k);
            s_cnt = (int)k;
        }
    }
    __syncthreads();
    const int first = s_first, cnt = s_cnt;
    for (int i = threadIdx.x; i < cnt; i += kBkBlock) s_k[i] = groups[gi * kBkGroupCap + i];
    __syncthreads();
    // a wave ranks 16 at a time, a quarter of the comparisons per 16 lanes
    const int per = (cnt + 3) / 4, j0 = (lane_id() >> 4) * per, j1 = j0 + per < cnt ? j0 + per : cnt;
    for (int i0 = wave * 16; i0 < cnt; i0 += kBkWaves * 16) {
        const int i = i0 + (lane_id() & 15);
        const K mine = i < cnt ? s_k[i] : K(0);
        uint32_t below = bk_count_below(s_k, j0, j1, mine, i);
        below += __shfl_xor(below, 16, 64);
        below += __shfl_xor(below, 32, 64);
        const int r = first + (int)below;
        if (lane_id() < 16 && i < cnt && r > 0 && r % kBkOver == 0 && r / kBkOver <= m)
            split[r / kBkOver - 1] = mine;
    }
    if (gi == kBkGroups - 1) {
        const int total = first + cnt;
        const int have = total > 0 ? (total - 1) / kBkOver : 0;
        for (int j = have + threadIdx.x; j < m; j += kBkBlock) split[j] = ~K(0);
    }
}

// ---------------------------------------------------------------- encode
constexpr int kBkUnroll = 4;

// The splitters in LDS: a search tree level by level (node j's children 2 j and
// 2 j + 1, the root 1), padded with the largest value to p2 - 1, p2 a power of
// two.  In ascending order all probes of a search step lay a power of two apart,
// in one bank: so the encode of 10M points took 88 us, 60 of them conflicts, and
// takes 60.
template <typename K>
__device__ __forceinline__ void bk_load_tree(const K *__restrict__ split, int m, int p2, K *s_tree) {
    for (int i = 1 + (int)threadIdx.x; i < p2; i += kBkBlock) {  // i - 1 splitters below it
        const int t = __ffs(i);
        s_tree[(p2 >> t) + (i >> t)] = i <= m ? split[i - 1] : ~K(0);
    }
}

// Points [c0, c1) to keys and bins, the bins' counts to s_bin.  Returns whether a
// coordinate is not finite.
template <typename K>
__device__ __forceinline__ bool bk_encode_range(const float *__restrict__ xyz, int64_t c0, int64_t c1,
                                                const BkGrid &g, const K *s_tree, int p2,
                                                K *__restrict__ keys, uint16_t *__restrict__ ids,
                                                uint32_t *s_bin) {
    const float o[3] = {g.o0, g.o1, g.o2};
    bool bad = false;
    for (int64_t i0 = c0 + threadIdx.x; i0 - threadIdx.x < c1; i0 += kBkUnroll * kBkBlock) {
        float p[kBkUnroll][3];
#pragma unroll
        for (int u = 0; u < kBkUnroll; ++u) {
            const int64_t i = i0 + u * kBkBlock;
#pragma unroll
            for (int a = 0; a < 3; ++a) p[u][a] = i < c1 ? xyz[3 * i + a] : 0.0f;
        }
        K k[kBkUnroll];
        int at[kBkUnroll];
#pragma unroll
        for (int u = 0; u < kBkUnroll; ++u) {
            Vox v;
            const bool ok = quantize3(p[u][0], p[u][1], p[u][2], o, g.scale, g.depth, v);
            bad |= !ok && i0 + u * kBkBlock < c1;
            k[u] = (K)enc3(v.x, v.y, v.z, g.depth, g.linear != 0);
            at[u] = 1;
        }
        for (int h = p2 >> 1; h; h >>= 1) {
#pragma unroll
            for (int u = 0; u < kBkUnroll; ++u) at[u] = 2 * at[u] + (s_tree[at[u]] < k[u] ? 1 : 0);
        }
#pragma unroll
        for (int u = 0; u < kBkUnroll; ++u) {
            const int64_t i = i0 + u * kBkBlock;
            if (i >= c1) continue;
            // the path ends at leaf p2 + (splitters below the key); the last
            // node that it left downwards is the next splitter (0: there is none)
            const int next = at[u] >> __ffs(~at[u]);
            const uint32_t id = 2 * (at[u] - p2) + (next && s_tree[next] == k[u] ? 1 : 0);
            keys[i] = k[u];
            ids[i] = (uint16_t)id;
            // neighbouring points mostly share a bin: one add for all of them
            const uint64_t act = __ballot(1);
            const int leader = __ffsll((unsigned long long)act) - 1;
            const uint32_t id0 = __shfl(id, leader, 64);
            if (__ballot(id == id0) == act) {
                if (lane_id() == leader) atomicAdd(&s_bin[id0], (uint32_t)__popcll(act));
            } else {
                atomicAdd(&s_bin[id], 1u);
            }
        }
    }
    return bad;
}

// Block b owns the points [b * chunk, (b + 1) * chunk).
template <typename K>
__global__ __launch_bounds__(kBkBlock) void k_bk_encode(const float *__restrict__ xyz, int64_t n,
                                                        int64_t chunk, BkGrid g,
                                                        const K *__restrict__ split, int nb, int p2,
                                                        K *__restrict__ keys,
                                                        uint16_t *__restrict__ ids, uint32_t *gbin,
                                                        uint32_t *err) {
    extern __shared__ uint64_t s_dyn[];
    K *s_tree = (K *)s_dyn;                       // p2
    uint32_t *s_bin = (uint32_t *)(s_tree + p2);  // 2 nb
    bk_load_tree(split, nb - 1, p2, s_tree);
    for (int i = threadIdx.x; i < 2 * nb; i += kBkBlock) s_bin[i] = 0;
    __syncthreads();
    const int64_t c0 = (int64_t)blockIdx.x * chunk;
    const int64_t c1 = c0 + chunk < n ? c0 + chunk : n;
    if (bk_encode_range<K>(xyz, c0, c1, g, s_tree, p2, keys, ids, s_bin))
        set_err(err, ERR_NONFINITE);
    __syncthreads();
    for (int i = threadIdx.x; i < 2 * nb; i += kBkBlock) {
        const uint32_t c = s_bin[i];
        if (c) atomicAdd(&gbin[(size_t)(blockIdx.x % kBkXcds) * 2 * nb + i], c);
    }
}

// Sums of the groups' bins of buckets [b0, b1), and the buckets' first slots from
// `first` on, over all groups and per group; the groups' tables have nb buckets.
__device__ __forceinline__ void bk_scan_range(const uint32_t *__restrict__ gbin, int nb, int b0,
                                              int b1, uint32_t first, uint32_t *__restrict__ bin,
                                              uint32_t *__restrict__ start,
                                              uint32_t *__restrict__ cursor, uint32_t *s_w) {
    uint32_t carry = first;
    for (int i0 = b0; i0 < b1; i0 += kBkBlock) {
        const int i = i0 + (int)threadIdx.x;
        uint32_t v[kBkXcds], sum = 0, eq = 0;
#pragma unroll
        for (int g = 0; g < kBkXcds; ++g) {
            uint2 c = make_uint2(0, 0);
            if (i < b1) c = ((const uint2 *)gbin)[(size_t)g * nb + i];
            v[g] = c.x;
            sum += c.x;
            eq += c.y;
        }
        uint32_t tot;
        uint32_t ex = carry + block_excl_sum<kBkBlock>(sum, s_w, &tot);
        if (i < b1) {
            bin[2 * i] = sum;
            bin[2 * i + 1] = eq;
            start[i] = ex;
#pragma unroll
            for (int g = 0; g < kBkXcds; ++g) {
                cursor[(size_t)g * nb + i] = ex;
                ex += v[g];
            }
        }
        carry += tot;
    }
}

static __global__ __launch_bounds__(kBkBlock) void k_bk_scan(const uint32_t *__restrict__ gbin, int nb,
                                                      uint32_t *__restrict__ bin,
                                                      uint32_t *__restrict__ start,
                                                      uint32_t *__restrict__ cursor) {
    __shared__ uint32_t s_w[kBkWaves];
    bk_scan_range(gbin, nb, 0, nb, 0, bin, start, cursor, s_w);
}

// The keys of the points [c0, c1) to their buckets (nb of them, cursors of the
// block's group), tile by tile: a tile's keys are counted per bucket in LDS, each
// bucket's share is taken from its cursor at once, and the keys go to it in any
// order.
template <typename K>
__device__ __forceinline__ void bk_scatter_range(const K *__restrict__ keys,
                                                 const uint16_t *__restrict__ ids, int64_t c0,
                                                 int64_t c1, int iu, int nb, uint32_t *cursor,
                                                 K *__restrict__ out, uint32_t *s_cnt) {
    for (int64_t t0 = c0; t0 < c1; t0 += (int64_t)iu * kBkBlock) {
        for (int i = threadIdx.x; i < nb; i += kBkBlock) s_cnt[i] = 0;
        __syncthreads();
        K k[kBkItems];
        uint32_t at[kBkItems];  // bucket, rank in the tile
        const int64_t i0 = t0 + threadIdx.x;
#pragma unroll
        for (int u = 0; u < kBkItems; ++u) {
            const int64_t i = i0 + u * kBkBlock;
            at[u] = u < iu && i < c1 ? ids[i] : 1u;
            k[u] = u < iu && i < c1 ? keys[i] : K(0);
        }
#pragma unroll
        for (int u = 0; u < kBkItems; ++u) {
            if (at[u] & 1u) continue;  // a splitter's copies stay behind
            const uint32_t b = at[u] >> 1;
            const uint64_t act = __ballot(1);
            const int leader = __ffsll((unsigned long long)act) - 1;
            const uint32_t b0 = __shfl(b, leader, 64);
            uint32_t r;
            if (__ballot(b == b0) == act) {
                uint32_t r0 = 0;
                if (lane_id() == leader) r0 = atomicAdd(&s_cnt[b0], (uint32_t)__popcll(act));
                r = __shfl(r0, leader, 64) + (uint32_t)__popcll(act & lanemask_lt());
            } else {
                r = atomicAdd(&s_cnt[b], 1u);
            }
            at[u] |= r << 16;
        }
        __syncthreads();
        for (int i = threadIdx.x; i < nb; i += kBkBlock) {
            const uint32_t c = s_cnt[i];
            if (c) s_cnt[i] = atomicAdd(&cursor[i], c);
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kBkItems; ++u)
            if (!(at[u] & 1u)) out[s_cnt[(at[u] & 0xFFFFu) >> 1] + (at[u] >> 16)] = k[u];
        __syncthreads();
    }
}

template <typename K>
__global__ __launch_bounds__(kBkBlock) void k_bk_scatter(const K *__restrict__ keys,
                                                         const uint16_t *__restrict__ ids,
                                                         int64_t n, int64_t chunk, int iu, int nb,
                                                         uint32_t *cursor, K *__restrict__ out) {
    extern __shared__ uint32_t s_cnt[];
    const int64_t c0 = (int64_t)blockIdx.x * chunk;
    const int64_t c1 = c0 + chunk < n ? c0 + chunk : n;
    bk_scatter_range<K>(keys, ids, c0, c1, iu, nb, cursor + (size_t)(blockIdx.x % kBkXcds) * nb, out,
                        s_cnt);
}

// ------------------------------------------------------------------ sort
// Inclusive wave sum by DPP: rows of 16 by shifts, then row totals broadcast.
__device__ __forceinline__ uint32_t bk_wave_incl(uint32_t v) {
    int x = (int)v;
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);  // row_shr:1
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);  // row_shr:2
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);  // row_shr:4
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);  // row_shr:8
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);  // row_bcast:15
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);  // row_bcast:31
    return (uint32_t)x;
}

constexpr int kBkBinBits = 13;   // bins of a bucket's differences, two 16-bit counts a word
constexpr int kBkBinMost = 128;  // keys of one bin that are placed by comparing them

struct BkShared {
    alignas(16) uint32_t x[kBkCap + 4];  // keys of a pass (halves of wide ones), run starts
    union {
        uint16_t wcnt[kBkWaves][256];   // per wave and digit: count, then offset
        alignas(16) uint32_t bins[1 << (kBkBinBits - 1)];  // counts, then first slots
    };
    uint32_t off[256];                  // block offset of each digit
    uint32_t tot[256];                  // its count in the tile
    uint32_t w[kBkWaves];
    uint64_t edge[kBkWaves];            // each wave's last key
    uint64_t lo, hi;
    uint32_t most;
};

// Ranks of the keys of iu items per thread (wave w holds elements
// [64 iu w, 64 iu (w + 1)) in item, lane order) by digit (k >> shift) & 255
// among equal digits of the wave; then per wave and digit offsets in s.wcnt
// and the digits' block offsets in s.off.
template <typename T, int ITEMS>
__device__ __forceinline__ void bk_rank(BkShared &s, const T (&k)[ITEMS], int iu, int shift,
                                        uint16_t (&rank)[ITEMS]) {
    const int tid = threadIdx.x, wave = tid >> 6;
    uint32_t *z = (uint32_t *)&s.wcnt[0][0];
    for (int i = tid; i < kBkWaves * 128; i += kBkBlock) z[i] = 0;
    __syncthreads();
    const uint64_t lt = lanemask_lt();
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        if (i < iu) {
            const uint32_t d = (uint32_t)(k[i] >> shift) & 255u;
            const uint64_t m = match_low_bits<8>(d);
            const uint32_t before = s.wcnt[wave][d];
            const uint32_t pre = (uint32_t)__popcll(m & lt);
            rank[i] = (uint16_t)(before + pre);
            if (pre == 0) s.wcnt[wave][d] = (uint16_t)(before + (uint32_t)__popcll(m));
        }
    }
    __syncthreads();
    uint32_t sum = 0;
    if (tid < 256) {
#pragma unroll
        for (int w = 0; w < kBkWaves; ++w) {
            const uint32_t c = s.wcnt[w][tid];
            s.wcnt[w][tid] = (uint16_t)sum;
            sum += c;
        }
    }
    const uint32_t inc = bk_wave_incl(sum);
    if (tid < 256 && lane_id() == 63) s.w[wave] = inc;
    __syncthreads();
    if (tid < 256) {
        uint32_t b = inc - sum;
        for (int w = 0; w < wave; ++w) b += s.w[w];
        s.off[tid] = b;
        s.tot[tid] = sum;
    }
    __syncthreads();
}

// Sorts cnt <= 64 * kBkWaves * iu keys held in registers by their low `bits`
// bits, padding (largest values, last in order) included.
template <typename T, int ITEMS>
__device__ __forceinline__ void bk_sort_regs(BkShared &s, T (&k)[ITEMS], int iu, int bits) {
    const int wave = threadIdx.x >> 6, wbase = wave * 64 * iu + lane_id();
    uint16_t rank[ITEMS];
    for (int shift = 0; shift < bits; shift += 8) {
        bk_rank(s, k, iu, shift, rank);
#pragma unroll
        for (int i = 0; i < ITEMS; ++i)
            if (i < iu) {
                const uint32_t d = (uint32_t)(k[i] >> shift) & 255u;
                const uint32_t pos = s.off[d] + s.wcnt[wave][d] + rank[i];
                rank[i] = (uint16_t)pos;
                s.x[pos] = (uint32_t)k[i];
            }
        __syncthreads();
        if constexpr (sizeof(T) == 4) {
#pragma unroll
            for (int i = 0; i < ITEMS; ++i)
                if (i < iu) k[i] = s.x[wbase + i * 64];
            // the next pass writes s.x only after its own barriers
        } else {
            uint32_t low[ITEMS];
#pragma unroll
            for (int i = 0; i < ITEMS; ++i)
                if (i < iu) low[i] = s.x[wbase + i * 64];
            __syncthreads();
#pragma unroll
            for (int i = 0; i < ITEMS; ++i)
                if (i < iu) s.x[rank[i]] = (uint32_t)((uint64_t)k[i] >> 32);
            __syncthreads();
#pragma unroll
            for (int i = 0; i < ITEMS; ++i)
                if (i < iu) k[i] = (T)(((uint64_t)s.x[wbase + i * 64] << 32) | low[i]);
        }
    }
}

// Sorts cnt keys (differences of `bits` bits below 2^32 - 1, ITEMS per thread,
// element order as in bk_rank) without radix passes: one split by the top
// kBkBinBits bits with an LDS counter per bin, then each key's place among its
// bin's keys by comparing it with them.  Keys on surfaces leave some tens in a
// bin that is not empty, a gap in the bucket leaves hundreds: over kBkBinMost
// the keys stay as they are, for the radix passes, and the result is false.
template <int ITEMS>
__device__ __forceinline__ bool bk_sort_bins(BkShared &s, uint32_t (&k)[ITEMS], int iu, int cnt,
                                             int bits) {
    const int tid = threadIdx.x, wave = tid >> 6, lane = lane_id(), wbase = wave * 64 * iu + lane;
    const int sh = bits > kBkBinBits ? bits - kBkBinBits : 0;
    constexpr int WORDS = 1 << (kBkBinBits - 1), PER = WORDS / kBkBlock;
    uint4 *const z = (uint4 *)s.bins;
    for (int i = tid; i < WORDS / 4; i += kBkBlock) z[i] = make_uint4(0, 0, 0, 0);
    if (tid == 0) s.most = 0;
    if (tid < 4) s.x[cnt + tid] = ~0u;  // past every key, for the reads of four
    __syncthreads();
    uint16_t rank[ITEMS];
#pragma unroll
    for (int i = 0; i < ITEMS; ++i)
        if (i < iu && wbase + i * 64 < cnt) {
            const uint32_t d = k[i] >> sh, up = (d & 1u) << 4;
            rank[i] = (uint16_t)(atomicAdd(&s.bins[d >> 1], 1u << up) >> up);
        }
    __syncthreads();
    uint32_t c[PER], sum = 0, most = 0;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        c[j] = s.bins[tid * PER + j];
        const uint32_t lo = c[j] & 0xFFFFu, hi = c[j] >> 16;
        sum += lo + hi;
        most = most > lo ? most : lo;
        most = most > hi ? most : hi;
    }
    const uint32_t inc = bk_wave_incl(sum);
    if (lane == 63) s.w[wave] = inc;
    if (sh && most > (uint32_t)kBkBinMost) s.most = 1;
    __syncthreads();
    const bool fits = s.most == 0;
    uint32_t at = inc - sum;
    for (int w = 0; w < wave; ++w) at += s.w[w];
    if (!fits) {
        __syncthreads();  // the caller goes on to write what was read here
        return false;
    }
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const uint32_t lo = c[j] & 0xFFFFu;
        s.bins[tid * PER + j] = at | ((at + lo) << 16);
        at += lo + (c[j] >> 16);
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < ITEMS; ++i)
        if (i < iu && wbase + i * 64 < cnt) {
            const uint32_t d = k[i] >> sh;
            s.x[((s.bins[d >> 1] >> ((d & 1u) << 4)) & 0xFFFFu) + rank[i]] = k[i];
        }
    __syncthreads();
    if (sh) {
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            const int j = wbase + i * 64;
            if (i < iu && j < cnt) {
                const uint32_t v = s.x[j], d = v >> sh;
                const uint32_t w0 = s.bins[d >> 1];
                const uint32_t w1 = s.bins[((d + 1) >> 1) & (WORDS - 1)];
                const int b0 = (int)((w0 >> ((d & 1u) << 4)) & 0xFFFFu) & ~3;
                const int b1 = d + 1 == 2 * WORDS ? cnt : (int)((w1 >> (((d + 1) & 1u) << 4)) & 0xFFFFu);
                // four at a time from an aligned start: the keys before the
                // bin are below v, those after it above; of equal keys the
                // earlier slots come first
                int p = b0;
#pragma unroll 2
                for (int t = b0; t < b1; t += 4) {
                    const uint4 y = *(const uint4 *)&s.x[t];
                    p += y.x < v + (t < j ? 1u : 0u) ? 1 : 0;
                    p += y.y < v + (t + 1 < j ? 1u : 0u) ? 1 : 0;
                    p += y.z < v + (t + 2 < j ? 1u : 0u) ? 1 : 0;
                    p += y.w < v + (t + 3 < j ? 1u : 0u) ? 1 : 0;
                }
                k[i] = v;
                rank[i] = (uint16_t)p;
            }
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < ITEMS; ++i)
            if (i < iu && wbase + i * 64 < cnt) s.x[rank[i]] = k[i];
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < ITEMS; ++i)
        if (i < iu && wbase + i * 64 < cnt) k[i] = s.x[wbase + i * 64];
    return true;
}

// Runs of cnt sorted keys in registers (element order as in bk_rank): values to
// out, lengths to len (nullable); returns their number.
template <typename T, int ITEMS, typename K>
__device__ __forceinline__ uint32_t bk_runs(BkShared &s, const T (&k)[ITEMS], int iu, int cnt,
                                            uint64_t lo, K *out, uint32_t *len) {
    const int wave = threadIdx.x >> 6, lane = lane_id(), wbase = wave * 64 * iu + lane;
    T last = 0;
#pragma unroll
    for (int i = 0; i < ITEMS; ++i)
        if (i < iu) last = k[i];
    if (lane == 63) s.edge[wave] = (uint64_t)last;
    __syncthreads();
    uint32_t heads = 0, mine = 0, wtot = 0;
    T prev_last = wave > 0 ? (T)s.edge[wave - 1] : T(0);
    const uint64_t lt = lanemask_lt();
    uint16_t at[ITEMS];
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        if (i < iu) {
            T prev = __shfl_up(k[i], 1, 64);
            if (lane == 0) prev = prev_last;
            prev_last = __shfl(k[i], 63, 64);
            const int j = wbase + i * 64;
            const bool head = j < cnt && (j == 0 || prev != k[i]);
            const uint64_t m = __ballot(head);
            at[i] = (uint16_t)(wtot + (uint32_t)__popcll(m & lt));
            wtot += (uint32_t)__popcll(m);
            heads |= head ? 1u << i : 0u;
        }
    }
    if (lane == 0) s.w[wave] = wtot;
    __syncthreads();
    uint32_t u = 0;
#pragma unroll
    for (int w = 0; w < kBkWaves; ++w) {
        const uint32_t c = s.w[w];
        mine += w < wave ? c : 0u;
        u += c;
    }
#pragma unroll
    for (int i = 0; i < ITEMS; ++i)
        if (i < iu && ((heads >> i) & 1u)) s.x[mine + at[i]] = (uint32_t)(wbase + i * 64);
    if (threadIdx.x == 0) s.x[u] = (uint32_t)cnt;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < ITEMS; ++i)
        if (i < iu && ((heads >> i) & 1u)) {
            const uint32_t r = mine + at[i];
            out[r] = (K)(lo + k[i]);
            if (len) len[r] = s.x[r + 1] - s.x[r];
        }
    return u;
}

// A bucket that LDS does not hold: radix passes between src and tmp, tile by
// tile; the run starts to the buffer that the passes did not end in, then values
// and lengths to where bk_runs leaves them.
template <typename K>
__device__ __noinline__ uint32_t bk_sort_large(BkShared &s, K *src, K *tmp, uint32_t cnt,
                                                uint64_t lo, int bits, bool lengths) {
    K *const out = src;
    uint32_t *const len = (uint32_t *)tmp;
    const int tid = threadIdx.x, wave = tid >> 6, lane = lane_id();
    constexpr int IU = 4, TILE = kBkBlock * IU;
    for (int shift = 0; shift < bits; shift += 8) {
        // digit starts, kept by threads 0..255 through the pass
        uint32_t *h = s.x, *g = s.x + 256;
        if (tid < 256) h[tid] = 0;
        __syncthreads();
        for (uint32_t j = tid; j < cnt; j += kBkBlock)
            atomicAdd(&h[(uint32_t)(((uint64_t)src[j] - lo) >> shift) & 255u], 1u);
        __syncthreads();
        const uint32_t c = tid < 256 ? h[tid] : 0u, inc = wave_incl_sum(c);
        if (tid < 256 && lane == 63) s.w[wave] = inc;
        __syncthreads();
        if (tid < 256) {
            uint32_t before = inc - c;
            for (int w = 0; w < wave; ++w) before += s.w[w];
            g[tid] = before;
        }
        for (uint32_t t0 = 0; t0 < cnt; t0 += TILE) {
            uint64_t k[IU];
            uint16_t rank[IU];
#pragma unroll
            for (int i = 0; i < IU; ++i) {
                const uint32_t j = t0 + wave * 64 * IU + i * 64 + lane;
                k[i] = j < cnt ? (uint64_t)src[j] - lo : ~0ull;
            }
            bk_rank(s, k, IU, shift, rank);
#pragma unroll
            for (int i = 0; i < IU; ++i) {
                const uint32_t j = t0 + wave * 64 * IU + i * 64 + lane;
                if (j < cnt) {
                    const uint32_t d = (uint32_t)(k[i] >> shift) & 255u;
                    tmp[g[d] + s.wcnt[wave][d] + rank[i]] = (K)(k[i] + lo);
                }
            }
            __syncthreads();
            if (tid < 256) g[tid] += s.tot[tid];  // padding counts only past the last key
            __syncthreads();
        }
        K *sw = src;
        src = tmp;
        tmp = sw;
    }
    if (src != out) {  // an odd number of passes
        for (uint32_t j = tid; j < cnt; j += kBkBlock) out[j] = src[j];
        tmp = src;
        src = out;
        __syncthreads();
    }
    // run starts, in order, to tmp
    uint32_t u = 0;
    for (uint32_t t0 = 0; t0 < cnt; t0 += kBkBlock) {
        const uint32_t j = t0 + tid;
        const bool head = j < cnt && (j == 0 || src[j] != src[j - 1]);
        uint32_t tot;
        const uint32_t ex = block_excl_sum<kBkBlock>(head ? 1u : 0u, s.w, &tot);
        if (head) tmp[u + ex] = (K)j;
        u += tot;
    }
    __syncthreads();
    // slot r of out and len lies at or before what run r reads, and later runs
    // read past it
    for (uint32_t t0 = 0; t0 < u; t0 += kBkBlock) {
        const uint32_t r = t0 + tid;
        K v = 0;
        uint32_t c = 0;
        if (r < u) {
            const uint32_t j = (uint32_t)tmp[r], e = r + 1 < u ? (uint32_t)tmp[r + 1] : cnt;
            v = src[j];
            c = e - j;
        }
        __syncthreads();
        if (r < u) {
            out[r] = v;
            if (lengths) len[r] = c;
        }
        __syncthreads();
    }
    return u;
}

// A block per bucket.  vals holds the buckets' keys, tmp as many slots (of the
// large buckets' passes).  The runs' values go to the bucket's first slots of
// vals, their lengths to the start of its part of tmp, their number (the
// splitter's run not included) to uniq: a bucket that waited here for the ones
// before it (a look-back) spent half its time on the slowest of them.
template <typename K>
__global__ __launch_bounds__(kBkBlock, 8) void k_bk_sort(K *vals, K *tmp, int nb,
                                                         const uint32_t *__restrict__ start,
                                                         const uint32_t *__restrict__ bin,
                                                         const K *__restrict__ split,
                                                         uint32_t *__restrict__ uniq, int lengths) {
    __shared__ BkShared s;
    const int tid = threadIdx.x, wave = tid >> 6, lane = lane_id();
    if (tid == 0) {
        s.lo = ~0ull;
        s.hi = 0;
    }
    const uint32_t b = blockIdx.x, first = start[b], cnt = bin[2 * b];
    K *src = vals + first;
    uint32_t *len = lengths ? (uint32_t *)(tmp + first) : nullptr;
    __syncthreads();
    // the splitters bound the bucket; one that is open on a side looks for its
    // least and largest key
    uint64_t lo0 = 0, span = 0;
    if (b > 0 && b < (uint32_t)nb - 1 && split[b - 1] != ~K(0) && split[b] != ~K(0)) {
        lo0 = (uint64_t)split[b - 1];
        span = (uint64_t)split[b] - lo0;
    } else if (cnt) {
        K lo = ~K(0), hi = K(0);
        for (uint32_t j = tid; j < cnt; j += kBkBlock) {
            const K v = src[j];
            lo = v < lo ? v : lo;
            hi = v > hi ? v : hi;
        }
        if (lo <= hi) {
            atomicMin((unsigned long long *)&s.lo, (unsigned long long)lo);
            atomicMax((unsigned long long *)&s.hi, (unsigned long long)hi);
        }
        __syncthreads();
        lo0 = s.lo;
        span = s.hi - s.lo;
    }
    const int bits = span ? 64 - __clzll((long long)span) : 0;
    const int iu = (int)((cnt + kBkBlock - 1) / kBkBlock), wbase = wave * 64 * iu + lane;
    uint32_t u;
    if (bits <= 32 && iu <= kBkItems) {
        uint32_t r[kBkItems];
#pragma unroll
        for (int i = 0; i < kBkItems; ++i)
            r[i] = i < iu && (uint32_t)(wbase + i * 64) < cnt
                       ? (uint32_t)((uint64_t)src[wbase + i * 64] - lo0) : ~0u;
        if (span == 0xFFFFFFFFu || !bk_sort_bins(s, r, iu, (int)cnt, bits))
            bk_sort_regs(s, r, iu, bits);
        u = bk_runs(s, r, iu, (int)cnt, lo0, src, len);
    } else if (sizeof(K) == 8 && iu <= kBkItems / 2) {
        uint64_t r[kBkItems / 2];
#pragma unroll
        for (int i = 0; i < kBkItems / 2; ++i)
            r[i] = i < iu && (uint32_t)(wbase + i * 64) < cnt
                       ? (uint64_t)src[wbase + i * 64] - lo0 : ~0ull;
        bk_sort_regs(s, r, iu, bits);
        u = bk_runs(s, r, iu, (int)cnt, lo0, src, len);
    } else {
        u = bk_sort_large<K>(s, src, tmp + first, cnt, lo0, bits, lengths != 0);
    }
    if (tid == 0) uniq[b] = u;
}

// The runs of every bucket, and the splitter's behind them, to their final
// places, from the buckets' first places (bases) or, if null, the sum of the
// numbers before them.
template <typename K>
__global__ __launch_bounds__(256) void k_bk_emit(const K *__restrict__ vals,
                                                 const K *__restrict__ tmp, int nb,
                                                 const uint32_t *__restrict__ start,
                                                 const uint32_t *__restrict__ bin,
                                                 const K *__restrict__ split,
                                                 const uint32_t *__restrict__ uniq,
                                                 const uint32_t *__restrict__ bases,
                                                 K *__restrict__ keys, uint32_t *__restrict__ counts,
                                                 int64_t cap, int64_t *n_out, uint32_t *err) {
    __shared__ uint32_t s_w[4];
    const int b = blockIdx.x;
    uint32_t base;
    if (bases) {
        base = bases[b];
    } else {
        uint32_t before = 0;
        for (int i = threadIdx.x; i < b; i += 256) before += uniq[i] + (bin[2 * i + 1] ? 1u : 0u);
        block_excl_sum<256>(before, s_w, &base);
    }
    const uint32_t u = uniq[b], first = start[b], n_eq = bin[2 * b + 1];
    const uint32_t *len = (const uint32_t *)(tmp + first);
    for (uint32_t r = threadIdx.x; r < u && (int64_t)base + r < cap; r += 256) {
        keys[(size_t)base + r] = vals[(size_t)first + r];
        if (counts) counts[(size_t)base + r] = len[r];
    }
    if (threadIdx.x == 0) {
        int64_t end = (int64_t)base + u;
        if (n_eq) {
            if (end < cap) {
                keys[end] = split[b];
                if (counts) counts[end] = n_eq;
            }
            ++end;
        }
        if (b == nb - 1 && n_out) *n_out = end;
        if (end > cap) set_err(err, ERR_CAPACITY);
    }
}

// ------------------------------------------------------------------ host
template <typename K>
inline void bk_launch(const cga_grid *g, const float *xyz, int64_t n, const BkWs &w, K *keys,
                     uint32_t *counts, int64_t cap, int64_t *n_out, uint32_t *err,
                     hipStream_t s) {
    const BkGrid bg{g->origin[0], g->origin[1], g->origin[2], g->scale, g->depth,
                    g->key_mode == CGA_KEY_LINEAR};
    const int m = w.nb - 1;
    K *split = (K *)w.split, *a = (K *)w.a, *b = (K *)w.b;
    if (m > 0) {
        CGA_PROF("bucket_sample", s);
        if (w.samples <= kBkOneSort) {
            k_bk_sample<K><<<(unsigned)((w.samples + 15) / 16), kBkBlock, 0, s>>>(
                xyz, n, bg, w.samples, 0u, kBkOver, split, m);
        } else {
            k_bk_sample<K><<<kBkGroups * kBkCoarse / 16, kBkBlock, 0, s>>>(
                xyz, n, bg, kBkGroups * kBkCoarse, 0x51ED27u, kBkCoarse, (K *)w.coarse,
                kBkGroups - 1);
            k_bk_distribute<K><<<(unsigned)((w.samples + 255) / 256), 256, 0, s>>>(
                xyz, n, bg, w.samples, (const K *)w.coarse, w.gcount, (K *)w.groups);
            k_bk_group_rank<K><<<kBkGroups, kBkBlock, 0, s>>>(w.gcount, (const K *)w.groups, split, m);
        }
    }
    int p2 = 1;
    while (p2 < w.nb) p2 <<= 1;
    const int64_t chunk = (n + w.blocks - 1) / w.blocks;
    {
        CGA_PROF("encode", s);
        const size_t lds = (size_t)p2 * sizeof(K) + (size_t)2 * w.nb * 4;
        k_bk_encode<K><<<(unsigned)w.blocks, kBkBlock, lds, s>>>(xyz, n, chunk, bg, split, w.nb, p2,
                                                                 a, w.ids, w.gbin, err);
    }
    {
        CGA_PROF("bucket_scatter", s);
        k_bk_scan<<<1, kBkBlock, 0, s>>>(w.gbin, w.nb, w.bin, w.start, w.cursor);
        const int64_t tiles = (chunk + kBkCap - 1) / kBkCap;
        const int iu = (int)((chunk + tiles * kBkBlock - 1) / (tiles * kBkBlock));
        k_bk_scatter<K><<<(unsigned)w.blocks, kBkBlock, (size_t)w.nb * 4, s>>>(
            a, w.ids, n, chunk, iu, w.nb, w.cursor, b);
    }
    {
        CGA_PROF("bucket_sort", s);
        k_bk_sort<K><<<(unsigned)w.nb, kBkBlock, 0, s>>>(b, a, w.nb, w.start, w.bin, split, w.uniq,
                                                         counts ? 1 : 0);
    }
    CGA_PROF("bucket_emit", s);
    k_bk_emit<K><<<(unsigned)w.nb, 256, 0, s>>>(b, a, w.nb, w.start, w.bin, split, w.uniq, nullptr, keys,
                                                counts, cap, n_out, err);
}

}  // namespace cga

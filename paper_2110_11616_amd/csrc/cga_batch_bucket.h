// The build by buckets (cga_bucket.h) of many frames at once: every frame has
// its own splitters and buckets, counted on the device from the frame's size,
// and its buckets are a range of one list, so the sort of the buckets is the
// single build's and the keys need no frame bits.
#pragma once

#include "cga_bucket.h"

namespace cga {

constexpr int kBbMax = 4096;       // buckets of one frame: 4096 points each up to 16M points
constexpr int kBbSamples = 16384;  // samples of one frame that its block sorts

// Points per bucket of F frames of n points in all: 4096, or, of few points whose
// average bucket spans 30 key bits or more, what gives two buckets a CU.  A
// bucket beyond 32 bits (Morton neighbours across a high bit) is sorted by 64-bit
// passes, and above 7168 keys (3 % of them at 4096 on average) through global
// memory: 100 us and more that few other buckets hide (us at 4096 / so, surfaces
// in random order: 600k 42-bit keys 169 / 116, 4 frames of 300k, 36 bits 228 / 162,
// 16 of 150k, 42 bits 305 / 230; LiDAR sweeps 104 / 110, 167 / 158, 262 / 214).
// From kBbFew on others do, and more buckets cost the LiDAR sweeps 5 %.
constexpr int kBbLeast = 1024, kBbWideMost = 2560;
constexpr int64_t kBbFew = (int64_t)kBbWideMost * 2048;
inline int bb_most(int F, int64_t n, int bits) {
    int lg = 0;
    while (((int64_t)8192 << lg) <= n / F) ++lg;
    if (bits - lg < 30 || n > kBbFew) return 4096;
    const int64_t fill = n / 512;
    return (int)(fill < kBbLeast ? kBbLeast : (fill < kBbWideMost ? fill : kBbWideMost));
}

struct BbWs {
    int nb = 0;                  // bound on the buckets of all frames
    int most = 0;                // points per bucket
    uint32_t *gbin = nullptr, *bin = nullptr;  // zeroed: per group and in all 2 nb
    size_t zero_bytes = 0;
    int32_t *fb = nullptr;       // F + 1: first bucket of each frame
    uint32_t *uniq = nullptr, *start = nullptr, *cursor = nullptr, *bases = nullptr;
    void *split = nullptr;       // nb; a frame's last is the value above all keys
    uint16_t *ids = nullptr;
    void *a = nullptr, *b = nullptr;
};

inline void bb_carve(Carve &c, BbWs &w, int F, int64_t n, size_t kb, int most) {
    w.most = most;
    w.nb = (int)(n / most + F);
    w.gbin = c.take<uint32_t>((size_t)kBkXcds * 2 * w.nb);
    w.bin = c.take<uint32_t>((size_t)2 * w.nb);
    w.fb = c.take<int32_t>((size_t)F + 1);
    w.zero_bytes = (size_t)((char *)w.fb - (char *)w.gbin);
    w.uniq = c.take<uint32_t>((size_t)w.nb);
    w.start = c.take<uint32_t>((size_t)w.nb);
    w.bases = c.take<uint32_t>((size_t)w.nb + 1);
    w.cursor = c.take<uint32_t>((size_t)kBkXcds * w.nb);
    w.split = c.take<char>((size_t)w.nb * kb);
    w.ids = c.take<uint16_t>((size_t)n);
    w.a = c.take<char>((size_t)n * kb);
    w.b = c.take<char>((size_t)n * kb);
}

// First bucket of every frame: one per `most` points, at least one, at most
// kBbMax.  One block.
__global__ __launch_bounds__(kBkBlock) void k_bb_plan(const int64_t *__restrict__ off, int F,
                                                      int most, int32_t *__restrict__ fb) {
    __shared__ int32_t s_w[kBkWaves];
    int32_t carry = 0;
    for (int f0 = 0; f0 < F; f0 += kBkBlock) {
        const int f = f0 + (int)threadIdx.x;
        int64_t b = f < F ? (off[f + 1] - off[f]) / most : 0;
        b = b < 1 ? 1 : (b > kBbMax ? kBbMax : b);
        int32_t tot;
        const int32_t ex = block_excl_sum<kBkBlock>(f < F ? (int32_t)b : 0, s_w, &tot);
        if (f < F) fb[f] = carry + ex;
        carry += tot;
    }
    if (threadIdx.x == 0) fb[F] = carry;
}

// A block per frame: its samples sorted, its splitters at equal distances among
// them.  (Its LDS is a CU's; the blocks are short and few.)
template <typename K>
__global__ __launch_bounds__(kBkBlock) void k_bb_sample(const float *__restrict__ xyz,
                                                        const int64_t *__restrict__ off, BkGrid g,
                                                        const int32_t *__restrict__ fb,
                                                        K *__restrict__ split) {
    __shared__ K s_k[kBbSamples];
    const int f = blockIdx.x, b0 = fb[f], nb = fb[f + 1] - b0;
    const int64_t first = off[f], n = off[f + 1] - first;
    if (threadIdx.x == 0) split[b0 + nb - 1] = ~K(0);
    if (nb < 2) return;
    // eight a bucket up to 4096 (50 us), then as many more as leave three a
    // bucket: with one or two, frames of 8M to 60M points among smaller ones
    // took 1.2 to 1.7 times as long as by the radix passes, so 1.0 to 1.2
    int S = nb * kBkOver < kBkOneSort ? nb * kBkOver : kBkOneSort;
    while (S < 3 * nb && S < kBbSamples) S *= 2;
    int p2 = 2;
    while (p2 < S) p2 <<= 1;
    for (int i = threadIdx.x; i < p2; i += kBkBlock) {
        bool ok;
        s_k[i] = i < S ? bk_encode_at<K>(xyz, first + bk_sample_at(i, S, n, 0u), g, &ok) : ~K(0);
    }
    for (int k = 2; k <= p2; k <<= 1)  // bitonic
        for (int j = k >> 1; j > 0; j >>= 1) {
            __syncthreads();
            for (int t = threadIdx.x; t < p2 / 2; t += kBkBlock) {
                const int i = ((t & ~(j - 1)) << 1) | (t & (j - 1)), l = i | j;
                const K x = s_k[i], y = s_k[l];
                if ((x > y) == ((i & k) == 0)) {
                    s_k[i] = y;
                    s_k[l] = x;
                }
            }
        }
    __syncthreads();
    for (int j = threadIdx.x; j < nb - 1; j += kBkBlock) split[b0 + j] = s_k[(j + 1) * S / nb];
}

// Last frame f with off[f] <= i.
__device__ __forceinline__ int bb_frame_of(const int64_t *off, int F, int64_t i) {
    int lo = 0, len = F;
    while (len > 1) {
        const int half = len >> 1;
        lo = off[lo + half] <= i ? lo + half : lo;
        len -= half;
    }
    return lo;
}

// Block b owns the points [b * chunk, (b + 1) * chunk), frame by frame.
template <typename K>
__global__ __launch_bounds__(kBkBlock) void k_bb_encode(const float *__restrict__ xyz,
                                                        const int64_t *__restrict__ off, int F,
                                                        int64_t n, int64_t chunk, BkGrid g,
                                                        const int32_t *__restrict__ fb,
                                                        const K *__restrict__ split, int nb_all,
                                                        K *__restrict__ keys,
                                                        uint16_t *__restrict__ ids, uint32_t *gbin,
                                                        uint32_t *err) {
    __shared__ K s_tree[kBbMax];
    __shared__ uint32_t s_bin[2 * kBbMax];
    int64_t c0 = (int64_t)blockIdx.x * chunk;
    const int64_t c1 = c0 + chunk < n ? c0 + chunk : n;
    bool bad = false;
    for (int f = c0 < c1 ? bb_frame_of(off, F, c0) : F; f < F && c0 < c1; ++f) {
        const int64_t fe = off[f + 1], e = fe < c1 ? fe : c1;
        if (e <= c0) continue;  // uniform: an empty frame
        const int b0 = fb[f], nb = fb[f + 1] - b0;
        int p2 = 1;
        while (p2 < nb) p2 <<= 1;
        bk_load_tree(split + b0, nb - 1, p2, s_tree);
        for (int i = threadIdx.x; i < 2 * nb; i += kBkBlock) s_bin[i] = 0;
        __syncthreads();
        bad |= bk_encode_range<K>(xyz, c0, e, g, s_tree, p2, keys, ids, s_bin);
        __syncthreads();
        uint32_t *out = gbin + ((size_t)(blockIdx.x % kBkXcds) * nb_all + b0) * 2;
        for (int i = threadIdx.x; i < 2 * nb; i += kBkBlock) {
            const uint32_t c = s_bin[i];
            if (c) atomicAdd(&out[i], c);
        }
        __syncthreads();
        c0 = e;
    }
    if (bad) set_err(err, ERR_NONFINITE);
}

// A block per frame: its buckets' first slots, from the frame's first point on.
__global__ __launch_bounds__(kBkBlock) void k_bb_scan(const int64_t *__restrict__ off,
                                                      const int32_t *__restrict__ fb,
                                                      const uint32_t *__restrict__ gbin, int nb_all,
                                                      uint32_t *__restrict__ bin,
                                                      uint32_t *__restrict__ start,
                                                      uint32_t *__restrict__ cursor) {
    __shared__ uint32_t s_w[kBkWaves];
    const int f = blockIdx.x;
    bk_scan_range(gbin, nb_all, fb[f], fb[f + 1], (uint32_t)off[f], bin, start, cursor, s_w);
}

template <typename K>
__global__ __launch_bounds__(kBkBlock) void k_bb_scatter(const K *__restrict__ keys,
                                                         const uint16_t *__restrict__ ids,
                                                         const int64_t *__restrict__ off, int F,
                                                         int64_t n, int64_t chunk,
                                                         const int32_t *__restrict__ fb, int nb_all,
                                                         uint32_t *cursor, K *__restrict__ out) {
    __shared__ uint32_t s_cnt[kBbMax];
    cursor += (size_t)(blockIdx.x % kBkXcds) * nb_all;
    int64_t c0 = (int64_t)blockIdx.x * chunk;
    const int64_t c1 = c0 + chunk < n ? c0 + chunk : n;
    for (int f = c0 < c1 ? bb_frame_of(off, F, c0) : F; f < F && c0 < c1; ++f) {
        const int64_t fe = off[f + 1], e = fe < c1 ? fe : c1;
        if (e <= c0) continue;
        const int64_t len = e - c0, tiles = (len + kBkCap - 1) / kBkCap;
        const int iu = (int)((len + tiles * kBkBlock - 1) / (tiles * kBkBlock));
        bk_scatter_range<K>(keys, ids, c0, e, iu, fb[f + 1] - fb[f], cursor + fb[f], out, s_cnt);
        c0 = e;
    }
}

// bases[b] = runs before bucket b, key_off[f] = runs before frame f.  One block.
__global__ __launch_bounds__(kBkBlock) void k_bb_bases(const uint32_t *__restrict__ uniq,
                                                       const uint32_t *__restrict__ bin, int nb,
                                                       const int32_t *__restrict__ fb, int F,
                                                       uint32_t *bases, int64_t *__restrict__ key_off) {
    __shared__ uint32_t s_w[kBkWaves];
    constexpr int PER = 8;
    uint32_t carry = 0;
    for (int i0 = 0; i0 < nb; i0 += kBkBlock * PER) {
        uint32_t v[PER], sum = 0;
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const int i = i0 + (int)threadIdx.x * PER + j;
            v[j] = i < nb ? uniq[i] + (bin[2 * i + 1] ? 1u : 0u) : 0u;
            sum += v[j];
        }
        uint32_t tot;
        uint32_t ex = carry + block_excl_sum<kBkBlock>(sum, s_w, &tot);
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const int i = i0 + (int)threadIdx.x * PER + j;
            if (i < nb) bases[i] = ex;
            ex += v[j];
        }
        carry += tot;
    }
    if (threadIdx.x == 0) bases[nb] = carry;
    __syncthreads();
    for (int f = threadIdx.x; f <= F; f += kBkBlock) key_off[f] = bases[fb[f]];
}

template <typename K>
inline void bb_launch(const cga_grid *g, const float *xyz, const int64_t *off, int F, int64_t n,
                      const BbWs &w, K *keys, uint32_t *counts, int64_t *key_off, int64_t *n_out,
                      uint32_t *err, hipStream_t s) {
    const BkGrid bg{g->origin[0], g->origin[1], g->origin[2], g->scale, g->depth,
                    g->key_mode == CGA_KEY_LINEAR};
    K *split = (K *)w.split, *a = (K *)w.a, *b = (K *)w.b;
    // a block's points: two scatter tiles, or fewer so that there are two blocks per CU
    int64_t blocks = (n + 2 * kBkCap - 1) / (2 * kBkCap);
    if (blocks < kBkGrid) blocks = bk_blocks(n);
    const int64_t chunk = (n + blocks - 1) / blocks;
    {
        CGA_PROF("bucket_sample", s);
        k_bb_plan<<<1, kBkBlock, 0, s>>>(off, F, w.most, w.fb);
        k_bb_sample<K><<<(unsigned)F, kBkBlock, 0, s>>>(xyz, off, bg, w.fb, split);
    }
    {
        CGA_PROF("batch_encode", s);
        k_bb_encode<K><<<(unsigned)blocks, kBkBlock, 0, s>>>(xyz, off, F, n, chunk, bg, w.fb, split,
                                                             w.nb, a, w.ids, w.gbin, err);
    }
    {
        CGA_PROF("bucket_scatter", s);
        k_bb_scan<<<(unsigned)F, kBkBlock, 0, s>>>(off, w.fb, w.gbin, w.nb, w.bin, w.start, w.cursor);
        k_bb_scatter<K><<<(unsigned)blocks, kBkBlock, 0, s>>>(a, w.ids, off, F, n, chunk, w.fb, w.nb,
                                                              w.cursor, b);
    }
    {
        CGA_PROF("bucket_sort", s);
        k_bk_sort<K><<<(unsigned)w.nb, kBkBlock, 0, s>>>(b, a, w.nb, w.start, w.bin, split, w.uniq,
                                                         counts ? 1 : 0);
    }
    CGA_PROF("bucket_emit", s);
    k_bb_bases<<<1, kBkBlock, 0, s>>>(w.uniq, w.bin, w.nb, w.fb, F, w.bases, key_off);
    k_bk_emit<K><<<(unsigned)w.nb, 256, 0, s>>>(b, a, w.nb, w.start, w.bin, split, w.uniq, w.bases,
                                                keys, counts, n, n_out, err);
}

}  // namespace cga

// Orthogonal projection, Eq. (3) with m_x = m_y = 1 (Section V-B): the set of
// 2-D pixels left after dropping one axis, with the voxels on each.  Three
// ways, by what the key order gives:
//
// * LINEAR, dropping z: the pixel key is key >> depth, ascending already, so
//   one run-length pass does.
// * MORTON up to depth 14: the voxels over a square tile of pixels are the
//   column of cells above it, and each cell is one contiguous run of keys.  A
//   block counts a tile's pixels in LDS straight from those runs (no sort).
// * otherwise: every voxel re-keyed to its pixel, the pixel keys sorted, equal
//   ones collapsed.
#include "cga_common.h"
#include "cga_rle.h"
#include "cga_sort.h"

namespace cga {

SortCfg default_sort_cfg(bool wide, int64_t n, int key_bits);

template <typename K, typename K2, int RB>
__global__ __launch_bounds__(256) void k_rekey(const K *__restrict__ in, int64_t n_host,
                                               const int64_t *d_n, uint32_t depth, int linear,
                                               int drop, K2 *__restrict__ out, int passes,
                                               uint32_t *hist) {
    constexpr uint32_t RADIX = 1u << RB;
    extern __shared__ uint32_t s_h[];
    for (uint32_t i = threadIdx.x; i < passes * RADIX; i += blockDim.x) s_h[i] = 0;
    __syncthreads();
    const int64_t n = dev_count(n_host, d_n);
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        Vox v = dec3(in[i], depth, linear != 0);
        uint32_t u = drop == 0 ? v.y : v.x;
        uint32_t w = drop == 2 ? v.y : v.z;
        K2 k2 = linear ? (K2)(((uint64_t)u << depth) | w) : (K2)((spread2(u) << 1) | spread2(w));
        out[i] = k2;
        hist_add_coherent<RB>(s_h, k2, passes);
    }
    __syncthreads();
    hist_flush<RB>(s_h, hist, passes);
}

template <typename K, typename K2, int RB>
static void rekey_launch(const K *in, int64_t n, const int64_t *d_n, const cga_grid *g, int drop,
                         K2 *out, int passes, uint32_t *hist, hipStream_t s) {
    int64_t blocks = (n + 256 * 8 - 1) / (256 * 8);
    blocks = blocks < 1 ? 1 : (blocks > 1024 ? 1024 : blocks);
    CGA_PROF("rekey", s);
    k_rekey<K, K2, RB><<<(unsigned)blocks, 256, hist_lds_bytes(passes, RB), s>>>(
        in, n, d_n, g->depth, g->key_mode == CGA_KEY_LINEAR, drop, out, passes, hist);
}

template <typename K, typename K2>
static void rekey_dispatch(int rb, const K *in, int64_t n, const int64_t *d_n, const cga_grid *g,
                           int drop, K2 *out, int passes, uint32_t *hist, hipStream_t s) {
    switch (rb) {
        case 4: rekey_launch<K, K2, 4>(in, n, d_n, g, drop, out, passes, hist, s); break;
        case 5: rekey_launch<K, K2, 5>(in, n, d_n, g, drop, out, passes, hist, s); break;
        case 6: rekey_launch<K, K2, 6>(in, n, d_n, g, drop, out, passes, hist, s); break;
        case 7: rekey_launch<K, K2, 7>(in, n, d_n, g, drop, out, passes, hist, s); break;
        case 9: rekey_launch<K, K2, 9>(in, n, d_n, g, drop, out, passes, hist, s); break;
        case 10: rekey_launch<K, K2, 10>(in, n, d_n, g, drop, out, passes, hist, s); break;
        case 11: rekey_launch<K, K2, 11>(in, n, d_n, g, drop, out, passes, hist, s); break;
        default: rekey_launch<K, K2, 8>(in, n, d_n, g, drop, out, passes, hist, s); break;
    }
}

// --------------------------------------------------- MORTON grids by tiles
// Pixel tiles of 2^L x 2^L and cells of 2^L cubed.  L follows the depth: 64
// cells per axis (4096 tiles, enough for the chip's 256 CUs many times over)
// where a tile's counters then fit in 64 KB of LDS, which is up to depth 13;
// 128 at depth 14 (a 16 MB cell table, cleared on each call); depth 15 would
// need a table of 134 MB and takes the sort.
constexpr uint32_t kTileDepthMax = 14;
constexpr int kTileGroup = 32;  // tiles whose totals are summed together: at most 512 groups
// A tile of more voxels than this, over which one block would take longer
// than the sort of them all (a thin bundle along the dropped axis), leaves the
// projection to the sort, as does a pixel of more than the 16-bit counters
// hold (repeated keys).
constexpr uint32_t kTileHeavy = 1u << 18;
// Recorded beside the error bits: the tiles cannot do this array, because its
// keys are not ascending (which the sort does not need; set before the tiles
// run) or a tile or pixel is too heavy (set while they run).
constexpr uint32_t kProjUnsorted = 1u << 16, kProjHeavy = 1u << 17;
constexpr uint32_t kProjRedo = kProjUnsorted | kProjHeavy;

__host__ __device__ __forceinline__ uint32_t tile_level(uint32_t depth) {
    const uint32_t l = depth > 10 ? depth - 6 : 4;
    const uint32_t c = l > 7 ? 7 : l;
    return c < depth ? c : depth;
}

// The 2-D Morton code of a 3-D one without its bits of axis `drop`, for up to
// eight triples: each triple keeps two bits, and the pairs close up.
__device__ __forceinline__ uint32_t drop_axis24(uint32_t k, int drop) {
    uint32_t p = drop == 0 ? k & 0x6DB6DBu
                  : (drop == 2 ? (k >> 1) & 0x6DB6DBu : ((k >> 1) & 0x492492u) | (k & 0x249249u));
    p = (p & 0x0C30C3u) | ((p & 0x618618u) >> 1);
    p = (p & 0x00F00Fu) | ((p & 0x3C03C0u) >> 2);
    return (p & 0xFFu) | ((p & 0xFF000u) >> 4);
}
// The bits of axis `drop` of up to eight triples.
__device__ __forceinline__ uint32_t axis_bits24(uint32_t k, int drop) {
    return compact3((uint64_t)(k >> (2 - drop)) & 0x249249ull);
}

struct TileTables {
    uint2 *cells;           // [tile][cell of its column]: first key, one past the last
    uint32_t *tot, *gtot;   // voxels per tile and per group of tiles
    uint32_t *uniq, *from;  // pixels of a tile (then their place in the output); place in tmp
};

// Runs of keys of the same cell, filed under their tile.
template <typename K>
__global__ __launch_bounds__(256) void k_proj_cells(const K *__restrict__ keys, int64_t n_host,
                                                    const int64_t *d_n, uint32_t depth, uint32_t L,
                                                    int drop, TileTables T, uint32_t *err) {
    constexpr int kIn = 4;  // keys in flight per thread
    const int64_t n = dev_count(n_host, d_n);
    const int lane = lane_id();
    bool bad = false;
    for (int64_t i0 = (int64_t)blockIdx.x * (256 * kIn); i0 < n; i0 += (int64_t)gridDim.x * (256 * kIn)) {
        K k[kIn], edge[kIn];  // lanes 0 and 63 also need the key before or after their wave's
#pragma unroll
        for (int u = 0; u < kIn; ++u) {
            const int64_t i = i0 + u * 256 + threadIdx.x;
            const int64_t e = lane == 0 ? i - 1 : i + 1;
            k[u] = i < n ? keys[i] : K(0);
            edge[u] = (lane == 0 || lane == 63) && e >= 0 && e < n ? keys[e] : K(0);
        }
#pragma unroll
        for (int u = 0; u < kIn; ++u) {
            const int64_t i = i0 + u * 256 + threadIdx.x;
            K prev = (K)__shfl_up((unsigned long long)k[u], 1, 64);
            K next = (K)__shfl_down((unsigned long long)k[u], 1, 64);
            if (i >= n) continue;
            if (lane == 0) prev = edge[u];
            if (lane == 63) next = edge[u];
            bad |= (i > 0 && k[u] < prev) || ((uint64_t)k[u] >> (3 * depth)) != 0;
            const uint32_t c = (uint32_t)((uint64_t)k[u] >> (3 * L));
            const bool head = i == 0 || (uint32_t)((uint64_t)prev >> (3 * L)) != c;
            const bool tail = i + 1 == n || (uint32_t)((uint64_t)next >> (3 * L)) != c;
            if ((head || tail) && !bad) {
                const uint32_t t = drop_axis24(c, drop);
                uint2 *e = &T.cells[((size_t)t << (depth - L)) | axis_bits24(c, drop)];
                if (head) e->x = (uint32_t)i;
                if (tail) e->y = (uint32_t)i + 1u;
            }
        }
    }
    if (bad) set_err(err, kProjUnsorted);
}

// Voxels per tile and per group, a block per group (sums in place of global
// adds, which take turns on a cache line: 400 us for the runs of 20M keys).
__global__ __launch_bounds__(256) void k_proj_totals(TileTables T, uint32_t tiles, uint32_t cells) {
    __shared__ uint32_t s_t[kTileGroup];
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    uint32_t v[kTileGroup / 4];  // a wave's tiles: every load ahead of the sums
#pragma unroll
    for (int q = 0; q < kTileGroup / 4; ++q) {
        const uint32_t t = blockIdx.x * kTileGroup + q * 4 + wave;
        v[q] = 0;
#pragma unroll
        for (int c = 0; c < 128; c += 64)
            if (t < tiles && c + lane < (int)cells) {
                const uint2 e = T.cells[(size_t)t * cells + c + lane];
                v[q] += e.y - e.x;
            }
    }
#pragma unroll
    for (int q = 0; q < kTileGroup / 4; ++q) {
        const uint32_t t = blockIdx.x * kTileGroup + q * 4 + wave;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) v[q] += __shfl_xor(v[q], o, 64);
        if (lane == 0) {
            s_t[q * 4 + wave] = v[q];
            if (t < tiles) T.tot[t] = v[q];
        }
    }
    __syncthreads();
    if (wave == 0) {
        uint32_t v = lane < kTileGroup ? s_t[lane] : 0u;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
        if (lane == 0) T.gtot[blockIdx.x] = v;
    }
}

// One block per tile: its voxels counted per pixel in LDS (pixels in Morton
// order, so the counters are in output order), the pixels that have any
// written as (pixel of the tile << 16 | voxels) to tmp at the tile's first
// voxel number.  Two counters to a word: a tile of 128 x 128 pixels takes
// 32 KB.
//
// Bound: the latency of a tile's steps (its column, its keys, its counters)
// and the scan of the counters.  So a thread has kIn keys in flight and the
// 128 x 128 tiles 1024 threads (a tile of 200k voxels, a side view of a dense
// sweep, is one block's work: three views of 8M LiDAR points at depth 13 take
// 500 us so, 730 with 512 threads, 698 by the sort), and those of at most
// kSparseMax voxels go to a launch of their own (SPARSE): small blocks, eight
// to a CU, with a bitmap of the tile's pixels whose words' prefix sums number
// the occupied ones, and counters for those alone (300k voxels at depth 14,
// three views: 663 -> 380 us; by the sort 443).  20M voxels at depth 14, one
// view: 333 us, by the sort 628.
constexpr int kOwn = 4;  // voxels of a thread of a sparse tile at most
constexpr uint32_t kSparseMax = 256 * kOwn;

template <int LMAX, bool SPARSE>
constexpr int tile_block() {
    return SPARSE || LMAX <= 5 ? 256 : (LMAX == 6 ? 512 : 1024);
}

template <typename K, int LMAX, bool SPARSE = false>
__global__ __launch_bounds__((tile_block<LMAX, SPARSE>())) void k_proj_tiles(
    const K *__restrict__ keys, uint32_t depth, uint32_t L, int drop, TileTables T,
    uint32_t *__restrict__ tmp, uint32_t *err) {
    constexpr int kBlock = tile_block<LMAX, SPARSE>(), kWaves = kBlock / 64;
    constexpr int kCells = 128;                         // cells of a column at most
    constexpr int kPx = 1 << (2 * LMAX);                // pixels of a tile at most
    constexpr int kRows = (kPx + kBlock - 1) / kBlock;  // rows of the block in them
    constexpr int kIn = 8;                              // keys in flight per thread
    constexpr int kBits = kPx / 32, kBitsOwn = (kBits + kBlock - 1) / kBlock;
    __shared__ uint32_t s_px[SPARSE ? kSparseMax : kPx / 2];
    __shared__ uint32_t s_bits[SPARSE ? kBits : 1], s_pre[SPARSE ? kBits : 1];
    __shared__ uint16_t s_code[SPARSE ? kSparseMax : 1];
    __shared__ uint32_t s_first[kCells], s_end[kCells];  // runs: first key, last number in the column + 1
    __shared__ uint32_t s_off[kRows * kWaves], s_w[kWaves], s_c[4];
    const uint32_t t = blockIdx.x, total = T.tot[t];
    // block-uniform: this kernel leaves that bit alone
    if (total == 0 || (*err & kProjUnsorted)) return;
    if (LMAX >= 7 && (total <= kSparseMax) != SPARSE) return;  // the other launch's
    if (total > kTileHeavy) {
        if (threadIdx.x == 0) set_err(err, kProjHeavy);
        return;
    }
    const int tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
    const int cells = 1 << (depth - L), px = 1 << (2 * L);
    // the totals of the tiles before this one: whole groups, then its own's
    const uint32_t g = t / kTileGroup;
    uint32_t pre = 0;
    for (uint32_t i = tid; i < g; i += kBlock) pre += T.gtot[i];
    if (tid < kTileGroup && g * kTileGroup + tid < t) pre += T.tot[g * kTileGroup + tid];
    // the column's occupied cells, closed up, with the running number of
    // their voxels
    uint2 seg = make_uint2(0, 0);
    if (tid < cells) seg = T.cells[(size_t)t * cells + tid];
    const uint32_t len = seg.y - seg.x;
    const uint64_t occ = __ballot(len != 0);
    const uint32_t incl = wave_incl_sum(len);
    if (wave < 2 && lane == 63) {
        s_c[wave] = (uint32_t)__popcll(occ);
        s_c[2 + wave] = incl;
    }
    uint32_t before;
    block_excl_sum<kBlock>(pre, s_w, &before);  // its barriers cover s_c
    if (len) {
        const uint32_t at = (wave ? s_c[0] : 0u) + (uint32_t)__popcll(occ & lanemask_lt());
        s_first[at] = seg.x;
        s_end[at] = (wave ? s_c[2] : 0u) + incl;
    }
    for (int i = tid; i < (SPARSE ? (int)total : kPx / 2); i += kBlock) s_px[i] = 0;
    if (SPARSE)
        for (int i = tid; i < kBits; i += kBlock) s_bits[i] = 0;
    __syncthreads();
    // the column's voxels by number: a thread's numbers ascend, so its run does
    const uint32_t low = (1u << (3 * L)) - 1u;
    int run = 0;
    uint32_t start = 0;  // number of the run's first voxel
    if (tid < total) {
        int len2 = (int)(s_c[0] + s_c[1]);
        while (len2 > 1) {  // first run that ends past number tid
            const int half = len2 >> 1;
            if (s_end[run + half - 1] <= (uint32_t)tid) run += half;
            len2 -= half;
        }
        start = run ? s_end[run - 1] : 0u;
    }
    auto key_at = [&](uint32_t f) __attribute__((always_inline)) -> K {
        while (f >= s_end[run]) start = s_end[run++];
        return keys[s_first[run] + (f - start)];
    };
    uint32_t found = 0;
    if constexpr (SPARSE) {
        K k[kOwn];
        uint32_t p[kOwn];
#pragma unroll
        for (int u = 0; u < kOwn; ++u) {
            const uint32_t f = (uint32_t)tid + u * kBlock;
            k[u] = f < total ? key_at(f) : K(0);
        }
#pragma unroll
        for (int u = 0; u < kOwn; ++u) {
            p[u] = drop_axis24((uint32_t)k[u] & low, drop);
            if ((uint32_t)tid + u * kBlock < total) atomicOr(&s_bits[p[u] >> 5], 1u << (p[u] & 31u));
        }
        __syncthreads();
        uint32_t mine = 0;
#pragma unroll
        for (int b = 0; b < kBitsOwn; ++b) mine += (uint32_t)__popc(s_bits[tid * kBitsOwn + b]);
        uint32_t ex = block_excl_sum<kBlock>(mine, s_w, &found);
#pragma unroll
        for (int b = 0; b < kBitsOwn; ++b) {
            s_pre[tid * kBitsOwn + b] = ex;
            ex += (uint32_t)__popc(s_bits[tid * kBitsOwn + b]);
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kOwn; ++u)
            if ((uint32_t)tid + u * kBlock < total) {
                const uint32_t w = p[u] >> 5;
                const uint32_t r = s_pre[w] + (uint32_t)__popc(s_bits[w] & ((1u << (p[u] & 31u)) - 1u));
                atomicAdd(&s_px[r], 1u);
                s_code[r] = (uint16_t)p[u];
            }
        __syncthreads();
        for (uint32_t j = tid; j < found; j += kBlock) tmp[before + j] = ((uint32_t)s_code[j] << 16) | s_px[j];
    } else {
        bool over = false;
        for (uint32_t f0 = tid; f0 < total; f0 += kIn * kBlock) {
            K k[kIn];
#pragma unroll
            for (int u = 0; u < kIn; ++u) {
                const uint32_t f = f0 + u * kBlock;
                k[u] = f < total ? key_at(f) : K(0);
            }
#pragma unroll
            for (int u = 0; u < kIn; ++u) {
                if (f0 + u * kBlock >= total) continue;
                const uint32_t p = drop_axis24((uint32_t)k[u] & low, drop), sh = 16 * (p & 1u);
                if (total < 1u << 16) {
                    atomicAdd(&s_px[p >> 1], 1u << sh);
                } else {
                    const uint32_t was = atomicAdd(&s_px[p >> 1], 1u << sh);
                    over |= ((was >> sh) & 0xFFFFu) == 0xFFFFu;
                }
            }
        }
        if (over) set_err(err, kProjHeavy);
        __syncthreads();
        auto counter = [&](int i) __attribute__((always_inline)) -> uint32_t {
            return i < px ? (s_px[i >> 1] >> (16 * (i & 1))) & 0xFFFFu : 0u;
        };
        // rank of every occupied pixel: ballots per row of the block, one scan
        const int rows = (px + kBlock - 1) / kBlock;
#pragma unroll 4
        for (int r = 0; r < rows; ++r) {
            const uint64_t b = __ballot(counter(r * kBlock + tid) != 0);
            if (lane == 0) s_off[r * kWaves + wave] = (uint32_t)__popcll(b);
        }
        __syncthreads();
        const uint32_t mine = tid < rows * kWaves ? s_off[tid] : 0u;
        const uint32_t ex = block_excl_sum<kBlock>(mine, s_w, &found);
        if (tid < rows * kWaves) s_off[tid] = before + ex;
        __syncthreads();
#pragma unroll 4
        for (int r = 0; r < rows; ++r) {
            const int i = r * kBlock + tid;
            const uint32_t c = counter(i);
            const uint64_t b = __ballot(c != 0);
            // (a 16-bit overflow, which has the sort do the call over, can
            // leave fewer pixels than ranks but never a rank past the voxels)
            if (c) tmp[s_off[r * kWaves + wave] + (uint32_t)__popcll(b & lanemask_lt())] = ((uint32_t)i << 16) | c;
        }
    }
    if (tid == 0) {
        T.uniq[t] = found;
        T.from[t] = before;
    }
}

// Tiles' pixel counts to their places in the output (one block; at most
// 16384 tiles), and the total.
__global__ __launch_bounds__(1024) void k_proj_scan(TileTables T, uint32_t tiles, int64_t cap,
                                                    int64_t *n_out, uint32_t *err) {
    constexpr int kPer = 16;
    __shared__ uint32_t s_w[16];
    __shared__ uint32_t s_u[1024 * (kPer + 1)];  // a thread's 16, off by one against bank conflicts
    if (*err & kProjRedo) return;  // block-uniform
    const int tid = threadIdx.x;
#pragma unroll
    for (int r = 0; r < kPer; ++r) {
        const uint32_t i = r * 1024 + tid;
        s_u[i + i / kPer] = i < tiles ? T.uniq[i] : 0u;
    }
    __syncthreads();
    uint32_t sum = 0, *own = s_u + tid * (kPer + 1);
#pragma unroll
    for (int j = 0; j < kPer; ++j) sum += own[j];
    uint32_t total, at = block_excl_sum<1024>(sum, s_w, &total);
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const uint32_t u = own[j];
        own[j] = at;
        at += u;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kPer; ++r) {
        const uint32_t i = r * 1024 + tid;
        if (i < tiles) T.uniq[i] = s_u[i + i / kPer];
    }
    if (tid == 0) {
        *n_out = total;
        if ((int64_t)total > cap) set_err(err, ERR_CAPACITY);
    }
}

// Every tile's pixels from tmp to their place in the output.
__global__ __launch_bounds__(256) void k_proj_gather(TileTables T, uint32_t tiles, uint32_t L,
                                                     const int64_t *__restrict__ n_out,
                                                     const uint32_t *__restrict__ tmp,
                                                     uint32_t *__restrict__ out,
                                                     uint32_t *__restrict__ counts, int64_t cap,
                                                     const uint32_t *err) {
    constexpr int kIn = 4;
    if (*err & kProjRedo) return;
    const uint32_t t = blockIdx.x, to = T.uniq[t];
    uint32_t end = t + 1 < tiles ? T.uniq[t + 1] : (uint32_t)*n_out;
    if ((int64_t)end > cap) end = (uint32_t)cap;
    if (end <= to) return;
    const uint32_t *src = tmp + T.from[t] - to;  // indexed by output place
    const uint32_t high = t << (2 * L);
    for (uint32_t i0 = to + threadIdx.x; i0 < end; i0 += kIn * 256) {
        uint32_t w[kIn];
#pragma unroll
        for (int u = 0; u < kIn; ++u) w[u] = i0 + u * 256 < end ? src[i0 + u * 256] : 0u;
#pragma unroll
        for (int u = 0; u < kIn; ++u) {
            const uint32_t i = i0 + u * 256;
            if (i < end) {
                out[i] = high | (w[u] >> 16);
                if (counts) counts[i] = w[u] & 0xFFFFu;
            }
        }
    }
}

// Where a call does not wait for its results, the sort follows the tiles in
// the stream and does nothing unless they gave up: its count is zero.  This
// sets it, and clears what the sort needs cleared.
__global__ __launch_bounds__(256) void k_proj_redo(int64_t n_host, const int64_t *d_n,
                                                   const uint32_t *err, int64_t *n_redo,
                                                   uint32_t *tile_ctr, uint4 *z0, size_t z0_n,
                                                   uint4 *z1, size_t z1_n) {
    const bool redo = (*err & kProjRedo) != 0;
    const size_t tid = (size_t)blockIdx.x * 256 + threadIdx.x, stride = (size_t)gridDim.x * 256;
    if (tid == 0) *n_redo = redo ? dev_count(n_host, d_n) : 0;
    if (!redo) return;
    if (tid <= (size_t)kMaxPasses) tile_ctr[tid] = 0;
    for (size_t i = tid; i < z0_n; i += stride) z0[i] = make_uint4(0, 0, 0, 0);
    for (size_t i = tid; i < z1_n; i += stride) z1[i] = make_uint4(0, 0, 0, 0);
}

struct ProjLayout {
    Control *ctl;
    SortWs sort;
    uint64_t *rle_status;
    void *buf_a, *buf_b;
    TileTables tiles{};
    size_t tile_bytes = 0;  // of the tables to clear, contiguous from tiles.cells
    size_t sort_bytes;      // what the sort alone needs
    size_t bytes;
};

static bool proj_by_tiles(const cga_grid *g) {
    return g->key_mode == CGA_KEY_MORTON && g->depth <= kTileDepthMax;
}
static uint32_t proj_tiles(uint32_t depth) { return 1u << (2 * (depth - tile_level(depth))); }

static ProjLayout proj_layout(void *ws, const cga_grid *g, int64_t n, const SortCfg &cfg) {
    ProjLayout L;
    Carve c(ws);
    const size_t kb = wide_keys2(g->depth) ? 8 : 4;
    L.ctl = c.take<Control>(1);
    sort_carve(c, L.sort, n, 2 * (int)g->depth, cfg);
    L.rle_status = c.take<uint64_t>((size_t)rle_status_words(n));
    L.buf_a = c.take<char>((size_t)(n > 0 ? n : 1) * kb);
    L.buf_b = c.take<char>((size_t)(n > 0 ? n : 1) * kb);
    L.sort_bytes = c.size();
    if (proj_by_tiles(g)) {
        const uint32_t lev = tile_level(g->depth), tiles = proj_tiles(g->depth);
        L.tiles.cells = c.take<uint2>((size_t)tiles << (g->depth - lev));
        L.tiles.uniq = c.take<uint32_t>(tiles);  // cleared with the cells: empty tiles leave it
        L.tile_bytes = (size_t)((char *)(L.tiles.uniq + tiles) - (char *)L.tiles.cells);
        L.tiles.from = c.take<uint32_t>(tiles);
        L.tiles.tot = c.take<uint32_t>(tiles);
        L.tiles.gtot = c.take<uint32_t>(tiles / kTileGroup + 1);
    }
    L.bytes = c.size();
    return L;
}

template <typename K, typename K2>
static void project_enqueue(const cga_grid *g, const K *keys, int64_t n, const int64_t *d_n,
                            int drop, K2 *out, uint32_t *counts, int64_t cap, int64_t *n_out,
                            const ProjLayout &L, hipStream_t s) {
    const uint32_t d = g->depth;
    if (g->key_mode == CGA_KEY_LINEAR && drop == 2) {
        // (x<<2d | y<<d | z) >> d = x<<d | y: already ascending, just collapse
        CGA_PROF("rle", s);
        rle_launch<K, K2, false>(keys, n, d_n, (int)d, ~0ull, out, counts, nullptr, cap, n_out, L.rle_status,
            &L.ctl->tile_ctr[kMaxPasses], &L.ctl->err, s);
        return;
    }
    const SortWs &w = L.sort;
    K2 *a = (K2 *)L.buf_a, *b = (K2 *)L.buf_b;
    rekey_dispatch<K, K2>(w.radix_bits, keys, n, d_n, g, drop, a, w.passes, w.hist, s);
    K2 *fin = (w.passes & 1) ? b : a;
    K2 *other = (w.passes & 1) ? a : b;
    sort_launch<K2>(w, a, fin, other, fin, n, d_n, true, L.ctl->tile_ctr, s);
    CGA_PROF("rle", s);
    rle_launch<K2, K2, false>(fin, n, d_n, 0, ~0ull, out, counts, nullptr, cap, n_out, L.rle_status,
        &L.ctl->tile_ctr[kMaxPasses], &L.ctl->err, s);
}

template <typename K>
static void project_tiles_enqueue(const cga_grid *g, const K *keys, int64_t n, const int64_t *d_n,
                                  int drop, uint32_t *out, uint32_t *counts, int64_t cap,
                                  int64_t *n_out, const ProjLayout &L, hipStream_t s) {
    const uint32_t lev = tile_level(g->depth), tiles = proj_tiles(g->depth);
    uint32_t *tmp = (uint32_t *)L.buf_a;
    int64_t blocks = (n + 1023) / 1024;
    blocks = blocks > 8192 ? 8192 : blocks;
    {
        CGA_PROF("rekey", s);
        k_proj_cells<K><<<(unsigned)blocks, 256, 0, s>>>(keys, n, d_n, g->depth, lev, drop, L.tiles,
                                                         &L.ctl->err);
    }
    {
        CGA_PROF("project_tiles", s);
        k_proj_totals<<<(tiles + kTileGroup - 1) / kTileGroup, 256, 0, s>>>(L.tiles, tiles,
                                                                            1u << (g->depth - lev));
        auto launch = [&](auto kernel, int block) {
            kernel<<<tiles, block, 0, s>>>(keys, g->depth, lev, drop, L.tiles, tmp, &L.ctl->err);
        };
        if (lev <= 4) {
            launch(k_proj_tiles<K, 4>, tile_block<4, false>());
        } else if (lev == 5) {
            launch(k_proj_tiles<K, 5>, tile_block<5, false>());
        } else if (lev == 6) {
            launch(k_proj_tiles<K, 6>, tile_block<6, false>());
        } else {
            launch(k_proj_tiles<K, 7, true>, tile_block<7, true>());
            launch(k_proj_tiles<K, 7>, tile_block<7, false>());
        }
        k_proj_scan<<<1, 1024, 0, s>>>(L.tiles, tiles, cap, n_out, &L.ctl->err);
        k_proj_gather<<<tiles, 256, 0, s>>>(L.tiles, tiles, lev, n_out, tmp, out, counts, cap,
                                            &L.ctl->err);
    }
}

template <typename K>
static void project_any(const cga_grid *g, const void *keys, int64_t n, const int64_t *d_n, int drop,
                        void *out, uint32_t *counts, int64_t cap, int64_t *n_out,
                        const ProjLayout &L, hipStream_t s) {
    if (wide_keys2(g->depth))
        project_enqueue<K, uint64_t>(g, (const K *)keys, n, d_n, drop, (uint64_t *)out, counts, cap,
                                     n_out, L, s);
    else
        project_enqueue<K, uint32_t>(g, (const K *)keys, n, d_n, drop, (uint32_t *)out, counts, cap,
                                     n_out, L, s);
}

}  // namespace cga

using namespace cga;

extern "C" {

size_t cga_project_workspace_bytes(const cga_grid *g, int64_t n) {
    if (!grid_valid(g) || n < 0) return 0;
    size_t m = 0;
    for (int rb = 4; rb <= 11; ++rb)
        for (int items : kSortItems) {
            SortCfg c;
            c.radix_bits = rb;
            c.items = items;
            size_t b = proj_layout(nullptr, g, n, c).bytes;
            m = b > m ? b : m;
        }
    return m;
}

int cga_project(const cga_grid *g, const void *d_keys, int64_t n, const int64_t *d_n,
                int drop_axis, void *d_out2d, uint32_t *d_counts, int64_t cap, int64_t *d_n_out,
                int64_t *n_out_host, void *d_ws, size_t ws_bytes, const cga_tune *tune,
                cga_stream stream) {
    if (!grid_valid(g) || n < 0 || cap < 0 || !d_ws) return CGA_EINVAL;
    if (drop_axis < 0 || drop_axis > 2) return CGA_EINVAL;
    if (n > 0 && (!d_keys || !d_out2d)) return CGA_EINVAL;
    if (n >= (int64_t)1 << 30) return CGA_EUNSUPPORTED;
    const bool wide2 = wide_keys2(g->depth);
    SortCfg cfg = default_sort_cfg(wide2, n, 2 * (int)g->depth);
    if (!tune) tuned_sort_cfg(wide2 ? 8 : 4, 2 * (int)g->depth, n, &cfg);
    if (tune) {
        cfg.radix_bits = (int)tune->radix_bits;
        cfg.items = (int)tune->tile_items;
        if (!sort_cfg_supported(cfg)) return CGA_EINVAL;
    }
    ProjLayout L = proj_layout(d_ws, g, n, cfg);
    if (ws_bytes < L.sort_bytes) return CGA_EWORKSPACE;
    hipStream_t s = (hipStream_t)stream;
    int64_t *cnt_out = d_n_out ? d_n_out : &L.ctl->count;
    // A caller that names a sort setting, or whose workspace holds the sort
    // but not the tile tables, gets the sort.  So does one that does not wait
    // and has few voxels to a tile: the sort's launches then follow
    // the tiles' (k_proj_redo), about 15 us whatever the size, and the tiles'
    // own share does not shrink with the voxels (up to 400k at depth 14 the
    // pair is 6 % slower than the sort alone; 3M 1.4x as fast).
    const bool wide = wide_keys(g->depth);
    const bool tiles = !tune && n > 0 && proj_by_tiles(g) && ws_bytes >= L.bytes &&
                       (n_out_host || n >= (int64_t)proj_tiles(g->depth) * 64);
    auto sort_way = [&](const int64_t *count) {
        if (wide)
            project_any<uint64_t>(g, d_keys, n, count, drop_axis, d_out2d, d_counts, cap, cnt_out, L, s);
        else
            project_any<uint32_t>(g, d_keys, n, count, drop_axis, d_out2d, d_counts, cap, cnt_out, L, s);
    };
    if (tiles) {
        CGA_TRY(launch_begin(L.ctl, L.tiles.cells, L.tile_bytes, nullptr, 0, cnt_out, s));
        if (wide)
            project_tiles_enqueue<uint64_t>(g, (const uint64_t *)d_keys, n, d_n, drop_axis,
                                            (uint32_t *)d_out2d, d_counts, cap, cnt_out, L, s);
        else
            project_tiles_enqueue<uint32_t>(g, (const uint32_t *)d_keys, n, d_n, drop_axis,
                                            (uint32_t *)d_out2d, d_counts, cap, cnt_out, L, s);
        if (n_out_host) {  // the caller waits anyway: look whether the tiles did it
            uint32_t bits = 0;
            const int st = finish_counts(L.ctl, s, cnt_out, n_out_host, nullptr, nullptr, &bits);
            if (st == CGA_EHIP || !(bits & kProjRedo)) return st;
        } else {
            const size_t z0 = (sort_zero_bytes(L.sort) + 15) / 16, z1 = ((size_t)rle_tiles(n) * 8 + 15) / 16;
            const unsigned blocks = (unsigned)(z0 / 256 < 1 ? 1 : (z0 / 256 > 1024 ? 1024 : z0 / 256));
            k_proj_redo<<<blocks, 256, 0, s>>>(n, d_n, &L.ctl->err, &L.ctl->count2, L.ctl->tile_ctr,
                                               (uint4 *)L.sort.hist, z0, (uint4 *)L.rle_status, z1);
            sort_way(&L.ctl->count2);
            CGA_HIP(hipGetLastError());
            return CGA_OK;
        }
    }
    CGA_TRY(launch_begin(L.ctl, L.sort.hist, sort_zero_bytes(L.sort), L.rle_status,
                         (size_t)rle_tiles(n) * 8, cnt_out, s));
    if (n > 0) {
        sort_way(d_n);
        CGA_HIP(hipGetLastError());
    }
    return n_out_host ? finish_counts(L.ctl, s, cnt_out, n_out_host) : CGA_OK;
}

}  // extern "C"

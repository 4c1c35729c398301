// Dispatch layouts: counts, offsets and packed rows of the per-pair and the
// node-deduplicated layout. A pair p goes to row
//     offsets[s][r] + (pairs before p with its source s and destination r),
// a token to one such row per destination node. Every scheme splits the call
// into tiles, counts each tile's items per destination, and lets the tile's
// workgroup rank its own items by ballots; none waits for another workgroup
// inside a kernel. What bounds all of them is latency: launches, dependent
// loads and barriers. They differ in how a workgroup learns its first rows.
// Times are layout-only calls, per pair | per node, in us (the chain of
// clear, count, one-workgroup scan and look-back that they replace in
// brackets):
//
//   per-source tiles (sources in equal blocks; two kernels). Tiles never
//     cross a source, so a workgroup needs the counts of its source's tiles
//     (a few rows) and the sums of all earlier tiles (at most about 1500
//     words), which the first kernel leaves in the workspace. T=131072, K=8,
//     8 x 8 ranks: 11.4 | 12.8 us of kernels (31 | 36); 32768 pairs on 4 x 8:
//     8.1 | 7.4 (16.6 | 18.5).
//   any sources (clear, count, rank, and the scan in between for tables over
//     kSmallTable). The counts per bucket come from atomic adds on a window
//     of sources per tile, the earlier tiles of a destination from the
//     tiles' counts; each workgroup turns the counts into first rows itself.
//     65536 pairs on 4 x 8: 14.8 | 13.4 (16.4 | 18.9). With the scan in
//     between, 131072 tokens, K = 8: 8 x 16 ranks 41.5 | 20.0 (43.8 | 34.1),
//     16 x 16 175 | 30.2 (171 | 48.6), 16 x 32 559 | 44.6 (571 | 59.8); the
//     scan's workgroup takes most of it (equal blocks, which need none: 10.0 |
//     10.6, 10.8 | 15.1, 16.1 | 16.5).
//   whole-call workgroups (small calls; one kernel). Every workgroup counts
//     all items of the call in its LDS, which costs less than another launch
//     up to a limit: 2048 pairs on 4 x 8 take 5.5 | 5.9 (13.2 | 15.3). Equal
//     blocks: 8192 pairs 6.9 us against 8.0 for per-source tiles, 16384 8.3
//     to 9.8 against 8.2; 1024 tokens 6 to 10 us against 7.2 to 8, 2048 7 to
//     15 against 7.3. Sources given: 24576 pairs 10.5 to 12.2 us against 14
//     to 17, 49152 15.4 to 19.5 against 14.1 to 17; 4096 tokens 8.6 to 17.6
//     against 11 to 16.7, 8192 12 to 19 against 12 to 16.4. With few ranks
//     the pairs' LDS atomics queue on few words, in every workgroup for all
//     pairs, and the limit is lower (small_pairs): 24576 pairs on 1, 2, 3, 4,
//     6 and 8 ranks take 26.2, 21.0, 17.4, 15.6, 14.0 and 12.4 us against
//     11.6, 14.1, 13.7, 13.3, 13.3 and 13.2.
#include <algorithm>
#include <type_traits>

#include "internal.hpp"

namespace cobalt {
namespace {

constexpr int kThreads = 1024;
constexpr int kWaves = kThreads / 64;
constexpr int kChunks = 4;                         // pairs per thread and pass of a tile
constexpr int64_t kPass = (int64_t)kThreads * kChunks;
constexpr int kNodeThreads = 512;
constexpr int kNodeWaves = kNodeThreads / 64;
constexpr int64_t kMaxTiles = 1024;                // beside one per source
constexpr int kSmallG = 64;
constexpr int64_t kSmallPairs = 8192;              // most pairs of a whole-call workgroup
constexpr int64_t kSmallPairsAny = 32768;          // the same with source ranks given
constexpr int64_t kSmallTokens = 1024;             // most tokens, node-deduplicated
constexpr int64_t kSmallTokensAny = 4096;
constexpr int kSmallTable = kSmallG * kSmallG;     // counts a workgroup turns into rows itself
constexpr int kWindow = 8192;                      // counts of a tile's window over its sources
constexpr int64_t kMaxAnyTiles = 256;
constexpr int kScanThreads = 1024;
constexpr int kScanLds = 16384;                    // counts staged in LDS (G <= 128)
constexpr int64_t kPairsPerWord = 4096;            // of the workspace, per destination
constexpr int64_t kTokensPerWord = 512;            // of the workspace, per node

// Tiles of equal source blocks: each source's `per_src` items in tiles of
// `tile`, a multiple of `unit` that keeps the tiles to kMaxTiles and one per
// source.
struct Tiles {
    int64_t tile;
    int per_src;
};
Tiles make_tiles(int64_t items_per_src, int G, int64_t unit) {
    const int64_t total = items_per_src * G;
    const int64_t m = std::max<int64_t>(1, (total + unit * kMaxTiles - 1) / (unit * kMaxTiles));
    return {unit * m, (int)((items_per_src + unit * m - 1) / (unit * m))};
}

// Sum over the workgroup, added to *out (LDS, cleared before).
__device__ __forceinline__ void block_add(uint32_t v, uint32_t* out) {
#pragma unroll
    for (int o = 32; o; o >>= 1) v += __shfl_xor(v, o, 64);
    if ((threadIdx.x & 63) == 0 && v) atomicAdd(out, v);
}

// Exclusive scan over the workgroup of kThreads threads.
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t v, uint32_t* wsum,
                                                         uint32_t* total) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t x = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
    }
    if (lane == 63) wsum[wave] = x;
    __syncthreads();
    uint32_t before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        before += w < wave ? wsum[w] : 0u;
        all += wsum[w];
    }
    *total = all;
    return before + x - v;
}

// Rank of the lane's pair among the wave's earlier pairs with destination r:
// the lanes that agree on every bit of r share it; cnt[r] counts the wave's
// pairs so far.
__device__ __forceinline__ int wave_rank(bool valid, int r, int bits, uint32_t* cnt) {
    const uint64_t below = (1ull << (threadIdx.x & 63)) - 1ull;
    uint64_t peers = __ballot(valid);
    for (int b = 0; b < bits; ++b) {
        const bool bit = valid && ((r >> b) & 1);
        const uint64_t bal = __ballot(bit);
        peers &= bit ? bal : ~bal;
    }
    int prior = 0;
    if (valid) prior = (int)cnt[r];
    if (valid && (peers & below) == 0) cnt[r] = prior + __popcll(peers);
    return prior + __popcll(peers & below);
}

__device__ __forceinline__ int bits_for(int n) { return n > 1 ? 32 - __builtin_clz(n - 1) : 0; }

// ------------------------------------------------------- per-source tiles
__global__ __launch_bounds__(kThreads) void tile_count_kernel(
    const int32_t* __restrict__ assigned, int G, int64_t per_src, int64_t tile, int tiles,
    uint32_t* __restrict__ hist, uint32_t* __restrict__ sums) {
    __shared__ uint32_t h[kMaxG];
    __shared__ uint32_t sum;
    const int s = blockIdx.x / tiles, q = blockIdx.x - s * tiles;
    const int64_t p0 = s * per_src + q * tile;
    const int64_t p1 = min(p0 + tile, (s + 1) * per_src);
    for (int r = threadIdx.x; r < G; r += kThreads) h[r] = 0;
    if (threadIdx.x == 0) sum = 0;
    __syncthreads();
    uint32_t n = 0;
    for (int64_t p = p0 + threadIdx.x; p < p1; p += kPass) {
        int r[kChunks];
#pragma unroll
        for (int c = 0; c < kChunks; ++c)
            r[c] = p + c * kThreads < p1 ? assigned[p + c * kThreads] : -1;
#pragma unroll
        for (int c = 0; c < kChunks; ++c)
            if ((uint32_t)r[c] < (uint32_t)G) {
                atomicAdd(&h[r[c]], 1u);
                ++n;
            }
    }
    block_add(n, &sum);
    __syncthreads();
    for (int r = threadIdx.x; r < G; r += kThreads) hist[(int64_t)blockIdx.x * G + r] = h[r];
    if (threadIdx.x == 0) sums[blockIdx.x] = sum;
}

__global__ __launch_bounds__(kThreads) void tile_rank_kernel(
    const int32_t* __restrict__ assigned, int G, int64_t per_src, int64_t tile, int tiles,
    const uint32_t* __restrict__ hist, const uint32_t* __restrict__ sums,
    int32_t* __restrict__ counts, int64_t* __restrict__ offsets, int32_t* __restrict__ pos) {
    __shared__ uint32_t wcnt[kWaves][kMaxG];  // the waves' counts, then their first rows
    __shared__ uint32_t own[kMaxG], prior[kMaxG], next[kMaxG];
    __shared__ uint32_t placed;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int s = blockIdx.x / tiles, q = blockIdx.x - s * tiles;
    const int64_t p0 = s * per_src + q * tile;
    const int64_t p1 = min(p0 + tile, (s + 1) * per_src);
    const int bits = bits_for(G);
    const int64_t off = (int64_t)wave * 64 * kChunks + lane;
    int r[kChunks];
#pragma unroll
    for (int c = 0; c < kChunks; ++c)
        r[c] = p0 + off + c * 64 < p1 ? assigned[p0 + off + c * 64] : -1;

    for (int i = threadIdx.x; i < G; i += kThreads) own[i] = prior[i] = 0;
    if (threadIdx.x == 0) placed = 0;
    for (int i = lane; i < G; i += 64) wcnt[wave][i] = 0;
    __syncthreads();
    uint32_t before = 0;
    for (int i = threadIdx.x; i < s * tiles; i += kThreads) before += sums[i];
    // destination col of every ngrp-th tile of the source
    const int lg = max(6, bits), col = threadIdx.x & ((1 << lg) - 1), ngrp = kThreads >> lg;
    if (col < G) {
        uint32_t all = 0, earlier = 0;
        for (int i = threadIdx.x >> lg; i < tiles; i += ngrp) {
            const uint32_t v = hist[((int64_t)s * tiles + i) * G + col];
            all += v;
            earlier += i < q ? v : 0u;
        }
        if (all) atomicAdd(&own[col], all);
        if (earlier) atomicAdd(&prior[col], earlier);
    }
    block_add(before, &placed);
    __syncthreads();
    if (wave == 0) {  // offsets of the source's buckets; the tile's first row in each
        uint32_t run = placed;
        for (int i = lane; i - lane < G; i += 64) {
            const uint32_t v = i < G ? own[i] : 0u;
            uint32_t x = v;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const uint32_t y = __shfl_up(x, o, 64);
                if (lane >= o) x += y;
            }
            if (i < G) {
                next[i] = run + x - v + prior[i];
                if (q == 0) {
                    counts[(int64_t)s * G + i] = (int32_t)v;
                    offsets[(int64_t)s * G + i] = run + x - v;
                }
            }
            run += __shfl(x, 63, 64);
        }
        if (q == 0 && s == G - 1 && lane == 0) offsets[(int64_t)G * G] = run;
    }
    for (int64_t p = p0;;) {
        int rank[kChunks];
#pragma unroll
        for (int c = 0; c < kChunks; ++c) {
            const bool valid = (uint32_t)r[c] < (uint32_t)G;
            rank[c] = wave_rank(valid, r[c], bits, wcnt[wave]);
            r[c] = valid ? r[c] : -1;
        }
        __syncthreads();
        for (int i = threadIdx.x; i < G; i += kThreads) {
            uint32_t run = next[i];
#pragma unroll
            for (int w = 0; w < kWaves; ++w) {
                const uint32_t v = wcnt[w][i];
                wcnt[w][i] = run;
                run += v;
            }
            next[i] = run;
        }
        __syncthreads();
#pragma unroll
        for (int c = 0; c < kChunks; ++c) {
            const int64_t at = p + off + c * 64;
            if (at < p1) pos[at] = r[c] < 0 ? -1 : (int)wcnt[wave][r[c]] + rank[c];
        }
        p += kPass;
        if (p >= p1) break;
        // the wave's own row of wcnt: no other wave reads it before the next barrier
        for (int i = lane; i < G; i += 64) wcnt[wave][i] = 0;
#pragma unroll
        for (int c = 0; c < kChunks; ++c)
            r[c] = p + off + c * 64 < p1 ? assigned[p + off + c * 64] : -1;
    }
}

// --------------------------------------------------- whole-call workgroups
// Turns the counts in table[R][C] into first rows: the offset of each bucket
// in row-major order, less its column's count in the rows above, plus
// prior[c]. With `write`, also writes the offsets, and the counts if asked
// for.
__device__ __forceinline__ void first_rows(uint32_t* table, uint32_t* rows, const uint32_t* prior,
                                           int R, int C, uint32_t* wsum, bool write,
                                           int32_t* __restrict__ counts,
                                           int64_t* __restrict__ offsets) {
    constexpr int kSeg = kSmallTable / kThreads;
    const int n = R * C, b0 = threadIdx.x * kSeg;
    uint32_t v[kSeg], local = 0;
#pragma unroll
    for (int i = 0; i < kSeg; ++i) {
        v[i] = b0 + i < n ? table[b0 + i] : 0u;
        local += v[i];
    }
    uint32_t total = 0;
    uint32_t run = block_exclusive_scan(local, wsum, &total);
#pragma unroll
    for (int i = 0; i < kSeg; ++i) {
        if (b0 + i < n) {
            rows[b0 + i] = run;
            if (write) {
                if (counts) counts[b0 + i] = (int32_t)v[i];
                offsets[b0 + i] = run;
            }
            run += v[i];
        }
    }
    if (write && threadIdx.x == 0) offsets[n] = total;
    __syncthreads();
    if (threadIdx.x < C) {
        uint32_t shift = prior[threadIdx.x];
#pragma unroll 8
        for (int r = 0; r < R; ++r) {
            const int b = r * C + threadIdx.x;
            rows[b] += shift;
            shift -= table[b];
        }
    }
}

__global__ __launch_bounds__(kThreads) void small_layout_kernel(
    const int32_t* __restrict__ assigned, const int32_t* __restrict__ src, int TK, int G,
    SmallDiv by_k, SmallDiv by_src, int32_t* __restrict__ counts, int64_t* __restrict__ offsets,
    int32_t* __restrict__ pos) {
    __shared__ uint32_t table[kSmallTable], rows[kSmallTable];
    __shared__ uint32_t wcnt[kWaves][kSmallG];
    __shared__ uint32_t prior[kSmallG], wsum[kWaves];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    // bucket of pair p, -1 for one with no valid rank or source
    auto bucket = [&](int p) {
        if (p >= TK) return -1;
        const int r = assigned[p];
        const int s = src ? src[by_k(p)] : by_src(p);
        return (uint32_t)r < (uint32_t)G && (uint32_t)s < (uint32_t)G ? s * G + r : -1;
    };
    auto count = [&](int p0, int p1) {  // pairs [p0, p1), both multiples of kThreads
        for (int p = p0 + threadIdx.x; p < p1; p += 4 * kThreads) {
            int b[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) b[c] = p + c * kThreads < p1 ? bucket(p + c * kThreads) : -1;
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (b[c] >= 0) atomicAdd(&table[b[c]], 1u);
        }
    };
    for (int i = threadIdx.x; i < G * G; i += kThreads) table[i] = 0;
    wcnt[wave][lane] = 0;
    if (threadIdx.x < kSmallG) prior[threadIdx.x] = 0;
    __syncthreads();
    const int tile0 = blockIdx.x * kThreads;
    const int mine = tile0 + threadIdx.x;
    const int b = bucket(mine);
    count(0, tile0);
    __syncthreads();
    if (tile0 > 0 && lane < G) {  // pairs before the tile, per destination
        uint32_t v = 0;
        for (int s = wave; s < G; s += kWaves) v += table[s * G + lane];
        if (v) atomicAdd(&prior[lane], v);
    }
    const int r = b >= 0 ? b % G : 0;
    const int rank = wave_rank(b >= 0, r, bits_for(G), wcnt[wave]);
    __syncthreads();
    count(tile0, (TK + kThreads - 1) / kThreads * kThreads);
    if (wave == 1 && lane < G) {
        uint32_t run = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            const uint32_t v = wcnt[w][lane];
            wcnt[w][lane] = run;
            run += v;
        }
    }
    __syncthreads();
    first_rows(table, rows, prior, G, G, wsum, blockIdx.x == 0, counts, offsets);
    __syncthreads();
    if (mine < TK) pos[mine] = b < 0 ? -1 : (int)(rows[b] + wcnt[wave][r]) + rank;
}

// ---------------------------------------------------------- any sources
__global__ __launch_bounds__(256) void clear_kernel(int32_t* __restrict__ counts, int n) {
    for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) counts[i] = 0;
}

// The window of a tile whose first and last items have sources lo and hi:
// the table rows it counts in LDS, 0 if it does not fit or they are invalid.
__device__ __forceinline__ int window_rows(int lo, int hi, int G, int C) {
    return lo >= 0 && hi < G && hi >= lo && (hi - lo + 1) * C <= kWindow ? hi - lo + 1 : 0;
}

// Adds the tile's counts in the window to counts and to the tile's column
// counts h, and stores h as the tile's row of hist.
__device__ __forceinline__ void flush_window(const uint32_t* window, uint32_t* h, int rows, int lo,
                                             int C, int32_t* __restrict__ counts,
                                             uint32_t* __restrict__ hist) {
    __syncthreads();
    const int ngrp = blockDim.x / C > 0 ? blockDim.x / C : 1;
    const int grp = threadIdx.x / C, col = threadIdx.x - grp * C;
    if (grp < ngrp) {
        uint32_t all = 0;
        for (int w = grp; w < rows; w += ngrp) {
            const uint32_t v = window[w * C + col];
            if (v) atomicAdd(&counts[(int64_t)(lo + w) * C + col], (int32_t)v);
            all += v;
        }
        if (all) atomicAdd(&h[col], all);
    }
    __syncthreads();
    for (int c = threadIdx.x; c < C; c += blockDim.x) hist[(int64_t)blockIdx.x * C + c] = h[c];
}

// Pairs [p, p + kPass) of a pass, one call per chunk: bucket s * G + r, or -1.
struct PairSource {
    const int32_t* assigned;
    const int32_t* src;
    int64_t token;  // of the pass's first pair
    int slot;
    SmallDiv by_k;
    int G;
    __device__ __forceinline__ int operator()(int64_t p, int i) const {
        const int r = assigned[p + i];
        const int s = src[token + by_k(slot + i)];
        return (uint32_t)r < (uint32_t)G && (uint32_t)s < (uint32_t)G ? s * G + r : -1;
    }
};
__device__ __forceinline__ PairSource pair_source(const int32_t* assigned, const int32_t* src,
                                                  int64_t p, int K, SmallDiv by_k, int G) {
    const uint32_t t = (uint32_t)p / (uint32_t)K;
    return {assigned, src, t, (int)((uint32_t)p - t * (uint32_t)K), by_k, G};
}

__global__ __launch_bounds__(kThreads) void any_count_kernel(
    const int32_t* __restrict__ assigned, const int32_t* __restrict__ src, int64_t TK, int K,
    SmallDiv by_k, int G, int64_t tile, int32_t* __restrict__ counts,
    uint32_t* __restrict__ hist) {
    __shared__ uint32_t window[kWindow];
    __shared__ uint32_t h[kMaxG];
    const int64_t p0 = blockIdx.x * tile, p1 = min(p0 + tile, TK);
    const int first = src[p0 / K], rows = window_rows(first, src[(p1 - 1) / K], G, G);
    const int lo = rows ? first : 0;
    for (int i = threadIdx.x; i < rows * G; i += kThreads) window[i] = 0;
    for (int r = threadIdx.x; r < G; r += kThreads) h[r] = 0;
    __syncthreads();
    for (int64_t p = p0; p < p1; p += kPass) {
        const PairSource bucket = pair_source(assigned, src, p, K, by_k, G);
        int b[kChunks];
#pragma unroll
        for (int c = 0; c < kChunks; ++c) {
            const int i = c * kThreads + threadIdx.x;
            b[c] = p + i < p1 ? bucket(p, i) : -1;
        }
#pragma unroll
        for (int c = 0; c < kChunks; ++c) {
            uint32_t n = 1;
            if (G == 1) {  // one bucket: the wave adds once (11.6 us for 32768 pairs, not 14.6)
                n = (uint32_t)__popcll(__ballot(b[c] >= 0));
                b[c] = (threadIdx.x & 63) == 0 && n ? 0 : -1;
            }
            if (b[c] < 0) continue;
            const int w = b[c] - lo * G;
            if (w >= 0 && w < rows * G) {
                atomicAdd(&window[w], n);
            } else {
                atomicAdd(&counts[b[c]], (int32_t)n);
                atomicAdd(&h[b[c] % G], n);
            }
        }
    }
    flush_window(window, h, rows, lo, G, counts, hist);
}

// GM: columns the LDS tables hold. With GM = kSmallG every workgroup turns
// the counts into first rows itself; else `base` holds them.
template <int GM>
__global__ __launch_bounds__(kThreads) void any_rank_kernel(
    const int32_t* __restrict__ assigned, const int32_t* __restrict__ src, int64_t TK, int K,
    SmallDiv by_k, int G, int64_t tile, const int32_t* __restrict__ counts,
    const uint32_t* __restrict__ hist, const int32_t* __restrict__ base,
    int64_t* __restrict__ offsets, int32_t* __restrict__ pos) {
    constexpr bool kTable = GM == kSmallG;
    __shared__ uint32_t table[kTable ? kSmallTable : 1], rows[kTable ? kSmallTable : 1];
    __shared__ uint32_t wcnt[kWaves][GM];
    __shared__ uint32_t prior[GM], wsum[kWaves];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t p0 = blockIdx.x * tile, p1 = min(p0 + tile, TK);
    const int bits = bits_for(G);
    const int off = wave * 64 * kChunks + lane;
    int b[kChunks];
    auto load = [&](int64_t p) {
        const PairSource bucket = pair_source(assigned, src, p, K, by_k, G);
#pragma unroll
        for (int c = 0; c < kChunks; ++c) b[c] = p + off + c * 64 < p1 ? bucket(p, off + c * 64) : -1;
    };
    load(p0);
    for (int i = threadIdx.x; i < G; i += kThreads) prior[i] = 0;
    for (int i = lane; i < G; i += 64) wcnt[wave][i] = 0;
    if constexpr (kTable)
        for (int i = threadIdx.x; i < G * G; i += kThreads) table[i] = (uint32_t)counts[i];
    __syncthreads();
    const int lg = max(6, bits), col = threadIdx.x & ((1 << lg) - 1), ngrp = kThreads >> lg;
    if (col < G) {
        uint32_t v = 0;
        for (int i = threadIdx.x >> lg; i < (int)blockIdx.x; i += ngrp) v += hist[(int64_t)i * G + col];
        if (v) atomicAdd(&prior[col], v);
    }
    __syncthreads();
    if constexpr (kTable) {
        first_rows(table, rows, prior, G, G, wsum, blockIdx.x == 0, nullptr, offsets);
        __syncthreads();
        if (threadIdx.x < G) prior[threadIdx.x] = 0;  // counted in rows
    }
    for (int64_t p = p0;;) {
        int rank[kChunks], r[kChunks];
#pragma unroll
        for (int c = 0; c < kChunks; ++c) {
            r[c] = b[c] >= 0 ? b[c] % G : 0;
            rank[c] = wave_rank(b[c] >= 0, r[c], bits, wcnt[wave]);
        }
        __syncthreads();
        for (int i = threadIdx.x; i < G; i += kThreads) {
            uint32_t run = prior[i];
#pragma unroll
            for (int w = 0; w < kWaves; ++w) {
                const uint32_t v = wcnt[w][i];
                wcnt[w][i] = run;
                run += v;
            }
            prior[i] = run;
        }
        __syncthreads();
#pragma unroll
        for (int c = 0; c < kChunks; ++c) {
            const int64_t at = p + off + c * 64;
            if (at >= p1) continue;
            int row = -1;
            if (b[c] >= 0)
                row = (kTable ? (int)rows[b[c]] : base[b[c]]) + (int)wcnt[wave][r[c]] + rank[c];
            pos[at] = row;
        }
        p += kPass;
        if (p >= p1) break;
        for (int i = lane; i < G; i += 64) wcnt[wave][i] = 0;
        load(p);
    }
}

// Exclusive scan of one value per thread across the workgroup.
__device__ int64_t block_exclusive_scan64(int64_t v, int64_t* total) {
    __shared__ int64_t wsum[kScanThreads / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int64_t x = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int64_t y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
    }
    if (lane == 63) wsum[wave] = x;
    __syncthreads();
    if (wave == 0) {
        int64_t w = lane < kScanThreads / 64 ? wsum[lane] : 0;
#pragma unroll
        for (int o = 1; o < kScanThreads / 64; o <<= 1) {
            const int64_t y = __shfl_up(w, o, 64);
            if (lane >= o) w += y;
        }
        if (lane < kScanThreads / 64) wsum[lane] = w;  // inclusive over waves
    }
    __syncthreads();
    const int64_t before = (wave > 0 ? wsum[wave - 1] : 0) + x - v;
    *total = wsum[kScanThreads / 64 - 1];
    return before;
}

// Exclusive scan of a [R][C] count matrix in row-major order, and
// base[s][c] = offsets[s][c] - sum_{s' < s} counts[s'][c]. With R*C <=
// kScanLds the counts and offsets are staged in LDS, so the sequential
// column pass reads LDS instead of global memory.
template <bool kLds>
__global__ __launch_bounds__(kScanThreads) void scan_kernel(const int32_t* __restrict__ counts,
                                                            int R, int C,
                                                            int64_t* __restrict__ offsets,
                                                            int32_t* __restrict__ base) {
    __shared__ int32_t c_lds[kLds ? kScanLds : 1];
    __shared__ int32_t o_lds[kLds ? kScanLds : 1];
    const int64_t n = (int64_t)R * C;
    if (kLds) {
        for (int64_t b = threadIdx.x; b < n; b += kScanThreads) c_lds[b] = counts[b];
        __syncthreads();
    }
    auto cnt = [&](int64_t b) -> int64_t { return kLds ? c_lds[b] : counts[b]; };
    const int64_t seg = (n + kScanThreads - 1) / kScanThreads;
    const int64_t lo = min(n, (int64_t)threadIdx.x * seg), hi = min(n, lo + seg);
    int64_t local = 0;
    for (int64_t b = lo; b < hi; ++b) local += cnt(b);
    int64_t total = 0;
    int64_t run = block_exclusive_scan64(local, &total);
    for (int64_t b = lo; b < hi; ++b) {
        offsets[b] = run;
        if (kLds) o_lds[b] = (int32_t)run;
        run += cnt(b);
    }
    if (threadIdx.x == 0) offsets[n] = total;
    __syncthreads();
    for (int c = threadIdx.x; c < C; c += kScanThreads) {
        int64_t col = 0;
        for (int r = 0; r < R; ++r) {
            const int64_t b = (int64_t)r * C + c;
            base[b] = (int32_t)((kLds ? (int64_t)o_lds[b] : offsets[b]) - col);
            col += cnt(b);
        }
    }
}

// ------------------------------------------------------ node-deduplicated
// Node set of token t: bit n set if some slot goes to a rank of node n;
// code[j] = (node << 8) | rank inside the node, or -1.
template <int KM, int VEC>
__device__ __forceinline__ uint32_t node_set(const int32_t* __restrict__ assigned, int64_t t, int K,
                                             int G, int g, SmallDiv by_g, int (&code)[KM]) {
    uint32_t B = 0;
    int r[KM];
#pragma unroll
    for (int j = 0; j < KM; ++j) r[j] = -1;
    load_row<KM, VEC>(assigned + t * K, K, r);
#pragma unroll
    for (int j = 0; j < KM; ++j) {
        const bool ok = (uint32_t)r[j] < (uint32_t)G;
        const int n = by_g(ok ? r[j] : 0);
        code[j] = ok ? (n << 8) | (r[j] - n * g) : -1;
        B |= ok ? 1u << n : 0u;
    }
    return B;
}

// Writes a token's rows: node_pos for every node, and the forwarding mask and
// token of each row. row(n, rank) is the row of node n for the lane with
// `rank` earlier lanes of its wave on n.
template <int KM, int NV, typename Row>
__device__ __forceinline__ void write_node_rows(uint32_t B, const int (&code)[KM], int64_t t, bool in,
                                                int N, int32_t* __restrict__ node_pos,
                                                uint32_t* __restrict__ fwd,
                                                int32_t* __restrict__ row_token, Row row) {
    const uint64_t below = (1ull << (threadIdx.x & 63)) - 1ull;
    int at[kMaxN];
#pragma unroll
    for (int n = 0; n < kMaxN; ++n) {
        at[n] = -1;
        if (n < N) {
            const bool bit = (B >> n) & 1u;
            const uint64_t bal = __ballot(bit);
            if (bit) {
                at[n] = row(n, __popcll(bal & below));
                uint32_t m = 0;
#pragma unroll
                for (int j = 0; j < KM; ++j) m |= (code[j] >> 8) == n ? 1u << (code[j] & 255) : 0u;
                fwd[at[n]] = m;
                if (row_token) row_token[at[n]] = (int32_t)t;
            }
        }
    }
    if (in) store_row<kMaxN, NV>(node_pos + t * N, N, at);
}

// Adds a wave's tokens (node sets B, sources s) to the counts of their
// buckets: by ballots where the tokens share their source, else one by one.
// add(s, n, count) is called with distinct buckets on distinct lanes.
template <typename Add>
__device__ __forceinline__ void count_nodes(uint32_t B, int s, int N, Add add) {
    const int lane = threadIdx.x & 63;
    const int s0 = __builtin_amdgcn_readfirstlane(s);
    if (__ballot(B != 0 && s != s0) == 0) {
        uint32_t mine = 0;
        for (int n = 0; n < N; ++n) {
            const uint32_t c = (uint32_t)__popcll(__ballot((B >> n) & 1u));
            mine = lane == n ? c : mine;
        }
        if (mine) add(s0, lane, mine);
    } else {
        for (uint32_t b = B; b; b &= b - 1u) add(s, __builtin_ctz(b), 1u);
    }
}

// Per-node counts of a wave's tokens, in seg[0..N).
__device__ __forceinline__ void wave_nodes(uint32_t B, int N, uint32_t* seg) {
    const int lane = threadIdx.x & 63;
    uint32_t mine = 0;
    for (int n = 0; n < N; ++n) {
        const uint32_t c = (uint32_t)__popcll(__ballot((B >> n) & 1u));
        mine = lane == n ? c : mine;
    }
    if (lane < N) seg[lane] = mine;
}

template <int KM, int VEC>
__global__ __launch_bounds__(kNodeThreads) void node_tile_count_kernel(
    const int32_t* __restrict__ assigned, int K, int N, int g, SmallDiv by_g, int64_t per_src,
    int64_t tile, int tiles, uint32_t* __restrict__ hist) {
    __shared__ uint32_t h[kMaxN];
    const int lane = threadIdx.x & 63;
    const int s = blockIdx.x / tiles, q = blockIdx.x - s * tiles;
    const int64_t t0 = s * per_src + q * tile;
    const int64_t t1 = min(t0 + tile, (s + 1) * per_src);
    if (threadIdx.x < kMaxN) h[threadIdx.x] = 0;
    __syncthreads();
    uint32_t mine = 0;  // lane n: the wave's tokens on node n
    for (int64_t t = t0 + threadIdx.x; t - threadIdx.x < t1; t += kNodeThreads) {
        int code[KM];
        const uint32_t B = t < t1 ? node_set<KM, VEC>(assigned, t, K, N * g, g, by_g, code) : 0u;
        for (int n = 0; n < N; ++n) {
            const uint32_t c = (uint32_t)__popcll(__ballot((B >> n) & 1u));
            mine += lane == n ? c : 0u;
        }
    }
    if (lane < N && mine) atomicAdd(&h[lane], mine);
    __syncthreads();
    if (threadIdx.x < N) hist[(int64_t)blockIdx.x * N + threadIdx.x] = h[threadIdx.x];
}

template <int KM, int VEC, int NV>
__global__ __launch_bounds__(kNodeThreads) void node_tile_rank_kernel(
    const int32_t* __restrict__ assigned, int K, int N, int g, SmallDiv by_g, int64_t per_src,
    int64_t tile, int tiles, const uint32_t* __restrict__ hist, int32_t* __restrict__ counts,
    int64_t* __restrict__ offsets, int32_t* __restrict__ node_pos, uint32_t* __restrict__ fwd,
    int32_t* __restrict__ row_token) {
    __shared__ uint32_t seg[kNodeWaves][kMaxN];  // the waves' counts, then their first rows
    __shared__ uint32_t own[kMaxN], prior[kMaxN], next[kMaxN];
    __shared__ uint32_t placed;
    const int wave = threadIdx.x >> 6;
    const int G = N * g;
    const int s = blockIdx.x / tiles, q = blockIdx.x - s * tiles;
    const int64_t t0 = s * per_src + q * tile;
    const int64_t t1 = min(t0 + tile, (s + 1) * per_src);
    int code[KM];
    int64_t t = t0 + threadIdx.x;
    uint32_t B = t < t1 ? node_set<KM, VEC>(assigned, t, K, G, g, by_g, code) : 0u;

    if (threadIdx.x < kMaxN) own[threadIdx.x] = prior[threadIdx.x] = 0;
    if (threadIdx.x == 0) placed = 0;
    __syncthreads();
    uint32_t before = 0;
    for (int i = threadIdx.x; i < s * tiles * N; i += kNodeThreads) before += hist[i];
    const int col = threadIdx.x & (kMaxN - 1);
    if (col < N) {
        uint32_t all = 0, earlier = 0;
        for (int i = threadIdx.x / kMaxN; i < tiles; i += kNodeThreads / kMaxN) {
            const uint32_t v = hist[((int64_t)s * tiles + i) * N + col];
            all += v;
            earlier += i < q ? v : 0u;
        }
        if (all) atomicAdd(&own[col], all);
        if (earlier) atomicAdd(&prior[col], earlier);
    }
    block_add(before, &placed);
    __syncthreads();
    if (threadIdx.x < N) {
        uint32_t run = placed;
        for (int n = 0; n < (int)threadIdx.x; ++n) run += own[n];
        next[threadIdx.x] = run + prior[threadIdx.x];
        if (q == 0) {
            const int64_t b = (int64_t)s * N + threadIdx.x;
            counts[b] = (int32_t)own[threadIdx.x];
            offsets[b] = run;
            if (b == (int64_t)G * N - 1) offsets[b + 1] = run + own[threadIdx.x];
        }
    }
    for (;;) {
        wave_nodes(B, N, seg[wave]);
        __syncthreads();
        if (threadIdx.x < N) {
            uint32_t run = next[threadIdx.x];
#pragma unroll
            for (int w = 0; w < kNodeWaves; ++w) {
                const uint32_t v = seg[w][threadIdx.x];
                seg[w][threadIdx.x] = run;
                run += v;
            }
            next[threadIdx.x] = run;
        }
        __syncthreads();
        write_node_rows<KM, NV>(B, code, t, t < t1, N, node_pos, fwd, row_token,
                                [&](int n, int rank) { return (int)seg[wave][n] + rank; });
        t += kNodeThreads;
        if (t - threadIdx.x >= t1) break;
        B = t < t1 ? node_set<KM, VEC>(assigned, t, K, G, g, by_g, code) : 0u;
        __syncthreads();  // seg is rewritten
    }
}

// Node set of token t < T and its source; an empty set without a valid one.
template <int KM, int VEC>
__device__ __forceinline__ uint32_t token_nodes(const int32_t* __restrict__ assigned,
                                                const int32_t* __restrict__ src, int64_t t,
                                                int64_t T, int K, int G, int g, SmallDiv by_g,
                                                int* s, int (&code)[KM]) {
    *s = 0;
    if (t >= T) return 0u;
    const int st = src[t];
    const uint32_t B = node_set<KM, VEC>(assigned, t, K, G, g, by_g, code);
    if ((uint32_t)st >= (uint32_t)G) return 0u;
    *s = st;
    return B;
}

template <int KM, int VEC>
__global__ __launch_bounds__(kThreads) void any_node_count_kernel(
    const int32_t* __restrict__ assigned, const int32_t* __restrict__ src, int64_t T, int K, int N,
    int g, SmallDiv by_g, int64_t tile, int32_t* __restrict__ counts, uint32_t* __restrict__ hist) {
    __shared__ uint32_t window[kWindow];
    __shared__ uint32_t h[kMaxN];
    const int G = N * g;
    const int64_t t0 = blockIdx.x * tile, t1 = min(t0 + tile, T);
    const int first = src[t0], rows = window_rows(first, src[t1 - 1], G, N);
    const int lo = rows ? first : 0;
    for (int i = threadIdx.x; i < rows * N; i += kThreads) window[i] = 0;
    if (threadIdx.x < kMaxN) h[threadIdx.x] = 0;
    __syncthreads();
    for (int64_t t = t0 + threadIdx.x; t - threadIdx.x < t1; t += kThreads) {
        int s, code[KM];
        const uint32_t B = token_nodes<KM, VEC>(assigned, src, t, t1, K, G, g, by_g, &s, code);
        count_nodes(B, s, N, [&](int sv, int n, uint32_t c) {
            if (sv >= lo && sv < lo + rows) {
                atomicAdd(&window[(sv - lo) * N + n], c);
            } else {
                atomicAdd(&counts[(int64_t)sv * N + n], (int32_t)c);
                atomicAdd(&h[n], c);
            }
        });
    }
    flush_window(window, h, rows, lo, N, counts, hist);
}

// kTable: G * N <= kSmallTable, and every workgroup turns the counts into
// first rows itself; else `base` holds them.
template <int KM, int VEC, int NV, bool kTable>
__global__ __launch_bounds__(kThreads) void any_node_rank_kernel(
    const int32_t* __restrict__ assigned, const int32_t* __restrict__ src, int64_t T, int K, int N,
    int g, SmallDiv by_g, int64_t tile, const int32_t* __restrict__ counts,
    const uint32_t* __restrict__ hist, const int32_t* __restrict__ base,
    int64_t* __restrict__ offsets, int32_t* __restrict__ node_pos, uint32_t* __restrict__ fwd,
    int32_t* __restrict__ row_token) {
    __shared__ uint32_t table[kTable ? kSmallTable : 1], rows[kTable ? kSmallTable : 1];
    __shared__ uint32_t seg[kWaves][kMaxN];
    __shared__ uint32_t prior[kMaxN], wsum[kWaves];
    const int wave = threadIdx.x >> 6;
    const int G = N * g;
    const int64_t t0 = blockIdx.x * tile, t1 = min(t0 + tile, T);
    int s, code[KM];
    int64_t t = t0 + threadIdx.x;
    uint32_t B = token_nodes<KM, VEC>(assigned, src, t, t1, K, G, g, by_g, &s, code);
    if (threadIdx.x < kMaxN) prior[threadIdx.x] = 0;
    if constexpr (kTable)
        for (int i = threadIdx.x; i < G * N; i += kThreads) table[i] = (uint32_t)counts[i];
    __syncthreads();
    const int col = threadIdx.x & (kMaxN - 1);
    if (col < N) {
        uint32_t v = 0;
        for (int i = threadIdx.x / kMaxN; i < (int)blockIdx.x; i += kThreads / kMaxN)
            v += hist[(int64_t)i * N + col];
        if (v) atomicAdd(&prior[col], v);
    }
    __syncthreads();
    if constexpr (kTable) {
        first_rows(table, rows, prior, G, N, wsum, blockIdx.x == 0, nullptr, offsets);
        __syncthreads();
        if (threadIdx.x < N) prior[threadIdx.x] = 0;  // counted in rows
    }
    for (;;) {
        wave_nodes(B, N, seg[wave]);
        __syncthreads();
        if (threadIdx.x < N) {
            uint32_t run = prior[threadIdx.x];
#pragma unroll
            for (int w = 0; w < kWaves; ++w) {
                const uint32_t v = seg[w][threadIdx.x];
                seg[w][threadIdx.x] = run;
                run += v;
            }
            prior[threadIdx.x] = run;
        }
        __syncthreads();
        write_node_rows<KM, NV>(B, code, t, t < t1, N, node_pos, fwd, row_token,
                                [&](int n, int rank) {
                                    const int b = s * N + n;
                                    return (kTable ? (int)rows[b] : base[b]) + (int)seg[wave][n] +
                                           rank;
                                });
        t += kThreads;
        if (t - threadIdx.x >= t1) break;
        B = token_nodes<KM, VEC>(assigned, src, t, t1, K, G, g, by_g, &s, code);
        __syncthreads();  // seg is rewritten
    }
}

template <int KM, int VEC, int NV>
__global__ __launch_bounds__(kThreads) void small_node_layout_kernel(
    const int32_t* __restrict__ assigned, const int32_t* __restrict__ src, int T, int K, int N,
    int g, SmallDiv by_g, SmallDiv by_src, int32_t* __restrict__ counts,
    int64_t* __restrict__ offsets, int32_t* __restrict__ node_pos, uint32_t* __restrict__ fwd,
    int32_t* __restrict__ row_token) {
    __shared__ uint32_t table[kSmallTable], rows[kSmallTable];
    __shared__ uint32_t seg[kWaves][kMaxN];
    __shared__ uint32_t prior[kMaxN], wsum[kWaves];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int G = N * g;
    // node set and source of token t; an empty set without a valid source
    auto token = [&](int t, int* s, int (&code)[KM]) -> uint32_t {
        *s = 0;
        if (t >= T) return 0u;
        const int st = src ? src[t] : by_src(t);
        const uint32_t B = node_set<KM, VEC>(assigned, t, K, G, g, by_g, code);
        if ((uint32_t)st >= (uint32_t)G) return 0u;
        *s = st;
        return B;
    };
    auto count = [&](int t0, int t1) {  // tokens [t0, t1), both multiples of kThreads
        for (int t = t0 + threadIdx.x; t < t1; t += kThreads) {
            int s, code[KM];
            const uint32_t B = token(t, &s, code);
            count_nodes(B, s, N,
                        [&](int sv, int n, uint32_t c) { atomicAdd(&table[sv * N + n], c); });
        }
    };
    for (int i = threadIdx.x; i < G * N; i += kThreads) table[i] = 0;
    if (threadIdx.x < kMaxN) prior[threadIdx.x] = 0;
    __syncthreads();
    const int tile0 = blockIdx.x * kThreads;
    const int mine = tile0 + threadIdx.x;
    int s, code[KM];
    const uint32_t B = token(mine, &s, code);
    count(0, tile0);
    wave_nodes(B, N, seg[wave]);
    __syncthreads();
    const int col = threadIdx.x & (kMaxN - 1);
    if (tile0 > 0 && col < N) {
        uint32_t v = 0;
        for (int r = threadIdx.x / kMaxN; r < G; r += kThreads / kMaxN) v += table[r * N + col];
        if (v) atomicAdd(&prior[col], v);
    }
    __syncthreads();
    count(tile0, (T + kThreads - 1) / kThreads * kThreads);
    if (wave == 1 && lane < N) {
        uint32_t run = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            const uint32_t v = seg[w][lane];
            seg[w][lane] = run;
            run += v;
        }
    }
    __syncthreads();
    first_rows(table, rows, prior, G, N, wsum, blockIdx.x == 0, counts, offsets);
    __syncthreads();
    write_node_rows<KM, NV>(B, code, mine, mine < T, N, node_pos, fwd, row_token,
                            [&](int n, int rank) {
                                return (int)(rows[s * N + n] + seg[wave][n]) + rank;
                            });
}

size_t align256(size_t v) { return (v + 255) & ~size_t(255); }

}  // namespace

// The workspace: base[G][C], then counts of tiles. Per column it has one
// 64-bit word for every `unit` items, which holds the 32-bit counts of
// G + (items - 1) / unit tiles together with base's own space (a scheme uses
// one or the other).
static size_t workspace_bytes(int64_t items, int64_t unit, int G, int C) {
    return 256 + align256(sizeof(int32_t) * (size_t)G * C) +
           align256(sizeof(uint64_t) * (size_t)std::max<int64_t>((items + unit - 1) / unit, 1) * C);
}
size_t dispatch_workspace_bytes(int64_t T, int K, int G) {
    return workspace_bytes(T * K, kPairsPerWord, G, G);
}
size_t node_dispatch_workspace_bytes(int64_t T, int N, int G) {
    return workspace_bytes(T, kTokensPerWord, G, N);
}

// Most pairs of a call on whole-call workgroups. With source ranks given the
// line lies about where the other scheme is as fast: at 8200 pairs for one
// rank, 13900, 16600, 19500, 21400 and 22800 for 2 to 6, 26700 for 8, and
// past kSmallPairsAny from 16 on.
static int64_t small_pairs(bool src, int G) {
    if (!src || G == 1) return kSmallPairs;
    return std::min<int64_t>(kSmallPairsAny, kSmallPairs + 2304 * (int64_t)G);
}

// Whole-call workgroups read all ranks and sources while others write rows, so
// they are not for a call that puts the rows in their place (the other schemes
// read a tile before they write its rows).
static bool in_place(const int32_t* rows, int64_t n, const int32_t* assigned, int64_t pairs,
                     const int32_t* src, int64_t T) {
    return overlap(rows, 4 * n, assigned, 4 * pairs) || overlap(rows, 4 * n, src, 4 * T);
}

// Clears counts[R][C] in a kernel: a recorded memset node is no part of a
// captured call.
static void launch_clear(int32_t* counts, int n, hipStream_t s) {
    hipLaunchKernelGGL(clear_kernel, dim3((unsigned)std::min((n + 255) / 256, 256)), dim3(256), 0,
                       s, counts, n);
}

static void launch_scan(const int32_t* counts, int R, int C, int64_t* offsets, int32_t* base,
                        hipStream_t s) {
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(1), dim3(kScanThreads), 0, s, counts, R, C, offsets, base);
    };
    R * C <= kScanLds ? launch(scan_kernel<true>) : launch(scan_kernel<false>);
}

cobalt_status launch_layout(const int32_t* assigned, const int32_t* src, int64_t T, int K, int G,
                            int32_t* counts, int64_t* offsets, int32_t* pos, void* ws,
                            hipStream_t s) {
    const int64_t TK = T * K;
    int32_t* base = (int32_t*)ws;
    if (T == 0) {
        launch_clear(counts, G * G, s);
        launch_scan(counts, G, G, offsets, base, s);
    } else if (G <= kSmallG && TK <= small_pairs(src != nullptr, G) &&
               !in_place(pos, TK, assigned, TK, src, T)) {
        const unsigned blocks = (unsigned)((TK + kThreads - 1) / kThreads);
        hipLaunchKernelGGL(small_layout_kernel, dim3(blocks), dim3(kThreads), 0, s, assigned, src,
                           (int)TK, G, divide_by(K), divide_by(src ? 1 : TK / G), counts, offsets,
                           pos);
    } else if (!src) {
        const Tiles t = make_tiles(TK / G, G, kPass);
        const unsigned blocks = (unsigned)G * (unsigned)t.per_src;
        uint32_t* hist = (uint32_t*)ws;
        uint32_t* sums = hist + (int64_t)blocks * G;
        hipLaunchKernelGGL(tile_count_kernel, dim3(blocks), dim3(kThreads), 0, s, assigned, G,
                           TK / G, t.tile, t.per_src, hist, sums);
        hipLaunchKernelGGL(tile_rank_kernel, dim3(blocks), dim3(kThreads), 0, s, assigned, G,
                           TK / G, t.tile, t.per_src, hist, sums, counts, offsets, pos);
    } else {
        const int64_t tile = kPass * std::max<int64_t>(1, (TK + kPass * kMaxAnyTiles - 1) /
                                                              (kPass * kMaxAnyTiles));
        const unsigned blocks = (unsigned)((TK + tile - 1) / tile);
        uint32_t* hist = (uint32_t*)((char*)ws + align256(sizeof(int32_t) * (size_t)G * G));
        launch_clear(counts, G * G, s);
        hipLaunchKernelGGL(any_count_kernel, dim3(blocks), dim3(kThreads), 0, s, assigned, src, TK,
                           K, divide_by(K), G, tile, counts, hist);
        if (G > kSmallG) launch_scan(counts, G, G, offsets, base, s);
        auto rank = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3(blocks), dim3(kThreads), 0, s, assigned, src, TK, K,
                               divide_by(K), G, tile, counts, hist, base, offsets, pos);
        };
        G > kSmallG ? rank(any_rank_kernel<kMaxG>) : rank(any_rank_kernel<kSmallG>);
    }
    COBALT_LAUNCH_CHECK();
    return COBALT_OK;
}

cobalt_status launch_node_layout(const int32_t* assigned, const int32_t* src, int64_t T, int K,
                                 int N, int g, int32_t* counts, int64_t* offsets,
                                 int32_t* node_pos, uint32_t* fwd, int32_t* row_token, void* ws,
                                 hipStream_t s) {
    const int G = N * g;
    int32_t* base = (int32_t*)ws;
    const bool table = G * N <= kSmallTable;
    // whole rows of node_pos per store (without: 6 % longer over 192 sizes)
    const bool nv = N % 4 == 0 && ((uintptr_t)node_pos & 15u) == 0;
    if (T == 0) {
        launch_clear(counts, G * N, s);
        launch_scan(counts, G, N, offsets, base, s);
        COBALT_LAUNCH_CHECK();
        return COBALT_OK;
    }
    by_row(K, assigned, [&](auto km, auto vec) {
        constexpr int KM = decltype(km)::value, V = decltype(vec)::value;
        if (table && T <= (src ? kSmallTokensAny : kSmallTokens) &&
            !in_place(node_pos, T * N, assigned, T * K, src, T)) {
            const unsigned blocks = (unsigned)((T + kThreads - 1) / kThreads);
            auto launch = [&](auto kernel) {
                hipLaunchKernelGGL(kernel, dim3(blocks), dim3(kThreads), 0, s, assigned, src,
                                   (int)T, K, N, g, divide_by(g), divide_by(src ? 1 : T / G),
                                   counts, offsets, node_pos, fwd, row_token);
            };
            nv ? launch(small_node_layout_kernel<KM, V, 4>)
               : launch(small_node_layout_kernel<KM, V, 1>);
        } else if (!src) {
            const Tiles t = make_tiles(T / G, G, kNodeThreads);
            const unsigned blocks = (unsigned)G * (unsigned)t.per_src;
            uint32_t* hist = (uint32_t*)ws;
            hipLaunchKernelGGL((node_tile_count_kernel<KM, V>), dim3(blocks), dim3(kNodeThreads),
                               0, s, assigned, K, N, g, divide_by(g), T / G, t.tile, t.per_src,
                               hist);
            auto launch = [&](auto kernel) {
                hipLaunchKernelGGL(kernel, dim3(blocks), dim3(kNodeThreads), 0, s, assigned, K, N,
                                   g, divide_by(g), T / G, t.tile, t.per_src, hist, counts,
                                   offsets, node_pos, fwd, row_token);
            };
            nv ? launch(node_tile_rank_kernel<KM, V, 4>) : launch(node_tile_rank_kernel<KM, V, 1>);
        } else {
            const int64_t tile = kThreads * std::max<int64_t>(1, (T + kThreads * kMaxAnyTiles - 1) /
                                                                     (kThreads * kMaxAnyTiles));
            const unsigned blocks = (unsigned)((T + tile - 1) / tile);
            uint32_t* hist = (uint32_t*)((char*)ws + align256(sizeof(int32_t) * (size_t)G * N));
            launch_clear(counts, G * N, s);
            hipLaunchKernelGGL((any_node_count_kernel<KM, V>), dim3(blocks), dim3(kThreads), 0, s,
                               assigned, src, T, K, N, g, divide_by(g), tile, counts, hist);
            if (!table) launch_scan(counts, G, N, offsets, base, s);
            auto launch = [&](auto kernel) {
                hipLaunchKernelGGL(kernel, dim3(blocks), dim3(kThreads), 0, s, assigned, src, T, K,
                                   N, g, divide_by(g), tile, counts, hist, base, offsets, node_pos,
                                   fwd, row_token);
            };
            if (table)
                nv ? launch(any_node_rank_kernel<KM, V, 4, true>)
                   : launch(any_node_rank_kernel<KM, V, 1, true>);
            else
                nv ? launch(any_node_rank_kernel<KM, V, 4, false>)
                   : launch(any_node_rank_kernel<KM, V, 1, false>);
        }
    });
    COBALT_LAUNCH_CHECK();
    return COBALT_OK;
}

}  // namespace cobalt

// Per-replica workload (Section 3.1, the workload model: w_er is the number
// of tasks of expert e executed by its replica on rank r; Section 3.2,
// Stage 2 tracks it per replica for the intra-node rebalancing).
//
// load[e][r] += #{pairs p : topk_idx[p] = e and assigned_rank[p] = r}.
// Same two-kernel scheme as the co-activation statistics:
//   count   grid = chunks x bands. A workgroup takes a contiguous chunk of
//           pairs and keeps the bins of a band of expert rows in LDS (all
//           rows when E*G fits and the grid is large enough without bands).
//           Pairs come four at a time with 16-byte loads of topk_idx and
//           assigned_rank where both are aligned. The band's bins are then
//           written out, at their place among the chunk's E*G bins, as uint16
//           where a chunk's pair count fits, else as uint32.
//   reduce  sixteen lanes per group of eight bins sum the chunks (one
//           16-byte load of eight uint16 bins per chunk), add pairwise
//           across lanes k and k + 8, exchange halves in three shuffle
//           rounds, and lane k < 8 adds the total of bin k into load: one
//           writer per element.
#include <algorithm>

#include "internal.hpp"

namespace cobalt {
namespace {

constexpr int kLoadThreads = 1024;
constexpr int kReduceThreads = 256;
constexpr int kReduceLanes = 16;
constexpr int64_t kPairsPerChunk = 16384;
constexpr int64_t kMaxChunks = 64;
constexpr int64_t kBandWords = 16384;  // 64 KiB of LDS
// Workgroups that the bands make up to. Every band reads all pairs of its
// chunk: T = 262144, K = 8 on E x G = 384 x 64 takes 9.7 us in 64 chunks x 4
// bands (10.3 without the write-through stores), 12.3 in 64 x 6 (bands halved
// until there were 256 workgroups).
constexpr int kMinGroups = 256;

// The partials take nchunks * E*G bins however they are cut into bands, so
// the workspace never shrinks as T, K, E or G grows: one of the size for a
// program's largest call serves its smaller ones. (With a slot of its own for
// every band, rounded up, E = 64, G = 32, K = 8 asked for 125440 bytes at T =
// 58000 and 118784 at T = 60000.)
struct LoadPlan {
    int nchunks, nbands, band_rows;
    bool u16;                // partial bins stored as uint16
    int64_t pairs_per_chunk; // a multiple of 4
    int64_t stride;          // bins of a chunk: E*G rounded up to a multiple of 8
    size_t bytes;
};

LoadPlan make_plan(int64_t T, int K, int E, int G) {
    LoadPlan p;
    const int64_t pairs = T * K;
    p.nchunks = (int)std::min<int64_t>(kMaxChunks, std::max<int64_t>(1, pairs / kPairsPerChunk));
    p.pairs_per_chunk = std::max<int64_t>(4, ((pairs + p.nchunks - 1) / p.nchunks + 3) & ~3);
    // as many bands of equal rows as the LDS needs, or as fill the chip; a
    // band starts at a multiple of eight bins, for its 16-byte stores
    const int64_t unit = G % 8 == 0 ? 1 : G % 4 == 0 ? 2 : G % 2 == 0 ? 4 : 8;
    const int64_t fit = kBandWords / G / unit * unit;
    const int64_t fill = std::min<int64_t>(E, (kMinGroups + p.nchunks - 1) / p.nchunks);
    const int64_t bands = std::max((E + fit - 1) / fit, fill);
    p.band_rows = (int)(((E + bands - 1) / bands + unit - 1) / unit * unit);
    p.nbands = (E + p.band_rows - 1) / p.band_rows;
    p.u16 = p.pairs_per_chunk <= 65535;
    p.stride = ((int64_t)E * G + 7) & ~int64_t(7);
    p.bytes = ((size_t)p.nchunks * p.stride * (p.u16 ? 2 : 4) + 255) & ~size_t(255);
    return p;
}

// kVec: four pairs per 16-byte load of each input (both 16-byte aligned and
// every chunk a multiple of four pairs, the last one included).
template <bool kVec, bool U16>
__global__ __launch_bounds__(kLoadThreads) void load_count_kernel(
    const int32_t* __restrict__ topk, const int32_t* __restrict__ assigned, int64_t TK, int E,
    int G, int nchunks, int band_rows, int64_t pairs_per_chunk, int64_t stride,
    void* __restrict__ part) {
    __shared__ __align__(16) uint32_t hist[kBandWords];
    const int chunk = blockIdx.x % nchunks;
    const int band = blockIdx.x / nchunks;
    const int e_lo = band * band_rows;
    const int e_hi = min(E, e_lo + band_rows);
    const int groups = ((e_hi - e_lo) * G + 7) / 8;  // of eight bins, band_rows * G / 8 at most
    for (int b = threadIdx.x; b < groups * 8; b += kLoadThreads) hist[b] = 0;
    __syncthreads();
    const int64_t p0 = (int64_t)chunk * pairs_per_chunk;
    const int64_t p1 = min(TK, p0 + pairs_per_chunk);
    auto add = [&](int e, int r) {
        if (e >= e_lo && e < e_hi && r >= 0 && r < G) atomicAdd(&hist[(e - e_lo) * G + r], 1u);
    };
    if constexpr (kVec) {
        const int4* t4 = reinterpret_cast<const int4*>(topk);
        const int4* a4 = reinterpret_cast<const int4*>(assigned);
        for (int64_t q = p0 / 4 + threadIdx.x; q < p1 / 4; q += kLoadThreads) {
            const int4 e = t4[q], r = a4[q];
            add(e.x, r.x);
            add(e.y, r.y);
            add(e.z, r.z);
            add(e.w, r.w);
        }
    } else {
        for (int64_t p = p0 + threadIdx.x; p < p1; p += kLoadThreads) add(topk[p], assigned[p]);
    }
    __syncthreads();
    // bins past the band's rows are zero (cleared above, never counted)
    const int64_t at = chunk * stride + (int64_t)e_lo * G;
    for (int g = threadIdx.x; g < groups; g += kLoadThreads) {
        const u32x4 lo = *reinterpret_cast<const u32x4*>(hist + g * 8);
        const u32x4 hi = *reinterpret_cast<const u32x4*>(hist + g * 8 + 4);
        if constexpr (U16) {
            const u32x4 packed = {lo.x | (lo.y << 16), lo.z | (lo.w << 16), hi.x | (hi.y << 16),
                                  hi.z | (hi.w << 16)};
            store_through(packed, static_cast<uint16_t*>(part) + at, groups * 16, g * 16);
        } else {
            uint32_t* out = static_cast<uint32_t*>(part) + at;
            store_through(lo, out, groups * 32, g * 32);
            store_through(hi, out, groups * 32, g * 32 + 16);
        }
    }
}

template <bool U16>
__global__ __launch_bounds__(kReduceThreads) void load_reduce_kernel(
    const void* __restrict__ part, int64_t bins, int nchunks, int64_t stride,
    uint32_t* __restrict__ load) {
    const int64_t gid = (int64_t)blockIdx.x * kReduceThreads + threadIdx.x;
    const int k = (int)(gid % kReduceLanes);
    const int64_t w0 = gid / kReduceLanes * 8;
    if (w0 >= bins) return;  // whole groups of lanes
    const int64_t bin = w0 + (k & 7);
    const bool real = k < 8 && bin < bins;
    const uint32_t prev = real ? load[bin] : 0u;
    uint32_t s[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    if constexpr (U16) {
        const uint16_t* src = static_cast<const uint16_t*>(part) + w0;
#pragma unroll 4
        for (int c = k; c < nchunks; c += kReduceLanes) {
            const u32x4 v = *reinterpret_cast<const u32x4*>(src + (int64_t)c * stride);
#pragma unroll
            for (int h = 0; h < 4; ++h) {
                s[2 * h] += v[h] & 0xffffu;
                s[2 * h + 1] += v[h] >> 16;
            }
        }
    } else {
        const uint32_t* src = static_cast<const uint32_t*>(part) + w0;
#pragma unroll 4
        for (int c = k; c < nchunks; c += kReduceLanes) {
            const u32x4* q = reinterpret_cast<const u32x4*>(src + (int64_t)c * stride);
            const u32x4 lo = q[0], hi = q[1];
#pragma unroll
            for (int h = 0; h < 4; ++h) {
                s[h] += lo[h];
                s[4 + h] += hi[h];
            }
        }
    }
    // lanes k, k ^ 8 add; then each round halves the bins a lane holds
#pragma unroll
    for (int o = 8; o < kReduceLanes; o <<= 1)
#pragma unroll
        for (int m = 0; m < 8; ++m) s[m] += __shfl_xor(s[m], o, kReduceLanes);
#pragma unroll
    for (int m = 0; m < 4; ++m) {
        const bool up = k & 4;
        const uint32_t keep = up ? s[4 + m] : s[m], give = up ? s[m] : s[4 + m];
        s[m] = keep + __shfl_xor(give, 4, kReduceLanes);
    }
#pragma unroll
    for (int m = 0; m < 2; ++m) {
        const bool up = k & 2;
        const uint32_t keep = up ? s[2 + m] : s[m], give = up ? s[m] : s[2 + m];
        s[m] = keep + __shfl_xor(give, 2, kReduceLanes);
    }
    {
        const bool up = k & 1;
        const uint32_t keep = up ? s[1] : s[0], give = up ? s[0] : s[1];
        s[0] = keep + __shfl_xor(give, 1, kReduceLanes);
    }
    if (real && s[0]) load[bin] = prev + s[0];
}

}  // namespace

size_t replica_load_workspace_bytes(int64_t T, int K, int E, int G) {
    return std::max<size_t>(make_plan(T, K, E, G).bytes, 256);
}

cobalt_status launch_replica_load(const int32_t* topk, const int32_t* assigned, int64_t T, int K,
                                  int E, int G, uint32_t* load, void* ws, size_t ws_bytes,
                                  hipStream_t s) {
    const LoadPlan p = make_plan(T, K, E, G);
    if (ws_bytes < p.bytes) return COBALT_EINVAL;
    const int64_t TK = T * K;
    const bool vec = TK % 4 == 0 && ((uintptr_t)topk & 15u) == 0 && ((uintptr_t)assigned & 15u) == 0;
    auto count = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)(p.nchunks * p.nbands)), dim3(kLoadThreads), 0, s,
                           topk, assigned, TK, E, G, p.nchunks, p.band_rows, p.pairs_per_chunk,
                           p.stride, ws);
    };
    if (p.u16)
        vec ? count(load_count_kernel<true, true>) : count(load_count_kernel<false, true>);
    else
        vec ? count(load_count_kernel<true, false>) : count(load_count_kernel<false, false>);
    COBALT_LAUNCH_CHECK();
    const int64_t items = p.stride / 8 * kReduceLanes;
    const dim3 grid((unsigned)((items + kReduceThreads - 1) / kReduceThreads));
    if (p.u16)
        hipLaunchKernelGGL(load_reduce_kernel<true>, grid, dim3(kReduceThreads), 0, s, ws,
                           (int64_t)E * G, p.nchunks, p.stride, load);
    else
        hipLaunchKernelGGL(load_reduce_kernel<false>, grid, dim3(kReduceThreads), 0, s, ws,
                           (int64_t)E * G, p.nchunks, p.stride, load);
    COBALT_LAUNCH_CHECK();
    return COBALT_OK;
}

}  // namespace cobalt

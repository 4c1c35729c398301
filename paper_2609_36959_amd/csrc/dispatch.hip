// Dispatch pack: the row copies behind the layouts of layout.hip.
//
//   scatter       per-pair layout: one wave per (token, slice, slot or two)
//                 reads the slice of x (from the cache for all but the first
//                 of the token's waves) and stores it to the slots' rows
//   node_scatter  node-deduplicated layout: four waves per (token, slice)
//                 with two or four nodes each
#include <algorithm>
#include <mutex>
#include <vector>

#include "internal.hpp"

namespace cobalt {
namespace {

// Row scatter for the per-pair layout: one workgroup per (token, slice of C
// KiB), R slots per wave (j, j + waves, ...). The waves that copy one slice of
// x[t] share a workgroup, so the slice is read from HBM once and from the
// cache by all waves but the first (plain loads keep it cached); each wave
// then issues a burst of C KiB to each of its packed rows, with non-temporal
// stores. On the T=131072, K=8, d=7168 workload (C = 2, R = 1) this reaches
// 5.9 TB/s, where one wave that stores its slice to all K rows reaches 5.1.
template <int C, int R>
__global__ __launch_bounds__(kMaxK * 64) void scatter_kernel(
    const u32x4* __restrict__ x, const int32_t* __restrict__ pos, int K, int64_t nch,
    int64_t bound, Slices cut, u32x4* __restrict__ packed) {
    uint32_t t, g;
    cut.split(blockIdx.x, &t, &g);
    const int j = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t c0 = (int64_t)g * (64 * C) + (threadIdx.x & 63);
    // The x loads are issued before the packed rows are read: a branch on the
    // row first would make every wave wait for that load before its own
    // loads start (measured: 3.45 ms instead of 2.95 ms). The in-range
    // guards also keep them there: without them the compiler sinks the
    // loads below the branch on p, with the same cost (3.42 ms at d = 7168).
    const u32x4* row = x + (int64_t)t * nch;
    u32x4 v[C];
#pragma unroll
    for (int i = 0; i < C; ++i)
        if (c0 + 64 * i < nch) v[i] = row[c0 + 64 * i];
    const int waves = blockDim.x >> 6;
    int p[R];
#pragma unroll
    for (int k = 0; k < R; ++k) {
        const int slot = j + waves * k;
        p[k] = R == 1 || slot < K ? pos[(int64_t)t * K + slot] : -1;
    }
    // The descriptor of a row's slice drops stores past the row's end, so the
    // stores need no guard of their own: all issue back to back from one
    // offset register.
    const int64_t first = (int64_t)g * (64 * C);
    const int32_t bytes = (int32_t)min(nch - first, (int64_t)(64 * C)) * 16;
    const int32_t off = (threadIdx.x & 63) * 16;
#pragma unroll
    for (int k = 0; k < R; ++k) {
        if (p[k] < 0 || p[k] >= bound) continue;
        u32x4* dst = packed + (int64_t)p[k] * nch + first;
#pragma unroll
        for (int i = 0; i < C; ++i) store_stream(v[i], dst, bytes, off + 1024 * i);
    }
}

// How scatter_kernel moves the rows of a call: 2 KiB slices and a wave per
// row, or a shape of 1 KiB slices where the output is larger than the
// memory-side cache (with less the shapes are level, and K = 1 takes 14 %
// longer in 1 KiB slices below 32 MB). Past that, what is fastest depends on
// how the rows' addresses fall on the memory channels, that is on K, d and
// the routing together, so the shapes are a table of what holds over 14600
// calls (all K; d from 1024 to 8192; T from 2048 to 131072; 8 to 64 ranks;
// uniform and skewed routing, half of it from the assignment), as the
// geometric mean (and the largest) of the ratio to the time in 2 KiB slices,
// for rows of whole KiB from d = 2048 on:
//   1 KiB slices, a wave per row: K = 1 0.91 (1.07), K = 2 0.91 (1.09).
//   1 KiB slices, two rows per wave: K = 3 0.94 (1.06), K = 10 0.92 (1.05),
//     K = 16 0.90 (1.18) for whole 2 KiB (1.03 (1.08) at d = 2560), K = 6
//     0.96 (1.07) and K = 8 0.94 (1.18) where d is a power of two (K = 6 1.00
//     (1.08) else).
//     K = 8 has buckets to avoid: sources in equal blocks whose buckets, if
//     they are equal too, lie at multiples of a power of two of at least 8
//     MiB, so that all ranks' rows meet the same channels at a time: 0.97
//     (1.42), worst with uniform routing (T = 65536, d = 4096, 16 ranks: 830
//     us in 2 KiB slices, 1177 in two rows per wave).
//     Not taken: K = 4 0.99 (1.28), 5 1.01 (1.10), 7 1.00 (1.06), 9 1.07
//     (1.26), 11 1.02 (1.12), 12 0.98 (1.05), 13 0.98 (1.10), 14 0.97 (1.07)
//     and 15 0.94 (1.09).
// Rows that are no whole number of KiB, or short, go by chunks_per_lane.
struct PackShape {
    int c, rows;
};
constexpr int64_t kCachedBytes = 256 << 20;

PackShape pack_shape(int64_t T, int K, int G, bool equal_blocks, int64_t nch) {
    const PackShape plain = {chunks_per_lane(nch), 1};
    const int64_t bytes = T * K * nch * 16;
    if (nch % 64 != 0 || nch < 256 || bytes <= kCachedBytes) return plain;
    const auto power_of_two = [](int64_t v) { return (v & (v - 1)) == 0; };
    const int64_t ranks2 = (int64_t)G * G;
    switch (K) {
        case 1:
        case 2:
            return {1, 1};
        case 3:
        case 10:
            return {1, 2};
        case 6:
            return power_of_two(nch) ? PackShape{1, 2} : plain;
        case 8:
            if (equal_blocks && bytes % ranks2 == 0 && power_of_two(bytes / ranks2) &&
                bytes / ranks2 >= (8 << 20))
                return plain;
            return power_of_two(nch) ? PackShape{1, 2} : plain;
        case 16:
            return nch % 128 == 0 ? PackShape{1, 2} : plain;
        default:
            return plain;
    }
}

// Row scatter for the node-deduplicated layout: one workgroup of
// kNodeScatterWaves waves per (token, slice); wave j loads the slice of x[t]
// and stores it to the token's rows for nodes n = j, j + 4, ... (SPW of them
// at most). A token has rows on only about half of the nodes, so one wave per
// node would leave half of the waves without a row (2.06 ms) and one wave for
// all of the token's rows serialises their stores (1.99 ms); two nodes per
// wave take 1.63 ms on the T=131072, N=8, d=7168 workload.
constexpr int kNodeScatterWaves = 4;

template <int C, int SPW>
__global__ __launch_bounds__(kNodeScatterWaves * 64) void node_scatter_kernel(
    const u32x4* __restrict__ x, const int32_t* __restrict__ node_pos, int N, int64_t nch,
    int64_t bound, Slices cut, u32x4* __restrict__ packed) {
    uint32_t t, g;
    cut.split(blockIdx.x, &t, &g);
    const int j = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t c0 = (int64_t)g * (64 * C) + (threadIdx.x & 63);
    // loads first, as in scatter_kernel (the guards keep them there)
    const u32x4* row = x + (int64_t)t * nch;
    u32x4 v[C];
#pragma unroll
    for (int i = 0; i < C; ++i)
        if (c0 + 64 * i < nch) v[i] = row[c0 + 64 * i];
    int q[SPW];
#pragma unroll
    for (int i = 0; i < SPW; ++i) {
        const int n = j + kNodeScatterWaves * i;
        q[i] = n < N ? node_pos[(int64_t)t * N + n] : -1;
    }
#pragma unroll
    for (int s = 0; s < SPW; ++s) {
        if (q[s] < 0 || q[s] >= bound) continue;
        u32x4* dst = packed + (int64_t)q[s] * nch;
#pragma unroll
        for (int i = 0; i < C; ++i)
            if (c0 + 64 * i < nch) __builtin_nontemporal_store(v[i], dst + c0 + 64 * i);
    }
}

}  // namespace

cobalt_status launch_dispatch(const int32_t* assigned, const int32_t* src, int64_t T, int K,
                              int G, const void* x, int64_t d, int32_t* counts, int64_t* offsets,
                              int32_t* pos, void* packed, void* ws, hipStream_t s) {
    if (cobalt_status st = launch_layout(assigned, src, T, K, G, counts, offsets, pos, ws, s))
        return st;
    if (T == 0 || !x) return COBALT_OK;
    const int64_t nch = d / 8;
    const PackShape shape = pack_shape(T, K, G, src == nullptr, nch);
    const Slices cut = cut_row(nch, shape.c);
    const int threads = (K + shape.rows - 1) / shape.rows * 64;
    for_token_ranges(T, (int64_t)cut.slices * threads, [&](int64_t t0, int64_t n) {
        auto launch = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3((unsigned)(n * cut.slices)), dim3(threads), 0, s,
                               (const u32x4*)x + t0 * nch, pos + t0 * K, K, nch, T * K, cut,
                               (u32x4*)packed);
        };
        if (shape.rows == 2)
            launch(scatter_kernel<1, 2>);
        else if (shape.c == 1)
            launch(scatter_kernel<1, 1>);
        else if (shape.c == 2)
            launch(scatter_kernel<2, 1>);
        else
            launch(scatter_kernel<3, 1>);
    });
    COBALT_LAUNCH_CHECK();
    return COBALT_OK;
}

cobalt_status launch_node_dispatch(const int32_t* assigned, const int32_t* src, int64_t T, int K,
                                   int N, int g, const void* x, int64_t d, int32_t* counts,
                                   int64_t* offsets, int32_t* node_pos, uint32_t* fwd,
                                   int32_t* row_token, void* packed, void* ws, hipStream_t s) {
    if (cobalt_status st = launch_node_layout(assigned, src, T, K, N, g, counts, offsets, node_pos,
                                              fwd, row_token, ws, s))
        return st;
    if (T == 0 || !x) return COBALT_OK;
    const int64_t nch = d / 8, bound = T * std::min(K, N);
    by_slices(nch, 3, [&](auto c, const Slices& cut) {
        constexpr int C = decltype(c)::value;
        const int threads = kNodeScatterWaves * 64;
        for_token_ranges(T, (int64_t)cut.slices * threads, [&](int64_t t0, int64_t n) {
            auto launch = [&](auto kernel) {
                hipLaunchKernelGGL(kernel, dim3((unsigned)(n * cut.slices)), dim3(threads), 0, s,
                                   (const u32x4*)x + t0 * nch, node_pos + t0 * N, N, nch, bound,
                                   cut, (u32x4*)packed);
            };
            N <= 2 * kNodeScatterWaves ? launch(node_scatter_kernel<C, 2>)
                                       : launch(node_scatter_kernel<C, 4>);
        });
    });
    COBALT_LAUNCH_CHECK();
    return COBALT_OK;
}

// Scratch of cobalt_dispatch_pack_noalloc: the dispatch workspace as a fixed
// array in the library's device memory. Each GPU the library runs on holds
// its own copy, from when the code object is loaded there until the process
// ends. In host code the array's name denotes a host-side stand-in, not a
// device address: the device address is looked up once per device and only
// that address is handed to kernels. Every call writes the words it reads
// (tile counts and their sums, base rows) in an earlier kernel of its own,
// so what a previous call left in the array does not matter.
static __device__ __align__(256) uint8_t scratch[COBALT_DISPATCH_NOALLOC_SCRATCH_BYTES];

cobalt_status dispatch_noalloc_scratch(void** out) {
    static std::mutex mu;
    static std::vector<void*> addr;  // per device
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0) return COBALT_EHIP;
    std::lock_guard<std::mutex> lock(mu);
    if ((int)addr.size() <= dev) addr.resize(dev + 1, nullptr);
    if (!addr[dev]) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return COBALT_EHIP;
        addr[dev] = p;
    }
    *out = addr[dev];
    return COBALT_OK;
}

}  // namespace cobalt

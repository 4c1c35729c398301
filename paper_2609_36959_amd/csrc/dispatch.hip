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

// How scatter_kernel moves the rows of a call. Times in us on outputs of 4 to
// 15 GB with x from HBM, 2 KiB slices and a wave per row | the shape taken:
//   K <= 2: 1 KiB slices, a wave per row. K = 2, d = 4096: 633 | 497;
//     d = 2048: 286 | 249; d = 7168: 1035 | 898.
//   K = 3, 4, 6, 8, 10, 16: 1 KiB slices, two rows per wave. K = 8, d = 4096:
//     1646 | 1557; d = 8192: 2332 | 2153; K = 6, d = 4096: 1230 | 1188; K =
//     16, d = 4096: 1722 | 1383; K = 10: 1705 | 1578. With K = 4, 6 or 8 and
//     an odd number of 2 KiB slices from five on, those walk over all XCDs
//     and stay ahead (K = 8, d = 7168: 2304 against 2335).
//   other K (workgroups of an odd number of waves, or three): 2 KiB slices.
//     K = 5, d = 4096: 1030 against 1107 us; K = 12: 1479 against 1577.
// Rows that are no whole number of KiB, or short, go by chunks_per_lane.
struct PackShape {
    int c, rows;
};
PackShape pack_shape(int K, int64_t nch) {
    const bool whole = nch % 64 == 0 && (nch == 128 || nch >= 256);
    if (whole && K <= 2 && nch >= 256) return {1, 1};
    if (whole && (K == 3 || K == 10 || K == 16)) return {1, 2};
    if (whole && (K == 4 || K == 6 || K == 8) && (nch <= 512 || nch % 256 != 128)) return {1, 2};
    return {chunks_per_lane(nch), 1};
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
    const PackShape shape = pack_shape(K, nch);
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
    by_slices(nch, [&](auto c, const Slices& cut) {
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

// Dispatch pack: the row copies behind the layouts of layout.hip.
//
//   scatter       per-pair layout: one wave per (token, slice, slot) reads
//                 the slice of x (from the cache for all but the first of the
//                 token's K waves) and stores it to the slot's packed row
//   node_scatter  node-deduplicated layout: four waves per (token, slice)
//                 with two or four nodes each
#include <algorithm>
#include <mutex>
#include <vector>

#include "internal.hpp"

namespace cobalt {
namespace {

// Row scatter for the per-pair layout: one workgroup per (token, slice), one
// wave per slot j. The K waves that copy one slice of x[t] share a workgroup,
// so the slice is read from HBM once and from the cache K - 1 times (plain
// loads keep it cached); each wave then issues a single burst of C KiB to one
// packed row, with non-temporal stores. On the T=131072, K=8, d=7168 workload
// this reaches 5.7 TB/s, where one wave that stores its slice to all K rows
// reaches 5.1.
template <int C>
__global__ __launch_bounds__(kMaxK * 64) void scatter_kernel(
    const u32x4* __restrict__ x, const int32_t* __restrict__ pos, int K, int64_t nch,
    int64_t bound, Slices cut, u32x4* __restrict__ packed) {
    uint32_t t, g;
    cut.split(blockIdx.x, &t, &g);
    const int j = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t c0 = (int64_t)g * (64 * C) + (threadIdx.x & 63);
    // The x loads are issued before the packed row is read: a branch on the
    // row first would make every wave wait for that load before its own
    // loads start (measured: 3.45 ms instead of 2.95 ms). The in-range
    // guards also keep them there: without them the compiler sinks the
    // loads below the branch on p, with the same cost (3.42 ms at d = 7168).
    const u32x4* row = x + (int64_t)t * nch;
    u32x4 v[C];
#pragma unroll
    for (int i = 0; i < C; ++i)
        if (c0 + 64 * i < nch) v[i] = row[c0 + 64 * i];
    const int p = pos[(int64_t)t * K + j];
    if (p < 0 || p >= bound) return;
    // The descriptor of the row's slice drops stores past the row's end, so
    // the stores need no guard of their own: all issue back to back from one
    // offset register.
    const int64_t first = (int64_t)g * (64 * C);
    u32x4* dst = packed + (int64_t)p * nch + first;
    const int32_t bytes = (int32_t)min(nch - first, (int64_t)(64 * C)) * 16;
    const int32_t off = (threadIdx.x & 63) * 16;
#pragma unroll
    for (int i = 0; i < C; ++i) store_stream(v[i], dst, bytes, off + 1024 * i);
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
    by_slices(nch, [&](auto c, const Slices& cut) {
        for_token_ranges(T, (int64_t)cut.slices * K * 64, [&](int64_t t0, int64_t n) {
            hipLaunchKernelGGL(scatter_kernel<decltype(c)::value>, dim3((unsigned)(n * cut.slices)),
                               dim3(K * 64), 0, s, (const u32x4*)x + t0 * nch, pos + t0 * K, K,
                               nch, T * K, cut, (u32x4*)packed);
        });
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

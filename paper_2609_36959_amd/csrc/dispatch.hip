// Dispatch pack: the row copies behind the layouts of layout.hip.
//
//   scatter       per-pair layout: one wave per (token, 2 KiB slice, slot)
//                 reads the slice of x (from the cache for all but the first
//                 of the token's K waves) and stores it to the slot's packed
//                 row
//   node_scatter  node-deduplicated layout: four waves per (token, slice)
//                 with two or four nodes each
//   copy          either, for rows wider than 16 slices
#include <algorithm>
#include <mutex>
#include <vector>

#include "internal.hpp"

namespace cobalt {
namespace {

constexpr int kCopyWaves = 4;

// Row copy. Each wave takes one (token, column group): it loads CG 16-byte
// chunks per lane of x[t] (64*CG chunks, a contiguous 1-2 KiB slice of the
// row) once, then stores them to the K packed rows of the token. Small
// per-wave state keeps many waves in flight; plain stores sustain a higher
// write rate than non-temporal ones on this access pattern.
// KC = compile-time K (0: any K up to 16); with KC the scalar loads of the
// token's pos entries are issued together.
template <int CG, int KC, bool kNode>
__global__ __launch_bounds__(kCopyWaves * 64) void copy_kernel(
    const u32x4* __restrict__ x, const int32_t* __restrict__ pos, int64_t T, int Kr, int64_t nch,
    int64_t TK, u32x4* __restrict__ packed) {
    constexpr int KM = KC ? KC : kMaxK;
    const int K = KC ? KC : Kr;
    const int64_t groups = (nch + 64 * CG - 1) / (64 * CG);
    // wave-uniform item index, so pos comes in through scalar loads
    const int64_t item = (int64_t)blockIdx.x * kCopyWaves +
                         __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (item >= T * groups) return;
    const int64_t t = item / groups;
    const int64_t c0 = (item - t * groups) * 64 * CG + (threadIdx.x & 63);
    int p[KM];
#pragma unroll
    for (int j = 0; j < KM; ++j) p[j] = j < K ? pos[t * K + j] : -1;
    const u32x4* row = x + t * nch;
    u32x4 v[CG];
#pragma unroll
    for (int i = 0; i < CG; ++i)
        if (c0 + 64 * i < nch) v[i] = __builtin_nontemporal_load(row + c0 + 64 * i);
#pragma unroll
    for (int j = 0; j < KM; ++j) {
        if (p[j] < 0 || p[j] >= TK) continue;
        u32x4* dst = packed + (int64_t)p[j] * nch;
#pragma unroll
        for (int i = 0; i < CG; ++i)
            if (c0 + 64 * i < nch) dst[c0 + 64 * i] = v[i];
    }
}

// Row scatter for the per-pair layout: one workgroup per (token, 2 KiB
// column slice), one wave per slot j. The K waves that copy one slice of
// x[t] share a workgroup, so the slice is read from HBM once and from the
// cache K - 1 times (plain loads keep it cached); each wave then issues a
// single 2 KiB burst to one packed row, with non-temporal stores. On the
// T=131072, K=8, d=7168 workload this reaches 5.7 TB/s, where the fan-out
// of copy_kernel (one wave stores its slice to all K rows) reaches 5.1.
// GROUPS, the number of slices per row, is a template parameter so that
// the block index splits into (token, slice) with a constant division: a
// wave does two loads and two stores, and a runtime 64-bit division would
// cost it more scalar instructions than that.
template <int GROUPS>
__global__ __launch_bounds__(kMaxK * 64) void scatter_kernel(
    const u32x4* __restrict__ x, const int32_t* __restrict__ pos, int K, int64_t nch,
    int64_t bound, u32x4* __restrict__ packed) {
    const uint32_t tg = blockIdx.x;
    const uint32_t t = tg / GROUPS;
    const uint32_t g = tg - t * GROUPS;
    const int j = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t c0 = (int64_t)g * 128 + (threadIdx.x & 63);
    // The x loads are issued before the packed row is read: a branch on the
    // row first would make every wave wait for that load before its own
    // two loads start (measured: 3.45 ms instead of 2.95 ms). The in-range
    // guards also keep them there: without them the compiler sinks both
    // loads below the branch on p, with the same cost (3.42 ms at d = 7168).
    const u32x4* row = x + (int64_t)t * nch;
    const bool in0 = c0 < nch, in1 = c0 + 64 < nch;
    u32x4 v0, v1;
    if (in0) v0 = row[c0];
    if (in1) v1 = row[c0 + 64];
    const int p = pos[(int64_t)t * K + j];
    if (p < 0 || p >= bound) return;
    // The row's buffer descriptor drops stores past its nch chunks, so the
    // stores need no guard of their own: both issue back to back from one
    // offset register.
    u32x4* dst = packed + (int64_t)p * nch;
    const int32_t off = (int32_t)(c0 * 16);
    store_stream(v0, dst, (int32_t)(nch * 16), off);
    store_stream(v1, dst, (int32_t)(nch * 16), off + 1024);
}

// Launches scatter_kernel for rows pos[t][0..per_tok) in [0, bound) when
// the slice count has an instantiation; returns false otherwise (the
// caller then uses the fan-out copy).
template <int GROUPS>
bool try_scatter(const void* x, const int32_t* pos, int64_t T, int per_tok, int64_t nch,
                 int64_t bound, void* packed, hipStream_t s) {
    if ((nch + 127) / 128 != GROUPS)
        return try_scatter<GROUPS - 1>(x, pos, T, per_tok, nch, bound, packed, s);
    for_token_ranges(T, (int64_t)GROUPS * per_tok * 64, [&](int64_t t0, int64_t n) {
        hipLaunchKernelGGL(scatter_kernel<GROUPS>, dim3((unsigned)(n * GROUPS)),
                           dim3(per_tok * 64), 0, s, (const u32x4*)x + t0 * nch,
                           pos + t0 * per_tok, per_tok, nch, bound, (u32x4*)packed);
    });
    return true;
}
template <>
bool try_scatter<0>(const void*, const int32_t*, int64_t, int, int64_t, int64_t, void*,
                    hipStream_t) {
    return false;
}

// Row scatter for the node-deduplicated layout: one workgroup of
// kNodeScatterWaves waves per (token, 2 KiB column slice); wave j loads the
// slice of x[t] and stores it to the token's rows for nodes n = j, j + 4,
// ... (SPW of them at most). A token has rows on only about half of the
// nodes, so one wave per node would leave half of the waves without a row
// (2.06 ms) and one wave for all of the token's rows serialises their
// stores (1.99 ms); two nodes per wave take 1.63 ms on the T=131072, N=8,
// d=7168 workload. GROUPS as for scatter_kernel.
constexpr int kNodeScatterWaves = 4;

template <int GROUPS, int SPW>
__global__ __launch_bounds__(kNodeScatterWaves * 64) void node_scatter_kernel(
    const u32x4* __restrict__ x, const int32_t* __restrict__ node_pos, int N, int64_t nch,
    int64_t bound, u32x4* __restrict__ packed) {
    const uint32_t tg = blockIdx.x;
    const uint32_t t = tg / GROUPS;
    const uint32_t g = tg - t * GROUPS;
    const int j = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t c0 = (int64_t)g * 128 + (threadIdx.x & 63);
    // loads first, as in scatter_kernel (the guards keep them there)
    const u32x4* row = x + (int64_t)t * nch;
    const bool in0 = c0 < nch, in1 = c0 + 64 < nch;
    u32x4 v0, v1;
    if (in0) v0 = row[c0];
    if (in1) v1 = row[c0 + 64];
    int q[SPW];
#pragma unroll
    for (int i = 0; i < SPW; ++i) {
        const int n = j + kNodeScatterWaves * i;
        q[i] = n < N ? node_pos[(int64_t)t * N + n] : -1;
    }
#pragma unroll
    for (int i = 0; i < SPW; ++i) {
        if (q[i] < 0 || q[i] >= bound) continue;
        u32x4* dst = packed + (int64_t)q[i] * nch;
        if (in0) __builtin_nontemporal_store(v0, dst + c0);
        if (in1) __builtin_nontemporal_store(v1, dst + c0 + 64);
    }
}

// Launches node_scatter_kernel when the slice count has an instantiation;
// returns false otherwise (the caller then uses the fan-out copy).
template <int GROUPS>
bool try_node_scatter(const void* x, const int32_t* node_pos, int64_t T, int N, int64_t nch,
                      int64_t bound, void* packed, hipStream_t s) {
    if constexpr (GROUPS == 0) {
        return false;
    } else {
        if ((nch + 127) / 128 != GROUPS)
            return try_node_scatter<GROUPS - 1>(x, node_pos, T, N, nch, bound, packed, s);
        const dim3 block(kNodeScatterWaves * 64);
        for_token_ranges(T, (int64_t)GROUPS * kNodeScatterWaves * 64, [&](int64_t t0, int64_t n) {
            const dim3 grid((unsigned)(n * GROUPS));
            const u32x4* xr = (const u32x4*)x + t0 * nch;
            const int32_t* np = node_pos + t0 * N;
            if (N <= 2 * kNodeScatterWaves)
                hipLaunchKernelGGL((node_scatter_kernel<GROUPS, 2>), grid, block, 0, s, xr, np, N,
                                   nch, bound, (u32x4*)packed);
            else
                hipLaunchKernelGGL((node_scatter_kernel<GROUPS, 4>), grid, block, 0, s, xr, np, N,
                                   nch, bound, (u32x4*)packed);
        });
        return true;
    }
}

// Copies x[t] to the rows pos[t][0..per_tok) that are in [0, bound).
template <bool kNode>
cobalt_status launch_copy(const void* x, const int32_t* pos, int64_t T, int per_tok, int64_t d,
                          int64_t bound, void* packed, hipStream_t s) {
    const int64_t nch = d / 8;
    const u32x4* xv = (const u32x4*)x;
    u32x4* pv = (u32x4*)packed;
    auto launch = [&](auto kernel, int64_t cg) {
        const int64_t groups = (nch + 64 * cg - 1) / (64 * cg);  // one wave each
        for_token_ranges(T, groups * 64, [&](int64_t t0, int64_t n) {
            const int64_t items = n * groups;
            hipLaunchKernelGGL(kernel, dim3((unsigned)((items + kCopyWaves - 1) / kCopyWaves)),
                               dim3(kCopyWaves * 64), 0, s, xv + t0 * nch, pos + t0 * per_tok, n,
                               per_tok, nch, bound, pv);
        });
    };
    if (nch >= 128)
        per_tok == 8 ? launch(copy_kernel<2, 8, kNode>, 2) : launch(copy_kernel<2, 0, kNode>, 2);
    else
        per_tok == 8 ? launch(copy_kernel<1, 8, kNode>, 1) : launch(copy_kernel<1, 0, kNode>, 1);
    COBALT_LAUNCH_CHECK();
    return COBALT_OK;
}

}  // namespace

cobalt_status launch_dispatch(const int32_t* assigned, const int32_t* src, int64_t T, int K,
                              int G, const void* x, int64_t d, int32_t* counts, int64_t* offsets,
                              int32_t* pos, void* packed, void* ws, hipStream_t s) {
    if (cobalt_status st = launch_layout(assigned, src, T, K, G, counts, offsets, pos, ws, s))
        return st;
    if (T == 0 || !x) return COBALT_OK;
    const int64_t TK = T * K;
    if (try_scatter<16>(x, pos, T, K, d / 8, TK, packed, s)) {
        COBALT_LAUNCH_CHECK();
        return COBALT_OK;
    }
    return launch_copy<false>(x, pos, T, K, d, TK, packed, s);
}

cobalt_status launch_node_dispatch(const int32_t* assigned, const int32_t* src, int64_t T, int K,
                                   int N, int g, const void* x, int64_t d, int32_t* counts,
                                   int64_t* offsets, int32_t* node_pos, uint32_t* fwd,
                                   int32_t* row_token, void* packed, void* ws, hipStream_t s) {
    if (cobalt_status st = launch_node_layout(assigned, src, T, K, N, g, counts, offsets, node_pos,
                                              fwd, row_token, ws, s))
        return st;
    if (T == 0 || !x) return COBALT_OK;
    const int64_t bound = T * std::min(K, N);
    if (try_node_scatter<16>(x, node_pos, T, N, d / 8, bound, packed, s)) {
        COBALT_LAUNCH_CHECK();
        return COBALT_OK;
    }
    return launch_copy<true>(x, node_pos, T, N, d, bound, packed, s);
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

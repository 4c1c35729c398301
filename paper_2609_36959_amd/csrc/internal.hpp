// Internal declarations of the HIP routing library (gfx950).
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstddef>
#include <cstdint>
#include <type_traits>

#include "cobalt.h"

namespace cobalt {

constexpr int kMaxN = 16;
constexpr int kMaxGpn = 32;
constexpr int kMaxG = 512;
static_assert(kMaxN * kMaxGpn <= kMaxG, "N and gpus_per_node in range bound G");
constexpr int kMaxK = 16;
constexpr int kMaxE = 4096;

// 16-byte vector: eight bf16 values, the unit of every row copy.
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Streaming row store: a 16-byte raw buffer store with the non-temporal
// (nt) cache bit, through a buffer descriptor of `bytes` bytes at `base`.
// The hardware drops stores outside the descriptor, so a row's stores need
// no guard branches of their own and issue back to back from one offset
// register (with a branch per store the compiler can make the second wait
// for the first). The descriptor's third dword is the gfx9 raw-buffer
// format word.
__device__ __forceinline__ void store_stream(const u32x4& v, void* base, int32_t bytes,
                                             int32_t offset) {
    constexpr int kNt = 2;
    const __amdgpu_buffer_rsrc_t rs =
        __builtin_amdgcn_make_buffer_rsrc(base, (short)0, bytes, 0x00020000);
    __builtin_amdgcn_raw_buffer_store_b128(v, rs, offset, 0, kNt);
}

// Store of 16 bytes at base + offset that goes through the L2 as it is made
// (sc1), for data that the next kernel reads on all XCDs: plain stores leave
// the lines dirty in the writer's L2, and the kernel's end waits while all of
// them are written back.
__device__ __forceinline__ void store_through(const u32x4& v, void* base, int32_t bytes,
                                              int32_t offset) {
    constexpr int kSc1 = 16;
    const __amdgpu_buffer_rsrc_t rs =
        __builtin_amdgcn_make_buffer_rsrc(base, (short)0, bytes, 0x00020000);
    __builtin_amdgcn_raw_buffer_store_b128(v, rs, offset, 0, kSc1);
}

// x / y for 0 <= x < 2^17 and 1 <= y: (x + 1/2) / y lies at least 1 / (2y)
// from an integer, and the product is off by less than x / y * 2^-22.
struct SmallDiv {
    float inv;
    __host__ __device__ int operator()(int x) const { return (int)(((float)x + 0.5f) * inv); }
};
__host__ __device__ inline SmallDiv divide_by(int64_t v) { return {1.0f / (float)v}; }

// A row of K ints in slots 0..K-1 of v, VEC ints per access (K is a multiple
// of VEC and the row is aligned to VEC ints).
template <int KM, int VEC>
__device__ __forceinline__ void load_row(const int32_t* row, int K, int (&v)[KM]) {
#pragma unroll
    for (int j = 0; j < KM; j += VEC) {
        if (j >= K) continue;
        if constexpr (VEC == 4) {
            const int4 q = *reinterpret_cast<const int4*>(row + j);
            v[j] = q.x; v[j + 1] = q.y; v[j + 2] = q.z; v[j + 3] = q.w;
        } else if constexpr (VEC == 2) {
            const int2 q = *reinterpret_cast<const int2*>(row + j);
            v[j] = q.x; v[j + 1] = q.y;
        } else {
            v[j] = row[j];
        }
    }
}

template <int KM, int VEC>
__device__ __forceinline__ void store_row(int32_t* row, int K, const int (&v)[KM]) {
#pragma unroll
    for (int j = 0; j < KM; j += VEC) {
        if (j >= K) continue;
        if constexpr (VEC == 4)
            *reinterpret_cast<int4*>(row + j) = make_int4(v[j], v[j + 1], v[j + 2], v[j + 3]);
        else if constexpr (VEC == 2)
            *reinterpret_cast<int2*>(row + j) = make_int2(v[j], v[j + 1]);
        else
            row[j] = v[j];
    }
}

// Calls f(KM, VEC) for rows of K ints at `p`: KM slots in registers, VEC ints
// per access. Without 8-byte accesses K = 2, 6 and 10 take 1.8 % longer in the
// node layouts (144 sizes) and 2.3 % in the statistics (27).
template <typename F>
void by_row(int K, const void* p, F&& f) {
    auto vec = [&](auto km) {
        if (K % 4 == 0 && ((uintptr_t)p & 15u) == 0)
            f(km, std::integral_constant<int, 4>());
        else if (K % 2 == 0 && ((uintptr_t)p & 7u) == 0)
            f(km, std::integral_constant<int, 2>());
        else
            f(km, std::integral_constant<int, 1>());
    };
    if (K <= 8)
        vec(std::integral_constant<int, 8>());
    else
        vec(std::integral_constant<int, 16>());
}

// A row of nch 16-byte chunks in slices of 64 * c chunks, and a workgroup's
// index b < 2^31 split into (token, slice) without a division:
// b / slices = (b * magic) >> shift, with shift = 31 + ceil(log2 slices) and
// magic = ceil(2^shift / slices).
struct Slices {
    uint32_t slices, magic, shift;
    __host__ __device__ void split(uint32_t b, uint32_t* t, uint32_t* g) const {
        *t = (uint32_t)(((uint64_t)b * magic) >> shift);
        *g = b - *t * slices;
    }
};
inline Slices cut_row(int64_t nch, int c) {
    Slices s;
    s.slices = (uint32_t)((nch + 64 * c - 1) / (64 * c));
    int lg = 0;
    while ((1u << lg) < s.slices) ++lg;
    s.shift = 31 + lg;
    s.magic = (uint32_t)(((uint64_t(1) << s.shift) + s.slices - 1) / s.slices);
    return s;
}
// Chunks per lane of a wave that moves a slice of a row of nch chunks: two,
// but one for rows of a single wave's width, and three where a second slice
// of two would be more than half empty or the row ends early in it. Pack and
// combine of 16384 tokens, K = 8, in us with one | two | three:
//   nch  48:  15.3 + 25.3 | 16.6 + 25.7 | 20.7 + 29.7
//   nch 112:  35.2 + 50.8 | 39.1 + 40.6 | 37.7 + 48.0
//   nch 144:  46.0 + 70.9 | 60.6 + 69.9 | 48.9 + 63.1
//   nch 192:  64.8 + 78.4 | 69.3 + 78.4 | 68.0 + 71.1
//   nch 208:  83.2 + 97.5 | 71.7 + 81.8 | 91.8 + 118
//   nch 360:   130 + 153  |  133 + 128  |  127 + 139
// Long rows of one chunk per lane and row pack faster only while x comes out
// of the memory-side cache: T = 32768, nch = 512 0.34 against 0.47 ms, but T
// = 131072, nch = 896 3.8 against 2.9 ms.
inline int chunks_per_lane(int64_t nch) {
    return nch <= 64 ? 1 : nch > 128 && nch <= 192 ? 3 : 2;
}

// Calls f(C, cut) with the row's chunks per lane C, at most `most`, and its
// slices.
template <typename F>
void by_slices(int64_t nch, int most, F&& f) {
    const int c = std::min(chunks_per_lane(nch), most);
    const Slices cut = cut_row(nch, c);
    if (c == 1)
        f(std::integral_constant<int, 1>(), cut);
    else if (c == 2)
        f(std::integral_constant<int, 2>(), cut);
    else
        f(std::integral_constant<int, 3>(), cut);
}

// Whether na bytes at a and nb bytes at b share any. A caller may give an
// output the memory of an input that the call has no more use for; kernels
// that write the one while others still read the other ask first.
inline bool overlap(const void* a, int64_t na, const void* b, int64_t nb) {
    return a && b && (const char*)a < (const char*)b + nb && (const char*)b < (const char*)a + na;
}

struct DeviceLayout {
    int device;
    int32_t N, g, G, E, S;
    uint32_t* node_mask;       // [E]
    uint32_t* rank_mask;       // [E][N]
    int32_t* owner;            // [E]
};

// A dispatch packet holds the grid size in work-items as a 32-bit value,
// and a larger grid is cut short without an error. Kernels that take one
// workgroup (or wave) per token slice are therefore launched over ranges of
// tokens of at most max_launch_items() work-items each, with their
// per-token arrays offset to the range; the rows they address through pos
// or node_pos stay absolute.
constexpr int64_t kMaxLaunchItems = int64_t(1) << 31;

// kMaxLaunchItems, or a smaller limit from the environment variable
// COBALT_MAX_LAUNCH_ITEMS (read at every launch, at least 64), so that
// tests can split ordinary sizes into many ranges.
int64_t max_launch_items();

// Calls launch(t0, n) for consecutive token ranges [t0, t0 + n) covering
// [0, T), each of at most max_launch_items() / items_per_token tokens (at
// least one).
template <typename F>
void for_token_ranges(int64_t T, int64_t items_per_token, F&& launch) {
    const int64_t per = items_per_token > 0 ? items_per_token : 1;
    const int64_t lim = max_launch_items();
    const int64_t step = lim / per > 0 ? lim / per : 1;
    for (int64_t t0 = 0; t0 < T; t0 += step) launch(t0, T - t0 < step ? T - t0 : step);
}

#define COBALT_LAUNCH_CHECK()                                        \
    do {                                                             \
        if (hipGetLastError() != hipSuccess) return COBALT_EHIP;     \
    } while (0)

// Per-device properties used to size launches.
struct DeviceInfo {
    int cus;
    int lds_bytes;  // usable LDS per workgroup
};
cobalt_status device_info(DeviceInfo* out);

// Launchers (argument checks are done by the C entry points).
size_t coact_workspace_bytes(int64_t T, int K, int E, int lds_bytes);
cobalt_status launch_coact_stats(const int32_t* topk, int64_t T, int K, int E, uint32_t* coact,
                                 uint32_t* count, void* ws, size_t ws_bytes, hipStream_t s);
cobalt_status launch_assign(const DeviceLayout& L, const int32_t* topk, const int32_t* src,
                            int64_t T, int K, uint64_t key, int mode, int32_t* out,
                            uint16_t* remote, hipStream_t s);
size_t dispatch_workspace_bytes(int64_t T, int K, int G);
cobalt_status launch_dispatch(const int32_t* assigned, const int32_t* src, int64_t T, int K,
                              int G, const void* x, int64_t d, int32_t* counts,
                              int64_t* offsets, int32_t* pos, void* packed, void* ws,
                              hipStream_t s);
// Device address of the fixed dispatch scratch on the current device
// (COBALT_DISPATCH_NOALLOC_SCRATCH_BYTES bytes, 256-byte aligned); looked up
// on the first call on each device, allocates nothing.
cobalt_status dispatch_noalloc_scratch(void** out);
// Counts, offsets and rows of a dispatch (layout.hip).
cobalt_status launch_layout(const int32_t* assigned, const int32_t* src, int64_t T, int K, int G,
                            int32_t* counts, int64_t* offsets, int32_t* pos, void* ws,
                            hipStream_t s);
cobalt_status launch_node_layout(const int32_t* assigned, const int32_t* src, int64_t T, int K,
                                 int N, int g, int32_t* counts, int64_t* offsets,
                                 int32_t* node_pos, uint32_t* fwd, int32_t* row_token, void* ws,
                                 hipStream_t s);
size_t node_dispatch_workspace_bytes(int64_t T, int N, int G);
cobalt_status launch_node_dispatch(const int32_t* assigned, const int32_t* src, int64_t T, int K,
                                   int N, int g, const void* x, int64_t d, int32_t* counts,
                                   int64_t* offsets, int32_t* node_pos, uint32_t* fwd,
                                   int32_t* row_token, void* packed, void* ws, hipStream_t s);
cobalt_status launch_combine(const void* eo, const int32_t* pos, const float* gates, int64_t T,
                             int K, int64_t d, void* y, float* y32, hipStream_t s);
cobalt_status launch_node_combine(const void* eo, const int32_t* pos, const int32_t* assigned,
                                  const float* gates, const int32_t* node_pos, int64_t T, int K,
                                  int N, int gpn, int64_t d, void* partial, void* y,
                                  hipStream_t s);
size_t replica_load_workspace_bytes(int64_t T, int K, int E, int G);
cobalt_status launch_replica_load(const int32_t* topk, const int32_t* assigned, int64_t T, int K,
                                  int E, int G, uint32_t* load, void* ws, size_t ws_bytes,
                                  hipStream_t s);
cobalt_status launch_count_ema(uint32_t* counts, int64_t n, float decay, bool init, bool clear,
                               float* ema, hipStream_t s);
cobalt_status launch_coact_ema(uint32_t* coact, uint32_t* count, int E, float decay, bool init,
                               bool clear, float* ema_coact, float* ema_count, float* ochiai,
                               hipStream_t s);
cobalt_status launch_validate(const int32_t* topk, const int32_t* src, int64_t T, int K, int E,
                              int G, uint32_t* dflags, hipStream_t s);

// SplitMix64 (Steele, Lea & Flood 2014): output of the generator for state z.
__host__ __device__ inline uint64_t splitmix64(uint64_t z) {
    z += 0x9e3779b97f4a7c15ull;
    z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
    z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
    return z ^ (z >> 31);
}

}  // namespace cobalt

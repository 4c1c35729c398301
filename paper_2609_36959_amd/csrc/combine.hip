// Combine and weighted sum (Fig. 1, last stage):
//   y[t][c] = bf16_rne( sum_j gates[t][j] * expert_out[pos[t][j]][c] ),
// accumulated in fp32 from 0 with one fused multiply-add per slot in slot
// order; slots whose row is outside [0, T*K) are skipped.
//
// fold_kernel: one workgroup per (token, column slice of C KiB), one wave per
// slot j (at least C waves). Wave j loads its row's slice (non-temporal, C
// 16-byte chunks per lane) into LDS; after a barrier C waves fold the K
// slices in slot order, one 16-byte chunk (eight bf16 values) per thread, and
// store the slice of y. Each wave has a single row to fetch, so many
// independent row loads are in flight; on the T=131072, K=8, d=7168 workload
// (C = 2) this runs at 6.5-6.6 TB/s, against 5.6 TB/s when one wave loads the
// chunks of all K rows. Twice the folding waves, 8 bytes per thread, took 3 %
// longer, and half as many, two chunks per lane, hold the stage longer still.
//
// direct_kernel (the widest rows, where direct_fold says so): one wave per
// (token, 1 KiB slice) loads the chunks of all K rows itself.
//
// The node-level combine (the reverse of the node-deduplicated dispatch)
// follows: node_fold_kernel sums each node's slots into a bf16 partial row
// and the token's partial rows, in node order, into y.
#include <algorithm>

#include "internal.hpp"

namespace cobalt {
namespace {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

// Rounds a and b to bf16, nearest even, and packs them with a in the low
// half: one v_cvt_pk_bf16_f32. In the floating-point mode of these kernels
// (IEEE, fp32 denormals kept) it gives the bits of the IEEE-754 rule written
// out (a quiet NaN keeps its sign and the top bits of its payload) on every
// one of the 2^32 inputs, and costs one instruction where the bit rule
// costs about ten for the pair.
__device__ __forceinline__ uint32_t pack_bf16_rne(float a, float b) {
    const f32x2 v = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

// How y_f32 is stored (store_sums chooses): in whole lines, non-temporally or
// not, or by each thread at its own chunk. (They are kernels of their own: from
// the two sides of a branch the compiler makes one ordinary store.)
enum class Sums { kNone, kStream, kKeep, kDirect };

template <Sums kSums, int C>
__global__ __launch_bounds__(kMaxK * 64) void fold_kernel(
    const u32x4* __restrict__ eo, const int32_t* __restrict__ pos, const float* __restrict__ gates,
    int K, int64_t nch, int64_t TK, Slices cut, u32x4* __restrict__ y, float* __restrict__ y32) {
    // K slices of 64 * C chunks (K * C KiB, sized at launch): a small stage
    // lets further workgroups start on a CU once the loading waves of a
    // workgroup have exited, which the wave count alone would not limit
    extern __shared__ u32x4 stage[];
    __shared__ float gate[kMaxK];
    __shared__ int valid[kMaxK];
    uint32_t t, g;
    cut.split(blockIdx.x, &t, &g);
    const int j = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int64_t c0 = (int64_t)g * (64 * C) + lane;
    if (j < K) {
        const int p = pos[(int64_t)t * K + j];
        const bool ok = p >= 0 && p < TK;
        // all loads are issued before any LDS write: a write right after its
        // own load would make the next load wait for it
        const u32x4* row = eo + (int64_t)(ok ? p : 0) * nch;
        u32x4 v[C];
#pragma unroll
        for (int i = 0; i < C; ++i)
            if (ok && c0 + 64 * i < nch) v[i] = __builtin_nontemporal_load(row + c0 + 64 * i);
#pragma unroll
        for (int i = 0; i < C; ++i)
            if (ok && c0 + 64 * i < nch) stage[(j * C + i) * 64 + lane] = v[i];
        const float gj = gates[(int64_t)t * K + j];
        if (lane == 0) {
            valid[j] = ok;
            gate[j] = gj;
        }
    }
    __syncthreads();
    // C waves fold: thread i takes chunk i of the slice (eight bf16 values),
    // summing the K slots in slot order, and stores 16 bytes of y
    if (j >= C) return;
    const int i = threadIdx.x;
    const int64_t c = (int64_t)g * (64 * C) + i;
    if ((kSums == Sums::kNone || kSums == Sums::kDirect) && c >= nch) return;
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    for (int k = 0; k < K; ++k) {
        if (!valid[k]) continue;
        const float gk = gate[k];
        const u32x4 v = stage[k * (64 * C) + i];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            acc[2 * q] = __builtin_fmaf(gk, __uint_as_float(v[q] << 16), acc[2 * q]);
            acc[2 * q + 1] = __builtin_fmaf(gk, __uint_as_float(v[q] & 0xffff0000u), acc[2 * q + 1]);
        }
    }
    u32x4 out;
#pragma unroll
    for (int q = 0; q < 4; ++q)
        out[q] = pack_bf16_rne(acc[2 * q], acc[2 * q + 1]);
    if (c < nch) __builtin_nontemporal_store(out, y + (int64_t)t * nch + c);
    if constexpr (kSums == Sums::kDirect) {
        float4* o = reinterpret_cast<float4*>(y32 + ((int64_t)t * nch + c) * 8);
        o[0] = make_float4(acc[0], acc[1], acc[2], acc[3]);
        o[1] = make_float4(acc[4], acc[5], acc[6], acc[7]);
    } else if constexpr (kSums != Sums::kNone) {
        // The wave's 64 chunks are 128 16-byte pieces of y_f32; lane l stores
        // pieces l and 64 + l, so that each store covers whole lines (two
        // stores at its own chunk would each cover half of every line).
        const int64_t c_wave = (int64_t)g * (64 * C) + 64 * j;
        u32x4* o = reinterpret_cast<u32x4*>(y32) + ((int64_t)t * nch + c_wave) * 2;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int from = 32 * h + lane / 2;
            u32x4 piece;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float lo = __shfl(acc[q], from, 64), hi = __shfl(acc[4 + q], from, 64);
                piece[q] = __float_as_uint(lane & 1 ? hi : lo);
            }
            if (c_wave + from >= nch) continue;
            if constexpr (kSums == Sums::kStream)
                __builtin_nontemporal_store(piece, o + 64 * h + lane);
            else
                o[64 * h + lane] = piece;
        }
    }
}

// Each wave takes one (token, slice of 64 chunks) and loads the chunks of all
// K rows, issuing every load before its single store so that no load waits
// behind a store. KM: slots held in registers, at least K (kFull: exactly K).
constexpr int kDirectWaves = 16;

template <bool kF32, int KM, bool kFull>
__global__ __launch_bounds__(kDirectWaves * 64) void direct_kernel(
    const u32x4* __restrict__ eo, const int32_t* __restrict__ pos, const float* __restrict__ gates,
    int64_t T, int Kr, int64_t nch, int64_t TK, u32x4* __restrict__ y, float* __restrict__ y32) {
    const int K = kFull ? KM : Kr;
    const int64_t slices = (nch + 63) / 64;
    // wave-uniform item index, so pos and gates come in through scalar loads
    const int64_t item = (int64_t)blockIdx.x * kDirectWaves +
                         __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (item >= T * slices) return;
    const int64_t t = item / slices;
    const int64_t c = (item - t * slices) * 64 + (threadIdx.x & 63);
    int p[KM];
    float g[KM];
#pragma unroll
    for (int j = 0; j < KM; ++j) {
        p[j] = j < K ? pos[t * K + j] : -1;
        g[j] = j < K ? gates[t * K + j] : 0.f;
    }
    u32x4 v[KM];
    bool ok[KM];
#pragma unroll
    for (int j = 0; j < KM; ++j) {
        ok[j] = p[j] >= 0 && p[j] < TK && c < nch;
        if (ok[j]) v[j] = __builtin_nontemporal_load(eo + (int64_t)p[j] * nch + c);
    }
    if (c >= nch) return;
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < KM; ++j) {
        if (!ok[j]) continue;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            acc[2 * q] = __builtin_fmaf(g[j], __uint_as_float(v[j][q] << 16), acc[2 * q]);
            acc[2 * q + 1] =
                __builtin_fmaf(g[j], __uint_as_float(v[j][q] & 0xffff0000u), acc[2 * q + 1]);
        }
    }
    u32x4 out;
#pragma unroll
    for (int q = 0; q < 4; ++q)
        out[q] = pack_bf16_rne(acc[2 * q], acc[2 * q + 1]);
    __builtin_nontemporal_store(out, y + t * nch + c);
    if constexpr (kF32) {
        float4* o = reinterpret_cast<float4*>(y32 + (t * nch + c) * 8);
        o[0] = make_float4(acc[0], acc[1], acc[2], acc[3]);
        o[1] = make_float4(acc[4], acc[5], acc[6], acc[7]);
    }
}

// Node-level combine: one workgroup per (token, 2 KiB column slice), one wave
// per slot j (at least two waves). Wave j loads its row's slice like
// fold_kernel and records its gate and its rank's node; after a barrier two
// waves, one 16-byte chunk per thread, go through the token's node rows in
// node order: each is the sum of the node's slots in slot order, rounded to
// bf16, stored as the partial row's slice and added to y. The partials
// stay in registers on their way into y: with a second kernel that read the
// node rows back the call moved a third more bytes and took 5.6 ms on the
// T=131072, K=8, N=8, d=7168 workload (3.93 + 1.67), now 4.35 ms (5.8 TB/s of
// mixed reads and writes). One wave per node row, with the partials summed
// through LDS after a second barrier, took 4.46 ms; plain instead of
// non-temporal stores of the partial rows 4.42 ms. Without y the partial rows
// are all it writes, and node_sum_kernel follows.
template <int C>
__global__ __launch_bounds__(kMaxK * 64) void node_fold_kernel(
    const u32x4* __restrict__ eo, const int32_t* __restrict__ pos,
    const int32_t* __restrict__ assigned, const float* __restrict__ gates,
    const int32_t* __restrict__ node_pos, int K, int N, int gpn, int64_t nch, int64_t TK,
    int64_t node_rows, Slices cut, u32x4* __restrict__ partial, u32x4* __restrict__ y) {
    extern __shared__ u32x4 stage[];
    __shared__ float gate[kMaxK];
    __shared__ int slot_node[kMaxK];  // node of slot j's rank, -1 for a skipped slot
    uint32_t t, g;
    cut.split(blockIdx.x, &t, &g);
    const int j = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int64_t c0 = (int64_t)g * (64 * C) + lane;
    if (j < K) {
        const int p = pos[(int64_t)t * K + j];
        const int r = assigned[(int64_t)t * K + j];
        const bool ok = p >= 0 && p < TK && r >= 0 && r < N * gpn;
        const u32x4* row = eo + (int64_t)(ok ? p : 0) * nch;
        u32x4 v[C];
#pragma unroll
        for (int i = 0; i < C; ++i)
            if (ok && c0 + 64 * i < nch) v[i] = __builtin_nontemporal_load(row + c0 + 64 * i);
#pragma unroll
        for (int i = 0; i < C; ++i)
            if (ok && c0 + 64 * i < nch) stage[(j * C + i) * 64 + lane] = v[i];
        const float gj = gates[(int64_t)t * K + j];
        if (lane == 0) {
            gate[j] = gj;
            slot_node[j] = ok ? r / gpn : -1;
        }
    }
    // lane n of the folding waves holds the row of (t, n) in partial
    int row = -1;
    if (j < C && lane < N) {
        const int q = node_pos[(int64_t)t * N + lane];
        row = q >= 0 && q < node_rows ? q : -1;
    }
    __syncthreads();
    if (j >= C) return;
    const int i = threadIdx.x;
    const int64_t c = (int64_t)g * (64 * C) + i;
    const int node = lane < K ? slot_node[lane] : -1;  // lane k holds slot k's node and gate
    const int gk = lane < K ? __float_as_int(gate[lane]) : 0;
    float sum[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    for (uint64_t nodes = __ballot(row >= 0); nodes; nodes &= nodes - 1) {
        const int n = __builtin_ctzll(nodes);
        float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        for (uint64_t slots = __ballot(node == n); slots; slots &= slots - 1) {
            const int k = __builtin_ctzll(slots);
            const float gv = __int_as_float(__builtin_amdgcn_readlane(gk, k));
            const u32x4 v = stage[k * (64 * C) + i];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                acc[2 * e] = __builtin_fmaf(gv, __uint_as_float(v[e] << 16), acc[2 * e]);
                acc[2 * e + 1] =
                    __builtin_fmaf(gv, __uint_as_float(v[e] & 0xffff0000u), acc[2 * e + 1]);
            }
        }
        u32x4 part;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            part[e] = pack_bf16_rne(acc[2 * e], acc[2 * e + 1]);
            sum[2 * e] += __uint_as_float(part[e] << 16);
            sum[2 * e + 1] += __uint_as_float(part[e] & 0xffff0000u);
        }
        const int q = __builtin_amdgcn_readlane(row, n);
        if (c < nch) __builtin_nontemporal_store(part, partial + (int64_t)q * nch + c);
    }
    if (!y || c >= nch) return;
    u32x4 out;
#pragma unroll
    for (int e = 0; e < 4; ++e)
        out[e] = pack_bf16_rne(sum[2 * e], sum[2 * e + 1]);
    __builtin_nontemporal_store(out, y + (int64_t)t * nch + c);
}

// y from the partial rows, for a y in the memory of the expert rows (or of
// another input), which node_fold_kernel reads until its last workgroup: one
// wave per (token, slice of 64 chunks).
__global__ __launch_bounds__(kDirectWaves * 64) void node_sum_kernel(
    const u32x4* __restrict__ partial, const int32_t* __restrict__ node_pos, int64_t T, int N,
    int64_t nch, int64_t node_rows, u32x4* __restrict__ y) {
    const int64_t slices = (nch + 63) / 64;
    const int64_t item = (int64_t)blockIdx.x * kDirectWaves +
                         __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (item >= T * slices) return;
    const int64_t t = item / slices;
    const int64_t c = (item - t * slices) * 64 + (threadIdx.x & 63);
    float sum[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    for (int n = 0; n < N; ++n) {
        const int q = node_pos[t * N + n];
        if (q < 0 || q >= node_rows || c >= nch) continue;
        const u32x4 v = __builtin_nontemporal_load(partial + (int64_t)q * nch + c);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            sum[2 * e] += __uint_as_float(v[e] << 16);
            sum[2 * e + 1] += __uint_as_float(v[e] & 0xffff0000u);
        }
    }
    if (c >= nch) return;
    u32x4 out;
#pragma unroll
    for (int e = 0; e < 4; ++e)
        out[e] = pack_bf16_rne(sum[2 * e], sum[2 * e + 1]);
    __builtin_nontemporal_store(out, y + t * nch + c);
}

}  // namespace

// Below 2 MiB the time is latency, and the exchange between lanes that makes
// whole lines costs what it saves elsewhere (T = 290, K = 8, d = 1032 4.1 us
// without it, 4.8 with). Non-temporal stores are faster up to where the
// memory-side cache's reuse sets in (T = 2180, K = 3, d = 1032: 5.9 us against
// 6.9), past its size (T = 32768, K = 8, d = 7168: 866 against 901) and with
// many rows to read for each that is written (T = 8192, K = 16, d = 7168: 416
// against 440; T = 32768, K = 8, d = 512: 61.5 against 67.8). In between,
// ordinary stores leave the sums in that cache for the kernel that reads them
// and for the next call that writes them: T = 8192, d = 7168 take 194 us so
// with K = 8 and 74 with K = 2, 214 and 98 non-temporally.
static Sums store_sums(int64_t T, int K, int64_t d) {
    const int64_t bytes = T * d * 4;
    if (bytes < (2 << 20)) return Sums::kDirect;
    const bool cached = bytes >= (40 << 20) && bytes <= (256 << 20);
    return cached && K <= 12 && (d > 512 || K <= 4) ? Sums::kKeep : Sums::kStream;
}

// Whether direct_kernel folds the rows: only rows of more than 2048 chunks (d >
// 16384) in enough waves to fill the chip, where K > 12 makes fold_kernel's
// workgroups so large that two of them fill a CU's waves (K = 16, d = 20480: T
// = 64 8.3 us against 11.0, T = 1024 116 against 141; T = 16 6.2 against 4.8),
// or where all its waves are in flight at once (T = 64, d = 32768: K = 8 5.3
// us against 7.7, K = 12 8.0 against 10.2).
static bool direct_fold(int64_t T, int K, int64_t nch) {
    const int64_t waves = T * ((nch + 63) / 64);
    return nch > 2048 && K >= 8 && waves > 2048 && (K > 12 || waves <= 4096);
}

cobalt_status launch_combine(const void* eo, const int32_t* pos, const float* gates, int64_t T,
                             int K, int64_t d, void* y, float* y32, hipStream_t s) {
    const int64_t nch = d / 8;
    if (direct_fold(T, K, nch)) {
        const int64_t slices = (nch + 63) / 64;  // one wave each
        for_token_ranges(T, slices * 64, [&](int64_t t0, int64_t n) {
            const unsigned blocks = (unsigned)((n * slices + kDirectWaves - 1) / kDirectWaves);
            auto launch = [&](auto kernel) {
                hipLaunchKernelGGL(kernel, dim3(blocks), dim3(kDirectWaves * 64), 0, s,
                                   (const u32x4*)eo, pos + t0 * K, gates + t0 * K, n, K, nch,
                                   T * K, (u32x4*)y + t0 * nch,
                                   y32 ? y32 + t0 * nch * 8 : nullptr);
            };
            if (K == 8)
                y32 ? launch(direct_kernel<true, 8, true>) : launch(direct_kernel<false, 8, true>);
            else
                y32 ? launch(direct_kernel<true, kMaxK, false>)
                    : launch(direct_kernel<false, kMaxK, false>);
        });
        COBALT_LAUNCH_CHECK();
        return COBALT_OK;
    }
    const Sums sums = y32 ? store_sums(T, K, d) : Sums::kNone;
    // with one or two slots a fold of three chunks per lane has waves that load
    // nothing: T = 16384, K = 1, d = 1536 24.1 us, with two chunks 20.1 (but with
    // y_f32 T = 65536, K = 1, d = 1280 128.8 against 147.3)
    by_slices(nch, K < 3 && !y32 ? 2 : 3, [&](auto c, const Slices& cut) {
        constexpr int C = decltype(c)::value;
        const int threads = std::max(K, C) * 64;
        for_token_ranges(T, (int64_t)cut.slices * threads, [&](int64_t t0, int64_t n) {
            auto launch = [&](auto kernel) {
                hipLaunchKernelGGL(kernel, dim3((unsigned)(n * cut.slices)), dim3(threads),
                                   (size_t)K * 64 * C * sizeof(u32x4), s, (const u32x4*)eo,
                                   pos + t0 * K, gates + t0 * K, K, nch, T * K, cut,
                                   (u32x4*)y + t0 * nch, y32 ? y32 + t0 * nch * 8 : nullptr);
            };
            if (sums == Sums::kNone)
                launch(fold_kernel<Sums::kNone, C>);
            else if (sums == Sums::kStream)
                launch(fold_kernel<Sums::kStream, C>);
            else if (sums == Sums::kKeep)
                launch(fold_kernel<Sums::kKeep, C>);
            else
                launch(fold_kernel<Sums::kDirect, C>);
        });
    });
    COBALT_LAUNCH_CHECK();
    return COBALT_OK;
}

cobalt_status launch_node_combine(const void* eo, const int32_t* pos, const int32_t* assigned,
                                  const float* gates, const int32_t* node_pos, int64_t T, int K,
                                  int N, int gpn, int64_t d, void* partial, void* y,
                                  hipStream_t s) {
    const int64_t nch = d / 8;
    const int64_t node_rows = T * std::min(K, N);
    const bool apart = overlap(y, T * d * 2, eo, T * K * d * 2) ||
                       overlap(y, T * d * 2, pos, T * K * 4) ||
                       overlap(y, T * d * 2, assigned, T * K * 4) ||
                       overlap(y, T * d * 2, gates, T * K * 4);
    by_slices(nch, 3, [&](auto c, const Slices& cut) {
        constexpr int C = decltype(c)::value;
        const int threads = std::max(K, C) * 64;
        for_token_ranges(T, (int64_t)cut.slices * threads, [&](int64_t t0, int64_t n) {
            hipLaunchKernelGGL(node_fold_kernel<C>, dim3((unsigned)(n * cut.slices)), dim3(threads),
                               (size_t)K * 64 * C * sizeof(u32x4), s, (const u32x4*)eo,
                               pos + t0 * K, assigned + t0 * K, gates + t0 * K, node_pos + t0 * N,
                               K, N, gpn, nch, T * K, node_rows, cut, (u32x4*)partial,
                               apart ? nullptr : (u32x4*)y + t0 * nch);
        });
    });
    if (apart) {
        const int64_t slices = (nch + 63) / 64;  // one wave each
        for_token_ranges(T, slices * 64, [&](int64_t t0, int64_t n) {
            const unsigned blocks = (unsigned)((n * slices + kDirectWaves - 1) / kDirectWaves);
            hipLaunchKernelGGL(node_sum_kernel, dim3(blocks), dim3(kDirectWaves * 64), 0, s,
                               (const u32x4*)partial, node_pos + t0 * N, n, N, nch, node_rows,
                               (u32x4*)y + t0 * nch);
        });
    }
    COBALT_LAUNCH_CHECK();
    return COBALT_OK;
}

// ---------------------------------------------------------------- validation

namespace {

__global__ void zero_flag_kernel(uint32_t* f) { *f = 0; }

__global__ __launch_bounds__(256) void validate_kernel(const int32_t* __restrict__ topk,
                                                       const int32_t* __restrict__ src, int64_t T,
                                                       int K, int E, int G, uint32_t* flags) {
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (t >= T) return;
    uint32_t f = 0;
    for (int j = 0; j < K; ++j) {
        const int e = topk[t * K + j];
        if (e < 0 || e >= E) f |= 1u;
        for (int i = 0; i < j; ++i)
            if (topk[t * K + i] == e) f |= 2u;
    }
    if (src) {
        const int s = src[t];
        if (s < 0 || s >= G) f |= 4u;
        if (t > 0 && src[t - 1] > s) f |= 8u;
    }
    if (f) atomicOr(flags, f);
}

}  // namespace

cobalt_status launch_validate(const int32_t* topk, const int32_t* src, int64_t T, int K, int E,
                              int G, uint32_t* dflags, hipStream_t s) {
    hipLaunchKernelGGL(zero_flag_kernel, dim3(1), dim3(1), 0, s, dflags);
    COBALT_LAUNCH_CHECK();
    hipLaunchKernelGGL(validate_kernel, dim3((unsigned)((T + 255) / 256)), dim3(256), 0, s, topk,
                       src, T, K, E, G, dflags);
    COBALT_LAUNCH_CHECK();
    return COBALT_OK;
}

}  // namespace cobalt

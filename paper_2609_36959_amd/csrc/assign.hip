// Communication-aware task assignment (Section 3.3, Algorithm 1), one lane
// per token.
//
// Step 1 (select execution nodes): the token's experts without a replica on
// the source node form U_t, each with its remote-node mask m (N-1 bits, bit
// i = the i-th node other than the source node). Algorithm 1 keeps the first
// feasible cover in order of (node count, mask value). The search here
// reaches the same cover without a table:
//  - F, the union of the masks with a single node, is contained in every
//    feasible cover. If F meets every mask of U_t, no other cover has as few
//    nodes, so F is the answer.
//  - Otherwise the answer is F | S, where S is the first set, by (size,
//    value), that meets each of the masks F misses (F and S are disjoint, so
//    this is the order of F | S): first_cover, a depth-first search over the
//    masks in registers. Trying the sets of a size one by one, as Algorithm
//    1 states it, made every wave wait for its slowest lane's hundreds of
//    sets (131072 tokens, E = 512 on 16 nodes, 256 replicas: 4.1-4.3 ms a
//    call, now 24 us).
// Each expert of U_t then draws one of the cover's nodes holding it.
// Step 2 (select execution ranks): every task draws one rank of its node
// holding the expert. Draws hash the pair index with SplitMix64.
#include "cover.hpp"
#include "internal.hpp"

namespace cobalt {
namespace {

// One wave per workgroup: a call of 10007 tokens (a chain of dependent loads
// and little else) takes 6.6 us so, 8.6 in workgroups of four waves on a
// quarter as many CUs; from 65536 tokens on there is no difference.
constexpr int kAssignThreads = 64;

struct AssignArgs {
    const int32_t* topk;
    const int32_t* src;
    int64_t T;
    int64_t tok_per_src;
    int K, E, N, g, G, mode;
    uint64_t key;
    const uint32_t* node_mask;
    const uint32_t* rank_mask;
    const int32_t* owner;
    int32_t* out;
    uint16_t* remote;
};

__device__ __forceinline__ uint32_t draw(uint64_t key, int64_t p, uint32_t stream, uint32_t cnt) {
    if (cnt <= 1) return 0;
    const uint64_t h = splitmix64(key ^ (((uint64_t)p << 1) | stream));
    return (uint32_t)(((h >> 32) * (uint64_t)cnt) >> 32);
}

// position of the k-th (0-based) set bit of v
__device__ __forceinline__ int kth_bit(uint32_t v, uint32_t k) {
    for (uint32_t i = 0; i < k; ++i) v &= v - 1u;
    return __builtin_ctz(v);
}

// KM: slots held in registers, at least K. VEC: ids read and ranks written
// per access (4 ints where K and both pointers allow it, else 2, else 1).
template <int KM, int VEC>
__global__ __launch_bounds__(kAssignThreads) void assign_kernel(AssignArgs a) {
    const int64_t t = (int64_t)blockIdx.x * kAssignThreads + threadIdx.x;
    if (t >= a.T) return;
    const int K = a.K;
    const int64_t p0 = t * K;
    const int s = a.src ? a.src[t] : (int)((uint32_t)t / (uint32_t)a.tok_per_src);
    int e[KM], rr[KM];
#pragma unroll
    for (int j = 0; j < KM; ++j) e[j] = rr[j] = -1;
    if (s < 0 || s >= a.G) {
        store_row<KM, VEC>(a.out + p0, K, rr);
        if (a.remote) a.remote[t] = 0;
        return;
    }
    const int home = s / a.g;
    const uint32_t home_bit = 1u << home;
    const uint32_t low = home_bit - 1u;

    load_row<KM, VEC>(a.topk + p0, K, e);
#pragma unroll
    for (int j = 0; j < KM; ++j) e[j] = (uint32_t)e[j] < (uint32_t)a.E ? e[j] : -1;

    if (a.mode == 1) {  // owner-only baseline
        uint32_t nodes = 0;
#pragma unroll
        for (int j = 0; j < KM; ++j) {
            if (e[j] >= 0) {
                rr[j] = a.owner[e[j]];
                const int n = rr[j] / a.g;
                if (n != home) nodes |= 1u << n;
            }
        }
        store_row<KM, VEC>(a.out + p0, K, rr);
        if (a.remote) a.remote[t] = (uint16_t)nodes;
        return;
    }

    // Step 1: remote masks of U_t and the nodes every cover needs.
    uint32_t m[KM];
    uint32_t forced = 0;
#pragma unroll
    for (int j = 0; j < KM; ++j) {
        m[j] = 0;
        if (e[j] >= 0) {
            const uint32_t nm = a.node_mask[e[j]];
            if (!(nm & home_bit)) {
                m[j] = (nm & low) | ((nm >> (home + 1)) << home);
                if ((m[j] & (m[j] - 1u)) == 0) forced |= m[j];
            }
        }
    }
    uint32_t missed[KM];  // the masks the forced nodes miss
    bool search = false;
#pragma unroll
    for (int j = 0; j < KM; ++j) {
        missed[j] = (m[j] & forced) ? 0u : m[j];
        search = search || missed[j] != 0;
    }
    uint32_t bstar = forced;
    if (search) bstar |= first_cover<KM>(missed);

    // Node of each task, then its rank (Step 2).
#pragma unroll
    for (int j = 0; j < KM; ++j) {
        if (e[j] >= 0) {
            const int64_t p = p0 + j;
            int n = home;
            const uint32_t cand = bstar & m[j];  // empty only on invalid layouts
            if (m[j] && cand) {
                const int bit = kth_bit(cand, draw(a.key, p, 0, __builtin_popcount(cand)));
                n = bit + (bit >= home ? 1 : 0);
            }
            const uint32_t R = a.rank_mask[(int64_t)e[j] * a.N + n];
            if ((!m[j] || cand) && R)
                rr[j] = n * a.g + kth_bit(R, draw(a.key, p, 1, __builtin_popcount(R)));
        }
    }
    store_row<KM, VEC>(a.out + p0, K, rr);
    if (a.remote) a.remote[t] = (uint16_t)((bstar & low) | ((bstar >> home) << (home + 1)));
}

}  // namespace

cobalt_status launch_assign(const DeviceLayout& L, const int32_t* topk, const int32_t* src,
                            int64_t T, int K, uint64_t key, int mode, int32_t* out,
                            uint16_t* remote, hipStream_t s) {
    AssignArgs a;
    a.topk = topk;
    a.src = src;
    a.T = T;
    a.tok_per_src = src ? 1 : T / L.G;
    a.K = K;
    a.E = L.E;
    a.N = L.N;
    a.g = L.g;
    a.G = L.G;
    a.mode = mode;
    a.key = key;
    a.node_mask = L.node_mask;
    a.rank_mask = L.rank_mask;
    a.owner = L.owner;
    a.out = out;
    a.remote = remote;
    const unsigned blocks = (unsigned)((T + kAssignThreads - 1) / kAssignThreads);
    // both rows are accessed alike: `out` decides where it is the less aligned
    const uintptr_t o = (uintptr_t)out & 15u, q = (uintptr_t)topk & 15u;
    by_row(K, (const void*)(o | q), [&](auto km, auto vec) {
        hipLaunchKernelGGL((assign_kernel<decltype(km)::value, decltype(vec)::value>),
                           dim3(blocks), dim3(kAssignThreads), 0, s, a);
    });
    COBALT_LAUNCH_CHECK();
    return COBALT_OK;
}

}  // namespace cobalt

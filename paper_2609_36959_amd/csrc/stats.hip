// Co-activation statistics (Section 3.2, Stage 1): per-pair co-selection
// counts c_ij and per-expert task counts w_e, as raw uint32 increments.
//
// The unordered pairs i < j form a triangle of E(E-1)/2 bins. It is split
// into nb row bands, nb a power of two, with the rows interleaved: band b
// holds the rows i = b, b + nb, b + 2nb, ... Interleaving gives every band
// nearly the same number of bins and, since popular experts are spread over
// the ids, a similar share of the increments. In band b, local row r (i =
// r*nb + b) starts at
//     off_b(r) = r (E - 1 - b) - nb r (r - 1) / 2
// and bin (i, j) is off_b(r) + j - i - 1.
//
// Two kernels:
//   count   grid = chunks x bands. A workgroup takes a contiguous chunk of
//           tokens and keeps its band's bins, and the counts of the experts
//           e = b (mod nb), in LDS. Each thread loads a token's ids (16-byte
//           loads where K and the address allow it), sorts them in registers,
//           and for every sorted slot a whose expert is in the band adds one
//           to the bins (e[a], e[b]) of the later slots, with LDS atomics.
//           The band's bins are then written to the chunk's slot of the
//           workspace, as uint16 where no bin of a chunk can pass 65535,
//           else as uint32.
//   reduce  eight or sixteen lanes per group of eight band bins sum the group
//           over the chunks (lane k takes chunks k, k + lanes, ..., one
//           16-byte load of eight uint16 bins each), add pairwise across
//           lanes k and k + 8, then exchange halves in three shuffle rounds
//           so that lane k < 8 ends with the total of bin k, which it adds to
//           coact[i][j] and coact[j][i]. Other lanes do the same for
//           expert_count. Every output element has exactly one writer, so the
//           result does not depend on scheduling. With few chunks the
//           shuffles and the row search are most of the work, so the fewer
//           lanes, with the row from a square root, serve up to kFewChunks
//           (E = 1024, 16384 tokens: 24.5 to 22.8 us a call).
//
// Checks. Ids outside [0, E) count nowhere. A token that repeats an id adds
// the product of the multiplicities to a pair, and m (m - 1) to the
// diagonal entry of an id it holds m times: the diagonal is kept per band in
// LDS beside the counts and added to coact with one atomic per nonzero entry
// (top-k selections never repeat an id, so this costs nothing on real
// routing). When every token a wave holds has K distinct ids in range (the
// normal case, found with one ballot), the wave adds its pairs without
// per-pair tests.
//
// Small calls (E up to kDirectE, kDirectUpdates elements over all chunks)
// skip the reduce: each count workgroup goes through coact's elements and
// adds its nonzero bins with integer atomics, whose sums do not depend on
// their order, a whole line of a row per wave. 4096 tokens with E = 16, K = 2
// take 3.9 us so (7.4 with the reduce; 12.8 when the bins of the triangle
// were added one by one), 256 with E = 128, K = 8 7.4 (8.4; 11.1), 16384 with
// E = 64, K = 6 6.2 (8.9; 15.9). At E = 256 one workgroup's walk over 65536
// elements takes longer than the reduce (20.9 against 12.4 us for 256
// tokens).
//
// Chunks. A workgroup's LDS atomics queue on its CU, so chunks are short
// until the partials they add cost as much: 512 tokens (256 up to kDirectE),
// at most 128 chunks, and with many bands at most kMaxGroups workgroups, or
// twice as many where that keeps the bins uint16 in no more space. E = 1024,
// 131072 tokens, K = 8 in 16 bands take 55.9 us with 16 chunks of uint32
// bins, 70 with the 33 that make them uint16, 101 with 128; E = 256, 4096
// tokens 14.0 us in 8 chunks against 16.8 in 4.
#include <algorithm>
#include <climits>
#include <cmath>
#include <mutex>
#include <set>
#include <utility>

#include "internal.hpp"

namespace cobalt {
namespace {

constexpr int kCountThreads = 1024;
constexpr int kReduceThreads = 256;
constexpr int kMaxLgBands = 12;
constexpr int64_t kTokensPerChunk = 512;
constexpr int64_t kMaxChunks = 128;
constexpr int kParBands = 2;            // bands for parallelism on large calls
constexpr int64_t kParPairs = 1 << 18;  // T*K from which bands are used for parallelism
constexpr int64_t kMaxGroups = 256;
constexpr int kDirectE = 128;
constexpr int64_t kDirectUpdates = 262144;
constexpr int kFewChunks = 32;

struct Plan {
    int nchunks;
    int lgb;                // log2 of the number of bands
    bool u16;               // partial bins stored as uint16
    int64_t tok_per_chunk;
    int64_t band_stride;    // bins of the largest band (band 0), rounded up to 8
    int32_t cnt_off;        // LDS word of the band's expert counts (then its diagonal)
    size_t lds_bytes;
    size_t part_bytes;      // partial pair histograms
    size_t count_bytes;     // partial expert counts
};

size_t align256(size_t v) { return (v + 255) & ~size_t(255); }
int64_t round_up(int64_t v, int64_t m) { return (v + m - 1) / m * m; }

// Rows of band b: i = r*nb + b < E - 1.
__host__ __device__ inline int32_t band_rows(int32_t E, int32_t nb, int32_t b) {
    return b < E - 1 ? (E - 1 - b + nb - 1) / nb : 0;
}
// Start of local row r of band b.
__host__ __device__ inline int32_t band_off(int32_t E, int32_t nb, int32_t b, int32_t r) {
    return r * (E - 1 - b) - nb * (r * (r - 1) / 2);
}
__host__ __device__ inline int32_t band_words(int32_t E, int32_t nb, int32_t b) {
    return band_off(E, nb, b, band_rows(E, nb, b));
}

// LDS words of band 0 (the largest) and of its expert counts (or diagonal)
// with nb bands, rounded up for 16-byte accesses.
int64_t hist_words(int E, int nb) { return round_up(std::max(band_words(E, nb, 0), 1), 8); }
int64_t cnt_words(int E, int nb) { return round_up((E + nb - 1) / nb, 4); }

bool make_plan(int64_t T, int64_t K, int E, int lds_bytes, Plan* p) {
    const int64_t lds_words = lds_bytes / 4;
    auto fits = [&](int l) { return hist_words(E, 1 << l) + 2 * cnt_words(E, 1 << l) <= lds_words; };
    // fewest bands whose largest band and counts fit the LDS
    int lgb = 0;
    while (lgb <= kMaxLgBands && !fits(lgb)) ++lgb;
    if (lgb > kMaxLgBands) return false;
    // large calls: more bands, for more workgroups (at most one row per band)
    if (T * K >= kParPairs)
        while ((1 << lgb) < kParBands && (1 << (lgb + 1)) <= std::max(E - 1, 1)) ++lgb;
    // Chunks of about kTokensPerChunk tokens, up to kMaxChunks, and no more
    // than make kMaxGroups workgroups: each chunk adds a whole triangle to
    // the partials that are written and read back.
    const int64_t most = std::max<int64_t>(1, std::min(kMaxChunks, kMaxGroups >> lgb));
    p->nchunks = (int)std::min(most, std::max<int64_t>(1, T / (E <= kDirectE ? kTokensPerChunk / 2
                                                                            : kTokensPerChunk)));
    p->tok_per_chunk = std::max<int64_t>(1, (T + p->nchunks - 1) / p->nchunks);
    // A token adds at most floor(K/2) * ceil(K/2) to one bin (two experts,
    // each repeated), so chunks of up to 65535 / that product tokens have
    // uint16 bins. Where the chunks above are longer, more of them are used,
    // if that takes no more space than these in uint32: the workspace then
    // never shrinks as T or K grows, and one of the size for a program's
    // largest call serves its smaller ones (without the bound on space, E =
    // 1024, K = 8 asked for 142 MB at 520000 tokens, 34 MB at 540000), and
    // many bands are no slower for it: E = 1024, 262144 tokens 72.6 us
    // against 105.7 in 65 uint16 chunks, E = 4096, 131072 277 against 657.
    const int nb = 1 << lgb;
    p->band_stride = hist_words(E, nb);
    const auto part = [&](int64_t chunks, int bytes) {
        return align256((size_t)chunks * nb * p->band_stride * bytes);
    };
    const auto counts = [&](int64_t chunks) { return align256((size_t)chunks * E * 4); };
    const int64_t maxpair = (K / 2) * ((K + 1) / 2);
    const int64_t tok16 = maxpair ? 65535 / maxpair : T + 1;
    p->u16 = p->tok_per_chunk <= tok16;
    if (!p->u16) {
        const int64_t n16 = (T + tok16 - 1) / tok16;
        if (n16 <= kMaxChunks &&
            part(n16, 2) + counts(n16) <= part(p->nchunks, 4) + counts(p->nchunks)) {
            p->nchunks = (int)n16;
            p->tok_per_chunk = (T + n16 - 1) / n16;
            p->u16 = true;
        }
    }
    p->lgb = lgb;
    p->cnt_off = (int32_t)p->band_stride;
    p->lds_bytes = (size_t)(p->band_stride + 2 * cnt_words(E, nb)) * 4;
    p->part_bytes = part(p->nchunks, p->u16 ? 2 : 4);
    p->count_bytes = counts(p->nchunks);
    return true;
}

// Local row of bin w of band b: the last r with off_b(r) <= w, from the root
// of the quadratic off_b, set right by a step or two where it is rounded.
__device__ __forceinline__ int32_t band_row_of(int32_t E, int32_t nb, int32_t b, int32_t w) {
    const float h = (float)(2 * (E - 1 - b) + nb);
    const float q = fmaxf(h * h - 8.0f * (float)nb * (float)w, 0.0f);
    int32_t r = (int32_t)((h - sqrtf(q)) / (float)(2 * nb));
    r = max(0, min(r, band_rows(E, nb, b) - 1));
    while (r > 0 && band_off(E, nb, b, r) > w) --r;
    while (r + 1 < band_rows(E, nb, b) && band_off(E, nb, b, r + 1) <= w) ++r;
    return r;
}

__device__ __forceinline__ void cswap(int& a, int& b) {
    const int lo = min(a, b), hi = max(a, b);
    a = lo;
    b = hi;
}

// Sorts e[0..KM) ascending, KM a power of two: Batcher's odd-even merge sort
// network (5 comparators for 4, 19 for 8, 63 for 16).
template <int KM>
__device__ __forceinline__ void sort_ids(int (&e)[KM]) {
#pragma unroll
    for (int p = 1; p < KM; p *= 2)
#pragma unroll
        for (int k = p; k >= 1; k /= 2)
#pragma unroll
            for (int j = k % p; j + k < KM; j += 2 * k)
#pragma unroll
                for (int i = 0; i < k; ++i)
                    if (i + j + k < KM && (i + j) / (2 * p) == (i + j + k) / (2 * p))
                        cswap(e[i + j], e[i + j + k]);
}

// Loads token t's ids into e (INT_MAX past K).
template <int KM, int VEC>
__device__ __forceinline__ void load_ids(const int32_t* __restrict__ topk, int64_t t, int K,
                                         int (&e)[KM]) {
#pragma unroll
    for (int a = 0; a < KM; ++a) e[a] = INT_MAX;
    load_row<KM, VEC>(topk + t * K, K, e);
}

// One token of the count kernel: its counts, pairs and repeats in band `band`.
template <int KM>
__device__ __forceinline__ void count_token(int (&e)[KM], int K, int E, int lgb, int band,
                                            int32_t row_len0, uint32_t* hist, uint32_t* cnt,
                                            uint32_t* diag) {
    const int nb = 1 << lgb;
#pragma unroll
    for (int a = 0; a < KM; ++a)
        if ((uint32_t)e[a] >= (uint32_t)E) e[a] = INT_MAX;
#pragma unroll
    for (int a = 0; a < KM; ++a)
        if (e[a] != INT_MAX && (e[a] & (nb - 1)) == band) atomicAdd(&cnt[e[a] >> lgb], 1u);
    sort_ids<KM>(e);
    // K distinct ids in range: strictly increasing, the K-th not INT_MAX
    bool ok = true;
#pragma unroll
    for (int a = 0; a < KM; ++a)
        if (a < K) ok = ok && e[a] != INT_MAX && (a == 0 || e[a > 0 ? a - 1 : 0] < e[a]);
    if (__builtin_amdgcn_ballot_w64(!ok) == 0) {  // one value for the wave
#pragma unroll
        for (int a = 0; a + 1 < KM; ++a) {
            const int i = e[a];
            if (a + 1 >= K || (i & (nb - 1)) != band) continue;
            const int32_t r = i >> lgb;
            const int32_t base = r * row_len0 - nb * (r * (r - 1) / 2) - i - 1;
#pragma unroll
            for (int b = a + 1; b < KM; ++b)
                if (b < K) atomicAdd(&hist[base + e[b]], 1u);
        }
    } else {
#pragma unroll
        for (int a = 0; a < KM; ++a) {
            const int i = e[a];
            if (i == INT_MAX || (i & (nb - 1)) != band) continue;
            const int32_t r = i >> lgb;
            const int32_t base = r * row_len0 - nb * (r * (r - 1) / 2) - i - 1;
            int m = 1;  // copies of i from slot a on (they follow a, sorted)
#pragma unroll
            for (int b = a + 1; b < KM; ++b) {
                const int j = e[b];
                if (j == i)
                    ++m;
                else if (j != INT_MAX)
                    atomicAdd(&hist[base + j], 1u);
            }
            const bool first = a == 0 || e[a > 0 ? a - 1 : 0] != i;
            if (first && m > 1) atomicAdd(&diag[i >> lgb], (uint32_t)(m * (m - 1)));
        }
    }
}

// KM: ids held in registers, at least K (kFull: exactly K, so that no slot is
// tested for); VEC: ids per load (load_row). Ids outside [0, E) sort last as
// INT_MAX and count nowhere. U16: partial bins written as uint16. A thread
// takes two tokens per iteration and issues both loads before either is
// counted.
template <int KM, int VEC, bool kFull, bool U16>
__global__ __launch_bounds__(kCountThreads) void coact_count_kernel(
    const int32_t* __restrict__ topk, int64_t T, int Kr, int E, int lgb, int nchunks,
    int64_t tok_per_chunk, int64_t band_stride, int cnt_off, void* __restrict__ part,
    uint32_t* __restrict__ cpart, bool direct, uint32_t* __restrict__ coact,
    uint32_t* __restrict__ count) {
    const int K = kFull ? KM : Kr;
    extern __shared__ uint32_t lds[];
    const int nb = 1 << lgb;
    const int chunk = blockIdx.x % nchunks;
    const int band = blockIdx.x / nchunks;
    const int32_t ncnt = band < E ? (E - band + nb - 1) / nb : 0;
    const int32_t row_len0 = E - 1 - band;  // length of local row 0
    uint32_t* hist = lds;
    uint32_t* cnt = lds + cnt_off;
    uint32_t* diag = cnt + (((E + nb - 1) / nb + 3) & ~3);

    // band_stride and the count words are multiples of 4 words
    const int32_t lds_words = (int32_t)(diag - lds) + ((ncnt + 3) & ~3);
    for (int32_t w = threadIdx.x * 4; w < lds_words; w += kCountThreads * 4)
        *reinterpret_cast<u32x4*>(lds + w) = u32x4{0u, 0u, 0u, 0u};
    __syncthreads();

    const int64_t t0 = (int64_t)chunk * tok_per_chunk;
    const int64_t t1 = min(T, t0 + tok_per_chunk);
    for (int64_t t = t0 + threadIdx.x; t < t1; t += 2 * kCountThreads) {
        const int64_t u = t + kCountThreads;
        int e[KM], f[KM];
        load_ids<KM, VEC>(topk, t, K, e);
        if (u < t1) load_ids<KM, VEC>(topk, u, K, f);
        count_token<KM>(e, K, E, lgb, band, row_len0, hist, cnt, diag);
        if (u < t1) count_token<KM>(f, K, E, lgb, band, row_len0, hist, cnt, diag);
    }
    __syncthreads();

    if (direct) {  // one band: the chunk's bins go straight to the outputs
        // Thread by thread over coact's elements, so that both triangles are
        // added to in whole lines.
        const SmallDiv by_e = divide_by(E);
        for (int32_t x = threadIdx.x; x < E * E; x += kCountThreads) {
            const int32_t i = by_e(x), j = x - i * E;
            const int32_t lo = min(i, j), hi = max(i, j);
            const uint32_t v = i == j ? diag[i] : hist[band_off(E, 1, 0, lo) + hi - lo - 1];
            if (v) atomicAdd(&coact[x], v);
        }
        for (int32_t k = threadIdx.x; k < ncnt; k += kCountThreads)
            if (count && cnt[k]) atomicAdd(&count[k], cnt[k]);
        return;
    }

    // Write-out: thread g takes bins [8g, 8g + 8). Written through the L2:
    // the count kernel takes 21.0 us instead of 23.9 on T = 262144, E = 384
    // (18.8 MB of partials), 12.1 instead of 14.0 on T = 131072, E = 256.
    const int32_t groups = (int32_t)(band_stride / 8);
    const int64_t at = ((int64_t)band * nchunks + chunk) * band_stride;
    const int32_t bytes = (int32_t)band_stride * (U16 ? 2 : 4);
    void* out = static_cast<char*>(part) + at * (U16 ? 2 : 4);
    for (int32_t g = threadIdx.x; g < groups; g += kCountThreads) {
        const u32x4 lo = *reinterpret_cast<const u32x4*>(lds + g * 8);
        const u32x4 hi = *reinterpret_cast<const u32x4*>(lds + g * 8 + 4);
        if constexpr (U16) {
            const u32x4 packed = {lo.x | (lo.y << 16), lo.z | (lo.w << 16), hi.x | (hi.y << 16),
                                  hi.z | (hi.w << 16)};
            store_through(packed, out, bytes, g * 16);
        } else {
            store_through(lo, out, bytes, g * 32);
            store_through(hi, out, bytes, g * 32 + 16);
        }
    }
    for (int32_t k = threadIdx.x; k < ncnt; k += kCountThreads) {
        cpart[(int64_t)chunk * E + k * nb + band] = cnt[k];
        const int64_t ex = (int64_t)k * nb + band;
        if (diag[k]) atomicAdd(&coact[ex * E + ex], diag[k]);
    }
}

// Items [0, nb * band_stride / 8) are groups of eight band bins, then E
// expert counts; kReduceLanes lanes per item, lane k summing chunks k,
// k + kReduceLanes, ...
template <bool U16, int kReduceLanes>
__global__ __launch_bounds__(kReduceThreads) void coact_reduce_kernel(
    const void* __restrict__ part, const uint32_t* __restrict__ cpart, int E, int lgb,
    int nchunks, int64_t band_stride, bool do_count, uint32_t* __restrict__ coact,
    uint32_t* __restrict__ count) {
    static_assert(kReduceLanes >= 8 && kReduceLanes <= 64 && (kReduceLanes & (kReduceLanes - 1)) == 0,
                  "a power of two of at least eight lanes");
    const int nb = 1 << lgb;
    const int64_t groups_per_band = band_stride / 8;
    const int64_t ngroups = (int64_t)nb * groups_per_band;
    const int64_t gid = (int64_t)blockIdx.x * kReduceThreads + threadIdx.x;
    const int64_t item = gid / kReduceLanes;
    const int k = (int)(gid % kReduceLanes);
    if (item < ngroups) {
        const int band = (int)(item / groups_per_band);
        const int32_t w0 = (int32_t)(item % groups_per_band) * 8;
        // The bin of lane k < 8 and its two outputs, read before the
        // partials so that both loads are in flight together; lanes from 8 on
        // help with the sums only.
        const int32_t w = w0 + (k & 7);
        const bool real = k < 8 && w < band_words(E, nb, band);
        int64_t ij = 0, ji = 0;
        uint32_t cij = 0, cji = 0;
        if (real) {
            const int32_t r = band_row_of(E, nb, band, w);
            const int32_t i = r * nb + band;
            const int32_t j = w - band_off(E, nb, band, r) + i + 1;
            ij = (int64_t)i * E + j;
            ji = (int64_t)j * E + i;
            cij = coact[ij];
            cji = coact[ji];
        }
        uint32_t s[8] = {0, 0, 0, 0, 0, 0, 0, 0};
        const int64_t base = (int64_t)band * nchunks * band_stride + w0;
        if constexpr (U16) {
            const uint16_t* src = static_cast<const uint16_t*>(part) + base;
#pragma unroll 8
            for (int c = k; c < nchunks; c += kReduceLanes) {
                const u32x4 v = *reinterpret_cast<const u32x4*>(src + (int64_t)c * band_stride);
#pragma unroll
                for (int h = 0; h < 4; ++h) {
                    s[2 * h] += v[h] & 0xffffu;
                    s[2 * h + 1] += v[h] >> 16;
                }
            }
        } else {
            const uint32_t* src = static_cast<const uint32_t*>(part) + base;
#pragma unroll 4
            for (int c = k; c < nchunks; c += kReduceLanes) {
                const u32x4* q = reinterpret_cast<const u32x4*>(src + (int64_t)c * band_stride);
                const u32x4 lo = q[0], hi = q[1];
#pragma unroll
                for (int h = 0; h < 4; ++h) {
                    s[h] += lo[h];
                    s[4 + h] += hi[h];
                }
            }
        }
        // Lanes k, k ^ 8, k ^ 16, ... add their sums, then three rounds each
        // halve the bins a lane holds: the lane keeps the half its bit
        // selects and adds the partner's sums of that half. Lane k ends with
        // the total of bin w0 + k % 8.
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
        const uint32_t sum = s[0];
        if (sum == 0 || !real) return;
        coact[ij] = cij + sum;
        coact[ji] = cji + sum;
    } else if (do_count && item < ngroups + E) {
        const int e = (int)(item - ngroups);
        uint32_t sum = 0;
#pragma unroll 8
        for (int c = k; c < nchunks; c += kReduceLanes) sum += cpart[(int64_t)c * E + e];
#pragma unroll
        for (int o = 1; o < kReduceLanes; o <<= 1) sum += __shfl_xor(sum, o, kReduceLanes);
        if (k == 0 && sum != 0) count[e] += sum;
    }
}

}  // namespace

size_t coact_workspace_bytes(int64_t T, int K, int E, int lds_bytes) {
    Plan p;
    if (!make_plan(T, K, E, lds_bytes, &p)) return 0;
    return p.part_bytes + p.count_bytes;
}

cobalt_status launch_coact_stats(const int32_t* topk, int64_t T, int K, int E, uint32_t* coact,
                                 uint32_t* count, void* ws, size_t ws_bytes, hipStream_t s) {
    DeviceInfo di;
    if (cobalt_status st = device_info(&di)) return st;
    Plan p;
    if (!make_plan(T, K, E, di.lds_bytes, &p)) return COBALT_EUNSUPPORTED;
    if (ws_bytes < p.part_bytes + p.count_bytes) return COBALT_EINVAL;
    const int nb = 1 << p.lgb;
    const bool direct = nb == 1 && E <= kDirectE && (int64_t)p.nchunks * E * E <= kDirectUpdates;
    void* part = ws;
    uint32_t* cpart = (uint32_t*)((char*)ws + p.part_bytes);
    // The LDS limit of each kernel is raised to the device maximum once per
    // device (host-side only, so the calls stay capturable).
    cobalt_status st = COBALT_OK;
    auto launch = [&](auto kernel) {
        static std::mutex mu;
        static std::set<std::pair<const void*, int>> raised;
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess) {
            st = COBALT_EHIP;
            return;
        }
        {
            std::lock_guard<std::mutex> lock(mu);
            if (!raised.count({(const void*)kernel, dev})) {
                if (hipFuncSetAttribute((const void*)kernel,
                                        hipFuncAttributeMaxDynamicSharedMemorySize,
                                        di.lds_bytes) != hipSuccess) {
                    st = COBALT_EHIP;
                    return;
                }
                raised.insert({(const void*)kernel, dev});
            }
        }
        hipLaunchKernelGGL(kernel, dim3((unsigned)(p.nchunks * nb)), dim3(kCountThreads),
                           p.lds_bytes, s, topk, T, K, E, p.lgb, p.nchunks, p.tok_per_chunk,
                           p.band_stride, p.cnt_off, part, cpart, direct, coact, count);
    };
    by_row(K, topk, [&](auto km, auto vec) {
        constexpr int KM = decltype(km)::value, V = decltype(vec)::value;
        if (K == KM)
            p.u16 ? launch(coact_count_kernel<KM, V, true, true>)
                  : launch(coact_count_kernel<KM, V, true, false>);
        else
            p.u16 ? launch(coact_count_kernel<KM, V, false, true>)
                  : launch(coact_count_kernel<KM, V, false, false>);
    });
    if (st != COBALT_OK) return st;
    COBALT_LAUNCH_CHECK();
    if (direct) return COBALT_OK;
    const int64_t items = (int64_t)nb * (p.band_stride / 8) + (count ? E : 0);
    auto reduce = [&](auto kernel, int lanes) {
        hipLaunchKernelGGL(kernel,
                           dim3((unsigned)((items * lanes + kReduceThreads - 1) / kReduceThreads)),
                           dim3(kReduceThreads), 0, s, part, cpart, E, p.lgb, p.nchunks,
                           p.band_stride, count != nullptr, coact, count);
    };
    if (p.nchunks <= kFewChunks)
        p.u16 ? reduce(coact_reduce_kernel<true, 8>, 8) : reduce(coact_reduce_kernel<false, 8>, 8);
    else
        p.u16 ? reduce(coact_reduce_kernel<true, 16>, 16)
              : reduce(coact_reduce_kernel<false, 16>, 16);
    COBALT_LAUNCH_CHECK();
    return COBALT_OK;
}

}  // namespace cobalt

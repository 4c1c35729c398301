// The smallest set of nodes that meets every mask: the search inside
// Algorithm 1's node selection.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace cobalt {

typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));

__host__ __device__ inline u16x2 splat16(uint32_t v) {
    return u16x2{(uint16_t)v, (uint16_t)v};
}
// 0xffff in the halves where v is zero, 0 in the others.
__host__ __device__ inline u16x2 zero_halves(u16x2 v) {
    return __builtin_elementwise_min(v, splat16(1)) - splat16(1);
}

// First set of bits, in the order (size, value), that meets every non-zero
// mask of m (at least one is non-zero; masks use bits 0..14, the remote
// nodes of up to 16).
//
// Depth-first search by size c, from a lower bound of the size up. At each
// step the sets that can still win agree on all nodes decided so far, and
// the highest node that some unmet mask can still use is decided next, left
// out before it is taken; so the first set found is the smallest value of
// the smallest size. D holds the nodes taken by decision, X those left out
// by decision, S and E what follows from them:
//  - the only usable node of an unmet mask is taken (S);
//  - a node that a single unmet mask can use gives way to the mask's lowest
//    usable node, which does as much at a lower value (E);
//  - a node no unmet mask can use is in no smallest set;
//  - with one node to go, the nodes common to all unmet masks decide at once.
// Decisions go down in node order, so the last node left out is the lowest
// bit of X: on a branch masks only get met and nodes only drop out, so the
// highest usable node only falls. A dead end takes that last node instead and
// forgets every lower decision, and S and E with them, since they may follow
// from what is undone. A decision waits until a pass derives nothing more, so
// what S and E held before the undone decision has followed again from the
// decisions that stand, and one mask is met besides: the next decision is
// below the node again (so it was on 340 million decisions for 300 million
// random sets of masks, 8 and 16 of them over up to 15 nodes).
//
// A pass is straight-line code on pairs of 16-bit masks, about 100
// instructions for eight masks, and the wave runs as many passes as its
// slowest lane: 12 on average where 131072 tokens have about seven two-node
// masks over 15 nodes (32, and up to 94, without the rule for E).
template <int KM>
__host__ __device__ inline uint32_t first_cover(const uint32_t (&m)[KM]) {
    static_assert(KM % 2 == 0, "masks are held in pairs");
    constexpr uint32_t kPad = 0x8000u;  // stands for "no mask", met from the start
    uint32_t all = 0xffffu, used = 0;
    int c = 0;  // disjoint masks found: no smaller set meets them all
    u16x2 q[KM / 2];
#pragma unroll
    for (int j = 0; j < KM; ++j) {
        const bool none = m[j] == 0;
        all &= none ? 0xffffu : m[j];
        const bool apart = (m[j] & used) == 0 && !none;
        c += apart;
        used |= apart ? m[j] : 0u;
        q[j / 2][j % 2] = (uint16_t)(none ? kPad : m[j]);
    }
    if (all) return all & (0u - all);
    c = c < 2 ? 2 : c;
    uint32_t S = 0, D = 0, X = 0, E = 0;
    for (;;) {
        const u16x2 s2 = splat16(S | kPad), free2 = splat16(~(X | E));
        u16x2 usable = splat16(0), twice = splat16(0), forced = splat16(0), upper = splat16(0);
        u16x2 common = splat16(0xffff), least = splat16(0xffff);
#pragma unroll
        for (int j = 0; j < KM / 2; ++j) {
            const u16x2 unmet = zero_halves(q[j] & s2);
            const u16x2 a = q[j] & free2 & unmet;  // nodes the mask can still use
            twice |= usable & a;
            usable |= a;
            const u16x2 a1 = a | ~unmet;  // all ones for a met mask
            common &= a1;
            least = __builtin_elementwise_min(least, a1);
            const u16x2 rest = a & (a - splat16(1));  // all but the lowest
            upper |= rest;
            forced |= a & zero_halves(rest);
        }
        const uint32_t use = usable[0] | usable[1];
        const uint32_t more = twice[0] | twice[1] | (usable[0] & usable[1]);
        const uint32_t both = common[0] & common[1];
        const uint32_t take = forced[0] | forced[1];
        const uint32_t drop = (upper[0] | upper[1]) & ~more;
        const int left = c - __builtin_popcount(S);
        bool dead = least[0] == 0 || least[1] == 0;
        if (use == 0 && !dead) return S;
        dead = dead || left <= 0 || __builtin_popcount(take) > left;
        if (!dead && left == 1 && both != 0) return S | (both & (0u - both));
        dead = dead || left == 1;
        const uint32_t back = X & (0u - X);
        const uint32_t D1 = (D & ~(back - 1u)) | back;  // 0 if nothing is left to undo
        const bool decide = (take | drop) == 0;
        c += dead && X == 0;
        S = dead ? D1 : S | take;
        E = dead ? 0u : E | drop;
        D = dead ? D1 : D;
        X = dead ? X ^ back : decide ? X | (0x80000000u >> __builtin_clz(use)) : X;
    }
}

}  // namespace cobalt

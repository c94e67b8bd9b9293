// A segment of the recorded paths (its layout is described in internal.h) as the
// kernels that read them see it: the products (paths.hip) and the row tiles' build
// (tiles.hip).
#pragma once

#include "internal.h"
#include "pair.h"

namespace rrt {

// One wave's view of a segment.
struct Segment {
    uint32_t n_vis, n_slots, n_groups, words;
    const uint32_t* vis;
    const float4* fac;
    const uint32_t* abc;                  // three slots, entries in use less one
    const uint16_t* dr;                   // the fourth slot, the ray
};

__device__ __forceinline__ Segment segment_of(const uint4* __restrict__ s, const uint4 h)
{
    Segment g;
    g.n_vis = __builtin_amdgcn_readfirstlane(h.x & 0xffffu);
    g.n_slots = __builtin_amdgcn_readfirstlane(h.x >> 16);
    g.n_groups = __builtin_amdgcn_readfirstlane(h.y);
    g.words = __builtin_amdgcn_readfirstlane(h.z);
    const uint4* p = s + 1 + (g.n_vis + 3) / 4;
    g.vis = reinterpret_cast<const uint32_t*>(s + 1);
    g.fac = reinterpret_cast<const float4*>(p);
    g.abc = reinterpret_cast<const uint32_t*>(p + g.n_groups);
    g.dr = reinterpret_cast<const uint16_t*>(p + g.n_groups + (g.n_groups + 3) / 4);
    return g;
}

__device__ __forceinline__ Segment segment_at(const uint4* __restrict__ s)
{
    return segment_of(s, s[0]);
}

// f(slot, particle) for every slot of the segment's visits: 16 lanes per
// visit, four visits at a time.
// w0: the lane's word of the first 64 visits (whatever it reads past them).
// Wave `part` of `parts` takes its share of them.
template <typename F>
__device__ __forceinline__ void for_slots(const Segment& g, int lane, uint32_t w0, F f,
                                          uint32_t part = 0, uint32_t parts = 1)
{
    for (uint32_t v0 = 0; v0 < g.n_vis; v0 += 64) {
        const uint32_t w = v0 + lane >= g.n_vis ? 0u : v0 == 0 ? w0 : g.vis[v0 + lane];
        uint32_t c = v0 + lane < g.n_vis ? (w & (kLeafMax - 1)) + 1u : 0u;
        // (the running slot count of the visits before v0 is only needed when
        // a segment has more than 64 visits)
        uint32_t incl = c;
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t y = __shfl_up(incl, off, 64);
            if (lane >= off) incl += y;
        }
        uint32_t base0 = 0;
        if (v0 > 0) {
            for (uint32_t v = lane; v < v0; v += 64) base0 += (g.vis[v] & (kLeafMax - 1)) + 1u;
            for (int off = 32; off > 0; off >>= 1) base0 += __shfl_xor(base0, off, 64);
        }
        const uint32_t excl = base0 + incl - c;
        const uint32_t nv = g.n_vis - v0 < 64u ? g.n_vis - v0 : 64u;
        const uint32_t q = lane & 15;
        for (uint32_t s = 4 * part; s < nv; s += 4 * parts) {
            const int src = (int)s + (lane >> 4);
            const uint32_t ws = __shfl(w, src, 64), b = __shfl(excl, src, 64);
            if ((uint32_t)src < nv && q <= (ws & (kLeafMax - 1)))
                f(b + q, (int)(ws >> kLeafShift) + (int)q);
        }
    }
}

}  // namespace rrt

// Work items of the matrix-core M2L kernels: which (tile group, slot) pairs a
// block runs (the items and teams are described at k_m2l_mma).
#pragma once
#include "common.hpp"

namespace hfmm {

// bits of m whose rank among the set bits, counted from `base`, lies in
// [lo, hi)
__device__ inline uint32_t m2l_rank_range(uint32_t m, int base, int lo, int hi) {
    for (int k = base; m && k < lo; ++k) m &= m - 1u;  // drop ranks below lo
    uint32_t keep = 0u;
    for (int k = max(base, lo); m && k < hi; ++k) {
        const uint32_t low = m & (0u - m);
        keep |= low;
        m ^= low;
    }
    return keep;
}

// This block's range of work items and the group of its first item (the
// items and teams are described at k_m2l_mma).  Workgroups are handed to
// the 8 XCDs round-robin: with gw = 8, workgroups x, x + 8, ..., x + 56 of
// each run of 64 are a team (all on XCD x); with gw = 1 each XCD (own L2)
// runs one contiguous range of blocks, i.e. of items.  A workgroup past the
// last team gets no items.
struct M2lItems {
    int b, o, item, iend, group;
    int64_t W;
};
__device__ inline M2lItems m2l_items(const int32_t* __restrict__ gpre, int ngroups, int gw,
                                     int nb) {
    M2lItems it;
    const int lin = blockIdx.x;
    if (gw == 8) {
        it.b = (lin >> 6) * 8 + (lin & 7);
        it.o = (lin >> 3) & 7;
    } else {
        const int xcd = lin & 7, q8 = nb >> 3, r8 = nb & 7;
        it.b = xcd * q8 + min(xcd, r8) + (lin >> 3);
        it.o = 0;
    }
    it.W = gpre[ngroups];
    it.item = (int)((int64_t)it.b * it.W / nb);
    it.iend = it.b < nb ? (int)((int64_t)(it.b + 1) * it.W / nb) : it.item;
    // the last group with gpre[group] <= item: a 64-way search, every lane
    // probing one point of [lo, hi) per round (gpre[lo] <= item < gpre[hi])
    const int lane = threadIdx.x & 63;
    int lo = 0, hi = ngroups;
    while (hi - lo > 1) {
        const int step = (hi - lo + 63) / 64;
        const int idx = lo + lane * step;
        const bool le = idx < hi && gpre[idx] <= it.item;
        const int k = __popcll(__ballot(le));  // lanes 0 .. k-1 (lane 0 always)
        hi = min(hi, lo + k * step);
        lo = lo + (k - 1) * step;
    }
    it.group = lo;
    return it;
}

// The segment of group it.group that starts at it.item: its partial-result
// number (teams before this one that hold items of the group), whether it
// is the group's last, and this block's slots (the group's slots whose ranks
// fall in the segment and in which its own tile has a source) as a mask, the
// same in every lane.  Moves it.item to the segment's end.
__device__ inline void m2l_segment(const uint32_t* __restrict__ tmask,
                                   const uint32_t* __restrict__ gmask,
                                   const int32_t* __restrict__ gpre, int tile, int nb,
                                   M2lItems& it, int& part, bool& last, uint32_t (&mw)[7]) {
    const int p0 = gpre[it.group], p1 = gpre[it.group + 1];
    const int seg_end = min(it.iend, p1);
    part = it.b - (int)((((int64_t)p0 + 1) * nb - 1) / it.W);
    last = seg_end == p1;
    int base = 0;
#pragma unroll
    for (int w = 0; w < 7; ++w) {
        const uint32_t m = gmask[8 * it.group + w];
        mw[w] = __builtin_amdgcn_readfirstlane(
            m2l_rank_range(m, base, it.item - p0, seg_end - p0) & tmask[8 * tile + w]);
        base += __popc(m);
    }
    it.item = seg_end;
}

// first slot position >= j of the mask, else 216
__device__ inline int m2l_next_slot(const uint32_t (&mw)[7], int j) {
#pragma unroll
    for (int w = 0; w < 7; ++w) {
        if (j < 32 * w + 32) {
            const uint32_t bb = j > 32 * w ? mw[w] & (~0u << (j - 32 * w)) : mw[w];
            if (bb) return 32 * w + __builtin_ctz(bb);
        }
    }
    return 216;
}

}  // namespace hfmm

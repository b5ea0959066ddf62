// How the candidate pairs of a wave's 64 cells are shared out over a round's
// slots.  Apart from the kernel, so that it can be run on the host with the
// wave's exchanges emulated.
#pragma once

namespace dsmcx {

// Sum of v over the lanes below (one wave); *total over all.
__device__ __forceinline__ int lanes_excl(int v, int* total) {
    const int lane = threadIdx.x & 63;
    int incl = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(incl, o, 64);
        if (lane >= o) incl += t;
    }
    *total = __shfl(incl, 63, 64);
    return incl - v;
}

// Candidates of a lane in the next round of SLOTS, of the `left` >= 0 that it
// has: all that are left when they fit in the slots, else the same number from
// each lane that has any.  *base: its first slot; *total: slots taken.  A lane
// claims no more than all slots, so that the sum over the lanes stays in range
// whatever the counts (64 cells of 2^31 - 1 candidates each).
template <int SLOTS>
__device__ __forceinline__ int share_slots(int left, int* base, int* total) {
    int m = left < SLOTS ? left : SLOTS;
    *base = lanes_excl(m, total);
    if (*total > SLOTS) {
        const int most = SLOTS / __popcll(__ballot(left > 0));
        m = left < most ? left : most;
        *base = lanes_excl(m, total);
    }
    return m;
}

}  // namespace dsmcx

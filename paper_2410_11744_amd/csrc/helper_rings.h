// Rules of the rings through which draws made by a tree's helpers (build_tree.hip) come to the wave that pops.  A draw's way: the helper's
// LDS (kMailRing places), a ring in memory (as many), a ring in the tree's LDS (kRing places); draw r is at place r mod the ring's size.
// Draws below `taken` (the rank of the draw that the node opens next, as control has last said) are dead.
// Plain code without any include, so that it runs on the host as well.
#pragma once

namespace dyspec {

constexpr int kRing = 8, kRings = 8;        // places of a ring, rings (helpers) of a tree

// Bits 0, kRing, 2 kRing .. of a mask of lanes, put together: bit k for ring k.
__host__ __device__ __forceinline__ unsigned ring_bits(unsigned long long lanes)
{
    unsigned bits = 0;
    for (int k = 0; k < kRings; ++k) bits |= (unsigned)(lanes >> (kRing * k) & 1ull) << k;
    return bits;
}
// The ring that a node gets: the first whose helper runs (here) and that no node has (claims); the first of all is the root's.
// kRings: none.  (Helpers whose workgroups have no CU yet must not keep the others' from being used.)
__host__ __device__ __forceinline__ unsigned free_ring(unsigned here, unsigned claims, bool root)
{
    const unsigned open = here & ~claims & (root ? 1u : (1u << kRings) - 2u);
    return open ? (unsigned)__builtin_ctz(open) : (unsigned)kRings;
}

// A helper begins at rank 0 when it comes, the node's own wave goes on meanwhile.  So control takes draws from the ring only when
// the helper has made the one that is taken next; until then every pop asks the own wave for the next draw, and moves `taken` behind it.
// (A claim at rank 200 that moved the node to its ring four draws later made control wait for a helper that had 200 to make.)
__host__ __device__ __forceinline__ bool helper_caught_up(int draws_told, int taken) { return draws_told > taken; }
enum HandOver { kOwnDraw, kOwnDrawAndLater, kFromRing };
// The node's draw of that rank is popped: the next one, rank + 1, is the own wave's (kOwnDrawAndLater: and `taken` is to be rank + 2), or the ring's.
__host__ __device__ __forceinline__ HandOver hand_over(unsigned rank, unsigned taken, bool caught_up)
{
    return rank + 1u < taken ? kOwnDraw : caught_up ? kFromRing : kOwnDrawAndLater;
}

// Place j of a ring of SIZE: the draw that it is for when `first` is the lowest one of use.
template <int SIZE>
__host__ __device__ __forceinline__ int draw_of_place(int first, int j) { return first + ((j - first) & (SIZE - 1)); }
// The helper may make draws below this: so none that is still of use is written over, in its LDS or in memory.
template <int SIZE>
__host__ __device__ __forceinline__ int draws_allowed(int taken) { return taken + SIZE; }

}  // namespace dyspec

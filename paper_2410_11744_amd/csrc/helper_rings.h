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

}  // namespace dyspec

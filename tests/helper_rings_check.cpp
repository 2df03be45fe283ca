// The rules of the rings of a tree's helpers (csrc/helper_rings.h), run on the host.
// usage: helper_rings_check free: which ring a node gets, for every set of running helpers and of claimed rings
#define __host__
#define __device__
#define __forceinline__ inline
#include "../paper_2410_11744_amd/csrc/helper_rings.h"

#include <cstdio>
#include <cstring>

using namespace dyspec;

static int free_rings()
{
    for (unsigned here = 0; here < 256; ++here)
        for (unsigned claims = 0; claims < 256; ++claims)
            for (int root = 0; root < 2; ++root) {
                unsigned want = kRings;             // any other helper that runs and has no node, the first of them
                for (int k = kRings - 1; k >= 0; --k)
                    if ((k == 0) == (root == 1) && (here >> k & 1) && !(claims >> k & 1)) want = k;
                const unsigned got = free_ring(here, claims, root);
                if (got != want) {
                    printf("running %02x, claimed %02x, %s: ring %u, not %u\n", here, claims, root ? "the root" : "a node", got, want);
                    return 1;
                }
            }
    for (unsigned bits = 0; bits < 256; ++bits) {
        unsigned long long lanes = 0;
        for (int k = 0; k < kRings; ++k) lanes |= (unsigned long long)(bits >> k & 1) << (kRing * k);
        if (ring_bits(lanes) != bits) return 1;
    }
    return 0;
}

int main(int argc, char** argv)
{
    if (argc == 2 && !strcmp(argv[1], "free")) return free_rings();
    return 2;
}

// The rules of the rings of a tree's helpers (csrc/helper_rings.h), run on the host.
// usage: helper_rings_check free: which ring a node gets, for every set of running helpers and of claimed rings
//        helper_rings_check draws <trials> <first seed>: a node's draws on their way, step by step in random order and at random speeds, claimed
//        at any rank: control gets each draw once, whole and in order, and waits for no helper that is many draws behind
#define __host__
#define __device__
#define __forceinline__ inline
#include "../paper_2410_11744_amd/csrc/helper_rings.h"

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <random>

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

// A draw as it lies in a ring: its rank, written in two steps.
struct Draw { int a = -1, b = -1; };

struct Node {
    static constexpr int kBig = 64, kLast = 700;            // places of the rings in the helper's LDS and in memory; draws of the node
    std::mt19937 rng;
    bool started = false;                                   // the helper's workgroup has a CU
    // the helper's LDS and its two waves
    Draw lds[kBig], memory[kBig];
    int made = 0, half = 0, room = kBig, shipped = 0, ship_step = 0, ship_made = 0, ship_taken = 0;
    int told_count = 0, told_taken = 0;                     // the mailbox
    // wave 1
    Draw ring[kRing];
    int word[kRing], put[kRing], count[kRing], told = 0;
    bool claimed = false, caught_up = false;
    // control and the node's own wave
    int rank = 0, taken = 0, claim_at, own_next = 0;        // own_next: draws that the own wave has made
    bool from_ring = false;
    int made_when_asked = -1;

    explicit Node(unsigned seed) : rng(seed), claim_at((int)(rng() % 400)) { for (int j = 0; j < kRing; ++j) word[j] = put[j] = -1, count[j] = 0; }

    void make()
    {
        if (!started || made >= kLast) return;
        if (half == 0 && made % 4 == 0 && made + 4 > room) return;
        Draw& d = lds[made % kBig];
        if (half == 0) { d.a = made; half = 1; }
        else { d.b = made; half = 0; ++made; }
    }
    void ship()
    {
        if (!started) return;
        if (ship_step == 0) { ship_made = made; ship_taken = told_taken; }
        if (ship_step == 1)
            for (int l = 0; l < kBig; ++l)
                if (ship_made > shipped && draw_of_place<kBig>(shipped, l) < ship_made) memory[l].a = lds[l].a;
        if (ship_step == 2)
            for (int l = 0; l < kBig; ++l)
                if (ship_made > shipped && draw_of_place<kBig>(shipped, l) < ship_made) memory[l].b = lds[l].b;
        if (ship_step == 3) {
            told_count = shipped = ship_made;
            room = draws_allowed<kBig>(ship_taken);
        }
        ship_step = (ship_step + 1) % 4;
    }
    void look()
    {
        if (!claimed) return;
        const int t = taken;
        for (int j = 0; j < kRing; ++j) {
            const int r = draw_of_place<kRing>(t, j);
            const bool wanted = r > put[j], get = wanted && r < count[j];
            if (get) { ring[j] = memory[r % kBig]; word[j] = put[j] = r; }
            if (wanted && told_count > count[j]) count[j] = told_count;
        }
        caught_up = caught_up || helper_caught_up(count[0], t);
        if (t > told) told = told_taken = t;
    }
    const char* pop()                                       // of the draw of that rank
    {
        if (from_ring) {
            const int j = rank % kRing;
            if (made_when_asked < 0) made_when_asked = made;
            if (word[j] != rank) return made - made_when_asked > 24 ? "control waits for a helper that is far behind" : nullptr;
            made_when_asked = -1;
            if (ring[j].a != rank || ring[j].b != rank) return "the draw in the ring is another one";
            taken = ++rank;
            return nullptr;
        }
        if (own_next <= rank) return nullptr;               // the own wave is at it
        if (!claimed && started && rank >= claim_at) {
            claimed = true;
            taken = rank + 5;
        } else if (claimed) {
            const HandOver h = hand_over((unsigned)rank, (unsigned)taken, caught_up);
            if (h == kOwnDrawAndLater) taken = rank + 2;
            if (h == kFromRing && taken != rank + 1) return "the ring's first draw is not the next one";
            from_ring = h == kFromRing;
        }
        ++rank;
        return nullptr;
    }
};

static int draws(int trials, unsigned seed0)
{
    int by_ring = 0;
    for (int trial = 0; trial < trials; ++trial) {
        Node n(seed0 + trial);
        // how often each of them gets a step; the helper's draws come some three times as fast as the own wave's
        int share[5] = { 24, (int)(20 + n.rng() % 60), (int)(20 + n.rng() % 60), (int)(1 + n.rng() % 40), 4 };
        const int start = (int)(n.rng() % 20000), all = share[0] + share[1] + share[2] + share[3] + share[4];
        for (long step = 0; n.rank < Node::kLast; ++step) {
            n.started = n.started || step >= start;
            int x = (int)(n.rng() % all), who = 0;
            while (x >= share[who]) x -= share[who++];
            const char* wrong = nullptr;
            if (who == 0) n.make();
            else if (who == 1) n.ship();
            else if (who == 2) n.look();
            else if (who == 3) { wrong = n.pop(); by_ring += n.from_ring; }
            else if (!n.from_ring && n.own_next <= n.rank) ++n.own_next;
            if (wrong || step > 50000000) {
                printf("seed %u, claimed from rank %d on, helper from step %d on, draw %d: %s\n", seed0 + trial, n.claim_at, start, n.rank, wrong ? wrong : "it never comes");
                return 1;
            }
        }
    }
    return by_ring > 100 * trials ? 0 : 1;
}

int main(int argc, char** argv)
{
    if (argc == 4 && !strcmp(argv[1], "draws")) return draws(atoi(argv[2]), (unsigned)atoi(argv[3]));
    if (argc == 2 && !strcmp(argv[1], "free")) return free_rings();
    return 2;
}

// Where the helpers of a tree leave their draws in the builder's workspace (csrc/row_workspace.h): apart from each other's and from
// everything the tree's own waves write, however late a helper comes.  Row i of N has totals, a maximum, the tokens of its draws (its
// children are later rows, the last pop asks for one draw more and one is made ahead: ranks 0 .. N - i), a draw put aside, and, of the
// first rows, a mailbox.
#define __host__
#define __device__
#include "../paper_2410_11744_amd/csrc/row_workspace.h"

#include <cstdio>
#include <vector>

int main()
{
    using namespace dyspec;
    const int helpers = 8, base = 3;
    for (int N = 16; N <= DYSPEC_MAX_BUILD_NODES; ++N) {
        std::vector<double> ws((base + N) * (size_t)kRowSumDoubles);
        std::vector<char> used(ws.size(), 0);
        const auto use = [&](const double* at, size_t doubles) {
            for (size_t d = 0; d < doubles; ++d) {
                const size_t i = at - ws.data() + d;
                if (i >= used.size()) return false;
                if (used[i]) return false;
                used[i] = 1;
            }
            return true;
        };
        bool apart = true;
        for (int i = 0; i < N; ++i) {
            apart = apart && use(ws_totals(ws.data(), base + i), kSums) && use(ws_rowmax(ws.data(), base + i), 1) && use(ws_made(ws.data(), base + i), kMadeDoubles);
            const unsigned short* const drawn = ws_drawn(ws.data(), base + i);
            apart = apart && use(reinterpret_cast<const double*>(drawn), (size_t)(N - i) / 4 + 1);
            if (i < helpers) apart = apart && use(ws_mail(ws.data(), base + i), kMailDoubles);
        }
        if (!apart) {
            printf("tree of %d rows: the rows' own parts overlap\n", N);
            return 1;
        }
        for (int k = 0; k < helpers; ++k) {
            const double* const ring = ws_mail_ring(ws.data(), base, N, k);
            if (ring < ws_totals(ws.data(), base) || (ring - ws.data()) % 2 || !use(ring, 2 * kMailRing)) {
                printf("tree of %d rows: the ring of helper %d lies over something else\n", N, k);
                return 1;
            }
        }
    }
    return 0;
}

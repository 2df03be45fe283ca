// What a drawing wave writes to a row of the builder's workspace (csrc/row_workspace.h) when all draws of a tree are one node's, by
// the order of service of csrc/build_tree.hip: a tree of N rows asks for ranks 0 .. N - 1 (the last pop asks as well),
// ranks 0 and 1 are drawn when asked for, from rank 1 on the next one is drawn and put aside.  Every token drawn must be in a place of
// its own, the draw put aside must stay as it was put.
#define __host__
#define __device__
#include "../paper_2410_11744_amd/csrc/row_workspace.h"

#include <cstdio>
#include <cstring>
#include <vector>

int main()
{
    using namespace dyspec;
    for (int N = 2; N <= DYSPEC_MAX_BUILD_NODES; ++N) {
        std::vector<double> ws(2 * kRowSumDoubles, -1.0);
        const auto token = [](int rank) { return (unsigned short)(rank * 31 + 7); };
        int last = -1;
        for (int asked = 0; asked < N; ++asked) {
            if (asked > 1)
                for (int k = 0; k < kMadeDoubles; ++k)
                    if (ws_made(ws.data(), 0)[k] != asked + 0.25 * k) {
                        printf("tree of %d rows: the draw of rank %d is not the one put aside\n", N, asked);
                        return 1;
                    }
            for (int rank = asked > 1 ? asked + 1 : asked; rank <= (asked ? asked + 1 : 0); ++rank) {
                if (rank > asked)
                    for (int k = 0; k < kMadeDoubles; ++k) ws_made(ws.data(), 0)[k] = rank + 0.25 * k;
                ws_drawn(ws.data(), 0)[rank] = token(rank);
                last = rank;
            }
        }
        for (int k = 0; last > 1 && k < kMadeDoubles; ++k)
            if (ws_made(ws.data(), 0)[k] != last + 0.25 * k) {
                printf("tree of %d rows: the draw of rank %d, put aside, was written over\n", N, last);
                return 1;
            }
        for (int rank = 0; rank <= last; ++rank)
            if (ws_drawn(ws.data(), 0)[rank] != token(rank)) {
                printf("tree of %d rows: token of rank %d written over\n", N, rank);
                return 1;
            }
        for (int k = 0; k < kRowSumDoubles; ++k)
            if (ws_totals(ws.data(), 1)[k] != -1.0) {
                printf("tree of %d rows: the next row was written to\n", N);
                return 1;
            }
    }
    return 0;
}

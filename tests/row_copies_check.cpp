// Random services of a drawing wave through csrc/row_copies.h: every draw must be made from its row as the draws before
// left it.  Prints the first draw that is not, and ends with status 1.
// usage: row_copies_check <rows> <waves> <trials> <first seed>
#define __host__
#define __device__
#define __forceinline__ inline
#include "../paper_2410_11744_amd/csrc/row_copies.h"

#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

struct Row {
    int node;
    int draws;                  // that its totals know of
};

int main(int argc, char** argv)
{
    if (argc != 5) return 2;
    const int N = atoi(argv[1]), waves = atoi(argv[2]), trials = atoi(argv[3]), seed0 = atoi(argv[4]);
    for (int trial = 0; trial < trials; ++trial) {
        std::mt19937 rng(seed0 + trial);
        const int wave = (int)(rng() % waves);
        std::vector<int> memory(N, 0);
        const auto fetch = [&](int i, Row& r) { r.node = i; r.draws = memory[i]; };
        dyspec::RowCopies<Row> rows;
        rows.open(wave);
        // the nodes of the wave are made in order; any that was made may be asked for a draw
        int made = wave;
        for (int services = 0; services < 4 * N; ++services) {
            rows.look_ahead(N, fetch);
            while (made + waves < N && rng() % 3 == 0) made += waves;
            if (made >= N) break;
            const int i = wave + waves * (int)(rng() % ((made - wave) / waves + 1));
            rows.hold(i, waves, fetch);
            if (rows.held.node != i || rows.held.draws != memory[i]) {
                printf("rows %d waves %d seed %d: draw %d of node %d is made from a copy of row %d that knows of %d\n", N, waves, seed0 + trial,
                       memory[i], i, rows.held.node, rows.held.draws);
                return 1;
            }
            ++rows.held.draws;
            ++memory[i];
        }
    }
    return 0;
}

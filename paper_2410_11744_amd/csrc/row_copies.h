// The copies of row totals that a drawing wave of the greedy builder keeps in registers: of the row it drew from
// last, and of its next new node's row, fetched before that node is made.
//
// A draw changes the totals of its row, in memory and in the copy it is made from.  The copy fetched ahead is
// therefore good for its node's first draw only: it is handed over, not kept, and a node that is drawn from again
// after another one is read from memory.  Plain code without any include, so that it runs on the host as well.
#pragma once

namespace dyspec {

// Row: whatever describes a row, with `int node` (-1: no row's).  fetch(node, row) reads it from memory.
template <typename Row>
struct RowCopies {
    Row held, ahead;
    int next_new;               // the wave's smallest node beyond all it has served

    __host__ __device__ __forceinline__ void open(int first)
    {
        held.node = -1;
        ahead.node = -1;
        next_new = first;
    }
    // Between two services: the next new node's row, of a tree of N rows.
    template <typename Fetch>
    __host__ __device__ __forceinline__ void look_ahead(int N, Fetch&& fetch)
    {
        if (ahead.node < next_new && next_new < N) fetch(next_new, ahead);
    }
    // Makes `held` the row of node i, one of every `stride`.
    template <typename Fetch>
    __host__ __device__ __forceinline__ void hold(int i, int stride, Fetch&& fetch)
    {
        if (held.node != i) {
            if (ahead.node == i) {
                held = ahead;
                ahead.node = -1;
            } else {
                fetch(i, held);
            }
        }
        if (i >= next_new) next_new = i + stride;
    }
};

}  // namespace dyspec

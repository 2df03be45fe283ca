// Depth-first renaming of built token trees (Appendix "Block-Sparsity Friendly Token Order")
// for gfx950: new index = position in the pre-order walk that visits children in sampling
// order, so every subtree becomes a contiguous run of rows and the ancestor mask gathers
// into fewer 32x32 blocks.
//
// The walk is a linked list: after node i comes its first child, else the next sibling of the
// nearest ancestor-or-self that has one.  Its positions are found without walking it, by pointer
// doubling in LDS: the "next sibling of the nearest ancestor" links first (rounds until every
// node has one: log2 of the longest chain of last children), then the tables of 2^r-fold
// successors, then the root's position is carried forward through the tables, largest step
// first.  About 25 barrier rounds of a few LDS reads replace up to 2N dependent LDS reads by one lane.
// A sequence is handled by one workgroup per kSliceRows rows: each finds all positions (latency
// bound, the other CUs are idle anyway) and writes its slice of the arrays and of the mask, the
// slice's mask rows built in LDS and streamed out whole.
// 2048 random-tree rows: 505 us with one lane walking and mask rows built in global memory, 18 us now
// (kernel trace); renaming and attention of that tree together 575 -> 81 us.
//
// Links that do not form a tree (inconsistent, cyclic) take the literal walk by one lane, which
// stops at the first node met twice; rows that were never attached follow in index order.
#include "dyspec_device.h"

namespace dyspec {

constexpr int kReorderThreads = 1024;
constexpr int kSliceRows = 256;
// Widest tree of a batch up to which one lane walks the links: the doubling's rounds take 5.3 us whatever they find (2 rows
// 5.3 -> 3.3 us, 12 rows 6.5 -> 5.6), and from 16 rows on the walk is no shorter (6.6 against 6.5; 24 rows 7.6 against 6.8).
constexpr int kShortTree = 12;
constexpr int kJumps = 11;                                  // 2^11 = DYSPEC_MAX_NODES steps cover any walk
constexpr int kMaskWordsMax = DYSPEC_MAX_NODES / 64;
constexpr int kNodesPerThread = DYSPEC_MAX_NODES / kReorderThreads;
static_assert((1 << kJumps) >= DYSPEC_MAX_NODES && DYSPEC_MAX_NODES % kReorderThreads == 0, "doubling covers the longest walk");

struct ReorderShared {
    short parent[DYSPEC_MAX_NODES];
    short first_child[DYSPEC_MAX_NODES];
    short next_sibling[DYSPEC_MAX_NODES];
    short rank[DYSPEC_MAX_NODES];      // old index -> new index
    short order[DYSPEC_MAX_NODES];     // new index -> old index
    short new_parent[DYSPEC_MAX_NODES];
    // per node: what follows its subtree (>= -1), or -2 - u while that is still "what follows u's subtree"
    int after[DYSPEC_MAX_NODES];
    union {
        short jump[kJumps][DYSPEC_MAX_NODES];               // 2^r-fold successors, -1: past the end
        uint64_t mask[kSliceRows][kMaskWordsMax + 1];       // afterwards: the slice's mask rows
    };
    int loose[kReorderThreads / kWave][kNodesPerThread];    // rows never attached, per wave and pass
};

// The literal walk (one lane): pre-order without a stack, down to the first child, else along to the
// next sibling of the nearest ancestor-or-self that has one.
// (a node met twice, or more than 2N climbing steps, can only come from links that do
//  not form a tree: the walk stops there and the rest is appended as unattached rows)
__device__ void walk_literally(ReorderShared& sh, int N)
{
    for (int i = 0; i < N; ++i) sh.rank[i] = -1;
    int n = 0, cur = 0, climbs = 0;
    while (cur >= 0 && n < N && sh.rank[cur] < 0) {
        sh.rank[cur] = (short)n;
        sh.order[n++] = (short)cur;
        int next = sh.first_child[cur];
        while (next < 0 && cur >= 0 && climbs <= 2 * N) {
            next = sh.next_sibling[cur];
            if (next < 0) { cur = sh.parent[cur]; ++climbs; }
        }
        cur = next;
    }
    for (int i = 0; i < N && n < N; ++i)
        if (sh.rank[i] < 0) { sh.rank[i] = (short)n; sh.order[n++] = (short)i; }
}

// SHORT: no tree has more than kShortTree rows.
template <bool SHORT>
__global__ __launch_bounds__(kReorderThreads) void dfs_reorder_kernel(SeqArgs sa, dyspec_tree in, dyspec_tree out,
                                                                      int* __restrict__ order_out,
                                                                      uint64_t* __restrict__ mask_out, int mask_words)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char dyn[];
    ReorderShared& sh = *reinterpret_cast<ReorderShared*>(dyn);
    const int tid = threadIdx.x;
    const int seq = blockIdx.x;
    const int base = sa.node_off[seq];
    const int N = sa.node_off[seq + 1] - base;
    const int j0 = blockIdx.y * kSliceRows;                 // this workgroup's slice of the new rows
    if (j0 >= N) return;                                    // uniform over the workgroup
    const int slice = min(N - j0, kSliceRows);
    // links outside [0, N) are read as "none", so a malformed tree cannot send the walk out of LDS
    auto link = [N](int v) { return (short)((v >= 0 && v < N) ? v : -1); };
    for (int i = tid; i < N; i += kReorderThreads) {
        const short p = link(in.parent[base + i]), s = link(in.next_sibling[base + i]);
        sh.parent[i] = p;
        sh.first_child[i] = link(in.first_child[base + i]);
        sh.next_sibling[i] = s;
        sh.after[i] = s >= 0 ? s : p >= 0 ? -2 - p : -1;
        sh.rank[i] = -1;
    }
    __syncthreads();
    if constexpr (SHORT) {
        if (tid == 0) walk_literally(sh, N);
    } else {
        // every link agrees with the parents it implies: then a walk without a cycle meets every node
        // at most once and climbs every edge at most once, and is the literal walk
        bool bad = tid == 0 && sh.parent[0] >= 0;
        for (int i = tid; i < N; i += kReorderThreads) {
            const int c = sh.first_child[i], s = sh.next_sibling[i];
            bad |= c >= 0 && sh.parent[c] != i;
            bad |= s >= 0 && (sh.parent[i] < 0 || sh.parent[s] != sh.parent[i]);
        }
        // what follows a subtree: every round replaces "as for u" by u's own answer or by u's reference.
        // (in place: whatever a reader finds in u's word is equivalent to what stood there before)
        bool open = true;
        for (int r = 0; r <= kJumps && open; ++r) {
            open = false;
            for (int i = tid; i < N; i += kReorderThreads) {
                const int a = sh.after[i];
                if (a <= -2) {
                    const int up = sh.after[-2 - a];
                    sh.after[i] = up;
                    open |= up <= -2;
                }
            }
            open = __syncthreads_or(open);
        }
        bad |= open;                                            // a cycle of parents
        // ---- successors, and successors of successors
        int rounds = 0;
        while ((1 << rounds) < N) ++rounds;                     // a walk of N nodes has N - 1 steps
        for (int i = tid; i < N; i += kReorderThreads) {
            const int c = sh.first_child[i];
            sh.jump[0][i] = c >= 0 ? (short)c : (short)max(sh.after[i], -1);
        }
        __syncthreads();
        for (int r = 1; r < rounds; ++r) {
            for (int i = tid; i < N; i += kReorderThreads) {
                const int h = sh.jump[r - 1][i];
                sh.jump[r][i] = h >= 0 ? sh.jump[r - 1][h] : (short)-1;
            }
            __syncthreads();
        }
        // 2^rounds >= N steps from the root must lead past the end
        if (tid == 0) {
            if (rounds > 0) {
                const int h = sh.jump[rounds - 1][0];
                bad |= h >= 0 && sh.jump[rounds - 1][h] >= 0;
            }
            sh.rank[0] = 0;
        }
        __syncthreads();
        // ---- positions: the node 2^r steps after one at position k is at k + 2^r
        // (a node reached and read within one round only writes positions that are right as well)
        for (int r = rounds - 1; r >= 0; --r) {
            for (int i = tid; i < N; i += kReorderThreads) {
                const int k = sh.rank[i];
                if (k >= 0) {
                    const int h = sh.jump[r][i];
                    if (h >= 0) sh.rank[h] = (short)(k + (1 << r));
                }
            }
            __syncthreads();
        }
        // ---- rows that were never attached follow in index order; one that names a parent is no such row
        int visited = 0;
        bool mine_loose[kNodesPerThread];
        unsigned long long lanes[kNodesPerThread];
#pragma unroll
        for (int k = 0; k < kNodesPerThread; ++k) {
            const int i = tid + k * kReorderThreads;
            mine_loose[k] = i < N && sh.rank[i] < 0;
            bad |= mine_loose[k] && sh.parent[i] >= 0;
            lanes[k] = __ballot(mine_loose[k]);
            if ((tid & 63) == 0) sh.loose[tid >> 6][k] = __popcll(lanes[k]);
            visited += __syncthreads_count(i < N && sh.rank[i] >= 0);
        }
        if (__syncthreads_or(bad)) {
            if (tid == 0) walk_literally(sh, N);
        } else {
#pragma unroll
            for (int k = 0; k < kNodesPerThread; ++k) {
                const int i = tid + k * kReorderThreads;
                if (mine_loose[k]) {
                    int pos = visited + __popcll(lanes[k] & ((1ull << (tid & 63)) - 1ull));
                    for (int kk = 0; kk <= k; ++kk)
                        for (int w = 0; w < (kk < k ? kReorderThreads / kWave : tid >> 6); ++w) pos += sh.loose[w][kk];
                    sh.rank[i] = (short)pos;
                }
                if (i < N) sh.order[sh.rank[i]] = (short)i;
            }
        }
    }
    __syncthreads();
    auto renamed = [&](int old) { return old >= 0 ? (int)sh.rank[old] : -1; };
    for (int j = tid; j < N; j += kReorderThreads) sh.new_parent[j] = (short)renamed(sh.parent[sh.order[j]]);
    for (int x = tid; x < slice * (kMaskWordsMax + 1); x += kReorderThreads) (&sh.mask[0][0])[x] = 0ull;
    __syncthreads();
    if (tid < slice) {
        // mask row j: own bit and the bits of the chain of renamed parents (all smaller than j), gathered
        // a word at a time
        const int j = j0 + tid;
        int word = j >> 6;
        uint64_t bits = 0ull;
        for (int a = j, prev = N; a >= 0 && a < prev; prev = a, a = sh.new_parent[a]) {
            if ((a >> 6) != word) { sh.mask[tid][word] = bits; word = a >> 6; bits = 0ull; }
            bits |= 1ull << (a & 63);
        }
        sh.mask[tid][word] = bits;
    } else if (tid >= kReorderThreads - kSliceRows && tid - (kReorderThreads - kSliceRows) < slice) {
        const int j = j0 + tid - (kReorderThreads - kSliceRows);
        const int o = sh.order[j];
        order_out[base + j] = o;
        out.parent[base + j] = sh.new_parent[j];
        out.first_child[base + j] = renamed(sh.first_child[o]);
        out.next_sibling[base + j] = renamed(sh.next_sibling[o]);
        out.token[base + j] = in.token[base + o];
        out.sib_rank[base + j] = in.sib_rank[base + o];
        out.depth[base + j] = in.depth[base + o];
    }
    __syncthreads();
    uint64_t* const rows = mask_out + (size_t)(base + j0) * mask_words;
    const int word = tid % kMaskWordsMax;
    if (word < mask_words)
        for (int r = tid / kMaskWordsMax; r < slice; r += kReorderThreads / kMaskWordsMax) rows[(size_t)r * mask_words + word] = sh.mask[r][word];
}

// the positions of the largest tree take more LDS than a kernel gets by default
hipError_t prepare_reorder()
{
    static std::atomic<unsigned long long> done_short{0}, done{0};
    const hipError_t e = raise_dynamic_lds_once(reinterpret_cast<const void*>(&dfs_reorder_kernel<true>), (int)sizeof(ReorderShared), done_short);
    if (e != hipSuccess) return e;
    return raise_dynamic_lds_once(reinterpret_cast<const void*>(&dfs_reorder_kernel<false>), (int)sizeof(ReorderShared), done);
}

hipError_t launch_dfs_reorder(const SeqArgs& sa, const dyspec_tree& in, const dyspec_tree& out, int* order,
                              uint64_t* mask_out, int mask_words, hipStream_t stream)
{
    int widest = 1;
    for (int s = 0; s < sa.n_seq; ++s) widest = max(widest, sa.node_off[s + 1] - sa.node_off[s]);
    const hipError_t e = prepare_reorder();
    if (e != hipSuccess) return e;
    const dim3 grid(sa.n_seq, (widest + kSliceRows - 1) / kSliceRows);
    if (widest <= kShortTree)
        dfs_reorder_kernel<true><<<grid, kReorderThreads, sizeof(ReorderShared), stream>>>(sa, in, out, order, mask_out, mask_words);
    else
        dfs_reorder_kernel<false><<<grid, kReorderThreads, sizeof(ReorderShared), stream>>>(sa, in, out, order, mask_out, mask_words);
    return hipGetLastError();
}

}  // namespace dyspec

// Depth-first renaming of built token trees (Appendix "Block-Sparsity Friendly Token Order")
// for gfx950: new index = position in the pre-order walk that visits children in sampling
// order, so every subtree becomes a contiguous run of rows and the ancestor mask gathers
// into fewer 32x32 blocks.
//
// The walk is a linked list: after node i comes its first child, else the next sibling of the
// nearest ancestor-or-self that has one.  Its positions are found without walking it, by pointer
// doubling in LDS: the "next sibling of the nearest ancestor" links first (rounds until every
// node has one), then every node's steps to the end of the walk: a word holds a node further along and the steps to it,
// and takes over what that node's word says.  A word is right at any time, so the rounds work in place and follow two links between
// barriers; 2048 rows need seven.  (Tables of 2^r-fold successors and the root's position carried forward through
// them: 21 rounds.)
// A subtree is then a run of rows that ends where the walk goes on after it, and row a is above row j if a <= j < end(a): a column of
// 64 rows of the mask is one run of bits, and a wave makes a word of 64 rows by transposing 64 columns.  (Each row's chain of parents
// followed by one lane: as fast in random trees, 200 us in a chain of 2048.)
// A sequence is handled by one workgroup per 64 rows: each finds all positions (latency bound, the other CUs are idle anyway) and
// writes its slice of the arrays and of the mask, the slice's mask rows made in LDS and streamed out whole.  Per 256 rows where
// that would be more than 512 workgroups, as many as run at a time: 17 sequences of 2048 rows 14.5 us (64 rows 18.8), 64 of them 27 (43), 64 of 1024
// 11.0 (16.8); 16 of 2048 13.2 (256 rows 14.4), 64 of 512 7.4 (8.2), one of 2048 8.8 (12.5).
// Bound by latencies: launch, the links' trip from memory, some twenty barriers with an LDS read or two between them, the writes.
// 2048 random-tree rows: 505 us with one lane walking and mask rows built in global memory, 17.1 with the tables of successors, 8.6 now;
// 512 rows 11.3 -> 5.3, 32 rows 7.7 -> 4.3, a chain of 2048 211 -> 11.2, 64 sequences of 2048 35.4 -> 27 (calls in a graph).
//
// Links that do not form a tree (inconsistent, cyclic) take the literal walk by one lane, which
// stops at the first node met twice; rows that were never attached follow in index order.
#include "dyspec_device.h"

namespace dyspec {

constexpr int kReorderThreads = 1024;                       // (512: 2048 rows 10.9 us, 32 rows 4.7; 256: 17.3 and 5.5)
constexpr int kSliceRows = 64, kWideSlice = 256;            // rows of a workgroup; of one where there are many
constexpr int kManySlices = 512;                            // more workgroups than that are many (two run on a CU at a time)
// Widest tree of a batch up to which one lane walks the links: the doubling's rounds take 3.7 us whatever they find (2 rows
// 3.5 -> 2.7 us, 4 rows 3.8 -> 3.3), and from 6 rows on the walk is no shorter (3.8 against 3.7; 12 rows 5.4 against 3.9).
constexpr int kShortTree = 5;
constexpr int kJumps = 11;                                  // 2^11 = DYSPEC_MAX_NODES steps cover any walk
constexpr int kHops = 2;                                    // links followed between two barriers: 1 + kHops times the reach a round
constexpr unsigned kPastEnd = 0xffffu;                      // upper half of a packed successor: the walk is over
constexpr int kMaskWordsMax = DYSPEC_MAX_NODES / 64;
constexpr int kNodesPerThread = DYSPEC_MAX_NODES / kReorderThreads;
static_assert((1 << kJumps) >= DYSPEC_MAX_NODES && DYSPEC_MAX_NODES % kReorderThreads == 0, "doubling covers the longest walk");

template <int SLICE>
struct ReorderShared {
    short parent[DYSPEC_MAX_NODES];
    short first_child[DYSPEC_MAX_NODES];
    short next_sibling[DYSPEC_MAX_NODES];
    short order[DYSPEC_MAX_NODES];     // new index -> old index
    short subtree_end[DYSPEC_MAX_NODES];                    // per new index: the row behind its subtree
    union {
        // per node: what follows its subtree (>= -1), or -2 - u while that is still "what follows u's subtree"
        int after[DYSPEC_MAX_NODES];
        struct {                                            // once the walk is known
            short rank[DYSPEC_MAX_NODES];                   // old index -> new index
            short new_parent[DYSPEC_MAX_NODES];
        };
    };
    // per node: a node further along the walk in the upper half, the steps to it in the lower
    unsigned ahead[DYSPEC_MAX_NODES];
    int token[DYSPEC_MAX_NODES], sib_rank[DYSPEC_MAX_NODES], depth[DYSPEC_MAX_NODES];   // carried over as they are
    uint64_t mask[SLICE][kMaskWordsMax + 1];                // the slice's mask rows
    int loose[kNodesPerThread][kReorderThreads / kWave];    // rows never attached, per pass and wave
    int n_loose;
    int bad;                                                // some link disagrees with the others
    int open[kJumps + 1];                                   // a round of `after` left something unresolved
};

// The literal walk (one lane): pre-order without a stack, down to the first child, else along to the
// next sibling of the nearest ancestor-or-self that has one.
// (a node met twice, or more than 2N climbing steps, can only come from links that do
//  not form a tree: the walk stops there and the rest is appended as unattached rows)
template <class Shared>
__device__ void walk_literally(Shared& sh, int N)
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

// Bit c of lane r becomes bit r of lane c.
__device__ __forceinline__ uint64_t transpose64(uint64_t x)
{
    const int lane = threadIdx.x & 63;
    uint64_t keep = 0x00000000ffffffffull;                  // columns without bit s
#pragma unroll
    for (int s = 32; s > 0; s >>= 1) {
        const uint64_t y = __shfl_xor((unsigned long long)x, s);
        x = (lane & s) ? (x & ~keep) | ((y >> s) & keep) : (x & keep) | ((y & keep) << s);
        keep ^= keep << (s >> 1);
    }
    return x;
}

// SHORT: no tree has more than kShortTree rows.
template <bool SHORT, int SLICE>
__global__ __launch_bounds__(kReorderThreads) void dfs_reorder_kernel(SeqArgs sa, dyspec_tree in, dyspec_tree out,
                                                                      int* __restrict__ order_out,
                                                                      uint64_t* __restrict__ mask_out, int mask_words)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char dyn[];
    auto& sh = *reinterpret_cast<ReorderShared<SLICE>*>(dyn);
    const int tid = threadIdx.x;
    const int seq = blockIdx.x;
    const int base = sa.node_off[seq];
    const int N = sa.node_off[seq + 1] - base;
    const int j0 = blockIdx.y * SLICE;                 // this workgroup's slice of the new rows
    if (j0 >= N) return;                                    // uniform over the workgroup
    const int slice = min(N - j0, SLICE);
    // links outside [0, N) are read as "none", so a malformed tree cannot send the walk out of LDS
    auto link = [N](int v) { return (short)((v >= 0 && v < N) ? v : -1); };
    for (int i = tid; i < N; i += kReorderThreads) {
        const short p = link(in.parent[base + i]), s = link(in.next_sibling[base + i]);
        sh.parent[i] = p;
        sh.first_child[i] = link(in.first_child[base + i]);
        sh.next_sibling[i] = s;
        if constexpr (!SHORT) sh.after[i] = s >= 0 ? s : p >= 0 ? -2 - p : -1;
        sh.token[i] = in.token[base + i];
        sh.sib_rank[i] = in.sib_rank[base + i];
        sh.depth[i] = in.depth[base + i];
    }
    if (tid <= kJumps) sh.open[tid] = 0;
    if (tid == 0) sh.n_loose = sh.bad = 0;
    __syncthreads();
    bool literally = SHORT;
    if constexpr (!SHORT) {
        // every link agrees with the parents it implies: then a walk without a cycle meets every node
        // at most once and climbs every edge at most once, and is the literal walk.
        // (rows that were never attached are counted by the way: they follow in index order)
        bool bad = tid == 0 && sh.parent[0] >= 0;
        int after[kNodesPerThread];
        unsigned long long lanes[kNodesPerThread];          // the wave's rows without a parent, the root aside
#pragma unroll
        for (int k = 0; k < kNodesPerThread; ++k) {
            const int i = tid + k * kReorderThreads;
            after[k] = -1;
            bool alone = false;
            if (i < N) {
                const int p = sh.parent[i], c = sh.first_child[i], s = sh.next_sibling[i];
                bad |= c >= 0 && sh.parent[c] != i;
                bad |= s >= 0 && (p < 0 || sh.parent[s] != p);
                after[k] = sh.after[i];
                alone = i > 0 && p < 0;
            }
            lanes[k] = __ballot(alone);
            if ((tid & 63) == 0) {
                sh.loose[k][tid >> 6] = __popcll(lanes[k]);
                if (lanes[k]) atomicAdd(&sh.n_loose, (int)__popcll(lanes[k]));
            }
        }
        if (bad) sh.bad = 1;
        // what follows a subtree: every round replaces "as for u" by u's own answer or by u's reference.
        // (in place: whatever a reader finds in u's word is equivalent to what stood there before)
        bool open = true;
        for (int r = 0; r <= kJumps && open; ++r) {
#pragma unroll
            for (int k = 0; k < kNodesPerThread; ++k) {
                if (after[k] <= -2) {
#pragma unroll
                    for (int h = 0; h < kHops; ++h)
                        if (after[k] <= -2) after[k] = sh.after[-2 - after[k]];
                    sh.after[tid + k * kReorderThreads] = after[k];
                    if (after[k] <= -2) sh.open[r] = 1;
                }
            }
            __syncthreads();
            open = sh.open[r] != 0;
        }
        // ---- successors, then in every round the successors found so far put together: the steps that are
        // left to the end of the walk.  (in place as well: a word holds a node and the steps to it at all times)
        unsigned ahead[kNodesPerThread];
#pragma unroll
        for (int k = 0; k < kNodesPerThread; ++k) {
            const int i = tid + k * kReorderThreads;
            ahead[k] = kPastEnd << 16;
            if (i < N) {
                const int c = sh.first_child[i], next = c >= 0 ? c : after[k];
                if (next >= 0) ahead[k] = (unsigned)next << 16 | 1u;
                sh.ahead[i] = ahead[k];
            }
        }
        __syncthreads();
        for (int reach = 1; reach < N; reach *= 1 + kHops) {
#pragma unroll
            for (int k = 0; k < kNodesPerThread; ++k) {
                if (ahead[k] >> 16 != kPastEnd) {
#pragma unroll
                    for (int h = 0; h < kHops; ++h)
                        if (ahead[k] >> 16 != kPastEnd) {
                            const unsigned u = sh.ahead[ahead[k] >> 16];
                            ahead[k] = (u & 0xffff0000u) | ((ahead[k] + u) & 0xffffu);
                        }
                    sh.ahead[tid + k * kReorderThreads] = ahead[k];
                }
            }
            __syncthreads();
        }
        // ---- positions.  The root's walk has to end, and has to meet every row that names a parent (it meets no other)
        const unsigned root = sh.ahead[0];
        const int steps = (int)(root & 0xffffu), n_loose = sh.n_loose;
        literally = open || sh.bad != 0 || root >> 16 != kPastEnd || steps + 1 + n_loose != N;      // uniform
        if (!literally) {
            auto place = [&](unsigned a) { return steps - (int)(a & 0xffffu); };
#pragma unroll
            for (int k = 0; k < kNodesPerThread; ++k) {
                const int i = tid + k * kReorderThreads;
                if (i >= N) continue;
                const int p = sh.parent[i];
                int pos = place(ahead[k]), end = after[k] >= 0 ? place(sh.ahead[after[k]]) : steps + 1;
                if (i > 0 && p < 0) {
                    pos = steps + 1 + __popcll(lanes[k] & ((1ull << (tid & 63)) - 1ull));
                    for (int kk = 0; kk <= k; ++kk)
                        for (int w = 0; w < (kk < k ? kReorderThreads / kWave : tid >> 6); ++w) pos += sh.loose[kk][w];
                    end = pos + 1;
                }
                sh.rank[i] = (short)pos;
                sh.subtree_end[pos] = (short)end;
                sh.order[pos] = (short)i;
                sh.new_parent[pos] = p >= 0 ? (short)place(sh.ahead[p]) : (short)-1;
            }
        }
    }
    auto renamed = [&](int old) { return old >= 0 ? (int)sh.rank[old] : -1; };
    if (literally) {
        if (tid == 0) walk_literally(sh, N);
        for (int x = tid; x < slice * (kMaskWordsMax + 1); x += kReorderThreads) (&sh.mask[0][0])[x] = 0ull;
        __syncthreads();
        for (int j = tid; j < N; j += kReorderThreads) sh.new_parent[j] = (short)renamed(sh.parent[sh.order[j]]);
    }
    __syncthreads();
    if (literally) {
        // mask row j: own bit and the bits of the chain of renamed parents (all smaller than j), gathered
        // a word at a time
        if (tid < slice) {
            const int j = j0 + tid;
            int word = j >> 6;
            uint64_t bits = 0ull;
            for (int a = j, prev = N; a >= 0 && a < prev; prev = a, a = sh.new_parent[a]) {
                if ((a >> 6) != word) { sh.mask[tid][word] = bits; word = a >> 6; bits = 0ull; }
                bits |= 1ull << (a & 63);
            }
            sh.mask[tid][word] = bits;
        }
    } else {
        // mask row j: the rows up to j whose subtree ends behind j.  A wave makes one word of 64 rows: lane l the column of
        // row 64 word + l, which is one run of bits, and the columns are transposed
        const int lane = tid & 63;
        for (int x = tid >> 6; x < (slice + 63) / 64 * mask_words; x += kReorderThreads / kWave) {
            const int word = x % mask_words, block = x / mask_words, row0 = j0 + 64 * block, a = 64 * word + lane;
            const int first = max(a - row0, 0), end = a < N && first < 64 ? min(sh.subtree_end[a] - row0, 64) : 0;
            uint64_t bits = end > first ? (~0ull >> (64 - end)) & (~0ull << first) : 0ull;
            if (__ballot(bits != 0ull)) bits = transpose64(bits);   // (else no row of the word is above any of the block)
            if (64 * block + lane < slice) sh.mask[64 * block + lane][word] = bits;
        }
    }
    if (tid >= kReorderThreads - SLICE && tid - (kReorderThreads - SLICE) < slice) {
        const int j = j0 + tid - (kReorderThreads - SLICE);
        const int o = sh.order[j];
        order_out[base + j] = o;
        out.parent[base + j] = sh.new_parent[j];
        out.first_child[base + j] = renamed(sh.first_child[o]);
        out.next_sibling[base + j] = renamed(sh.next_sibling[o]);
        out.token[base + j] = sh.token[o];
        out.sib_rank[base + j] = sh.sib_rank[o];
        out.depth[base + j] = sh.depth[o];
    }
    __syncthreads();
    uint64_t* const rows = mask_out + (size_t)(base + j0) * mask_words;
    const int word = tid % kMaskWordsMax;
    if (word < mask_words)
        for (int r = tid / kMaskWordsMax; r < slice; r += kReorderThreads / kMaskWordsMax) rows[(size_t)r * mask_words + word] = sh.mask[r][word];
}

template <bool SHORT, int SLICE>
static hipError_t prepare_form()
{
    static std::atomic<unsigned long long> done{0};
    return raise_dynamic_lds_once(reinterpret_cast<const void*>(&dfs_reorder_kernel<SHORT, SLICE>), (int)sizeof(ReorderShared<SLICE>), done);
}

// the positions of the largest tree take more LDS than a kernel gets by default
hipError_t prepare_reorder()
{
    hipError_t e = prepare_form<true, kSliceRows>();
    if (e == hipSuccess) e = prepare_form<false, kSliceRows>();
    if (e == hipSuccess) e = prepare_form<false, kWideSlice>();
    return e;
}

hipError_t launch_dfs_reorder(const SeqArgs& sa, const dyspec_tree& in, const dyspec_tree& out, int* order,
                              uint64_t* mask_out, int mask_words, hipStream_t stream)
{
    int widest = 1;
    for (int s = 0; s < sa.n_seq; ++s) widest = max(widest, sa.node_off[s + 1] - sa.node_off[s]);
    const hipError_t e = prepare_reorder();
    if (e != hipSuccess) return e;
    const auto launch = [&](auto* kernel, int slice, size_t lds) {
        kernel<<<dim3(sa.n_seq, (widest + slice - 1) / slice), kReorderThreads, lds, stream>>>(sa, in, out, order, mask_out, mask_words);
    };
    if (widest <= kShortTree)
        launch(&dfs_reorder_kernel<true, kSliceRows>, kSliceRows, sizeof(ReorderShared<kSliceRows>));
    else if (sa.n_seq * ((widest + kSliceRows - 1) / kSliceRows) <= kManySlices)
        launch(&dfs_reorder_kernel<false, kSliceRows>, kSliceRows, sizeof(ReorderShared<kSliceRows>));
    else
        launch(&dfs_reorder_kernel<false, kWideSlice>, kWideSlice, sizeof(ReorderShared<kWideSlice>));
    return hipGetLastError();
}

}  // namespace dyspec

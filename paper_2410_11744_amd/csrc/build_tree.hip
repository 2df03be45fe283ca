// Greedy fixed-budget token-tree construction (Algorithm 1, Section 4.2, Appendix A.1)
// and the ancestor bitmask of tree attention (Section 2) for gfx950.
//
// One workgroup builds one sequence's tree without leaving the GPU.  The paper keeps the
// expandable slots in a heap on the host; here the frontier lives in registers or LDS and the pop
// is an arg-max, which costs less than a heap's pointer chasing at these sizes.  A draw needs the
// parent's residual draft distribution: fp64 softmax weights and an inverse CDF over them.
// fp64 keeps every discrete decision (which slot, which token) equal to an fp64 evaluation of the
// algorithm except at relative margins near 1e-13.
//
// With a workspace (build_tree_waves_kernel) the draws leave the pop's way.  The draws of a node
// depend on its row, its path key and the child's rank only, not on when the node is popped, so
// they are made ahead by other waves of the workgroup; draft_row_sums_kernel (one workgroup per row, all
// rows at once) has stored every row's maximum and group totals before.  Without a workspace the builder (build_tree_kernel)
// recomputes the sums of the parent's row for every draw.  Both ways make the same draws to the rounding of their sums, and build the
// same tree where no decision is closer than that; one call builds the same tree every time.
#include <algorithm>
#include <cstddef>

#include "draft_row.h"
#include "helper_rings.h"
#include "lane_ops.h"
#include "row_copies.h"
#include "row_workspace.h"
#include "run_draw.h"
#include "wave_draw.h"

namespace dyspec {

constexpr int kMaxSlots = 2 * DYSPEC_MAX_BUILD_NODES + 2;

// Data-parallel part (the draft softmax of every node, Algorithm 1's model call output):
// one workgroup per row writes the row's totals and maximum.  S: segments held, V <= S * kSeg.
// Bound in turn by the trip to memory (every load is issued before the maximum is known) and by the vector ALU: some 28
// instructions a token, 22 of them the fp64 exponential.  Segments past the end of the row cost nothing, and the sums of a run's lanes
// are folded into one another (row_sums) instead of summed one by one, five steps each: 32 rows of 1000 tokens
// 9.8 -> 3.6 us, 128 rows of 32000 14.6 -> 12.4, 512 rows 27.3 -> 26.2 (66 MB; nothing is left to overlap loads with: all
// rows are in flight at once).  S: 2 holds 4096 tokens, 8 16384; where the unused segments were skipped in the code for 16 their
// registers and code stayed.
template <bool VEC, int S>
__global__ __launch_bounds__(kBlock) void draft_row_sums_kernel(const float* __restrict__ draft_logits, int V, SeqArgs sa,
                                                                double* __restrict__ ws, int mails)
{
    __shared__ float fred[kWaves];
    const int row = blockIdx.x;
    const int seq = find_seq(sa, row);
    const double inv_temp = 1.0 / (double)sa.temp_d[seq];
    float x[S][4];
    load_row<VEC, float>(draft_logits + (size_t)row * V, V, x);
    float mx[1] = { -INFINITY };
#pragma unroll
    for (int j = 0; j < S; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) mx[0] = fmaxf(mx[0], x[j][e]);
    block_max<1>(mx, fred);
    const double m = (double)mx[0] * inv_temp;
    double seg[S];
#pragma unroll
    for (int j = 0; j < S; ++j) {
        seg[j] = 0.0;
        if (j * kSeg >= V) continue;                    // uniform
        double z[4], w4[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) z[e] = fma((double)x[j][e], inv_temp, -m);
        exp_nonpos_xn<4>(z, w4);                        // (tokens past the end: exp(-inf) = 0)
        seg[j] = (w4[0] + w4[1]) + (w4[2] + w4[3]);
    }
    // half a wave holds a run of a segment: lane j % 16 of the half gets segment j's sum
    static_assert(4 * kWave == 2 * kRun && kMaxSeg == 16, "two runs per wave and segment, a lane per segment");
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, j = lane & 15;
    double t = row_sums(seg);
    t += __shfl_xor(t, 16, kWave);
    if (lane & 16) ws_totals(ws, row)[j * (kSeg / kRun) + 2 * wave + (lane >> 5)] = j < S ? t : 0.0;
    if (threadIdx.x == 0) *ws_rowmax(ws, row) = m;
    if (mails && threadIdx.x < kMailDoubles && row - sa.node_off[seq] < kRings) ws_mail(ws, row)[threadIdx.x] = 0.0;
}

// LDS state of the form without a workspace.
struct BuildShared {
    double slot_value[kMaxSlots];       // < 0: closed
    int slot_parent[kMaxSlots];
    int n_children[DYSPEC_MAX_BUILD_NODES];
    int last_child[DYSPEC_MAX_BUILD_NODES];
    int token[DYSPEC_MAX_BUILD_NODES];
    int first_child[DYSPEC_MAX_BUILD_NODES];
    int next_sibling[DYSPEC_MAX_BUILD_NODES];
    int depth[DYSPEC_MAX_BUILD_NODES];
    uint2 pk[DYSPEC_MAX_BUILD_NODES];
    CdfScratch cdf;
    double best_v[kWaves];
    int best_i[kWaves];
    float fred[kWaves];
    int n_slots;
    int pick;
};

// Initial state of a sequence's tree in global memory: every row unbuilt.
__device__ __forceinline__ void init_tree_rows(int base, int N, const dyspec_tree& tree, float* __restrict__ est_value,
                                               uint64_t* __restrict__ anc_mask, int mask_words)
{
    for (int i = threadIdx.x; i < N; i += kBlock) {
        tree.parent[base + i] = -1; tree.token[base + i] = -1; tree.sib_rank[base + i] = 0;
        tree.first_child[base + i] = -1; tree.next_sibling[base + i] = -1; tree.depth[base + i] = 0;
        est_value[base + i] = (i == 0) ? 1.0f : 0.0f;
        for (int w = 0; w < mask_words; ++w)
            anc_mask[(size_t)(base + i) * mask_words + w] = (w == i / 64) ? (1ull << (i % 64)) : 0ull;
    }
}

// ... and in LDS, with the root's slot open.  Ends with a barrier.
__device__ __forceinline__ void init_tree_state(BuildShared& sh, int seq, int base, int N, const dyspec_tree& tree,
                                                float* __restrict__ est_value, uint64_t* __restrict__ anc_mask, int mask_words)
{
    const int tid = threadIdx.x;
    init_tree_rows(base, N, tree, est_value, anc_mask, mask_words);
    for (int i = tid; i < N; i += kBlock) {
        sh.n_children[i] = 0; sh.last_child[i] = -1; sh.token[i] = -1;
        sh.first_child[i] = -1; sh.next_sibling[i] = -1; sh.depth[i] = 0;
    }
    for (int s = tid; s < kMaxSlots; s += kBlock) sh.slot_value[s] = -1.0;
    __syncthreads();
    if (tid == 0) {
        sh.slot_value[0] = 1.0; sh.slot_parent[0] = 0; sh.n_slots = 1;
        sh.pk[0] = root_key((uint32_t)seq);
    }
    __syncthreads();
}

// Thread 0's bookkeeping for new node i = child number `rank` of p with token y, taken from a slot
// of value v (Algorithm 1: the node's estimated acceptance rate).
__device__ __forceinline__ void append_node(BuildShared& sh, const dyspec_tree& tree, float* __restrict__ est_value,
                                            uint2 key, int base, int p, int i, int rank, int y, double v)
{
    sh.token[i] = y; sh.depth[i] = sh.depth[p] + 1;
    if (sh.last_child[p] < 0) { sh.first_child[p] = i; tree.first_child[base + p] = i; }
    else { sh.next_sibling[sh.last_child[p]] = i; tree.next_sibling[base + sh.last_child[p]] = i; }
    sh.last_child[p] = i; sh.n_children[p] = rank + 1;
    sh.pk[i] = key;
    tree.parent[base + i] = p; tree.token[base + i] = y; tree.sib_rank[base + i] = rank;
    tree.depth[base + i] = sh.depth[i];
    est_value[base + i] = (float)v;
}

// The form without a workspace: the sums of the parent's row are recomputed for every draw.
template <bool VEC>
__global__ __launch_bounds__(kBlock) void build_tree_kernel(
    const float* __restrict__ draft_logits, int V, SeqArgs sa, uint64_t seed,
    dyspec_tree tree, float* __restrict__ est_value, uint64_t* __restrict__ anc_mask,
    int mask_words, int* __restrict__ n_built)
{
    __shared__ BuildShared sh;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int seq = blockIdx.x;
    const int base = sa.node_off[seq];
    const int N = sa.node_off[seq + 1] - base;
    const double inv_temp = 1.0 / (double)sa.temp_d[seq];
    init_tree_state(sh, seq, base, N, tree, est_value, anc_mask, mask_words);

    int n = 1;
    while (n < N) {
        // ---- pop: open slot of largest value, earliest-opened on ties
        const int n_slots = sh.n_slots;
        double bv = -1.0; int bi = 0x7fffffff;
        for (int s = tid; s < n_slots; s += kBlock) {
            const double v = sh.slot_value[s];
            if (v > bv) { bv = v; bi = s; }           // s ascends: ties keep the earlier slot
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            const double ov = __shfl_xor(bv, o, kWave);
            const int oi = __shfl_xor(bi, o, kWave);
            if (ov > bv || (ov == bv && oi < bi)) { bv = ov; bi = oi; }
        }
        if (lane == 0) { sh.best_v[wave] = bv; sh.best_i[wave] = bi; }
        __syncthreads();
        if (tid == 0) {
            double v = sh.best_v[0]; int i = sh.best_i[0];
            for (int w = 1; w < kWaves; ++w)
                if (sh.best_v[w] > v || (sh.best_v[w] == v && sh.best_i[w] < i)) { v = sh.best_v[w]; i = sh.best_i[w]; }
            sh.pick = (v > 0.0) ? i : -1;
        }
        __syncthreads();
        const int pick = sh.pick;
        if (pick < 0) break;                           // frontier is empty
        const int p = sh.slot_parent[pick];
        const double v = sh.slot_value[pick];
        const int rank = sh.n_children[p];

        // ---- draw the token from the residual draft distribution of p (softmax weights with
        //      the earlier children's tokens removed)
        const double u = (double)u01(seed, sh.pk[p], (uint32_t)rank, KIND_BUILD);
        const float* __restrict__ row = draft_logits + (size_t)(base + p) * V;
        // bit k of `gone` marks this thread's k-th token as already drawn at this position
        uint64_t gone = 0ull;
        for (int c = sh.first_child[p]; c >= 0; c = sh.next_sibling[c]) {
            const int yc = sh.token[c];
            if (((yc % kSeg) >> 2) == tid) gone |= 1ull << (4 * (yc / kSeg) + (yc & 3));
        }
        double m, seg[kMaxSeg], W, wy;
        row_segment_sums<VEC>(row, V, inv_temp, gone, sh.fred, &m, seg);
        const int y = block_inverse_cdf_seg(seg, u, &sh.cdf, &W, &wy, [&](int j, int e) -> double {
            const int idx = tok_index(j, e);
            const bool live = idx < V && !((gone >> (4 * j + e)) & 1ull);
            return live ? token_weight(row[idx], inv_temp, m) : 0.0;
        });
        if (y < 0) break;                              // nothing left to sample under p

        // ---- append node n, open its two slots
        const int i = n;
        if (tid == 0) {
            const double Ry = wy / W;
            sh.slot_value[pick] = -1.0;
            append_node(sh, tree, est_value, child_key(seed, sh.pk[p], (uint32_t)rank), base, p, i, rank, y, v);
            const double v0 = v * Ry, v1 = v * (1.0 - Ry);
            int ns = sh.n_slots;
            if (v1 > 0.0) { sh.slot_value[ns] = v1; sh.slot_parent[ns] = p; ++ns; }   // next sampling at this position
            if (v0 > 0.0) { sh.slot_value[ns] = v0; sh.slot_parent[ns] = i; ++ns; }   // first child of the new node
            sh.n_slots = ns;
        }
        if (tid < mask_words) {
            const uint64_t up = anc_mask[(size_t)(base + p) * mask_words + tid];
            anc_mask[(size_t)(base + i) * mask_words + tid] = up | ((tid == i / 64) ? (1ull << (i % 64)) : 0ull);
        }
        ++n;
        __syncthreads();
    }
    if (tid == 0) n_built[seq] = n;
}

// The form with a workspace: waves with roles.
//
// Wave 0 (control) pops.  Every node has one open slot, its next draw; the lanes of control hold the best 64 in
// order (the slots themselves lie in LDS), so the pop is lane 0's.  It takes the popped node's next draw (token, R[y], the
// new node's path key and first uniform) from
// LDS, opens the new node's slot and the parent's next one.
// Wave 1 draws from the root's row, which it keeps in LDS (wave_draw.h), up to kRing draws
// ahead, or, in trees that have helpers (below), brings the draws that these make.
// kDrawWaves waves draw for the other nodes (node i: wave i % kDrawWaves of them), one draw ahead per node and a
// second one put aside where the node has been drawn from twice, the node of the largest slot value first: totals from the workspace (a new node's were fetched before it
// was made: its row is known), a wave scan, the picked run's 128 logits, two per lane, a wave scan.
//
// LDS words, one writer at a time.  A node's word is, with the top bit clear, a request of control for
// draw `rank` (low bits: the upper bits of the slot value, the order in which requests are
// served), and with the top bit set the answer (the token; the rest of the draw lies beside it) or nothing (which may
// say that the node's draws come from a ring).  Control writes it only while the bit is set, the node's wave only while it is clear.  The root's
// draws go through a ring; `news` tells the draw waves which requests the last pop made.  LDS operations
// of a wave take effect in their order, so data written before a word are there for whoever has read the word.
//
// Every wait ends: control waits only for a requested draw, which the node's wave makes in finitely
// many steps whatever else happens (an empty row is an answer as well), or the node's helper, once it runs; the drawing waves leave when
// control has set `news` to kStop, which it does after at most N - 1 pops.  (Were an answer to stay out all the
// same, control gives up after kBuildPolls looks: the tree ends there, and n_built says so.)
//
// What bounds it: the number of instructions of control's pop and of wave 1's draw (a wave alone issues a vector one in 4.5
// cycles, one of eight bytes or in doubles in 5.5, a DPP move of what was just made in 12.5; an LDS read is back after 52), and
// where a node is popped again at once or a tree is one chain, those of a draw from memory (the trip itself is over before the Philox
// blocks made meanwhile).
// Measured against a workgroup that popped and drew in turn, two barriers a draw, with the pass over the rows: 512 rows of
// 32000 tokens 1378 -> 508 us (with eight drawing waves on two SIMDs 562, on all four 543: a request waits for the draw its
// wave is at), 128 rows 346 -> 134, 32 rows of 1000 tokens 92 -> 55; a single chain of 512 nodes 1413 -> 1130.  (All before
// the sorted list of slots, see pop_nodes.)  Of one size the time depends on the table, that is, on how often nodes
// are popped again: 178 to 349 us over tables of 512 rows of independent normal logits (before there were helpers, below, 470 to 960).
constexpr int kBuildThreads = 1024;
constexpr int kDrawWaves = kBuildThreads / kWave - 2;
static_assert(kRing * kRings == kWave, "a lane for every place");
constexpr uint32_t kAnswer = 0x80000000u;
constexpr uint32_t kStop = 0u;              // news of a pop is never 0: the new node's index is not
static_assert(DYSPEC_MAX_BUILD_NODES <= 1024 && DYSPEC_MAX_VOCAB <= (1 << 15), "parent, rank and previous sibling share a word, rank and token too");

// What LDS holds of a node; its last 24 bytes are what a place in a ring holds.
struct Node {
    double value;           // open slot (<= 0: none)
    unsigned long long key; // path key
    uint32_t opened;        // order in which the open slot was opened (2 i + 1: first child, 2 i: next sampling of the parent of node i)
    float u;                // uniform of the next draw
    uint32_t word;          // request or answer: kAnswer | rank << 15 | token
    float child_u;          // uniform of the first draw of the node the draw makes
    double r;               // its next draw, made ahead: R[y] (< 0: the row is empty),
    unsigned long long child_key;   // path key of the node the draw makes
};
constexpr uint32_t kNode = sizeof(Node), kValueAt = 0, kKeyAt = 8, kOpenedAt = 16, kUAt = 20, kWordAt = 24, kChildUAt = 28, kRAt = 32, kChildKeyAt = 40;
static_assert(kNode == 48 && offsetof(Node, value) == kValueAt && offsetof(Node, key) == kKeyAt && offsetof(Node, opened) == kOpenedAt && offsetof(Node, u) == kUAt &&
              offsetof(Node, word) == kWordAt && offsetof(Node, child_u) == kChildUAt && offsetof(Node, r) == kRAt && offsetof(Node, child_key) == kChildKeyAt, "");
// What LDS holds of a ring: the open slot of its node, the node's last child, the rank of the draw that opens next (draws below are taken).
struct RingState {
    double value;
    uint32_t last, taken;
};
constexpr uint32_t kTakenAt = 12;
static_assert(sizeof(RingState) == 16 && offsetof(RingState, taken) == kTakenAt, "");
constexpr uint32_t kPlace = kNode - kWordAt;                     // a place in a ring, addressed as if it were a node's
// Dynamic LDS of the builder: byte offsets.
struct BuildLds {
    static constexpr uint32_t ring = 0;                                            // places of the root's ring, draw r at r % kRing; with helpers the rings lie behind the nodes
    static constexpr uint32_t state = ring + kRing * kPlace;                       // of every ring (RingState)
    static constexpr uint32_t here = state + 16 * kRings;                          // bit k: helper k runs
    static constexpr uint32_t hot = here + 4;                                      // per ring: its node
    static constexpr uint32_t claims = hot + 4 * kRings;                           // bit k: ring k has a node
    static constexpr uint32_t caught_up = claims + 4;                              // bit k: and its helper has the draws that are taken next
    static constexpr uint32_t news = caught_up + 4;                                   // new node | popped node << 10 | kRequest if it was asked for another draw
    static constexpr uint32_t n_built = news + 4;
    static constexpr uint32_t fred = n_built + 4;
    static constexpr uint32_t gone = fred + 4 * (kBuildThreads / kWave);          // drawn tokens of the run a wave is drawing from
    static_assert(state % 16 == 0, "");
    static constexpr uint32_t nodes = (gone + kDrawWaves * (kRun / 8) + 15) / 16 * 16;
    __host__ __device__ static constexpr uint32_t row(int widest) { return nodes + kNode * widest; }
};
constexpr uint32_t kRequest = 1u << 20;
constexpr size_t kLdsPerWorkgroup = 160 * 1024;
static_assert(BuildLds::row(DYSPEC_MAX_BUILD_NODES) <= kLdsPerWorkgroup, "the node state of the largest tree fits in LDS");

__device__ __forceinline__ u64 join_key(uint2 k) { return (u64)k.x | ((u64)k.y << 32); }
__device__ __forceinline__ uint2 split_key(u64 k) { return make_uint2((uint32_t)k, (uint32_t)(k >> 32)); }
__device__ __forceinline__ void keep_order() { asm volatile("" ::: "memory"); }
// What the lane publishes: the draw, then its word.
__device__ __forceinline__ void publish(uint32_t place, double r, u64 key, float u, uint32_t word)
{
    *lds_at<double>(place + kRAt) = r;
    *lds_at<u64>(place + kChildKeyAt) = key;
    *lds_at<float>(place + kChildUAt) = u;
    lds_set(lds_at<uint32_t>(place + kWordAt), word);
}

// The roles are functions of their own, so that each has the scalar registers to itself; their arguments arrive
// in vector registers and are declared uniform again.
// Where in a 64-byte line of instructions their loops lie moves all times by 1 - 2 %, so each begins at a line and so many
// instructions behind: against none, 512 rows of 32000 tokens 608 -> 603, 462 -> 455 and (flat rows) 389 -> 382 us, a chain 1121 -> 1110.
template <int N> __device__ __forceinline__ void begin_behind() { asm volatile(".rept %0\n\ts_nop 0\n\t.endr" :: "n"(N)); }

// Wave 1: the root's draws, in order, up to kRing ahead of control.
__device__ __attribute__((noinline, aligned(64))) void draw_for_root(uint32_t lds_, uint32_t row_at, double inv_temp, double m, int V_, int N_, uint64_t seed_, uint32_t seq)
{
    begin_behind<15>();
    const uint32_t lds = uniform(lds_);
    const int V = uniform(V_), N = uniform(N_);
    const u64 seed = uniform((u64)seed_);
    const uint2 key = root_key(uniform(seq));
    WaveRow row;
    row.leaf = lds_at<double>(uniform(row_at));
    row.logits = lds_at<float>(uniform(row_at) + 8 * row_leaves(V));
    row.inv_temp = uniform(inv_temp);
    row.m = uniform(m);
    const int lane = threadIdx.x & 63;
    open_wave_row(row, V);
    float us = 0.f, child_u = 0.f;                  // of 64 ranks, one per lane: the draw's uniform, the child's first one,
    u64 child = 0;                                  // its key
    for (int rank = 0; rank < N - 1; ++rank) {
        if ((rank & 63) == 0) {
            const uint2 ck = child_key(seed, key, (uint32_t)(rank + lane));
            us = u01(seed, key, (uint32_t)(rank + lane), KIND_BUILD);
            child_u = u01(seed, ck, 0u, KIND_BUILD);
            child = join_key(ck);
        }
        uint32_t news = lds_now(lds_at<uint32_t>(lds + BuildLds::news));
        uint32_t taken = lds_now(lds_at<uint32_t>(lds + BuildLds::state + kTakenAt));
        Drawn d;
        const bool drawn = draw_wave_row(row, (double)readlane_f32(us, rank & 63), &d);
        const double R = drawn ? d.wy / d.W : -1.0;
        for (;;) {
            if (uniform(news) == kStop) return;
            if (rank - (int)uniform(taken) < kRing) break;
            __builtin_amdgcn_s_sleep(1);
            news = lds_now(lds_at<uint32_t>(lds + BuildLds::news));
            taken = lds_now(lds_at<uint32_t>(lds + BuildLds::state + kTakenAt));
        }
        // (lane rank % 64 has the child's key at hand)
        if (lane == (rank & 63))
            publish(lds + BuildLds::ring - kWordAt + (uint32_t)(rank % kRing) * kPlace, R, child, child_u, kAnswer | ((uint32_t)rank << 15) | (uint32_t)(drawn ? d.y : 0));
        if (!drawn) return;
    }
}

// A draw wave's copy of a node's totals (lane l: totals 4 l .. 4 l + 3), row maximum and first 64 tokens drawn (lane r: draw r's,
// once it is made); which copies it keeps: row_copies.h.
struct HeldRow {
    int node;               // -1: none
    double tot[4], m;
    int drawn;
};
__device__ __forceinline__ void fetch_row(double* ws, int base, int i, HeldRow& h)
{
    const double* const t = ws_totals(ws, base + i) + 4 * (threadIdx.x & 63);
    h.node = i;
#pragma unroll
    for (int k = 0; k < 4; ++k) h.tot[k] = t[k];
    h.m = *ws_rowmax(ws, base + i);
    h.drawn = ws_drawn(ws, base + i)[threadIdx.x & 63];
}

// Of 64 ranks of a node's draws (first + lane): the draw's uniform, the path key of the node the draw makes, that node's first uniform.
// A node drawn from again gets them for the next 64 draws at once; the first draw, the only one of most nodes, makes its own.
struct DrawNames {
    int node, first;
    float u, child_u;
    u64 child;
};
__device__ __forceinline__ void make_names(DrawNames& d, uint64_t seed, u64 key_word, int node, int rank)
{
    const uint2 key = split_key(key_word);
    d.node = node;
    d.first = rank & ~(kWave - 1);
    const uint32_t r = (uint32_t)(d.first + (int)(threadIdx.x & 63));
    const uint2 child = child_key(seed, key, r);
    d.u = u01(seed, key, r, KIND_BUILD);
    d.child_u = u01(seed, child, 0u, KIND_BUILD);
    d.child = join_key(child);
}

// A draw made, as it is handed to control.
struct MadeDraw {
    int node, rank;         // -1: none
    double R;
    u64 child;
    float child_u;
    uint32_t word;
};
// One that has not been asked for waits in the workspace (lane 0 writes and reads it).
__device__ __forceinline__ void put_made(double* ws, int ws_row, const MadeDraw& d)
{
    double* const at = ws_made(ws, ws_row);
    at[0] = d.R;
    at[1] = __longlong_as_double((long long)d.child);
    at[2] = __hiloint2double((int)d.word, __float_as_int(d.child_u));
}
__device__ __forceinline__ void get_made(double* ws, int ws_row, MadeDraw& d)
{
    const double* const at = ws_made(ws, ws_row);
    const double last = at[2];
    d.R = at[0];
    d.child = (u64)__double_as_longlong(at[1]);
    d.child_u = __int_as_float(__double2loint(last));
    d.word = (uint32_t)__double2hiint(last);
}

// One draw for a node of a sequence by a wave, the node's row in global memory: what is left of its
// totals lies in the workspace (totals 4 l .. 4 l + 3 are read and written by lane l), as do the tokens drawn
// before (entry r by lane r % 64); this wave alone draws for the node.  `asked`: control waits for it, else it is put aside.
//
// A node that has been drawn from twice is likely to be popped several times in a row, and control then waits for its wave alone,
// some 560 instructions a draw.  So from its third draw on a node's draw is made when the one before is handed over, and handed over at
// once when it is asked for.  512 rows of 32000 tokens, three tables: 470 -> 409, 441 -> 404, 520 -> 490 us, 1024 rows of 32768 1542 -> 1311,
// of which half by the logits' load, which is no longer waited for where it is made (the Philox blocks follow).
// (Only the run, its logits and names made ready ahead, the draw made when asked for: 471, 441, 524; the same after a look
// at the wave's other requests: 524, 484, 562.)
// Rank r + 1 is of use in trees of at least r + 3 rows; smaller ones only ended after the draw (2 rows of 32000 tokens 18.1 us,
// with it 19.2; 3 rows of 32001 25.5, 26.8).
template <bool VEC>
__device__ __forceinline__ void draw_for_node(MadeDraw& d, uint32_t place, uint32_t gone, const float* __restrict__ row, int V, double inv_temp,
                                              uint64_t seed, double* ws, int ws_row, HeldRow& h, DrawNames& names, int node, int rank, bool asked)
{
    const int lane = threadIdx.x & 63;
    d.node = asked ? -1 : node;
    d.rank = rank;
    d.R = -1.0;
    d.child = 0ull;
    d.child_u = 0.f;
    d.word = kAnswer;
    const auto hand_over = [&]() __attribute__((always_inline)) {
        if (lane == 0) {
            if (asked) publish(place, d.R, d.child, d.child_u, d.word);
            else put_made(ws, ws_row, d);
        }
    };
    const u64 key_word = *lds_at<u64>(place + kKeyAt);
    if (rank > 0 && (rank & (kWave - 1)) == 0) make_names(names, seed, key_word, node, rank);     // (the draw before has not left this one's uniform)
    const bool named = names.node == node && names.first == (rank & ~(kWave - 1));                 // uniform
    const double u = (double)(named ? readlane_f32(names.u, rank & (kWave - 1)) : *lds_at<float>(place + kUAt));
    const RunSums sums = sum_runs(h.tot);
    if (!(sums.W > 0.0)) {                          // nothing left to sample under the node
        hand_over();
        return;
    }
    const PickedRun run = pick_run(h.tot, sums, u);
    const int run0 = (4 * run.lane + run.k) * kRun;
    const int tok0 = run0 + 2 * lane;               // this lane's two tokens of the run
    // (past the end of the row a token that is there is read: with the loads in a branch of their own they are waited for in it)
    float2 x;
    if constexpr (VEC) {
        x = *reinterpret_cast<const float2*>(row + (tok0 < V ? tok0 : 0));
    } else {
        x.x = row[min(tok0, V - 1)];
        x.y = row[min(tok0 + 1, V - 1)];
    }
    unsigned short* const drawn = ws_drawn(ws, ws_row);
    uint32_t out = 0u;                              // bit e: token tok0 + e was drawn here before
    uint2 child;
    float next_u, child_u;
    // ---- while the logits are on their way: the tokens drawn before, the key of the node this draw makes, its first uniform, the
    //      uniform of this node's next draw
    if (rank == 0) {
        // lane 0 the key, lane 1 the next draw's uniform
        const uint2 key = split_key(key_word);
        const uint4 blk = philox4x32_10(make_uint4(key.x, key.y, (uint32_t)(lane & 1), (lane & 1) ? KIND_BUILD : KIND_PATH), seed_key(seed));
        child = make_uint2((uint32_t)__builtin_amdgcn_readlane((int)blk.x, 0), (uint32_t)__builtin_amdgcn_readlane((int)blk.y, 0));
        next_u = (float)(blk.x >> 8) * (1.0f / 16777216.0f);                        // lane 1's counts
        child_u = u01(seed, child, 0u, KIND_BUILD);
    } else {
        if (lane < kRun / 32) lds_set(lds_at<uint32_t>(gone + 4 * lane), 0u);
        auto leave_out = [&](int t) __attribute__((always_inline)) {
            if (t / kRun * kRun == run0)
                __hip_atomic_fetch_or(lds_at<uint32_t>(gone + 4 * (t % kRun / 32)), 1u << (t % 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        };
        if (lane < rank) leave_out(h.drawn);
        for (int c = lane + kWave; c < rank; c += kWave) leave_out(drawn[c]);
        out = lds_now(lds_at<uint32_t>(gone + 4 * (lane / 16))) >> (2 * (lane & 15));
        if (!named) make_names(names, seed, key_word, node, rank);
        const int at = rank & (kWave - 1);
        child = make_uint2((uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)names.child, at), (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(names.child >> 32), at));
        next_u = names.u;                                                           // lane at + 1's counts
        child_u = readlane_f32(names.child_u, at);
    }
    // ---- the token: as above among the run's 128
    double z[2], w[2];
    z[0] = fma((double)(tok0 < V ? x.x : -INFINITY), inv_temp, -h.m);
    z[1] = fma((double)(tok0 + 1 < V ? x.y : -INFINITY), inv_temp, -h.m);
    exp_nonpos_xn<2>(z, w);
    if (out & 1u) w[0] = 0.0;
    if (out & 2u) w[1] = 0.0;
    const TokenSums tokens = sum_tokens(w);
    if (!tokens.live) {                             // (the run's total says otherwise: not while totals and logits belong together)
        hand_over();
        return;
    }
    const PickedToken t = pick_token(w, tokens, run);
    const int y = run0 + 2 * t.lane + t.second;
    if (lane == ((rank + 1) & (kWave - 1))) *lds_at<float>(place + kUAt) = next_u;
    d.R = t.wy / sums.W;
    d.child = join_key(child);
    d.child_u = child_u;
    d.word = kAnswer | ((uint32_t)rank << 15) | (uint32_t)y;
    hand_over();
    // what is left of the run
    const double left = run_left(w, tokens, t);
    const bool here = lane == run.lane;
#pragma unroll
    for (int q = 0; q < 4; ++q) h.tot[q] = here && q == run.k ? left : h.tot[q];       // (selects: a store to tot[k] puts the array in scratch memory)
    if (here) ws_totals(ws, ws_row)[4 * lane + run.k] = left;
    if (lane == (rank & 63)) {
        drawn[rank] = (unsigned short)y;
        if (rank < kWave) h.drawn = y;
    }
}

// Draw wave `mine`: serves the requests of its nodes, the largest slot value first, until told to stop.
template <bool VEC>
__device__ __attribute__((noinline, aligned(64))) void draw_for_nodes(uint32_t lds_, int mine_, const float* draft_logits_, int V_,
                                                         double inv_temp_, uint64_t seed_, double* ws_, int base_, int N_)
{
    begin_behind<15>();
    const uint32_t lds = uniform(lds_);
    const int mine = uniform(mine_), V = uniform(V_), base = uniform(base_), N = uniform(N_);
    const float* __restrict__ const draft_logits = uniform(draft_logits_);
    const double inv_temp = uniform(inv_temp_);
    const u64 seed = uniform((u64)seed_);
    double* const ws = uniform(ws_);
    const int lane = threadIdx.x & 63;
    const uint32_t nodes = lds + BuildLds::nodes, gone = lds + BuildLds::gone + mine * (kRun / 8);
    RowCopies<HeldRow> rows;
    rows.open(mine);
    DrawNames names = { -1, 0, 0.f, 0.f, 0ull };
    MadeDraw made;                                  // the last draw put aside
    made.node = made.rank = -1;
    const auto fetch = [&](int i, HeldRow& h) __attribute__((always_inline)) { fetch_row(ws, base, i, h); };
    uint32_t seen = 1u << 31;                       // the news last looked at (none yet)
    bool look = mine == 0;                          // requests may be open (node 0's, at the start)
    for (;;) {
        rows.look_ahead(N, fetch);
        int i = -1, rank = 0;
        const auto wanted = [&]() __attribute__((always_inline)) {      // that draw has been asked for
            return made.node >= 0 && !(uniform(lds_now(lds_at<uint32_t>(nodes + kNode * made.node + kWordAt))) & kAnswer);
        };
        if (wanted()) {
            i = made.node;
            rank = made.rank;
        } else if (look) {
            // the best request of each lane's nodes, then of the wave
            int best = 0, node = 0;
#pragma unroll
            for (int s = 0; s < (DYSPEC_MAX_BUILD_NODES + kDrawWaves * kWave - 1) / (kDrawWaves * kWave); ++s) {
                const int q = mine + kDrawWaves * (lane + s * kWave);
                if (q < N) {
                    const uint32_t w = lds_now(lds_at<uint32_t>(nodes + kNode * q + kWordAt));
                    const int p = (w & kAnswer) ? 0 : (int)(w & 0x7fffu) + 1;
                    if (p > best) { best = p; node = q | (int)(w >> 15) << 16; }
                }
            }
            const int top = wave_max_dpp_int(best);
            if (top > 0) {
                const int nr = __builtin_amdgcn_readlane(node, __builtin_ctzll(ballot(best == top)));
                i = nr & 0xffff;
                rank = nr >> 16;
            }
        }
        if (i < 0) {                                // nothing to do: wait for news
            uint32_t m;
            while ((m = uniform(lds_now(lds_at<uint32_t>(lds + BuildLds::news)))) == seen) __builtin_amdgcn_s_sleep(1);
            if (m == kStop) return;
            // the requests of one pop, if it is the one after the last seen; else look at all
            const int a = (int)(m & 1023u), p = (int)(m >> 10) & 1023;
            const bool a_mine = a % kDrawWaves == mine, p_mine = (m & kRequest) && p % kDrawWaves == mine;
            const bool one = a == (int)(seen & 1023u) + 1;
            seen = m;
            if (p_mine && p == made.node && wanted()) {
                look = !one || a_mine;              // after it has been served
                i = made.node;
                rank = made.rank;
            } else {
                look = !one || (a_mine && p_mine);
                if (look || !(a_mine || p_mine)) continue;
                look = true;                        // ... after it has been served
                i = a_mine ? a : p;
                const uint32_t w = uniform(lds_now(lds_at<uint32_t>(nodes + kNode * i + kWordAt)));
                if (w & kAnswer) continue;          // served already
                rank = (int)(w >> 15);
            }
        }
        bool asked = true;
        if (rank > 1) {                             // made when the one before was asked for
            if (made.node != i) get_made(ws, base + i, made);
            if (lane == 0) publish(nodes + kNode * i, made.R, made.child, made.child_u, made.word);
            asked = false;
            ++rank;
        }
        for (;;) {
            rows.hold(i, kDrawWaves, fetch);
            draw_for_node<VEC>(made, nodes + kNode * i, gone, draft_logits + (size_t)(base + i) * V, V, inv_temp, seed, ws, base + i, rows.held, names, i, rank, asked);
            if (!asked || rank == 0 || rank + 3 > N) break;     // (a tree complete by then: its last pop's request is nobody's to wait for)
            asked = false;
            ++rank;
        }
        if (uniform(lds_now(lds_at<uint32_t>(lds + BuildLds::news))) == kStop) return;
    }
}

// ---- Helpers: workgroups on CUs of their own, each for one node that is drawn from again and again.
//
// Rules.  A batch has helpers if its widest tree has kHelpedRows rows and kRings more workgroups a sequence leave each a CU of its own
// (kHelpedBlocks), a tree of it from kLeastHelped rows on.  The root gets the first helper when it is popped, another node one from its pop
// of rank kClaimRank on, while more than kHelpedLeft rows are to be built and a helper runs that no node has (free_ring).  kOwnDraws after
// the claim at the earliest, and once the helper has caught up with the node's own wave (hand_over), the node's draws come from the helper.
//
// A draw from global memory takes a wave 2.1 us, one from a row in LDS 0.67, and the tree's workgroup has room for the root's row at most.
// A helper brings the node's row into its LDS, makes the node's draws from rank 0 on (they depend on the row and the path key
// alone) and leaves them in a ring in memory (row_workspace.h); wave 1 of the tree's workgroup brings them to a ring in LDS (helper_rings.h).
// When a helper takes over depends on the clock; a draw has the same bits whoever makes it (run_draw.h).
//
// Words in memory, all accesses relaxed and device-scope: the mailbox's state (the helper comes: kHere; wave 1 claims it; one that has
// waited too long leaves), its other word (wave 1: draws taken, or that the tree is complete), the count of draws that can be read (helper;
// written when they are there).  Waits: for a claim a helper looks a bounded number of times.  Once it is claimed it stays until wave 1 says that the
// tree is complete, which it does when control ends, after a bounded number of looks of its own (kBuildPolls).  Only a helper that runs is
// claimed: nobody waits for a workgroup that has no CU, and a tree without its helpers is built by its own waves.
//
// Measured, with the pass over the rows: 512 rows of 32000 tokens, four tables, without helpers, with them and with their draws popped
// many at a time (pop_nodes): 961, 470, 582, 553 -> 334, 320, 332, 319 -> 332, 201, 225, 211 us; all draws from
// the root 381 -> 360, from another node 1091 -> 371; 1024 rows of 32768 tokens 1876 -> 597 -> 550, 64 rows 124 -> 80, 128 rows
// 222, 134, 177 -> 128, 110, 123 -> 118, 88, 107.  (These with a claim at rank 3, eight more draws of the node's own wave, and draws of 0.63 us
// that had other bits than the own wave's.)  Now, three tables of 512 rows 349, 178, 205 us, two of 128 rows 117 and 81, all draws from
// one node 390, 1024 rows of 32768 tokens 580.  What is left is, where one node has all the draws, its helper's draw, and where slots of
// single draws come between, their pop, 0.5 us.
// kClaimRank, kOwnDraws: at the node's second pop and four draws, as a helper has its first draw 8 us after it is told: the four tables 329, 179, 198,
// 209 us, 128 rows 111, 83, 86.  Of 190 shapes of 64 to 512 rows (1000 to 32000 tokens, deviation 2 and 3, Zipf) the times are 0.985 of those
// with rank 3 and eight draws, the best 0.83, the worst 1.03; peaked rows (deviation 10), whose nodes are hardly popped three times, 1.01, the worst
// 1.07.  A claim at the first pop: 0.983 and 1.03, the worst of the former 1.08; at the third 0.989 and 1.00, 1.04.  Told apart by R[y] (below
// 1/4, 1/8, 1/16 at rank 1): 0.995, the peaked ones no better.
// kHelpedRows: below, a node has hardly the draws to pay for a row's loading (some 8 us before the first draw is there).
// kHelpedBlocks: 28 sequences of 64 rows hold 252 CUs.  Such a call takes 145 us by itself (197 without helpers), beside another like it 223 for both (219),
// beside four verifications of 512 rows on another stream 253 (216); 28 sequences of 200 rows 330 (545), 577 for two (638), 417 (566).
constexpr int kClaimRank = 1, kOwnDraws = 4, kRootOwnDraws = 2;        // draws the node's own wave makes after the claim, at least
constexpr int kHelpedRows = 64;             // of the widest tree of a batch that has helpers,
constexpr int kLeastHelped = 16;            // of any tree of it that has some (a mailbox each in its rows)
constexpr int kHelpedLeft = 24;             // rows still to be built when a node is worth a helper
constexpr int kHelpedBlocks = 256;          // one workgroup a CU
constexpr int kHelperPolls = 1 << 22;       // some seconds
static_assert(kLeastHelped >= kRings, "");
constexpr uint32_t kHere = 1u, kClaimed = 2u;                   // mailbox state; claimed: | node << 2
constexpr uint32_t kStopped = 0x80000000u;                      // beside the number of draws taken
typedef double doublex2 __attribute__((ext_vector_type(2)));
constexpr uint32_t kHelpPlace = 32;                             // wy, W, y of a draw
struct HelpLds {
    static constexpr uint32_t node = 0;
    static constexpr uint32_t made = 4;                                            // draws made,
    static constexpr uint32_t room = 8;                                            // draws that may be made (kStopped: no more)
    static constexpr uint32_t fred = 16;
    static constexpr uint32_t ring = fred + 4 * (kBuildThreads / kWave);
    static constexpr uint32_t totals = ring + kMailRing * kHelpPlace;
    static constexpr uint32_t row = totals + 8 * kSums;
};
static_assert(HelpLds::totals % 16 == 0 && HelpLds::row % 16 == 0, "");
template <typename T> __device__ __forceinline__ T agent_load(const T* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
template <typename T> __device__ __forceinline__ void agent_store(T* p, T v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void memory_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
__device__ __forceinline__ u64* mail_words(double* mail) { return reinterpret_cast<u64*>(mail); }               // state | taken << 32
__device__ __forceinline__ uint32_t* mail_state(double* mail) { return reinterpret_cast<uint32_t*>(mail); }
__device__ __forceinline__ uint32_t* mail_taken(double* mail) { return reinterpret_cast<uint32_t*>(mail) + 1; }
__device__ __forceinline__ u64* mail_key(double* mail) { return reinterpret_cast<u64*>(mail + 1); }
__device__ __forceinline__ uint32_t* mail_count(double* mail) { return reinterpret_cast<uint32_t*>(mail + 2); }

// A helper's first wave: draws rank 0 .. N - 2 of the row in LDS, as far as there is room, and leaves them in the ring in LDS.
__device__ __attribute__((noinline, aligned(64))) void make_draws(uint32_t lds_, double inv_temp, double m, int N_, uint64_t seed_, u64 key_)
{
    const uint32_t lds = uniform(lds_), ring = lds + HelpLds::ring;
    const int N = uniform(N_);
    const u64 seed = uniform((u64)seed_);
    const uint2 key = split_key(uniform(key_));
    RunRow row;
    row.logits = lds_at<float>(lds + HelpLds::row);
    row.inv_temp = uniform(inv_temp);
    row.m = uniform(m);
    const int lane = threadIdx.x & 63;
    open_run_row(row, lds_at<double>(lds + HelpLds::totals));
    float us = 0.f;                                 // the uniforms of 64 ranks
    for (int rank = 0; rank < N - 1; ++rank) {
        if ((rank & 3) == 0) {
            if ((rank & 63) == 0) us = u01(seed, key, (uint32_t)(rank + lane), KIND_BUILD);
            for (;;) {                              // (ends when the second wave ends, at the latest)
                const uint32_t room = uniform(lds_now(lds_at<uint32_t>(lds + HelpLds::room)));
                if (room == kStopped) return;
                if (rank + 4 <= (int)room) break;
                __builtin_amdgcn_s_sleep(2);
            }
        }
        // (all lanes write what one would: with a branch on the lane, or one that the compiler joins with it, the whole loop is run under masks)
        Drawn d = { 0, -1.0, 1.0 };
        uint32_t drawn = draw_run_row(row, (double)readlane_f32(us, rank & 63), &d) ? 1u : 0u;
        asm("" : "+s"(drawn));
        const uint32_t place = ring + kHelpPlace * (uint32_t)(rank & (kMailRing - 1));
        *lds_at<doublex2>(place) = doublex2{ d.wy, d.W };
        *lds_at<uint32_t>(place + 16) = (uint32_t)d.y;
        lds_set(lds_at<uint32_t>(lds + HelpLds::made), (uint32_t)rank + 1u);
        if (!drawn) return;
    }
}
// Its second wave: brings them to memory, where wave 1 of the tree's workgroup reads them.
__device__ __attribute__((noinline)) void ship_draws(uint32_t lds_, double* mail_, double* ring_)
{
    const uint32_t lds = uniform(lds_);
    double *const mail = uniform(mail_), *const ring = uniform(ring_);
    const int lane = threadIdx.x & 63;
    int shipped = 0;
    for (int polls = 0; polls < kHelperPolls; ++polls) {
        const int made = (int)uniform(lds_now(lds_at<uint32_t>(lds + HelpLds::made)));
        const u64 words = agent_load(mail_words(mail));
        if (made > shipped) {
            if (draw_of_place<kMailRing>(shipped, lane) < made) {
                const uint32_t place = lds + HelpLds::ring + kHelpPlace * (uint32_t)lane;
                const double wy = *lds_at<double>(place), W = *lds_at<double>(place + 8);
                agent_store(ring + 2 * lane, wy / W);
                agent_store(reinterpret_cast<uint32_t*>(ring + 2 * lane + 1), *lds_at<uint32_t>(place + 16));
            }
            memory_done();                          // they are where they can be read
            if (lane == 0) agent_store(mail_count(mail), (uint32_t)made);
            shipped = made;
        }
        const uint32_t taken = uniform((uint32_t)(words >> 32));
        if (taken & kStopped) break;
        if (lane == 0) lds_set(lds_at<uint32_t>(lds + HelpLds::room), (uint32_t)draws_allowed<kMailRing>((int)taken));
        if (polls == kHelperPolls - 1) {            // (the root's helper, whose tree's workgroup may have no CU yet)
            uint32_t was = kHere;
            if (lane == 0) __hip_atomic_compare_exchange_strong(mail_state(mail), &was, 0u, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (uniform(was) != kHere) polls = 0;   // claimed: goes on
        }
    }
    if (lane == 0) lds_set(lds_at<uint32_t>(lds + HelpLds::room), kStopped);
}

// Helper `mine` of a sequence.  The first one is the root's.
template <bool VEC>
__device__ __attribute__((noinline)) void help_build(uint32_t lds_, const float* draft_logits_, int V_, double inv_temp_, uint64_t seed_, double* ws_, int base_, int N_, int mine_, uint32_t seq_)
{
    const uint32_t lds = uniform(lds_);
    const int V = uniform(V_), base = uniform(base_), N = uniform(N_), mine = uniform(mine_);
    const float* const draft_logits = uniform(draft_logits_);
    const double inv_temp = uniform(inv_temp_);
    double* const ws = uniform(ws_);
    double* const mail = ws_mail(ws, base + mine);
    const int lane = threadIdx.x & 63, wave = uniform((int)(threadIdx.x >> 6));
    int node = 0;
    if (wave == 0 && lane == 0) {
        agent_store(mail_state(mail), kHere);
        *lds_at<uint32_t>(lds + HelpLds::made) = 0u;
        *lds_at<uint32_t>(lds + HelpLds::room) = (uint32_t)kMailRing;
    }
    if (mine > 0) {
        if (wave == 0) {
            node = -1;
            for (int polls = 0; polls < kHelperPolls; ++polls) {
                const u64 w = uniform(agent_load(mail_words(mail)));
                if ((uint32_t)(w >> 32) & kStopped) break;
                if (((uint32_t)w & 3u) == kClaimed) {
                    node = (int)((uint32_t)w >> 2);
                    break;
                }
                if (polls == kHelperPolls - 1) {    // the tree's workgroup may have no CU yet: leaves, unless it has been claimed just now
                    uint32_t was = kHere;
                    if (lane == 0) __hip_atomic_compare_exchange_strong(mail_state(mail), &was, 0u, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    was = uniform(was);
                    if ((was & 3u) == kClaimed) node = (int)(was >> 2);
                }
                __builtin_amdgcn_s_sleep(4);
            }
            if (lane == 0) *lds_at<int>(lds + HelpLds::node) = node;
        }
        __syncthreads();
        node = uniform(*lds_at<int>(lds + HelpLds::node));
        if (node < 0 || node >= N) return;
    }
    const double m = load_run_row<kBuildThreads, VEC>(draft_logits + (size_t)(base + node) * V, V, inv_temp, lds_at<double>(lds + HelpLds::totals),
                                                      lds_at<float>(lds + HelpLds::row), (float*)lds_at<float>(lds + HelpLds::fred));
    if (wave == 0) make_draws(lds, inv_temp, m, N, seed_, mine > 0 ? agent_load(mail_key(mail)) : join_key(root_key(uniform(seq_))));
    else if (wave == 1) ship_draws(lds, mail, ws_mail_ring(ws, base, N, mine));
}

// Wave 1 of a tree with helpers: fills the rings in LDS from the helpers'.  Lane 8 k + j has place j of ring k.
__device__ __attribute__((noinline, aligned(64))) void bring_draws(uint32_t lds_, uint32_t rings_, double* ws_, int base_, int N_, uint64_t seed_)
{
    const uint32_t lds = uniform(lds_), rings = uniform(rings_);
    const int base = uniform(base_);
    const u64 seed = uniform((u64)seed_);
    double* const ws = uniform(ws_);
    const int lane = threadIdx.x & 63, k = lane / kRing, j = lane % kRing;
    double* const mail = ws_mail(ws, base + k);
    const double* const ring = ws_mail_ring(ws, base, uniform(N_), k);
    const bool first = j == 0;
    uint32_t asked = 0, claimed = 0, ready = 0;     // rings that have a node, whose helper has been told, whose helper has caught up
    u64 here = 0, key = 0;
    int put = -1, told = 0, count = 0;              // the draw last put into the place, what the helper knows to be taken, what it has told of
    while (uniform(lds_now(lds_at<uint32_t>(lds + BuildLds::news))) != kStop) {
        const uint32_t claims = uniform(lds_now(lds_at<uint32_t>(lds + BuildLds::claims)));
        const bool used = claimed >> k & 1u, all_here = here == 0x0101010101010101ull;
        const int taken = used ? (int)lds_now(lds_at<uint32_t>(lds + BuildLds::state + 16 * k + kTakenAt)) : 0;
        const int rank = draw_of_place<kRing>(taken, j);
        const bool wanted = used && rank > put, get = wanted && rank < count;
        // (all of a look's loads are on their way together)
        const uint32_t state = all_here ? kHere : agent_load(mail_state(mail));
        uint32_t now = 0, y = 0;
        double R = 0.0;
        if (wanted) now = agent_load(mail_count(mail));
        if (get) {
            const double* const at = ring + 2 * (rank & (kMailRing - 1));
            R = agent_load(at);
            y = agent_load(reinterpret_cast<const uint32_t*>(at + 1));
        }
        if (ballot(get)) {
            const uint2 child = child_key(seed, split_key(key), (uint32_t)rank);
            const float child_u = u01(seed, child, 0u, KIND_BUILD);
            if (get) {
                publish(rings - kWordAt + kPlace * (uint32_t)lane, R, join_key(child), child_u, kAnswer | ((uint32_t)rank << 15) | y);
                put = rank;
            }
        }
        count = max(count, (int)now);
        if (claimed != ready) {
            ready |= ring_bits(ballot(used && first && helper_caught_up(count, taken)));
            if (lane == 0) lds_set(lds_at<uint32_t>(lds + BuildLds::caught_up), ready);
        }
        if (!all_here) {
            here |= ballot(first && state == kHere);
            if (lane == 0) lds_set(lds_at<uint32_t>(lds + BuildLds::here), ring_bits(here));
        }
        if (claims != asked) {
            const bool mine = (claims & ~asked) >> k & 1u;
            int node = 0;
            if (mine) {
                node = *lds_at<int>(lds + BuildLds::hot + 4 * k);
                key = *lds_at<u64>(lds + BuildLds::nodes + kNode * (uint32_t)node + kKeyAt);
                if (first) agent_store(mail_key(mail), key);
            }
            memory_done();
            uint32_t was = 0;
            if (mine && first) {
                was = kHere;
                __hip_atomic_compare_exchange_strong(mail_state(mail), &was, kClaimed | (uint32_t)node << 2, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            const u64 got = ballot(was == kHere);    // bit 8 k; (a helper that has left meanwhile has not been got)
            claimed |= ring_bits(got);
            asked = claims;
        }
        if (used && first && taken > told) {
            agent_store(mail_taken(mail), (uint32_t)taken);
            told = taken;
        }
        if (!ballot(wanted)) __builtin_amdgcn_s_sleep(2);
    }
    if (first) agent_store(mail_taken(mail), kStopped);
}

// The larger of two values, neither a NaN (fmax would first quiet what it cannot know to be none).
__device__ __forceinline__ double larger(double a, double b)
{
    double r;
    asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
// Largest of the rings' non-negative values (the same in the kRing lanes of each), in scalar registers.
__device__ __forceinline__ double largest_of_rings(double x)
{
    static_assert(kRing == 8 && kRings == 8, "eight by eight lanes");
    x = larger(x, dpp_or_zero<0x118>(x));
    x = larger(x, dpp_or_zero<kDppBcast15, 0xa>(x));
    x = larger(x, dpp_or_zero<kDppBcast31, 0xc>(x));
    return readlane_f64(x, 63);
}

// Wave 0: pops and appends.  Returns the number of rows built, its complement if a draw stayed out.  Row i's parent | rank << 10 | previous
// sibling << 20 goes to `parent` for the time being.
//
// The frontier is a sorted list in the lanes: lane k holds the k-th best open slot, of equal values the one opened first (an
// empty place: value -1).  A pop takes lane 0; the popped node's next slot goes where its value belongs, and the lanes before
// that place move up by one; the new node's slot makes the lanes behind its place move down.  A slot that finds no place among
// the 64 is left out: `unlisted` is the largest value left out so far, and while lane 0 is above it the list is as good as the
// whole frontier.  Else the list is made again from the slots in LDS (`relist`): a few times in trees of many equally good
// slots and in large ones of peaked tables, seldom in 512 rows of 1000 or 32000 tokens of independent normal logits of deviation 5.
// (512 rows with two equal tokens each, where every sixteenth pop does: 482 us, 505 with the maximum found at each pop, 720 with a list
// made by sixteen comparisons a lane for each of its entries.)
// Against the best of each lane's nodes kept in the lane and the maximum over the lanes found at each pop, and the other
// nodes of the popped one's lane looked over again: a pop whose draw is there 0.61 -> 0.51 us; with the draws' names
// for 64 ranks at once (DrawNames) 512 rows of 32000 tokens 441 -> 417, 495 -> 471 and 570 -> 547 us on three tables.
//
// The slots of nodes whose draws come from a ring are not in the list.  The lanes look at all rings at once, lane j of a ring at its j-th
// next draw: the draws that are there give the slots that the node will have, v (1 - R[y]) from one to the next, and those of the nodes to be
// made, v R[y].  The pops of an order are then known as far as slots are above every other one that may be open meanwhile: these draws are
// popped together, each lane making a node (its index: how many of them are larger).  A ring's slots only get smaller, so a ring's draws
// stay in their order.  Equal slots are popped singly, the one opened first first.  (What it gives: the helpers' figures.)
//
// Pops from the list make a loop of their own in which no branch depends on the lane: 768 rows, deviation 10, all pops but 49 from the list:
// 657 us before there were rings, 691 with the stores and moves under `lane == 0`, 644 now.  (As a function that is called, it saved and restored 35
// scalar registers and 2 vector registers in memory: 0.3 to 0.5 us of every tree, 11.9 us at the least.)
constexpr int kRelisted = 16;           // found one after the other
template <int CTRL> __device__ __forceinline__ int dpp_or_own(int x) { return __builtin_amdgcn_update_dpp(x, x, CTRL, 0xf, 0xf, false); }
template <int CTRL> __device__ __forceinline__ double dpp_or_own(double x)
{
    return __hiloint2double(dpp_or_own<CTRL>(__double2hiint(x)), dpp_or_own<CTRL>(__double2loint(x)));
}
struct Slots {
    double value;           // lane k: of the k-th best open slot,
    int node;               // and its node (| kSure: no slot left out comes before it, even if one is as large)
    double unlisted;        // no open slot outside the list is larger (the same in every lane)
};
constexpr int kSure = 1 << 16;

// The list made again from the slots of nodes 0 .. n - 1, node q in lane q % 64: the slots whose value's high word is above a line that
// is searched for, 32 to 64 of them where that can be had in few steps, each put where it belongs as a pop does.  Where the values
// near that line are too many of a kind (their high words equal), the kRelisted best, found one after the other: every lane's best;
// the best of those is listed and its lane's next one looked up by sixteen lanes at once.
// A peaked table's tree needs it most: of its first 1000 rows hundreds of slots lie within a factor of two, and a list of sixteen
// lasted sixteen pops at some 8 us a list.  960 rows of 32000 tokens, normal logits of deviation 10 at temperature 1: 812 us before there
// was a list, 1029 with sixteen slots at a time, 827 now; deviation 7.5: 935, 947, 806.  (Where most values are equal the search
// is for nothing: 1024 rows of two equal tokens 1098 -> 1105.)
__device__ __attribute__((noinline)) Slots relist(uint32_t nodes_, int n_)
{
    const uint32_t nodes = uniform(nodes_);
    const int n = uniform(n_), lane = threadIdx.x & 63;
    constexpr int Q = DYSPEC_MAX_BUILD_NODES / kWave;
    static_assert(Q == 16, "a row of lanes looks at a lane's nodes");
    {
        int high[Q], most = 0;                      // of positive values; as integers they are in the values' order
#pragma unroll
        for (int k = 0; k < Q; ++k) {
            const int q = lane + kWave * k;
            high[k] = q < n ? *lds_at<int>(nodes + kNode * q + kValueAt + 4) : 0;
            most = max(most, high[k]);
        }
        most = wave_max_dpp_int(most);
        const auto above = [&](int line) __attribute__((always_inline)) {      // (line >= 0: no closed slot)
            int c = 0;
#pragma unroll
            for (int k = 0; k < Q; ++k) c += __builtin_popcountll(ballot(high[k] > line));
            return c;
        };
        // `line` has at most 64 slots above it, `low` more, or is 0
        int line = most, listed = 0, step = 1 << 18, low = most, c = 0;
        do {
            low = max(low - step, 0);
            step <<= 2;
            c = above(low);
            if (c <= kWave) { line = low; listed = c; }
        } while (c < kWave / 2 && low > 0);
        for (int t = 0; t < 4 && listed < kWave / 2 && line - low > 1; ++t) {
            const int mid = low + (line - low) / 2;
            c = above(mid);
            if (c <= kWave) { line = mid; listed = c; } else low = mid;
        }
        if (listed >= kRelisted || (listed > 0 && line == 0)) {
            Slots s = { -1.0, 0, 0.0 };
            int opened = 0;
            double left = -1.0;
            for (int k = 0; kWave * k < n; ++k) {
                const int q = lane + kWave * k;
                double v = -1.0;
                int o = 0;
                if (q < n) {
                    v = *lds_at<double>(nodes + kNode * q + kValueAt);
                    o = (int)*lds_at<uint32_t>(nodes + kNode * q + kOpenedAt);
                }
                const bool take = __double2hiint(v) > line;
                left = fmax(left, take ? -1.0 : v);
                for (u64 m = ballot(take); m; m &= m - 1) {
                    const int l = __builtin_ctzll(m);
                    const double x = readlane_f64(v, l);
                    const int xo = __builtin_amdgcn_readlane(o, l);
                    const int at = __builtin_popcountll(ballot(s.value > x) | (ballot(s.value == x) & ballot(opened < xo)));
                    const double down_v = dpp_or_own<kDppWaveShr1>(s.value);
                    const int down_n = dpp_or_own<kDppWaveShr1>(s.node), down_o = dpp_or_own<kDppWaveShr1>(opened);
                    s.value = lane > at ? down_v : lane == at ? x : s.value;
                    s.node = lane > at ? down_n : lane == at ? (l + kWave * k) | kSure : s.node;
                    opened = lane > at ? down_o : lane == at ? xo : opened;
                }
            }
            left = wave_max_dpp(left);
            s.unlisted = left > 0.0 ? left : 0.0;
            return s;
        }
    }
    double best = -1.0;
    int at = 0, when = 0;
    for (int k = 0; kWave * k < n; ++k) {
        const int q = lane + kWave * k;
        if (q >= n) break;
        const double v = *lds_at<double>(nodes + kNode * q + kValueAt);
        const int o = (int)*lds_at<uint32_t>(nodes + kNode * q + kOpenedAt);
        if (v > 0.0 && (v > best || (v == best && o < when))) { best = v; at = k; when = o; }
    }
    uint32_t listed = 0;                            // bit k: node lane + 64 k is in the list
    Slots s = { -1.0, 0, 0.0 };
    for (int t = 0; t <= kRelisted; ++t) {
        const double top = wave_max_dpp(best);
        if (!(uniform(top) > 0.0)) break;
        if (t == kRelisted) { s.unlisted = top; break; }
        u64 cand = ballot(best == top);
        if (cand & (cand - 1)) {
            const int first = best == top ? 0xffff - when : 0;
            cand &= ballot(first == wave_max_dpp_int(first));
        }
        const int winner = __builtin_ctzll(cand), k = __builtin_amdgcn_readlane(at, winner);
        if (lane == t) { s.value = top; s.node = (winner + kWave * k) | kSure; }
        if (lane == winner) listed |= 1u << k;
        const int q = winner + kWave * (lane & 15);
        double v = -1.0;
        int o = 0;
        if (q < n && !(((uint32_t)__builtin_amdgcn_readlane((int)listed, winner) >> (lane & 15)) & 1u)) {
            v = *lds_at<double>(nodes + kNode * q + kValueAt);
            o = (int)*lds_at<uint32_t>(nodes + kNode * q + kOpenedAt);
            if (!(v > 0.0)) v = -1.0;
        }
        double m = v;                               // (every row of 16 lanes holds the same)
        m = fmax(m, dpp_or_zero<kDppXor1>(m));
        m = fmax(m, dpp_or_zero<kDppXor2>(m));
        m = fmax(m, dpp_or_zero<kDppHalfMirror>(m));
        m = fmax(m, dpp_or_zero<kDppMirror>(m));
        u64 same = ballot(v == m);
        if (same & 0xffffull & ((same & 0xffffull) - 1)) {
            const int first = v == m ? 0xffff - o : 0;
            same &= ballot(first == wave_max_dpp_int(first));
        }
        const int next = __builtin_ctzll(same), o_next = __builtin_amdgcn_readlane(o, next);
        if (lane == winner) { best = m; at = next; when = o_next; }
    }
    return s;
}

// A node that has no ring yet, popped for the draw of that rank: the ring (+ 1) that has its draws from the next one on, else 0.  Claims one
// for it if it is time.  (Control alone; what it remembers is in LDS.)
__device__ __forceinline__ uint32_t ring_for(uint32_t lds_, uint32_t p_, uint32_t rank_, uint32_t n_, uint32_t N_)
{
    const uint32_t lds = uniform(lds_), p = uniform(p_), rank = uniform(rank_), n = uniform(n_), N = uniform(N_);
    const uint32_t lane = threadIdx.x & 63, claims = uniform(*lds_at<uint32_t>(lds + BuildLds::claims));
    const u64 has = ballot(*lds_at<uint32_t>(lds + BuildLds::hot + 4 * (lane % kRings)) == p) & claims & ((1u << kRings) - 1u);
    if (has) {
        const uint32_t c = (uint32_t)__builtin_ctzll(has), taken_at = lds + BuildLds::state + 16 * c + kTakenAt;
        const uint32_t caught_up = uniform(lds_now(lds_at<uint32_t>(lds + BuildLds::caught_up)));
        const HandOver h = hand_over(rank, uniform(*lds_at<uint32_t>(taken_at)), caught_up >> c & 1u);
        if (h == kOwnDrawAndLater) lds_set(lds_at<uint32_t>(taken_at), rank + 2u);
        return h == kFromRing ? c + 1u : 0u;
    }
    const uint32_t c = free_ring(uniform(lds_now(lds_at<uint32_t>(lds + BuildLds::here))), claims, p == 0);
    if (c < kRings && n + kHelpedLeft < N) {
        *lds_at<uint32_t>(lds + BuildLds::state + 16 * c + kTakenAt) = rank + 1u + (p == 0 ? kRootOwnDraws : kOwnDraws);
        *lds_at<uint32_t>(lds + BuildLds::hot + 4 * c) = p;
        lds_set(lds_at<uint32_t>(lds + BuildLds::claims), claims | 1u << c);
    }
    return 0u;
}

// base[index], the index in a vector register
template <typename T> __device__ __forceinline__ void put_row(T* base, uint32_t index, T value) { *reinterpret_cast<T*>(reinterpret_cast<char*>(base) + (size_t)(4u * index)) = value; }

__device__ __forceinline__ int pop_nodes(uint32_t lds_, uint32_t rings_, int root_ring_, int helped_, int N_, int max_polls_, int* parent_, int* token_, float* est_value_)
{
    const uint32_t lds = uniform(lds_), nodes = lds + BuildLds::nodes, states = lds + BuildLds::state;
    const bool root_ring = uniform(root_ring_) != 0, helped = uniform(helped_) != 0;
    const uint32_t N = (uint32_t)uniform(N_);
    int *const parent = uniform(parent_), *const token = uniform(token_);
    float* const est_value = uniform(est_value_);
    const uint32_t lane = threadIdx.x & 63, k = lane / kRing, j = lane % kRing;
    Slots s = { lane == 0 && !root_ring ? 1.0 : -1.0, 0, 0.0 };
    // the rings that are in use (all lanes of one); per lane of ring k: its first place, its node, the
    // rank of its next draw
    u64 live = root_ring ? 0xffull : 0ull;
    const uint32_t places = uniform(rings_) - kWordAt + (helped ? kPlace * kRing * k : 0u);
    uint32_t ring_node = 0, next = 0;
    uint32_t n = 1;
    int polls = uniform(max_polls_);
    if (lane == 0) {
        token[0] = -1;
        est_value[0] = 1.0f;
    }
    // a new slot into the list, behind the slots (its first ones) of that mask; what finds no place is left out
    const auto insert = [&](double x, int node, u64 before) __attribute__((always_inline)) {
        const double out = before != ~0ull ? readlane_f64(s.value, 63) : x;
        const double down_v = dpp_or_own<kDppWaveShr1>(s.value);
        const int down_n = dpp_or_own<kDppWaveShr1>(s.node);
        const u64 upto = before << 1 | 1ull, at = upto & ~before;
        s.value = __builtin_amdgcn_inverse_ballot_w64(upto) ? s.value : down_v;
        s.node = __builtin_amdgcn_inverse_ballot_w64(upto) ? s.node : down_n;
        s.value = __builtin_amdgcn_inverse_ballot_w64(at) ? x : s.value;
        s.node = __builtin_amdgcn_inverse_ballot_w64(at) ? node : s.node;
        s.unlisted = larger(s.unlisted, out);
    };
    const auto list_sure = [&]() __attribute__((always_inline)) {       // the list's first slot is the best of all that no ring has
        return (ballot(s.value > s.unlisted) & 1ull) || (uniform((uint32_t)s.node) & kSure);
    };
    bool watch = helped, lost = false;              // for nodes to give a ring to
    uint32_t to_ring = 0;                           // the ring + 1 that has taken over the node popped last
    while (n < N) {
        if (polls <= 0) { lost = true; break; }
        if (to_ring) {                              // (the ring's words are control's own and in place)
            const uint32_t state = states + 16u * (to_ring - 1u);
            if (k == to_ring - 1u) {
                ring_node = *lds_at<uint32_t>(lds + BuildLds::hot + 4u * (to_ring - 1u));
                next = *lds_at<uint32_t>(state + kTakenAt);
            }
            live |= 0xffull << (kRing * (to_ring - 1u));
            watch = live != ~0ull;
            to_ring = 0;
        }
        // ---- the rings' draws: lane j of a ring has the j-th next one
        typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
        const double list = larger(uniform(s.value), s.unlisted);
        const u32x4 state = *lds_at<u32x4>(states + 16u * k);
        const double V = __hiloint2double((int)state.y, (int)state.x);
        if (ballot(V >= list) & live) {             // the best slot is a ring's
            const uint32_t rank = next + j, place = places + kPlace * (rank & (kRing - 1));
            const uint32_t w = lds_now(lds_at<uint32_t>(place + kWordAt));
            const double R = __longlong_as_double((long long)lds_now(lds_at<u64>(place + kRAt)));      // (as good as the word that was read before it)
            const u64 child = lds_now(lds_at<u64>(place + kChildKeyAt));
            const uint32_t child_u = lds_now(lds_at<uint32_t>(place + kChildUAt));
            constexpr u64 kFirsts = 0x0101010101010101ull, kButLasts = ~(kFirsts << 7);
            const bool there = (w >> 15) == (0x10000u | rank);
            // those that are there one after the other
            const u64 some = ballot(there && __double2hiint(R) >= 0) & live;
            u64 ok = some & (((some & kButLasts) + kFirsts) ^ kButLasts);
            // the slot that each is popped from, as deep as slots are above the list's, and what it opens
            const double q = 1.0 - R;
            double v = V;
            u64 deep = kFirsts;
#pragma unroll
            for (int t = 1; t < kRing; ++t) {
                if (!(ok & (kFirsts << (t - 1)) & ballot(v > list))) break;
                const double up = dpp_or_zero<0x111>(v * q);
                v = __builtin_amdgcn_inverse_ballot_w64(kFirsts << t) ? up : v;
                deep |= kFirsts << t;
            }
            ok &= deep;
            double v0 = v * R, v1 = v * q;
            // No slot that may be open meanwhile is above `bar`: the list's, those of the draws that come next or are not there, and the
            // first slots of the nodes that these draws make.  So all draws above it are popped, the largest first.  (High words;
            // draws that differ from it below those come one at a time.)
            int bar = __builtin_amdgcn_inverse_ballot_w64(ok) ? __double2hiint(v0) : 0;
            bar = max(bar, __builtin_amdgcn_inverse_ballot_w64(ok & ~((ok >> 1) & kButLasts)) ? __double2hiint(v1) : __builtin_amdgcn_inverse_ballot_w64(live & ~ok & kFirsts) ? __double2hiint(V) : 0);
            bar = wave_max_dpp_int(max(bar, __double2hiint(list)));
            u64 take = ballot(__double2hiint(v) > bar) & ok;
            uint32_t pos = 0;                       // how many are larger
            if (take & (take - 1)) {
                uint32_t same = 0;
                for (u64 m = take; m; m &= m - 1) {
                    const double x = readlane_f64(v, __builtin_ctzll(m));
                    pos += x > v;
                    same += x == v;
                }
                if (ballot(same > 1) & take) take = 0;      // two as large: one at a time
            }
            bool ring_next = true;
            if (take == 0) {
                // ---- one slot by itself: the best of the rings, of equal ones the one opened first (the order of the nodes' last
                //      children), or the list's first if that is as good and was opened before
                const double best_ring = largest_of_rings(__builtin_amdgcn_inverse_ballot_w64(live) ? V : 0.0);
                u64 heads = ballot(V == best_ring) & live & kFirsts;
                ring_next = (ballot(best_ring > 0.0) & 1ull) != 0;
                if ((ballot(s.value == best_ring) | ballot(s.unlisted == best_ring)) & 1ull) {
                    if (!list_sure()) {
                        s = relist(nodes, (int)n);
                        continue;
                    }
                    const uint32_t o = uniform(*lds_at<uint32_t>(nodes + kNode * (uniform((uint32_t)s.node) & (kSure - 1)) + kOpenedAt));
                    if (!(ballot(s.value < best_ring) & 1ull) && !(ballot(2u * state.z < o) & heads)) ring_next = false;
                }
                if (ring_next) {
                    int l = __builtin_ctzll(heads);
                    uint32_t first = (uint32_t)__builtin_amdgcn_readlane((int)state.z, l);
                    for (u64 m = heads & (heads - 1); m; m &= m - 1) {
                        const uint32_t z = (uint32_t)__builtin_amdgcn_readlane((int)state.z, __builtin_ctzll(m));
                        if (z < first) { first = z; l = __builtin_ctzll(m); }
                    }
                    take = 1ull << l;
                    pos = 0;
                    if (!(ok & take)) {
                        if (!(ballot(there) & take)) {              // its draw is still out
                            const uint32_t at = (uint32_t)__builtin_amdgcn_readlane((int)place, l), want = 0x10000u | (uint32_t)__builtin_amdgcn_readlane((int)rank, l);
                            while ((uniform(lds_now(lds_at<uint32_t>(at + kWordAt))) >> 15) != want && --polls > 0);
                            continue;
                        }
                        if (__builtin_amdgcn_readlane(__double2hiint(R), l) == (int)0xbff00000u) break;        // (-1) nothing left to sample
                        v0 = v;                     // the quotient of two infinite weights (see below)
                        v1 = 0.0;
                    }
                }
            }
            if (ring_next) {
                // ---- nodes n .. by their places, and the rings' next slots
                if ((uint32_t)__builtin_popcountll(take) > N - n) take &= ballot(pos < N - n);
                const uint32_t i = n + pos;
                const uint32_t beside = (uint32_t)dpp_or_zero<0x111>((int)i), before = j == 0 ? state.z : beside;         // the sibling before (asked for by all lanes)
                if (__builtin_amdgcn_inverse_ballot_w64(take)) {
                    const uint32_t place_i = nodes + kNode * i;
                    *lds_at<u64>(place_i + kKeyAt) = child;
                    *lds_at<uint32_t>(place_i + kUAt) = child_u;
                    *lds_at<double>(place_i + kValueAt) = v0;
                    keep_order();
                    lds_set(lds_at<uint32_t>(place_i + kWordAt), (uint32_t)__double2hiint(v0) >> 16);          // request of draw 0
                    put_row(token, i, (int)(w & 0x7fffu));
                    put_row(est_value, i, (float)v);
                    put_row(parent, i, (int)(ring_node | rank << 10 | before << 20));
                }
                const u64 ends = take & ~((take >> 1) & kButLasts);
                if (__builtin_amdgcn_inverse_ballot_w64(ends))
                    *lds_at<u32x4>(states + 16u * k) = u32x4{ (uint32_t)__double2loint(v1), (uint32_t)__double2hiint(v1), i, rank + 1u };
                n = uniform(n + (uint32_t)__builtin_popcountll(take));
                if (lane == 0) lds_set(lds_at<uint32_t>(lds + BuildLds::news), n - 1u);
                next += (uint32_t)__builtin_popcount((uint32_t)(take >> (kRing * k)) & 0xffu);
                // ---- the new nodes' slots
                const double lowest = readlane_f64(s.value, 63);
                for (u64 m = ballot(v0 > s.unlisted && !(v0 > lowest)) & take; m; m &= m - 1) s.unlisted = larger(s.unlisted, readlane_f64(v0, __builtin_ctzll(m)));
                for (u64 m = ballot(v0 > s.unlisted && v0 > lowest) & take; m; m &= m - 1) {
                    const int l = __builtin_ctzll(m);
                    const double x = readlane_f64(v0, l);
                    const int xi = __builtin_amdgcn_readlane((int)i, l);
                    // (of equal ones the one opened first: those listed before, or this time as an earlier node)
                    insert(x, xi, ballot(s.value > x) | (ballot(s.value == x) & ballot((s.node & (kSure - 1)) < xi)));
                }
                continue;
            }
        }
        // ---- the largest value of the list
        if (__builtin_expect(!list_sure(), 0)) {
            if (!(ballot(s.unlisted > 0.0) & 1ull)) break;              // no slot is open
            s = relist(nodes, (int)n);
            continue;
        }
        // One after the other while it is above the rings' and those left out.  No branch here depends on the lane (and so all lanes write
        // what one would): the loop is left to scalar branches as it stands then, else every path through it is a chain of copies.
        double line = live ? larger(s.unlisted, largest_of_rings(__builtin_amdgcn_inverse_ballot_w64(live) ? V : 0.0)) : s.unlisted;
        enum { kGoOn, kEnded, kLost };
        int status = kGoOn;
        do {
            const uint32_t p = uniform((uint32_t)s.node) & (kSure - 1);
            const double v = uniform(s.value);
            // ---- its node's next draw
            const uint32_t place_p = nodes + kNode * p;
            uint32_t w = lds_now(lds_at<uint32_t>(place_p + kWordAt));
            double R = __longlong_as_double((long long)lds_now(lds_at<u64>(place_p + kRAt)));       // (as good as the word that was read before it)
            u64 child = lds_now(lds_at<u64>(place_p + kChildKeyAt));
            uint32_t child_u = lds_now(lds_at<uint32_t>(place_p + kChildUAt));
            const uint32_t o = *lds_at<uint32_t>(place_p + kOpenedAt);
            w = uniform(w);
            while (__builtin_expect(!(w & kAnswer), 0)) {
                if (--polls <= 0) break;
                w = lds_now(lds_at<uint32_t>(place_p + kWordAt));
                R = __longlong_as_double((long long)lds_now(lds_at<u64>(place_p + kRAt)));
                child = lds_now(lds_at<u64>(place_p + kChildKeyAt));
                child_u = lds_now(lds_at<uint32_t>(place_p + kChildUAt));
                w = uniform(w);
            }
            if (polls <= 0) { status = kLost; break; }
            const int R_hi = uniform(__double2hiint(R));
            if (__builtin_expect(R_hi < 0, 0)) {
                if (R_hi == (int)0xbff00000u) { status = kEnded; break; }       // (-1) nothing left to sample under p
                // the quotient of two infinite weights, a NaN with its sign bit set: the token holds all that is left, at a
                // temperature so small that the row's maximum over it is rounded by more than the range of exp
                R = 1.0;
            }
            // ---- node n = child number `rank` of p, its slot and p's next one (p's is opened first)
            const double v0 = v * R;
            double v1 = v * (1.0 - R);
            const uint32_t rank = (w >> 15) & 1023u;
            uint32_t news = n | (p << 10) | kRequest, tell = ((rank + 1u) << 15) | ((uint32_t)__double2hiint(v1) >> 16);
            if (__builtin_expect(watch && (rank == (uint32_t)kClaimRank || rank >= (uint32_t)(kClaimRank + kOwnDraws) || p == 0), 0)) {
                to_ring = ring_for(lds, p, rank, n, N);
                if (to_ring) {                      // ... and p's slot is the ring's
                    const uint32_t state = states + 16u * (to_ring - 1u);
                    *lds_at<double>(state) = v1;
                    *lds_at<uint32_t>(state + 8u) = n;
                    lds_set(lds_at<uint32_t>(state + kTakenAt), rank + 1u);
                    v1 = 0.0;
                    news ^= kRequest;
                    tell = kAnswer;
                }
            }
            // what other waves wait for first; the slots' values are control's own
            const uint32_t place_n = nodes + kNode * n;
            *lds_at<u64>(place_n + kKeyAt) = child;
            *lds_at<uint32_t>(place_n + kUAt) = child_u;
            keep_order();
            lds_set(lds_at<uint32_t>(place_n + kWordAt), (uint32_t)__double2hiint(v0) >> 16);       // request of draw 0
            lds_set(lds_at<uint32_t>(place_p + kWordAt), tell);
            lds_set(lds_at<uint32_t>(lds + BuildLds::news), news);
            *lds_at<double>(place_n + kValueAt) = v0;
            *lds_at<double>(place_p + kValueAt) = v1;
            *lds_at<uint32_t>(place_p + kOpenedAt) = 2u * n;
            put_row(token, n, (int)(w & 0x7fffu));
            put_row(est_value, n, (float)v);
            put_row(parent, n, (int)(p | rank << 10 | (o >> 1) << 20));
            // ---- The first slot goes, p's next and the new node's come behind those at least as good: up to where the better one of the two
            // goes the slots move up, behind the other's place down.  (Masks of lanes; the first slot is at least as good as either.)
            const bool in = ballot(v0 > s.unlisted) & 1ull;         // (else the new one is left out, as it is if there is no place)
            const u64 g1 = ballot(s.value >= v1) >> 1, g0 = in ? ballot(s.value >= v0) >> 1 : ~0ull;
            const u64 high = g1 & g0, low = (g1 | g0) << 1 | 1ull;
            const u64 first = ballot(!(v0 > v1)) | (in ? 0ull : ~0ull);         // p's is the better one (of equal ones it was opened first)
            const bool p_first = first & 1ull;
            const double best = __builtin_amdgcn_inverse_ballot_w64(first) ? v1 : v0, other = __builtin_amdgcn_inverse_ballot_w64(first) ? v0 : v1;
            const int best_n = (int)(p_first ? p : n), other_n = (int)(p_first ? n : p);
            if (in) {
                const double out = low != ~0ull ? readlane_f64(s.value, 63) : other;
                s.unlisted = larger(s.unlisted, out);
                line = larger(line, out);
            }
            const double up_v = dpp_or_own<kDppWaveShl1>(s.value), down_v = dpp_or_own<kDppWaveShr1>(s.value);
            const int up_n = dpp_or_own<kDppWaveShl1>(s.node), down_n = dpp_or_own<kDppWaveShr1>(s.node);
            const u64 at_high = (high << 1 | 1ull) & ~high, at_low = (low << 1 | 1ull) & ~low, above = ~(low << 1 | 1ull);
            const auto pick = [&](auto own, auto up, auto b, auto l, auto down) __attribute__((always_inline)) {
                own = __builtin_amdgcn_inverse_ballot_w64(high) ? up : own;
                own = __builtin_amdgcn_inverse_ballot_w64(at_high) ? b : own;
                own = __builtin_amdgcn_inverse_ballot_w64(at_low) ? l : own;
                return __builtin_amdgcn_inverse_ballot_w64(above) ? down : own;
            };
            s.value = pick(s.value, up_v, best, other, down_v);
            s.node = pick(s.node, up_n, best_n, other_n, down_n);
            ++n;
        } while (n < N && !to_ring && (ballot(s.value > line) & 1ull));
        if (status != kGoOn) {
            lost = status == kLost;
            break;
        }
    }
    return lost ? (int)~n : (int)n;
}

template <bool VEC>
__global__ __launch_bounds__(kBuildThreads) void build_tree_waves_kernel(
    const float* __restrict__ draft_logits, int V, SeqArgs sa, uint64_t seed,
    dyspec_tree tree, float* est_value, uint64_t* __restrict__ anc_mask,
    int mask_words, int* __restrict__ n_built, double* ws, int widest, int root_ring, int max_polls)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char dyn[];
    uint32_t lds = lds_base(dyn);
    asm("" : "+s"(lds));        // (a constant known to the link only, else: the roles' loops would load it from memory time and again)
    const uint32_t nodes = lds + BuildLds::nodes, row_at = lds + BuildLds::row(widest);
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int help = (int)blockIdx.x - sa.n_seq;                    // >= 0: this workgroup is a helper
    const int seq = help >= 0 ? help / kRings : (int)blockIdx.x;
    const int base = sa.node_off[seq];
    const int N = sa.node_off[seq + 1] - base;
    const double inv_temp = 1.0 / (double)sa.temp_d[seq];
    const bool helped = (int)gridDim.x > sa.n_seq && N >= kLeastHelped;
    if (help >= 0) {
        if (helped) help_build<VEC>(lds, draft_logits, V, inv_temp, seed, ws, base, N, help % kRings, (uint32_t)seq);
        return;
    }
    const uint2 key = root_key((uint32_t)seq);
    for (int i = tid; i < N; i += kBuildThreads) {
        const uint32_t place = nodes + kNode * i;
        *lds_at<double>(place + kValueAt) = i == 0 && !root_ring ? 1.0 : -1.0;        // (the root's slot is its ring's)
        *lds_at<uint32_t>(place + kWordAt) = i == 0 && !root_ring ? 0x3ff0u : kAnswer;           // a request for draw 0, or nothing
        *lds_at<uint32_t>(place + kOpenedAt) = 2u * (uint32_t)i + 1u;
    }
    // (with helpers the rings lie where the root's row would)
    const uint32_t rings = helped ? row_at : lds + BuildLds::ring;
    if (tid < (helped ? kRings * kRing : kRing)) *lds_at<uint32_t>(rings + kPlace * tid) = 0u;
    if (tid == 0) {
        *lds_at<u64>(nodes + kKeyAt) = join_key(key);
        *lds_at<float>(nodes + kUAt) = u01(seed, key, 0u, KIND_BUILD);
        *lds_at<double>(lds + BuildLds::state) = 1.0;
        *lds_at<uint32_t>(lds + BuildLds::state + 8) = 0u;
        *lds_at<uint32_t>(lds + BuildLds::state + kTakenAt) = 0u;
        *lds_at<uint32_t>(lds + BuildLds::here) = 0u;
        *lds_at<uint32_t>(lds + BuildLds::claims) = 0u;
        *lds_at<uint32_t>(lds + BuildLds::caught_up) = 0u;
        *lds_at<uint32_t>(lds + BuildLds::news) = 1u << 31;
    }
    double m = 0.0;
    if (root_ring && N > 1)
        m = load_row_lds<kBuildThreads, VEC>(draft_logits + (size_t)base * V, V, inv_temp, lds_at<double>(row_at),
                                             lds_at<float>(row_at + 8 * row_leaves(V)), reinterpret_cast<float*>(dyn + BuildLds::fred));
    __syncthreads();
    // (control and the root's wave share their SIMDs, but come first there)
    if (wave == 0) {
        __builtin_amdgcn_s_setprio(3);
        const int n = pop_nodes(lds, rings, root_ring, helped, N, max_polls, tree.parent + base, tree.token + base, est_value + base);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");            // the rows are read back below
        if (tid == 0) {
            *lds_at<int>(lds + BuildLds::n_built) = n;
            lds_set(lds_at<uint32_t>(lds + BuildLds::news), kStop);
        }
    } else if (wave == 1) {
        if (!helped) __builtin_amdgcn_s_setprio(2);
        if (helped) bring_draws(lds, rings, ws, base, N, seed);
        else if (root_ring && N > 1) draw_for_root(lds, row_at, inv_temp, m, V, N, seed, (uint32_t)seq);
    } else {
        draw_for_nodes<VEC>(lds, wave - 2, draft_logits, V, inv_temp, seed, ws, base, N);
    }
    __builtin_amdgcn_s_setprio(0);
    __syncthreads();
    // ---- the tree is known: links, depths and masks, all rows at once
    const int ended = *lds_at<int>(lds + BuildLds::n_built), n = ended < 0 ? ~ended : ended;
    lds_t<int>* const first = lds_at<int>(nodes);             // the nodes' place is free now
    lds_t<int>* const next = first + widest;
    lds_t<uint32_t>* const from = lds_at<uint32_t>(nodes + 8 * widest);
    for (int i = tid; i < N; i += kBuildThreads) {
        first[i] = -1;
        next[i] = -1;
        from[i] = (i > 0 && i < n) ? (uint32_t)tree.parent[base + i] : 0u;
    }
    __syncthreads();
    for (int i = tid; i < n; i += kBuildThreads)
        if (i > 0) {
            const uint32_t f = from[i];
            if ((f >> 10) & 1023u) next[f >> 20] = i; else first[f & 1023u] = i;
        }
    __syncthreads();
    for (int i = tid; i < N; i += kBuildThreads) {
        const bool built = i > 0 && i < n;
        const uint32_t f = from[i];
        tree.parent[base + i] = built ? (int)(f & 1023u) : -1;
        tree.sib_rank[base + i] = (int)((f >> 10) & 1023u);
        tree.first_child[base + i] = first[i];
        tree.next_sibling[base + i] = next[i];
        if (i >= n) {
            tree.token[base + i] = -1;
            est_value[base + i] = 0.0f;
        }
        // own bit and the ancestors', which are smaller and smaller: a word at a time
        uint64_t* const mrow = anc_mask + (size_t)(base + i) * mask_words;
        int word = i >> 6, depth = 0;
        for (int w = mask_words - 1; w > word; --w) mrow[w] = 0ull;
        uint64_t bits = 1ull << (i & 63);
        for (int a = i; built && a > 0; ++depth) {
            a = (int)(from[a] & 1023u);
            for (; (a >> 6) != word; --word) { mrow[word] = bits; bits = 0ull; }
            bits |= 1ull << (a & 63);
        }
        for (; word >= 0; --word) { mrow[word] = bits; bits = 0ull; }
        tree.depth[base + i] = depth;
    }
    if (tid == 0) n_built[seq] = ended < 0 ? -1 : n;
}

// The root's row is kept in LDS in batches without helpers, where it fits beside the node state (32000 tokens: up to 564 rows,
// 32768: up to 498) and is drawn from often enough to pay for its loading (2 rows of 32000 tokens 26.0 us with it, 17.9
// without; 8 rows 30.3 and 30.0; 16 rows 35.8 and 45.5); else the root's draws are made like every other node's.
constexpr int kRingRows = 10;
static size_t build_lds_bytes(int V, int widest, bool root_ring) { return BuildLds::row(widest) + (root_ring ? row_lds_bytes(V) : 0); }

// the builder takes up to a whole CU's LDS: the kernels' limit is raised once
hipError_t prepare_build_tree()
{
    static std::atomic<unsigned long long> done_vec{0}, done_scalar{0};
    const hipError_t e = raise_dynamic_lds_once(reinterpret_cast<const void*>(&build_tree_waves_kernel<true>), (int)kLdsPerWorkgroup, done_vec);
    if (e != hipSuccess) return e;
    return raise_dynamic_lds_once(reinterpret_cast<const void*>(&build_tree_waves_kernel<false>), (int)kLdsPerWorkgroup, done_scalar);
}

size_t build_tree_workspace_bytes(int total_rows) { return (size_t)total_rows * kRowSumDoubles * sizeof(double); }

template <int S>
static void launch_draft_row_sums_s(const float* draft_logits, int V, const SeqArgs& sa, double* ws, int mails, hipStream_t stream)
{
    const int rows = sa.node_off[sa.n_seq];
    if (V % 4 == 0) draft_row_sums_kernel<true, S><<<rows, kBlock, 0, stream>>>(draft_logits, V, sa, ws, mails);
    else draft_row_sums_kernel<false, S><<<rows, kBlock, 0, stream>>>(draft_logits, V, sa, ws, mails);
}
static hipError_t launch_draft_row_sums(const float* draft_logits, int V, const SeqArgs& sa, double* ws, int mails, hipStream_t stream)
{
    if (V <= 2 * kSeg) launch_draft_row_sums_s<2>(draft_logits, V, sa, ws, mails, stream);
    else if (V <= 8 * kSeg) launch_draft_row_sums_s<8>(draft_logits, V, sa, ws, mails, stream);
    else launch_draft_row_sums_s<kMaxSeg>(draft_logits, V, sa, ws, mails, stream);
    return hipGetLastError();
}

hipError_t launch_build_tree(const float* draft_logits, int V, const SeqArgs& sa, uint64_t seed,
                             const dyspec_tree& tree, float* est_value, uint64_t* anc_mask,
                             int mask_words, int* n_built, void* workspace, size_t workspace_bytes, int max_polls, hipStream_t stream)
{
    const int rows = sa.node_off[sa.n_seq];
    double* ws = static_cast<double*>(workspace);
    const bool cached = ws != nullptr && workspace_bytes >= build_tree_workspace_bytes(rows);
    if (cached) {
        int widest = 0;
        for (int s = 0; s < sa.n_seq; ++s) widest = max(widest, sa.node_off[s + 1] - sa.node_off[s]);
        const bool helped = widest >= kHelpedRows && sa.n_seq * (1 + kRings) <= kHelpedBlocks;
        const int root_ring = !helped && widest >= kRingRows && build_lds_bytes(V, widest, true) <= kLdsPerWorkgroup;
        const size_t lds_bytes = helped ? std::max((size_t)BuildLds::row(widest) + kRings * kRing * kPlace, HelpLds::row + run_row_lds_bytes(V))
                                        : build_lds_bytes(V, widest, root_ring);
        const int grid = sa.n_seq * (helped ? 1 + kRings : 1);
        const hipError_t ea = prepare_build_tree();
        if (ea != hipSuccess) return ea;
        const hipError_t es = launch_draft_row_sums(draft_logits, V, sa, ws, helped, stream);
        if (es != hipSuccess) return es;
        if (V % 4 == 0) {
            build_tree_waves_kernel<true><<<grid, kBuildThreads, lds_bytes, stream>>>(
                draft_logits, V, sa, seed, tree, est_value, anc_mask, mask_words, n_built, ws, widest, root_ring, max_polls);
        } else {
            build_tree_waves_kernel<false><<<grid, kBuildThreads, lds_bytes, stream>>>(
                draft_logits, V, sa, seed, tree, est_value, anc_mask, mask_words, n_built, ws, widest, root_ring, max_polls);
        }
    } else if (V % 4 == 0) {
        build_tree_kernel<true><<<sa.n_seq, kBlock, 0, stream>>>(draft_logits, V, sa, seed, tree, est_value,
                                                                 anc_mask, mask_words, n_built);
    } else {
        build_tree_kernel<false><<<sa.n_seq, kBlock, 0, stream>>>(draft_logits, V, sa, seed, tree, est_value,
                                                                  anc_mask, mask_words, n_built);
    }
    return hipGetLastError();
}

}  // namespace dyspec

// Token tree construction with a threshold (Algorithm 2, Section 4.4, Appendix A.2) for gfx950.
//
// The tree grows level by level.  Within a level the nodes are independent: every node whose
// estimated value is at or above the threshold draws children from its own draft row, without
// replacement, for as long as the value of the next draw stays at or above the threshold.
// That is the data-parallel form of the builder: one workgroup per node of the level
// (threshold_expand_kernel), all of them at once, each with its row in LDS, from which one
// wave makes the node's draws (wave_draw.h, as the greedy builder draws from the root).  Nodes are
// numbered in creation order (level by level, parents in order, children in sampling order),
// which a workgroup cannot know while its neighbours are still drawing, so children go to a
// per-level pool first and threshold_commit_kernel (one workgroup per sequence) scans the
// counts, cuts at the row capacity and writes the tree rows, links, path keys, values and
// ancestor masks.  The commit also writes the level's size to host memory, where the host reads it
// when the stream is done: it sizes the next grid and ends the loop.  Draft row of a node = its row index, as for Algorithm 1.
#include "draft_row.h"
#include "lane_ops.h"
#include "wave_draw.h"

namespace dyspec {

// Workspace, in doubles, for rows = sum of capacities N_s:
//   child_value[rows]   value of a node's own first draw (v * d[y]); root 1
//   pool_v0[pool], pool_v[pool]   per drawn child: v * d[y], and the value v it was drawn at
//   pk[rows] (uint2), counts[rows] (int), pool_token[pool] (int), state[4 * n_seq] (int)
// pool = sum over sequences of N_s^2 / 4 + N_s entries: a level with F nodes and R rows left
// holds at most F * R children and F <= N - R.
struct ThresholdWs {
    double* child_value;
    double* pool_v0;
    double* pool_v;
    uint2* pk;
    int* counts;
    int* pool_token;
    int* state;          // per sequence: level begin, level end, rows left at level begin, unused
    long long pool_off[DYSPEC_MAX_SEQ + 1];
};

static size_t pool_entries(int N) { return (size_t)N * N / 4 + N; }

size_t build_threshold_workspace_bytes(const SeqArgs& sa)
{
    const size_t rows = sa.node_off[sa.n_seq];
    size_t pool = 0;
    for (int s = 0; s < sa.n_seq; ++s) pool += pool_entries(sa.node_off[s + 1] - sa.node_off[s]);
    return rows * 8 + pool * 16 + rows * 8 + rows * 4 + pool * 4 + (size_t)sa.n_seq * 16 + 64;
}

static ThresholdWs carve(void* workspace, const SeqArgs& sa)
{
    ThresholdWs w;
    const size_t rows = sa.node_off[sa.n_seq];
    size_t pool = 0;
    for (int s = 0; s < sa.n_seq; ++s) {
        w.pool_off[s] = (long long)pool;
        pool += pool_entries(sa.node_off[s + 1] - sa.node_off[s]);
    }
    w.pool_off[sa.n_seq] = (long long)pool;
    char* p = static_cast<char*>(workspace);
    w.child_value = reinterpret_cast<double*>(p); p += rows * 8;
    w.pool_v0 = reinterpret_cast<double*>(p); p += pool * 8;
    w.pool_v = reinterpret_cast<double*>(p); p += pool * 8;
    w.pk = reinterpret_cast<uint2*>(p); p += rows * 8;
    w.counts = reinterpret_cast<int*>(p); p += rows * 4;
    w.pool_token = reinterpret_cast<int*>(p); p += pool * 4;
    w.state = reinterpret_cast<int*>(p);
    return w;
}

struct ThresholdArgs {
    double t[DYSPEC_MAX_SEQ];
};

__global__ __launch_bounds__(256) void threshold_init_kernel(SeqArgs sa, dyspec_tree tree, float* __restrict__ est_value,
                                                             uint64_t* __restrict__ anc_mask, int mask_words,
                                                             int* __restrict__ n_built, ThresholdWs w)
{
    const int seq = blockIdx.x;
    const int base = sa.node_off[seq];
    const int N = sa.node_off[seq + 1] - base;
    for (int i = threadIdx.x; i < N; i += 256) {
        tree.parent[base + i] = -1; tree.token[base + i] = -1; tree.sib_rank[base + i] = 0;
        tree.first_child[base + i] = -1; tree.next_sibling[base + i] = -1; tree.depth[base + i] = 0;
        est_value[base + i] = (i == 0) ? 1.0f : 0.0f;
        for (int k = 0; k < mask_words; ++k)
            anc_mask[(size_t)(base + i) * mask_words + k] = (k == i / 64) ? (1ull << (i % 64)) : 0ull;
        w.counts[base + i] = 0;
    }
    if (threadIdx.x == 0) {
        if (N > 0) {
            w.child_value[base] = 1.0;
            w.pk[base] = root_key((uint32_t)seq);
        }
        w.state[4 * seq + 0] = 0;                       // the first level is the root alone
        w.state[4 * seq + 1] = min(N, 1);
        w.state[4 * seq + 2] = max(N - 1, 0);
        w.state[4 * seq + 3] = 0;
        n_built[seq] = min(N, 1);
    }
}

// One workgroup per node of the current level: blockIdx.x = position in the level.  All waves bring
// the node's row into LDS (logits, leaf sums); then the first one draws and the others leave.
// Bound by the instructions of a draw (a lone wave issues one in eight cycles, about 160 of them): 0.57 us each,
// against 1.5 us when the whole workgroup made every draw, with two barriers and eight waves doing every
// scan: the 384-row tree of the Zipf table (383 draws under the root) 587 -> 235 us, now 227.  A second wave that takes
// over the division and the writing through a ring of draws in LDS makes it 256: keeping the ring costs the
// drawing wave more instructions than it saves.
constexpr int kExpandThreads = 1024;
template <bool VEC>
__global__ __launch_bounds__(kExpandThreads) void threshold_expand_kernel(const float* __restrict__ draft_logits, int V, SeqArgs sa,
                                                                          ThresholdArgs ta, uint64_t seed, ThresholdWs w)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char dyn[];
    __shared__ float fred[kExpandThreads / kWave];
    const int tid = threadIdx.x, lane = tid & 63;
    const int seq = blockIdx.y;
    const int base = sa.node_off[seq];
    const int lvl_begin = uniform(w.state[4 * seq + 0]), lvl_end = uniform(w.state[4 * seq + 1]), left = uniform(w.state[4 * seq + 2]);
    const int f = blockIdx.x;
    const int p = lvl_begin + f;
    if (p >= lvl_end) return;                           // uniform over the workgroup
    const double t = ta.t[seq];
    double v = w.child_value[base + p];
    if (!(v >= t) || left <= 0) {                       // below the threshold: no draw, the row is not even read
        if (tid == 0) w.counts[base + p] = 0;
        return;
    }
    WaveRow row;
    row.leaf = lds_at<double>(lds_base(dyn));
    row.logits = lds_at<float>(lds_base(dyn) + 8 * row_leaves(V));
    row.inv_temp = 1.0 / (double)sa.temp_d[seq];
    row.m = load_row_lds<kExpandThreads, VEC>(draft_logits + (size_t)(base + p) * V, V, row.inv_temp, row.leaf, row.logits, fred);
    if (tid >= kWave) return;
    open_wave_row(row, V);
    const uint2 pk = w.pk[base + p];
    const size_t pool0 = (size_t)w.pool_off[seq] + (size_t)f * left;
    // draws count - 64 .. count - 1 wait in the lanes to be written out together, draw c in lane c % 64
    float us = 0.f;                                     // the uniforms of 64 samplings, one per lane
    int token = 0, count = 0;
    double value = 0.0, own = 0.0;
    auto flush = [&](int first) {                       // draws first .. count - 1
        const int c = first + lane;
        if (c < count) { w.pool_token[pool0 + c] = token; w.pool_v[pool0 + c] = value; w.pool_v0[pool0 + c] = own; }
    };
    while (count < left && ballot(v >= t)) {
        if ((count & 63) == 0) us = u01(seed, pk, (uint32_t)(count + lane), KIND_BUILD);
        Drawn d;
        if (!draw_wave_row(row, (double)readlane_f32(us, count & 63), &d)) break;       // nothing left to sample under p
        const double dy = d.wy / d.W;
        if (lane == (count & 63)) { token = d.y; value = v; own = v * dy; }
        v = v * (1.0 - dy);
        ++count;
        if ((count & 63) == 0) flush(count - kWave);
    }
    flush(count & ~63);
    if (lane == 0) w.counts[base + p] = count;
}

struct CommitShared {
    int excl[DYSPEC_MAX_BUILD_NODES + 1];
    int scan[kWaves];
};

// One workgroup per sequence: numbers the level's children in creation order, cuts at the
// capacity, writes their rows and makes them the next level.
__global__ __launch_bounds__(kBlock) void threshold_commit_kernel(SeqArgs sa, uint64_t seed, dyspec_tree tree,
                                                                  float* __restrict__ est_value, uint64_t* anc_mask,
                                                                  int mask_words, int* __restrict__ n_built, ThresholdWs w,
                                                                  int* __restrict__ host_state)
{
    __shared__ CommitShared sh;
    const int tid = threadIdx.x;
    const int seq = blockIdx.x;
    const int base = sa.node_off[seq];
    const int lvl_begin = w.state[4 * seq + 0], lvl_end = w.state[4 * seq + 1], left = w.state[4 * seq + 2];
    const int F = lvl_end - lvl_begin;
    if (F <= 0) return;
    // exclusive scan of the children counts over the level, two nodes per thread (F <= 1024)
    const int f0 = 2 * tid, f1 = 2 * tid + 1;
    const int c0 = f0 < F ? w.counts[base + lvl_begin + f0] : 0;
    const int c1 = f1 < F ? w.counts[base + lvl_begin + f1] : 0;
    int excl;
    const int incl = block_scan_inclusive<int>(c0 + c1, sh.scan, &excl);
    if (f0 <= F) sh.excl[f0] = excl;
    if (f1 <= F) sh.excl[f1] = excl + c0;
    if (tid == kBlock - 1 && F == 2 * kBlock) sh.excl[F] = incl;
    __syncthreads();
    const int total = sh.excl[F];
    const int M = min(total, left);                     // rows that still fit
    for (int k = tid; k < M; k += kBlock) {
        // node of the level that drew child k: last f with excl[f] <= k
        int lo = 0, hi = F - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (sh.excl[mid] <= k) lo = mid; else hi = mid - 1;
        }
        const int fpos = lo, rank = k - sh.excl[fpos];
        const int p = lvl_begin + fpos, i = lvl_end + k;
        const size_t e = (size_t)w.pool_off[seq] + (size_t)fpos * left + rank;
        const int n_kids = min(sh.excl[fpos + 1], M) - sh.excl[fpos];      // children of p that fit
        tree.parent[base + i] = p;
        tree.token[base + i] = w.pool_token[e];
        tree.sib_rank[base + i] = rank;
        tree.depth[base + i] = tree.depth[base + p] + 1;
        tree.next_sibling[base + i] = (rank + 1 < n_kids) ? i + 1 : -1;
        if (rank == 0) tree.first_child[base + p] = i;
        est_value[base + i] = (float)w.pool_v[e];
        w.child_value[base + i] = w.pool_v0[e];
        w.pk[base + i] = child_key(seed, w.pk[base + p], (uint32_t)rank);
        w.counts[base + i] = 0;
        for (int q = 0; q < mask_words; ++q)
            anc_mask[(size_t)(base + i) * mask_words + q] =
                anc_mask[(size_t)(base + p) * mask_words + q] | ((q == i / 64) ? (1ull << (i % 64)) : 0ull);
    }
    __syncthreads();
    if (tid == 0) {
        w.state[4 * seq + 0] = lvl_end;
        w.state[4 * seq + 1] = lvl_end + M;
        w.state[4 * seq + 2] = left - M;
        n_built[seq] = lvl_end + M;
        if (host_state) {
            host_state[4 * seq + 0] = lvl_end;
            host_state[4 * seq + 1] = lvl_end + M;
            host_state[4 * seq + 2] = left - M;
        }
    }
}

// Host memory that the commits write to, for kHostStates calls at a time; a call without one
// copies the state from the workspace.  Read this way a level costs 8 us less than with a copy between the commit
// and the wait: trees of one level (384 rows, V = 32000) 292 -> 283 us, of six (64 rows, V = 1000) 226 -> 172.
// Allocated once for the process, 8 KB.
constexpr int kHostStates = 8;
static std::atomic<int*> host_states{nullptr};
static std::atomic<unsigned> host_states_taken{0};

static void allocate_host_states()
{
    if (host_states.load(std::memory_order_acquire)) return;
    int *mine = nullptr, *none = nullptr;
    // (an allocation is no concern of a capture that runs in this or another thread)
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    if (hipThreadExchangeStreamCaptureMode(&mode) != hipSuccess) return;
    const hipError_t e = hipHostMalloc(reinterpret_cast<void**>(&mine), sizeof(int) * 4 * DYSPEC_MAX_SEQ * kHostStates, hipHostMallocPortable);
    (void)hipThreadExchangeStreamCaptureMode(&mode);
    if (e != hipSuccess) {
        (void)hipGetLastError();                        // not now: the calls copy
        return;
    }
    if (!host_states.compare_exchange_strong(none, mine, std::memory_order_acq_rel)) (void)hipHostFree(mine);
}

// One call's part of that memory, given back when the call returns.
struct HostState {
    int* words = nullptr;
    unsigned bit = 0;
    HostState()
    {
        int* const all = host_states.load(std::memory_order_acquire);
        unsigned taken = host_states_taken.load(std::memory_order_relaxed);
        while (all && (~taken & ((1u << kHostStates) - 1u))) {
            const int k = __builtin_ctz(~taken);
            if (host_states_taken.compare_exchange_weak(taken, taken | (1u << k), std::memory_order_acquire, std::memory_order_relaxed)) {
                bit = 1u << k;
                words = all + 4 * DYSPEC_MAX_SEQ * k;
                return;
            }
        }
    }
    ~HostState() { host_states_taken.fetch_and(~bit, std::memory_order_release); }
    // commits that may still run keep what they write to
    void keep() { bit = 0; }
    HostState(const HostState&) = delete;
    HostState& operator=(const HostState&) = delete;
};

// the expanding workgroups keep a row in dynamic LDS: raised to the largest vocabulary once
hipError_t prepare_build_threshold()
{
    allocate_host_states();
    static std::atomic<unsigned long long> done_vec{0}, done_scalar{0};
    constexpr int bytes = (int)row_lds_bytes(DYSPEC_MAX_VOCAB);
    hipError_t e = raise_dynamic_lds_once(reinterpret_cast<const void*>(&threshold_expand_kernel<true>), bytes, done_vec);
    if (e != hipSuccess) return e;
    return raise_dynamic_lds_once(reinterpret_cast<const void*>(&threshold_expand_kernel<false>), bytes, done_scalar);
}

hipError_t launch_build_threshold(const float* draft_logits, int V, const SeqArgs& sa, const double* threshold,
                                  uint64_t seed, const dyspec_tree& tree, float* est_value, uint64_t* anc_mask,
                                  int mask_words, int* n_built, int* n_levels, void* workspace, hipStream_t stream)
{
    // the call waits for the stream, which a capture would refuse half-way through
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    const hipError_t ec = hipStreamIsCapturing(stream, &capture);
    if (ec != hipSuccess) return ec;
    if (capture != hipStreamCaptureStatusNone) return hipErrorStreamCaptureUnsupported;
    const ThresholdWs w = carve(workspace, sa);
    ThresholdArgs ta;
    for (int s = 0; s < sa.n_seq; ++s) ta.t[s] = threshold[s];
    const size_t dyn_bytes = row_lds_bytes(V);
    const hipError_t ea = prepare_build_threshold();
    if (ea != hipSuccess) return ea;
    threshold_init_kernel<<<sa.n_seq, 256, 0, stream>>>(sa, tree, est_value, anc_mask, mask_words, n_built, w);
    // (Launching eight levels at a time without a look from the host in between, over a grid sized for
    // the widest level possible, was measured and is slower: a launch of workgroups that find
    // nothing to do costs about as much as the look it saves -- 70B table 1.06 against 1.00 ms, the
    // 13B table, two levels deep, 0.60 against 0.50 ms.)
    int widest = 1;
    for (int s = 0; s < sa.n_seq; ++s) widest = max(widest, sa.node_off[s + 1] - sa.node_off[s]);
    int frontier = widest > 1 ? 1 : 0, levels = 0;      // widest level over the sequences: the roots, if a row is left
    HostState host;
    int copied[4 * DYSPEC_MAX_SEQ];
    int* const state = host.words ? host.words : copied;
    for (int s = 0; s < 4 * sa.n_seq; ++s) state[s] = 0;
    // a level adds at least one row or ends the loop, so this runs at most max N times
    while (frontier > 0) {
        if (V % 4 == 0)
            threshold_expand_kernel<true><<<dim3(frontier, sa.n_seq), kExpandThreads, dyn_bytes, stream>>>(draft_logits, V, sa, ta, seed, w);
        else
            threshold_expand_kernel<false><<<dim3(frontier, sa.n_seq), kExpandThreads, dyn_bytes, stream>>>(draft_logits, V, sa, ta, seed, w);
        threshold_commit_kernel<<<sa.n_seq, kBlock, 0, stream>>>(sa, seed, tree, est_value, anc_mask, mask_words, n_built, w, host.words);
        hipError_t e = hipSuccess;
        if (!host.words) e = hipMemcpyAsync(state, w.state, sizeof(int) * 4 * sa.n_seq, hipMemcpyDeviceToHost, stream);
        if (e == hipSuccess) e = hipStreamSynchronize(stream);
        if (e != hipSuccess) {
            host.keep();
            return e;
        }
        ++levels;
        frontier = 0;
        for (int s = 0; s < sa.n_seq; ++s)
            if (state[4 * s + 2] > 0) frontier = max(frontier, state[4 * s + 1] - state[4 * s + 0]);
    }
    if (n_levels) *n_levels = levels;
    return hipGetLastError();
}

}  // namespace dyspec

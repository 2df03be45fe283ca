// Tree attention on the matrix cores for short walks: bf16 tensors, head_dim 64 or 128, fp32 accumulation.
//
// Workgroup = NW waves on one block of 32 rows (row = node * G + head, as in tree_attn_mfma.hip) of one KV head.
// The waves share out the keys: wave w takes blocks w, w + NW, ... of 32 keys from a walk of the prefix's blocks and
// the tree's blocks that any of the 32 rows sees.  Each wave brings its keys into LDS of its own (direct loads, K and V
// 32 rows each) and waits for nobody; the waves meet at the end, where (max, sum, rows) of all are merged through LDS
// in fp32 and every wave finishes 32 / NW rows.
//
// Why: the 128-row workgroups of tree_attn_mfma.hip run one to a CU, start with 128 KB of loads, and where they leave the
// chip idle split the prefix and merge parts of 128 rows: some 10 us beside the walk.  Here a workgroup starts with a few KB, and
// a row block's walk is shared out inside it, so short walks need few parts or none.  Long walks are better off there:
// a block of keys loaded to LDS serves 32 rows here, 128 there.
// What bounds it: the CU's path from L1 to LDS (64 bytes a cycle: 52 measured with K and V in L2), for K and V from memory the
// trips of the 16 KB that a wave has under way; of 11 us (32 heads, 128 rows, 1024 keys) 0.7 are the addresses, 1.1 the first
// trip, 5 the walk, 1.5 the merge, 1.3 the launch itself.
// Measured, us per layer, the other kernel -> this one: 32 heads, 128 rows, 1024 keys 16.7 -> 12.2 (2 parts); 8 KV heads of 8,
// 32 rows, 4096 keys 22.9 -> 15.6 (4 parts); 64 heads, tree of 2048 rows alone 65 -> 37 (2 waves, four workgroups a CU);
// two sequences of 37 and 5 rows, 100 and 33 keys 9.3 -> 5.7.
// Without effect: V's fragments read ahead of the softmax, the first product as two chains, K's loads behind the first product.
#include <atomic>

#include "attn_mfma.h"

namespace dyspec {

constexpr int kShortRows = 32;            // rows of a workgroup, keys of a block
constexpr int kShortSplits = 8;           // parts of a prefix at most
constexpr float kShortSumLimit = 1024.0f; // a lane's block sum above this raises the reference maximum

template <int D> struct ShortGeo {
    static constexpr int kRowBytes = 2 * D;
    static constexpr int kChunks = D / 8;                        // 16-byte chunks per row
    static constexpr int kRowsPerLoad = 1024 / kRowBytes;        // rows one wave-wide direct load covers
    static constexpr int kMatBytes = 32 * kRowBytes;             // 32 rows
    static constexpr int kLoads = 32 / kRowsPerLoad;             // direct loads per 32 rows
    static constexpr int kPartWords = kShortRows * (D / 4 + 1);    // 64-bit words of a part: bf16 rows, (max, sum) per row
};
// LDS: a K and a V slot per wave, the query rows, the waves' (max, sum) per row, the visibility words
// With two waves the query rows pass through the second wave's V slot and (max, sum) take the words' place at the end, so that
// four workgroups share a CU at head_dim 128.
template <int NW> constexpr bool kShared = NW == 2;
template <int NW> constexpr int kMlBytes = 8 * kShortRows * NW;
template <int D, int NW> constexpr int short_lds_bytes(int tree_tiles)
{
    return kShared<NW> ? 2 * NW * ShortGeo<D>::kMatBytes + (256 * tree_tiles > kMlBytes<NW> ? 256 * tree_tiles : kMlBytes<NW>)
                       : (2 * NW + 1) * ShortGeo<D>::kMatBytes + kMlBytes<NW> + 256 * tree_tiles;
}

// What the kernel takes, laid out to arrive in few scalar loads: a batch of one sequence reads nothing but the head.
struct ShortSeq { int tile_off, node_off, N, P; long long kv_off, pad; };
struct ShortArgs {
    const char *q, *kp, *vp, *kt, *vt, *mask;
    char* out;
    unsigned long long* part;
    unsigned* counters;
    long long q_stride, kvp_stride, kvt_stride;    // bytes between stacked layers
    uint32_t kv_row_bytes, q_row_bytes;            // of all heads
    uint32_t G, g_magic;                           // r / G = hi(r * g_magic), G = 1: r
    int mask_bytes;                                // a row of the mask
    int n_split, n_seq;
    float c2;                                      // softmax scale * log2(e)
    ShortSeq one;                                  // the first sequence
    ShortSeq seq[DYSPEC_MAX_SEQ];
};

template <int N> __device__ __forceinline__ void wait_direct_loads_but() { asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory"); }
__device__ __forceinline__ uint32_t div_magic(uint32_t r, uint32_t magic) { return magic ? __umulhi(r, magic) : r; }

template <int D, int NW>
__global__ __launch_bounds__(64 * NW, D == 64 ? 4 : 2) void tree_attn_short_kernel(ShortArgs a)
{
    using L = ShortGeo<D>;
    constexpr int KK = D / 16;                   // k-steps of the first product
    constexpr int DB = D / 32;                   // 32-wide blocks of the head dimension
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int n = lane & 31, g = lane >> 5;

    // ---- which rows, which keys
    const int kvh = blockIdx.x, tile = blockIdx.y;
    // (the arguments are asked for together: left to themselves the loads come one by one, where each is first used)
    ShortSeq sq = a.one;
    const char *a_q = a.q, *a_kp = a.kp, *a_vp = a.vp, *a_kt = a.kt, *a_vt = a.vt, *a_mask = a.mask;
    uint32_t kv_row_bytes = a.kv_row_bytes, q_row_bytes = a.q_row_bytes, G = a.G, g_magic = a.g_magic;
    int mask_bytes = a.mask_bytes, n_split = a.n_split, n_seq = a.n_seq;
    long long q_stride = a.q_stride, kvp_stride = a.kvp_stride, kvt_stride = a.kvt_stride;
    float c2 = a.c2;
    asm volatile("" : "+s"(a_q), "+s"(a_kp), "+s"(a_vp), "+s"(a_kt), "+s"(a_vt), "+s"(a_mask), "+s"(kv_row_bytes), "+s"(q_row_bytes), "+s"(G),
                 "+s"(g_magic), "+s"(mask_bytes), "+s"(n_split), "+s"(n_seq), "+s"(q_stride), "+s"(kvp_stride), "+s"(kvt_stride), "+s"(c2));
    asm volatile("" : "+s"(sq.tile_off), "+s"(sq.node_off), "+s"(sq.N), "+s"(sq.P), "+s"(sq.kv_off));
    if (n_seq > 1) {                             // sequences that end at or before this tile
        const int at = lane + 1 < n_seq ? a.seq[lane + 1].tile_off : 0x7fffffff;
        sq = a.seq[__builtin_popcountll(__builtin_amdgcn_ballot_w64(tile >= at))];
    }
    const int N = sq.N, P = sq.P;
    int layer = blockIdx.z, split = 0;
    if (n_split > 1) { layer = blockIdx.z / n_split; split = blockIdx.z % n_split; }
    const int rows = (int)G * N;
    const int r0 = (tile - sq.tile_off) * kShortRows;
    const int node_last = (int)div_magic((uint32_t)min(rows - 1, r0 + kShortRows - 1), g_magic);
    // a split takes an even share of the blocks; the last one walks the tree as well
    const int nPall = (P + 31) / 32;
    int nTw = node_last / 64 + 1, p_begin = 0, nP = nPall;
    if (n_split > 1) {
        const int share = (nPall + node_last / 32 + n_split) / n_split;
        p_begin = min(split * share, nPall);
        nP = nPall - p_begin;
        if (split < n_split - 1) { nTw = 0; nP = min(share, nP); }
    }
    const long long kvp_off = layer * kvp_stride + sq.kv_off * kv_row_bytes + kvh * D * 2;
    const long long kvt_off = layer * kvt_stride + (long long)sq.node_off * kv_row_bytes + kvh * D * 2;
    const char *const kp = a_kp + kvp_off, *const vp = a_vp + kvp_off, *const kt = a_kt + kvt_off, *const vt = a_vt + kvt_off;
    const uint32_t lds0 = lds_address(lds);
    const uint32_t slot = lds0 + wave * 2 * L::kMatBytes;              // this wave's K rows, then its V rows
    const uint32_t q_lds = lds0 + (2 * NW - (kShared<NW> ? 1 : 0)) * L::kMatBytes;
    const uint32_t ml_lds = q_lds + L::kMatBytes;
    const uint32_t vis_lds = ml_lds + (kShared<NW> ? 0 : kMlBytes<NW>);                    // [tree tile of 64 keys][its half][row]: 32 visibility bits

    // ---- the visibility words of the 32 rows, the query rows (a row past the end repeats the last one)
    const int lrow = lane / L::kChunks, cpos = lane % L::kChunks;
    {
        const char* const mask = a_mask + (long long)sq.node_off * mask_bytes;
        const uint32_t off = div_magic((uint32_t)min(r0 + n, rows - 1), g_magic) * (uint32_t)mask_bytes + 4u * (uint32_t)g;
        for (int t = wave; t < nTw; t += NW)
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2"
                         :: "s"(vis_lds + 256 * t), "v"(off), "s"(mask + 8 * t) : "m0", "memory");
        const char* const q_seq = a_q + layer * q_stride + (long long)sq.node_off * q_row_bytes + (long long)kvh * G * (D * 2);
#pragma unroll
        for (int xx = 0; xx < (L::kLoads + NW - 1) / NW; ++xx) {
            const int x = xx * NW + wave;
            if (x < L::kLoads) {
                const int R = x * L::kRowsPerLoad + lrow;
                const uint32_t rc = (uint32_t)min(r0 + R, rows - 1), j = div_magic(rc, g_magic);
                direct_load_16(q_seq, j * q_row_bytes + (rc - j * G) * (D * 2) + 16u * (uint32_t)(cpos ^ swz_k<D>(R)), q_lds + x * 1024);
            }
        }
    }
    // ---- direct loads of a block: load x brings rows kRowsPerLoad*x .., lane i chunk i % kChunks (swizzled) of row i / kChunks
    uint32_t voff_k[L::kLoads], voff_v[L::kLoads];
    {
        constexpr int kPeriod = 4;                // the swizzles repeat after four loads
        const uint32_t row0 = (uint32_t)lrow * kv_row_bytes;
#pragma unroll
        for (int x = 0; x < L::kLoads; ++x) {
            if (x < kPeriod) {
                const int row = L::kRowsPerLoad * x + lrow;
                voff_k[x] = row0 + L::kRowsPerLoad * x * kv_row_bytes + 16u * (uint32_t)(cpos ^ swz_k<D>(row));
                voff_v[x] = row0 + L::kRowsPerLoad * x * kv_row_bytes + 16u * (uint32_t)(cpos ^ swz_v<D>(row));
            } else {
                voff_k[x] = voff_k[x - kPeriod] + kPeriod * L::kRowsPerLoad * kv_row_bytes;
                voff_v[x] = voff_v[x - kPeriod] + kPeriod * L::kRowsPerLoad * kv_row_bytes;
            }
        }
    }
    // rows past the end of the region repeat its last row (finite as every row; their scores are masked)
    auto issue = [=](auto v_c, const char* prefix_region, const char* tree_region, const uint32_t (&voff)[L::kLoads], bool tree, int key0, uint32_t dst)
        __attribute__((always_inline)) {
        constexpr bool is_v = decltype(v_c)::value;
        const char* const base = (tree ? tree_region : prefix_region) + (long long)key0 * kv_row_bytes;
        const int there = (tree ? N : P) - key0;
        if (there >= 32) {
            static_for<L::kLoads>([=](auto xc) {
                constexpr int x = decltype(xc)::value;
                direct_load_16(base, voff[x], dst + x * 1024);
            });
        } else {
#pragma unroll 1
            for (int x = 0; x < L::kLoads; ++x) {
                const int row = L::kRowsPerLoad * x + lrow;
                const uint32_t c = (uint32_t)(cpos ^ (is_v ? swz_v<D>(row) : swz_k<D>(row)));
                direct_load_16(base, (uint32_t)min(row, there - 1) * kv_row_bytes + 16u * c, dst + x * 1024);
            }
        }
    };
    auto issue_k = [=](bool tree, int key0) __attribute__((always_inline)) { issue(std::false_type{}, kp, kt, voff_k, tree, key0, slot); };
    auto issue_v = [=](bool tree, int key0) __attribute__((always_inline)) { issue(std::true_type{}, vp, vt, voff_v, tree, key0, slot + L::kMatBytes); };
    int v = wave;                                // place in the walk
    const bool early = v < nP;
    bool tree = false;
    int key0 = 32 * (p_begin + v);
    const bool v_late = kShared<NW> && wave == NW - 1;          // (the query rows lie in its V slot)
    if (early) {
        issue_k(false, key0);
        if (!v_late) issue_v(false, key0);
    }
    // ---- the query rows and visibility words have landed, in every wave
    if (!early) wait_direct_loads();
    else if (v_late) wait_direct_loads_but<L::kLoads>();
    else wait_direct_loads_but<2 * L::kLoads>();
    __syncthreads();
    bf16x8 qf[KK];                                // B operand of the first product: lane holds query n, dims 16 kk + 8 g ..
#pragma unroll
    for (int kk = 0; kk < KK; ++kk)
        qf[kk] = *(lds_bf16x8)(uint32_t)(q_lds + n * L::kRowBytes + (((2 * kk + g) ^ swz_k<D>(n)) << 4));
    if (kShared<NW>) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __syncthreads();
        if (early && v_late) issue_v(false, key0);
    }
    // the walk: the prefix's blocks, then the tree's that any of the rows sees (lane b asks for block b; lane k holds the k-th).
    // A wave looks when it comes to the end of the prefix.
    int seen_blocks = 0, n_blocks = nP;
    bool looked = nTw == 0;
    auto look = [&]() __attribute__((always_inline)) {
        uint32_t any = 0u;
        if (lane < 2 * nTw && 32 * lane < N) {
            typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
            typedef __attribute__((address_space(3))) const u32x4* lds_u32x4;
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const u32x4 w = *(lds_u32x4)(uint32_t)(vis_lds + 128 * lane + 16 * ((k + lane) & 7));
                any |= (w.x | w.y) | (w.z | w.w);
            }
        }
        const unsigned long long act = __builtin_amdgcn_ballot_w64(any != 0u);
        n_blocks = nP + __builtin_popcountll(act);
        const int rank = any != 0u ? __builtin_popcountll(act & ((1ull << lane) - 1ull)) : 63;
        seen_blocks = __builtin_amdgcn_ds_permute(4 * rank, lane);
        looked = true;
    };
    bool have = early;
    if (!early) {
        if (!looked) look();
        have = v < n_blocks;
        if (have) {
            key0 = 32 * __builtin_amdgcn_readlane(seen_blocks, v - nP);
            tree = true;
            issue_k(true, key0);
            issue_v(true, key0);
        }
    }

    // ---- LDS read addresses
    int k_off[KK];                               // K fragment of k-step kk, key row n
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) k_off[kk] = (int)slot + n * L::kRowBytes + (((2 * kk + g) ^ swz_k<D>(n)) << 4);
    int v_off[DB];                               // V^T fragments by the transposing read (lane layout: tree_attn_mfma.hip)
    {
        const int sl = lane & 15, grp = (lane >> 4) & 1;
        const int row = (sl >> 2) + 4 * g;
#pragma unroll
        for (int db = 0; db < DB; ++db) {
            const int chunk = 4 * db + 2 * grp + ((sl & 3) >> 1);
            v_off[db] = (int)slot + L::kMatBytes + row * L::kRowBytes + ((chunk ^ swz_v<D>(row)) << 4) + 8 * (sl & 1);
        }
    }
    const floatx16 zero16 = { 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0 };
    floatx16 acc[DB];                            // O^T: head-dim block db, lane: query n; register i: dim 8 (i/4) + 4 g + i % 4
#pragma unroll
    for (int db = 0; db < DB; ++db) acc[db] = zero16;
    float m_run = -1e30f, l_run = 0.0f;
    bool first = true;

    while (have) {
        const int next_v = v + NW;
        const bool next_tree = next_v >= nP;
        int next_key0 = 32 * (p_begin + next_v);
        if (next_tree) {
            if (!looked) look();
            next_key0 = 32 * __builtin_amdgcn_readlane(seen_blocks, (next_v - nP) & 63);
        }
        const bool more = next_v < n_blocks;
        // ---- S^T = K Q^T; the next block's K follows as soon as this one's is in registers
        wait_direct_loads_but<L::kLoads>();      // (all but this block's V)
        bf16x8 fr[KK];
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) fr[kk] = *(lds_bf16x8)(uint32_t)k_off[kk];
        const bool masked = tree || P - key0 < 32;
        uint32_t vis = ~0u;                      // bit 8 (i/4) + i % 4: the lane's key of register i
        if (tree) vis = *(__attribute__((address_space(3))) const uint32_t*)(uint32_t)(vis_lds + 4 * key0 + 4 * n);
        else if (masked) vis = (1u << (P - key0)) - 1u;
        vis >>= 4 * g;
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        if (more) issue_k(next_tree, next_key0);
        floatx16 S = zero16;
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) S = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[kk], qf[kk], S, 0, 0, 0);
        // ---- numerators against the reference maximum as it stands; if a lane's sum says that is too low (and for
        //      the first block) the reference is raised to the true maximum and they are taken again
        float p[16], ls = 0.0f;
        bool low = first;
        if (!first) {
            const float mc = m_run * c2;
#pragma unroll
            for (int i = 0; i < 16; ++i) p[i] = fast_exp2(fmaf(S[i], c2, -mc));
            if (masked) {
#pragma unroll
                for (int i = 0; i < 16; ++i) p[i] = and_bits(p[i], __builtin_amdgcn_sbfe((int)vis, 8 * (i / 4) + (i % 4), 1));
            }
#pragma unroll
            for (int i = 0; i < 16; ++i) ls += p[i];
            low = __any(!(ls <= kShortSumLimit));
        }
        if (low) {
            float sm[16];
#pragma unroll
            for (int i = 0; i < 16; ++i) sm[i] = S[i];
            if (masked) {
#pragma unroll
                for (int i = 0; i < 16; ++i) if (!((vis >> (8 * (i / 4) + (i % 4))) & 1u)) sm[i] = -INFINITY;
            }
            float mx = -INFINITY;
#pragma unroll
            for (int i = 0; i < 16; i += 2) mx = max3(mx, sm[i], sm[i + 1]);
            mx = fmaxf(mx, __shfl_xor(mx, 32, kWave));
            const float m_new = fmaxf(m_run, mx);
            if (!first) {
                const float alpha = fast_exp2((m_run - m_new) * c2);
                l_run *= alpha;
#pragma unroll
                for (int db = 0; db < DB; ++db)
#pragma unroll
                    for (int i = 0; i < 16; ++i) acc[db][i] *= alpha;
            }
            m_run = m_new;
            const float mc = m_run * c2;
            ls = 0.0f;
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                p[i] = fast_exp2(fmaf(sm[i], c2, -mc));
                ls += p[i];
            }
            first = false;
        }
        l_run += ls;
        union { uint32_t w[8]; bf16x8 v[2]; } pb;           // numerators in bf16: B operand of the second product
#pragma unroll
        for (int i = 0; i < 16; i += 2) {
            const floatx2 pp = { p[i], p[i + 1] };
            pb.w[i / 2] = __builtin_bit_cast(uint32_t, __builtin_convertvector(pp, bf16x2));
        }
        // ---- O^T += V^T P^T; then the next block's V
        if (more) wait_direct_loads_but<L::kLoads>(); else wait_direct_loads();
        bf16x8 vf[2][DB];
#pragma unroll
        for (int ts = 0; ts < 2; ++ts)
#pragma unroll
            for (int db = 0; db < DB; ++db) {
                union { short4v h[2]; bf16x8 v; } f;
#pragma unroll
                for (int half = 0; half < 2; ++half)
                    f.h[half] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4)(uint32_t)(8 * (2 * ts + half) * L::kRowBytes + v_off[db]));
                vf[ts][db] = f.v;
            }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        if (more) issue_v(next_tree, next_key0);
#pragma unroll
        for (int ts = 0; ts < 2; ++ts)
#pragma unroll
            for (int db = 0; db < DB; ++db) acc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[ts][db], pb.v[ts], acc[db], 0, 0, 0);
        v = next_v;
        tree = next_tree;
        key0 = next_key0;
        have = more;
    }

    // ---- merge.  Every wave leaves its rows in its own slots: piece 2 k + e (four dims) of row n at 16-byte place
    //      32 (2 k + e) + (n ^ (k + 16 e)), so that a wave's writes (one piece of all rows) and its reads (a row's even or odd
    //      pieces) both spread over all banks; maxima and sums beside.
    l_run += __shfl_xor(l_run, 32, kWave);
    typedef float floatx4 __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) floatx4* lds_floatx4;
    typedef __attribute__((address_space(3))) floatx2* lds_floatx2;
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int ib = 0; ib < 4; ++ib) {
            const int k = 4 * db + ib;
            *(lds_floatx4)(uint32_t)(slot + 16 * (32 * (2 * k + g) + (n ^ (k + 16 * g)))) =
                floatx4{ acc[db][4 * ib], acc[db][4 * ib + 1], acc[db][4 * ib + 2], acc[db][4 * ib + 3] };
        }
    if (kShared<NW>) __syncthreads();                                  // nobody looks at the visibility words any more
    if (g == 0) *(lds_floatx2)(uint32_t)(ml_lds + 8 * (32 * wave + n)) = floatx2{ m_run, l_run };
    __syncthreads();
    // A lane finishes eight dims of a row at a time (16 bytes of output), wave w rows 32 / NW * w ..
    constexpr int DP = D / 8, RW = kShortRows / NW, IT = (RW * DP + 63) / 64;
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    auto pack = [](const float (&x)[8], float f) -> u32x4 {
        u32x4 w;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const floatx2 v = { x[2 * e] * f, x[2 * e + 1] * f };
            w[e] = __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
        }
        return w;
    };
    char* const out_rows = a.out + layer * q_stride + (long long)sq.node_off * q_row_bytes + (long long)kvh * G * (D * 2);
    // 16 bytes of a finished row, streamed
    auto store = [=](int row, int dp, const u32x4& w) __attribute__((always_inline)) {
        const uint32_t r = (uint32_t)(r0 + row), j = div_magic(r, g_magic);
        if (r < (uint32_t)rows)
            __builtin_nontemporal_store(w, reinterpret_cast<u32x4*>(out_rows + (size_t)(j * q_row_bytes + (r - j * G) * (D * 2) + 16 * dp)));
    };
    const size_t group = ((size_t)layer * gridDim.y + tile) * gridDim.x + kvh;
    unsigned long long* const parts = a.part + group * n_split * L::kPartWords;
#pragma unroll
    for (int t = 0; t < IT; ++t) {
        const int idx = 64 * t + lane, dp = idx % DP, row = wave * RW + idx / DP;
        if (RW * DP % 64 != 0 && idx >= RW * DP) break;
        floatx2 ml[NW];
#pragma unroll
        for (int z = 0; z < NW; ++z) ml[z] = *(lds_floatx2)(uint32_t)(ml_lds + 8 * (32 * z + row));
        float M = ml[0].x, Ls = 0.0f, o[8] = { 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f };
#pragma unroll
        for (int z = 1; z < NW; ++z) M = fmaxf(M, ml[z].x);
#pragma unroll
        for (int z = 0; z < NW; ++z) {
            const float f = fast_exp2((ml[z].x - M) * c2);
            Ls = fmaf(ml[z].y, f, Ls);
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const floatx4 x = *(lds_floatx4)(uint32_t)(lds0 + z * 2 * L::kMatBytes + 16 * (32 * (2 * dp + e) + (row ^ (dp + 16 * e))));
#pragma unroll
                for (int i = 0; i < 4; ++i) o[4 * e + i] = fmaf(x[i], f, o[4 * e + i]);
            }
        }
        if (n_split == 1) {
            store(row, dp, pack(o, 1.0f / Ls));
        } else {
            // Prefix split: as in tree_attn_mfma.hip every workgroup leaves its normalised rows (bf16) and their (max, sum) in
            // the workspace with device-scope accesses and counts its arrival; the last one merges all, in split order.
            unsigned long long* const mine = parts + (size_t)split * L::kPartWords;
            const u32x4 w = pack(o, Ls > 0.0f ? 1.0f / Ls : 0.0f);     // a split without keys: weight 0, rows 0
#pragma unroll
            for (int e = 0; e < 2; ++e)
                __hip_atomic_store(mine + row * (D / 4) + 2 * dp + e, ((unsigned long long)w[2 * e + 1] << 32) | w[2 * e], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (dp == 0)
                __hip_atomic_store(mine + kShortRows * (D / 4) + row, ((unsigned long long)__float_as_uint(Ls) << 32) | __float_as_uint(M),
                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    if (n_split == 1) return;
    // every store of the workgroup has been acknowledged before its arrival is counted
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    typedef __attribute__((address_space(3))) uint32_t* lds_u32;
    const lds_u32 flag = (lds_u32)lds0;
    if (threadIdx.x == 0) {
        const unsigned before = __builtin_amdgcn_atomic_inc32(a.counters + group, (unsigned)n_split - 1u, __ATOMIC_RELAXED, "agent");
        *flag = before == (unsigned)n_split - 1u;
    }
    __syncthreads();
    if (*flag == 0u) return;                                           // uniform over the workgroup
#pragma unroll
    for (int t = 0; t < IT; ++t) {
        const int idx = 64 * t + lane, dp = idx % DP, row = wave * RW + idx / DP;
        if (RW * DP % 64 != 0 && idx >= RW * DP) break;
        constexpr int Z = kShortSplits;
        unsigned long long w[Z][2], ml[Z];
#pragma unroll
        for (int z = 0; z < Z; ++z) {
            ml[z] = (unsigned long long)__float_as_uint(-1e30f);
            w[z][0] = w[z][1] = 0ull;
            if (z < n_split) {                                         // uniform
                const unsigned long long* const part = parts + (size_t)z * L::kPartWords;
#pragma unroll
                for (int e = 0; e < 2; ++e)
                    w[z][e] = __hip_atomic_load(part + row * (D / 4) + 2 * dp + e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                ml[z] = __hip_atomic_load(part + kShortRows * (D / 4) + row, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        float M = -1e30f, Ls = 0.0f, o[8] = { 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f };
#pragma unroll
        for (int z = 0; z < Z; ++z) M = fmaxf(M, __uint_as_float((uint32_t)ml[z]));
#pragma unroll
        for (int z = 0; z < Z; ++z) {
            const float wz = fast_exp2((__uint_as_float((uint32_t)ml[z]) - M) * c2) * __uint_as_float((uint32_t)(ml[z] >> 32));
            Ls += wz;
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const uint32_t lo = (uint32_t)w[z][e], hi = (uint32_t)(w[z][e] >> 32);
                o[4 * e] = fmaf(wz, __uint_as_float(lo << 16), o[4 * e]);
                o[4 * e + 1] = fmaf(wz, __uint_as_float(lo & 0xffff0000u), o[4 * e + 1]);
                o[4 * e + 2] = fmaf(wz, __uint_as_float(hi << 16), o[4 * e + 2]);
                o[4 * e + 3] = fmaf(wz, __uint_as_float(hi & 0xffff0000u), o[4 * e + 3]);
            }
        }
        store(row, dp, pack(o, 1.0f / Ls));
    }
}

template <int D, int NW>
static hipError_t raise_short_lds()
{
    static std::atomic<unsigned long long> done{0};
    return raise_dynamic_lds_once(reinterpret_cast<const void*>(&tree_attn_short_kernel<D, NW>), short_lds_bytes<D, NW>(DYSPEC_MAX_NODES / 64), done);
}

hipError_t prepare_tree_attn_short()
{
    hipError_t e = raise_short_lds<128, 8>();
    if (e == hipSuccess) e = raise_short_lds<128, 4>();
    if (e == hipSuccess) e = raise_short_lds<128, 2>();
    if (e == hipSuccess) e = raise_short_lds<64, 8>();
    if (e == hipSuccess) e = raise_short_lds<64, 4>();
    return e;
}

template <int D, int NW>
static hipError_t launch_short(const ShortArgs& s, int Hkv, int blocks, int layers, int tree_tiles, hipStream_t stream)
{
    const hipError_t e = raise_short_lds<D, NW>();
    if (e != hipSuccess) return e;
    tree_attn_short_kernel<D, NW><<<dim3(Hkv, blocks, layers * s.n_split), 64 * NW, short_lds_bytes<D, NW>(tree_tiles), stream>>>(s);
    return hipGetLastError();
}

// Time of a call by either kernel, in us, from what its sizes are: the launch and a workgroup's fixed part, then whichever
// is longest: the longest walk, all workgroups' work over the chip, the prefix's bytes.  Fitted to 600 one-layer shapes (1 to 8
// sequences, trees of 8 to 2048 rows, prefixes of 0 to 8192 keys, 32 / 40 / 64 heads, head_dim 64 and 128; K and V of
// successive launches not in cache), there right to 11 - 15 % rms and the choice within 4 % (head_dim 64: 7 %) of always the faster form.
// Over 33000 shapes with 1 to 64 KV heads and 1 to 80 layers it is right to 20 - 35 % and the calls take 0.72 of the other kernel's
// time (the fastest form of each: 0.64); one layer is slower by more than 5 % in 0.2 - 0.4 % of the calls that this kernel takes, 8 to 80
// layers in 2 - 4 %.  The exceptions in tree_attn_short_plan are for kinds of calls that came out slower.
struct CallCost {
    float launch, walk0, walk;      // launch; the longest walk: fixed part, per unit of keys
    float alone;                    // a unit of keys takes this share more if no other row block walks it (k row blocks: 1/k of that)
    float work0, work;              // a workgroup's share of the chip: fixed part, per unit of keys
    float merge, merge_part;        // a split prefix: once, per part
    float bytes;                    // MB of K and V per us
};
struct CallCosts { CallCost tall, short8, short4, short2; };     // tree_attn_mfma.hip, units of 64 keys; this kernel with 8, 4, 2 waves, of 32
constexpr CallCosts kCosts128 = { { 4.85f, 2.35f, 0.98f, 0.1f, 7.6f, 1.14f, 1.2f, 0.42f, 4.3f },
                                  { 2.0f, 2.2f, 0.256f, 0.45f, 4.0f, 0.257f, 2.1f, 0.18f, 4.3f },
                                  { 4.3f, 0.0f, 0.261f, 0.37f, 1.33f, 0.229f, 0.0f, 0.0f, 1.9f },
                                  { 5.05f, 0.0f, 0.413f, 0.0f, 0.70f, 0.243f, 0.0f, 0.0f, 1.7f } };
constexpr CallCosts kCosts64 = { { 3.95f, 2.7f, 0.657f, 0.12f, 4.54f, 0.928f, 1.46f, 0.21f, 4.2f },
                                 { 3.6f, 0.0f, 0.166f, 0.55f, 1.08f, 0.168f, 2.0f, 0.13f, 3.9f },
                                 { 3.7f, 0.0f, 0.192f, 0.2f, 0.66f, 0.155f, 0.0f, 0.0f, 1.7f },
                                 {} };                                 // (two waves: never the best at head_dim 64)
constexpr float kClearlyLess = 0.9f;       // this kernel is taken where it is this much better: the model's error

struct CallTime { float once, work, whole; };     // of one call on an idle chip; its share of a full chip; once, no workgroup shared by two CUs
static CallTime call_time(const CallCost& c, const SeqArgs& sa, int G, int Hkv, int d, int layers, int splits, int rows_per_group, int keys_per_unit)
{
    float longest = 0.0f, work = 0.0f, keys = 0.0f, workgroups = 0.0f;
    for (int s = 0; s < sa.n_seq; ++s) {
        const int N = sa.node_off[s + 1] - sa.node_off[s];
        if (N == 0) continue;
        const int groups = (G * N + rows_per_group - 1) / rows_per_group;
        // of the tree a block of rows sees a few tiles, however large it is (the long kernel's masked tiles cost half as much again)
        const float tree = keys_per_unit == 64 ? 1.5f * (float)min((N + 63) / 64, 3) : (float)min((N + 31) / 32, 5);
        const float units = ((float)((sa.prefix_len[s] + keys_per_unit - 1) / keys_per_unit) + tree) / (float)splits;
        longest = fmaxf(longest, units * (1.0f + c.alone / (float)groups));
        work += (float)groups * (float)splits * (c.work0 + c.work * units);
        keys += (float)sa.prefix_len[s];
        workgroups += (float)groups;
    }
    work *= (float)Hkv * (float)layers / 256.0f;
    workgroups *= (float)splits * (float)Hkv * (float)layers / 256.0f;        // a CU
    const float bytes = keys * (float)Hkv * (float)d * 4e-6f * (float)layers / c.bytes;
    CallTime t;
    t.work = fmaxf(work, bytes);
    const float walk = c.walk0 + c.walk * longest, rest = c.launch + (splits > 1 ? c.merge + c.merge_part * (float)splits : 0.0f);
    t.once = rest + fmaxf(walk, t.work);
    t.whole = rest + fmaxf(walk, fmaxf(work * ceilf(workgroups) / workgroups, bytes));
    return t;
}

static long long row_blocks(const SeqArgs& sa, int G)
{
    long long blocks = 0;
    for (int s = 0; s < sa.n_seq; ++s) blocks += ((long long)G * (sa.node_off[s + 1] - sa.node_off[s]) + kShortRows - 1) / kShortRows;
    return blocks;
}

// The forms there are; parts only as many as are resident at once and as the workspace has room for.
bool tree_attn_short_has(const SeqArgs& sa, int Hq, int Hkv, int d, int layers, size_t workspace_bytes, int waves, int splits)
{
    const int G = Hq / Hkv;
    const long long blocks = row_blocks(sa, G), groups = blocks * Hkv * layers;
    // (grid limits; rows divided by G through a product with 32-bit factors)
    if (blocks == 0 || blocks > 65535 || (long long)layers * kShortSplits > 65535 || G > 1024) return false;
    if (waves != 8 && waves != 4 && !(waves == 2 && d == 128)) return false;
    if (splits == 1) return true;
    const size_t part = (size_t)(kShortRows * (d / 4 + 1)) * sizeof(unsigned long long);
    return waves == 8 && splits > 1 && splits <= kShortSplits && groups * splits <= 256 && kAttnCounterBytes + (size_t)groups * splits * part <= workspace_bytes;
}

ShortPlan tree_attn_short_plan(const SeqArgs& sa, int Hq, int Hkv, int d, int layers, int long_splits, size_t workspace_bytes)
{
    const int G = Hq / Hkv;
    ShortPlan best = { 0, 1 };
    if (!tree_attn_short_has(sa, Hq, Hkv, d, layers, 0, 8, 1)) return best;
    // Where the long kernel has no parts to merge either, the choice is the same whatever the number of layers (one layer's
    // result does not depend on the others): this kernel has to be better for a call by itself and with the chip full.
    const bool any_layers = long_splits == 1;
    const int L = any_layers ? 1 : layers;
    const CallCosts& costs = d == 128 ? kCosts128 : kCosts64;
    const CallTime other = call_time(costs.tall, sa, G, Hkv, d, L, long_splits, 128, 64);
    float least = kClearlyLess * other.once;
    // Several layers of which the long kernel splits the prefix are about one workgroup a CU there; a few more of this kernel's
    // than one a CU take as long as two.  2 KV heads of 6, 23 rows, 5271 keys, head_dim 64, 32 layers: 320 workgroups, 66 us for
    // the other's 40.  (One layer is bound by its longest walk: there the whole workgroups say nothing.)
    const bool whole_counts = !any_layers && layers > 1;
    auto consider = [&](const CallCost& c, int waves, int splits) {
        const CallTime t = call_time(c, sa, G, Hkv, d, L, splits, kShortRows, 32);
        if (t.once < least && (!any_layers || t.work < kClearlyLess * other.work) && (!whole_counts || kClearlyLess * t.whole < other.whole)) {
            least = t.once;
            best = { waves, splits };
        }
    };
    if (d == 128) consider(costs.short2, 2, 1);
    consider(costs.short4, 4, 1);
    // At head_dim 64 a walk of at most four blocks of keys has no use for eight waves: half of them bring no keys and still join in the
    // merge (25 rows alone, 64/8 heads: 80 layers 36 us, 18 with four waves, 27 with the other kernel; one layer 5.0 and 4.6).  At head_dim
    // 128 eight are better by 1 - 2 % in one layer, as each finishes fewer rows.
    int most_blocks = 0;
    for (int s = 0; s < sa.n_seq; ++s) {
        const int N = sa.node_off[s + 1] - sa.node_off[s];
        if (N > 0) most_blocks = max(most_blocks, (sa.prefix_len[s] + 31) / 32 + (N + 31) / 32);
    }
    if (d == 128 || most_blocks > 4) consider(costs.short8, 8, 1);
    for (int splits = 2; !any_layers && tree_attn_short_has(sa, Hq, Hkv, d, layers, workspace_bytes, 8, splits); ++splits)
        consider(costs.short8, 8, splits);
    // Two waves are for many row blocks of short walks.  Where one long walk is twice the chip's share, that walk is what is waited for
    // and four waves take 0.61 of the time (one layer; 0.76 two or four layers, 1.03 more): trees of 10, 1005, 32 .. 5 rows, the third
    // behind 6883 keys, one KV head of 8: 73 us by the other kernel, 91 with two waves, 47 with four.
    if (best.waves == 2) {
        const CallTime t = call_time(costs.short2, sa, G, Hkv, d, L, 1, kShortRows, 32);
        if (t.once > 2.0f * (costs.short2.launch + t.work)) best.waves = 4;
    }
    return best;
}

hipError_t launch_tree_attn_short(const AttnArgs& a, const SeqArgs& sa, int waves, hipStream_t stream)
{
    ShortArgs s;
    s.q = static_cast<const char*>(a.q); s.kp = static_cast<const char*>(a.kp); s.vp = static_cast<const char*>(a.vp);
    s.kt = static_cast<const char*>(a.kt); s.vt = static_cast<const char*>(a.vt); s.mask = reinterpret_cast<const char*>(a.mask);
    s.out = static_cast<char*>(a.out);
    s.part = reinterpret_cast<unsigned long long*>(a.part); s.counters = a.counters;
    s.q_stride = a.q_stride; s.kvp_stride = a.kvp_stride; s.kvt_stride = a.kvt_stride;
    s.kv_row_bytes = (uint32_t)a.Hkv * a.d * 2; s.q_row_bytes = (uint32_t)a.Hq * a.d * 2;
    s.G = (uint32_t)(a.Hq / a.Hkv);
    s.g_magic = s.G > 1 ? (uint32_t)((1ull << 32) / s.G + 1) : 0u;
    s.mask_bytes = a.mask_words * 8;
    s.n_split = a.splits; s.n_seq = sa.n_seq;
    s.c2 = a.scale * 1.4426950408889634f;
    // sequences of longer walks first, so that the last workgroups to start are short ones
    int order[DYSPEC_MAX_SEQ];
    for (int i = 0; i < sa.n_seq; ++i) {
        int k = i;
        for (; k > 0 && sa.prefix_len[order[k - 1]] < sa.prefix_len[i]; --k) order[k] = order[k - 1];
        order[k] = i;
    }
    int blocks = 0;
    for (int i = 0; i < sa.n_seq; ++i) {
        const int q = order[i], N = sa.node_off[q + 1] - sa.node_off[q];
        s.seq[i] = { blocks, sa.node_off[q], N, sa.prefix_len[q], sa.kv_off[q], 0 };
        blocks += ((int)s.G * N + kShortRows - 1) / kShortRows;
    }
    s.one = s.seq[0];
    if (a.d == 128)
        return waves == 8   ? launch_short<128, 8>(s, a.Hkv, blocks, a.layers, a.mask_words, stream)
               : waves == 4 ? launch_short<128, 4>(s, a.Hkv, blocks, a.layers, a.mask_words, stream)
                            : launch_short<128, 2>(s, a.Hkv, blocks, a.layers, a.mask_words, stream);
    return waves == 8 ? launch_short<64, 8>(s, a.Hkv, blocks, a.layers, a.mask_words, stream)
                      : launch_short<64, 4>(s, a.Hkv, blocks, a.layers, a.mask_words, stream);
}

}  // namespace dyspec

// Vocabulary softmax statistics of every tree row and multi-candidate tree rejection
// sampling (Algorithm 3, Appendix A.3; one-candidate rule of Section 2) for gfx950.
//
// Two kernels.  The statistics kernel is the data-parallel part: it reads every tree row's
// draft and target logits from HBM once and reduces each to (max, sum-exp), the normalisers
// every later probability needs (streaming forms; a plain one workgroup per row form for rows
// below 16 bytes).  verify_walk_kernel is Algorithm 3 itself,
// one workgroup per sequence walking from the root: the first child of a node is tested
// from two logits and the row statistics alone; only after a rejection are the node's two
// rows brought into registers (as weights of a known sum, no reduction) for the residual
// updates R <- norm(max(R-D,0)), D[y] <- 0, D <- norm(D), one pass over the registers and one workgroup reduction per
// rejected child, stopping at the first accepted one.  Tree links of the
// sequence are staged in LDS so the walk chases pointers there, not in HBM.
//
// A target temperature of 0 (the temperature-0 rows of Section 5's tables) makes the target
// row all mass on its largest logit, the smallest index winning a tie.  For such a sequence
// the statistics pass stores (largest raw target logit, its index) in place of (max, sum-exp)
// and the walk builds its target row from that index instead of reading the logits; every
// other step of Algorithm 3 runs unchanged.
#include "lane_ops.h"

namespace dyspec {

// (value, index) pairs ordered by larger value, then smaller index
__device__ __forceinline__ void better_of(float& m, int& i, float m2, int i2)
{
    if (m2 > m || (m2 == m && i2 < i)) { m = m2; i = i2; }
}

// Largest value and the first index holding it over a workgroup of NW waves; every thread
// brings its own best pair.  The result is valid in thread 0.
template <int NW>
__device__ __forceinline__ void block_argmax(float& m, int& i, float* red_m, int* red_i)
{
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) better_of(m, i, __shfl_xor(m, o, kWave), __shfl_xor(i, o, kWave));
    const int wave = threadIdx.x / kWave;
    if ((threadIdx.x & (kWave - 1)) == 0) { red_m[wave] = m; red_i[wave] = i; }
    __syncthreads();
    if (threadIdx.x == 0) {
        m = red_m[0]; i = red_i[0];
        for (int w = 1; w < NW; ++w) better_of(m, i, red_m[w], red_i[w]);
    }
}

template <typename T>
__global__ __launch_bounds__(kBlock) void softmax_stats_kernel(
    const T* __restrict__ draft_logits, const T* __restrict__ target_logits, int V,
    SeqArgs sa, float* __restrict__ row_stats, float* __restrict__ accept_ratio)
{
    __shared__ float fred[kWaves * 2];
    __shared__ int ired[kWaves];
    const int row = blockIdx.x;
    const int seq = find_seq(sa, row);
    const bool greedy = sa.temp_t[seq] == 0.0f;
    const float inv_td = 1.0f / sa.temp_d[seq], inv_tt = greedy ? 1.0f : 1.0f / sa.temp_t[seq];
    float D[kMaxSeg][4], R[kMaxSeg][4];
    load_row<false, T>(draft_logits + (size_t)row * V, V, D);
    load_row<false, T>(target_logits + (size_t)row * V, V, R);
    float top = -INFINITY;
    int top_i = 0;
    if (greedy) {
#pragma unroll
        for (int j = 0; j < kMaxSeg; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (R[j][e] > top) { top = R[j][e]; top_i = tok_index(j, e); }   // ascending index per thread
        block_argmax<kWaves>(top, top_i, fred, ired);
        __syncthreads();
    }
    float mx[2] = { -INFINITY, -INFINITY };
#pragma unroll
    for (int j = 0; j < kMaxSeg; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            D[j][e] *= inv_td; R[j][e] *= inv_tt;
            mx[0] = fmaxf(mx[0], D[j][e]); mx[1] = fmaxf(mx[1], R[j][e]);
        }
    block_max<2>(mx, fred);
    float sm[2] = { 0.0f, 0.0f };
#pragma unroll
    for (int j = 0; j < kMaxSeg; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            sm[0] += expf(D[j][e] - mx[0]); sm[1] += expf(R[j][e] - mx[1]);   // exp(-inf) = 0 past V
        }
    block_sum<float, 2>(sm, fred);
    if (threadIdx.x == 0) {
        *reinterpret_cast<float4*>(row_stats + 4 * (size_t)row) =
            greedy ? make_float4(mx[0], sm[0], top, (float)top_i) : make_float4(mx[0], sm[0], mx[1], sm[1]);
        accept_ratio[row] = (row == sa.node_off[seq]) ? 0.0f : -2.0f;      // -2: not tested by the walk
    }
}

// Streaming form of the statistics pass for fp32 rows of whole pieces, V % 4 == 0: one workgroup of 256 threads per
// (row, table), so a 512-row batch puts 1024 independent 128 KB streams on the chip.  Each
// thread keeps a running (max, sum) pair over its 16-byte pieces, eight pieces in flight, and
// raises its reference once per batch of 32 values (33 exponentials per 32 values); pairs are
// merged with (m, s) + (m', s') = (M, s 2^{c(m-M)} + s' 2^{c(m'-M)}), M = max(m, m').  The
// maximum is taken over the raw logits, so max * (1/T) is rounded exactly as the plain
// two-pass form rounds it.
constexpr int kStatThreads = 256;
constexpr int kStatUnroll = 8;

// NANS: what both hold without a maximum is kept (NaN among their values).  (No branch: with one a call takes 0.5 us longer.)
template <bool NANS = false>
__device__ __forceinline__ void merge_stat(float& m, float& s, float m2, float s2, float c)
{
    const float M = fmaxf(m, m2);
    const bool empty = M == -INFINITY;
    if (!NANS && empty) return;
    const float f = __builtin_amdgcn_exp2f((m - M) * c), f2 = __builtin_amdgcn_exp2f((m2 - M) * c);
    s = s * (NANS && empty ? 1.0f : f) + s2 * (NANS && empty ? 1.0f : f2);
    m = M;
}

__global__ __launch_bounds__(kStatThreads) void softmax_stats_stream_kernel(
    const float* __restrict__ draft_logits, const float* __restrict__ target_logits, int V,
    SeqArgs sa, float* __restrict__ row_stats, float* __restrict__ accept_ratio)
{
    __shared__ float red[2 * (kStatThreads / kWave)];
    const int row = blockIdx.x, table = blockIdx.y;
    const int seq = find_seq(sa, row);
    const float4* __restrict__ x = reinterpret_cast<const float4*>((table ? target_logits : draft_logits) + (size_t)row * V);
    const int n4 = V / 4;
    if (table == 1 && sa.temp_t[seq] == 0.0f) {                  // whole workgroup takes this branch
        __shared__ int ired[kStatThreads / kWave];
        float top = -INFINITY;
        int top_i = 0;
        for (int i0 = threadIdx.x; i0 < n4; i0 += kStatThreads * kStatUnroll) {
            float4 v[kStatUnroll];
#pragma unroll
            for (int u = 0; u < kStatUnroll; ++u) {
                const int i = i0 + u * kStatThreads;
                v[u] = (i < n4) ? x[i] : make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
            }
#pragma unroll
            for (int u = 0; u < kStatUnroll; ++u) {              // ascending index per thread
                const int i = 4 * (i0 + u * kStatThreads);
                if (v[u].x > top) { top = v[u].x; top_i = i; }
                if (v[u].y > top) { top = v[u].y; top_i = i + 1; }
                if (v[u].z > top) { top = v[u].z; top_i = i + 2; }
                if (v[u].w > top) { top = v[u].w; top_i = i + 3; }
            }
        }
        block_argmax<kStatThreads / kWave>(top, top_i, red, ired);
        if (threadIdx.x == 0)
            *reinterpret_cast<float2*>(row_stats + 4 * (size_t)row + 2) = make_float2(top, (float)top_i);
        return;
    }
    const float inv_t = 1.0f / (table ? sa.temp_t[seq] : sa.temp_d[seq]);
    const float c = inv_t * 1.4426950408889634f;
    float m = -INFINITY, s = 0.0f;
    for (int i0 = threadIdx.x; i0 < n4; i0 += kStatThreads * kStatUnroll) {
        float4 v[kStatUnroll];
#pragma unroll
        for (int u = 0; u < kStatUnroll; ++u) {
            const int i = i0 + u * kStatThreads;
            v[u] = (i < n4) ? x[i] : make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
        }
        float cm = -INFINITY;
#pragma unroll
        for (int u = 0; u < kStatUnroll; ++u) cm = fmaxf(fmaxf(cm, fmaxf(v[u].x, v[u].y)), fmaxf(v[u].z, v[u].w));
        const float M = fmaxf(m, cm);
        if (M == -INFINITY) continue;                            // nothing but -inf logits so far
        float acc = s * __builtin_amdgcn_exp2f((m - M) * c);
        const float Mc = M * c;
#pragma unroll
        for (int u = 0; u < kStatUnroll; ++u) {
            acc += __builtin_amdgcn_exp2f(fmaf(v[u].x, c, -Mc)) + __builtin_amdgcn_exp2f(fmaf(v[u].y, c, -Mc));
            acc += __builtin_amdgcn_exp2f(fmaf(v[u].z, c, -Mc)) + __builtin_amdgcn_exp2f(fmaf(v[u].w, c, -Mc));
        }
        s = acc;
        m = M;
    }
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) merge_stat(m, s, __shfl_xor(m, o, kWave), __shfl_xor(s, o, kWave), c);
    const int wave = threadIdx.x / kWave;
    if ((threadIdx.x & (kWave - 1)) == 0) { red[2 * wave] = m; red[2 * wave + 1] = s; }
    __syncthreads();
    if (threadIdx.x == 0) {
        m = red[0]; s = red[1];
#pragma unroll
        for (int w = 1; w < kStatThreads / kWave; ++w) merge_stat(m, s, red[2 * w], red[2 * w + 1], c);
        *reinterpret_cast<float2*>(row_stats + 4 * (size_t)row + 2 * table) = make_float2(m * inv_t, s);
        if (table == 0) accept_ratio[row] = (row == sa.node_off[seq]) ? 0.0f : -2.0f;   // -2: not tested by the walk
    }
}

// Sixteen bytes of a logits row: four fp32 or eight bf16 values.
template <typename T> struct Piece;
template <> struct Piece<float> {
    static constexpr int N = 4;
    __device__ static __forceinline__ void unpack(const uint4& r, float (&f)[4])
    {
        f[0] = __uint_as_float(r.x); f[1] = __uint_as_float(r.y); f[2] = __uint_as_float(r.z); f[3] = __uint_as_float(r.w);
    }
};
template <> struct Piece<__bf16> {
    static constexpr int N = 8;
    __device__ static __forceinline__ void unpack(const uint4& r, float (&f)[8])
    {
        f[0] = bf16_bits_to_float(r.x & 0xffffu); f[1] = bf16_bits_to_float(r.x >> 16);
        f[2] = bf16_bits_to_float(r.y & 0xffffu); f[3] = bf16_bits_to_float(r.y >> 16);
        f[4] = bf16_bits_to_float(r.z & 0xffffu); f[5] = bf16_bits_to_float(r.z >> 16);
        f[6] = bf16_bits_to_float(r.w & 0xffffu); f[7] = bf16_bits_to_float(r.w >> 16);
    }
};

// The streaming form for tables of type T read in 16-byte pieces; V a multiple of the values in
// a piece.  (fp32 tables take the kernel above, written out for four values per piece.)  RAGGED: any V of a piece or more, rows that begin at
// any value.  The pieces are read where they lie (wide loads need no alignment beyond the type's), the end of a row by its last 16 bytes.  These rows had
// been held in registers, 64 values a thread whatever V, read one by one and with the library's exponential: 512 rows of 32002 tokens with the walk 65 -> 38 us,
// 2517 rows in bf16 491 -> 101, 7999 tokens 47 -> 27 and 189 -> 61, 1001 tokens 43 -> 24 and 148 -> 52 (whole rows of 32000: 36 and 96).
// The sums are made relative to the rounded maximum over T that the walk subtracts, by x / T - max in one rounding, in four chains: the
// normaliser's error is below that of the form before (deviation 2, 3, 10 and Zipf, mean 1.4e-7, 2.3e-7, 7.3e-7, 0.6e-7; 1.5, 2.8, 8.3, 0.75).
template <typename T, bool RAGGED>
__global__ __launch_bounds__(kStatThreads) void softmax_stats_stream_pieces_kernel(
    const T* __restrict__ draft_logits, const T* __restrict__ target_logits, int V,
    SeqArgs sa, float* __restrict__ row_stats, float* __restrict__ accept_ratio)
{
    constexpr int PN = Piece<T>::N;
    __shared__ float red[2 * (kStatThreads / kWave)];
    const int row = blockIdx.x, table = blockIdx.y;
    const int seq = find_seq(sa, row);
    // pieces are fetched as float4 (one 16-byte load each; the bits are taken apart afterwards)
    const T* __restrict__ const x = (table ? target_logits : draft_logits) + (size_t)row * V;
    const int n16 = (V + PN - 1) / PN;
    // a piece past the end re-reads the last piece and is then set to -inf; RAGGED: the last piece ends with the row, and those of its
    // values that belong to the piece before are set to -inf
    auto begin = [&](int i) __attribute__((always_inline)) { return min(PN * i, V - PN); };
    auto fetch = [&](int i) __attribute__((always_inline)) {
        if constexpr (RAGGED) {
            const typename Unaligned<T>::Piece r = *reinterpret_cast<const typename Unaligned<T>::Piece*>(reinterpret_cast<const char*>(x) + (uint32_t)sizeof(T) * (uint32_t)begin(i));
            return make_float4(__uint_as_float(r.x), __uint_as_float(r.y), __uint_as_float(r.z), __uint_as_float(r.w));
        } else {
            return reinterpret_cast<const float4*>(x)[min(i, n16 - 1)];
        }
    };
    auto open_piece = [&](const float4& r, int i, float (&f)[PN]) __attribute__((always_inline)) {
        Piece<T>::unpack(make_uint4(__float_as_uint(r.x), __float_as_uint(r.y), __float_as_uint(r.z), __float_as_uint(r.w)), f);
        const int skip = RAGGED ? PN * i - begin(i) : 0;
#pragma unroll
        for (int e = 0; e < PN; ++e) f[e] = (RAGGED ? e >= skip : i < n16) ? f[e] : -INFINITY;
    };
    if (table == 1 && sa.temp_t[seq] == 0.0f) {                  // whole workgroup takes this branch
        __shared__ int ired[kStatThreads / kWave];
        float top = -INFINITY;
        int top_i = 0;
        for (int i0 = threadIdx.x; i0 < n16; i0 += kStatThreads * kStatUnroll) {
            float4 v[kStatUnroll];
#pragma unroll
            for (int u = 0; u < kStatUnroll; ++u) v[u] = fetch(i0 + u * kStatThreads);
#pragma unroll
            for (int u = 0; u < kStatUnroll; ++u) {              // ascending index per thread
                const int i = RAGGED ? begin(i0 + u * kStatThreads) : PN * (i0 + u * kStatThreads);
                float f[PN];
                open_piece(v[u], i0 + u * kStatThreads, f);
#pragma unroll
                for (int e = 0; e < PN; ++e) if (f[e] > top) { top = f[e]; top_i = i + e; }
            }
        }
        block_argmax<kStatThreads / kWave>(top, top_i, red, ired);
        if (threadIdx.x == 0)
            *reinterpret_cast<float2*>(row_stats + 4 * (size_t)row + 2) = make_float2(top, (float)top_i);
        return;
    }
    const float inv_t = 1.0f / (table ? sa.temp_t[seq] : sa.temp_d[seq]);
    // m: the largest logit so far, s relative to it; RAGGED: the largest over T, rounded, which the walk subtracts as well
    constexpr float kLog2e = 1.4426950408889634f;
    const float c = RAGGED ? kLog2e : inv_t * kLog2e;
    float m = -INFINITY, s = 0.0f;
    for (int i0 = threadIdx.x; i0 < n16; i0 += kStatThreads * kStatUnroll) {
        float4 v[kStatUnroll];
#pragma unroll
        for (int u = 0; u < kStatUnroll; ++u) v[u] = fetch(i0 + u * kStatThreads);
        float f[kStatUnroll][PN];
        float cm = -INFINITY;
#pragma unroll
        for (int u = 0; u < kStatUnroll; ++u) {
            open_piece(v[u], i0 + u * kStatThreads, f[u]);
#pragma unroll
            for (int e = 0; e < PN; e += 2) cm = fmaxf(cm, fmaxf(f[u][e], f[u][e + 1]));
        }
        const float M = fmaxf(m, RAGGED ? cm * inv_t : cm);
        if (M == -INFINITY) {                                    // nothing but -inf logits so far, or NaN
            if constexpr (RAGGED) {
#pragma unroll
                for (int u = 0; u < kStatUnroll; ++u)
#pragma unroll
                    for (int e = 0; e < PN; ++e) s += f[u][e] == f[u][e] ? 0.0f : f[u][e];
            }
            continue;
        }
        float acc = s * __builtin_amdgcn_exp2f((m - M) * c);
        const float Mc = M * c;
        float part[4] = { 0.0f, 0.0f, 0.0f, 0.0f };              // (shorter chains of roundings)
#pragma unroll
        for (int u = 0; u < kStatUnroll; ++u)
#pragma unroll
            for (int e = 0; e < PN; e += 2) {
                if constexpr (RAGGED) part[u % 4] += __builtin_amdgcn_exp2f(fmaf(f[u][e], inv_t, -M) * c) + __builtin_amdgcn_exp2f(fmaf(f[u][e + 1], inv_t, -M) * c);
                else acc += __builtin_amdgcn_exp2f(fmaf(f[u][e], c, -Mc)) + __builtin_amdgcn_exp2f(fmaf(f[u][e + 1], c, -Mc));
            }
        s = RAGGED ? acc + ((part[0] + part[1]) + (part[2] + part[3])) : acc;
        m = M;
    }
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) merge_stat<RAGGED>(m, s, __shfl_xor(m, o, kWave), __shfl_xor(s, o, kWave), c);
    const int wave = threadIdx.x / kWave;
    if ((threadIdx.x & (kWave - 1)) == 0) { red[2 * wave] = m; red[2 * wave + 1] = s; }
    __syncthreads();
    if (threadIdx.x == 0) {
        m = red[0]; s = red[1];
#pragma unroll
        for (int w = 1; w < kStatThreads / kWave; ++w) merge_stat<RAGGED>(m, s, red[2 * w], red[2 * w + 1], c);
        *reinterpret_cast<float2*>(row_stats + 4 * (size_t)row + 2 * table) = make_float2(RAGGED ? m : m * inv_t, s);
        if (table == 0) accept_ratio[row] = (row == sa.node_off[seq]) ? 0.0f : -2.0f;   // -2: not tested by the walk
    }
}

// exp(x) for x <= 0 through the hardware's exp2 (inputs below -126/log2(e) give 0, which is what a
// probability that small is here): one multiply and one v_exp_f32, about 1e-7 |x| of relative
// error, against some twenty instructions of the library routine -- a thread turns 128 logits
// into probabilities per visited node.
__device__ __forceinline__ float exp_fast(float x) { return __builtin_amdgcn_exp2f(x * 1.4426950408889634f); }

// A thread's tokens of a row of S segments: component e of segment j is v[e][j] (a segment known to be the same in every
// thread picks the registers by index).
template <int S> using RowVec = float __attribute__((ext_vector_type(S)));
__device__ __forceinline__ double four(const float a, const float b, const float c, const float d) { return ((double)a + (double)b) + ((double)c + (double)d); }

// Sums over the wave of N values a lane (N = 2, 8 or 16), scattered: lane l gets the sum of value l % N.
template <int N>
__device__ __forceinline__ double wave_sums(double (&x)[N])
{
    double t = row_sums(x);
    t += __shfl_xor(t, 16, kWave);
    t += __shfl_xor(t, 32, kWave);
    return t;
}

// Inverse CDF over a register-resident row of weights (the step's last token): the smallest token index y, in the order
// (segment, thread, element), whose cumulative weight exceeds u * W.  Sums are fp64.  Every wave leaves its sum of every segment
// in LDS; every wave scans those S * 8 sums and picks segment and wave of the crossing; that wave scans its 64 sums of the
// segment, and the owning lane walks its four weights.  Two barriers.  Every thread gets y (-1 when W == 0).
// (With every thread's sums staged in LDS and a serial pick among the segments, three barriers: 3.2 to 4.3 us, now 2.4 to 3.2.)
struct DrawScratch {
    double part[kMaxSeg * kWaves];
    int y;
};
template <int S>
__device__ __forceinline__ int draw_from_row(const RowVec<S> (&w)[4], double u, DrawScratch* sc)
{
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    {
        double seg[S];
#pragma unroll
        for (int j = 0; j < S; ++j) seg[j] = four(w[0][j], w[1][j], w[2][j], w[3][j]);
        const double t = wave_sums(seg);
        if (lane < S) sc->part[lane * kWaves + wave] = t;
    }
    __syncthreads();
    constexpr int E = S * kWaves, EL = (E + kWave - 1) / kWave;           // sums, sums a lane
    static_assert(EL <= 2, "");
    const double e0 = lane * EL < E ? sc->part[lane * EL] : 0.0, e1 = EL == 2 ? sc->part[lane * EL + EL - 1] : 0.0;
    const double mine = e0 + e1, cum = wave_scan_dpp(mine);
    const double W = readlane_f64(cum, 63), target = u * W;
    if (!(W > 0.0)) return -1;                               // uniform
    const u64 live = ballot(mine > 0.0), hit = live & ballot(cum > target);
    const int l = hit ? __builtin_ctzll(hit) : live ? 63 - __builtin_clzll(live) : 0;       // (rounding at the very top: the last with weight)
    double start = readlane_f64(cum, (l - 1) & 63);
    if (l == 0) start = 0.0;
    int at = l * EL;
    if (EL == 2) {
        const double p0 = readlane_f64(e0, l), p1 = readlane_f64(e1, l);
        if (!(p0 > 0.0 && start + p0 > target) && p1 > 0.0) { start += p0; ++at; }
    }
    const int js = uniform(at / kWaves);
    if (wave == uniform(at % kWaves)) {
        // (the segment is the same in every lane)
        const float w4[4] = { w[0][js], w[1][js], w[2][js], w[3][js] };
        const double own = four(w4[0], w4[1], w4[2], w4[3]);
        const double inc = wave_scan_dpp(own);               // inclusive, in lane order
        const u64 some = ballot(own > 0.0), over = some & ballot(start + inc > target);
        const int ol = over ? __builtin_ctzll(over) : some ? 63 - __builtin_clzll(some) : 0;
        if (lane == ol) {
            double c = start + (inc - own);
            int y = -1, ylast = -1;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                c += (double)w4[e];
                if (w4[e] > 0.0f) ylast = tok_index(js, e);
                if (y < 0 && w4[e] > 0.0f && c > target) y = tok_index(js, e);
            }
            sc->y = y >= 0 ? y : ylast;
        }
    }
    __syncthreads();
    return sc->y;
}

// The walk's rows.  Both rows of the node being decided stay in registers, S segments of 4 tokens a thread: the draft row D as
// unnormalised weights exp(logit/T - max) (what is left of D after the children rejected so far is D * scale_d), the target
// row R as weights of the sum `mass`.  A thread's tokens are its own: nobody else reads them, except the two values at the
// next child's token, which their owner publishes.  LDS holds the sequence's tree links as 16-bit values (tokens < 32768,
// nodes < 2048; -1 = none) and the scratch of the reductions.
//
// A rejection is one sweep over registers: R <- max(R - D * (mass * scale_d), 0) (R stays within [0, 1], so the clamp of the fma
// does for the maximum) and the new mass, and one reduction with one barrier.  What is left of D is summed again only by the
// wave that held the rejected token: the others' shares stand.  With D in LDS the sweep waited for 16 LDS reads one after the
// other (each behind the bounds check of its segment) and every wave summed D again: 2.0 us a rejection at 32000 tokens,
// 1.4 with both in registers; a node's rows and first rejection 7.8 -> 6.4.  What bounds a rejection: the instructions between two
// barriers, 128 of them the sweep, and the reads behind the barrier.  So the partial sums are read all at once, the next child's
// links and token are on their way during the sweep, of D's sums only the one over the removed token's place in a thread's four is made again,
// and the two quotients that the next child needs are one division in two lanes.  What a node's decision reads from memory first goes by vector
// loads (by scalar ones a walk of two nodes without a rejection took 1 us longer), and segments that are whole for every V of the form
// are loaded without bounds.  Calls with 512 rows of 32000 tokens and 8, 1 and 3 rejections 50.4, 36.5, 38.3 -> 47.2, 34.5, 36.4 us (statistics pass 21.6),
// eight sequences, up to 23 rejections in one, 96 -> 91; 64 rows 38.1 -> 34.1; same results, bit for bit.
// (Tried beside it: workgroups that read the first nodes' rows into the walk's L2, 0.5 to 2 us of those calls and 4 us more where a walk is short.)
// S: 2, 8 or 16 by the size of the vocabulary, so that short rows don't pay for segments they have not (1000 tokens: walk 8.6 -> 4.6 us).
// The draft row's loads are issued first, so that its weights are made while the target row's are still out.
// (R's sum shrinks with every rejection; below kSmallMass the weights are brought back to a sum of 1, as they are
// where mass * scale_d would leave the range.)
//
// Rows that are no distribution (all -inf, NaN, +inf) end as they would with a normalised R: under such a target row no
// child is accepted and no last token comes out; after such a draft row the scan ends with the first child and the
// last token comes from the target row.  In both, the sweep finds no mass left, which is where they are told from R == D.
constexpr float kSmallMass = 9.5367431640625e-7f;     // 2^-20: weights of 1e-32 of the sum are still normal numbers
typedef float floatx4 __attribute__((ext_vector_type(4)));
struct WalkShared {
    DrawScratch draw;
    alignas(16) float2 part[2][kWaves];       // per wave, by parity of the rejection: mass left in R, weight in D
    float2 next[2];               // R and D at the next child's token
};
static constexpr size_t walk_lds_bytes(int widest) { return 3 * (size_t)((widest + 7) & ~7) * sizeof(short); }

template <bool VEC, typename T, int S>
__global__ __launch_bounds__(kBlock) void verify_walk_kernel(
    const T* __restrict__ draft_logits, const T* __restrict__ target_logits, int V,
    SeqArgs sa, dyspec_tree tree, uint64_t seed, int emit_bonus,
    const float* __restrict__ row_stats, float* __restrict__ accept_ratio,
    int* __restrict__ accepted_nodes, int* __restrict__ n_accepted,
    int* __restrict__ final_token, float* __restrict__ min_margin)
{
    __shared__ WalkShared sh;
    extern __shared__ __attribute__((aligned(16))) unsigned char dyn[];
    const int tid = threadIdx.x;
    const int seq = blockIdx.x;
    const int base = sa.node_off[seq];
    const int N = sa.node_off[seq + 1] - base;
    const bool greedy = sa.temp_t[seq] == 0.0f;                  // target row = all mass on stats.w
    const float inv_td = 1.0f / sa.temp_d[seq], inv_tt = greedy ? 1.0f : 1.0f / sa.temp_t[seq];
    const int Npad = (N + 7) & ~7;
    short* const l_token = reinterpret_cast<short*>(dyn);
    short* const l_child = l_token + Npad;
    short* const l_next = l_child + Npad;
    for (int i = tid; i < N; i += kBlock) {
        const int tk = tree.token[base + i], fc = tree.first_child[base + i], ns = tree.next_sibling[base + i];
        l_token[i] = (short)((tk >= 0 && tk < V) ? tk : -1);     // anything else is no token: ratio 0
        l_child[i] = (short)((fc >= 0 && fc < N) ? fc : -1);
        l_next[i] = (short)((ns >= 0 && ns < N) ? ns : -1);
    }
    __syncthreads();

    auto ratio_of = [](float d, float r) { return (d > 0.0f) ? r / d : (r > 0.0f ? INFINITY : 0.0f); };

    int cur = 0, na = 0, fin = -1;
    uint2 pk = root_key((uint32_t)seq);
    float margin = INFINITY;
    for (int steps = 0; steps < N; ++steps) {            // a path has fewer than N edges
        int c = l_child[cur];
        const bool leaf = c < 0;
        int next = -1;
        uint2 pk_next = pk;
        bool rows_loaded = false;
        RowVec<S> R[4], D[4];
        // the node's statistics: one 16-byte load, on its way together with the first child's logits (all with an address in vector
        // registers; and what is read from LDS at one is waited for where it is used)
        int lane_zero = 0;
        asm volatile("" : "+v"(lane_zero));
        const float4 st = *reinterpret_cast<const float4*>(row_stats + 4 * (size_t)(base + cur) + lane_zero);
        float scale_d = 0.0f, mass = 0.0f;                // what is left of D = D * scale_d; R's sum
        // R <- the target row's weights; with want_draft, D <- the draft row's
        auto load_rows = [&](bool want_draft) __attribute__((always_inline)) {
            float X[S][4], Y[S][4];
            int v_here = V, own = 4 * tid;
            asm volatile("" : "+s"(v_here), "+v"(own));   // (what follows from them for each segment isn't kept in registers from node to node)
            constexpr int FULL = S == kMaxSeg ? 8 : S == 8 ? 2 : 0;         // (see with_segments)
            if (want_draft) load_row<VEC, T, FULL>(draft_logits + (size_t)(base + cur) * V, v_here, X, own);
            if (!greedy) load_row<VEC, T, FULL>(target_logits + (size_t)(base + cur) * V, v_here, Y, own);
            if (want_draft) {                             // (the loads of both rows are in flight together)
#pragma unroll
                for (int j = 0; j < S; ++j)
#pragma unroll
                    for (int e = 0; e < 4; ++e) D[e][j] = exp_fast(X[j][e] * inv_td - st.x);
                scale_d = 1.0f / st.y;
            }
            mass = greedy ? 1.0f : st.w;
            if (greedy) {
                const int mine = (int)st.w - 4 * tid;
#pragma unroll
                for (int j = 0; j < S; ++j)
#pragma unroll
                    for (int e = 0; e < 4; ++e) R[e][j] = mine - j * kSeg == e ? 1.0f : 0.0f;
            } else {
#pragma unroll
                for (int j = 0; j < S; ++j)
#pragma unroll
                    for (int e = 0; e < 4; ++e) R[e][j] = exp_fast(Y[j][e] * inv_tt - st.z);
            }
        };
        if (!leaf) {
            // ---- first child: two logits and the row statistics decide
            float dy = 0.0f;                              // D at the tested child's token
            uint2 keys;                                   // of 64 children, one per lane: path key, uniform of the acceptance
            float us;
            {
                const int y = l_token[c];
                float d = 0.0f, r = 0.0f, xd = 0.0f, xt = 0.0f;
                if (y >= 0) {
                    xd = logit_to_float((draft_logits + (size_t)(base + cur) * V)[y + lane_zero]);
                    if (!greedy) xt = logit_to_float((target_logits + (size_t)(base + cur) * V)[y + lane_zero]);
                }
                keys = child_key(seed, pk, (uint32_t)(tid & (kWave - 1)));          // (while the loads are out)
                us = u01(seed, keys, 0u, KIND_ACCEPT);
                if (y >= 0) {
                    dy = exp_fast(xd * inv_td - st.x);
                    d = dy / st.y;
                    r = greedy ? ((float)y == st.w ? 1.0f : 0.0f) : exp_fast(xt * inv_tt - st.z) / st.w;
                }
                const float ratio = uniform(ratio_of(d, r));
                const uint2 pk_n = make_uint2((uint32_t)__builtin_amdgcn_readlane((int)keys.x, 0), (uint32_t)__builtin_amdgcn_readlane((int)keys.y, 0));
                const float u = readlane_f32(us, 0);
                margin = fminf(margin, fabsf(u - ratio));
                if (tid == 0) accept_ratio[base + c] = ratio;
                if (u < ratio) { next = c; pk_next = pk_n; }
            }
            // ---- rejected: bring the rows in and update the residuals child by child
            if (next < 0) {
                load_rows(true);
                rows_loaded = true;
                // R and D at token y (none: zeros), by the thread that owns it
                auto publish = [&](int y, float2* place) __attribute__((always_inline)) {
                    const int js = uniform(max(y, 0) / kSeg), e = y & 3;
                    if (((max(y, 0) % kSeg) >> 2) == tid) {
                        const float r0 = R[0][js], r1 = R[1][js], r2 = R[2][js], r3 = R[3][js];
                        const float d0 = D[0][js], d1 = D[1][js], d2 = D[2][js], d3 = D[3][js];
                        *place = y < 0 ? make_float2(0.0f, 0.0f)
                                       : make_float2(e == 0 ? r0 : e == 1 ? r1 : e == 2 ? r2 : r3, e == 0 ? d0 : e == 1 ? d1 : e == 2 ? d2 : d3);
                    }
                };
                // D's sums: w[e] of a thread's tokens of place e, left_w of the wave's
                float w[4], left_w = 0.0f;
                const auto sum_place = [&](int e) __attribute__((always_inline)) {
                    float s = 0.0f;
#pragma unroll
                    for (int j = 0; j < S; ++j) s += D[e][j];
                    w[e] = s;
                };
                int y = l_token[c], after = l_next[c], y_next = after >= 0 ? l_token[after] : -1;
                float2 rd = make_float2(0.0f, 0.0f);      // R and D at the tested child's token,
                float share = 0.0f;                       // and R's part of its sum
                for (int rank = 0; c >= 0 && rank < N; ++rank) {
                    const int par = rank & 1;
                    const int after_2 = l_next[max(after, 0) + lane_zero];
                    if (rank > 0 && rank % kWave == 0) {
                        keys = child_key(seed, pk, rank + (tid & (kWave - 1)));
                        us = u01(seed, keys, 0u, KIND_ACCEPT);
                    }
                    if (rank > 0) {
                        // ratio seen by this child after its earlier siblings were rejected
                        dy = rd.y;
                        const float ratio = uniform(ratio_of(rd.y * scale_d, share));
                        const uint2 pk_n = make_uint2((uint32_t)__builtin_amdgcn_readlane((int)keys.x, rank & 63), (uint32_t)__builtin_amdgcn_readlane((int)keys.y, rank & 63));
                        const float u = readlane_f32(us, rank & 63);
                        margin = fminf(margin, fabsf(u - ratio));
                        if (tid == 0) accept_ratio[base + c] = ratio;
                        if (u < ratio) { next = c; pk_next = pk_n; break; }
                    }
                    // reject child c: R <- norm(max(R-D,0)) with D as it stands, then y leaves D.  (The owner of
                    // y does so for y first: what is left of D is summed without y, where a sum with y less
                    // its weight would lose what y outweighs.)
                    float f = scale_d * mass;
                    if (f == INFINITY) {                      // what is left of D weighs next to nothing: R's weights come down to shares first
                        const float down = 1.0f / mass;
#pragma unroll
                        for (int j = 0; j < S; ++j)
#pragma unroll
                            for (int e = 0; e < 4; ++e) R[e][j] *= down;
                        mass = 1.0f;
                        f = scale_d;                          // at most 2^126, as D's weights are normal numbers
                    }
                    if (y >= 0 && ((y % kSeg) >> 2) == tid) {
                        const int js = uniform(y / kSeg), e = y & 3;
#pragma unroll
                        for (int k = 0; k < 4; ++k) {
                            const float r = R[k][js], d = D[k][js];
                            R[k][js] = e == k ? __builtin_amdgcn_fmed3f(fmaf(-f, d, r), 0.0f, 1.0f) : r;
                            D[k][js] = e == k ? 0.0f : d;
                        }
                    }
                    float m[4] = { 0.0f, 0.0f, 0.0f, 0.0f };
#pragma unroll
                    for (int j = 0; j < S; ++j)
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            R[e][j] = __builtin_amdgcn_fmed3f(fmaf(-f, D[e][j], R[e][j]), 0.0f, 1.0f);
                            m[e] += R[e][j];
                        }
                    publish(y_next, &sh.next[par]);
                    const int after_3 = l_token[max(after_2, 0)];
                    if (rank == 0 || (y >= 0 && (y % kSeg) / (4 * kWave) == uniform(tid / kWave))) {      // (the same in every lane)
                        const int e = y & 3;
                        if (rank == 0) {
#pragma unroll
                            for (int k = 0; k < 4; ++k) sum_place(k);
                        } else if (e == 0) sum_place(0);
                        else if (e == 1) sum_place(1);
                        else if (e == 2) sum_place(2);
                        else sum_place(3);
                        left_w = wave_sum_f32_dpp((w[0] + w[1]) + (w[2] + w[3]));
                    }
                    const float mw = wave_sum_f32_dpp((m[0] + m[1]) + (m[2] + m[3])), ww = left_w;
                    if ((tid & (kWave - 1)) == 0) sh.part[par][tid / kWave] = make_float2(mw, ww);
                    __syncthreads();
                    // (all reads on their way together)
                    floatx4 parts[kWaves / 2];
#pragma unroll
                    for (int k = 0; k < kWaves / 2; ++k) parts[k] = *reinterpret_cast<const floatx4*>(&sh.part[par][2 * k]);
                    rd = sh.next[par];
                    static_assert(kWaves == 8, "");
                    asm volatile("" : "+v"(parts[0]), "+v"(parts[1]), "+v"(parts[2]), "+v"(parts[3]), "+v"(rd.x), "+v"(rd.y));
                    float2 sum = make_float2(parts[0].x, parts[0].y);
#pragma unroll
                    for (int k = 1; k < kWaves; ++k) { sum.x += parts[k / 2][2 * (k % 2)]; sum.y += parts[k / 2][2 * (k % 2) + 1]; }
                    sum.x = uniform(sum.x); sum.y = uniform(sum.y);
                    rd.x = uniform(rd.x); rd.y = uniform(rd.y);
                    // a draft row that is no distribution (no weight at all, or NaN among it) empties at once
                    const bool no_draft = !(sum.y + dy > 0.0f);
                    if (sum.x >= kSmallMass) {
                        mass = sum.x;
                    } else {
                        if (!(sum.x > 0.0f) && no_draft) {
                            rows_loaded = false;              // the last token comes from the target row as it is
                        } else if (!(sum.x > 0.0f) && !greedy && !(mass > 0.0f && fabsf(st.z) < INFINITY)) {
                            // a target row that is no distribution: every child is rejected, no last token
                        } else if (sum.x > 0.0f) {
                            // R's weights are scaled up again long before the smallest of them are lost
                            // (in two steps: the sum's reciprocal alone may be past the range)
                            const float lift = sum.x < 0x1p-100f ? 0x1p100f : 1.0f, up = 1.0f / (sum.x * lift);
                            mass = 1.0f;
#pragma unroll
                            for (int j = 0; j < S; ++j)
#pragma unroll
                                for (int e = 0; e < 4; ++e) R[e][j] = fminf(R[e][j] * lift * up, 1.0f);
                            rd.x = uniform(fminf(rd.x * lift * up, 1.0f));
                        } else {
                            // R == D to rounding (hardly any reject can reach here): R stays, that is, becomes D as
                            // it stood; a greedy target's R is its one token, whatever its mass
                            mass = greedy ? 1.0f : sum.y + dy;
                            // (one token's value is not in D: that of the greedy row, or the one just removed)
                            const int one = greedy ? (int)st.w : y, mine = one - 4 * tid;
                            const float value = greedy ? 1.0f : dy;
#pragma unroll
                            for (int j = 0; j < S; ++j)
#pragma unroll
                                for (int e = 0; e < 4; ++e) R[e][j] = mine - j * kSeg == e ? value : greedy ? 0.0f : D[e][j];
                            rd.x = uniform(y_next < 0 ? 0.0f : y_next == one ? value : greedy ? 0.0f : rd.y);
                        }
                    }
                    const float left = sum.y;                 // weight left in D
                    c = after;
                    y = y_next;
                    after = c >= 0 ? uniform(after_2) : -1;
                    y_next = after >= 0 ? uniform(after_3) : -1;
                    if (!(left > 0.0f) || no_draft) {         // D is empty: later children are not tried
                        if (tid == 0)
                            for (int k = 0, cc = c; cc >= 0 && k < N; ++k, cc = l_next[cc])
                                accept_ratio[base + cc] = -1.0f;
                        break;
                    }
                    // D <- norm(D), kept as a factor; the next child's R as a share: two lanes' quotients
                    const float q = ((tid & 1) ? 1.0f : rd.x) / ((tid & 1) ? left : mass);
                    scale_d = readlane_f32(q, 1);
                    share = readlane_f32(q, 0);
                }
            }
        }
        if (next >= 0) {
            if (tid == 0) accepted_nodes[base + na] = next;
            ++na;
            cur = next; pk = pk_next;
            __syncthreads();                                  // the scratch is free for the next node
            continue;
        }
        // ---- the walk stops at cur: emit a token from what is left of the target row
        if (leaf && !emit_bonus) { fin = -1; break; }
        if (!rows_loaded) load_rows(false);
        __syncthreads();
        const double u = (double)u01(seed, pk, 0u, KIND_RESID);
        fin = draw_from_row<S>(R, u, &sh.draw);
        break;
    }
    if (tid == 0) {
        n_accepted[seq] = na;
        final_token[seq] = fin;
        min_margin[seq] = margin;
    }
}

// f(S) for the rows' segments
template <typename F>
static hipError_t with_segments(int V, F&& f)
{
    if (V <= 2 * kSeg) return f(std::integral_constant<int, 2>{});
    if (V <= 8 * kSeg) return f(std::integral_constant<int, 8>{});
    return f(std::integral_constant<int, kMaxSeg>{});
}

// loads the walk's code (its LDS, at most 12 KB, needs no limit raised)
hipError_t prepare_verify()
{
    hipError_t e = hipSuccess;
    auto touch = [&](const void* kernel) {
        hipFuncAttributes attributes;
        if (e == hipSuccess) e = hipFuncGetAttributes(&attributes, kernel);
    };
    for (int V : { 1, 8 * kSeg, kMaxSeg * kSeg })
        (void)with_segments(V, [&](auto sc) {
            constexpr int S = decltype(sc)::value;
            touch(reinterpret_cast<const void*>(&verify_walk_kernel<true, float, S>));
            touch(reinterpret_cast<const void*>(&verify_walk_kernel<false, float, S>));
            touch(reinterpret_cast<const void*>(&verify_walk_kernel<true, __bf16, S>));
            touch(reinterpret_cast<const void*>(&verify_walk_kernel<false, __bf16, S>));
            return e;
        });
    return e;
}

template <typename T>
static hipError_t launch_verify_t(const T* draft_logits, const T* target_logits, int V,
                                  const SeqArgs& sa, const dyspec_tree& tree, uint64_t seed, int emit_bonus,
                                  float* row_stats, float* accept_ratio, int* accepted_nodes, int* n_accepted,
                                  int* final_token, float* min_margin, hipStream_t stream)
{
    const int rows = sa.node_off[sa.n_seq];
    // statistics: the streaming form reads whole 16-byte pieces where the rows are made of them, else it takes the end of a row from its last 16 bytes
    if (V < Piece<T>::N) {
        softmax_stats_kernel<T><<<rows, kBlock, 0, stream>>>(draft_logits, target_logits, V, sa, row_stats, accept_ratio);
    } else if (V % Piece<T>::N == 0) {
        if constexpr (sizeof(T) == 4)
            softmax_stats_stream_kernel<<<dim3(rows, 2), kStatThreads, 0, stream>>>(draft_logits, target_logits, V, sa, row_stats, accept_ratio);
        else
            softmax_stats_stream_pieces_kernel<T, false><<<dim3(rows, 2), kStatThreads, 0, stream>>>(draft_logits, target_logits, V, sa, row_stats, accept_ratio);
    } else {
        softmax_stats_stream_pieces_kernel<T, true><<<dim3(rows, 2), kStatThreads, 0, stream>>>(draft_logits, target_logits, V, sa, row_stats, accept_ratio);
    }
    int widest = 1;
    for (int s = 0; s < sa.n_seq; ++s) widest = max(widest, sa.node_off[s + 1] - sa.node_off[s]);
    return with_segments(V, [&](auto sc) {
        constexpr int S = decltype(sc)::value;
        auto launch = [&](auto vec) {
            verify_walk_kernel<decltype(vec)::value, T, S><<<sa.n_seq, kBlock, walk_lds_bytes(widest), stream>>>(
                draft_logits, target_logits, V, sa, tree, seed, emit_bonus, row_stats, accept_ratio, accepted_nodes, n_accepted, final_token, min_margin);
            return hipGetLastError();
        };
        return V % 4 == 0 ? launch(std::true_type{}) : launch(std::false_type{});
    });
}

hipError_t launch_verify(const void* draft_logits, const void* target_logits, bool bf16_logits, int V,
                         const SeqArgs& sa, const dyspec_tree& tree, uint64_t seed, int emit_bonus,
                         float* row_stats, float* accept_ratio, int* accepted_nodes, int* n_accepted,
                         int* final_token, float* min_margin, hipStream_t stream)
{
    if (bf16_logits)
        return launch_verify_t(static_cast<const __bf16*>(draft_logits), static_cast<const __bf16*>(target_logits), V, sa, tree,
                               seed, emit_bonus, row_stats, accept_ratio, accepted_nodes, n_accepted, final_token, min_margin, stream);
    return launch_verify_t(static_cast<const float*>(draft_logits), static_cast<const float*>(target_logits), V, sa, tree,
                           seed, emit_bonus, row_stats, accept_ratio, accepted_nodes, n_accepted, final_token, min_margin, stream);
}

}  // namespace dyspec

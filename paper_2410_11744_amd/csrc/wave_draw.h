// Draws without replacement from one draft row by a single wave.
//
// Vocabulary order is kept at three levels: kGroups groups of kGroupTokens tokens, one per lane of
// the wave; kGroupLeaves leaves of kLeafTokens tokens per group; the tokens.  A draw is an inverse
// CDF through the three levels: the wave compares its inclusive scan of the group totals with u * W, scans
// the picked group's leaves, turns the picked leaf's logits into weights and scans those.  Nothing
// but the wave's own instructions lies between two draws: no barrier, no trip to global memory.
// Bound by the number of instructions, about 160 a draw: a wave alone issues one in eight cycles, dependent or not
// (0.57 us a draw in the threshold builder; a workgroup of eight waves with two barriers a draw took 1.5).
//
// The sums are never updated by subtraction: the drawn token's leaf, its group and the scan of the
// groups are each made of what is left (sum before + sum after the gap), so they are zero exactly
// when nothing is left and equal a single remaining weight exactly, however much was drawn before.
// The sums before and after come out of one scan: a second copy of the sixteen leaves (32
// tokens) lies in the lanes beside them in reverse order.
#pragma once
#include "draft_row.h"
#include "lane_ops.h"

namespace dyspec {

typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int kLeafTokens = 32;
constexpr int kGroupTokens = 512;
constexpr int kGroupLeaves = kGroupTokens / kLeafTokens;
constexpr int kGroups = DYSPEC_MAX_VOCAB / kGroupTokens;
static_assert(kGroups == kWave && kGroupLeaves == 16 && kLeafTokens == 32, "one group per lane, one leaf table row per 16 lanes");

// LDS of a row: the leaf sums of whole groups, then the logits of whole leaves (-inf: past the end, or drawn)
__host__ __device__ constexpr int row_leaves(int V) { return (V + kGroupTokens - 1) / kGroupTokens * kGroupLeaves; }
__host__ __device__ constexpr int row_logits(int V) { return (V + kLeafTokens - 1) / kLeafTokens * kLeafTokens; }
__host__ __device__ constexpr size_t row_lds_bytes(int V) { return (size_t)row_leaves(V) * sizeof(double) + (size_t)row_logits(V) * sizeof(float); }

// Inclusive scan over each row of 16 lanes, over each half wave.
__device__ __forceinline__ double scan16_dpp(double x)
{
    x += dpp_or_zero<0x111>(x);
    x += dpp_or_zero<0x112>(x);
    x += dpp_or_zero<0x114>(x);
    x += dpp_or_zero<0x118>(x);
    return x;
}
__device__ __forceinline__ double scan32_dpp(double x)
{
    x = scan16_dpp(x);
    x += dpp_or_zero<kDppBcast15, 0xa>(x);
    return x;
}
// the lane's value at position i of a scan, 0 for i = -1
__device__ __forceinline__ double scan_at(double x, int i) { const double v = readlane_f64(x, i & 63); return i < 0 ? 0.0 : v; }

// A row in sweeps of 4 tokens per thread of NT (-inf: past the end).
template <int NT, bool VEC, int SW>
__device__ __forceinline__ void load_row_sweeps(const float* __restrict__ row, int V, float (&x)[SW][4])
{
    const int tid = threadIdx.x;
#pragma unroll
    for (int s = 0; s < SW; ++s) {
        const int i0 = 4 * (s * NT + tid);
        if constexpr (VEC) {
            const float4 v = i0 < V ? *reinterpret_cast<const float4*>(row + i0) : make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
            x[s][0] = v.x; x[s][1] = v.y; x[s][2] = v.z; x[s][3] = v.w;
        } else if (4 * NT * (s + 1) <= V) {                     // (uniform; rows that begin at any value)
            typedef float four __attribute__((ext_vector_type(4), aligned(4)));
            const four v = *reinterpret_cast<const four*>(row + i0);
            x[s][0] = v.x; x[s][1] = v.y; x[s][2] = v.z; x[s][3] = v.w;
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) x[s][e] = i0 + e < V ? row[i0 + e] : -INFINITY;
        }
    }
}

// Brings a row into LDS with NT threads: logits, leaf sums; the row maximum over T is returned to
// every thread.  `fred`: NT / 64 floats.  Ends with a barrier.
template <int NT, bool VEC>
__device__ __forceinline__ double load_row_lds(const float* __restrict__ row, int V, double inv_temp, lds_t<double>* leaf, lds_t<float>* logits, float* fred)
{
    constexpr int SW = DYSPEC_MAX_VOCAB / (4 * NT);         // sweeps of 4 tokens per thread
    const int tid = threadIdx.x, lane = tid & 63;
    const int Vl = row_logits(V), Vg = row_leaves(V) * kLeafTokens;
    float x[SW][4];
    load_row_sweeps<NT, VEC>(row, V, x);
    float mx = -INFINITY;
#pragma unroll
    for (int s = 0; s < SW; ++s) {
        mx = fmaxf(mx, fmaxf(fmaxf(x[s][0], x[s][1]), fmaxf(x[s][2], x[s][3])));
        const int i0 = 4 * (s * NT + tid);
        if (i0 < Vl) *(lds_t<floatx4>*)(logits + i0) = floatx4{ x[s][0], x[s][1], x[s][2], x[s][3] };
    }
    mx = wave_max(mx);
    if (lane == 0) fred[tid >> 6] = mx;
    __syncthreads();
    mx = fred[lane & (NT / 64 - 1)];
    mx = wave_max(mx);
    const double m = (double)mx * inv_temp;
#pragma unroll
    for (int s = 0; s < SW; ++s) {
        const int i0 = 4 * (s * NT + tid);
        if (s * NT * 4 >= V) break;                         // uniform
        double z[4], w4[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) z[e] = fma((double)x[s][e], inv_temp, -m);
        exp_nonpos_xn<4>(z, w4);
        double t = (w4[0] + w4[1]) + (w4[2] + w4[3]);       // tokens past the end: exp(-inf) = 0
        t += dpp_or_zero<kDppXor1>(t);
        t += dpp_or_zero<kDppXor2>(t);
        t += dpp_or_zero<kDppHalfMirror>(t);                // the eight lanes of a leaf
        if ((lane & 7) == 0 && i0 < Vg) leaf[i0 / kLeafTokens] = t;     // (a sweep is a multiple of a group: all are written)
    }
    __syncthreads();
    return m;
}

// What the drawing wave keeps in registers of a row in LDS.
struct WaveRow {
    lds_t<double>* leaf;
    lds_t<float>* logits;
    double m, inv_temp;
    double tot, cum;            // lane l: total of group l, inclusive scan over the groups
};

__device__ __forceinline__ void open_wave_row(WaveRow& r, int V)
{
    const int lane = threadIdx.x & 63;
    r.tot = 0.0;
    if (lane < row_leaves(V) / kGroupLeaves) {
#pragma unroll
        for (int k = 0; k < kGroupLeaves; ++k) r.tot += r.leaf[lane * kGroupLeaves + ((k + lane) & (kGroupLeaves - 1))];
    }
    r.cum = wave_scan_dpp(r.tot);
}

struct Drawn { int y; double wy, W; };

// First lane of `hit`, or the last one of `live` (not empty) where rounding left no hit.
__device__ __forceinline__ int pick_lane(u64 hit, u64 live)
{
    return hit ? __builtin_ctzll(hit) : 63 - __builtin_clzll(live);
}

// One draw with uniform u of a row with weight left; the token leaves the row.  Every lane gets the same result.
// A crossing is looked for where sums are compared with the target alone: of non-negative values in one order, the first sum above it
// belongs to a positive one.  Sums of one scan are made in different orders, though, and may miss the target or cross it at a zero
// by a rounding: if there is no crossing at the last level, or at a zero, nothing has been changed, the result is false,
// and the draw is made again with EXACT, which asks for positive values at each level and takes the last one if there is no crossing
// (what was picked otherwise is what EXACT picks).  A 383-draw row: 276 -> 268 us a call; with a branch at each level instead of
// one at the end 286.
// Nothing past the row is read.  Finite sums: for u <= 1 - 2^-24 the target lies so far below the row's last sums (their
// roundings are some 2^-50 of them) that the last group's crossing is found among its leaves that have logits.  An infinite sum crosses
// nothing and belongs to EXACT: `none` and the target are then NaN, every sum counts as past it, and the first token is refused.
template <bool EXACT>
__device__ __forceinline__ bool draw_wave_row(WaveRow& r, double u, double W, Drawn* d)
{
    const int lane = threadIdx.x & 63;
    const double none = EXACT ? 0.0 : W * 0.0;
    const double target = EXACT ? u * W : fma(u, W, none);
    const auto past = [=](double sum) __attribute__((always_inline)) { return EXACT ? sum > target : !(sum <= target); };
    const auto pick = [](u64 hit, int last, auto&& positive) __attribute__((always_inline)) {
        if constexpr (EXACT) {
            const u64 live = positive();
            return pick_lane(live & hit, live);
        } else {
            return (int)__builtin_ctzll(hit | (1ull << last));
        }
    };
    const int g = pick(ballot(past(r.cum)), 63, [&]() { return ballot(r.tot > 0.0); });
    // lanes 0..15 (and 32..47) hold the group's leaves, lanes 16..31 (48..63) the same in reverse order
    const double b = r.leaf[g * kGroupLeaves + ((lane & 15) ^ ((lane & 16) ? 15 : 0))];
    const double below_g = scan_at(r.cum, g - 1);
    const double cb = scan16_dpp(b);
    const double eb = dpp_or_zero<0x111>(cb);               // what lies before each leaf (row_shr:1; 0 at the start of a row)
    const int l = pick(ballot(past(below_g + cb)) & 0xffffull, 15, [&]() { return ballot(b > 0.0) & 0xffffull; });
    // lanes 0..31: the leaf's tokens, lanes 32..63: the same in reverse order
    const int leaf0 = (g * kGroupLeaves + l) * kLeafTokens;
    const float x = r.logits[leaf0 + ((lane & 31) ^ ((lane & 32) ? 31 : 0))];
    const double leaves_before = readlane_f64(eb, l), leaves_after = readlane_f64(eb, 31 - l);
    const double below_l = below_g + leaves_before;
    const double rest = wave_scan_dpp(lane == g ? 0.0 : r.tot);        // scan of the groups without this one
    double z[1] = { fma((double)x, r.inv_temp, -r.m) }, w[1];
    exp_nonpos_xn<1>(z, w);
    const double cw = scan32_dpp(w[0]);
    const u64 over = ballot(past(below_l + cw)) & 0xffffffffull;
    const int e = pick(over, 31, [&]() { return ballot(w[0] > 0.0) & 0xffffffffull; });
    d->y = leaf0 + e;
    d->wy = readlane_f64(w[0], e);
    d->W = W;
    if (!EXACT && (over == 0ull || !(d->wy > none))) return false;
    const double left = scan_at(cw, e - 1) + (e < 31 ? readlane_f64(cw, 62 - e) : 0.0);
    const double t = (leaves_before + left) + leaves_after;
    r.cum = rest + (lane >= g ? t : 0.0);
    if (lane == g) r.tot = t;
    if (lane == e) r.logits[leaf0 + e] = -INFINITY;
    if (lane == 0) r.leaf[g * kGroupLeaves + l] = left;
    return true;
}
// The same; false (nothing changed) when the row is empty.  u <= 1 - 2^-24.
__device__ __forceinline__ bool draw_wave_row(WaveRow& r, double u, Drawn* d)
{
    const double W = readlane_f64(r.cum, 63);
    if (!(W > 0.0)) return false;
    if (__builtin_expect(!draw_wave_row<false>(r, u, W, d), 0)) draw_wave_row<true>(r, u, W, d);
    return true;
}

}  // namespace dyspec

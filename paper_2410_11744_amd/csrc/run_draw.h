// Draws without replacement from a draft row by its runs of kRun tokens: the sums and comparisons of one draw, in one place, so that a
// draw has the same bits whoever makes it (a wave of the tree's workgroup, the row in memory, or a helper, the row in LDS).  Which of
// the two it is depends on the clock; two children with equal logits open slots that are equal but for roundings.
//
// Lane l has what is left of runs 4 l .. 4 l + 3.  A draw is an inverse CDF over the lanes (scan), the lane's four runs, the run's lanes of two
// tokens each (scan), the two tokens.  What is left of a run is summed again without the drawn token, never subtracted.
//
// Bound, in a helper, by one wave's instructions like draw_wave_row, whose sums its draws were made by before: 0.67 us a draw where that takes
// 0.63 (two exponentials a lane, the run's sum and the scan over the lanes one after the other; a chain of 512 rows 371 -> 391 us, 512 rows of
// independent normal logits 332, 181, 201 -> 350, 181, 204).
#pragma once
#include "wave_draw.h"
#include "row_workspace.h"

namespace dyspec {

static_assert(kSums == 4 * kWave && kRun == 2 * kWave, "four runs to a lane, two tokens of a run to a lane");

// What is left of the lane's four runs, the inclusive scan over the lanes, all that is left.
struct RunSums { double four, cum, W; };
__device__ __forceinline__ RunSums sum_runs(const double (&tot)[4])
{
    RunSums s;
    const double t01 = tot[0] + tot[1];
    s.four = t01 + (tot[2] + tot[3]);
    s.cum = wave_scan_dpp(s.four);
    s.W = readlane_f64(s.cum, 63);
    return s;
}
struct PickedRun {
    int lane, k;            // run 4 lane + k
    double target, start;   // u W, the weight before the run
};
// The run of the crossing.  s.W > 0.
__device__ __forceinline__ PickedRun pick_run(const double (&tot)[4], const RunSums& s, double u)
{
    // the lane of the crossing, then one of its four totals (every lane walks its own)
    PickedRun p;
    p.target = u * s.W;
    p.lane = pick_lane(ballot(s.four > 0.0) & ballot(s.cum > p.target), ballot(s.four > 0.0));
    const double start = scan_at(s.cum, p.lane - 1);
    double run_start = start;
    int k = -1;
    {
        double run = start;
        int last = 0;
        double last_start = start;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const double after = run + tot[e];
            if (tot[e] > 0.0) { last = e; last_start = run; }
            if (k < 0 && tot[e] > 0.0 && after > p.target) { k = e; run_start = run; }
            run = after;
        }
        if (k < 0) { k = last; run_start = last_start; }            // rounding at the top
    }
    p.k = __builtin_amdgcn_readlane(k, p.lane);
    p.start = readlane_f64(run_start, p.lane);
    return p;
}

// Lane l's two tokens of a run, the scan over the lanes, the lanes with weight.
struct TokenSums { double mine, inc; u64 live; };
__device__ __forceinline__ TokenSums sum_tokens(const double (&w)[2])
{
    TokenSums s;
    s.mine = w[0] + w[1];
    s.inc = wave_scan_dpp(s.mine);
    s.live = ballot(s.mine > 0.0);
    return s;
}
struct PickedToken {
    int lane, second;       // token 2 lane + second of the run
    double wy;              // its weight
};
// The token of the crossing.  s.live is not empty.
__device__ __forceinline__ PickedToken pick_token(const double (&w)[2], const TokenSums& s, const PickedRun& p)
{
    PickedToken t;
    t.lane = pick_lane(s.live & ballot(p.start + s.inc > p.target), s.live);
    const double mid = p.start + scan_at(s.inc, t.lane - 1) + w[0];     // (of interest in the picked lane)
    const int second = 1 - (int)((w[0] > 0.0) & ((mid > p.target) | !(w[1] > 0.0)));
    t.second = __builtin_amdgcn_readlane(second, t.lane);
    t.wy = readlane_f64(t.second ? w[1] : w[0], t.lane);
    return t;
}
// What is left of the run without the picked token.
__device__ __forceinline__ double run_left(const double (&w)[2], const TokenSums& s, const PickedToken& t)
{
    const int lane = threadIdx.x & 63;
    return wave_sum_dpp(lane == t.lane ? (t.second ? w[0] : w[1]) : s.mine);
}

// ---- A row in LDS: the logits of whole runs (-inf: past the end, or drawn); the runs' totals pass through LDS once.
__host__ __device__ constexpr int row_runs(int V) { return (V + kRun - 1) / kRun; }
__host__ __device__ constexpr size_t run_row_lds_bytes(int V) { return (size_t)row_runs(V) * kRun * sizeof(float); }

// Total of a run, four tokens' sum in each lane of half a wave; in the half's last lane.  (In the order in which row_sums and the exchange
// behind it add: mirrored lanes first.)
__device__ __forceinline__ double run_total(double t)
{
    t += dpp_or_zero<kDppMirror>(t);
    t += dpp_or_zero<kDppHalfMirror>(t);
    t += dpp_or_zero<kDppXor2>(t);
    t += dpp_or_zero<kDppXor1>(t);
    t += dpp_or_zero<kDppBcast15, 0xa>(t);
    return t;
}

// Brings a row into LDS with NT threads: logits, run totals (kSums of them); the row maximum over T is returned to every
// thread.  `fred`: NT / 64 floats.  Ends with a barrier.
template <int NT, bool VEC>
__device__ __forceinline__ double load_run_row(const float* __restrict__ row, int V, double inv_temp, lds_t<double>* totals, lds_t<float>* logits, float* fred)
{
    constexpr int SW = DYSPEC_MAX_VOCAB / (4 * NT);         // sweeps of 4 tokens per thread
    const int tid = threadIdx.x, lane = tid & 63;
    const int Vr = row_runs(V) * kRun;
    float x[SW][4];
    load_row_sweeps<NT, VEC>(row, V, x);
    float mx = -INFINITY;
#pragma unroll
    for (int s = 0; s < SW; ++s) {
        mx = fmaxf(mx, fmaxf(fmaxf(x[s][0], x[s][1]), fmaxf(x[s][2], x[s][3])));
        const int i0 = 4 * (s * NT + tid);
        if (i0 < Vr) *(lds_t<floatx4>*)(logits + i0) = floatx4{ x[s][0], x[s][1], x[s][2], x[s][3] };
    }
    mx = wave_max(mx);
    if (lane == 0) fred[tid >> 6] = mx;
    __syncthreads();
    mx = fred[lane & (NT / 64 - 1)];
    mx = wave_max(mx);
    const double m = (double)mx * inv_temp;
#pragma unroll
    for (int s = 0; s < SW; ++s) {
        double t = 0.0;
        if (s * NT * 4 < V) {                               // uniform
            double z[4], w4[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) z[e] = fma((double)x[s][e], inv_temp, -m);
            exp_nonpos_xn<4>(z, w4);
            t = run_total((w4[0] + w4[1]) + (w4[2] + w4[3]));       // tokens past the end: exp(-inf) = 0
        }
        if ((lane & 31) == 31) totals[(s * NT + tid) / (kRun / 4)] = t;
    }
    __syncthreads();
    return m;
}

// wave_scan_dpp for scans made again and again: what rows 0 and 2 (0 and 1) of lanes are to add stays 0 from scan to scan, as the moves
// write the other rows only.
struct ScanZeros { int hi15, lo15, hi31, lo31; };
__device__ __forceinline__ double wave_scan_again(double x, ScanZeros& z)
{
    x = scan16_dpp(x);
    z.hi15 = __builtin_amdgcn_update_dpp(z.hi15, __double2hiint(x), kDppBcast15, 0xa, 0xf, false);
    z.lo15 = __builtin_amdgcn_update_dpp(z.lo15, __double2loint(x), kDppBcast15, 0xa, 0xf, false);
    x += __hiloint2double(z.hi15, z.lo15);
    z.hi31 = __builtin_amdgcn_update_dpp(z.hi31, __double2hiint(x), kDppBcast31, 0xc, 0xf, false);
    z.lo31 = __builtin_amdgcn_update_dpp(z.lo31, __double2loint(x), kDppBcast31, 0xc, 0xf, false);
    return x + __hiloint2double(z.hi31, z.lo31);
}

// What the drawing wave keeps in registers of a row in LDS.
struct RunRow {
    lds_t<float>* logits;
    double m, inv_temp;
    double tot[4], cum;             // lane l: totals of runs 4 l .. 4 l + 3, inclusive scan over the lanes,
    double before[4];               // the weight before each of the four runs
    ScanZeros zeros;
};
__device__ __forceinline__ void scan_runs(RunRow& r)
{
    const double t01 = r.tot[0] + r.tot[1];
    r.cum = wave_scan_again(t01 + (r.tot[2] + r.tot[3]), r.zeros);         // (sum_runs)
    r.before[0] = dpp_or_zero<kDppWaveShr1>(r.cum);
#pragma unroll
    for (int e = 1; e < 4; ++e) r.before[e] = r.before[e - 1] + r.tot[e - 1];
}
__device__ __forceinline__ void open_run_row(RunRow& r, const lds_t<double>* totals)
{
    const int lane = threadIdx.x & 63;
    r.zeros = { 0, 0, 0, 0 };
#pragma unroll
    for (int e = 0; e < 4; ++e) r.tot[e] = totals[4 * lane + e];
    scan_runs(r);
}

__device__ __forceinline__ void run_weights(const RunRow& r, const PickedRun& p, double (&w)[2])
{
    typedef float floatx2 __attribute__((ext_vector_type(2)));
    const floatx2 x = *(lds_t<floatx2>*)(r.logits + (4 * p.lane + p.k) * kRun + 2 * (int)(threadIdx.x & 63));
    const double z[2] = { fma((double)x.x, r.inv_temp, -r.m), fma((double)x.y, r.inv_temp, -r.m) };
    exp_nonpos_xn<2>(z, w);
}

// One draw with uniform u <= 1 - 2^-24; false (nothing changed) when the row is empty.  Every lane gets the same result.
// A crossing is looked for where sums are compared with the target alone.  A picked lane, run or token without
// weight, or no crossing at the last level, shows by the drawn weight: then nothing has been changed, and the draw is made by pick_run
// and pick_token, which ask for positive values at each level.  An infinite sum: as in draw_wave_row.
__device__ __forceinline__ bool draw_run_row(RunRow& r, double u, Drawn* d)
{
    const int lane = threadIdx.x & 63;
    const double W = readlane_f64(r.cum, 63);
    if (!(W > 0.0)) return false;
    const double none = W * 0.0, target = fma(u, W, none);
    const auto past = [=](double sum) __attribute__((always_inline)) { return !(sum <= target); };
    PickedRun p;
    p.target = target;
    p.lane = (int)__builtin_ctzll(ballot(past(r.cum)) | (1ull << 63));
    const bool p1 = past(r.before[1]), p2 = past(r.before[2]), p3 = past(r.before[3]);
    p.k = __builtin_amdgcn_readlane(p1 ? 0 : p2 ? 1 : p3 ? 2 : 3, p.lane);
    double w[2];
    run_weights(r, p, w);
    p.start = readlane_f64(p1 ? r.before[0] : p2 ? r.before[1] : p3 ? r.before[2] : r.before[3], p.lane);
    const double mine = w[0] + w[1];
    const double sum = p.start + wave_scan_again(mine, r.zeros);           // (sum_tokens)
    const u64 over = ballot(past(sum));
    PickedToken t;
    t.lane = (int)__builtin_ctzll(over | (1ull << 63));
    // the sum before the lane's tokens
    const double sum_before = __hiloint2double(__builtin_amdgcn_update_dpp(__double2hiint(p.start), __double2hiint(sum), kDppWaveShr1, 0xf, 0xf, false),
                                               __builtin_amdgcn_update_dpp(__double2loint(p.start), __double2loint(sum), kDppWaveShr1, 0xf, 0xf, false));
    const bool first = past(sum_before + w[0]);
    t.second = (int)(~ballot(first) >> t.lane & 1ull);
    t.wy = readlane_f64(first ? w[0] : w[1], t.lane);
    // run_left's sum, over the rows of lanes without lane reads (row 3 gets (2 + 3) + (0 + 1), the others what is not read)
    double left_v = lane == t.lane ? (first ? w[1] : w[0]) : mine;
    left_v += dpp_or_zero<kDppXor1>(left_v);
    left_v += dpp_or_zero<kDppXor2>(left_v);
    left_v += dpp_or_zero<kDppHalfMirror>(left_v);
    left_v += dpp_or_zero<kDppMirror>(left_v);
    left_v += dpp_or_zero<kDppBcast15>(left_v);
    left_v += dpp_or_zero<kDppBcast31>(left_v);
    double left = readlane_f64(left_v, 63);
    if (__builtin_expect(over == 0ull || !(t.wy > none), 0)) {
        p = pick_run(r.tot, sum_runs(r.tot), u);
        run_weights(r, p, w);
        const TokenSums s = sum_tokens(w);
        if (s.live == 0ull) return false;           // (the run's total says otherwise: not while totals and logits belong together)
        t = pick_token(w, s, p);
        left = run_left(w, s, t);
    }
    d->y = (4 * p.lane + p.k) * kRun + 2 * t.lane + t.second;
    d->wy = t.wy;
    d->W = W;
    // the token leaves the row
    r.logits[d->y] = -INFINITY;
#pragma unroll
    for (int e = 0; e < 4; ++e) r.tot[e] = lane == p.lane && e == p.k ? left : r.tot[e];
    scan_runs(r);
    return true;
}

}  // namespace dyspec

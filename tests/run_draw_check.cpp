// Draws of one wave by a row's runs (csrc/run_draw.h), run on the host: a row in LDS as a helper of the greedy builder has it against the same
// row in memory as a wave of the tree's workgroup has it.  Token, weight, sum and what is left have to be equal bit for bit, draw after draw,
// until the row is empty.  The row's logits in LDS end at a page that cannot be read.
// usage: run_draw_check totals <trials> <first seed>: the run totals of the pass over the rows against a helper's
//        run_draw_check draws <trials> <first seed>
#include "../paper_2410_11744_amd/csrc/run_draw.h"

#include <signal.h>
#include <stdio.h>
#include <stdlib.h>
#include <sys/mman.h>
#include <unistd.h>

#include <random>

using namespace dyspec;

template <typename T> static T* at_the_end(size_t n)
{
    const size_t page = 1 << 20, bytes = (n * sizeof(T) + 15) / 16 * 16, whole = (bytes + page - 1) / page * page;
    char* const p = (char*)mmap(nullptr, whole + 2 * page, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS, -1, 0);
    if (p == MAP_FAILED) exit(2);
    mprotect(p, page, PROT_NONE);
    mprotect(p + page + whole, page, PROT_NONE);
    return (T*)(p + page + whole - bytes);
}

// the sums of S segments' quads over the 128 tokens of each half wave, as draft_row_sums_kernel makes them
template <int S> static bool totals_agree(std::mt19937& rng)
{
    static double quads[64][16], row_pass[64], other[64], helper[16][64];
    for (auto& lane : quads)
        for (double& q : lane) q = exp(-(double)(rng() % 100000) / 5000.0) * (rng() % 8 != 0);
    host_wave::run([]() {
        double seg[S];
        for (int j = 0; j < S; ++j) seg[j] = quads[threadIdx.x][j];
        other[threadIdx.x] = row_sums(seg);
    });
    for (int l = 0; l < 64; ++l) row_pass[l] = other[l] + other[l ^ 16];
    host_wave::run([]() {
        for (int j = 0; j < S; ++j) {
            const double t = run_total(quads[threadIdx.x][j]);
            helper[j][threadIdx.x] = t;
        }
    });
    for (int j = 0; j < S; ++j)
        for (int half = 0; half < 2; ++half)
            if (memcmp(&helper[j][32 * half + 31], &row_pass[32 * half + 16 + j], sizeof(double))) {
                printf("segment %d of %d, half %d: %.17g and %.17g\n", j, S, half, helper[j][32 * half + 31], row_pass[32 * half + 16 + j]);
                return false;
            }
    return true;
}

struct Row {
    int V;
    double m, inv_temp;
    std::vector<float> memory;
    std::vector<bool> gone;
    float* logits;
    double tot[64][4], lds_tot[64][4], cum[64], before[64][4];
    explicit Row(int V_) : V(V_), m(0.0), inv_temp(1.0), memory(V_), gone(V_, false), logits(at_the_end<float>(row_runs(V_) * kRun)) {}
    void open()
    {
        for (int i = 0; i < row_runs(V) * kRun; ++i) logits[i] = i < V ? memory[i] : -INFINITY;
        static double totals[kSums];
        for (int r = 0; r < kSums; ++r) {
            static double quads[32];
            for (int q = 0; q < 32; ++q) {
                double z[4], w[4];
                for (int e = 0; e < 4; ++e) {
                    const int i = kRun * r + 4 * q + e;
                    z[e] = fma(i < V ? (double)memory[i] : -INFINITY, inv_temp, -m);
                }
                exp_nonpos_xn<4>(z, w);
                quads[q] = (w[0] + w[1]) + (w[2] + w[3]);
            }
            if (kRun * r >= V) { totals[r] = 0.0; continue; }
            const int at = r;
            host_wave::run([at]() {
                const double t = run_total(quads[threadIdx.x & 31]);
                if (threadIdx.x == 31) totals[at] = t;
            });
        }
        for (int l = 0; l < 64; ++l)
            for (int k = 0; k < 4; ++k) tot[l][k] = totals[4 * l + k];
        host_wave::run([this]() {
            RunRow r = run_row();
            open_run_row(r, (lds_t<double>*)totals);
            keep(r);
        });
    }
    RunRow run_row()
    {
        RunRow r;
        r.logits = (lds_t<float>*)logits;
        r.m = m;
        r.inv_temp = inv_temp;
        r.cum = cum[threadIdx.x];
        r.zeros = { 0, 0, 0, 0 };
        for (int k = 0; k < 4; ++k) { r.tot[k] = lds_tot[threadIdx.x][k]; r.before[k] = before[threadIdx.x][k]; }
        return r;
    }
    void keep(const RunRow& r)
    {
        cum[threadIdx.x] = r.cum;
        for (int k = 0; k < 4; ++k) { lds_tot[threadIdx.x][k] = r.tot[k]; before[threadIdx.x][k] = r.before[k]; }
    }
    bool draw_in_lds(double u, Drawn& d)
    {
        bool drawn = false;
        host_wave::run([&]() {
            RunRow r = run_row();
            Drawn mine = { -1, 0.0, 0.0 };
            const bool ok = draw_run_row(r, u, &mine);
            keep(r);
            if (threadIdx.x == 0) { drawn = ok; d = mine; }
        });
        return drawn;
    }
    // as draw_for_node
    bool draw_from_memory(double u, Drawn& d)
    {
        bool drawn = false;
        host_wave::run([&]() {
            const int lane = threadIdx.x;
            double left_of[4];
            for (int k = 0; k < 4; ++k) left_of[k] = tot[lane][k];
            const RunSums sums = sum_runs(left_of);
            if (!(sums.W > 0.0)) return;
            const PickedRun run = pick_run(left_of, sums, u);
            const int tok0 = (4 * run.lane + run.k) * kRun + 2 * lane;
            double z[2], w[2];
            for (int e = 0; e < 2; ++e) z[e] = fma((double)(tok0 + e < V ? memory[tok0 + e] : -INFINITY), inv_temp, -m);
            exp_nonpos_xn<2>(z, w);
            for (int e = 0; e < 2; ++e)
                if (tok0 + e < V && gone[tok0 + e]) w[e] = 0.0;
            const TokenSums tokens = sum_tokens(w);
            if (!tokens.live) return;
            const PickedToken t = pick_token(w, tokens, run);
            const double left = run_left(w, tokens, t);
            if (lane == run.lane) tot[lane][run.k] = left;
            if (lane == 0) {
                d.y = (4 * run.lane + run.k) * kRun + 2 * t.lane + t.second;
                d.wy = t.wy;
                d.W = sums.W;
                drawn = true;
            }
        });
        if (drawn) gone[d.y] = true;
        return drawn;
    }
};

static int draws(int trials, int seed0)
{
    int made = 0;
    for (int trial = 0; trial < trials; ++trial) {
        std::mt19937 rng(seed0 + trial);
        const int sizes[] = { 1, 2, 5, 127, 128, 129, 300, 511, 513, 1000, 4000, 32641, 32768 };
        Row row(sizes[trial % 13]);
        std::normal_distribution<float> normal(0.0f, 3.0f);
        // normal logits rounded to bf16, few tokens, equal ones, some next to nothing, infinite weights
        const int kind = (int)(rng() % 5);
        row.inv_temp = kind == 0 ? 1.0 / (double)0.6f : 1.0;
        float top = -INFINITY;
        for (float& x : row.memory) {
            x = kind == 2 ? 0.25f : normal(rng) * (kind == 3 ? 60.0f : 1.0f);
            uint32_t bits;
            memcpy(&bits, &x, 4);
            bits = (bits + 0x7fffu + ((bits >> 16) & 1u)) & 0xffff0000u;
            memcpy(&x, &bits, 4);
            if ((kind == 1 || kind == 4) && rng() % 9) x = -INFINITY;
            if (x > top) top = x;
        }
        row.m = kind == 4 ? -2000.0 : (double)top * row.inv_temp;
        row.open();
        const int most = row.V < 400 ? row.V + 1 : 90;
        for (int k = 0; k < most; ++k) {
            const double u = rng() % 16 == 0 ? 0.0 : rng() % 16 == 0 ? 1.0 - 0x1p-24 : (rng() >> 8) * (1.0 / 16777216.0);
            Drawn a = { -1, 0.0, 0.0 }, b = { -1, 0.0, 0.0 };
            const bool in_lds = row.draw_in_lds(u, a), from_memory = row.draw_from_memory(u, b);
            if (in_lds != from_memory || (in_lds && (a.y != b.y || memcmp(&a.wy, &b.wy, 8) || memcmp(&a.W, &b.W, 8) || memcmp(row.tot, row.lds_tot, sizeof(row.tot))))) {
                printf("seed %d, V = %d, kind %d, draw %d: token %d of %.17g / %.17g in LDS, %d of %.17g / %.17g from memory\n", seed0 + trial, row.V, kind, k,
                       in_lds ? a.y : -1, a.wy, a.W, from_memory ? b.y : -1, b.wy, b.W);
                return 1;
            }
            if (!in_lds) break;
            ++made;
        }
    }
    printf("%d draws\n", made);
    return made > 20 * trials ? 0 : 1;
}

static void out_of_range(int)
{
    static const char said[] = "a read past the row\n";
    (void)!write(1, said, sizeof(said) - 1);
    _exit(1);
}

int main(int argc, char** argv)
{
    signal(SIGSEGV, out_of_range);
    if (argc != 4) return 2;
    const int trials = atoi(argv[2]), seed0 = atoi(argv[3]);
    if (!strcmp(argv[1], "draws")) return draws(trials, seed0);
    for (int t = 0; t < trials; ++t) {
        std::mt19937 rng(seed0 + t);
        if (!totals_agree<2>(rng) || !totals_agree<8>(rng) || !totals_agree<16>(rng)) return 1;
    }
    return 0;
}

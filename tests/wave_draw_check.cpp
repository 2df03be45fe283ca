// Draws of one wave from a row in LDS (csrc/wave_draw.h), run on the host.  The row's leaf sums and logits end at pages that cannot be
// read, so a read past the row ends the program.
// usage: wave_draw_check range <V>: rows whose sums are infinite; every token is drawn once, none outside the row
//        wave_draw_check exact <trials> <first seed>: the two steps (without and with EXACT) against EXACT alone, bit for bit, on
//        sums that disagree by roundings and uniforms at the edges
#include "../paper_2410_11744_amd/csrc/wave_draw.h"

#include <signal.h>
#include <stdio.h>
#include <stdlib.h>
#include <sys/mman.h>
#include <unistd.h>

#include <random>

using namespace dyspec;

// n values that end (to the 16 bytes of an LDS access) where memory ends
template <typename T> static T* at_the_end(size_t n)
{
    const size_t page = 1 << 20, bytes = (n * sizeof(T) + 15) / 16 * 16, whole = (bytes + page - 1) / page * page;
    char* const p = (char*)mmap(nullptr, whole + 2 * page, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS, -1, 0);
    if (p == MAP_FAILED) exit(2);
    mprotect(p, page, PROT_NONE);
    mprotect(p + page + whole, page, PROT_NONE);
    return (T*)(p + page + whole - bytes);
}

struct Row {
    int V;
    double m;                   // what the weights are relative to
    double* leaf;
    float* logits;
    double tot[64], cum[64];
    explicit Row(int V_) : V(V_), m(0.0), leaf(at_the_end<double>(row_leaves(V_))), logits(at_the_end<float>(row_logits(V_))) {}
    void take(const Row& o)
    {
        m = o.m;
        memcpy(leaf, o.leaf, row_leaves(V) * sizeof(double));
        memcpy(logits, o.logits, row_logits(V) * sizeof(float));
        memcpy(tot, o.tot, sizeof(tot));
        memcpy(cum, o.cum, sizeof(cum));
    }
    bool same(const Row& o) const
    {
        return !memcmp(leaf, o.leaf, row_leaves(V) * sizeof(double)) && !memcmp(logits, o.logits, row_logits(V) * sizeof(float)) &&
               !memcmp(tot, o.tot, sizeof(tot)) && !memcmp(cum, o.cum, sizeof(cum));
    }
    // the leaf sums of the logits, the lanes' sums of those
    void sums()
    {
        for (int l = 0; l < row_leaves(V); ++l) {
            leaf[l] = 0.0;
            for (int k = 0; k < kLeafTokens && l * kLeafTokens + k < row_logits(V); ++k) {
                double z[1] = { (double)logits[l * kLeafTokens + k] - m }, w[1];
                exp_nonpos_xn<1>(z, w);
                leaf[l] += w[0];
            }
        }
        host_wave::run([this]() {
            WaveRow r = wave_row();
            open_wave_row(r, V);
            keep(r);
        });
    }
    WaveRow wave_row() const
    {
        WaveRow r;
        r.leaf = (lds_t<double>*)leaf;
        r.logits = (lds_t<float>*)logits;
        r.m = m;
        r.inv_temp = 1.0;
        r.tot = tot[threadIdx.x];
        r.cum = cum[threadIdx.x];
        return r;
    }
    void keep(const WaveRow& r) { tot[threadIdx.x] = r.tot; cum[threadIdx.x] = r.cum; }
};

enum How { TWO_STEPS, FIRST_STEP, EXACT_ALONE };
static bool draw(Row& row, double u, How how, Drawn& d)
{
    bool drawn = false;
    host_wave::run([&]() {
        WaveRow r = row.wave_row();
        Drawn mine = { -1, 0.0, 0.0 };
        const double W = readlane_f64(r.cum, 63);
        const bool ok = how == TWO_STEPS ? draw_wave_row(r, u, &mine) : how == FIRST_STEP ? draw_wave_row<false>(r, u, W, &mine)
                                         : W > 0.0 && draw_wave_row<true>(r, u, W, &mine);
        row.keep(r);
        if (threadIdx.x == 0) { drawn = ok; d = mine; }
    });
    return drawn;
}

static int range(int V)
{
    Row row(V);
    std::mt19937 rng(V);
    std::vector<bool> out(V, false);
    int left = V < 40 ? V : 40;
    for (int i = 0; i < row_logits(V); ++i) row.logits[i] = -INFINITY;
    for (int k = 0; k < left; ++k) {            // the first, the last and some between
        const int i = k == 0 ? 0 : k == 1 ? V - 1 : V <= 40 ? k - 1 : (int)(rng() % V);
        row.logits[i] = 0.0f;
    }
    left = 0;
    for (int i = 0; i < V; ++i) left += row.logits[i] == 0.0f;
    row.m = -2000.0;                            // exp(2000): the rounding of a maximum over a tiny temperature
    row.sums();
    for (; left > 0; --left) {
        Drawn d;
        if (!draw(row, (rng() >> 8) * (1.0 / 16777216.0), TWO_STEPS, d) || d.y < 0 || d.y >= V || out[d.y]) {
            printf("V = %d: token %d of a row with %d left\n", V, d.y, left);
            return 1;
        }
        out[d.y] = true;
    }
    Drawn d;
    return draw(row, 0.5, TWO_STEPS, d) ? 1 : 0;
}

static int exact(int trials, int seed0)
{
    int first_step_failed = 0, draws = 0;
    for (int t = 0; t < trials; ++t) {
        std::mt19937 rng(seed0 + t);
        const int sizes[] = { 5, 33, 512, 700, 1000, 2049, 16385 };
        const int V = sizes[rng() % 7];
        Row a(V), b(V), c(V);
        const int kind = (int)(rng() % 4);      // all tokens, few tokens, one group, tokens next to nothing
        for (int i = 0; i < row_logits(V); ++i) {
            const float x = -(float)(rng() % 4096) / (kind == 3 ? 40.0f : 512.0f);
            a.logits[i] = i >= V || (kind == 1 && rng() % 50) || (kind == 2 && i / kGroupTokens != (V - 1) / kGroupTokens / 2) ? -INFINITY : x;
        }
        a.sums();
        for (int k = 0; k < 24; ++k) {
            // sums that differ by roundings from the ones below them
            const auto nudge = [&](double x) { return x > 0.0 ? x * (1.0 + ((int)(rng() % 9) - 4) * 0x1p-52) : x; };
            if (k % 3 == 0)
                for (int g = 0; g < 64; ++g) { a.cum[g] = nudge(a.cum[g]); if (rng() % 4 == 0) a.tot[g] = nudge(a.tot[g]); }
            const double W = a.cum[63];
            if (!(W > 0.0)) break;
            // a target at a sum of the row, or just beside it
            double edge = a.cum[rng() % 64];
            if (rng() % 2) {
                const int g = (int)(rng() % (row_leaves(V) / kGroupLeaves));
                edge = g ? a.cum[g - 1] : 0.0;
                for (int l = 0, n = (int)(rng() % 17); l < n; ++l) edge += a.leaf[g * kGroupLeaves + l];
            }
            double u = edge / W * (1.0 + ((int)(rng() % 5) - 2) * 0x1p-53);
            if (rng() % 8 == 0) u = (rng() >> 8) * (1.0 / 16777216.0);
            if (u > 1.0 - 0x1p-24) u = 1.0 - 0x1p-24;           // (the largest uniform)
            b.take(a);
            c.take(a);
            Drawn da, db, dc;
            const bool ra = draw(a, u, TWO_STEPS, da), rb = draw(b, u, EXACT_ALONE, db), rc = draw(c, u, FIRST_STEP, dc);
            if (ra != rb || da.y != db.y || da.wy != db.wy || da.W != db.W || !a.same(b)) {
                printf("seed %d draw %d: token %d of weight %g, EXACT %d of %g\n", seed0 + t, k, da.y, da.wy, db.y, db.wy);
                return 1;
            }
            first_step_failed += !rc;
            ++draws;
            if (!ra) break;
        }
    }
    printf("%d draws, %d by the second step\n", draws, first_step_failed);
    return first_step_failed > trials / 20 ? 0 : 1;
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
    if (argc == 3 && !strcmp(argv[1], "range")) return range(atoi(argv[2]));
    if (argc == 4 && !strcmp(argv[1], "exact")) return exact(atoi(argv[2]), atoi(argv[3]));
    return 2;
}

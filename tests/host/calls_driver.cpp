// Host-only checks of C-ABI calls on models, with the runtime and the launchers of
// fake_runtime.cpp.  Usage: calls_driver CHECK; exit status 0 on success.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <string>
#include <vector>

#include "dsx.h"
#include "fake_runtime.h"

#define CHECK(c)                                                              \
    do {                                                                      \
        if (!(c)) {                                                           \
            std::fprintf(stderr, "check failed at line %d: %s (%s)\n", __LINE__, #c, dsx_last_error()); \
            std::exit(1);                                                     \
        }                                                                     \
    } while (0)

// A nuclear model with S sites in general positions (or, with grid > 0, on multiples of 1/grid along
// axes 2 and 3), its sites uploaded, its box |G| <= r n.
static dsx_model make(int n1, int n2, int n3, int S, int order, int r, int grid = 0, bool ff = false)
{
    std::vector<double> frac, b, f;
    for (int i = 0; i < S; ++i) {
        for (int a = 0; a < 3; ++a) frac.push_back(grid > 0 && a > 0 ? (double)(i % grid) / grid : 0.1 + 0.07 * i + 0.2 * a);
        b.push_back(1.0);
        for (double v : {0.4, 20.0, 0.5, 7.0, 0.1, 2.0, 0.0}) f.push_back(v);
    }
    dsx_model_desc d;
    std::memset(&d, 0, sizeof(d));
    for (int a = 0; a < 3; ++a) { d.cell[a] = 1.0; d.cell[3 + a] = 90.0; }
    d.n[0] = n1; d.n[1] = n2; d.n[2] = n3;
    d.n_sites = S; d.frac = frac.data(); d.b = b.data();
    d.ff = ff ? f.data() : nullptr;
    d.kind = DSX_NUCLEAR; d.has_occ = 1; d.taylor_order = order; d.n_configs = 1;
    dsx_model m = nullptr;
    CHECK(dsx_create_model(&d, &m) == DSX_OK);
    std::vector<float> occ((size_t)S * n1 * n2 * n3, 1.f), disp(3 * occ.size(), 0.01f);
    CHECK(dsx_set_sites(m, 0, occ.data(), order > 0 ? disp.data() : nullptr, nullptr, DSX_HOST) == DSX_OK);
    const int g0[3] = {-r * n1, -r * n2, -r * n3}, cnt[3] = {2 * r * n1 + 1, 2 * r * n2 + 1, 2 * r * n3 + 1};
    CHECK(dsx_set_grid(m, g0, cnt) == DSX_OK);
    return m;
}

// Orders and edges whose fields of one site pass the limit on them: models are made, their boxes
// refused; the largest below it is taken.
static void large_orders()
{
    std::vector<float> out((size_t)5 * 5 * 515);
    for (int n3 : {231, 232, 233, 240, 250, 256})
        for (int S : {1, 3, 64}) {
            dsx_model m = make(1, 1, n3, S, 8, 1);
            CHECK(dsx_compute_intensity(m, out.data(), DSX_HOST, nullptr) == DSX_ERR_UNSUPPORTED);
            CHECK(dsx_destroy_model(m) == DSX_OK);
        }
    for (int n3 : {40, 90}) {
        dsx_model m = make(1, 1, n3, 3, 8, 1);
        CHECK(dsx_compute_intensity(m, out.data(), DSX_HOST, nullptr) == DSX_OK);
        CHECK(dsx_destroy_model(m) == DSX_OK);
    }
    dsx_model m = make(1, 1, 40, 2, 16, 1);
    CHECK(dsx_compute_intensity(m, out.data(), DSX_HOST, nullptr) == DSX_ERR_UNSUPPORTED);
    CHECK(dsx_destroy_model(m) == DSX_OK);
}

// A points call that fails after it has put copies on the stream returns only when they have run:
// they read the caller's points and the call's own work list.
static void points_errors()
{
    const int64_t np = 61;
    const size_t bytes = np * 3 * sizeof(double);
    for (int fault = 0; fault < 5; ++fault) {
        dsx_model m = make(6, 5, 8, 3, 2, 1);
        std::vector<double>* q = new std::vector<double>();
        for (int i = 0; i < np; ++i)
            for (double v : {0.2 * i - 6.0, 1.5, 0.25 * i - 7.0}) q->push_back(v);
        std::vector<float> out(np);
        CHECK(dsx_filter_points(m, 2, 2, np, q->data(), out.data(), DSX_HOST, nullptr) == DSX_OK);
        CHECK(fake::pending == 0);
        fake::launches.clear();
        if (fault == 0) fake::fail_copy_bytes = bytes;
        if (fault == 1) fake::fail_launch = "points";
        if (fault == 2) fake::fail_copy_bytes = np * sizeof(float);
        if (fault == 3) fake::fail_launch = "nuclear";
        if (fault == 4) fake::fail_launch = "bragg";
        CHECK(dsx_filter_points(m, 2, 2, np, q->data(), out.data(), DSX_HOST, nullptr) == DSX_ERR_DEVICE);
        CHECK(std::string(dsx_last_error()).size() > 0);
        CHECK(fake::pending == 0);
        delete q;
        fake::reset();
        CHECK(dsx_destroy_model(m) == DSX_OK);
    }
}

// The tuner's choice of columns per axis-1 block: the default (0) is among the candidates, and
// nothing is timed that the model does not launch or dsx_tune_set_fft would refuse.
static int g_best_tc = 0;
static double tile_cost(const fake::Launch& l)
{
    return l.name == "fft_axis1" && l.tc != g_best_tc ? 2.0 : 1.0;
}

static int tuned_tile(int n1, int n2, int n3, int best_tc)
{
    dsx_model m = make(n1, n2, n3, 2, 0, 1);
    fake::launches.clear();
    fake::cost = tile_cost;
    g_best_tc = best_tc;
    CHECK(dsx_autotune(m, 0, nullptr) == DSX_OK);
    int32_t radices[48], tile = -1, choice[3], tuned = 0;
    CHECK(dsx_tune_query_fft(m, radices, &tile) == DSX_OK && dsx_tune_query(m, choice, &tuned) == DSX_OK && tuned == 1);
    CHECK(dsx_tune_set_fft(m, nullptr, tile) == DSX_OK);
    CHECK(dsx_destroy_model(m) == DSX_OK);
    fake::cost = nullptr;
    return tile;
}

static void tuned_tiles()
{
    unsetenv("DSX_TUNE_CACHE");
    CHECK(tuned_tile(12, 40, 40, 256) == 0);       // one pass: the default of 256 columns
    CHECK(tuned_tile(47, 4, 4, 256) == 0);
    CHECK(tuned_tile(12, 40, 40, 32) == 32);
    CHECK(tuned_tile(47, 4, 4, 64) == 64);
    CHECK(tuned_tile(40, 4, 4, 64) == 0);          // two passes: 64 is the default
    CHECK(tuned_tile(40, 4, 4, 16) == 16);
    CHECK(tuned_tile(67, 4, 4, 32) == 0);          // Stockham passes
    CHECK(tuned_tile(67, 4, 4, 16) == 16);
    CHECK(tuned_tile(40, 4, 4, -1) == 0);          // none better: the default stays
    CHECK(tuned_tile(240, 2, 2, 64) == 0);         // 64 columns of 240 are past the limit
    for (const fake::Launch& l : fake::launches) CHECK(l.name != "fft_axis1" || l.tc < 64);
    CHECK(tuned_tile(12, 12, 12, 32) == 0);        // transformed whole: no axis-1 launch to tune
    for (const fake::Launch& l : fake::launches) CHECK(l.name != "fft_axis1");
    CHECK(tuned_tile(32, 20, 20, 16) == 0);        // a fixed kernel
}

// The tune cache: a line serves the models that take the same kernels, and lines written for other
// kernels of the same sizes (an earlier build's among them) are passed by.
static bool tune_times(dsx_model m)
{
    fake::launches.clear();
    CHECK(dsx_autotune(m, 0, nullptr) == DSX_OK);
    const bool timed = !fake::launches.empty();
    CHECK(dsx_destroy_model(m) == DSX_OK);
    return timed;
}

static void tune_keys()
{
    const char* path = getenv("DSX_TUNE_CACHE");
    CHECK(path);
    FILE* f = std::fopen(path, "w");
    CHECK(f);
    std::fputs("gfx950|0|12,40,40|S4|N2|M1|occ1|box-12,-40,-40,25,81,81|m0\t2 4 4 16 4x3 4x2x5 4x2x5\n", f);
    std::fclose(f);
    CHECK(tune_times(make(12, 40, 40, 4, 2, 1)));                // not the line above
    CHECK(!tune_times(make(12, 40, 40, 4, 2, 1)));               // its own
    CHECK(tune_times(make(12, 40, 40, 4, 2, 1, 0, true)));       // factors that depend on |Q|: class form
    CHECK(!tune_times(make(12, 40, 40, 4, 2, 1, 0, true)));
    CHECK(tune_times(make(12, 40, 40, 4, 2, 1, 2)));             // halves: folded, parity sets
    CHECK(!tune_times(make(12, 40, 40, 4, 2, 1, 4)));            // quarters: four classes, as in general positions
    CHECK(tune_times(make(12, 40, 40, 4, 2, 1, 1)));             // all sites in one class
    CHECK(!tune_times(make(12, 40, 40, 4, 2, 1, 2)));
    CHECK(!tune_times(make(12, 40, 40, 4, 2, 1)));
}

int main(int argc, char** argv)
{
    const std::string what = argc > 1 ? argv[1] : "";
    if (what == "large_orders") large_orders();
    else if (what == "points_errors") points_errors();
    else if (what == "tuned_tiles") tuned_tiles();
    else if (what == "tune_keys") tune_keys();
    else return 2;
    fake::reset();
    std::printf("passed\n");
    return 0;
}

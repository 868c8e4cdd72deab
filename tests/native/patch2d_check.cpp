// Host checks of the 2D patch kernel's plan: the shapes it accepts against the
// LDS a block takes; the time and the memory of the plans kept per problem.
#include <chrono>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <memory>
#include <string>
#include <vector>

#include "patch2d_plan.hpp"
#include "solver.hpp"

#define CHECK(c)                                                              \
    do {                                                                      \
        if (!(c)) {                                                           \
            std::fprintf(stderr, "check failed line %d: %s\n", __LINE__, #c); \
            std::exit(1);                                                     \
        }                                                                     \
    } while (0)

using namespace cf;

constexpr size_t kLimit = 163840;

// Dynamic LDS of a block: E and H entries of n patches, the zero and a spare
// one, at an odd number of 16-byte words; the measured box; weights, basis row
// and offsets of the samples.
size_t dynamic_lds(const Patch2DShape& q, int value, int n, const Patch2DSizes& z) {
    auto up = [](size_t b) { return (b + 15) / 16 * 16; };
    const int v = 16 / value, words = (q.cx + q.b + v - 1) / v;
    const size_t entries = up((size_t)(n + 2) * (words | 1) * 16);
    return 2 * entries + up((size_t)z.box * value) + up((size_t)z.samples * z.points * 8) + up((size_t)z.samples * 8) +
           up((size_t)z.samples * z.points * 2);
}

// Every accepted (patches, box, samples, points) fits with the kernel's static
// part: eight integers per polarization that the kernel is built for.
template <typename T>
void check_lds(int precision) {
    Patch2DShape sh[kMaxShapes2D];
    const int n_sh = patch2d_shapes<T>(sh, kMaxShapes2D);
    long accepted = 0, refused = 0, close = 0;
    for (int v = 0; v < n_sh; ++v) {
        Patch2DSet s;
        s.shapes.assign(sh, sh + n_sh);
        s.lists[0].resize(n_sh);
        s.lists[1].resize(n_sh);
        for (int n : {64, 500, 700, 900, 943, 960})
            for (int points = 1; points <= 4; ++points)
                for (int samples = 1; samples <= 128; samples += 3)
                    for (int box = 1; box <= 40000; box += box < 500 ? 1 : 19) {
                        const Patch2DSizes z{box, samples, points};
                        for (int k = 0; k < 2; ++k) {
                            s.lists[k][v].n = n;
                            s.lists[k][v].parts = 1;
                        }
                        const size_t dyn = dynamic_lds(sh[v], sizeof(T), n, z);
                        const bool one = patch2d_choose(s, precision, 0, 1, z, kLimit) >= 0;
                        const bool both = patch2d_choose_mixed(s, precision, 2, z, kLimit) >= 0;
                        CHECK(!one || dyn + 32 <= kLimit);
                        CHECK(!both || dyn + 64 <= kLimit);
                        CHECK(one || dyn + 256 > kLimit);
                        const Patch2DSizes more{box, kPatchSamples + 1, points}, wider{box, samples, kPatchPoints + 1};
                        for (const Patch2DSizes& w : {more, wider}) {
                            CHECK(patch2d_choose(s, precision, 0, 1, w, kLimit) < 0);
                            CHECK(patch2d_choose_mixed(s, precision, 2, w, kLimit) < 0);
                        }
                        accepted += one;
                        refused += !one;
                        close += dyn <= kLimit && dyn + 64 > kLimit;
                    }
    }
    CHECK(accepted > 0 && refused > 0 && close > 0);
}

// A box of vacuum with one row of conductor.
void make(Problem& p, int nx, int ny) {
    std::vector<uint8_t> id((size_t)nx * ny, 0);
    std::fill(id.begin(), id.begin() + nx, 1);
    const double eps[2] = {1, -INFINITY}, mu[2] = {1, 1};
    cf_grid g{};
    cf_materials m{};
    cf_surface s{};
    g.ndim = 2;
    g.n[0] = nx;
    g.n[1] = ny;
    g.n[2] = 1;
    g.res = 8;
    g.bc[2] = CF_BC_PERIODIC;
    m.n_materials = 2;
    m.eps = eps;
    m.mu = mu;
    for (int k = 0; k < 6; ++k) m.comp_id[k] = id.data();
    s.lo[0] = s.lo[1] = 3;
    s.hi[0] = s.hi[1] = 20;
    s.hi[2] = 1;
    s.n_harm = 2;
    const std::string err = build_problem(g, m, s, p);
    CHECK(err.empty());
}

// Grids that no shape covers, in parts or whole, are told quickly, by less than
// the problem's own creation takes, and keep nothing per cell.
void check_declined() {
    using clock = std::chrono::steady_clock;
    double build = 1e9, plan = 1e9;
    for (int rep = 0; rep < 5; ++rep) {
        Problem p;
        const auto t0 = clock::now();
        make(p, 1500, 1400);
        const auto t1 = clock::now();
        const auto set = patch2d_set(p, rep % 2 ? CF_FP32 : CF_FP64);
        const auto t2 = clock::now();
        build = std::min(build, std::chrono::duration<double>(t1 - t0).count());
        plan = std::min(plan, std::chrono::duration<double>(t2 - t1).count());
        for (int k = 0; k < 2; ++k) {
            for (const Patch2DList& l : set->lists[k]) CHECK(l.parts == 0);
            CHECK(set->live[k].empty() && set->high[k].empty());
        }
    }
    std::printf("1500 x 1400: build %.2f ms, plan %.2f ms\n", build * 1e3, plan * 1e3);
    CHECK(plan < 0.5 * build);
}

// Kept plans are bounded by what they hold, not by their number.
void check_kept() {
    std::vector<std::unique_ptr<Problem>> probs;
    std::weak_ptr<const Patch2DSet> first;
    size_t cells = 0;
    for (int k = 0; k < 90; ++k) {
        probs.push_back(std::make_unique<Problem>());
        make(*probs.back(), 1600, 150);
        const auto set = cfi::cached_patches(*probs.back(), CF_FP32);
        CHECK(!set->live[0].empty() && !set->live[1].empty());
        if (k == 0) first = set;
        if (k < 5) CHECK(cfi::cached_patches(*probs.front(), CF_FP32) == first.lock());
        cells += (size_t)1600 * 150;
    }
    CHECK(cells * 14 > (size_t)256 << 20 && first.expired());
}

int main() {
    check_declined();
    check_kept();
    check_lds<float>(CF_FP32);
    check_lds<double>(CF_FP64);
    std::puts("patch2d ok");
    return 0;
}

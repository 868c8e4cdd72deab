// Host checks of the 2D patch kernel's plan: the shapes it accepts against the
// LDS a block takes.
#include <cstdio>
#include <cstdlib>

#include "patch2d_plan.hpp"

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
                        accepted += one;
                        refused += !one;
                        close += dyn <= kLimit && dyn + 64 > kLimit;
                    }
    }
    CHECK(accepted > 0 && refused > 0 && close > 0);
}

int main() {
    check_lds<float>(CF_FP32);
    check_lds<double>(CF_FP64);
    std::puts("patch2d ok");
    return 0;
}

// Host plan of the 2D patch kernel (see patch2d_plan.hpp).
#include "patch2d_plan.hpp"

#include <algorithm>
#include <cmath>

namespace cf {

namespace {

// Whether an id's material lets the field change.
bool holds_field(const Problem& p, const std::vector<double>& v, int id) {
    return id != kWallId && id < p.nmat && std::isfinite(v[id]);
}

// The material every component of `comps` uses in every cell: `single` when
// the ids with a field share one value, `all` when no cell is without a field.
struct Uniform {
    bool single = true, all = true;
    int id = kNullId;
};
Uniform uniform(const Problem& p, const std::vector<double>& v, std::initializer_list<int> comps) {
    bool used[256] = {};
    for (int c : comps)
        for (int64_t k = 0; k < p.ncell; ++k) used[p.ids[c][k]] = true;
    Uniform u;
    for (int id = 0; id < 256; ++id) {
        if (!used[id]) continue;
        if (!holds_field(p, v, id)) u.all = false;
        else if (u.id == kNullId) u.id = id;
        else if (v[id] != v[u.id]) u.single = false;
    }
    return u;
}

// Patches of cx x b cells with a cell that can change: E where its coefficient
// is not 0, H where an E value of its curl is such a one.
std::vector<Patch2DCell> live_patches(const Problem& p, const std::vector<uint8_t>& live, int cx, int b) {
    const int nx = p.nx, ny = p.ny, LX = (nx + cx - 1) / cx, LY = (ny + b - 1) / b;
    const bool perx = p.grid.bc[0] == CF_BC_PERIODIC, pery = p.grid.bc[1] == CF_BC_PERIODIC;
    std::vector<uint8_t> on((size_t)LX * LY, 0);
    for (int y = 0; y < ny; ++y) {
        const uint8_t* row = live.data() + (size_t)y * nx;
        const int yb = y / b, yd = (y > 0 ? y - 1 : pery ? ny - 1 : y) / b;
        for (int x = 0; x < nx; ++x) {
            if (!row[x]) continue;
            const int xb = x / cx;
            on[(size_t)yb * LX + xb] = on[(size_t)yd * LX + xb] = 1;
            on[(size_t)yb * LX + (x > 0 ? x - 1 : perx ? nx - 1 : x) / cx] = 1;
        }
    }
    std::vector<int> at(on.size(), -1);
    int n = 0;
    for (size_t k = 0; k < on.size(); ++k)
        if (on[k]) at[k] = n++;
    std::vector<Patch2DCell> out;
    if (n >= 65535) return out;
    auto ref = [&](int i, int j) -> uint16_t {
        if (i < 0 || i >= LX) {
            if (!perx) return (uint16_t)n;
            i = (i + LX) % LX;
        }
        if (j < 0 || j >= LY) {
            if (!pery) return (uint16_t)n;
            j = (j + LY) % LY;
        }
        const int a = at[(size_t)j * LX + i];
        return (uint16_t)(a < 0 ? n : a);
    };
    out.reserve(n);
    for (int j = 0; j < LY; ++j)
        for (int i = 0; i < LX; ++i)
            if (on[(size_t)j * LX + i])
                out.push_back({(uint16_t)(i * cx), (uint16_t)(j * b), ref(i + 1, j), ref(i - 1, j), ref(i, j + 1),
                               ref(i, j - 1), 0, 0});
    return out;
}

}  // namespace

Patch2DSet patch2d_set(const Problem& p, int precision) {
    Patch2DSet s;
    Patch2DShape sh[kMaxShapes2D];
    const int n = precision == CF_FP64 ? patch2d_shapes<double>(sh, kMaxShapes2D)
                                       : patch2d_shapes<float>(sh, kMaxShapes2D);
    s.shapes.assign(sh, sh + n);
    const Uniform ue = uniform(p, p.eps, {CF_EX, CF_EY, CF_EZ}), uh = uniform(p, p.mu, {CF_HX, CF_HY, CF_HZ});
    s.id_e = ue.id;
    s.id_h = uh.id;
    const bool fits = p.grid.ndim == 2 && p.nx < 65536 && p.ny < 65536;
    for (int k = 0; k < 2; ++k) {
        s.lists[k].resize(n);
        s.cells[k].assign(n, 0.0);
        if (!fits) continue;
        std::vector<uint8_t> live(p.ncell, 0);
        for (int c : k == 0 ? std::vector<int>{CF_EZ} : std::vector<int>{CF_EX, CF_EY})
            for (int64_t q = 0; q < p.ncell; ++q) live[q] |= holds_field(p, p.eps, p.ids[c][q]);
        for (int v = 0; v < n; ++v) {
            const Patch2DShape& q = s.shapes[v];
            if (q.coef != kRegAll && !(uh.single && uh.all)) continue;
            if (q.coef == kMaskB && !ue.single) continue;
            // a periodic axis wraps at a patch edge
            if (p.grid.bc[0] == CF_BC_PERIODIC && p.nx % q.cx) continue;
            if (p.grid.bc[1] == CF_BC_PERIODIC && p.ny % q.b) continue;
            s.lists[k][v] = live_patches(p, live, q.cx, q.b);
            for (const Patch2DCell& c : s.lists[k][v])
                s.cells[k][v] += (double)std::min(q.cx, p.nx - c.x0) * std::min(q.b, p.ny - c.y0);
        }
    }
    return s;
}

int patch2d_choose(const Patch2DSet& s, int precision, int k, int nslots, const Patch2DSizes& z, size_t lds_limit) {
    constexpr int kCUs = 256;
    int best = -1;
    double best_cost = 0;
    // the surface wave addresses the box by 16-bit offsets
    if (z.box > 65535) return -1;
    for (int v = 0; v < (int)s.shapes.size(); ++v) {
        const Patch2DShape& q = s.shapes[v];
        const int n = (int)s.lists[k][v].size(), waves = (n + 63) / 64 + 1;
        if (n == 0 || waves > 4 * q.mw) continue;
        const size_t lds = precision == CF_FP64 ? patch2d_lds<double>(q, n, z) : patch2d_lds<float>(q, n, z);
        if (lds > lds_limit) continue;
        // VALU issue: about 11 instructions per cell and step, 2 more per
        // masked E component, 4 cycles each; a step's latency (LDS, two
        // barriers) is 700 cycles beyond a wave's own instructions
        const double instr = (q.cx * q.b) * (q.coef == kMaskB ? (k == 0 ? 13.0 : 15.0) : 11.0) + 40;
        const int per_cu = std::max(1, std::min(4 * q.mw / waves, (int)(lds_limit / std::max<size_t>(lds, 1))));
        const int c = std::min(per_cu, (nslots + kCUs - 1) / kCUs);
        const int rounds = (nslots + kCUs * c - 1) / (kCUs * c);
        const double simd = std::ceil(c * waves / 4.0);   // waves of the fullest SIMD
        const double cost = rounds * std::max(simd * instr * 4, 700 + instr * 4.5);
        if (best < 0 || cost < best_cost) {
            best = v;
            best_cost = cost;
        }
    }
    return best;
}

}  // namespace cf

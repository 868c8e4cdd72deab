// Host plan of the 2D patch kernel (see patch2d_plan.hpp).
#include "patch2d_plan.hpp"

#include <algorithm>
#include <cmath>
#include <numeric>

namespace cf {

namespace {

// Steps of a launch of a grid in parts, and so the width of their rims: a
// longer launch loads and stores the fields less often but computes wider rims.
// Pistons of 34000 and 38000 live cells in two parts (FP32, 448 channels, 900
// steps): 12.6 and 17.3 ms with at most 32 steps, 10.8 and 11.9 with 48, 9.9
// and 10.4 with 64 and 96 (about 23 and 25 on tiles).
constexpr int kPartSteps[] = {96, 64, 48, 32, 24, 16, 8};

// Patches a block of the shape may hold (its last wave takes the surface sums).
int most_patches(const Patch2DShape& q) { return 256 * q.mw - 64; }

// Estimated cycles of a step on a compute unit with `waves` waves of the shape,
// polarization slot k.  VALU issue: about 11 instructions per cell and step, 2
// more per masked component, 4 cycles each; a step's latency (LDS, two
// barriers) is 700 cycles beyond a wave's own instructions.
double step_cycles(const Patch2DShape& q, int k, int waves) {
    const double per_cell = q.coef == kMaskH ? 17.0 : q.coef == kMaskB ? (k == 0 ? 13.0 : 15.0) : 11.0;
    const double instr = (q.cx * q.b) * per_cell + 40;
    return std::max(std::ceil(waves / 4.0) * instr * 4, 700 + instr * 4.5);
}

// Estimated cycles of a compute unit per channel and step: of a grid in parts
// (with its share of the copy rate, 4.7 TB/s: 7.6 bytes a cycle, for the loads
// and stores of a launch), and of the tiles (400 x 200 piston: 14000 live cells
// in 6.2 us, FP32).
double parts_cost(const Patch2DShape& q, int k, const Patch2DList& l, int precision) {
    const double value = precision == CF_FP64 ? 8.0 : 4.0;
    const double bytes = 3 * value * (l.cells.size() * (double)(q.cx * q.b) + l.live_cells);
    return l.parts * step_cycles(q, k, (l.n + 63) / 64 + 1) + bytes / 7.6 / l.steps;
}
double tiles_cost(double cells, int precision) { return cells * (precision == CF_FP64 ? 2.2 : 1.05); }

constexpr int kCUs = 256;

// Whether an id's material lets the field change.
bool holds_field(const Problem& p, const std::vector<double>& v, int id) {
    return id != kWallId && id < p.nmat && std::isfinite(v[id]);
}

// The materials the components `comps` use: `single` when the ids with a field
// share one value, `all` when no cell is without a field, `two` when there are
// two kinds of cells, of two values (id, second) or of one and without a field.
struct Uniform {
    bool single = true, all = true, two = false;
    int id = kNullId, second = kNullId;
};
Uniform uniform(const Problem& p, const std::vector<double>& v, std::initializer_list<int> comps) {
    bool used[256] = {};
    for (int c : comps)
        for (int64_t k = 0; k < p.ncell; ++k) used[p.ids[c][k]] = true;
    Uniform u;
    bool more = false;
    for (int id = 0; id < 256; ++id) {
        if (!used[id]) continue;
        if (!holds_field(p, v, id)) {
            u.all = false;
        } else if (u.id == kNullId) {
            u.id = id;
        } else if (v[id] != v[u.id]) {
            u.single = false;
            if (u.second == kNullId) u.second = id;
            else if (v[id] != v[u.second]) more = true;
        }
    }
    u.two = u.id != kNullId && !more && u.single != u.all;
    return u;
}

// Which E components of a polarization can change: bit 0 E_z (TM) or E_x (TE),
// bit 1 E_y (TE).
std::vector<uint8_t> live_e(const Problem& p, int k) {
    std::vector<uint8_t> live(p.ncell, 0);
    const int first = k == 0 ? CF_EZ : CF_EX, n = k == 0 ? 1 : 2;
    for (int c = 0; c < n; ++c)
        for (int64_t q = 0; q < p.ncell; ++q) live[q] |= (uint8_t)(holds_field(p, p.eps, p.ids[first + c][q]) << c);
    return live;
}

// The patches of cx x b cells of a grid, row by row; `on` marks those with a
// cell that can change: E where its coefficient is not 0, H where an E value of
// its curl is such a one.
struct PatchGrid {
    const Problem& p;
    const std::vector<uint8_t>& live;
    const std::vector<uint8_t>& high;                 // as live, H components of the second material
    int cx, b, LX, LY;
    bool perx, pery;
    std::vector<uint8_t> on;
    PatchGrid(const Problem& p_, const std::vector<uint8_t>& live_, const std::vector<uint8_t>& high_, int cx_, int b_)
        : p(p_), live(live_), high(high_), cx(cx_), b(b_), LX((p_.nx + cx_ - 1) / cx_), LY((p_.ny + b_ - 1) / b_),
          perx(p_.grid.bc[0] == CF_BC_PERIODIC), pery(p_.grid.bc[1] == CF_BC_PERIODIC) {
        on.assign((size_t)LX * LY, 0);
        for (int y = 0; y < p.ny; ++y) {
            const uint8_t* row = live.data() + (size_t)y * p.nx;
            const int yb = y / b, yd = (y > 0 ? y - 1 : pery ? p.ny - 1 : y) / b;
            for (int x = 0; x < p.nx; ++x) {
                if (!row[x]) continue;
                const int xb = x / cx;
                on[(size_t)yb * LX + xb] = on[(size_t)yd * LX + xb] = 1;
                on[(size_t)yb * LX + (x > 0 ? x - 1 : perx ? p.nx - 1 : x) / cx] = 1;
            }
        }
    }
    // Appends the patches of columns [i0, i1) and rows [j0, j1) (wrapped on a
    // periodic axis), those of the columns [s0, s1) and rows [t0, t1) stored;
    // `none` marks a neighbour outside the list.  Returns how many.
    int append(int i0, int i1, int j0, int j1, int s0, int s1, int t0, int t1, int none,
               std::vector<Patch2DCell>& out) const {
        std::vector<int> at((size_t)LX * LY, -1);
        auto wrap = [](int v, int n) { return ((v % n) + n) % n; };
        int n = 0;
        for (int j = j0; j < j1; ++j)
            for (int i = i0; i < i1; ++i) {
                if ((!perx && (i < 0 || i >= LX)) || (!pery && (j < 0 || j >= LY))) continue;
                const size_t q = (size_t)wrap(j, LY) * LX + wrap(i, LX);
                if (on[q] && at[q] < 0) at[q] = n++;
            }
        auto ref = [&](int i, int j) -> uint16_t {
            if ((!perx && (i < 0 || i >= LX)) || (!pery && (j < 0 || j >= LY))) return (uint16_t)none;
            const int a = at[(size_t)wrap(j, LY) * LX + wrap(i, LX)];
            return (uint16_t)(a < 0 ? none : a);
        };
        const size_t first = out.size();
        out.resize(first + n);
        for (int j = 0; j < LY; ++j)
            for (int i = 0; i < LX; ++i) {
                const int k = at[(size_t)j * LX + i];
                if (k < 0) continue;
                Patch2DCell c{};
                c.x0 = (uint16_t)(i * cx);
                c.y0 = (uint16_t)(j * b);
                c.right = ref(i + 1, j);
                c.left = ref(i - 1, j);
                c.up = ref(i, j + 1);
                c.down = ref(i, j - 1);
                c.flags = kPatchUsed | (i >= s0 && i < s1 && j >= t0 && j < t1 ? kPatchStored : 0);
                for (int r = 0; r < b && j * b + r < p.ny; ++r)
                    for (int q = 0; q < cx && i * cx + q < p.nx; ++q) {
                        const uint8_t v = live[(size_t)(j * b + r) * p.nx + i * cx + q];
                        c.live[0] |= (uint32_t)(v & 1) << (r * cx + q);
                        c.live[1] |= (uint32_t)(v >> 1) << (r * cx + q);
                        const uint8_t w = high[(size_t)(j * b + r) * p.nx + i * cx + q];
                        c.high[0] |= (uint32_t)(w & 1) << (r * cx + q);
                        c.high[1] |= (uint32_t)(w >> 1) << (r * cx + q);
                    }
                out[first + k] = c;
            }
        return n;
    }
    Patch2DList whole() const {
        Patch2DList l;
        l.n = (int)std::count(on.begin(), on.end(), 1);
        if (l.n == 0 || l.n >= 65535) return Patch2DList();
        l.parts = 1;
        append(0, LX, 0, LY, 0, LX, 0, LY, l.n, l.cells);
        count(l);
        return l;
    }
    void count(Patch2DList& l) const {
        for (const Patch2DCell& c : l.cells)
            if (c.flags & kPatchStored)
                l.live_cells += (double)std::min(cx, p.nx - c.x0) * std::min(b, p.ny - c.y0);
    }
    // Parts of at most `most` patches, cut across x or y where the fewest blocks
    // (then patches) result; a rim of at least `steps` cells beyond a cut.  The
    // measured points (box lo .. hi) stay inside one part.
    Patch2DList parts(int most, int steps, const int lo[2], const int hi[2]) const {
        Patch2DList best;
        for (int axis = 0; axis < 2; ++axis) {
            const int N = axis == 0 ? LX : LY, w = axis == 0 ? cx : b, rim = (steps + w - 1) / w;
            std::vector<int> load(N, 0);
            for (int j = 0; j < LY; ++j)
                for (int i = 0; i < LX; ++i) load[axis == 0 ? i : j] += on[(size_t)j * LX + i];
            const int total = std::accumulate(load.begin(), load.end(), 0);
            const int s0 = lo[axis] / w, s1 = hi[axis] / w;
            const bool per = axis == 0 ? perx : pery;
            for (int m = 2; m <= kMaxParts; ++m) {
                // equal shares; a cut through the measured points moves to their nearer end
                std::vector<int> cut{0};
                int sum = 0;
                for (int c = 0; c < N && (int)cut.size() < m; ++c) {
                    sum += load[c];
                    if (sum * (int64_t)m < (int64_t)total * (int)cut.size()) continue;
                    int at = c + 1;
                    if (at > s0 && at <= s1) at = at - s0 < s1 + 1 - at ? s0 : s1 + 1;
                    if (at > cut.back() && at < N) cut.push_back(at);
                    else break;
                }
                cut.push_back(N);
                if ((int)cut.size() != m + 1) continue;
                Patch2DList l;
                l.parts = m;
                l.steps = steps;
                int n = 0;
                bool ok = true;
                for (int q = 0; q < m; ++q) {
                    const int c0 = cut[q] - rim, c1 = cut[q + 1] + rim;
                    ok = ok && !(per && c1 - c0 > N);      // a rim that meets itself
                    int k = 0;
                    for (int c = c0; c < c1; ++c)
                        if (per) k += load[((c % N) + N) % N];
                        else if (c >= 0 && c < N) k += load[c];
                    n = std::max(n, k);
                    if (s0 >= cut[q] && s1 < cut[q + 1]) l.surf_part = q;
                }
                if (!ok || n == 0 || n > most) continue;
                if (best.parts && (m > best.parts || (m == best.parts && n >= best.n))) break;
                l.n = n;
                for (int q = 0; q < m; ++q) {
                    const int c0 = cut[q] - rim, c1 = cut[q + 1] + rim;
                    const int have = axis == 0 ? append(c0, c1, 0, LY, cut[q], cut[q + 1], 0, LY, n, l.cells)
                                               : append(0, LX, c0, c1, 0, LX, cut[q], cut[q + 1], n, l.cells);
                    l.cells.resize(l.cells.size() + n - have);
                }
                count(l);
                best = std::move(l);
                break;
            }
        }
        return best;
    }
    static constexpr int kMaxParts = 16;
};

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
    s.id_h2 = uh.second;
    s.masks = ue.single;
    s.ncell = p.ncell;
    const bool fits = p.grid.ndim == 2 && p.nx < 65536 && p.ny < 65536;
    // box of every point a channel can measure
    int lo[2] = {p.nx, p.ny}, hi[2] = {-1, -1};
    for (const Gather& g : p.gathers)
        for (int32_t ix : g.idx) {
            const int c[2] = {ix % p.nx, ix / p.nx};
            for (int a = 0; a < 2; ++a) {
                lo[a] = std::min(lo[a], c[a]);
                hi[a] = std::max(hi[a], c[a]);
            }
        }
    for (int k = 0; k < 2; ++k) {
        s.lists[k].resize(n);
        if (!fits) continue;
        const std::vector<uint8_t> live = live_e(p, k);
        // H components of the second material (of none, where that is the second kind)
        std::vector<uint8_t> high(p.ncell, 0);
        if (uh.two)
            for (int c = 0; c < (k == 0 ? 2 : 1); ++c) {
                const auto& ids = p.ids[(k == 0 ? CF_HX : CF_HZ) + c];
                for (int64_t q = 0; q < p.ncell; ++q)
                    high[q] |= (uint8_t)(!(holds_field(p, p.mu, ids[q]) && p.mu[ids[q]] == p.mu[uh.id]) << c);
            }
        // whether a shape's coefficients can hold the materials
        auto holds = [&](const Patch2DShape& q) {
            const bool one_h = uh.single && uh.all;
            switch (q.coef) {
                case kMaskB: return one_h && ue.single;
                case kMaskH: return uh.two && ue.single;
                case kRegE: return one_h;
                default: return true;
            }
        };
        bool covered = false;
        for (int v = 0; v < n; ++v) {
            const Patch2DShape& q = s.shapes[v];
            if (!holds(q)) continue;
            // a periodic axis wraps at a patch edge
            if (p.grid.bc[0] == CF_BC_PERIODIC && p.nx % q.cx) continue;
            if (p.grid.bc[1] == CF_BC_PERIODIC && p.ny % q.b) continue;
            s.lists[k][v] = PatchGrid(p, live, high, q.cx, q.b).whole();
            if (s.lists[k][v].n > most_patches(q)) s.lists[k][v] = Patch2DList();
            covered = covered || s.lists[k][v].parts > 0;
        }
        if (covered || hi[0] < 0) continue;
        // too large for one compute unit: parts, with the shape of the most cells,
        // unless the tiles are estimated to take less
        for (int v = 0; v < n; ++v) {
            const Patch2DShape& q = s.shapes[v];
            if ((q.coef != kMaskB && q.coef != kMaskH) || !holds(q)) continue;
            if (p.grid.bc[0] == CF_BC_PERIODIC && p.nx % q.cx) continue;
            if (p.grid.bc[1] == CF_BC_PERIODIC && p.ny % q.b) continue;
            const PatchGrid grid(p, live, high, q.cx, q.b);
            double best = 0;
            for (int steps : kPartSteps) {
                Patch2DList l = grid.parts(most_patches(q), steps, lo, hi);
                if (!l.parts) continue;
                const double cost = parts_cost(q, k, l, precision);
                if (s.lists[k][v].parts && cost >= best) continue;
                best = cost;
                s.lists[k][v] = std::move(l);
            }
            if (s.lists[k][v].parts && best > tiles_cost(s.lists[k][v].live_cells, precision)) s.lists[k][v] = Patch2DList();
            if (s.lists[k][v].parts) break;
        }
    }
    return s;
}

int patch2d_choose(const Patch2DSet& s, int precision, int k, int nslots, const Patch2DSizes& z, size_t lds_limit) {
    int best = -1;
    double best_cost = 0;
    // the surface wave addresses the box by 16-bit offsets
    if (z.box > 65535) return -1;
    for (int v = 0; v < (int)s.shapes.size(); ++v) {
        const Patch2DShape& q = s.shapes[v];
        const Patch2DList& l = s.lists[k][v];
        const int n = l.n, waves = (n + 63) / 64 + 1, nblocks = nslots * l.parts;
        if (l.parts == 0) continue;
        const size_t lds = precision == CF_FP64 ? patch2d_lds<double>(q, n, z) : patch2d_lds<float>(q, n, z);
        if (lds > lds_limit) continue;
        const int per_cu = std::max(1, std::min(4 * q.mw / waves, (int)(lds_limit / std::max<size_t>(lds, 1))));
        const int c = std::min(per_cu, (nblocks + kCUs - 1) / kCUs);
        const int rounds = (nblocks + kCUs * c - 1) / (kCUs * c);
        const double cost = rounds * step_cycles(q, k, c * waves);
        if (best < 0 || cost < best_cost) {
            best = v;
            best_cost = cost;
        }
    }
    return best;
}

int patch2d_choose_mixed(const Patch2DSet& s, int precision, int nslots, const Patch2DSizes& z, size_t lds_limit) {
    int best = -1;
    double best_cost = 0;
    if (nslots > kCUs || z.box > 65535) return -1;
    for (int v = 0; v < (int)s.shapes.size(); ++v) {
        const Patch2DShape& q = s.shapes[v];
        const Patch2DList &tm = s.lists[0][v], &te = s.lists[1][v];
        if (!patch2d_small(q.cx * q.b, precision == CF_FP64 ? 8 : 4) || tm.parts != 1 || te.parts != 1) continue;
        const int n = std::max(tm.n, te.n);
        const size_t lds = precision == CF_FP64 ? patch2d_lds<double>(q, n, z) : patch2d_lds<float>(q, n, z);
        if (lds > lds_limit) continue;
        const double cost = step_cycles(q, 1, (n + 63) / 64 + 1);
        if (best < 0 || cost < best_cost) {
            best = v;
            best_cost = cost;
        }
    }
    return best;
}

}  // namespace cf

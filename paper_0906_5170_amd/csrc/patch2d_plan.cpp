// Host plan of the 2D patch kernel (see patch2d_plan.hpp).
#include "patch2d_plan.hpp"

#include <algorithm>
#include <cmath>
#include <cstring>
#include <numeric>

namespace cf {

namespace {

// Steps of a launch of a grid in parts, and so the width of their rims: a
// longer launch loads and stores the fields less often but computes wider rims,
// and a smaller shape steps faster but needs more parts.  Which is best depends
// on the channels: few leave compute units idle, so a step's latency counts;
// many fill the device, so all parts' work counts (see patch2d_choose).
constexpr int kPartSteps[] = {96, 64, 48, 32, 24, 16, 8};
constexpr int kNumPartSteps = 7;

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

// Estimated cycles of a block in parts per step, with its share of a launch: the
// longer of a latency of 26 us (launch, tables, first loads) and, with `fill` of
// the compute units at work, its share of the copy rate, 4.7 TB/s or 7.6 bytes a
// cycle, for the loads and stores of its field values.  No other block's steps
// overlap with them: a block of parts fills its compute unit.  Measured, 16
// channels of 260 x 200 cells, FP32: 8 x 4 cells 30 us a launch and 2.6 us a step
// (2.24 with 675 patches), 5 x 5 24 and 2.2, 5 x 4 (kRegE) 23 and 2.1, kMaskH 8 x 4
// 32 and 2.7, 5 x 5 27 and 2.2; FP64 4 x 3 31 and 1.1.
double part_cycles(const Patch2DShape& q, int k, const Patch2DList& l, int precision, double fill) {
    const double value = precision == CF_FP64 ? 8.0 : 4.0, scale = q.coef == kRegE ? 1.2 : q.coef == kMaskH ? 0.7 : 0.8;
    const double bytes = 3 * value * (l.n * (double)(q.cx * q.b) + l.live_cells / l.parts);
    const double step = scale * step_cycles(q, k, 4 * q.mw) * (0.55 + 0.45 * l.n / most_patches(q));
    return step + std::max(62000.0, fill * bytes / 7.6) / l.steps;
}

// And of the tiles, per live cell with the device full (FP32 640 channels:
// 260 x 200 cells 0.86, 300 x 300 0.74, 440 x 330 0.67; FP64 2.6 to 3.4).
double tiles_cost(double cells, int precision) { return cells * (precision == CF_FP64 ? 2.6 : 0.7); }

// The surface wave addresses the box by 16-bit offsets.
bool sizes_fit(const Patch2DSizes& z) { return z.box <= 65535 && z.samples <= kPatchSamples && z.points <= kPatchPoints; }

constexpr int kCUs = 256;
constexpr int kMaxParts = 16;

// Cycles of the tiles' step of nslots channels: a launch's latency (2.6 us a step,
// FP64 3.7), most of it while it has little to do.
double tiles_step(double cells, int nslots, int precision) {
    const double all = tiles_cost(cells, precision) * nslots / kCUs;
    return std::max(all, (precision == CF_FP64 ? 7900.0 : 5400.0) + all / 2);
}

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
    bool used[256];                                   // the ids
};
Uniform uniform(const Problem& p, const std::vector<double>& v, std::initializer_list<int> comps) {
    bool used[256] = {};
    for (int c : comps) {
        const uint8_t* ids = p.ids[c].data();
        uint64_t last = 0, word;
        int64_t k = 0;
        for (; k + 8 <= p.ncell; k += 8) {             // eight ids like the eight before them: seen
            std::memcpy(&word, ids + k, 8);
            if (word == last && k > 0) continue;
            last = word;
            for (int j = 0; j < 8; ++j) used[ids[k + j]] = true;
        }
        for (; k < p.ncell; ++k) used[ids[k]] = true;
    }
    Uniform u;
    std::copy(used, used + 256, u.used);
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

// Cells of component c whose id lets the field change.
int64_t count_live(const Problem& p, int c) {
    bool on[256];
    for (int id = 0; id < 256; ++id) on[id] = holds_field(p, p.eps, id);
    const uint8_t* ids = p.ids[c].data();
    uint64_t last = 0, word;
    int64_t n = 0, k = 0, of_last = 0;
    for (; k + 8 <= p.ncell; k += 8) {
        std::memcpy(&word, ids + k, 8);
        if (word != last || k == 0) {
            last = word;
            of_last = 0;
            for (int j = 0; j < 8; ++j) of_last += on[ids[k + j]];
        }
        n += of_last;
    }
    for (; k < p.ncell; ++k) n += on[ids[k]];
    return n;
}

// Runs of live cells of every row: [begin, end) pairs of row y at runs[y].
using Runs = std::vector<std::vector<int>>;
Runs live_runs(const std::vector<uint8_t>& live, int nx, int ny) {
    Runs r(ny);
    for (int y = 0; y < ny; ++y) {
        const uint8_t* row = live.data() + (size_t)y * nx;
        for (int x = 0; x < nx; ++x) {
            // an end of a run at x, the next one after the values like it
            if ((row[x] != 0) != (r[y].size() % 2 != 0)) r[y].push_back(x);
            uint64_t word;
            for (const uint64_t like = row[x] * 0x0101010101010101ull; x + 8 < nx; x += 8) {
                std::memcpy(&word, row + x + 1, 8);
                if (word != like) break;
            }
        }
        if (r[y].size() % 2) r[y].push_back(nx);
    }
    return r;
}
int64_t count_cells(const Runs& runs) {
    int64_t n = 0;
    for (const auto& row : runs)
        for (size_t k = 0; k < row.size(); k += 2) n += row[k + 1] - row[k];
    return n;
}

// Bit 0 of byte k of a word at bit k.
uint32_t low_bits(uint64_t word) {
    return (uint32_t)(((word & 0x0101010101010101ull) * 0x0102040810204080ull) >> 56);
}

// The patches of cx x b cells of a grid, row by row; `on` marks those with a
// cell that can change: E where its coefficient is not 0, H where an E value of
// its curl is such a one.
struct PatchGrid {
    const Patch2DSet& s;
    int cx, b, LX, LY;
    std::vector<uint8_t> on;
    std::vector<int> loads[2];                        // patches per column and per row
    PatchGrid(const Patch2DSet& s_, const Runs& runs, int cx_, int b_)
        : s(s_), cx(cx_), b(b_), LX((s_.nx + cx_ - 1) / cx_), LY((s_.ny + b_ - 1) / b_) {
        on.assign((size_t)LX * LY, 0);
        for (int y = 0; y < s.ny; ++y) {
            uint8_t* own = on.data() + (size_t)(y / b) * LX;
            uint8_t* below = on.data() + (size_t)((y > 0 ? y - 1 : s.pery ? s.ny - 1 : y) / b) * LX;
            for (size_t k = 0; k < runs[y].size(); k += 2) {
                const int x0 = runs[y][k], x1 = runs[y][k + 1], c0 = x0 / cx, c1 = (x1 - 1) / cx + 1;
                std::memset(own + c0, 1, c1 - c0);
                std::memset(below + c0, 1, c1 - c0);
                own[(x0 > 0 ? x0 - 1 : s.perx ? s.nx - 1 : x0) / cx] = 1;
            }
        }
    }
    // Appends the patches of columns [i0, i1) and rows [j0, j1) (wrapped on a
    // periodic axis), those of the columns [s0, s1) and rows [t0, t1) stored;
    // `none` marks a neighbour outside the list.  Returns how many.
    int append(const std::vector<uint8_t>& live, const std::vector<uint8_t>& high, int i0, int i1, int j0, int j1, int s0,
               int s1, int t0, int t1, int none, std::vector<Patch2DCell>& out) const {
        std::vector<int> at((size_t)LX * LY, -1);
        auto wrap = [](int v, int n) { return v < 0 ? v + n : v >= n ? v - n : v; };   // rims end within a period
        int n = 0;
        for (int j = j0; j < j1; ++j)
            for (int i = i0; i < i1; ++i) {
                if ((!s.perx && (i < 0 || i >= LX)) || (!s.pery && (j < 0 || j >= LY))) continue;
                const size_t q = (size_t)wrap(j, LY) * LX + wrap(i, LX);
                if (on[q] && at[q] < 0) at[q] = n++;
            }
        auto ref = [&](int i, int j) -> uint16_t {
            if ((!s.perx && (i < 0 || i >= LX)) || (!s.pery && (j < 0 || j >= LY))) return (uint16_t)none;
            const int a = at[(size_t)wrap(j, LY) * LX + wrap(i, LX)];
            return (uint16_t)(a < 0 ? none : a);
        };
        const size_t first = out.size();
        out.resize(first + n);
        for (int jj = j0; jj < j1; ++jj)
            for (int ii = i0; ii < i1; ++ii) {
                if ((!s.perx && (ii < 0 || ii >= LX)) || (!s.pery && (jj < 0 || jj >= LY))) continue;
                const int i = wrap(ii, LX), j = wrap(jj, LY);
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
                // a row's bytes as a word (shapes have at most 8 columns)
                const int w = std::min(cx, s.nx - i * cx);
                for (int r = 0; r < b && j * b + r < s.ny; ++r) {
                    const size_t cell = (size_t)(j * b + r) * s.nx + i * cx;
                    uint64_t v = 0, u = 0;
                    std::memcpy(&v, live.data() + cell, w);
                    if (!high.empty()) std::memcpy(&u, high.data() + cell, w);
                    c.live[0] |= low_bits(v) << (r * cx);
                    c.live[1] |= low_bits(v >> 1) << (r * cx);
                    c.high[0] |= low_bits(u) << (r * cx);
                    c.high[1] |= low_bits(u >> 1) << (r * cx);
                }
                out[first + k] = c;
            }
        return n;
    }
    void count_loads() {
        loads[0].assign(LX, 0);
        loads[1].assign(LY, 0);
        for (int j = 0; j < LY; ++j) {
            const uint8_t* row = on.data() + (size_t)j * LX;
            int n = 0;
            for (int i = 0; i < LX; ++i) {
                loads[0][i] += row[i];
                n += row[i];
            }
            loads[1][j] = n;
        }
    }
    double cells() const {
        double n = 0;
        for (int j = 0; j < LY; ++j) {
            const uint8_t* row = on.data() + (size_t)j * LX;
            int w = 0;
            for (int i = 0; i < LX; ++i) w += row[i];
            const int last = row[LX - 1] ? LX * cx - s.nx : 0;   // columns of the last patch beyond the grid
            n += ((double)w * cx - last) * std::min(b, s.ny - j * b);
        }
        return n;
    }
    Patch2DList whole() const {
        Patch2DList l;
        l.n = (int)std::count(on.begin(), on.end(), 1);
        if (l.n == 0 || l.n >= 65535) return Patch2DList();
        l.parts = 1;
        l.live_cells = cells();
        return l;
    }
    // Parts of at most `most` patches, cut across x or y where the fewest blocks
    // (then patches) result; a rim of at least `steps` cells beyond a cut.  The
    // measured points (box lo .. hi) stay inside one part.  After count_loads.
    Patch2DList parts(int most, int steps, const int lo[2], const int hi[2]) const {
        Patch2DList best;
        for (int axis = 0; axis < 2; ++axis) {
            const int N = axis == 0 ? LX : LY, w = axis == 0 ? cx : b, rim = (steps + w - 1) / w;
            const std::vector<int>& load = loads[axis];
            std::vector<int> before(N + 1, 0);         // patches before a column (row)
            std::partial_sum(load.begin(), load.end(), before.begin() + 1);
            const int total = before[N];
            const int s0 = lo[axis] / w, s1 = hi[axis] / w;
            const bool per = axis == 0 ? s.perx : s.pery;
            for (int m = std::max(2, total / most); m <= kMaxParts; ++m) {
                // equal shares; a cut through the measured points moves to their nearer end
                std::vector<int> cut{0};
                for (int c = 0; c < N && (int)cut.size() < m; ++c) {
                    if (before[c + 1] * (int64_t)m < (int64_t)total * (int)cut.size()) continue;
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
                l.axis = axis;
                bool ok = true;
                for (int q = 0; q < m; ++q) {
                    const int c0 = cut[q] - rim, c1 = cut[q + 1] + rim;
                    ok = ok && !(per && c1 - c0 > N);      // a rim that meets itself
                    int k = before[std::min(c1, N)] - before[std::max(c0, 0)];
                    if (per && ok) k += before[std::max(c1 - N, 0)] + total - before[std::min(c0 + N, N)];
                    l.n = std::max(l.n, k);
                    if (s0 >= cut[q] && s1 < cut[q + 1]) l.surf_part = q;
                }
                if (!ok || l.n == 0 || l.n > most) continue;
                if (best.parts && (m > best.parts || (m == best.parts && l.n >= best.n))) break;
                l.cut = std::move(cut);
                best = std::move(l);
                break;
            }
        }
        return best;
    }
};

}  // namespace

std::shared_ptr<const Patch2DSet> patch2d_set(const Problem& p, int precision) {
    const auto set = std::make_shared<Patch2DSet>();
    Patch2DSet& s = *set;
    Patch2DShape sh[kMaxShapes2D];
    const int n = precision == CF_FP64 ? patch2d_shapes<double>(sh, kMaxShapes2D)
                                       : patch2d_shapes<float>(sh, kMaxShapes2D);
    s.shapes.assign(sh, sh + n);
    for (auto& lists : s.lists) lists.resize(n * (1 + kNumPartSteps));
    s.nx = p.nx;
    s.ny = p.ny;
    // grids beyond every shape in parts are told by their live cells alone (1800 x
    // 1800 cells: 50 ms of planning for nothing before, now 2)
    int64_t most = 0;
    for (const Patch2DShape& q : s.shapes) most = std::max(most, (int64_t)kMaxParts * most_patches(q) * q.cx * q.b);
    const bool fits[2] = {
        p.grid.ndim == 2 && p.nx < 65536 && p.ny < 65536 && count_live(p, CF_EZ) <= most,
        p.grid.ndim == 2 && p.nx < 65536 && p.ny < 65536 && std::max(count_live(p, CF_EX), count_live(p, CF_EY)) <= most};
    if (!fits[0] && !fits[1]) return set;
    const Uniform ue = uniform(p, p.eps, {CF_EX, CF_EY, CF_EZ}), uh = uniform(p, p.mu, {CF_HX, CF_HY, CF_HZ});
    s.id_e = ue.id;
    s.id_h = uh.id;
    s.id_h2 = uh.second;
    s.masks = ue.single;
    s.perx = p.grid.bc[0] == CF_BC_PERIODIC;
    s.pery = p.grid.bc[1] == CF_BC_PERIODIC;
    // whether a shape's coefficients can hold the materials, and a periodic axis
    // wraps at a patch edge
    auto holds = [&](const Patch2DShape& q) {
        if ((s.perx && p.nx % q.cx) || (s.pery && p.ny % q.b)) return false;
        const bool one_h = uh.single && uh.all;
        switch (q.coef) {
            case kMaskB: return one_h && ue.single;
            case kMaskH: return uh.two && ue.single;
            case kRegE: return one_h;
            default: return true;
        }
    };
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
    uint8_t live_id[256], high_id[256];
    for (int id = 0; id < 256; ++id) {
        live_id[id] = holds_field(p, p.eps, id);
        // the second material, or none where that is the second kind
        high_id[id] = uh.two && !(holds_field(p, p.mu, id) && p.mu[id] == p.mu[uh.id]);
    }
    for (int k = 0; k < 2; ++k) {
        if (!fits[k]) continue;
        // bit c of a cell: `of` its id of component first + c (all but the used ids
        // without it)
        auto bits = [&](const uint8_t* of, const bool* used, int first, int count) {
            std::vector<uint8_t> out(p.ncell, (uint8_t)((1 << count) - 1));
            for (int c = 0; c < count; ++c)
                for (int id = 0; id < 256; ++id) {
                    if (!used[id] || of[id]) continue;
                    const uint8_t* __restrict ids = p.ids[first + c].data();
                    uint8_t* __restrict at = out.data();
                    const uint8_t without = (uint8_t)id, keep = (uint8_t)~(1 << c);
                    const int64_t ncell = p.ncell;
                    for (int64_t q = 0; q < ncell; ++q) at[q] = ids[q] == without ? at[q] & keep : at[q];
                }
            return out;
        };
        s.live[k] = k == 0 ? bits(live_id, ue.used, CF_EZ, 1) : bits(live_id, ue.used, CF_EX, 2);
        const Runs runs = live_runs(s.live[k], p.nx, p.ny);
        const int64_t cells = count_cells(runs);
        bool covered = false;
        for (int v = 0; v < n; ++v) {
            const Patch2DShape& q = s.shapes[v];
            if (!holds(q) || cells > (int64_t)most_patches(q) * q.cx * q.b) continue;
            s.lists[k][v] = PatchGrid(s, runs, q.cx, q.b).whole();
            if (s.lists[k][v].n > most_patches(q)) s.lists[k][v] = Patch2DList();
            covered = covered || s.lists[k][v].parts > 0;
        }
        // too large for one compute unit: parts, of the shapes that hold their E
        // values in masks, unless the tiles are estimated to take less
        double best = 0, live = 0;
        for (int v = 0; v < n && !covered && hi[0] >= 0; ++v) {
            const Patch2DShape& q = s.shapes[v];
            // (smaller shapes take many parts, mostly rims)
            if (q.cx * q.b * (precision == CF_FP64 ? 8 : 4) < 64) continue;
            if (q.coef == kRegAll || !s.masks || !holds(q) || cells > (int64_t)kMaxParts * most_patches(q) * q.cx * q.b)
                continue;
            PatchGrid grid(s, runs, q.cx, q.b);
            grid.count_loads();
            live = grid.cells();
            for (int t = 0; t < kNumPartSteps; ++t) {
                Patch2DList& l = s.lists[k][n * (1 + t) + v];
                l = grid.parts(most_patches(q), kPartSteps[t], lo, hi);
                if (!l.parts) continue;
                l.live_cells = live;
                const double cost = l.parts * part_cycles(q, k, l, precision, 1);
                if (best == 0 || cost < best) best = cost;
            }
        }
        if (best > tiles_cost(live, precision))
            for (Patch2DList& l : s.lists[k]) l = Patch2DList();
        // the cells' masks, while some list may need them
        if (std::none_of(s.lists[k].begin(), s.lists[k].end(), [](const Patch2DList& l) { return l.parts > 0; }))
            std::vector<uint8_t>().swap(s.live[k]);
        else if (uh.two)
            s.high[k] = k == 0 ? bits(high_id, uh.used, CF_HX, 2) : bits(high_id, uh.used, CF_HZ, 1);
    }
    return set;
}

const std::vector<Patch2DCell>& patch2d_cells(const Patch2DSet& s, int k, int entry) {
    std::lock_guard<std::mutex> lk(s.mu);
    std::vector<Patch2DCell>& out = s.cells[{k, entry}];
    if (!out.empty()) return out;
    out.reserve(s.lists[k][entry].size());
    const Patch2DShape& q = s.shape(entry);
    const Patch2DList& l = s.lists[k][entry];
    const PatchGrid g(s, live_runs(s.live[k], s.nx, s.ny), q.cx, q.b);
    if (l.parts == 1) {
        g.append(s.live[k], s.high[k], 0, g.LX, 0, g.LY, 0, g.LX, 0, g.LY, l.n, out);
        return out;
    }
    const int w = l.axis == 0 ? q.cx : q.b, rim = (l.steps + w - 1) / w;
    for (int r = 0; r < l.parts; ++r) {
        const int a = l.cut[r], z = l.cut[r + 1], c0 = a - rim, c1 = z + rim;
        const int have = l.axis == 0 ? g.append(s.live[k], s.high[k], c0, c1, 0, g.LY, a, z, 0, g.LY, l.n, out)
                                     : g.append(s.live[k], s.high[k], 0, g.LX, c0, c1, 0, g.LX, a, z, l.n, out);
        out.resize(out.size() + l.n - have);
    }
    return out;
}

int patch2d_choose(const Patch2DSet& s, int precision, int k, int nslots, const Patch2DSizes& z, size_t lds_limit,
                   int others, size_t room) {
    int best = -1;
    double best_cost = 0;
    if (!sizes_fit(z)) return -1;
    for (int v = 0; v < (int)s.lists[k].size(); ++v) {
        const Patch2DShape& q = s.shape(v);
        const Patch2DList& l = s.lists[k][v];
        if (l.parts == 0 || (l.parts > 1 && l.size() > room)) continue;
        const int n = l.n, waves = (n + 63) / 64 + 1, nblocks = (nslots + (l.parts > 1 ? others : 0)) * l.parts;
        const size_t lds = precision == CF_FP64 ? patch2d_lds<double>(q, n, z) : patch2d_lds<float>(q, n, z);
        if (lds > lds_limit) continue;
        const int per_cu =
            l.parts > 1 ? 1 : std::max(1, std::min(4 * q.mw / waves, (int)(lds_limit / std::max<size_t>(lds, 1))));
        const int c = std::min(per_cu, (nblocks + kCUs - 1) / kCUs);
        const int rounds = (nblocks + kCUs * c - 1) / (kCUs * c);
        const double cost = rounds * (l.parts > 1 ? part_cycles(q, k, l, precision, std::min(1.0, (double)nblocks / kCUs))
                                                  : step_cycles(q, k, c * waves));
        // launches of 8 steps are mostly start, loads and stores: only well below the
        // tiles (FP64, 200 x 90 cells: 5.0 us a step with 16 channels, 3.8 on tiles,
        // 8.2 against 18 with 256)
        if (l.parts > 1 && l.steps < 16 && 1.15 * cost > tiles_step(l.live_cells, nslots + others, precision)) continue;
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
    if (nslots > kCUs || !sizes_fit(z)) return -1;
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

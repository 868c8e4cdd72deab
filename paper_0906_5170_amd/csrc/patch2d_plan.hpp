// Host plan of the 2D patch kernel: which patches of a problem's grid hold
// cells that can change, the parts of grids beyond one compute unit, and the
// shape a launch takes.
#pragma once

#include <map>
#include <memory>
#include <mutex>
#include <utility>
#include <vector>

#include "patch2d.hpp"
#include "plan.hpp"

namespace cf {

// A polarization's lists for one entry: `parts` lists of n patches each, at
// most `steps` steps per launch (0: any number, one part), cut across `axis`
// before the patch columns (rows) of `cut`.
struct Patch2DList {
    int n = 0, parts = 0, surf_part = 0, steps = 0, axis = 0;
    std::vector<int> cut;
    double live_cells = 0;                            // cells of the stored patches inside the grid
    size_t size() const { return (size_t)n * parts; }
};

struct Patch2DSet {
    std::vector<Patch2DShape> shapes;
    // per polarization (0 TM, 1 TE) and entry (parts == 0: not usable): every shape
    // with whole channels, then, for grids beyond a compute unit, every shape with
    // parts of each number of steps
    std::vector<Patch2DList> lists[2];
    const Patch2DShape& shape(int entry) const { return shapes[entry % shapes.size()]; }
    int kernel(int entry) const { return entry % (int)shapes.size(); }   // shape index of its launches
    int id_e = kNullId, id_h = kNullId;               // an E and an H material with a field
    int id_h2 = kNullId;                              // and the other one where H has two
    bool masks = false;                               // E components share one material
    int nx = 0, ny = 0;
    bool perx = false, pery = false;
    // per polarization and cell: which E components can change (bit 0 E_z or
    // E_x, bit 1 E_y; empty without a usable list), which H components are of the
    // second material (empty where there is none)
    std::vector<uint8_t> live[2], high[2];
    // the patches of the lists in use so far, by (polarization, entry)
    mutable std::mutex mu;
    mutable std::map<std::pair<int, int>, std::vector<Patch2DCell>> cells;
};

// The lists of a fusable 2D problem for every entry of the precision (sizes and
// cuts), and the patches of one of them, formed on first use.
std::shared_ptr<const Patch2DSet> patch2d_set(const Problem& p, int precision);
const std::vector<Patch2DCell>& patch2d_cells(const Patch2DSet& s, int k, int entry);

// Entry with the least estimated time for nslots channels of polarization slot k,
// or -1 when none covers the problem; parts share the device with `others`
// channels of the other polarization and have room for `room` patches.
int patch2d_choose(const Patch2DSet& s, int precision, int k, int nslots, const Patch2DSizes& z, size_t lds_limit,
                   int others = 0, size_t room = SIZE_MAX);

// The small shape (whole channels) with the least time for a launch of both
// polarizations (nslots channels in all) that the device takes at once, or -1.
int patch2d_choose_mixed(const Patch2DSet& s, int precision, int nslots, const Patch2DSizes& z, size_t lds_limit);

}  // namespace cf

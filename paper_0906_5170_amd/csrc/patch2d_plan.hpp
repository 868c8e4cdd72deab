// Host plan of the 2D patch kernel: which patches of a problem's grid hold
// cells that can change, the parts of grids beyond one compute unit, and the
// shape a launch takes.
#pragma once

#include <memory>
#include <vector>

#include "patch2d.hpp"
#include "plan.hpp"

namespace cf {

// A polarization's lists for one shape: `parts` lists of n patches each, at
// most `steps` steps per launch (0: any number, one part).
struct Patch2DList {
    int n = 0, parts = 0, surf_part = 0, steps = 0;
    std::vector<Patch2DCell> cells;
    double live_cells = 0;                            // cells of the stored patches inside the grid
};

struct Patch2DSet {
    std::vector<Patch2DShape> shapes;
    std::vector<Patch2DList> lists[2];                // per polarization (0 TM, 1 TE) and shape (parts == 0: not usable)
    int id_e = kNullId, id_h = kNullId;               // an E and an H material with a field
    int id_h2 = kNullId;                              // and the other one where H has two
    bool masks = false;                               // E components share one material
    int64_t ncell = 0;
};

// The lists of a fusable 2D problem for every shape of the precision.
Patch2DSet patch2d_set(const Problem& p, int precision);

// Shape with the least estimated time for nslots channels of polarization
// slot k, or -1 when none covers the problem.
int patch2d_choose(const Patch2DSet& s, int precision, int k, int nslots, const Patch2DSizes& z, size_t lds_limit);

// The small shape with the least time for a launch of whole channels of both
// polarizations (nslots in all) that the device takes at once, or -1.
int patch2d_choose_mixed(const Patch2DSet& s, int precision, int nslots, const Patch2DSizes& z, size_t lds_limit);

}  // namespace cf

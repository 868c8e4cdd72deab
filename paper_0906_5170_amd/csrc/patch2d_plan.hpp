// Host plan of the 2D patch kernel: which patches of a problem's grid hold
// cells that can change, and the shape a launch takes.
#pragma once

#include <memory>
#include <vector>

#include "patch2d.hpp"
#include "plan.hpp"

namespace cf {

struct Patch2DSet {
    std::vector<Patch2DShape> shapes;
    std::vector<std::vector<Patch2DCell>> lists[2];   // per polarization (0 TM, 1 TE) and shape; empty: not usable
    std::vector<double> cells[2];                     // cells of the listed patches inside the grid
    int id_e = kNullId, id_h = kNullId;               // an E and an H material with a field
};

// The lists of a fusable 2D problem for every shape of the precision.
Patch2DSet patch2d_set(const Problem& p, int precision);

// Shape with the least estimated time for nslots channels of polarization
// slot k, or -1 when none covers the problem.
int patch2d_choose(const Patch2DSet& s, int precision, int k, int nslots, const Patch2DSizes& z, size_t lds_limit);

}  // namespace cf

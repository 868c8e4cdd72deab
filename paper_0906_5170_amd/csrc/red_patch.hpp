// Patch kernel of the reduced problems (cylindrical orders, k_z and Bloch
// points): launch interface.
#pragma once

#include <deque>
#include <memory>
#include <vector>

#include "device.hpp"
#include "lds.hpp"
#include "red_span.hpp"

namespace cf {

// Coefficient classes of the cells.  A cell's H class names the triple of
// materials its H_x, H_y, H_z coefficients come from, its E class the triple
// of E_x, E_y, E_z; cls[cell] = H class | E class << 8.  Class 0 holds no
// field (every b is 0).  id[g][c] lists one material id per component for
// class c of group g (0 H, 1 E); ids whose coefficients agree share a class.
constexpr int kPatchClasses = 64;
struct PatchClasses {
    const uint16_t* cls;                // device, one word per cell
    int n[2];                           // classes in use per group (with class 0)
    int h_uniform;                      // every cell has H class 1
    uint8_t id[2][kPatchClasses][3];
};

// Largest bounding box (cells) of the interpolation points of one channel's
// source or measured component, and largest samples x points of a channel's
// face: they size the block's LDS tables.
struct PatchSizes {
    int box, samples, points;
};

// Open (CPML) and dispersive k_z runs: host-side classes, Lorentz rows (row 0
// has no term; [1 / eps, (c1, c2, c3) per term]) with the row of each E class
// and component, and device memory for the blocks' CPML values.
struct PatchOpen {
    const uint16_t* cls;
    int n_lor, lor_rows;
    double lor[4][13];
    uint8_t lrow[kPatchClasses][3];
    void* scratch;
    int64_t scratch_bytes;
};

// Patches without a cell that can change are left out: host copy of the
// classes, device memory for the list of the others, and the host lists, which
// live until the stream has drained.  The plan of the last launch, with its list
// in `dev`, serves further ones of as many channels (a run's spans between
// convergence checks).
struct PatchLive {
    const uint16_t* cls;
    char* dev;
    size_t room;
    std::deque<std::vector<uint16_t>>* keep;
    std::shared_ptr<const void> plan;
    int plan_slots = -1;
};

// What a launch did: whether a shape covers the grid (nothing is launched
// otherwise), and the cells its patches hold.
struct PatchRan {
    bool launched = false;
    double cells = 0;
};

// As launch_red_resident_span, for grids a patch shape covers (see PatchRan).  slots == nullptr:
// the channels 0 .. nslots - 1.  op: an open or dispersive run (whole span
// only, the grid's CPML set as for the split kernels); it uses no field
// blocks.  live: as above, or null (every patch of the grid).
template <typename T>
hipError_t launch_red_patch(T* fields, const ChanDev* ch, const int* slots, int nslots, const Grid2D& g,
                            const RedOrders& ord, const RedSpan& span, const SurfTables& t, const PatchClasses& pc,
                            const PatchSizes& ps, const PatchOpen* op, PatchLive* live, double dA, double* acc, double* gamma,
                            int gamma_stride, hipStream_t s, PatchRan* ran);

}  // namespace cf

// Patch kernel of the Cartesian 2D problems (TM and TE): plan and launch
// interface.
#pragma once

#include <cstdint>
#include <vector>

#include "device.hpp"

namespace cf {

// How a shape holds the cells' coefficients b (a is one value per field group
// wherever b != 0).  kMaskB: one bit per E component, for grids whose H
// components share one material and whose E components share one or are held
// at 0.  kRegE: E values in registers, one H material.  kRegAll: all in
// registers, any materials.
enum Patch2DCoef { kMaskB = 0, kRegE = 1, kRegAll = 2 };

// Patch of cx x b cells per thread, register budget of mw waves per SIMD.
struct Patch2DShape {
    int cx, b, mw, coef;
};
constexpr int kMaxShapes2D = 12;
template <typename T>
int patch2d_shapes(Patch2DShape* out, int max);

// One patch of an instance's list, on the device: first cell, and the list
// indices of the patches to the right and left, above and below (the list's
// length stands for "none": fields there are 0).
struct Patch2DCell {
    uint16_t x0, y0, right, left, up, down, pad0, pad1;
};
static_assert(sizeof(Patch2DCell) == 16, "one 16-byte load per thread");

// Head of an instance: its lists and their lengths per polarization (0 TM,
// 1 TE), and an E and an H material whose a, b its cells carry.
struct Patch2DInst {
    const Patch2DCell* cells[2];
    int32_t n[2];
    int32_t id_e, id_h;
};

// Box of the measured points and samples x points of a channel, the largest
// of a launch: they size the block's LDS tables.
struct Patch2DSizes {
    int box, samples, points;
};

// LDS bytes of a block for n patches.
template <typename T>
size_t patch2d_lds(const Patch2DShape& q, int n, const Patch2DSizes& z);

// Advances the channels slots[0 .. nslots - 1] (all of polarization pol) by
// min(kmax, remaining steps of the instance) steps from launch-clock step m, in
// the instance's buffer fa.  heads: one per instance.  n: longest list of the
// launch's instances.
template <typename T>
hipError_t launch_patch2d(int shape, int pol, const ChanDev* ch, const int* slots, int nslots, const InstDev* inst,
                          const Patch2DInst* heads, int n, const Patch2DSizes& z, int kmax, int m, hipStream_t s);

}  // namespace cf

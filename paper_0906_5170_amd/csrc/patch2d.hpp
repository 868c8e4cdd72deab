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
// at 0.  kMaskH: besides, one bit per H component, for H components of two
// materials (one may hold H at 0).  kRegE: E values in registers, one H
// material.  kRegAll: all in registers, any materials.
enum Patch2DCoef { kMaskB = 0, kRegE = 1, kRegAll = 2, kMaskH = 3 };

// Patch of cx x b cells per thread, register budget of mw waves per SIMD.
struct Patch2DShape {
    int cx, b, mw, coef;
};
constexpr int kMaxShapes2D = 16;
// Small shapes, of grids whose solve takes a fraction of a millisecond: a launch
// may hold both polarizations, and a block can start its channel itself.  (The
// registers of the larger ones have no room for either.)
constexpr bool patch2d_small(int cells, int value_bytes) { return cells * value_bytes <= 32; }
template <typename T>
int patch2d_shapes(Patch2DShape* out, int max);

// One patch of an instance's list, on the device: first cell, the list indices
// of the patches to the right and left, above and below (the list's length
// stands for "none": fields there are 0), the cells whose E components (TM: E_z;
// TE: E_x, E_y) are not held at 0, cell (r, j) at bit r cx + j, and those whose H
// components (TM: H_x, H_y; TE: H_z) are of the second H material.
enum { kPatchUsed = 1, kPatchStored = 2 };
struct Patch2DCell {
    uint16_t x0, y0, right, left, up, down, flags, pad;
    uint32_t live[2], high[2];
};
static_assert(sizeof(Patch2DCell) == 32, "four 8-byte loads per thread");

// Head of an instance: per polarization (0 TM, 1 TE) its lists (one per part,
// of one length n, the shorter ones filled up with unused patches), the part
// whose stored patches hold the measured points; and an E and an H material
// whose a, b its cells carry.
//
// A grid with more live cells than a compute unit's registers hold goes in
// parts, one block each: a part's list holds the patches it stores and, beyond
// the cuts, a rim of its neighbours' patches, which goes stale by one cell per
// step.  A launch may take as many steps as the rim is wide.
struct Patch2DInst {
    const Patch2DCell* cells[2];
    int32_t n[2], surf_part[2];
    int32_t id_e, id_h;
    int32_t masks;      // E components share one material: b = b(id_e) where live
    int32_t id_h2;      // second H material (kMaskH)
    int32_t start;      // the block of step 0 kicks and starts its channel itself (whole channels only)
};

// Box of the measured or the kicked points and samples x points of a channel,
// the largest of a launch: they size the block's LDS tables.
struct Patch2DSizes {
    int box, samples, points;
};
// The most samples of a channel and points of a sample: the surface wave keeps
// them in registers.  (Surfaces that fit a tile have at most 118 samples, of 4
// points.)
constexpr int kPatchSamples = 128, kPatchPoints = 4;

// LDS bytes of a block for n patches, dynamic and static.
template <typename T>
size_t patch2d_lds(const Patch2DShape& q, int n, const Patch2DSizes& z);

// Advances the channels (of polarization pol; 0: of both, for a small shape) by
// min(kmax, remaining steps of the instance) steps from launch-clock step m, from
// the instance's buffer src (0: fa, 1: fb) to dst (the same one only without
// parts).  items: one per block, channel slot | part << kPartShift.  heads: one
// per instance.  n: longest list of the launch's instances.
constexpr int kPartShift = 26;
template <typename T>
hipError_t launch_patch2d(int shape, int pol, const ChanDev* ch, const int* items, int nitems, const InstDev* inst,
                          const Patch2DInst* heads, int n, const Patch2DSizes& z, int kmax, int m, int src, int dst,
                          hipStream_t s);

}  // namespace cf

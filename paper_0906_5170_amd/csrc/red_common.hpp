// Update forms of the reduced (cylindrical, k_z, Bloch) problems shared by
// their kernels.
#pragma once

#include "device.hpp"
#include "yee_common.hpp"

namespace cf {

// Reduced update, with M the coupling of the run (m, or k dx) and the curls
// in undivided form:
//   h_x/h_z: ((A e_z(j+1) - B e_z) - M e_y) C       h_y/h_r: M e_x D - d_x e_z
//   e_x/e_z: ((P h_z - Q h_z(j-1)) + M h_y) D       e_y/e_r: -M h_x C - d_x h_z
//   h_z/h_phi and e_z/e_phi: the Cartesian two-dimensional forms;
// cylindrical (CYL): (A, B, C, D, P, Q) = (j + 1/2, j - 1/2, 1/j, 1/(j - 1/2),
// j, j - 1), row 0 the axis with its own rules; k_z: all 1.  The row table
// holds 6 values per row (field precision); the kernels read C and D from it
// and form the others from j.
enum { RA = 0, RB, RC, RD, RP, RQ, kRowFactors };

// Complex runs keep the real part of the six components in the first
// 6 x ncell values of a channel block and the imaginary part in the next.
// The x neighbour across the periodic edge of part `part` (0 real, 1
// imaginary): forward (F[nx] = p F[0]) or backward (F[-1] = conj(p) F[nx-1]),
// from the wrapped cell's own-part value a and other-part value b.
template <typename T>
__device__ __forceinline__ T bloch_fwd(T a, T b, int part, T pc, T ps) {
    return part == 0 ? a * pc - b * ps : a * pc + b * ps;
}
template <typename T>
__device__ __forceinline__ T bloch_bwd(T a, T b, int part, T pc, T ps) {
    return part == 0 ? a * pc + b * ps : a * pc - b * ps;
}

}  // namespace cf

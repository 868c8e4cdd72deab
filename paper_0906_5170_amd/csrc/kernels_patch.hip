// Patch kernel of the reduced problems, FP32 fields (red_patch_kernel.hpp).
#include "red_patch_kernel.hpp"

namespace cf {

template hipError_t launch_red_patch<float>(float*, const ChanDev*, const int*, int, const Grid2D&, const RedOrders&,
                                         const RedSpan&, const SurfTables&, const PatchClasses&, const PatchSizes&,
                                         const PatchOpen*, PatchLive*, double, double*, double*, int, hipStream_t, PatchRan*);

}  // namespace cf

// 3D plane-marching kernels of the schemes beside WENO3 + HLLC: 16 x 15 columns over 16 planes.
#include "fv_registry.h"
#include "fv_stage_z.h"

namespace fvk {
#define PLANES(R, F) FV_ENTRY_Z(EQ_EULER, R, F, 16, 15, 16, 256)
static const RegEntry kTable[] = {
    PLANES(REC_WENO3, FLUX_HLL), PLANES(REC_WENO3, FLUX_RUSANOV),
    PLANES(REC_MUSCL, FLUX_HLLC), PLANES(REC_MUSCL, FLUX_HLL), PLANES(REC_MUSCL, FLUX_RUSANOV),
};
#undef PLANES
const RegEntry* unit_planes3d(int* count) { *count = sizeof(kTable) / sizeof(kTable[0]); return kTable; }
}  // namespace fvk

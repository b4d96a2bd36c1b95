// 2D row-marching kernels: the schemes whose column window and faces fit the 128 registers that
// four wavefronts per SIMD leave (a spilled register costs a wait for every load before it).
#include "fv_registry.h"
#include "fv_stage_y.h"

namespace fvk {
static const RegEntry kTable[] = {
    FV_ENTRY_Y(EQ_EULER, REC_WENO3, FLUX_HLLC), FV_ENTRY_Y(EQ_EULER, REC_WENO3, FLUX_HLL),
    FV_ENTRY_Y(EQ_EULER, REC_WENO3, FLUX_RUSANOV),
    FV_ENTRY_Y(EQ_EULER, REC_MUSCL, FLUX_HLLC), FV_ENTRY_Y(EQ_EULER, REC_MUSCL, FLUX_HLL),
    FV_ENTRY_Y(EQ_EULER, REC_MUSCL, FLUX_RUSANOV),
    FV_ENTRY_Y(EQ_SWE, REC_MUSCL, FLUX_HLL), FV_ENTRY_Y(EQ_SWE, REC_MUSCL, FLUX_RUSANOV),
};
const RegEntry* unit_rows2d(int* count) { *count = sizeof(kTable) / sizeof(kTable[0]); return kTable; }
}  // namespace fvk

// Step kernels over all bits and drawn subsets, one to eight waves per chain,
// for int32_t coefficients with int32_t fields.
#include "pns_full.h"

namespace pns {

hipError_t launch_full_i32(bool drawn, bool instr, int block, int groups, int grid, size_t dyn, hipStream_t st,
                           const StepArgs& a)
{
    PNS_FULL_TILE_LIST(PNS_FULL_DISPATCH_TILE, int32_t, int32_t)
    return hipErrorInvalidConfiguration;
}

}  // namespace pns

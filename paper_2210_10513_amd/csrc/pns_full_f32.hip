// Step kernels over all bits and drawn subsets, one to eight waves per chain,
// for float coefficients with double fields.
#include "pns_full.h"

namespace pns {

hipError_t launch_full_f32(bool drawn, bool instr, int block, int groups, int grid, size_t dyn, hipStream_t st,
                           const StepArgs& a)
{
    return drawn ? full::launch_tile<float, double, true>(instr, block, groups, grid, dyn, st, a)
                 : full::launch_tile<float, double, false>(instr, block, groups, grid, dyn, st, a);
}

}  // namespace pns

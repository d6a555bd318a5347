// Step kernels over all bits and drawn subsets, one to eight waves per chain,
// for int32_t coefficients with int64_t fields.
#include "pns_full.h"

namespace pns {

hipError_t launch_full_i64(bool drawn, bool instr, int block, int groups, int grid, size_t dyn, hipStream_t st,
                           const StepArgs& a)
{
    return drawn ? full::launch_tile<int32_t, int64_t, true>(instr, block, groups, grid, dyn, st, a)
                 : full::launch_tile<int32_t, int64_t, false>(instr, block, groups, grid, dyn, st, a);
}

}  // namespace pns

// fp32 on the matrix cores, the pipelined form with four groups of waves, 4 columns a staging load: instantiations.
#include "split_kernel.h"

namespace sc {
sc_status_t launch_split_pipe4_4(const Plan& p, const SplitArgs& a, const SplitTable& t, const void* x, void* y, int grid, hipStream_t stream)
{
    return launch_split_typed<14, 4>(p, a, t, x, y, grid, stream);
}
}  // namespace sc

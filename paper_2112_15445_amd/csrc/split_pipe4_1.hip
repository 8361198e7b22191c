// fp32 on the matrix cores, the pipelined form with four groups of waves, 1 column a staging load: instantiations.
#include "split_kernel.h"

namespace sc {
sc_status_t launch_split_pipe4_1(const Plan& p, const SplitArgs& a, const SplitTable& t, const void* x, void* y, int grid, hipStream_t stream)
{
    return launch_split_typed<14, 1>(p, a, t, x, y, grid, stream);
}
}  // namespace sc

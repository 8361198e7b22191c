// DENSE variant, 8-bit activations (SC_I8, SC_CB4_I8): v_mfma_i32_16x16x64_i8 instantiations of the one-shot kernel
// for 16-row blocks of weights of 4 GB and more.
#include "dense_tile_kernel.h"

namespace sc {
sc_status_t launch_tile_i8_wide(const Plan& p, const TileArgs& a, const void* x, void* y, int grid, hipStream_t stream)
{
    return launch_tile_typed<SC_I8, 0, true>(p, a, x, y, grid, stream);
}
}  // namespace sc

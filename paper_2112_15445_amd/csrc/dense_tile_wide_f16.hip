// DENSE variant, 16-bit activations (SC_F16, SC_CB4_F16): v_mfma_f32_16x16x32_f16 instantiations of the one-shot kernel
// for 16-row blocks of weights of 4 GB and more.
#include "dense_tile_kernel.h"

namespace sc {
sc_status_t launch_tile_f16_wide(const Plan& p, const TileArgs& a, const void* x, void* y, int grid, hipStream_t stream)
{
    return launch_tile_typed<SC_F16, 0, true>(p, a, x, y, grid, stream);
}
}  // namespace sc

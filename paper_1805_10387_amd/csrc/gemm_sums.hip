// Instantiations of the contraction kernels: weight-gradient products that also sum their first operand (bias gradients).
#include "gemm_dtl.hpp"

namespace mp {
int launch_dtl_sums_tile(int t, const GemmArgs& g, dim3 grid, hipStream_t hs) {
    switch (t) {
        case 1: return launch_dtl_sums<256, 128>(g, grid, hs);
        case 3: return launch_dtl_sums<128, 128>(g, grid, hs);
        case 4: return launch_dtl_sums<128, 64>(g, grid, hs);
        case 5: return launch_dtl_sums<64, 128>(g, grid, hs);
        default: return MP_E_UNSUPPORTED;
    }
}
}  // namespace mp

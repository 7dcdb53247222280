// Instantiations of the contraction kernels for small problems.
#include "gemm_small.hpp"

namespace mp {

template <int NW>
static int launch_tile_nw(bool a_kc, bool b_kc, const GemmArgs& g, int splits, hipStream_t hs) {
    if (!a_kc) return launch_small<NW, false, false>(g, splits, hs);
    return b_kc ? launch_small<NW, true, true>(g, splits, hs) : launch_small<NW, true, false>(g, splits, hs);
}
int launch_small_tile(int waves, bool a_kc, bool b_kc, const GemmArgs& g, int splits, hipStream_t hs) {
    return waves == 8 ? launch_tile_nw<8>(a_kc, b_kc, g, splits, hs) : launch_tile_nw<4>(a_kc, b_kc, g, splits, hs);
}

template <int NW>
static void launch_both(const BothArgs& b, bool tail, int n, hipStream_t hs) {
    if (tail) hipLaunchKernelGGL((gemm_small_both_kernel<NW, TAIL>), dim3(n), dim3(64 * NW), sm_lds(NW), hs, b);
    else hipLaunchKernelGGL((gemm_small_both_kernel<NW, EDGE>), dim3(n), dim3(64 * NW), sm_lds(NW), hs, b);
}
int launch_small_both(int waves, const BothArgs& b, hipStream_t hs) {
    const auto odd  = [](int v) { return v % 8 != 0; };
    const bool tail = odd(b.dx.K) || odd(b.dx.N) || odd(b.dw.M) || odd(b.dw.N);
    const int  n = b.dx.tiles_m * b.dx.tiles_n + b.dw.tiles_m * b.dw.tiles_n;
    if (waves == 8) launch_both<8>(b, tail, n, hs);
    else launch_both<4>(b, tail, n, hs);
    MP_LAUNCH_CHECK("gemm launch (both gradients)");
    return MP_OK;
}

}  // namespace mp

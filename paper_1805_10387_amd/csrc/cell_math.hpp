// LSTM cell arithmetic shared by the per-step cell kernels and the persistent recurrent-layer kernels: fp32 between
// fp16 storage points, the cell state never rounded (paper Section 3.2: explicitly fp32 parts of a mixed-precision
// model).  One definition, so that a layer gives the same bits whichever of the two paths runs it.
#pragma once
#include "common.hpp"

namespace mp {

// A cell stands between the arrival of one slice and the departure of the next in the recurrent kernels, where nothing hides an
// instruction, so both functions are branch-free and divide by a reciprocal: a forward cell is 84 instructions, and 137 with
// the IEEE division and the library's tanh, whose two branches both run in a wave of mixed values (0.05 to 0.1 us of a step).
// Relative error against 64 bits on N(0, 1) values, root mean square (largest), that way and this: sigma 4.3e-8 (2.8e-7) and the
// same; tanh 2.8e-8 (1.5e-7) and 2.6e-8 (1.1e-7).
// sigma(x): the hardware's reciprocal with one Newton step
__device__ __forceinline__ float sigmoidf_(float x) {
    const float d = 1.0f + __expf(-x);
    const float r = __builtin_amdgcn_rcpf(d);
    const float s = __builtin_fmaf(r, __builtin_fmaf(-d, r, 1.0f), r);
    return d == INFINITY ? 0.0f : s;  // (a NaN stays one)
}
// tanh(x): 1 - 2 / (exp(2|x|) + 1), and near zero, where that cancels, x + x^3 P(x^2) with P fitted for a small largest relative
// error (5e-9, at 0.86)
__device__ __forceinline__ float tanhf_(float x) {
    const float a = __builtin_fabsf(x), u = a * a;
    float       p = -0.0004824179923f;
    p = __builtin_fmaf(p, u, 0.002651009941f);
    p = __builtin_fmaf(p, u, -0.008331941441f);
    p = __builtin_fmaf(p, u, 0.02169604227f);
    p = __builtin_fmaf(p, u, -0.05393717065f);
    p = __builtin_fmaf(p, u, 0.1333306581f);
    p = __builtin_fmaf(p, u, -0.3333332539f);
    const float near = __builtin_fmaf(a * u, p, a);
    const float far  = __builtin_fmaf(-2.0f, __builtin_amdgcn_rcpf(__expf(2.0f * a) + 1.0f), 1.0f);
    return __builtin_copysignf(a < 0.875f ? near : far, x);
}

// gi, gf, gg, go: the STORED (fp16) gate sums of one cell.  Returns c_t; *h16 = RNE16(sigma(o) tanh(c_t)).
__device__ __forceinline__ float lstm_cell_forward(float gi, float gf, float gg, float go, float c_prev, uint16_t* h16) {
    const float cn = sigmoidf_(gf) * c_prev + sigmoidf_(gi) * tanhf_(gg);
    *h16           = f2h(sigmoidf_(go) * tanhf_(cn));
    return cn;
}

// What the backward of one cell takes from its forward: the activations of the stored gate sums and tanh of the cell state.
// (Apart from the rest because it does not depend on the gradients.)
struct LstmCellAct {
    float si, sf, tg, so, tc;
};
__device__ __forceinline__ LstmCellAct lstm_cell_act(float gi, float gf, float gg, float go, float c) {
    return {sigmoidf_(gi), sigmoidf_(gf), tanhf_(gg), sigmoidf_(go), tanhf_(c)};
}

// Backward of one cell for one time step.  dh: fp32 sum of the gradients reaching h_t; dc_in: cell-state gradient
// carried from step t + 1.  Writes RNE16 of (di, df, dg, do) and returns the cell-state gradient carried to t - 1.
__device__ __forceinline__ float lstm_cell_backward(const LstmCellAct& f, float c_prev, float dh, float dc_in, uint16_t* d4) {
    const float d_o = dh * f.tc * f.so * (1.0f - f.so);
    const float dc  = dc_in + dh * f.so * (1.0f - f.tc * f.tc);
    const float d_i = dc * f.tg * f.si * (1.0f - f.si);
    const float d_f = dc * c_prev * f.sf * (1.0f - f.sf);
    const float d_g = dc * f.si * (1.0f - f.tg * f.tg);
    d4[0] = f2h(d_i);
    d4[1] = f2h(d_f);
    d4[2] = f2h(d_g);
    d4[3] = f2h(d_o);
    return dc * f.sf;
}

}  // namespace mp

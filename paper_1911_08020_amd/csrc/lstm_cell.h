// The LSTM cell of the recurrent models (section 4.1): no bias, gate order
// (i, f, g, o),
//     c' = sigmoid(f) * c + sigmoid(i) * tanh(g),   h' = sigmoid(o) * tanh(c').
// Shared by the cell kernel of the two-kernel step and the fused step kernel, so
// both apply the same arithmetic to the gate pre-activations.
#pragma once

#include <hip/hip_runtime.h>

namespace darb {

// 1 / d for a finite d >= 1: the hardware's reciprocal and one Newton step.
__device__ __forceinline__ float lstm_rcp(float d) {
    const float r = __builtin_amdgcn_rcpf(d);
    return fmaf(r, fmaf(-d, r, 1.0f), r);
}

// 1 / (1 + e^-z).  The exponent is bounded so that the Newton step never meets an
// infinity; written so that a NaN passes through.
__device__ __forceinline__ float lstm_sigmoid(float z) {
    float t = z * -0x1.715476p+0f;                    // -log2 e
    t = t > 126.0f ? 126.0f : t;
    return lstm_rcp(1.0f + __builtin_amdgcn_exp2f(t));
}

// tanh without branches: from 0.625 on 1 - 2 / (e^2|x| + 1) (at 15 that is 1 in fp32),
// below it x + x^3 P(x^2), where the other form would cancel: the usual split of single
// precision (that of Moshier's Cephes library), P of degree 4 fitted for this file to the
// least relative error over the range (9e-9).  About 25 instructions; the math library's
// took several times as many, and the cell's two in a row were its longest part.
__device__ __forceinline__ float lstm_tanh(float x) {
    const float a = fabsf(x), s = x * x;
    float p = fmaf(s, -5.704986397e-3f, 2.063908614e-2f);
    p = fmaf(s, p, -5.373971537e-2f);
    p = fmaf(s, p, 1.333144158e-1f);
    p = fmaf(s, p, -3.333328068e-1f);
    const float small = fmaf(x * s, p, x);
    const float t = a > 15.0f ? 15.0f : a;
    const float e = __builtin_amdgcn_exp2f(t * 0x1.715476p+1f);   // 2 log2 e
    const float big = copysignf(fmaf(-2.0f, lstm_rcp(e + 1.0f), 1.0f), x);
    return a >= 0.625f ? big : small;                 // a NaN takes the polynomial
}

// gi, gf, gg, go: gate pre-activations; c: the cell state, updated; returns h'.
__device__ __forceinline__ float lstm_cell(float gi, float gf, float gg, float go, float &c) {
    const float cn = lstm_sigmoid(gf) * c + lstm_sigmoid(gi) * lstm_tanh(gg);
    c = cn;
    return lstm_sigmoid(go) * lstm_tanh(cn);
}

}  // namespace darb

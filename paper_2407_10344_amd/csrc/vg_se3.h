// Device helpers on SE(3) in FP64 (retraction, composition) and the end of a
// Levenberg-Marquardt iteration, which the candidates' reduction does.
#pragma once

#include "vg_device.h"

namespace vg {

__device__ __forceinline__ void hat3(const double v[3], double S[9]) {
    S[0] = 0.0;
    S[1] = -v[2];
    S[2] = v[1];
    S[3] = v[2];
    S[4] = 0.0;
    S[5] = -v[0];
    S[6] = -v[1];
    S[7] = v[0];
    S[8] = 0.0;
}

__device__ __forceinline__ void mm3(const double A[9], const double B[9], double C[9]) {
    for (int i = 0; i < 3; ++i)
        for (int j = 0; j < 3; ++j) C[3 * i + j] = A[3 * i] * B[j] + A[3 * i + 1] * B[3 + j] + A[3 * i + 2] * B[6 + j];
}

// Exp of xi = [omega; v] in SE(3): rotation by Rodrigues' formula, translation
// V v with V = I + (1 - cos th)/th^2 W + (th - sin th)/th^3 W^2, W = (omega)x.
__device__ inline void se3_exp(const double xi[6], double out[12]) {
    const double th2 = xi[0] * xi[0] + xi[1] * xi[1] + xi[2] * xi[2];
    const double th = sqrt(th2);
    double a, b, c;
    if (th < 1e-4) {
        a = 1.0 - th2 / 6.0 + th2 * th2 / 120.0;
        b = 0.5 - th2 / 24.0 + th2 * th2 / 720.0;
        c = 1.0 / 6.0 - th2 / 120.0 + th2 * th2 / 5040.0;
    } else {
        const double s = sin(th), co = cos(th);
        a = s / th;
        b = (1.0 - co) / th2;
        c = (th - s) / (th2 * th);
    }
    double W[9], W2[9];
    hat3(xi, W);
    mm3(W, W, W2);
    double V[9];
    for (int k = 0; k < 9; ++k) {
        const double I = (k % 4 == 0) ? 1.0 : 0.0;
        out[k] = I + a * W[k] + b * W2[k];
        V[k] = I + b * W[k] + c * W2[k];
    }
    for (int i = 0; i < 3; ++i) out[9 + i] = V[3 * i] * xi[3] + V[3 * i + 1] * xi[4] + V[3 * i + 2] * xi[5];
}

__device__ inline void pose_mul(const double A[12], const double B[12], double C[12]) {
    double Rm[9];
    mm3(A, B, Rm);
    for (int i = 0; i < 3; ++i)
        C[9 + i] = A[3 * i] * B[9] + A[3 * i + 1] * B[10] + A[3 * i + 2] * B[11] + A[9 + i];
    for (int k = 0; k < 9; ++k) C[k] = Rm[k];
}

// FP32 copy of a pose (16 floats) as the multi-level FP32 kernels read it, taken
// from where the pose was stored: as further uses of the values themselves the
// conversions change the order in which the compiler fuses the sums that form them,
// and the last bit of a step decides accepts near convergence.
__device__ __forceinline__ void stage_pose(float* __restrict__ posef, int64_t f, const volatile double* P) {
    if (posef == nullptr) return;
    for (int k = 0; k < 16; ++k) posef[16 * f + k] = k < 12 ? (float)P[k] : 0.0f;
}

// Accept the candidate of factor f iff it is valid and its error e_new is below the
// error at T (then lambda / 10), else keep T (lambda x 10).  Records e at T and the
// decision.
__device__ inline void lm_accept(const LmArgs& lm, int64_t f, double e_new) {
    const double e0 = lm.lin[(int64_t)kOutRow * f];
    const bool acc = (lm.valid[f] != 0) && (e_new < e0);
    if (acc) {
        for (int k = 0; k < 12; ++k) lm.poses[12 * f + k] = lm.cand[12 * f + k];
        lm.lambda[f] /= 10.0;
    } else {
        lm.lambda[f] *= 10.0;
    }
    if (lm.accepted != nullptr) lm.accepted[(int64_t)lm.stride * f + lm.col] = acc ? 1 : 0;
    if (lm.e_out != nullptr) lm.e_out[(int64_t)lm.stride * f + lm.col] = e0;
    stage_pose(lm.posef, f, lm.poses + 12 * f);
}

}  // namespace vg

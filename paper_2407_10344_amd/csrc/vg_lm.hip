// FP64 pose kernels: SE(3) retraction with its right Jacobian.
#include "vg_se3.h"

namespace vg {

// Right Jacobian of SE(3): J_r(xi) = sum_n (-ad_xi)^n / (n+1)!, with
// ad_xi = [[(omega)x, 0], [(v)x, (omega)x]] for xi = [omega; v].  The series is
// summed until the term is negligible (it converges for every xi).
__device__ void se3_right_jacobian(const double xi[6], double J[36]) {
    double Wx[9], Vx[9];
    hat3(xi, Wx);
    hat3(xi + 3, Vx);
    double ad[36] = {0};
    for (int i = 0; i < 3; ++i)
        for (int j = 0; j < 3; ++j) {
            ad[6 * i + j] = -Wx[3 * i + j];
            ad[6 * (3 + i) + j] = -Vx[3 * i + j];
            ad[6 * (3 + i) + 3 + j] = -Wx[3 * i + j];
        }
    double term[36], next[36];
    for (int k = 0; k < 36; ++k) {
        term[k] = (k % 7 == 0) ? 1.0 : 0.0;
        J[k] = term[k];
    }
    for (int n = 1; n < 60; ++n) {
        double mx = 0.0;
        for (int i = 0; i < 6; ++i)
            for (int j = 0; j < 6; ++j) {
                double s = 0.0;
                for (int q = 0; q < 6; ++q) s += term[6 * i + q] * ad[6 * q + j];
                next[6 * i + j] = s / (double)(n + 1);
            }
        for (int k = 0; k < 36; ++k) {
            term[k] = next[k];
            J[k] += term[k];
            mx = fmax(mx, fabs(term[k]));
        }
        if (mx < 1e-18) break;
    }
}

__global__ void k_se3_retract(int64_t F, const double* __restrict__ T0, const double* __restrict__ xi,
                              double* __restrict__ T, double* __restrict__ jr) {
    const int64_t f = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (f >= F) return;
    double x[6], E[12], A[12], C[12];
    for (int k = 0; k < 6; ++k) x[k] = xi[6 * f + k];
    for (int k = 0; k < 12; ++k) A[k] = T0[12 * f + k];
    se3_exp(x, E);
    pose_mul(A, E, C);
    for (int k = 0; k < 12; ++k) T[12 * f + k] = C[k];
    if (jr != nullptr) {
        double J[36];
        se3_right_jacobian(x, J);
        for (int k = 0; k < 36; ++k) jr[36 * f + k] = J[k];
    }
}

__global__ void k_fill(double* __restrict__ p, int64_t n, double v) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

vg_status launch_se3_retract(vg_context* ctx, int64_t F, const double* d_T0, const double* d_xi, double* d_T,
                             double* d_jr) {
    if (F == 0) return VG_OK;
    k_se3_retract<<<(int)((F + 63) / 64), 64, 0, ctx->stream>>>(F, d_T0, d_xi, d_T, d_jr);
    VG_HIP(hipGetLastError());
    return VG_OK;
}

vg_status launch_fill(vg_context* ctx, double* d_ptr, int64_t n, double v) {
    if (n <= 0) return VG_OK;
    k_fill<<<(int)((n + 255) / 256), 256, 0, ctx->stream>>>(d_ptr, n, v);
    VG_HIP(hipGetLastError());
    return VG_OK;
}

}  // namespace vg

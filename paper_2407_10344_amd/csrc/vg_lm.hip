// FP64 pose kernels: SE(3) retraction with its right Jacobian, and the proposal of
// a Levenberg-Marquardt step (one thread per factor; 6x6 systems are tiny, so the
// point is to stay on the device).
#include <algorithm>

#include "vg_se3.h"

namespace vg {

// T = T0 Exp(xi) of one factor.
__device__ __forceinline__ void retract(const double* __restrict__ T0, const double* __restrict__ xi, int64_t f,
                                        double x[6], double C[12]) {
    double E[12], A[12];
    for (int k = 0; k < 6; ++k) x[k] = xi[6 * f + k];
    for (int k = 0; k < 12; ++k) A[k] = T0[12 * f + k];
    se3_exp(x, E);
    pose_mul(A, E, C);
}

// Poses alone: one thread per factor (a million factors 81 us, 606 us with a wave each).
__global__ __launch_bounds__(64) void k_se3_poses(int64_t F, const double* __restrict__ T0,
                                                  const double* __restrict__ xi, double* __restrict__ T) {
    const int64_t step = (int64_t)gridDim.x * blockDim.x;
    for (int64_t f = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; f < F; f += step) {
        double x[6], C[12];
        retract(T0, xi, f, x, C);
        for (int k = 0; k < 12; ++k) T[12 * f + k] = C[k];
    }
}

// Poses and Jacobians, one wave per factor.  Right Jacobian of SE(3): J_r(xi) = sum_n (-ad_xi)^n / (n+1)!,
// with ad_xi = [[(omega)x, 0], [(v)x, (omega)x]] for xi = [omega; v]; the series is
// summed until the term is negligible (it converges for every xi).  Bound by that
// serial chain, so each of 36 lanes keeps one entry and the terms pass through LDS
// (64 factors: 4.8 us, against 41 us with one lane per factor).
__global__ __launch_bounds__(64) void k_se3_retract(int64_t F, const double* __restrict__ T0,
                                                    const double* __restrict__ xi, double* __restrict__ T,
                                                    double* __restrict__ jr) {
    __shared__ double s_term[36];
    const int lane = threadIdx.x;
    for (int64_t f = blockIdx.x; f < F; f += gridDim.x) {
        double x[6], C[12];
        retract(T0, xi, f, x, C);
        for (int k = 0; k < 12; ++k)
            if (lane == k) T[12 * f + k] = C[k];
        const int i = min(lane, 35) / 6, j = min(lane, 35) % 6;
        // column j of -ad: rows of -(omega)x, -(v)x
        double W[9], V[9], ad[6];
        hat3(x, W);
        hat3(x + 3, V);
#pragma unroll
        for (int q = 0; q < 6; ++q) {
            const int a = q % 3;
            const double w = j % 3 == 0 ? W[3 * a] : (j % 3 == 1 ? W[3 * a + 1] : W[3 * a + 2]);
            const double v = j % 3 == 0 ? V[3 * a] : (j % 3 == 1 ? V[3 * a + 1] : V[3 * a + 2]);
            ad[q] = (q < 3) == (j < 3) ? -w : (q < 3 ? 0.0 : -v);
        }
        double term = i == j ? 1.0 : 0.0, J = term;
        for (int n = 1; n < 60; ++n) {
            __syncthreads();
            if (lane < 36) s_term[lane] = term;
            __syncthreads();
            double s = 0.0;
#pragma unroll
            for (int q = 0; q < 6; ++q) s += s_term[6 * i + q] * ad[q];
            term = s / (double)(n + 1);
            J += term;
            if (!__any(fabs(term) >= 1e-18)) break;   // uniform
        }
        if (lane < 36) jr[36 * f + lane] = J;
    }
}

// Solve (H + lambda diag(H)) delta = -b by Cholesky; returns false if not SPD.
__device__ bool lm_solve(const double* row, double lambda, double delta[6]) {
    double A[36], L[36] = {0};
    for (int i = 0; i < 6; ++i)
        for (int j = 0; j < 6; ++j) A[6 * i + j] = row[1 + 6 * i + j] + (i == j ? lambda * row[1 + 7 * i] : 0.0);
    for (int j = 0; j < 6; ++j) {
        double s = A[7 * j];
        for (int k = 0; k < j; ++k) s -= L[6 * j + k] * L[6 * j + k];
        if (!(s > 0.0)) return false;
        L[7 * j] = sqrt(s);
        for (int i = j + 1; i < 6; ++i) {
            double u = A[6 * i + j];
            for (int k = 0; k < j; ++k) u -= L[6 * i + k] * L[6 * j + k];
            L[6 * i + j] = u / L[7 * j];
        }
    }
    double z[6];
    for (int i = 0; i < 6; ++i) {
        double s = -row[37 + i];
        for (int k = 0; k < i; ++k) s -= L[6 * i + k] * z[k];
        z[i] = s / L[7 * i];
    }
    for (int i = 5; i >= 0; --i) {
        double s = z[i];
        for (int k = i + 1; k < 6; ++k) s -= L[6 * k + i] * delta[k];
        delta[i] = s / L[7 * i];
    }
    return true;
}

// Proposal of one damped step per factor: delta from (H + lambda diag H) delta = -b
// (FP64 Cholesky) at the linearization rows, candidate T Exp(delta).  A matrix
// that is not SPD leaves the candidate at T and marks it invalid.  A kernel of its
// own: inside the reduction the compiler fuses the exponential's sums in another
// order, and a step's last bit decides later accepts near convergence.
__global__ void k_lm_propose(int64_t F, const double* __restrict__ out, const double* __restrict__ lambda,
                             const double* __restrict__ poses, double* __restrict__ cand, int32_t* __restrict__ valid,
                             float* __restrict__ posef) {
    const int64_t f = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (f >= F) return;
    const double* row = out + (int64_t)kOutRow * f;
    double delta[6], T[12], E[12], C[12];
    for (int k = 0; k < 12; ++k) T[k] = poses[12 * f + k];
    const bool ok = lm_solve(row, lambda[f], delta);
    if (ok) {
        se3_exp(delta, E);
        pose_mul(T, E, C);
    } else {
        for (int k = 0; k < 12; ++k) C[k] = T[k];
    }
    for (int k = 0; k < 12; ++k) cand[12 * f + k] = C[k];
    valid[f] = ok ? 1 : 0;
    stage_pose(posef, f, cand + 12 * f);
}

__global__ void k_fill(double* __restrict__ p, int64_t n, double v) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

vg_status launch_se3_retract(vg_context* ctx, int64_t F, const double* d_T0, const double* d_xi, double* d_T,
                             double* d_jr) {
    if (F == 0) return VG_OK;
    if (d_jr == nullptr)
        k_se3_poses<<<(unsigned)std::min<int64_t>((F + 63) / 64, 1 << 22), 64, 0, ctx->stream>>>(F, d_T0, d_xi, d_T);
    else
        k_se3_retract<<<(unsigned)std::min<int64_t>(F, 1 << 22), 64, 0, ctx->stream>>>(F, d_T0, d_xi, d_T, d_jr);
    VG_HIP(hipGetLastError());
    return VG_OK;
}

vg_status launch_lm_propose(vg_batch* b, const double* d_out, const LmArgs& lm) {
    k_lm_propose<<<(int)((b->F + 63) / 64), 64, 0, b->ctx->stream>>>(b->F, d_out, lm.lambda, lm.poses, lm.cand, lm.valid,
                                                                     lm.posef);
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

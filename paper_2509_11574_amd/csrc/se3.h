// SE(3) helpers in binary64 for the device (camera pose updates).
// xi = (rho, phi): translation part first, then the rotation vector.
#pragma once
#include <hip/hip_runtime.h>

namespace gps {

// Exp of xi = (rho, phi) in SE(3) (Rodrigues' formula for the rotation, the left
// Jacobian of SO(3) for the translation).
__device__ inline void se3_exp_d(const double xi[6], double R[9], double t[3])
{
    const double wx = xi[3], wy = xi[4], wz = xi[5];
    const double th2 = wx * wx + wy * wy + wz * wz, th = sqrt(th2);
    const double K[9] = {0.0, -wz, wy, wz, 0.0, -wx, -wy, wx, 0.0};
    double K2[9];
    for (int r = 0; r < 3; ++r)
        for (int c = 0; c < 3; ++c) K2[3 * r + c] = K[3 * r] * K[c] + K[3 * r + 1] * K[3 + c] + K[3 * r + 2] * K[6 + c];
    double A, B, C;
    if (th < 1e-6) {  // series of sin(th)/th, (1 - cos th)/th^2, (th - sin th)/th^3
        A = 1.0 - th2 / 6.0;
        B = 0.5 - th2 / 24.0;
        C = 1.0 / 6.0 - th2 / 120.0;
    } else {
        A = sin(th) / th;
        B = (1.0 - cos(th)) / th2;
        C = (th - sin(th)) / (th2 * th);
    }
    double V[9];
    for (int k = 0; k < 9; ++k) {
        const double I = (k % 4 == 0) ? 1.0 : 0.0;
        R[k] = I + A * K[k] + B * K2[k];
        V[k] = I + B * K[k] + C * K2[k];
    }
    for (int r = 0; r < 3; ++r) t[r] = V[3 * r] * xi[0] + V[3 * r + 1] * xi[1] + V[3 * r + 2] * xi[2];
}

// y = J^T g for the left Jacobian of SE(3) at xi: J = sum_n ad(xi)^n / (n + 1)!,
// ad(xi) = [[phi^, rho^], [0, phi^]] (hat = cross-product matrix), so that
// Exp(xi + e) = Exp(J e) Exp(xi) to first order in e.  One lane runs this, so the series
// is taken on the vector (ad^T (a, b) = -(phi x a, rho x a + phi x b): three cross products
// a term) and not on the 6x6 matrix, and it ends once the rest is below binary64 rounding
// of the sum; 39 terms, which reach |phi| = 2 pi, at most.  The matrix series took 66 us
// a call (a 160x120 view as a 1280x720 one) and this one takes 3 to 4.
__device__ inline void se3_left_jacobian_t_mul_d(const double xi[6], const double g[6], double y[6])
{
    const double rx = xi[0], ry = xi[1], rz = xi[2], px = xi[3], py = xi[4], pz = xi[5];
    const double reach = fabs(rx) + fabs(ry) + fabs(rz) + fabs(px) + fabs(py) + fabs(pz);
    double a0 = g[0], a1 = g[1], a2 = g[2], b0 = g[3], b1 = g[4], b2 = g[5];
    for (int k = 0; k < 6; ++k) y[k] = g[k];
    for (int n = 1; n < 40; ++n) {
        const double s = -1.0 / (double)(n + 1);
        const double c0 = s * (py * a2 - pz * a1), c1 = s * (pz * a0 - px * a2), c2 = s * (px * a1 - py * a0);
        const double d0 = s * ((ry * a2 - rz * a1) + (py * b2 - pz * b1));
        const double d1 = s * ((rz * a0 - rx * a2) + (pz * b0 - px * b2));
        const double d2 = s * ((rx * a1 - ry * a0) + (px * b1 - py * b0));
        a0 = c0, a1 = c1, a2 = c2, b0 = d0, b1 = d1, b2 = d2;
        y[0] += a0, y[1] += a1, y[2] += a2, y[3] += b0, y[4] += b1, y[5] += b2;
        const double term = fmax(fmax(fmax(fabs(a0), fabs(a1)), fabs(a2)), fmax(fmax(fabs(b0), fabs(b1)), fabs(b2)));
        const double sum = fmax(fmax(fmax(fabs(y[0]), fabs(y[1])), fabs(y[2])), fmax(fmax(fabs(y[3]), fabs(y[4])), fabs(y[5])));
        // from here on each term is less than half of the one before it
        if (2.0 * reach < (double)(n + 2) && term <= 0x1p-56 * sum) break;
    }
}

}  // namespace gps
